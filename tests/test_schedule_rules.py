"""Host rules of a solve's schedule (csrc/schedule.h), compiled for the CPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2103_10203_amd", "csrc")


def _program(tmp_path, body):
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text('#include <cstdio>\n#include <cstdlib>\n#include "schedule.h"\n'
                   "int main(int n, char** v) {\n" + body + "\n}\n")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I" + CSRC, str(src), "-o", str(exe)], check=True)

    def run(*args):
        return subprocess.run([str(exe), *map(str, args)], check=True, capture_output=True, text=True).stdout.split()
    return run


@pytest.fixture(scope="module")
def by_component(tmp_path_factory):
    run = _program(tmp_path_factory.mktemp("rule"), """
  long long a[8];
  for (int i = 0; i < 8; ++i) a[i] = atoll(v[i + 1]);
  std::printf("%d\\n", mor_sched::rows_by_component({a[0] != 0, a[1] != 0, a[2] != 0, a[3] != 0, a[4], (int)a[5],
                                                     a[6], a[7]}));
  return 0;""")
    return lambda **kw: run(*[int(x) for x in {
        "row_fast": 1, "default": 1, "dft": 0, "persistent": 0, "bytes": 1 << 20, "rb": 4, "rows": 256, "rves": 1,
        **kw}.values()]) == ["1"]


def test_small_calls_run_rows_by_component(by_component):
    assert by_component()
    assert by_component(rves=8) and not by_component(rves=9)          # 512 workgroups of four rows
    assert by_component(rows=257, rves=7) and not by_component(rows=257, rves=8)  # 65 workgroups each
    assert by_component(rows=2048) and not by_component(rows=2049)


@pytest.mark.parametrize("other", [{"persistent": 1}, {"dft": 1}, {"default": 0}, {"row_fast": 0}, {"rb": 0},
                                   {"bytes": 1 << 31}])
def test_other_forms_keep_their_row_kernel(by_component, other):
    for rves in (1, 8, 1000):
        assert not by_component(rves=rves, **other)
