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


MIB = 1 << 20
DEFAULT = (192 * MIB, 128)


@pytest.fixture(scope="module")
def cut(tmp_path_factory):
    run = _program(tmp_path_factory.mktemp("cut"), """
  for (int i = 1; i + 5 < n; i += 6) {
    const mor_sched::Cut c = mor_sched::cut_runs(atoll(v[i]), atoll(v[i + 1]), atoll(v[i + 2]), atoll(v[i + 3]),
                                                 atoll(v[i + 4]), atoll(v[i + 5]) != 0);
    std::printf("%lld %d\\n", (long long)c.runs, (int)c.pairs);
  }
  return 0;""")

    def one(*args):
        runs, pairs = run(*(int(a) for a in args))
        return int(runs), pairs == "1"
    one.many = lambda rows: run(*(int(a) for r in rows for a in r))
    return one


def test_runs_of_the_default_limits(cut):
    # bytes, RVEs, row workgroups, limit, minimum of RVEs, pairs possible
    assert cut(350 * MIB, 1024, 16384, *DEFAULT, 1) == (4, True)     # 1024 RVEs of 256^2
    assert cut(350 * MIB, 1024, 16384, *DEFAULT, 0) == (2, False)
    assert cut(43 * MIB, 128, 2048, *DEFAULT, 1) == (2, True)
    assert cut(21 * MIB, 64, 1024, *DEFAULT, 1) == (1, False)        # too few workgroups
    assert cut(10 * MIB, 512, 2048, *DEFAULT, 1) == (1, False)       # too few bytes
    assert cut(252 * MIB, 8, 32768, *DEFAULT, 1) == (4, True)        # eight of 128^3
    assert cut(300 * MIB, 2, 32768, *DEFAULT, 1) == (1, False)       # halves beyond half the limit


def test_a_set_minimum_bounds_every_run(cut):
    assert cut(252 * MIB, 8, 32768, 192 * MIB, 4, 1) == (2, False)   # runs of two are not allowed
    assert cut(252 * MIB, 8, 32768, 192 * MIB, 129, 1) == (1, False)
    assert cut(350 * MIB, 1024, 16384, 192 * MIB, 256, 1) == (4, True)
    assert cut(350 * MIB, 1024, 16384, 192 * MIB, 257, 1) == (2, False)
    assert cut(350 * MIB, 1024, 16384, 192 * MIB, 2 ** 63 - 1, 1) == (1, False)


def test_a_set_limit_bounds_what_is_in_flight(cut):
    # 100 MB and 8192 workgroups under 4 MiB: no eight runs of 12.5 MB in pairs
    assert cut(100e6, 512, 8192, 4 * MIB, 1, 1) == (24, False)
    assert cut(100e6, 512, 8192, 0, 1, 1) == (1, False)
    assert cut(100e6, 512, 8192, 2 ** 63 - 1, 1, 1) == (2, True)
    rows = []
    for limit in (1, 600 << 10, 4 * MIB, 40 * MIB, 192 * MIB, 1 << 40):
        for rves in (1, 2, 7, 128, 1536):
            for total in (3 * MIB, 90 * MIB, 352 * MIB, 40 << 30):
                for least in (1, 5, 128, 300):
                    for wgs in (64, 4096, 1 << 20):
                        rows.append((total, rves, wgs, limit, least, 1))
    out = cut.many(rows)
    for (total, rves, wgs, limit, least, _), runs, pairs in zip(rows, out[::2], out[1::2]):
        runs = int(runs)
        assert 1 <= runs <= rves
        if pairs == "1":
            assert 2 * total <= runs * limit and runs % 2 == 0
            assert least == 128 or rves // runs >= least
        else:
            assert runs == 1 or rves // runs >= least


def test_grids_side_by_side_within_the_cache_and_a_lowered_limit(tmp_path):
    run = _program(tmp_path, """
  std::printf("%d %d\\n", mor_sched::grids_side_by_side(atoll(v[1]), atoll(v[2]), atoll(v[3])),
              mor_sched::shares_device(atoll(v[2]), atoll(v[3])));
  return 0;""")
    assert run(3, 200 * MIB, 192 * MIB) == ["1", "0"]
    assert run(3, 257 * MIB, 1 << 40) == ["0", "1"]
    assert run(1, MIB, 192 * MIB) == ["0", "1"]
    assert run(3, 200 * MIB, 0) == ["1", "0"]
    assert run(3, 5 * MIB, 4 * MIB) == ["0", "0"]
    assert run(3, 4 * MIB, 4 * MIB) == ["1", "0"]
