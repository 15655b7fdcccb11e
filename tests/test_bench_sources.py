"""The counter summaries that bench.py quotes are tied to the sources of the
solve kernels: every source file but those of the plans, the network and the error
measures counts."""
import importlib.util
import os

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_solve_source_is_hashed():
    spec = importlib.util.spec_from_file_location("bench_sources", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    files = {f for f in os.listdir(os.path.join(ROOT, "paper_2103_10203_amd", "csrc")) if f.endswith((".h", ".hip"))}
    assert set(bench.SOLVE_SOURCES) == files - {"plan.hip", "mlp.hip", "error.hip"}
