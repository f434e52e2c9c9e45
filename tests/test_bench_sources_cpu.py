"""Host-only: what the hash that ties stored counters to the product's code covers."""
import glob
import importlib.util
import os

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_kernel_hash_covers_the_product_and_its_plan():
    """Every source of the windowed product, the plan among them (another cut of the
    orbits launches other kernels)."""
    spec = importlib.util.spec_from_file_location("bench_mod", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    files = glob.glob(os.path.join(ROOT, "paper_2001_01978_amd", "csrc", "window*"))
    assert len(files) >= 4
    assert {os.path.relpath(f, ROOT) for f in files} <= set(bench.KERNEL_SOURCES)
