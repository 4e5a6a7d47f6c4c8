"""bench.py's roofline entry names what bounds the kernel that it times (CPU only)."""
import importlib.util
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def bench():
    spec = importlib.util.spec_from_file_location("bench_module", os.path.join(ROOT, "bench.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def test_streaming_kernels_against_hbm(bench):
    r = bench.roofline_of("check", 0.1, 4e8, "")
    assert r["bound"] == "hbm" and r["unit"] == "GB/s" and r["achieved"] == pytest.approx(4000.0)
    assert r["frac"] == pytest.approx(4000.0 / bench.HBM_PEAK_GBS)


def test_frame_resident_kernel_against_issue(bench):
    counted = bench.FUSED_VALU["source_sha256"]
    r = bench.roofline_of("fused", 1.0, 4e7, counted)
    assert r["bound"] == "valu" and r["hbm"]["achieved"] == pytest.approx(40.0)
    assert r["frac"] == pytest.approx(bench.FUSED_VALU["insts_per_launch"] * 1e3 / bench.VALU_ISSUE_PEAK)
    for other in (bench.roofline_of("fused", 1.0, 4e7, "another source"),
                  bench.roofline_of("fused", 1.0, 4e7, counted, layered=True),
                  bench.roofline_of("fused", None, 4e7, counted)):
        assert other["bound"] == "valu" and other["achieved"] is None and other["frac"] is None

