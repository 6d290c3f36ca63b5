"""The benchmark rates the M2L against the instructions it issues (CPU only)."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402

RES = {"phases_fwd_ms": {"m2l": 2.0, "p2p": 0.1}, "phases_adj_ms": {"m2l": 2.0, "p2p": 0.1},
       "counts": {"m2l_rank": 116, "v_pairs": 1000, "p2p_pairs": 10}}


# p = 6 has 152 surface points, p = 7 218, p = 8 296
@pytest.mark.parametrize("precision,n,kernel,peak", [
    ("split_bf16", 152, "laplace", 2500.0), ("split_bf16", 296, "gravity", 2500.0),
    ("fp32", 56, "laplace", 2500.0), ("fp32", 152, "laplace", 2500.0),
    ("fp32", 218, "laplace", 157.3), ("fp32", 152, "gravity", 157.3), ("fp32", 296, "gravity", 157.3)])
def test_m2l_peak(precision, n, kernel, peak):
    r = bench.roofline(RES, n, precision, "none", 1, kernel)
    assert r["kernel"] == "k_m2l" and r["peak"] == peak
    assert r["frac"] == pytest.approx(2 * 116 * 116 * 1000 / 2e-3 / 1e12 / peak)
