"""Reweighting at the edges of its workgroups' shares and of the LDS histogram (16,384 bins), against the
FP64 oracle.  Tolerance: the bins' sums differ only in the order of FP64 additions (at most 2,049 terms, so
below 2,049 eps relative), and F = -kBT log of their ratio: 1e-10 kBT, the bar of the other reweighting tests."""
import math

import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 1023, 1024, 1025, 2049])
@pytest.mark.parametrize("nb", [[1], [16384], [16385], [3, 5]])
def test_edges_against_the_oracle(orc, T, nb):
    import paper_2510_06873_amd as P

    dims, kBT = len(nb), W.KBT_KJMOL
    s, V = W.biased_trace(T=T, dims=dims, seed=80 + T)
    lo, hi = [-math.pi] * dims, [math.pi] * dims
    dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (s, V)]
    F = P.fes_reweight(*dev, lo, hi, nb, kBT).cpu().numpy()
    Fr = orc.fes_reweight(s, V, lo, hi, nb, kBT)
    fin = np.isfinite(Fr)
    assert np.array_equal(np.isfinite(F), fin) and fin.any()
    assert np.max(np.abs(F[fin] - Fr[fin])) <= 1e-10 * kBT
