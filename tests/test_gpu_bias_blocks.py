"""The bias sum in one workgroup (up to 8,192 hills of capacity) and in several, at the edges of a thread's rounds
and of the capacity, 1-D, 2-D and periodic, against the FP64 oracle (1e-12 relative, as the other bias tests)."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [0, 1, 1024, 1025, 4097, 8192])
@pytest.mark.parametrize("capacity", [8192, 8193, 400000])
@pytest.mark.parametrize("dims,period", [(1, 0.0), (2, 0.0), (2, 6.0)])
def test_bias_and_deposit(orc, K, capacity, dims, period):
    from paper_2510_06873_amd import CV_EXTERNAL, Params, Pipeline

    sigma = [0.35, 0.2][:dims]
    cen = W.hill_centres(K, [-3.0] * dims, [3.0] * dims, seed=K + 5)
    hts = np.random.default_rng(6).uniform(0.2, 1.2, K)
    pipe = Pipeline(0, Params(cv_kind=CV_EXTERNAL, external_dims=dims, sigma=sigma, period=[period] * dims, w0=1.2,
                              gamma=10.0, kBT=W.KBT_KJMOL, hill_capacity=capacity))
    pipe.hills_set(cen, hts)
    x = np.array([0.3, -2.9][:dims])
    s = torch.from_numpy(x).cuda()
    per = [period] * dims if period else None
    V, dV = pipe.bias_eval(s)
    V, dV = V.item(), dV.cpu().numpy()
    Vr, dVr = orc.bias(cen, hts, sigma, x, period=per) if K else (0.0, np.zeros(dims))
    assert abs(V - Vr) <= 1e-12 * abs(Vr)
    assert np.max(np.abs(dV - dVr)) <= 1e-12 * (np.abs(dVr).max() + abs(Vr) / min(sigma))
    pipe.deposit_hill(s)
    if K == capacity:
        assert pipe.status(True) == -6
        assert pipe.hills_get()[1].shape[0] == K
    else:
        pipe.check()
        c, h = pipe.hills_get()
        assert h.shape[0] == K + 1 and np.array_equal(c[-1], x)
        want = 1.2 * np.exp(-Vr / (W.KBT_KJMOL * 9.0))
        assert abs(h[-1] - want) <= 1e-12 * want
