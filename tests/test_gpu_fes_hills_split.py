"""The free energy from hills, split over workgroups: the 2-D matrix product and the 1-D shares, at the
edges of their tiles and shares, against the FP64 oracle; and the direct sum that a captured stream takes.

Tolerance: a point sums K terms of at most one magnitude in FP64, so the two orders of summation and a
factor exp(-a) exp(-b) for exp(-a - b) (arguments up to ~700: relative error ~700 eps in a term that is then
below e^-700) differ by far less than 1e-12 of the largest value, the bar of the other FES tests."""
import math

import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
TWO_PI = 2 * math.pi


def context(dims, K, period):
    from paper_2510_06873_amd import CV_EXTERNAL, Params, Pipeline

    cen = W.hill_centres(K, [-math.pi] * dims, [math.pi] * dims, seed=70 + K + dims)
    hts = np.random.default_rng(71).uniform(0.2, 1.2, K)
    pipe = Pipeline(0, Params(cv_kind=CV_EXTERNAL, external_dims=dims, sigma=[0.35, 0.2][:dims], period=[period] * dims,
                              w0=1.2, gamma=10.0, kBT=W.KBT_KJMOL, hill_capacity=K + 3))
    pipe.hills_set(cen, hts)
    return pipe, cen, hts


@pytest.mark.parametrize("nb,K", [([1, 1], 1), ([128, 128], 33), ([129, 127], 300), ([1, 300], 40), ([257, 3], 1025),
                                  ([16], 1), ([256], 15), ([257], 4000)])
@pytest.mark.parametrize("period", [0.0, TWO_PI])
def test_split_sum_against_the_oracle(orc, nb, K, period):
    dims = len(nb)
    pipe, cen, hts = context(dims, K, period)
    lo, hi = [-math.pi] * dims, [math.pi] * dims
    F = pipe.fes_hills(lo, hi, nb).cpu().numpy()
    Fr = orc.fes_hills(cen, hts, [0.35, 0.2][:dims], lo, hi, nb, gamma=10.0, period=[period] * dims if period else None)
    assert np.max(np.abs(F - Fr)) <= 1e-12 * np.abs(Fr).max()
    assert np.array_equal(F, pipe.fes_hills(lo, hi, nb).cpu().numpy())  # a fixed order of summation


def test_captured_call_allocates_nothing_and_agrees():
    pipe, _, _ = context(2, 500, TWO_PI)
    lo, hi, nb = [-math.pi] * 2, [math.pi] * 2, [130, 40]
    F = pipe.fes_hills(lo, hi, nb)
    G = torch.zeros_like(F)
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    pipe.set_stream(stream)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        pipe.fes_hills(lo, hi, nb, G)
    for _ in range(3):
        G.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.max((F - G).abs()).item() <= 1e-12 * F.abs().max().item()
    pipe.set_stream(torch.cuda.current_stream())
