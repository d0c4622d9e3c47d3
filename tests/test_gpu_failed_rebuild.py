"""A batched rebuild that fails on one walker's box leaves the others usable: a rebuild captured before it goes on
working on the buffers it was captured with, between eager rebuilds, on positions it has not seen (cell starts, order
and rows as an eager context builds them)."""
import numpy as np
import pytest

import workloads as W
from tests.helpers import params_for
from tests.test_gpu_parity import to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

WL = dict(cv="q6", precision="fp32", r_c=3.6, skin=0.4, taper=0.2, cn_r0=2.5, bond_d0=0.7, bond_w=0.02, count_n0=5.5,
          count_w=0.25, sigma=[20.0], w0=W.W0_EV, gamma=10.0, kBT=W.KBT_EV, hills=dict(k=64))


def lists(pipe):
    nc, perm, start = pipe.cell_list()
    nbr, cnt = pipe.neighbor_lists()
    pipe.stream.synchronize()
    nbr, cnt = nbr.cpu().numpy(), cnt.cpu().numpy()
    return nc, perm.cpu().numpy(), start.cpu().numpy(), cnt, [row[:c] for row, c in zip(nbr, cnt)]


def same(a, b):
    assert a[0] == b[0]
    for x, y in zip(a[1:4], b[1:4]):
        assert np.array_equal(x, y)
    for x, y in zip(a[4], b[4]):
        assert np.array_equal(x, y)


def test_captured_rebuild_after_a_failed_batched_one():
    from paper_2510_06873_amd import Batch, GmError, Pipeline

    d = W.wurtzite_slab(nx=8, ny=4, nz=8, seed=5)
    box, n = np.asarray(d["box"], np.float64), len(d["pos"])
    rng = np.random.default_rng(3)
    frames = [to_dev(W.as_float4(W._wrap_f32(np.asarray(d["pos"], np.float64) + rng.normal(0.0, 0.5, (n, 3)), box)))
              for _ in range(4)]
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(st):
        def pipe_of():
            return Pipeline(n, params_for(WL, max_neighbors=128), stream=st)

        at, at2 = frames[0].clone(), frames[0].clone()
        F, F2 = torch.zeros((n, 4), device="cuda"), torch.zeros((n, 4), device="cuda")
        pipe, other, ref = pipe_of(), pipe_of(), pipe_of()
        for p in (pipe, other):
            p.build_neighbors_checked(at, box)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=st):
            pipe.build_neighbors(at, box)
        batch = Batch([pipe, other], [at, at2], [F, F2], stream=st)

        def check(k, replay):
            at.copy_(frames[k])
            if replay:
                graph.replay()
            else:
                pipe.build_neighbors(at, box)
            ref.build_neighbors_checked(frames[k], box)
            same(lists(pipe), lists(ref))

        check(1, True)
        with pytest.raises(GmError, match="BOX"):
            batch.build_some([0, 1], [box, [5.0, 5.0, 5.0]], stream=st)
        check(2, False)
        check(3, True)
        check(1, False)
        check(2, True)
        batch.close()
        for p in (pipe, other, ref):
            assert p.status(True) == 0
            p.close()
