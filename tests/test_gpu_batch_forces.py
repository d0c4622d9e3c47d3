"""Batched steps with hills, so that the bias forces are not zero, equal to the calls of a lone context bit for bit: CV,
V, forces and the deposited hill, for every CV and precision, on systems on both sides of the lines of pass 1 (the
caller's positions up to 131,072 atoms; the sorted copy in batches of FP64 coordination walkers with dense cells) and
of the CV's sum (256 workgroups), with atoms inside and outside the box."""
import numpy as np
import pytest

import workloads as W
from tests.helpers import params_for
from tests.test_gpu_parity import to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BASE = dict(taper=0.2, bond_d0=0.7, bond_w=0.02, count_n0=5.5, count_w=0.25, w0=W.W0_EV, gamma=10.0, kBT=W.KBT_EV,
            hills=dict(k=64))
WZ, FCC = dict(BASE, r_c=3.6, skin=0.4, cn_r0=2.5), dict(BASE, r_c=6.0, skin=0.5, cn_r0=3.0)


def structure(wl, size, outside):
    rng = np.random.default_rng(7)
    if wl is FCC:
        d = W.fcc_jittered(size, seed=31)
        pos, box = np.asarray(d["pos"], np.float64), d["box"]
    else:
        pos, _, box = W.wurtzite_ideal(*size)
    pos = W._wrap_f32(pos + rng.normal(0.0, 0.16, pos.shape), box)
    if outside:
        move = rng.integers(-1, 2, pos.shape) * (rng.random(pos.shape) < 0.01)
        pos = (pos.astype(np.float64) + move * box).astype(np.float32)
    return pos, box


@pytest.mark.parametrize("wl,cv,sizes", [(WZ, "q6", [(5, 4, 4), (12, 7, 8)]), (WZ, "q6", [(24, 12, 10)]),
                                         (WZ, "coord_q6", [(8, 4, 8), (14, 9, 9)]), (WZ, "coord", [(5, 4, 4), (21, 9, 11)]),
                                         (FCC, "coord", [6, 9, 14]), (WZ, "q6", [(33, 32, 16), (5, 4, 4)])])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("outside", [False, True])
def test_batched_step_equals_a_lone_one(wl, cv, sizes, precision, outside):
    from paper_2510_06873_amd import Batch, Pipeline

    prm = dict(wl, cv=cv, precision=precision, sigma=[0.3, 30.0] if cv == "coord_q6" else [0.3 if cv == "coord" else 30.0])
    dims = len(prm["sigma"])
    alone, batched, pos4, forces, want = [], [], [], [], []
    for size in sizes:
        pos, box = structure(wl, size, outside)
        n = len(pos)
        p4 = to_dev(W.as_float4(pos))
        pipe, twin = (Pipeline(n, params_for(prm, max_neighbors=160)) for _ in range(2))
        for p in (pipe, twin):
            p.build_neighbors_checked(p4, box)
        s0 = pipe.cv_forward(p4).cpu().numpy()[:dims]
        sig = np.array(prm["sigma"])
        cen, hts = W.hill_centres(40, s0 - 2 * sig, s0 + 2 * sig, seed=8), np.linspace(0.5, 1.5, 40) * prm["w0"]
        for p in (pipe, twin):
            p.hills_set(cen, hts)
        F = to_dev(W.external_forces(n, seed=3), pipe.fdtype)
        F0 = F.clone()
        got = []
        for _ in range(2):
            s = pipe.cv_forward(p4)
            V, dV = pipe.bias_eval()
            pipe.cv_backward(p4)
            pipe.apply_bias_forces(p4, F)
            pipe.deposit_hill()
            got.append((s.clone(), V.clone(), F.clone()))
        assert not torch.equal(F, F0) and pipe.status(True) == 0
        alone.append(pipe), batched.append(twin), pos4.append(p4), forces.append(F0), want.append(got)
    batch = Batch(batched, pos4, forces)
    for t in range(2):
        batch.step()
        batch.deposit()
        sb, Vb = batch.values()
        for k, got in enumerate(want):
            assert torch.equal(sb[k, :dims], got[t][0][:dims]) and torch.equal(Vb[k:k + 1], got[t][1].reshape(1))
            assert torch.equal(forces[k], got[t][2])
    batch.close()
    for a, b in zip(alone, batched):
        assert all(np.array_equal(x, y) for x, y in zip(a.hills_get(), b.hills_get()))
        a.close()
        b.close()
