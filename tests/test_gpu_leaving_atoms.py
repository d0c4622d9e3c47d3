"""Atoms that leave the box between the rebuild and the step (unwrapped, by less than half the skin), in FP64: the
pass that reads the caller's positions finds them itself, in the launch that tells the later passes.  More bricks
than run at once, bricks on every face with room for shifted coordinates, atoms outside in some of them only; CV and
forces against the FP64 oracle at the parity tests' bar, 1e-10, on several steps (the flag unset and set before)."""
import dataclasses

import numpy as np
import pytest

import workloads as W
from tests.helpers import oracle_cvs, params_for, rel_force_err
from tests.test_gpu_parity import to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

WZ = dict(taper=0.2, bond_d0=0.7, bond_w=0.02, count_n0=5.5, count_w=0.25, w0=W.W0_EV, gamma=10.0, kBT=W.KBT_EV,
          hills=dict(k=4), r_c=3.6, skin=0.4, cn_r0=2.5, precision="fp64")
W_PLANE = 3.19 * 3 ** 0.5 / 6  # height of the lattice's first plane above the face of axis 1


@pytest.mark.parametrize("cv", ["q6", "coord_q6"])
@pytest.mark.parametrize("cells,brick", [((12, 7, 8), (1, 1, 1)), ((13, 8, 9), (1, 1, 1)), ((21, 9, 11), (0, 0, 0))])
def test_leaving_the_box_after_the_rebuild(orc, cells, brick, cv):
    from paper_2510_06873_amd import Pipeline

    d = W.wurtzite_slab(*cells, seed=32)
    box = d["box"]
    # a plane of atoms on each face
    pos = W._wrap_f32(np.asarray(d["pos"], np.float64) - np.array([0.0, W_PLANE, 0.0]), box)
    n, rng = len(pos), np.random.default_rng(11)
    wl = dict(WZ, cv=cv, sigma=[20.0] * (1 if cv == "q6" else 2))
    pipe = Pipeline(n, dataclasses.replace(params_for(wl, max_neighbors=128), brick=brick))
    pipe.build_neighbors_checked(to_dev(W.as_float4(pos, d["species"])), box)
    # by at most 0.12 per axis from within 0.1 of a face, on a part of each face: the atoms of the other bricks
    # there stay inside
    given = pos.astype(np.float64)
    for axis in range(3):
        part = given[:, (axis + 1) % 3] < 0.4 * box[(axis + 1) % 3]
        low = part & (pos[:, axis] < 0.1)
        high = part & (pos[:, axis] > box[axis] - 0.1)
        assert low.sum() + high.sum() > 0
        given[low, axis] = -rng.uniform(0.0, 0.02, low.sum())
        given[high, axis] = box[axis] + rng.uniform(0.0, 0.02, high.sum())
    left = given.astype(np.float32)
    assert ((left < 0) | (left >= box)).any(1).sum() >= 4
    F_in = W.external_forces(n, seed=9)
    dv = torch.tensor([0.37] if cv == "q6" else [0.0, 0.37], dtype=torch.float64, device="cuda")
    for at in (left, pos, left):
        p4, F = to_dev(W.as_float4(at, d["species"])), to_dev(F_in, pipe.fdtype)
        s = pipe.cv_forward(p4).clone()
        pipe.cv_backward(p4)
        pipe.apply_bias_forces(p4, F, dv)
        assert pipe.status(True) == 0
        s_ref, g_ref, _ = oracle_cvs(orc, at, box, wl)
        assert np.all(np.abs(s.cpu().numpy()[:len(s_ref)] - s_ref) <= 1e-10 * np.abs(s_ref))
        got = F.cpu().numpy()[:, :3].astype(np.float64) - F_in[:, :3].astype(np.float64)
        assert rel_force_err(got, -0.37 * g_ref[-1]) <= 1e-10
    pipe.close()
