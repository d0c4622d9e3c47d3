"""FP32 q6 forces of unwrapped coordinates around 131,072 atoms (below, pass 1 reads the caller's positions; above, the
sorted copy), against the FP64 oracle on the same coordinates.

Tolerance: 1e-4 of the largest force, the bar of FP32 arithmetic on wrapped coordinates, and what rounding the images
adds.  A pair of atoms outside on opposite sides lies two box lengths apart; forming its image rounds each coordinate at
up to 2 L (half an ulp, 1.5e-5 A at L = 177 A).  The oracle says what that does: its own forces with the outside
atoms' coordinates, wrapped, each moved by one ulp at L (1.5e-5 A) up or down at random, three times over (the random
signs of the sum of pairs against their worst case)."""
import numpy as np
import pytest

import workloads as W
from tests.helpers import oracle_cvs, params_for, rel_force_err
from tests.test_gpu_parity import to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

WL = dict(taper=0.2, bond_d0=0.7, bond_w=0.02, count_n0=5.5, count_w=0.25, w0=W.W0_EV, gamma=10.0, kBT=W.KBT_EV,
          hills=dict(k=4), precision="fp32", r_c=3.6, skin=0.4, cn_r0=2.5, cv="q6", sigma=[20.0])


@pytest.mark.parametrize("cells", [(32, 32, 16), (33, 32, 16)])
def test_q6_forces(orc, cells):
    from paper_2510_06873_amd import Pipeline

    x, species, box = W.wurtzite_ideal(*cells)
    rng = np.random.default_rng(7)
    pos = W._wrap_f32(x + rng.normal(0.0, 0.16, x.shape), box)
    move = rng.integers(-1, 2, pos.shape) * (rng.random(pos.shape) < 0.01)
    out = (pos.astype(np.float64) + move * box).astype(np.float32)
    n, L = len(pos), np.asarray(box, np.float64)
    p4 = to_dev(W.as_float4(out, species))
    pipe = Pipeline(n, params_for(WL))
    pipe.build_neighbors_checked(p4, box)
    s = pipe.cv_forward(p4).cpu().numpy()
    pipe.cv_backward(p4)
    F = torch.zeros((n, 4), device="cuda")
    pipe.apply_bias_forces(p4, F, torch.ones(1, dtype=torch.float64, device="cuda"))
    assert pipe.status(True) == 0
    s_ref, g_ref, _ = oracle_cvs(orc, out, box, WL)
    assert abs(s[0] - s_ref[0]) <= 1e-5 * abs(s_ref[0])
    back = W._wrap_f32(out.astype(np.float64), L)
    step = np.float32(np.spacing(np.float32(L.max())))
    moved = back + step * rng.choice(np.array([-1.0, 1.0], np.float32), back.shape) * (move != 0).any(1)[:, None]
    moved = np.clip(moved, 0, np.nextafter(np.float32(L), np.float32(0))).astype(np.float32)
    (_, g_a, _), (_, g_b, _) = oracle_cvs(orc, back, box, WL), oracle_cvs(orc, moved, box, WL)
    tol = 1e-4 + 3.0 * rel_force_err(g_b[0], g_a[0])
    print("tolerance %.2e" % tol)
    assert tol < 1e-2
    assert rel_force_err(F.cpu().numpy()[:, :3], -g_ref[0]) <= tol
    pipe.close()
