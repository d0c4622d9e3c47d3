"""Passes 2-4 over halos that fit the LDS staging whole, in part, and barely at all (the rest read from global
memory), each against the FP64 oracle at the bars of the parity tests: CV 1e-5 (FP32) / 1e-10 (FP64), forces
1e-4 / 1e-10; and an adjoint asked for a second time on the same forward state, which must give the same bits."""
import dataclasses

import numpy as np
import pytest

import workloads as W
from tests.helpers import oracle_cvs, params_for, rel_force_err
from tests.test_gpu_parity import dev, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

WZ = dict(taper=0.2, bond_d0=0.7, bond_w=0.02, count_n0=5.5, count_w=0.25, w0=W.W0_EV, gamma=10.0, kBT=W.KBT_EV,
          hills=dict(k=4), r_c=3.6, skin=0.4, cn_r0=2.5)


@pytest.mark.parametrize("lds_kb", [0, 24, 8])  # FP32: 1,174, 331 and 90 slots, of about 410 in a halo
@pytest.mark.parametrize("cv", ["q6", "coord_q6"])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_part_staged_rows_against_the_oracle(orc, precision, cv, lds_kb):
    from paper_2510_06873_amd import Pipeline

    d = W.wurtzite_slab(4, 3, 4, seed=32)
    pos, box, n = d["pos"], d["box"], len(d["pos"])
    dims = 1 if cv == "q6" else 2
    wl = dict(WZ, cv=cv, precision=precision, sigma=[20.0, 20.0][:dims])
    prm = dataclasses.replace(params_for(wl, max_neighbors=128), brick=(2, 2, 2), tpa=2, lds_kb=lds_kb)
    ft = torch.float32 if precision == "fp32" else torch.float64
    pipe = Pipeline(n, prm)
    p4 = to_dev(W.as_float4(pos))
    pipe.build_neighbors_checked(p4, box)
    s = pipe.cv_forward(p4).cpu().numpy()
    seed = torch.tensor([0.0, 1.0][2 - dims:], dtype=torch.float64, device=dev())  # the q6 count's gradient
    out = []
    for _ in range(2):
        F = torch.zeros((n, 4), dtype=ft, device=dev())
        pipe.cv_backward(p4)
        pipe.apply_bias_forces(p4, F, seed)
        out.append(F.cpu().numpy())
    assert pipe.status(True) == 0
    pipe.close()
    s_ref, g_ref, _ = oracle_cvs(orc, pos, box, wl)
    tol_s, tol_f = (1e-5, 1e-4) if precision == "fp32" else (1e-10, 1e-10)
    assert np.all(np.abs(s[:dims] - s_ref) <= tol_s * np.abs(s_ref))
    assert rel_force_err(out[0][:, :3], -g_ref[-1]) <= tol_f
    assert np.array_equal(out[0], out[1])
