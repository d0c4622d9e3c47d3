"""The default bricks and lanes of systems on both sides of the choice's lines (few cells, below and above 8,192
atoms, both precisions, staging of a quarter, a third and a half of a CU), against the FP64 oracle at the bars
of the parity tests: CV 1e-5 (FP32) / 1e-10 (FP64), forces 1e-4 / 1e-10."""
import numpy as np
import pytest

import workloads as W
from tests.helpers import oracle_cvs, rel_force_err
from tests.test_gpu_parity import make_pipe, run_step

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BASE = dict(taper=0.2, bond_d0=0.7, bond_w=0.02, count_n0=5.5, count_w=0.25, w0=W.W0_EV, gamma=10.0, kBT=W.KBT_EV,
            hills=dict(k=4), sigma=[20.0])
FCC = dict(BASE, cv="coord", r_c=6.0, skin=0.5, cn_r0=3.0)
WZ = dict(BASE, cv="q6", r_c=3.6, skin=0.4, cn_r0=2.5)


@pytest.mark.parametrize("wl,cells", [(FCC, 6), (FCC, 9), (FCC, 14), (WZ, (4, 3, 4)), (WZ, (14, 8, 9)), (WZ, (15, 8, 9))])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_default_geometry_against_the_oracle(orc, wl, cells, precision):
    wl = dict(wl, precision=precision)
    d = W.fcc_jittered(cells, seed=31) if wl["cv"] == "coord" else W.wurtzite_slab(*cells, seed=32)
    pos, box, n = d["pos"], d["box"], len(d["pos"])
    pipe = make_pipe(wl, n, max_neighbors=128)
    F_in = W.external_forces(n, seed=9)
    s, F = run_step(pipe, pos, d["species"], box, F_in, [0.37])
    s_ref, g_ref, _ = oracle_cvs(orc, pos, box, wl)
    tol_s, tol_f = (1e-5, 1e-4) if precision == "fp32" else (1e-10, 1e-10)
    assert abs(s[0] - s_ref[0]) <= tol_s * abs(s_ref[0])
    # the coordination's gradient is 2/N of a pair sum: forces in units of it, so that the FP32 force they are
    # added to does not hide them
    scale = 1.0 if wl["cv"] == "q6" else n / 2.0
    if scale != 1.0:
        s, F = run_step(pipe, pos, d["species"], box, F_in, [scale])
    dv = 0.37 if scale == 1.0 else scale
    assert rel_force_err(F[:, :3] - F_in[:, :3].astype(np.float64), -dv * g_ref[0]) <= tol_f
