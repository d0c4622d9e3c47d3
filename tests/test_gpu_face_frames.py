"""FP64 bricks on periodic faces, whose coordinates are staged shifted: boxes with and without room for the shift on
each axis, atoms on the faces (0, -0 and the last float below the length) and, in one box, one atom outside it
(which takes the general images), against the FP64 oracle at the parity tests' bar, 1e-10."""
import dataclasses

import numpy as np
import pytest

import workloads as W
from tests.helpers import oracle_cvs, params_for, rel_force_err
from tests.test_gpu_parity import run_step

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

WZ = dict(taper=0.2, bond_d0=0.7, bond_w=0.02, count_n0=5.5, count_w=0.25, w0=W.W0_EV, gamma=10.0, kBT=W.KBT_EV,
          hills=dict(k=4), r_c=3.6, skin=0.4, cn_r0=2.5, precision="fp64")


@pytest.mark.parametrize("outside", [False, True])
@pytest.mark.parametrize("cv", ["q6", "coord_q6"])
@pytest.mark.parametrize("cells", [(12, 7, 8), (12, 3, 4), (4, 7, 8)])  # 9 x 9 x 10 cells, few on some axes
def test_faces_against_the_oracle(orc, cells, cv, outside):
    from paper_2510_06873_amd import Pipeline

    d = W.wurtzite_slab(*cells, seed=32)
    pos, box = np.array(d["pos"], np.float32), d["box"]
    n = len(pos)
    last = np.float32(box)
    last = np.where(last.astype(np.float64) >= box, np.nextafter(last, np.float32(0)), last)
    for axis in range(3):  # the three atoms nearest to a face are put on it
        near = np.argsort(np.minimum(pos[:, axis], box[axis] - pos[:, axis]))[:3]
        pos[near, axis] = np.array([0.0, -0.0, last[axis]], np.float32)
    wl = dict(WZ, cv=cv, sigma=[20.0] * (1 if cv == "q6" else 2))
    pipe = Pipeline(n, dataclasses.replace(params_for(wl, max_neighbors=128), brick=(1, 1, 1)))
    given = pos.copy()
    if outside:
        given[n // 2, 0] = np.float32(pos[n // 2, 0] + box[0])
        pos = given
    F_in = W.external_forces(n, seed=9)
    seed = [0.37] if cv == "q6" else [0.0, 0.37]
    s, F = run_step(pipe, given, d["species"], box, F_in, seed)
    s_ref, g_ref, _ = oracle_cvs(orc, pos, box, wl)
    assert np.all(np.abs(s[:len(s_ref)] - s_ref) <= 1e-10 * np.abs(s_ref))
    assert rel_force_err(F[:, :3] - F_in[:, :3].astype(np.float64), -0.37 * g_ref[-1]) <= 1e-10
    pipe.close()
