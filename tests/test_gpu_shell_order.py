"""Neighbour rows that list the pairs about the taper shell first: the lists a caller copies out keep the order of
lists that know no shell (exactly, also when rows are cut at max_neighbors), and forces on atoms that have moved
up to half the skin since the build, so that pairs cross the shell both ways, meet the FP64 oracle at the bars of
the parity tests: CV 1e-5 (FP32) / 1e-10 (FP64), forces 1e-4 / 1e-10."""
import dataclasses

import numpy as np
import pytest

import workloads as W
from tests.helpers import oracle_cvs, params_for, rel_force_err
from tests.test_gpu_parity import run_step, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

WZ = dict(taper=0.2, bond_d0=0.7, bond_w=0.02, count_n0=5.5, count_w=0.25, w0=W.W0_EV, gamma=10.0, kBT=W.KBT_EV,
          hills=dict(k=4), r_c=3.6, skin=0.4, cn_r0=2.5)


@pytest.mark.parametrize("kmax", [12, 20, 64])
@pytest.mark.parametrize("tpa", [1, 2, 4])
def test_copied_lists_keep_their_order(tpa, kmax):
    from paper_2510_06873_amd import Pipeline

    d = W.wurtzite_slab(7, 5, 5, seed=22)
    rows = []
    for cv in ("q6", "coord"):  # the coordination's lists know no shell
        wl = dict(WZ, cv=cv, precision="fp32", sigma=[20.0])
        pipe = Pipeline(len(d["pos"]), dataclasses.replace(params_for(wl, max_neighbors=kmax), brick=(2, 2, 2), tpa=tpa))
        pipe.build_neighbors(to_dev(W.as_float4(d["pos"])), d["box"])
        nbr, cnt = (t.cpu().numpy() for t in pipe.neighbor_lists())
        used = np.arange(nbr.shape[1])[None, :] < np.minimum(cnt, nbr.shape[1])[:, None]
        rows.append((cnt, np.where(used, nbr, -1)))
        pipe.close()
    assert np.array_equal(rows[0][0], rows[1][0]) and np.array_equal(rows[0][1], rows[1][1])


@pytest.mark.parametrize("tpa", [1, 2, 4])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_pairs_crossing_the_shell(orc, precision, tpa):
    from paper_2510_06873_amd import Pipeline

    d = W.wurtzite_slab(7, 5, 5, seed=22)
    box, n = d["box"], len(d["pos"])
    wl = dict(WZ, cv="q6", precision=precision, sigma=[20.0])
    step = np.random.default_rng(tpa).normal(size=(n, 3))
    step *= 0.199 / np.linalg.norm(step, axis=1, keepdims=True)  # every atom by just less than half the skin
    pos = (d["pos"] + step).astype(np.float32)
    pipe = Pipeline(n, dataclasses.replace(params_for(wl, max_neighbors=64), tpa=tpa))
    F_in = W.external_forces(n, seed=9)
    run_step(pipe, d["pos"], d["species"], box, F_in, [0.37])  # builds the lists at the first positions
    p4 = to_dev(W.as_float4(pos, d["species"]))
    s = pipe.cv_forward(p4).cpu().numpy()
    pipe.cv_backward(p4)
    F = to_dev(F_in, pipe.fdtype)
    pipe.apply_bias_forces(p4, F, torch.tensor([0.37], dtype=torch.float64, device=F.device))
    assert pipe.status(True) == 0
    s_ref, g_ref, _ = oracle_cvs(orc, pos, box, wl)
    tol_s, tol_f = (1e-5, 1e-4) if precision == "fp32" else (1e-10, 1e-10)
    assert abs(s[0] - s_ref[0]) <= tol_s * abs(s_ref[0])
    F = F.cpu().numpy().astype(np.float64)
    assert rel_force_err(F[:, :3] - F_in[:, :3].astype(np.float64), -0.37 * g_ref[0]) <= tol_f
    pipe.close()
