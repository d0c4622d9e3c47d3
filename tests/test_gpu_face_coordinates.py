"""Coordinates at the far face: exactly float(L) where that lies below L (inside the box) and the next float
(outside), against the oracle: neighbour sets bit-exact, CV and forces at the bars of the parity tests."""
import numpy as np
import pytest

import workloads as W
from tests.helpers import oracle_cvs, rel_force_err
from tests.test_gpu_parity import Q6CV, gpu_neighbor_sets, make_pipe, run_step

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("step", [0, 1])
def test_atoms_on_the_far_face(orc, step):
    d = W.wurtzite_slab(11, 6, 9, seed=23)
    pos, box = d["pos"].copy(), d["box"]
    axes = [a for a in range(3) if float(np.float32(box[a])) < box[a]]
    assert axes
    for a in axes:
        v = np.float32(box[a])
        near = np.argsort(-pos[:, a])[:3]
        pos[near, a] = v if step == 0 else np.nextafter(v, np.float32(np.inf))
        inside = pos[near, a].astype(np.float64) < box[a]
        assert inside.all() if step == 0 else not inside.any()
    n = len(pos)
    pipe = make_pipe(Q6CV, n)
    F_in = W.external_forces(n, seed=9)
    s, F = run_step(pipe, pos, d["species"], box, F_in, [0.37])
    off, nb = orc.neighbors(pos, box, 4.0)
    rows = gpu_neighbor_sets(pipe)
    for i in range(n):
        assert np.array_equal(rows[i], nb[off[i]:off[i + 1]]), i
    s_ref, g_ref, _ = oracle_cvs(orc, pos, box, Q6CV)
    assert abs(s[0] - s_ref[0]) <= 1e-5 * abs(s_ref[0])
    assert rel_force_err(F[:, :3] - F_in[:, :3].astype(np.float64), -0.37 * g_ref[0]) <= 1e-4
