"""FP32 q6 at and above 1,048,576 atoms (up to there the neighbour rows list the pairs about the taper shell first, above
they stay in slot order), against the FP64 oracle on one period of a box that is repeated along z.

Coordinates and box lengths are multiples of 2^-13 A, so that every copy (below 1,024 A) holds the same differences to
the bit.  Tolerances: the bars of FP32 arithmetic, 1e-5 of the CV and 1e-4 of the largest force."""
import numpy as np
import pytest

import workloads as W
from tests.helpers import oracle_cvs, params_for, rel_force_err
from tests.test_gpu_parity import to_dev
from tests.test_gpu_unwrapped_large import WL

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("copies", [8, 9])
def test_rows_of_repeated_boxes(orc, copies):
    from paper_2510_06873_amd import Pipeline

    x, species, box = W.wurtzite_ideal(32, 32, 16)
    grid = 2.0 ** -13
    box = np.round(np.asarray(box, np.float64) / grid) * grid
    pos = np.random.default_rng(11).normal(0.0, 0.16, x.shape) + x
    pos = np.mod(np.round(pos / grid) * grid, box)
    assert len(pos) == 1 << 17 and copies * box[2] < 1024
    big = np.concatenate([pos + [0.0, 0.0, k * box[2]] for k in range(copies)]).astype(np.float32)
    n = len(big)
    p4 = to_dev(W.as_float4(big, np.tile(species, copies)))
    pipe = Pipeline(n, params_for(WL))
    pipe.build_neighbors_checked(p4, box * [1, 1, copies])
    s = pipe.cv_forward(p4).cpu().numpy()
    pipe.cv_backward(p4)
    F = torch.zeros((n, 4), device="cuda")
    pipe.apply_bias_forces(p4, F, torch.ones(1, dtype=torch.float64, device="cuda"))
    assert pipe.status(True) == 0
    s_ref, g_ref, _ = oracle_cvs(orc, pos.astype(np.float32), box, WL)
    assert abs(s[0] - copies * s_ref[0]) <= 1e-5 * abs(copies * s_ref[0])
    assert rel_force_err(F.cpu().numpy()[:, :3], -np.tile(g_ref[0], (copies, 1))) <= 1e-4
    pipe.close()
