"""What the serving loop charges a walker is at least what its context holds after the first rebuild, plus its positions
and forces: halos that repeat an atom up to 27 times (a last brick of one cell on every axis, bricks of one cell), on
both sides of 131,072 atoms, wide rows, both precisions."""
import dataclasses

import numpy as np
import pytest

import workloads as W
from tests.test_gpu_parity import to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lattice,size,kind,brick", [
    ("fcc", 29, 1, (3, 3, 3)),          # 97,556 atoms in 16 cells per axis
    ("fcc", 29, 1, (0, 0, 0)), ("fcc", 33, 1, (4, 4, 4)), ("fcc", 9, 1, (1, 1, 1)),
    ("wz", (20, 12, 13), 2, (3, 3, 3)), ("wz", (20, 12, 13), 3, (0, 0, 0)), ("wz", (5, 4, 4), 3, (1, 1, 2))])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("kmax", [128, 512])
def test_charged_at_least_what_is_held(lattice, size, kind, brick, precision, kmax):
    from paper_2510_06873_amd import Params, Pipeline
    from paper_2510_06873_amd.serving import Request, device_bytes

    if lattice == "fcc":
        d = W.fcc_jittered(size, seed=31)
        pos, box = d["pos"], d["box"]
        r = dict(r_c=6.0, skin=0.5, cn_r0=3.0)
    else:
        pos, _, box = W.wurtzite_ideal(*size)
        pos = W._wrap_f32(pos, box)
        r = dict(r_c=3.6, skin=0.4, cn_r0=2.5)
    n = len(pos)
    prm = Params(cv_kind=kind, precision=precision, sigma=[1.0, 1.0], hill_capacity=1000, max_neighbors=kmax, brick=brick, **r)
    pipe = Pipeline(n, prm)
    pipe.build_neighbors_checked(to_dev(W.as_float4(pos)), box)
    held = pipe.device_bytes() + n * (16 + 4 * (8 if precision else 4))
    req = Request(0, 0.0, np.zeros((n, 4), np.float32), np.asarray(box), dataclasses.replace(prm), np.zeros((0, 1)),
                  np.zeros(0), np.zeros((n, 4), np.float32))
    assert held <= device_bytes(req)
    pipe.close()
