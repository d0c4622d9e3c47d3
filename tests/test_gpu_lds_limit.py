"""LDS budgets near the device's limit with halos that fill them, and rows as wide as they may be: the neighbour
build's staging and its rows fit together, and the lists are those of brute force (halos staged in part among them).
A budget that leaves nothing to stage in is refused before anything is launched."""
import numpy as np
import pytest

import workloads as W
from tests.test_gpu_build_rows import same_sets
from tests.test_gpu_parity import to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# r_list, LDS, brick, row width: a halo of 6 x 6 x 6 cells of 52 atoms; rows of 64 KiB beside it; the automatic brick
@pytest.mark.parametrize("r_list,lds_kb,brick,kmax", [(8.5, 160, (4, 4, 4), 256), (8.5, 150, (4, 4, 4), 256),
                                                      (8.5, 128, (4, 4, 4), 4096), (10.5, 160, (0, 0, 0), 512)])
@pytest.mark.parametrize("precision", [0, 1])
def test_dense_halos_near_the_limit(orc, r_list, lds_kb, brick, kmax, precision):
    from paper_2510_06873_amd import Params, Pipeline

    d = W.fcc_jittered(15, seed=31)
    pos, box = d["pos"], d["box"]
    pipe = Pipeline(len(pos), Params(cv_kind=1, precision=precision, r_c=r_list, skin=0.0, cn_r0=3.0, sigma=[1.0],
                                     hill_capacity=4, max_neighbors=kmax, lds_kb=lds_kb, brick=brick))
    p4 = to_dev(W.as_float4(pos))
    pipe.build_neighbors(p4, box)
    assert pipe.status(True) == 0
    same_sets(orc, pipe, pos, box, r_list)
    # the same list from the default budget gives the same CV
    s = pipe.cv_forward(p4).clone()
    other = Pipeline(len(pos), Params(cv_kind=1, precision=precision, r_c=r_list, skin=0.0, cn_r0=3.0, sigma=[1.0],
                                      hill_capacity=4, max_neighbors=kmax))
    other.build_neighbors(p4, box)
    assert torch.allclose(s, other.cv_forward(p4), rtol=1e-5 if precision == 0 else 1e-10, atol=0.0)
    pipe.close()
    other.close()


@pytest.mark.parametrize("kind", [1, 2, 3])
@pytest.mark.parametrize("precision", [0, 1])
def test_a_budget_below_the_static_arrays_is_refused(kind, precision):
    from paper_2510_06873_amd import GmError, Params, Pipeline

    d = W.wurtzite_slab(4, 3, 4, seed=32)
    pipe = Pipeline(len(d["pos"]), Params(cv_kind=kind, precision=precision, sigma=[1.0, 1.0], hill_capacity=4, lds_kb=1))
    with pytest.raises(GmError, match="HIP"):
        pipe.build_neighbors(to_dev(W.as_float4(d["pos"])), d["box"])
    pipe.close()
