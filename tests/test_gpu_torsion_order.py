"""Torsion forces: every atom's terms are added in torsion order, rounded to the force type after each term,
whatever the chunk a torsion falls into (64 at a time).  The same sums taken torsion by torsion, one call each,
must therefore give the same bits; the whole also agrees with the FP64 oracle's gradient (tolerance: 4 atoms per
torsion, at most 4 x count roundings of the running force; FP64 gradients of well-bent quadruples, 1e-14)."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count", [1, 63, 64, 65, 200])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_forces_equal_those_of_single_calls(orc, count, dtype):
    import paper_2510_06873_amd as P

    d = W.peptide_in_solvent(n_solvent=200)
    rng = np.random.default_rng(9 + count)
    # backbone quadruples of the chain, either way round: 10 atoms, so every atom is in many torsions
    at = rng.integers(0, 7, count)[:, None] + np.arange(4)
    quads = d["chain"][np.where(rng.random(count)[:, None] < 0.5, at, at[:, ::-1])].astype(np.int32)
    if count > 2:
        quads[count // 2, 1] = -1  # an index out of range: no force from this torsion
    pos = torch.from_numpy(W.as_float4(d["pos"])).cuda()
    n = pos.shape[0]
    q = torch.from_numpy(quads).cuda()
    dV = torch.from_numpy(rng.normal(size=count)).cuda()
    F0 = torch.from_numpy(rng.normal(size=(n, 4))).to(dtype).cuda()
    F, G = F0.clone(), F0.clone()
    P.torsion_forces(pos, q, d["box"], dV, F)
    for t in range(count):
        P.torsion_forces(pos, q[t:t + 1].contiguous(), d["box"], dV[t:t + 1].contiguous(), G)
    assert torch.equal(F, G)
    ok = (quads >= 0).all(1)
    ref = F0.cpu().numpy().astype(np.float64)
    _, grad = orc.torsions(d["pos"], d["box"], quads[ok])
    for t, g, f in zip(quads[ok], grad, dV.cpu().numpy()[ok]):
        for k in range(4):
            ref[t[k], :3] -= f * g[k]
    eps = 6e-8 if dtype == torch.float32 else 2e-16
    big = np.abs(ref).max() + np.abs(dV.cpu().numpy()).max() * max(np.abs(grad).max(), 1.0) * 8
    assert np.abs(F.cpu().numpy() - ref).max() <= ((4 * count + 8) * eps + 1e-14 * count) * big
