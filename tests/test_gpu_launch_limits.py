"""Batches of tiny lattices that need more threads than one launch may have
(2^32): the call must take them in several launches.  The last lattices are
compared with a call of their own."""
import pytest

from paper_2509_26269_amd import synth as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _plan(Lx, Ly, shells):
    from paper_2509_26269_amd import moto as M

    if shells == 3:
        return M, M.Plan.from_params(S.ham_3shell(Lx, Ly))
    return M, M.Plan.from_params(S.ham_pdfeir(Lx, Ly, n_shells=shells))


def _spins(plan, B):
    # every 64 lattices the same
    g = torch.Generator(device="cuda").manual_seed(B)
    m = torch.randn(64, 3, plan.N, generator=g, device="cuda")
    m = m / m.norm(dim=1, keepdim=True)
    return m.repeat(-(-B // 64), 1, 1)[:B].contiguous()


# 256 threads a tile: 2^24 tiles (and groups of vectors) of the gather, 2^24 of the many-shell tiles
@pytest.mark.parametrize("Lx,Ly,B,nvec,shells,layout", [(4, 4, (1 << 24) + 70, 1, 3, 1), (1, 2, (1 << 23) + 70, 8, 3, 0),
                                                        (3, 1, (1 << 23) + 70, 8, 3, 1), (1, 2, (1 << 22) + 70, 4, 4, 1)])
def test_hvp_of_many_tiny_lattices(Lx, Ly, B, nvec, shells, layout):
    M, plan = _plan(Lx, Ly, shells)
    m = _spins(plan, B)
    c = (m * m.roll(1, dims=0)).sum(1)
    V = m.repeat(1, nvec, 1)[:, : nvec * (3 - layout)].reshape(B, nvec, 3 - layout, plan.N).contiguous()
    W = torch.full_like(V, float("nan"))
    M.moto_tangent_hvp(plan, m, c, V, layout, W=W, batch=B)
    for lo, hi in ((0, 64), (B // 2, B // 2 + 64), (B - 64, B)):
        own = M.moto_tangent_hvp(plan, m[lo:hi].contiguous(), c[lo:hi].contiguous(), V[lo:hi].contiguous(), layout,
                                 batch=hi - lo)
        assert torch.equal(W[lo:hi], own)
    assert bool(torch.isfinite(W).all())


# 512 threads a tile
def test_energies_of_many_tiny_lattices():
    B = (1 << 23) + 70
    M, plan = _plan(1, 2, 4)
    m = _spins(plan, B)
    out = M.moto_energy_grad(plan, m)
    for lo, hi in ((0, 64), (B - 64, B)):
        own = M.moto_energy_grad(plan, m[lo:hi].contiguous())
        for x, y in zip(out[:4], own[:4]):
            assert torch.equal(x[lo:hi], y)
    assert all(bool(torch.isfinite(x).all()) for x in out[:4])
