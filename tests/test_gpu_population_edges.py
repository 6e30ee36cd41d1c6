"""Population eigen-solves at the edges of the narrow row kernels: rows that do
not fill a chunk, fewer and more chunks than blocks, block widths 3 and 4 (the
narrow kernels) and 5 (the general ones), members that stop at different
iterations.  A member of a population must give the bits of its own solve."""
import numpy as np
import pytest

from paper_2509_26269_amd import synth as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# 2 N rows: 70 (a chunk and six rows), 234, 1056, 33800 (529 chunks on 256 blocks)
@pytest.mark.parametrize("Lx,Ly", [(5, 7), (9, 13), (33, 16), (130, 130)])
@pytest.mark.parametrize("k,guard", [(1, 2), (2, 2), (2, 3)])
@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("masked", [False, True])
def test_member_equals_its_own_solve(Lx, Ly, k, guard, dt, masked):
    from paper_2509_26269_amd import moto as M

    p = S.ham_3shell(Lx, Ly)
    plan = M.Plan.from_params(p)
    hvp, tol = (M.MOTO_F64, 1e-9) if dt == "f64" else (M.MOTO_F32, 1e-5)
    rng = np.random.default_rng(Lx)
    start = S.skyrmion(Lx, Ly, min(Lx, Ly) / 5.0)
    m = np.stack([S.add_tilt_noise(start, s, rng) for s in (0.02, 0.3, 0.1)])
    md = torch.as_tensor(m, device="cuda").contiguous()
    mask = None
    if masked:
        mask = torch.as_tensor((rng.random((3, plan.N)) < 0.6).astype(np.uint8), device="cuda")
    opts = M.eig_opts(hvp, tol=tol, guard=guard, max_iter=60)
    pop = M.moto_min_modes_population(plan, md, k, hvp, mask=mask, opts=opts)
    for y in range(3):
        one = M.moto_min_modes(plan, md[y].contiguous(), k, hvp, mask=None if mask is None else mask[y].contiguous(),
                               opts=opts)
        assert (one.status, one.iters, one.n_hvp) == (pop.status[y], pop.iters[y], pop.n_hvp[y])
        assert torch.equal(one.evals, pop.evals[y]) and torch.equal(one.V, pop.V[y])
        if one.status == M.CONVERGED:
            assert float(one.resid.max()) <= tol * plan.hessian_norm_bound()


# the convergence control is taken inside the next iteration's first small step,
# except at the end of a chunk of iterations: the chunk length changes nothing
@pytest.mark.parametrize("Lx,Ly", [(9, 13), (130, 130)])
@pytest.mark.parametrize("k,guard", [(1, 0), (1, 1), (1, 2), (2, 2), (2, 3)])
@pytest.mark.parametrize("max_iter", [5, 60])
def test_chunk_length_changes_nothing(Lx, Ly, k, guard, max_iter):
    from paper_2509_26269_amd import moto as M

    p = S.ham_3shell(Lx, Ly)
    plan = M.Plan.from_params(p)
    m = S.add_tilt_noise(S.skyrmion(Lx, Ly, min(Lx, Ly) / 5.0), 0.1, np.random.default_rng(Ly))
    md = torch.as_tensor(m, device="cuda").contiguous()
    out = []
    for every in (1, 3, 8):
        opts = M.eig_opts(M.MOTO_F64, tol=1e-7, guard=guard, max_iter=max_iter, check_every=every)
        out.append(M.moto_min_modes(plan, md, k, M.MOTO_F64, opts=opts))
    for r in out[1:]:
        assert (r.status, r.iters, r.n_hvp) == (out[0].status, out[0].iters, out[0].n_hvp)
        assert torch.equal(r.evals, out[0].evals) and torch.equal(r.V, out[0].V)
        assert torch.equal(r.resid, out[0].resid)
    assert out[0].iters <= max_iter
