"""Masked populations whose Gram kernels get fewer workgroups a member than a
solve of their own (more than 4096 in all): sums are taken in other groups, so
the pairs agree to the tolerance of the solve and no longer bit for bit."""
import numpy as np
import pytest

from paper_2509_26269_amd import synth as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 2])
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_capped_population_agrees_with_own_solves(k, dt):
    from paper_2509_26269_amd import moto as M

    L, P = 96, 17  # 288 chunks of 64 rows: 256 workgroups alone, 241 a member in the population
    plan = M.Plan.from_params(S.ham_3shell(L, L))
    hvp, tol = (M.MOTO_F64, 1e-8) if dt == "f64" else (M.MOTO_F32, 1e-5)
    rng = np.random.default_rng(k)
    start = S.skyrmion(L, L, 6.0)
    m = torch.as_tensor(np.stack([S.add_tilt_noise(start, 0.02 * (1 + y % 3), rng) for y in range(P)]), device="cuda")
    x, y = np.meshgrid(np.arange(L), np.arange(L))
    disc = (((x - L / 2) ** 2 + (y - L / 2) ** 2) < 18.0**2).astype(np.uint8).ravel()
    mask = torch.as_tensor(np.tile(disc, (P, 1)), device="cuda").contiguous()
    opts = M.eig_opts(hvp, tol=tol, max_iter=400)
    pop = M.moto_min_modes_population(plan, m.contiguous(), k, hvp, mask=mask, opts=opts)
    bound = tol * plan.hessian_norm_bound()
    for b in (0, P // 2, P - 1):
        one = M.moto_min_modes(plan, m[b].contiguous(), k, hvp, mask=mask[b].contiguous(), opts=opts)
        assert one.status == pop.status[b] == M.CONVERGED
        assert float(pop.resid[b].max()) <= bound and float(one.resid.max()) <= bound
        # an eigenvalue lies within the residual norm of a computed one; FP32 products add 1e-6 of the bound
        slack = 2 * bound + (2e-6 * plan.hessian_norm_bound() if dt == "f32" else 0.0)
        assert float((pop.evals[b] - one.evals).abs().max()) <= slack
