"""Energy/gradient at the edges of its two forms: lattices of at most four
32 x 8 tiles take one workgroup and write their sums directly, larger ones a
workgroup per tile and a second reduction; the sums formed depend on what the
caller asks for, the vector outputs must not."""
import numpy as np
import pytest

import oracle as O
from paper_2509_26269_amd import synth as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# one tile, four tiles in a row / column / square, five, and sizes below a tile
@pytest.mark.parametrize("Lx,Ly", [(32, 8), (128, 8), (32, 32), (64, 16), (32, 33), (129, 8), (33, 17), (2, 3), (1, 40)])
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_energy_forms_agree_with_oracle(Lx, Ly, dt):
    from paper_2509_26269_amd import moto as M

    p = S.ham_3shell(Lx, Ly)
    p.B = (0.011, -0.017, 0.03)
    h = O.Ham(**p.asdict())
    plan = M.Plan.from_params(p)
    B = 3
    rng = np.random.default_rng(Lx * 100 + Ly)
    ms = np.stack([S.random_texture(h.N, rng) for _ in range(B)])
    md = torch.as_tensor(ms, dtype=torch.float64 if dt == "f64" else torch.float32, device="cuda")
    mask = torch.as_tensor((rng.random((B, h.N)) < 0.7).astype(np.uint8), device="cuda")
    full = M.moto_energy_grad(plan, md, mask=mask, want_dtheta=True)
    some = M.moto_energy_grad(plan, md, mask=mask)
    for a, b in zip(full[1:4], some[1:4]):
        assert torch.equal(a, b)
    # FP64 sums of N terms of size h_est in any order; FP32 terms carry their own rounding
    tol = (1e-13 if dt == "f64" else 2e-6) * h.h_est() * h.N
    ref = [O.energy_grad(h, md[b].double().cpu().numpy()) for b in range(B)]
    for E in (full[0], some[0]):
        assert np.abs(E.cpu().numpy() - np.array([r[0] for r in ref])).max() <= tol
    th = full[4].cpu().numpy()
    # E is linear in theta
    theta = np.array(list(p.J) + list(p.D) + [p.K] + list(p.B))
    assert np.abs(th @ theta - np.array([r[0] for r in ref])).max() <= 4 * tol
    vt = (1e-13 if dt == "f64" else 2e-6) * h.h_est()
    on = mask.cpu().numpy()
    for b in range(B):
        _, g, c, F = ref[b]
        assert np.abs(some[1][b].double().cpu().numpy() - g).max() <= vt
        assert np.abs(some[2][b].double().cpu().numpy() - c).max() <= vt
        assert np.abs(some[3][b].double().cpu().numpy() - F * on[b]).max() <= vt
