"""The gather and march forms of the frame-layout HVP are two schedules of one
sum: pinned in turn they must agree bit for bit, so that the size rule that
chooses between them cannot change a result.  The ambient form, which always
takes the gather, is compared with the oracle at the edges of its tiles."""
import numpy as np
import pytest

import oracle as O
from paper_2509_26269_amd import synth as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GATHER, MARCH = 12, (7, 8, 9)


def _M():
    from paper_2509_26269_amd import moto as M

    return M


# tiles are 32 x 8: exact, one short, one over, smaller than a tile, narrower than the halo's period
@pytest.mark.parametrize("Lx,Ly,B,nvec", [(32, 8, 2, 1), (31, 9, 1, 3), (33, 7, 3, 5), (64, 16, 1, 12), (4, 5, 2, 2),
                                          (129, 17, 2, 9), (300, 6, 1, 4)])
@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("masked", [False, True])
def test_gather_and_march_give_the_same_bits(Lx, Ly, B, nvec, dt, masked):
    M = _M()
    p = S.ham_3shell(Lx, Ly)
    plan = M.Plan.from_params(p)
    g = torch.Generator(device="cuda").manual_seed(Lx * 1000 + Ly)
    tdt, dtc = (torch.float64, M.MOTO_F64) if dt == "f64" else (torch.float32, M.MOTO_F32)
    m = torch.randn(B, 3, plan.N, generator=g, device="cuda", dtype=torch.float64)
    m = (m / m.norm(dim=1, keepdim=True)).to(tdt)
    c = torch.randn(B, plan.N, generator=g, device="cuda", dtype=tdt)
    V = torch.randn(B, nvec, 2, plan.N, generator=g, device="cuda", dtype=tdt)
    mask = (torch.rand(B, plan.N, generator=g, device="cuda") < 0.7).to(torch.uint8) if masked else None

    def run():
        W = torch.full_like(V, float("nan"))
        return M.moto_tangent_hvp(plan, m, c, V, mask=mask, W=W, batch=B)

    out = {"default": run()}
    for var in (GATHER,) + MARCH:
        if M.lib().moto_plan_set_hvp_variant(plan.handle, dtc, B, nvec, var) == 0:
            out[var] = run()
    assert len(out) >= 4
    for var, W in out.items():
        assert torch.equal(W, out[GATHER]), var


@pytest.mark.parametrize("Lx,Ly,B,nvec", [(32, 8, 1, 1), (33, 9, 2, 6), (3, 2, 2, 2), (1, 5, 1, 3), (70, 15, 1, 2)])
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_ambient_hvp_at_tile_edges(Lx, Ly, B, nvec, dt):
    M = _M()
    p = S.ham_3shell(Lx, Ly)
    h = O.Ham(**p.asdict())
    plan = M.Plan.from_params(p)
    rng = np.random.default_rng(7 * Lx + Ly)
    tdt = torch.float64 if dt == "f64" else torch.float32
    ms = np.stack([S.random_texture(h.N, rng) for _ in range(B)])
    md = torch.as_tensor(ms, dtype=tdt, device="cuda")
    ms = md.double().cpu().numpy()
    cs = np.stack([O.energy_grad(h, ms[b])[2] for b in range(B)])
    V = np.stack([S.random_tangent(ms[b], nvec, rng) for b in range(B)])
    mask = (rng.random((B, h.N)) < 0.8).astype(np.uint8)
    cd, Vd = (torch.as_tensor(x, dtype=tdt, device="cuda") for x in (cs, V))
    W = M.moto_tangent_hvp(plan, md, cd, Vd, M.MOTO_AMBIENT, mask=torch.as_tensor(mask, device="cuda"), batch=B)
    W = W.double().cpu().numpy()
    # an output is a sum of at most 57 products of the bond strength: 1e-12 and 1e-5 of the norm bound leave a
    # factor of 100 over the rounding of the inputs
    tol = (1e-12 if dt == "f64" else 1e-5) * h.h_est()
    for b in range(B):
        for j in range(nvec):
            ref = O.tangent_hvp(h, ms[b], cd[b].double().cpu().numpy(), Vd[b, j].double().cpu().numpy(), mask=mask[b])
            assert np.abs(W[b, j] - ref).max() <= tol * max(1.0, np.abs(V[b, j]).max()), (b, j)
