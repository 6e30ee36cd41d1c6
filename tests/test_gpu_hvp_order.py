"""The gather HVP's workgroup order on grids of every remainder by eight: each
lattice and vector must be worked on once, with the bits of the march."""
import pytest

from paper_2509_26269_amd import synth as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# one tile a lattice, so the grid is the batch (one vector) or a multiple of it
@pytest.mark.parametrize("B", [1, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16, 255, 2049])
@pytest.mark.parametrize("nvec", [1, 5])
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_every_lattice_once(B, nvec, dt):
    from paper_2509_26269_amd import moto as M

    plan = M.Plan.from_params(S.ham_3shell(20, 7))
    g = torch.Generator(device="cuda").manual_seed(B)
    tdt, dtc = (torch.float64, M.MOTO_F64) if dt == "f64" else (torch.float32, M.MOTO_F32)
    m = torch.randn(B, 3, plan.N, generator=g, device="cuda", dtype=torch.float64)
    m = (m / m.norm(dim=1, keepdim=True)).to(tdt)
    c = torch.randn(B, plan.N, generator=g, device="cuda", dtype=tdt)
    V = torch.randn(B, nvec, 2, plan.N, generator=g, device="cuda", dtype=tdt)
    out = []
    for var in (12, 8):  # gather, march
        assert M.lib().moto_plan_set_hvp_variant(plan.handle, dtc, B, nvec, var) == 0
        out.append(M.moto_tangent_hvp(plan, m, c, V, W=torch.full_like(V, float("nan")), batch=B))
    assert torch.equal(*out)


@pytest.mark.parametrize("B", [1, 7, 9, 11, 13, 255])
@pytest.mark.parametrize("nvec", [1, 5])
@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("masked", [False, True])
def test_every_ambient_lattice_once(B, nvec, dt, masked):
    """Ambient lattices of a batch against calls of their own."""
    from paper_2509_26269_amd import moto as M

    plan = M.Plan.from_params(S.ham_3shell(37, 9))
    g = torch.Generator(device="cuda").manual_seed(B)
    tdt = torch.float64 if dt == "f64" else torch.float32
    m = torch.randn(B, 3, plan.N, generator=g, device="cuda", dtype=torch.float64)
    m = (m / m.norm(dim=1, keepdim=True)).to(tdt)
    c = torch.randn(B, plan.N, generator=g, device="cuda", dtype=tdt)
    V = torch.randn(B, nvec, 3, plan.N, generator=g, device="cuda", dtype=tdt)
    mask = (torch.rand(B, plan.N, generator=g, device="cuda") < 0.7).to(torch.uint8) if masked else None
    W = M.moto_tangent_hvp(plan, m, c, V, M.MOTO_AMBIENT, mask=mask, W=torch.full_like(V, float("nan")), batch=B)
    for b in range(0, B, max(1, B // 9)):
        one = M.moto_tangent_hvp(plan, m[b : b + 1].contiguous(), c[b : b + 1].contiguous(), V[b : b + 1].contiguous(),
                                 M.MOTO_AMBIENT, mask=None if mask is None else mask[b : b + 1].contiguous())
        assert torch.equal(W[b : b + 1], one)
