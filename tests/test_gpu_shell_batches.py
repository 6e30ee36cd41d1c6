"""Many-shell kernels on batches of different lattices and vectors, ragged at
both tile sizes (32 x 16 and 64 x 32): every lattice and vector is its own."""
import numpy as np
import pytest

import oracle as O
from paper_2509_26269_amd import synth as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# (lattice, copies, vectors): 64 x 32 tiles for the HVP (512 of them and more) and 32 x 16
@pytest.mark.parametrize("Lx,Ly,B,nvec", [(65, 33, 128, 3), (65, 33, 9, 5), (5, 7, 300, 4)])
@pytest.mark.parametrize("ns", [7, 17, 35])
@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("layout", [0, 1])
def test_every_lattice_and_vector_is_its_own(Lx, Ly, B, nvec, ns, dt, layout):
    from paper_2509_26269_amd import moto as M

    p = S.ham_pdfeir(Lx, Ly, n_shells=ns)
    h = O.Ham(**p.asdict())
    plan = M.Plan.from_params(p)
    tdt = torch.float64 if dt == "f64" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(Lx + ns)
    m = torch.randn(B, 3, h.N, generator=g, device="cuda", dtype=torch.float64)
    m = (m / m.norm(dim=1, keepdim=True)).to(tdt)
    mask = (torch.rand(B, h.N, generator=g, device="cuda") < 0.8).to(torch.uint8)
    V = torch.randn(B, nvec, 3 - layout, h.N, generator=g, device="cuda", dtype=tdt)
    if layout == M.MOTO_AMBIENT:
        V = V - (V * m[:, None]).sum(2, keepdim=True) * m[:, None]
    V = V.contiguous()
    E, grad, c, F, _ = M.moto_energy_grad(plan, m, mask=mask)
    W = M.moto_tangent_hvp(plan, m, c, V, layout, mask=mask, batch=B)
    # rounding in the working precision times the norm bound; vectors are up to 5 long and the frames add to it
    tol = (1e-13 if dt == "f64" else 2e-6) * h.h_est()
    for b in (0, 1, B // 2, B - 1):
        mb, cb, on = m[b].double().cpu().numpy(), c[b].double().cpu().numpy(), mask[b].cpu().numpy()
        Eo, go, co, Fo = O.energy_grad(h, mb)
        assert abs(float(E[b]) - Eo) <= tol * h.N
        assert np.abs(grad[b].double().cpu().numpy() - go).max() <= tol
        assert np.abs(cb - co).max() <= tol
        assert np.abs(F[b].double().cpu().numpy() - Fo * on).max() <= tol
        for j in (0, nvec - 1):
            v = V[b, j].double().cpu().numpy()
            ref = O.tangent_hvp(h, mb, cb, O.from_frame(mb, v) if layout else v, mask=on)
            ref = O.to_frame(mb, ref) if layout else ref
            assert np.abs(W[b, j].double().cpu().numpy() - ref).max() <= 20 * tol, (b, j)
