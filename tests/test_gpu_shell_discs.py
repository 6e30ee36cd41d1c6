"""General-shell kernels at the edges of their discs (10, 20 and 36 shells) and
tiles (32 x 16 and 64 x 32 sites), against the oracle."""
import numpy as np
import pytest

import oracle as O
from paper_2509_26269_amd import synth as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _params(Lx, Ly, ns):
    p = S.ham_pdfeir(Lx, Ly, n_shells=min(ns, 35))
    p.J = (p.J + [1e-5])[:ns]
    p.D = [p.D[0]] + [0.0] * (ns - 1)
    p.B = (0.011, -0.017, 0.03)
    return p


# (lattice, copies of it): below a tile, one site over, exact; the last makes the 64 x 32 tiles the choice
@pytest.mark.parametrize("Lx,Ly,B,nvec", [(7, 5, 1, 1), (33, 17, 1, 2), (32, 16, 2, 1), (65, 33, 16, 16)])
@pytest.mark.parametrize("ns", [4, 10, 11, 20, 21, 36])
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_disc_edges(Lx, Ly, B, nvec, ns, dt):
    from paper_2509_26269_amd import moto as M

    p = _params(Lx, Ly, ns)
    h = O.Ham(**p.asdict())
    plan = M.Plan.from_params(p)
    rng = np.random.default_rng(100 * Lx + ns)
    tdt = torch.float64 if dt == "f64" else torch.float32
    m1, v1 = S.random_texture(h.N, rng), rng.standard_normal((2, h.N))
    on1 = (rng.random(h.N) < 0.8).astype(np.uint8)
    md = torch.as_tensor(m1, dtype=tdt, device="cuda").expand(B, 3, h.N).contiguous()
    mk = torch.as_tensor(on1, device="cuda").expand(B, h.N).contiguous()
    V = torch.as_tensor(v1, dtype=tdt, device="cuda").expand(B, nvec, 2, h.N).contiguous()
    E, g, c, F, _ = M.moto_energy_grad(plan, md, mask=mk)
    W = M.moto_tangent_hvp(plan, md, c, V, M.MOTO_FRAME, mask=mk, batch=B)
    # copies of one state: every copy equals the first bit for bit
    for t in (E, g, c, F, W):
        assert torch.equal(t, t[:1].expand_as(t))
    assert torch.equal(W, W[:, :1].expand_as(W))
    m_in, v_in, c_in = (x.double().cpu().numpy() for x in (md[0], V[0, 0], c[0]))
    Eo, go, co, Fo = O.energy_grad(h, m_in)
    # sums of at most 366 bonds: rounding in the working precision times the norm bound, with room for the order
    tol = (1e-13 if dt == "f64" else 2e-6) * h.h_est()
    assert abs(float(E[0]) - Eo) <= tol * h.N
    assert np.abs(g[0].double().cpu().numpy() - go).max() <= tol
    assert np.abs(c_in - co).max() <= tol
    assert np.abs(F[0].double().cpu().numpy() - Fo * on1).max() <= tol
    ref = O.to_frame(m_in, O.tangent_hvp(h, m_in, c_in, O.from_frame(m_in, v_in), mask=on1))
    # the frames add a few roundings of vectors up to 4 long
    assert np.abs(W[0, 0].double().cpu().numpy() - ref).max() <= 20 * tol
