"""More than three shells: how exact the field of the energies is, and what a
non-finite spin or vector reaches."""
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
    return p


def _exchange(h, m, t):
    """-2 sum_s J_s sum_{delta in s} m_{i+delta} in type t (couplings of m's own
    type), every shell added up before its coupling is applied."""
    u = m.astype(t).reshape(3, h.Ly, h.Lx)
    out = np.zeros_like(u)
    for s, J in enumerate(h.J):
        acc = np.zeros_like(u)
        for dx, dy, sh in O.shells(len(h.J)):
            if sh == s:
                acc = acc + np.roll(u, (-dy, -dx), axis=(1, 2))
        out = out + t(m.dtype.type(-2.0 * J)) * acc
    return out.reshape(3, -1)


# random spins and a texture; shell counts inside, at and beyond the discs of 10, 20 and 36
@pytest.mark.parametrize("state", ["random", "skyrmion"])
@pytest.mark.parametrize("ns", [4, 10, 11, 20, 21, 35])
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_field_as_exact_as_shell_sums(state, ns, dt):
    """The rms error of the gradient is that of adding shell by shell in the
    working precision, emulated here on the CPU.  The rms over 12288 values
    scatters by a percent; fused multiply-adds only lower it.  One running sum
    over the bonds has more than twice that error at 35 shells."""
    from paper_2509_26269_amd import moto as M

    L = 64
    p = _params(L, L, ns)
    p.K, p.B, p.D = 0.0, (0.0, 0.0, 0.0), [0.0] * ns
    h = O.Ham(**p.asdict())
    plan = M.Plan.from_params(p)
    t, tdt = (np.float64, torch.float64) if dt == "f64" else (np.float32, torch.float32)
    rng = np.random.default_rng(ns)
    m = S.random_texture(h.N, rng) if state == "random" else S.skyrmion(L, L, 9.0)
    m = m.astype(t)
    md = torch.as_tensor(np.ascontiguousarray(m), dtype=tdt, device="cuda")
    _, g, _, _, _ = M.moto_energy_grad(plan, md[None].contiguous())
    exact = _exchange(h, m, np.longdouble)
    err = np.sqrt(np.mean((g[0].cpu().numpy() - exact) ** 2))
    own = np.sqrt(np.mean((_exchange(h, m, t) - exact) ** 2))
    print(f"{state} ns {ns} {dt}: rms error {err / own:.3f} of the emulated sum's")
    assert err <= 1.25 * own


@pytest.mark.parametrize("ns", [4, 7, 11, 13, 21, 30])
@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_bad_spin_reaches_its_shells_only(ns, dt, bad):
    from paper_2509_26269_amd import moto as M

    L = 64
    p = _params(L, L, ns)
    plan = M.Plan.from_params(p)
    m = torch.as_tensor(S.random_texture(L * L, np.random.default_rng(ns)), device="cuda")
    md = m.to(torch.float64 if dt == "f64" else torch.float32)
    x0, y0 = 30, 31  # its disc spans several tiles
    md[0, x0 + L * y0] = bad
    _, g, _, _, _ = M.moto_energy_grad(plan, md[None].contiguous())
    touched = ~torch.isfinite(g[0]).all(0).cpu().numpy().reshape(L, L)
    want = np.zeros((L, L), bool)
    for dx, dy, _ in O.shells(ns):
        want[(y0 - dy) % L, (x0 - dx) % L] = True
    want[y0, x0] = touched[y0, x0]  # its own field holds the anisotropy only
    assert (touched == want).all()


@pytest.mark.parametrize("ns", [4, 7, 10, 11, 13, 21, 30, 36])
@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("layout", [0, 1])
def test_bad_vector_stays_in_the_rows_of_its_bonds(ns, dt, layout):
    """The HVP convolves whole rows of a disc that may hold more shells than the
    plan: a non-finite entry may reach further along a row, by 12 sites at
    most, but no row without a bond."""
    from paper_2509_26269_amd import moto as M

    L = 64
    p = _params(L, L, ns)
    plan = M.Plan.from_params(p)
    tdt = torch.float64 if dt == "f64" else torch.float32
    md = torch.as_tensor(S.random_texture(L * L, np.random.default_rng(ns)), device="cuda").to(tdt)[None].contiguous()
    c = M.moto_energy_grad(plan, md)[2]
    V = torch.zeros(1, 1, 3 - layout, L * L, dtype=tdt, device="cuda")
    x0, y0 = 30, 31
    V[0, 0, :, x0 + L * y0] = float("nan")
    W = M.moto_tangent_hvp(plan, md, c, V, layout)
    touched = ~torch.isfinite(W[0, 0]).all(0).cpu().numpy().reshape(L, L)
    bonds = [(dx, dy) for dx, dy, _ in O.shells(ns)]
    for dx, dy in bonds:
        assert touched[y0 - dy, x0 - dx]
    reach = max(abs(dy) for _, dy in bonds)
    ys, xs = np.nonzero(touched)
    assert np.abs(ys - y0).max() <= reach and np.abs(xs - x0).max() <= 12
