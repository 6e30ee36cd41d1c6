"""The order of the energy sums: lattices of at most four 32 x 8 tiles are summed
inside one workgroup, with the bits of the two launches that larger ones take
(tile sums first, then a butterfly over the tiles)."""
import numpy as np
import pytest

from paper_2509_26269_amd import synth as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _butterfly(x):
    """Sum over the last axis (64 lanes): partner 32 lanes away first."""
    while x.shape[-1] > 1:
        h = x.shape[-1] // 2
        x = x[..., :h] + x[..., h:]
    return x[..., 0]


def _sum_by_tiles(e, Lx, Ly):
    nx, ny = -(-Lx // 32), -(-Ly // 8)
    pad = np.zeros((ny * 8, nx * 32))
    pad[:Ly, :Lx] = e.reshape(Ly, Lx)
    tiles = pad.reshape(ny, 8, nx, 32).transpose(0, 2, 1, 3).reshape(ny * nx, 4, 64)  # tile, wave, lane
    waves = _butterfly(tiles)
    t = np.zeros(64)
    for i in range(4):
        t[: ny * nx] += waves[:, i]
    return _butterfly(t)


# one to four tiles, ragged ones, and five (the two launches)
@pytest.mark.parametrize("Lx,Ly", [(32, 8), (5, 7), (64, 8), (33, 9), (96, 8), (32, 24), (20, 19), (128, 8), (64, 16),
                                   (61, 13), (32, 40)])
@pytest.mark.parametrize("want_dtheta", [False, True])
def test_sums_in_the_order_of_the_two_launches(Lx, Ly, want_dtheta):
    """Without couplings and with B = (0, 0, 1) a site's energy is -m_z exactly."""
    from paper_2509_26269_amd import moto as M

    plan = M.Plan(Lx, Ly, [0.0], [0.0], 0.0, (0.0, 0.0, 1.0))
    N = Lx * Ly
    rng = np.random.default_rng(N)
    m = np.stack([S.random_texture(N, rng) for _ in range(40)])
    md = torch.as_tensor(m, device="cuda")
    E, _, _, _, dth = M.moto_energy_grad(plan, md, want_dtheta=want_dtheta)
    want = np.array([_sum_by_tiles(-mb[2], Lx, Ly) for mb in m])
    assert np.array_equal(E.cpu().numpy(), want)
    if want_dtheta:
        assert np.array_equal(dth[:, -1].cpu().numpy(), want)


# three and four tiles, one lattice below and at the batch that takes the two launches
@pytest.mark.parametrize("Lx,Ly,B", [(32, 32, 1023), (32, 32, 1024), (32, 24, 1365), (32, 24, 1366), (64, 8, 2049)])
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_batch_does_not_change_a_lattice(Lx, Ly, B, dt):
    from paper_2509_26269_amd import moto as M

    plan = M.Plan.from_params(S.ham_3shell(Lx, Ly))
    g = torch.Generator(device="cuda").manual_seed(B)
    m = torch.randn(B, 3, plan.N, generator=g, device="cuda", dtype=torch.float64)
    m = (m / m.norm(dim=1, keepdim=True)).to(torch.float64 if dt == "f64" else torch.float32)
    for dtheta in (False, True):
        all_ = M.moto_energy_grad(plan, m, want_dtheta=dtheta)
        for b in (0, B // 2, B - 1):
            one = M.moto_energy_grad(plan, m[b : b + 1].contiguous(), want_dtheta=dtheta)
            for x, y in zip(all_, one):
                assert x is None or torch.equal(x[b : b + 1], y)
