"""A backward pass takes the parameters that its forward pass read: also when its
plan has left the cache since, and never after theta was changed in place."""
import numpy as np
import pytest

from paper_2509_26269_amd import synth as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _passes(E, m, th, u):
    gm, gth = torch.autograd.grad(E, (m, th), create_graph=True)
    return (gm.detach(), gth.detach()) + torch.autograd.grad((gm * u).sum() + gth.sum(), (m, th))


@pytest.mark.parametrize("n", [1, 8, 9, 20])  # the cache holds eight plans
def test_derivatives_after_other_parameters(n):
    from paper_2509_26269_amd import autograd as A

    p = S.ham_3shell(9, 7)
    rng = np.random.default_rng(n)
    m = torch.as_tensor(S.add_tilt_noise(S.skyrmion(9, 7, 2.0), 0.2, rng), device="cuda").requires_grad_(True)
    u = torch.as_tensor(rng.standard_normal((3, 63)), device="cuda")
    ths = [(A.theta_of(p) * (1.0 + 0.01 * i)).requires_grad_(True) for i in range(n)]
    want = [_passes(A.energy(m, th, 9, 7), m, th, u) for th in ths]
    Es = [A.energy(m, th, 9, 7) for th in ths]
    for E, th, w in zip(Es, ths, want):
        for a, b in zip(_passes(E, m, th, u), w):
            assert torch.equal(a, b)


def test_theta_changed_in_place_is_refused():
    from paper_2509_26269_amd import autograd as A

    m = torch.as_tensor(S.skyrmion(9, 7, 2.0), device="cuda").requires_grad_(True)
    th = A.theta_of(S.ham_3shell(9, 7))
    E = A.energy(m, th, 9, 7)
    th.mul_(2.0)
    with pytest.raises(RuntimeError, match="modified by an inplace operation"):
        E.backward()
