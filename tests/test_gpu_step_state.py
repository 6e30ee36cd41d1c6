"""The step's state may begin at any double: a caller may cut it out of a larger
allocation."""
import pytest

from paper_2509_26269_amd import synth as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mem,k", [(1, 0), (8, 1), (16, 2)])
def test_state_aligned_to_doubles(mem, k):
    from paper_2509_26269_amd import moto as M

    plan = M.Plan.from_params(S.ham_3shell(33, 17))
    g = torch.Generator(device="cuda").manual_seed(mem)
    m0 = torch.randn(3, plan.N, generator=g, device="cuda", dtype=torch.float64)
    m0 = (m0 / m0.norm(dim=0)).contiguous()
    V = torch.randn(max(k, 1), 3, plan.N, generator=g, device="cuda", dtype=torch.float64)
    V = V / V.flatten(1).norm(dim=1)[:, None, None]
    opts = M.step_opts(mem=mem, tau_F=1e-12)
    out = []
    for shift in (0, 8):
        st = M.StepState(plan, mem=mem)
        whole = torch.zeros(st.nbytes + 16, dtype=torch.uint8, device="cuda")
        st.buf = whole[shift : shift + st.nbytes]
        assert st.buf.data_ptr() % 16 == shift
        m = m0.clone()
        for _ in range(mem + 3):
            F = M.moto_energy_grad(plan, m, want_grad=False, want_c=False)[3]
            M.moto_reflected_step(plan, m, F, V if k else None, k, st, opts)
        out.append((m, st.out.clone()))
        assert not whole[:shift].any() and not whole[shift + st.nbytes :].any()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
