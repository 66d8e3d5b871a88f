"""The low-rank pass with its pairs side by side (few items) and in turn (many): the same bits on every grid, with
pair counts around whole rounds of the four waves and items around whole workgroups of pencils."""
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1809_10186_amd as qc  # noqa: E402


@pytest.mark.parametrize("N,many", [(8, 70), (12, 40), (16, 260), (24, 260), (32, 35)])
@pytest.mark.parametrize("N_rho", [1, 2, 7, 8, 9, 17])
def test_side_by_side_gives_the_bits_of_in_turn(N, many, N_rho):
    plan = qc.Plan(N, 6.0, N_rho, sphere=W.sphere_rule(6), omega=0.81)
    f = torch.from_numpy(W.maxwellian_mixture(5, N, 6.0, 50 + N)).to("cuda").repeat(many // 5, 1, 1, 1)
    plan.set_chunk(many)
    a = plan.eval(f)
    for few in (1, 3):
        print(f"case N={N} N_rho={N_rho} items={few}", flush=True)
        assert torch.equal(plan.eval(f[:few].contiguous()), a[:few])
