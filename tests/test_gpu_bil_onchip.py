"""The bilinear gain loop on chip (FP32, N <= 32) against the two-pass schedule: the same operations in the same
order, so the same bits, below and above the launch size at which the library switches between them."""
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1809_10186_amd as qc  # noqa: E402


@pytest.mark.parametrize("N,N_rho,M,items,svd_tol", [
    (8, 16, 6, 15, 0.0), (8, 16, 6, 16, 0.0), (12, 7, 16, 37, 0.0), (16, 8, 12, 33, 1e-6), (24, 16, 12, 17, 0.0),
    (32, 13, 6, 4, 0.0), (32, 13, 6, 5, 0.0), (32, 5, 16, 70, 1e-6)])
def test_onchip_bilinear_gives_the_two_pass_bits(N, N_rho, M, items, svd_tol):
    print(f"case N={N} N_rho={N_rho} M={M} items={items} svd={svd_tol}", flush=True)
    svd = dict(svd_rank=0, svd_tol=svd_tol) if svd_tol else {}
    plan = qc.Plan(N, 6.0, N_rho, sphere=W.sphere_rule(M), omega=0.74, precision=qc.QCOLL_FP32, **svd)
    f = torch.from_numpy(W.maxwellian_mixture(items, N, 6.0, 70 + N)).to("cuda")
    g = torch.from_numpy(W.maxwellian_mixture(items, N, 6.0, 90 + N, noise=0.1)).to("cuda")
    a = plan.eval_bilinear(f, g)
    plan.set_schedule(1)
    assert torch.equal(a, plan.eval_bilinear(f, g))
