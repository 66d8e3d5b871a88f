"""The FP64 term loops at 32^3 with one term, one volume or all terms a workgroup and their sums by pencils or by
points: the same operations in the same order, so an item's bits do not depend on how many come with it."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1809_10186_amd as qc  # noqa: E402


@pytest.mark.parametrize("N_rho,M", [(1, 1), (2, 2), (3, 7), (4, 6), (8, 12), (16, 5)])
def test_any_number_of_items_gives_the_same_bits(N_rho, M):
    pts, w = W.sphere_rule(12)
    sph = np.ascontiguousarray(pts[:M]), np.full(M, 2.0 * np.pi / M)
    n = 40
    f = torch.from_numpy(W.maxwellian_mixture(n, 32, 6.0, 25)).to("cuda")
    g = torch.from_numpy(W.cotangent(f.cpu().numpy(), 26)).to("cuda")
    vss = qc.Plan(32, 6.0, N_rho, sphere=sph, omega=0.81, alpha=1.5)
    vhs = qc.Plan(32, 6.0, N_rho, sphere=sph, omega=0.81)
    Q = vss.eval(f)
    df, dw = vhs.vjp(f, g, want_domega=True)
    for few in (1, 2, 3, 5, 9, 17):
        print(f"case N_rho={N_rho} M={M} items={few}", flush=True)
        a, b = f[n - few:].contiguous(), g[n - few:].contiguous()
        assert torch.equal(vss.eval(a), Q[n - few:])
        d, x = vhs.vjp(a, b, want_domega=True)
        assert torch.equal(d, df[n - few:]) and torch.equal(x, dw[n - few:])
        assert torch.equal(vhs.vjp(a, b)[0], df[n - few:])
