"""The FP64 on-chip term loops at N = 32 (VJP of VHS kernels, gain of VSS kernels) against the two-pass schedule and
the oracle, at launch sizes around their sub-chunks, odd M and few nodes.  Both sides are FP64: their difference is
bounded by the FP64 parity tolerance of the library, 1e-12 of the largest value."""
import numpy as np
import pytest

import workloads as W
from oracle import adjoint, spectral

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1809_10186_amd as qc  # noqa: E402

TOL = 1e-12


def _rel(a, b):
    d = (a - b).abs().flatten(1).amax(1) / b.abs().flatten(1).amax(1)
    return float(d.max())


def _rule(M):
    """The M = 12 rule, or its first M points with their weights scaled to 2 pi."""
    pts, w = W.sphere_rule(12)
    if M == 12:
        return pts, w
    w = np.full(M, 2.0 * np.pi / M)
    return np.ascontiguousarray(pts[:M]), w


@pytest.mark.parametrize("N_rho,M,items", [(3, 5, 1), (16, 12, 3), (4, 6, 17), (1, 1, 33)])
def test_vjp_terms_on_chip_match_two_passes(N_rho, M, items):
    print(f"case vjp N_rho={N_rho} M={M} items={items}", flush=True)
    sph = _rule(M)
    f = W.maxwellian_mixture(items, 32, 6.0, 21)
    g = W.cotangent(f, 22)
    fg, gg = (torch.from_numpy(x).to("cuda") for x in (f, g))
    plan = qc.Plan(32, 6.0, N_rho, sphere=sph, omega=0.81)
    df, dw = plan.vjp(fg, gg, want_domega=True)
    one, wone = plan.vjp(fg[items - 1:].contiguous(), gg[items - 1:].contiguous(), want_domega=True)
    assert torch.equal(one[0], df[items - 1]) and torch.equal(wone[0], dw[items - 1])
    plan.set_schedule(1)
    df2, dw2 = plan.vjp(fg, gg, want_domega=True)
    e, ew = _rel(df, df2), float(((dw - dw2).abs() / (gg * fg).abs().flatten(1).sum(1)).max())
    print(f"df {e:.3e} domega (of sum |f g|) {ew:.3e}", flush=True)
    assert e <= TOL and ew <= TOL
    if items == 1:
        P = spectral.Params(32, 6.0, N_rho, sph[0], sph[1], 0.81)
        ref = adjoint.vjp_f(f[0], g[0], P)
        assert np.abs(df[0].cpu().numpy() - ref).max() <= TOL * np.abs(ref).max()


@pytest.mark.parametrize("N_rho,M,items", [(3, 5, 1), (16, 12, 2), (4, 6, 17), (2, 1, 66)])
def test_vss_terms_on_chip_match_two_passes(N_rho, M, items):
    print(f"case vss N_rho={N_rho} M={M} items={items}", flush=True)
    sph = _rule(M)
    f = W.maxwellian_mixture(items, 32, 6.0, 23)
    fg = torch.from_numpy(f).to("cuda")
    plan = qc.Plan(32, 6.0, N_rho, sphere=sph, omega=0.81, alpha=1.5)
    Q = plan.eval(fg)
    assert torch.equal(plan.eval(fg[items - 1:].contiguous())[0], Q[items - 1])
    out = torch.empty_like(fg)
    plan.eval_noalloc(fg, out)
    assert torch.equal(out, Q)
    plan.set_schedule(1)
    e = _rel(Q, plan.eval(fg))
    print(f"Q {e:.3e}", flush=True)
    assert e <= TOL
    if items == 1:
        P = spectral.Params(32, 6.0, N_rho, sph[0], sph[1], 0.81, vss_alpha=1.5)
        ref = spectral.collide(f[0], P)
        assert np.abs(Q[0].cpu().numpy() - ref).max() <= TOL * np.abs(ref).max()
