"""The 1-D driver's transport, wall densities and fused Runge-Kutta updates at every compile-time node count (K = 1..4)
and past it, against the oracle's scheme: FP64 throughout, 1e-12 of the largest value after one step."""
import numpy as np
import pytest

import workloads as W
from oracle import rkdg, spectral

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1809_10186_amd as qc  # noqa: E402


@pytest.mark.parametrize("order,rk,n_elem", [(0, 2, 3), (1, 3, 1), (2, 1, 2), (3, 2, 2), (4, 3, 2), (6, 2, 1)])
def test_step_matches_the_oracle(order, rk, n_elem):
    print(f"case order={order} rk={rk} elements={n_elem}", flush=True)
    N, L, Nr = 8, 5.0, 3
    sph = W.sphere_rule(6)
    P = spectral.Params(N, L, Nr, sph[0], sph[1], 1.0)
    faces = np.cumsum(np.r_[0.0, 0.3 + 0.1 * np.arange(n_elem)])
    F = W.maxwellian_mixture(n_elem * (order + 1), N, L, 5).reshape(n_elem, order + 1, N, N, N)
    ref = rkdg.Dg1d(faces, order, P, 0.7, rkdg.Bc("wall", u=(0.1, 0.0, 0.0), T=0.9), rkdg.Bc("wall", T=1.2))
    want = ref.step(F, 0.003, rk=rk)
    plan = qc.Plan(N, L, Nr, sphere=sph, omega=1.0)
    d = qc.Dg1d(plan, faces, order, 0.7, qc.Bc("wall", u=(0.1, 0.0, 0.0), T=0.9), qc.Bc("wall", T=1.2))
    Fg = torch.from_numpy(F.copy()).to("cuda")
    d.step(Fg, 0.003, rk=rk)
    err = np.abs(Fg.cpu().numpy() - want).max() / np.abs(want).max()
    moved = np.abs(want - F).max() / np.abs(want).max()
    print(f"rel {err:.3e} (step moved {moved:.1e})", flush=True)
    assert err <= 1e-12
