"""The fused adjoint (FP32) with sphere rules around and past the number of terms whose shift factors it holds at a
time, against the FP64 plan of the same rule."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1809_10186_amd as qc  # noqa: E402


@pytest.mark.parametrize("N,M", [(8, 256), (12, 256), (16, 127), (16, 128), (16, 129), (24, 128), (24, 129),
                                 (24, 256)])
def test_fused_adjoint_of_large_sphere_rules(N, M):
    print(f"case N={N} M={M}", flush=True)
    i = np.arange(M) + 0.5   # Fibonacci points of the half sphere, equal weights
    z, phi = i / M, np.pi * (1 + 5 ** 0.5) * i
    r = np.sqrt(1 - z * z)
    sph = np.ascontiguousarray(np.stack([r * np.cos(phi), r * np.sin(phi), z], 1)), np.full(M, 2 * np.pi / M)
    f = W.maxwellian_mixture(2, N, 6.0, 30 + N)
    g = W.cotangent(f, 3)
    f, g = torch.from_numpy(f).to("cuda"), torch.from_numpy(g).to("cuda")
    out = {}
    for prec in (qc.QCOLL_FP32, qc.QCOLL_FP64):
        plan = qc.Plan(N, 6.0, 2, sphere=sph, omega=0.81, precision=prec)
        out[prec] = [x.cpu().numpy() for x in plan.vjp(f, g, want_domega=True, through_conserve=True)]
    for a, b in zip(out[qc.QCOLL_FP32], out[qc.QCOLL_FP64]):
        err = np.abs(a - b).max() / np.abs(b).max()
        print(f"rel_linf={err:.3e}", flush=True)
        assert err <= 5e-5
