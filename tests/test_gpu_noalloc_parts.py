"""qcoll_eval_noalloc for FP64 VSS plans at 32^3 whose one item's term volumes pass the fixed scratch: the nodes go
through it in parts, with the bits of qcoll_eval."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1809_10186_amd as qc  # noqa: E402


def _rule(M):
    i = np.arange(M) + 0.5   # Fibonacci points of the half sphere, equal weights
    z, phi = i / M, np.pi * (1 + 5 ** 0.5) * i
    r = np.sqrt(1 - z * z)
    return np.ascontiguousarray(np.stack([r * np.cos(phi), r * np.sin(phi), z], 1)), np.full(M, 2 * np.pi / M)


# nodes a launch: 63 of 64, 14 of 16, 3 of 7 (whose last part of the sums is continued)
@pytest.mark.parametrize("N_rho,M", [(64, 16), (16, 67), (7, 255)])
def test_parts_of_the_nodes_give_the_bits_of_eval(N_rho, M):
    print(f"case N_rho={N_rho} M={M}", flush=True)
    plan = qc.Plan(32, 6.0, N_rho, sphere=_rule(M), omega=0.81, alpha=1.5)
    f = torch.from_numpy(W.maxwellian_mixture(2, 32, 6.0, 24)).to("cuda")
    out = torch.empty_like(f)
    plan.eval_noalloc(f, out)
    assert torch.equal(out, plan.eval(f))
