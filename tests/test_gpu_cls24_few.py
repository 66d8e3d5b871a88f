"""The FP64 gain loop at 24^3 with one workgroup per term against one per (pair, class): the same bits, whichever the
number of items or the workspace selects."""
import ctypes

import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1809_10186_amd as qc  # noqa: E402


@pytest.mark.parametrize("N_rho,M", [(1, 6), (4, 6), (5, 16), (8, 12)])
def test_one_workgroup_per_term_gives_the_same_bits(N_rho, M):
    plan = qc.Plan(24, 6.0, N_rho, sphere=W.sphere_rule(M), omega=0.81)
    n = 90
    f = torch.from_numpy(W.maxwellian_mixture(n, 24, 6.0, 33)).to("cuda")
    Q = plan.eval(f)
    split = 0
    for few in (1, 2, 3, 4, 8):
        print(f"case N_rho={N_rho} M={M} items={few}", flush=True)
        a = f[n - few:].contiguous()
        assert torch.equal(plan.eval(a), Q[n - few:])
        # the smallest workspace that is taken has no room for the terms' volumes
        volumes = few * N_rho * (M - 1) * 24 ** 3 * 16
        full = plan.workspace_bytes(few)
        ws = torch.empty(full, dtype=torch.uint8, device="cuda")
        out = torch.full_like(a, float("nan"))
        code = qc.lib().qcoll_eval(plan._h, few, qc._ptr(a), qc._ptr(out), qc._ptr(ws),
                                   ctypes.c_size_t(max(full - volumes, 0)), qc._stream(None))
        if code == 0:
            split += 1
            assert torch.equal(out, Q[n - few:])
    assert split > 0 or N_rho == 1
