"""Evaluations of a few items: the on-chip gain loop as one workgroup per
(item, node, sphere point) against one per (item, node).

Both run the same operations in the same order, so their results are the same
bits.  A workspace too small for the per-term volumes selects the second; a
workspace of qcoll_workspace_bytes the first, where the launch is small enough."""
import ctypes

import numpy as np
import pytest

import workloads as W
from oracle import spectral

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1809_10186_amd as qc  # noqa: E402


def _eval(plan, f, ws_bytes):
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
    Q = torch.full_like(f, float("nan"))
    code = qc.lib().qcoll_eval(plan._h, f.shape[0], qc._ptr(f), qc._ptr(Q), qc._ptr(ws), ctypes.c_size_t(ws_bytes),
                               qc._stream(None))
    assert code == 0, qc.lib().qcoll_last_error()
    torch.cuda.synchronize()
    return Q


@pytest.mark.parametrize("N,N_rho,M,items,precision", [
    (12, 5, 6, 1, qc.QCOLL_FP32), (12, 16, 16, 3, qc.QCOLL_FP32), (16, 1, 6, 1, qc.QCOLL_FP32),
    (16, 7, 12, 5, qc.QCOLL_FP32), (24, 3, 6, 2, qc.QCOLL_FP32), (24, 12, 16, 1, qc.QCOLL_FP32),
    (32, 16, 12, 1, qc.QCOLL_FP32), (32, 5, 6, 3, qc.QCOLL_FP32), (16, 8, 6, 1, qc.QCOLL_FP64),
    (16, 3, 16, 4, qc.QCOLL_FP64), (32, 4, 12, 1, qc.QCOLL_FP64), (32, 3, 6, 3, qc.QCOLL_FP64)])
def test_one_workgroup_per_term_gives_the_same_bits(N, N_rho, M, items, precision):
    print(f"case N={N} N_rho={N_rho} M={M} items={items} prec={precision}", flush=True)
    sph = W.sphere_rule(M)
    plan = qc.Plan(N, 6.0, N_rho, sphere=sph, omega=0.81, precision=precision)
    f = W.maxwellian_mixture(items, N, 6.0, 40 + N)
    fg = torch.from_numpy(f).to("cuda")
    full = plan.workspace_bytes(items)
    a = _eval(plan, fg, full)
    plan.set_schedule(2)
    few = _eval(plan, fg, full - 256 if full > 256 else full)
    assert torch.equal(a, few)
    # the same item inside a batch too large for the split
    n = 40
    big = fg[:1].repeat(n, 1, 1, 1).contiguous()
    assert torch.equal(_eval(plan, big, plan.workspace_bytes(n))[n - 1], a[0])
    if N <= 16:
        ref = spectral.collide(f[0], spectral.Params(N, 6.0, N_rho, sph[0], sph[1], 0.81))
        err = np.abs(a[0].cpu().numpy() - ref).max() / np.abs(ref).max()
        print(f"rel_linf={err:.3e}", flush=True)
        assert err <= (1e-12 if precision == qc.QCOLL_FP64 else 2e-5)


def test_workspace_of_a_larger_batch_serves_a_smaller_one():
    """A workspace sized for a batch that does not split holds every smaller
    call, whatever optional parts that call could use."""
    for precision in (qc.QCOLL_FP32, qc.QCOLL_FP64):
        plan = qc.Plan(16, 6.0, 8, sphere=W.sphere_rule(12), omega=0.81, precision=precision)
        f = torch.from_numpy(W.maxwellian_mixture(64, 16, 6.0, 9)).to("cuda")
        ws = plan.workspace_bytes(64)
        whole = _eval(plan, f, ws)
        for n in (1, 2, 3, 7, 20):
            assert torch.equal(_eval(plan, f[:n].contiguous(), ws), whole[:n])
