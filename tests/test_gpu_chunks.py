"""Items per chunk: the default, a chunk of 64 and a workspace sized for fewer items give the same bits; and the
bilinear gain loop, whose last pairs may take the two passes, gives those of the two-pass schedule."""
import ctypes

import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1809_10186_amd as qc  # noqa: E402


def _fields(items, N, seed):
    f = W.maxwellian_mixture(7, N, 6.0, seed)
    return torch.from_numpy(f).to("cuda").repeat((items + 6) // 7, 1, 1, 1)[:items].contiguous()


def _call(plan, op, f, g, ws_bytes):
    L = qc.lib()
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
    out = torch.full_like(f, float("nan"))
    n, w, s = f.shape[0], (qc._ptr(ws), ctypes.c_size_t(ws_bytes)), qc._stream(None)
    if op == 0:
        code = L.qcoll_eval(plan._h, n, qc._ptr(f), qc._ptr(out), *w, s)
    elif op == 1:
        code = L.qcoll_vjp(plan._h, n, qc._ptr(f), qc._ptr(g), qc._ptr(out), None, 1, *w, s)
    else:
        code = L.qcoll_eval_bilinear(plan._h, n, qc._ptr(f), qc._ptr(g), qc._ptr(out), *w, s)
    torch.cuda.synchronize()
    return code, out


@pytest.mark.parametrize("N,items,precision,alpha", [
    (8, 2100, qc.QCOLL_FP32, 1.0), (8, 300, qc.QCOLL_FP64, 1.0), (8, 300, qc.QCOLL_FP64, 1.5),
    (12, 1030, qc.QCOLL_FP32, 1.0), (12, 270, qc.QCOLL_FP64, 1.0), (16, 520, qc.QCOLL_FP32, 1.0),
    (16, 270, qc.QCOLL_FP64, 1.0), (16, 70, qc.QCOLL_FP32, 1.3), (24, 135, qc.QCOLL_FP64, 1.0),
    (24, 65, qc.QCOLL_FP32, 1.0), (32, 66, qc.QCOLL_FP64, 1.0)])
def test_default_chunk_and_smaller_workspaces(N, items, precision, alpha):
    print(f"case N={N} items={items} prec={precision} alpha={alpha}", flush=True)
    plan = qc.Plan(N, 6.0, 3, sphere=W.sphere_rule(6), omega=0.81, precision=precision, alpha=alpha)
    f, g = _fields(items, N, 3), _fields(items, N, 4)
    for op in (0, 1, 2):
        # the chunk a workspace always has to hold: the fused adjoint 256 items, the two-pass adjoint 32
        fused = precision == qc.QCOLL_FP32 and alpha == 1.0
        least = plan.workspace_bytes(64 if op != 1 or N == 32 else (256 if fused else 32), op)
        code, a = _call(plan, op, f, g, plan.workspace_bytes(items, op))
        assert code == 0, qc.lib().qcoll_last_error()
        code, b = _call(plan, op, f, g, least)
        assert code == 0, qc.lib().qcoll_last_error()
        assert torch.equal(a, b)
        assert _call(plan, op, f, g, plan.workspace_bytes(1, op) // 2)[0] != 0   # refused before any launch
        if op != 1:
            plan.set_chunk(64)
            code, c = _call(plan, op, f, g, plan.workspace_bytes(items, op))
            assert code == 0 and torch.equal(a, c)
            plan.set_chunk(0)


@pytest.mark.parametrize("N,N_rho,items", [(24, 4, 43), (24, 4, 44), (24, 4, 75), (24, 4, 111), (32, 3, 22),
                                           (32, 4, 40), (32, 4, 49), (32, 2, 129)])
def test_bilinear_pairs_past_the_last_full_set(N, N_rho, items):
    print(f"case N={N} N_rho={N_rho} items={items}", flush=True)
    plan = qc.Plan(N, 6.0, N_rho, sphere=W.sphere_rule(6), omega=0.74, precision=qc.QCOLL_FP32)
    f, g = _fields(items, N, 5), _fields(items, N, 6)
    a = plan.eval_bilinear(f, g)
    plan.set_schedule(1)
    assert torch.equal(a, plan.eval_bilinear(f, g))


def test_group_in_a_workspace_sized_for_fewer_items():
    f = _fields(300, 8, 8)
    plan = qc.Plan(8, 6.0, 4, sphere=W.sphere_rule(6), omega=0.81, precision=qc.QCOLL_FP32)
    small, whole = qc.Group([plan], [64]), qc.Group([plan], [300])
    want = whole.eval([f], conserve=False, use_graph=False)[0].clone()
    L = qc.lib()
    nb = L.qcoll_group_workspace_bytes(small._h, 0)
    assert nb < L.qcoll_group_workspace_bytes(whole._h, 0)
    ws, Q = torch.empty(nb, dtype=torch.uint8, device="cuda"), torch.zeros_like(f)
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    for _ in range(3):
        Q.zero_()
        torch.cuda.synchronize()
        assert L.qcoll_group_eval(whole._h, qc.Group._arr([f]), qc.Group._arr([Q]), 0, qc._ptr(ws),
                                  ctypes.c_size_t(nb), ctypes.c_void_p(st.cuda_stream), 1) == 0
        torch.cuda.synchronize()
        assert torch.equal(Q, want)
    assert L.qcoll_group_eval(whole._h, qc.Group._arr([f]), qc.Group._arr([Q]), 0, qc._ptr(ws),
                              ctypes.c_size_t(256), None, 0) != 0


@pytest.mark.parametrize("N,N_rho,items,few", [(8, 9, 20, 3), (12, 9, 20, 3), (16, 9, 131, 16), (16, 3, 131, 16),
                                               (24, 11, 60, 8), (32, 9, 18, 5), (32, 2, 18, 5)])
def test_low_rank_parts_in_turn_and_side_by_side(N, N_rho, items, few):
    """The low-rank pass sums its pairs in the same four parts at any number of items."""
    print(f"case N={N} N_rho={N_rho} items={items}", flush=True)
    plan = qc.Plan(N, 6.0, N_rho, sphere=W.sphere_rule(6), omega=0.81)
    f = _fields(items, N, 9)
    a = plan.eval(f)
    plan.set_chunk(few)
    assert torch.equal(a, plan.eval(f))
    assert torch.equal(a[:1], plan.eval(f[:1].contiguous()))
