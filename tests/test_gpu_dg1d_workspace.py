"""The 1-D driver's workspace holds the state volumes that a step of each order uses and no more, and a step writes
nothing past it."""
import ctypes

import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1809_10186_amd as qc  # noqa: E402


@pytest.mark.parametrize("inv_kn", [0.0, 1.0])
def test_state_volumes_by_order(inv_kn):
    N, E, K = 8, 3, 2
    plan = qc.Plan(N, 5.0, 3, sphere=W.sphere_rule(6), omega=0.81)
    d = qc.Dg1d(plan, [0.0, 0.3, 0.5, 1.0], K - 1, inv_kn, qc.Bc("wall", T=0.9), qc.Bc("wall", T=1.2))
    L = qc.lib()
    need = [int(L.qcoll_dg1d_workspace_bytes(d._h, rk)) for rk in range(4)]
    vol = E * K * N ** 3 * 8
    # L(F) in rk 1, the first stage in rk 2, two stages in rk 3
    assert [n - need[0] for n in need] == [0, vol, vol, 2 * vol]
    F0 = torch.from_numpy(W.maxwellian_mixture(E * K, N, 5.0, 6).reshape(E, K, N, N, N)).to("cuda")
    for rk in (1, 2, 3):
        want = d.step(F0.clone(), 0.002, rk=rk)
        ws = torch.full((need[rk] + 4096,), 0x5a, dtype=torch.uint8, device="cuda")
        F = F0.clone()
        torch.cuda.synchronize()
        assert L.qcoll_dg1d_step(d._h, qc._ptr(F), 0.002, rk, qc._ptr(ws), ctypes.c_size_t(need[rk]), None) == 0
        torch.cuda.synchronize()
        assert torch.equal(F, want) and bool((ws[need[rk]:] == 0x5a).all())
        assert L.qcoll_dg1d_step(d._h, qc._ptr(F), 0.002, rk, qc._ptr(ws), ctypes.c_size_t(need[rk] - 1), None) != 0
