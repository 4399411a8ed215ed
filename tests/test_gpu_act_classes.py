"""awq_act_scale_ws: the calibration statistic with the rows divided into classes is bit for bit the result of
the call without a workspace -- every number of classes, ragged column blocks, row counts with remainders of
the classes, of the phases and of the rows requested ahead, infinities and NaN."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,K", [(4096, 64), (4097, 1000), (4101, 1024), (6000, 2048), (4229, 2056), (4500, 4096),
                                 (8192, 4104), (8200, 8192), (12289, 4352), (20000, 8)])
def test_row_classes_equal_the_undivided_sums_bit_for_bit(T, K):
    import torch
    import paper_2306_00978_amd as awq
    lib = awq.load()
    need = lib.awq_act_scale_workspace_bytes(T, K)
    assert need > 0 and need % (4 * K) == 0
    g = torch.Generator(device="cuda").manual_seed(T + K)
    X = (torch.randn((T, K), generator=g, device="cuda") * 3).half()
    X[5, 0], X[T - 1, K - 1] = float("inf"), float("nan")
    ws = torch.full((need + 64,), 0xAB, dtype=torch.uint8, device="cuda")
    ref, out = (torch.full((K,), -1.0, device="cuda") for _ in range(2))
    for alpha in (0.5, 1.0):
        st = awq._stream()
        assert lib.awq_act_scale(X.data_ptr(), T, K, alpha, ref.data_ptr(), st) == 0
        assert lib.awq_act_scale_ws(X.data_ptr(), T, K, alpha, out.data_ptr(), ws.data_ptr(), need, st) == 0
        assert np.array_equal(ref.cpu().numpy().view(np.uint32), out.cpu().numpy().view(np.uint32))
        assert np.array_equal(awq.awq_act_scale(X, alpha).cpu().numpy().view(np.uint32), ref.cpu().numpy().view(np.uint32))
    assert bool((ws[need:] == 0xAB).all())
    assert lib.awq_act_scale_ws(X.data_ptr(), T, K, 0.5, out.data_ptr(), ws.data_ptr(), need - 4, st) == -5
    assert lib.awq_act_scale_ws(X.data_ptr(), T, K, 0.5, out.data_ptr(), ctypes.c_void_p(ws.data_ptr() + 4), need, st) == -4


@pytest.mark.parametrize("T,K,own", [(4249, 2240, False), (8200, 1024, True)])
def test_python_call_allocates_a_workspace_where_it_pays_and_only_if_it_may(T, K, own, monkeypatch):
    import torch
    import paper_2306_00978_amd as awq
    need = awq.awq_act_scale_workspace_bytes(T, K)
    assert need > 0
    X = (torch.randn((T, K), device="cuda") * 3).half()
    want = torch.empty(K, device="cuda")
    assert awq.load().awq_act_scale(X.data_ptr(), T, K, 0.5, want.data_ptr(), awq._stream()) == 0
    out, ws = torch.empty(K, device="cuda"), torch.zeros(need, dtype=torch.uint8, device="cuda")

    def allocations(**kw):
        out.fill_(-1.0)
        before = torch.cuda.memory_stats()["allocation.all.allocated"]
        awq.awq_act_scale(X, 0.5, out=out, **kw)
        after = torch.cuda.memory_stats()["allocation.all.allocated"]
        assert torch.equal(out, want)
        return after - before

    assert allocations(workspace=False) == 0
    assert allocations() == int(own)
    assert allocations(workspace=ws) == 0 and bool(ws.any())             # the caller's one was used
    with pytest.raises(awq.AwqError):
        awq.awq_act_scale(X, 0.5, out=out, workspace=ws[:need - 16])

    def full(*a, **kw):
        raise torch.OutOfMemoryError("no room")
    monkeypatch.setattr(torch, "empty", full)
    assert allocations() == 0
