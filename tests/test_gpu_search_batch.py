"""awq_search_scale with several candidates at a time against one at a time: the workspace that it is given decides."""
import pytest

pytestmark = pytest.mark.gpu


# 16 tokens: one at a time whatever the workspace; 17, 159: the tile kernel; 513 x 4112 and 2125 x 1040: the prefill kernel, ragged;
# 16, 17 and 33 points: one launch, two, three, the last one shorter; 3 x 128: a table of powers that needs a place of its own
@pytest.mark.parametrize("T,N,K,points", [(16, 64, 256, 3), (17, 16, 1280, 16), (17, 272, 1280, 17), (159, 1120, 2944, 20), (33, 32, 128, 33),
                                          (513, 4112, 1024, 5), (2125, 1040, 384, 7), (1000, 4112, 256, 1)])
def test_several_candidates_at_a_time(T, N, K, points):
    import torch
    import paper_2306_00978_amd as awq
    lib = awq.load()
    g = torch.Generator(device="cuda").manual_seed(T + N + K)
    W = (torch.randn((N, K), generator=g, device="cuda") * 0.02).half()
    gain = torch.ones(K, device="cuda")
    gain[torch.randperm(K, generator=g, device="cuda")[:max(1, K // 100)]] = 20.0
    X = (torch.randn((T, K), generator=g, device="cuda") * gain).half()
    alphas = [i / points for i in range(points)]
    least = lib.awq_search_scale_workspace_bytes(T, N, K, points, 128)
    most = lib.awq_search_scale_batch_workspace_bytes(T, N, K, points, 128)
    assert most >= least and (most > least) == (T > 16 and points > 1)
    one, all_of_them = None, None
    for size in sorted({least, (least + most) // 2, most - 1, most, most + 4096} - {least - 1}):
        workspace = torch.full((size + 256,), 0xA5, dtype=torch.uint8, device="cuda")
        best, losses, s = awq.awq_search_scale(W, X, alphas, workspace=workspace[:size])
        assert torch.equal(workspace[size:], torch.full_like(workspace[size:], 0xA5))
        if one is None:
            one = losses
        # other orders of fp32 sums: an output that rounds the other way changes the loss as the rounding of outputs itself
        # does, 1e-4 of it and a cross term of 2e-2 / sqrt(outputs) standard deviation at the most
        assert torch.all((losses / one - 1).abs() <= 1e-4 + 0.06 / (T * N) ** 0.5), (size, losses, one)
        assert int(best) == int(losses.argmin())
        assert torch.equal(s, awq.awq_act_scale(X, alphas[int(best)]))
        all_of_them = losses
    assert torch.equal(awq.awq_search_scale(W, X, alphas)[1], all_of_them)
    with pytest.raises(RuntimeError):
        awq.awq_search_scale(W, X, alphas, workspace=torch.empty(least - 1, dtype=torch.uint8, device="cuda"))
