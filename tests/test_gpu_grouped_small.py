"""Grouped 4-bit launches at five to eight tokens on both sides of the rule that keeps small ones with the streaming
kernel: all linears of short K, one that does not fit it, and a launch just beyond the size.  Against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = 2e-3


@pytest.mark.parametrize("M", [5, 6, 7])
@pytest.mark.parametrize("shapes", [
    [(1280, 1280), (160, 1280), (272, 3840)],
    [(640, 1152), (48, 8448)],                            # K beyond the register-resident activations
    [(16384, 2048), (16400, 2048)],                       # more than 32 MB
])
def test_grouped_launch_at_five_to_seven_tokens(M, shapes):
    import oracle
    import torch
    import paper_2306_00978_amd as awq
    g = np.random.default_rng(M)
    linears, expect = [], []
    for N, K in shapes:
        W = torch.randn((N, K), generator=torch.Generator().manual_seed(N + K)).mul_(0.02).half()
        x = g.standard_normal((M, K)).astype(np.float16)
        s = g.uniform(0.5, 2.0, K).astype(np.float32)
        Wdq = oracle.dequant(*oracle.quantize(W.numpy(), s))
        y = torch.full((M * N + 16,), float("nan"), dtype=torch.float16, device="cuda")
        packed = awq.awq_quantize_pack(W.cuda(), torch.from_numpy(s).cuda())
        linears.append((torch.from_numpy(x).cuda(), *packed, y[:M * N].view(M, N), N))
        expect.append((x, Wdq, y))
    awq.awq_w4a16_linear_multi(linears)
    for x, Wdq, y in expect:
        n = M * Wdq.shape[0]
        got = y.cpu().numpy()
        assert np.all(np.isnan(got[n:]))                   # nothing written past the end
        err = oracle.norm_error(got[:n].reshape(M, -1), oracle.matmul(x, Wdq), x, Wdq)
        assert err.max() <= TOL, err.max()
