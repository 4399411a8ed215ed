"""Grouped 3-bit launches at nine tokens and more, where the activations go through LDS: ragged last batches (groups of K
not a multiple of four), rows split over the two units of a workgroup and whole ones, a row block more than
whole steps.  Against the oracle, and the same launch twice."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = 2e-3


@pytest.mark.parametrize("M", [9, 13, 16])
@pytest.mark.parametrize("shapes", [
    [(1280, 1280), (160, 1280), (272, 4352), (2400, 384)],
    [(112, 2432), (32, 640), (16, 8448), (4112, 1408)],
    [(8192, 3968), (8192, 2048), (2048, 8192)],
])
def test_w3_rows_launch_against_the_oracle(M, shapes):
    import oracle
    import torch
    import paper_2306_00978_amd as awq
    if M != 16 and shapes[0][0] == 8192:
        pytest.skip("the large group at one size")
    g = np.random.default_rng(M)
    linears, expect = [], []
    for N, K in shapes:
        W = torch.randn((N, K), generator=torch.Generator().manual_seed(N + K)).mul_(0.02).half()
        x = g.standard_normal((M, K)).astype(np.float16)
        s = g.uniform(0.5, 2.0, K).astype(np.float32)
        Wdq = oracle.dequant(*oracle.quantize_w3(W.numpy(), s))
        y = torch.full((M * N + 16,), float("nan"), dtype=torch.float16, device="cuda")
        packed = awq.awq_quantize_pack_w3(W.cuda(), torch.from_numpy(s).cuda())
        linears.append((torch.from_numpy(x).cuda(), *packed, y[:M * N].view(M, N), N))
        expect.append((x, Wdq, y))
    awq.awq_w3a16_linear_multi(linears)
    first = [y.cpu().numpy().copy() for _, _, y in expect]
    awq.awq_w3a16_linear_multi(linears)
    for (x, Wdq, y), got in zip(expect, first):
        n = M * Wdq.shape[0]
        assert np.all(np.isnan(got[n:]))                   # nothing written past the end
        assert np.array_equal(got[:n].view(np.uint16), y.cpu().numpy()[:n].view(np.uint16))
        err = oracle.norm_error(got[:n].reshape(M, -1), oracle.matmul(x, Wdq), x, Wdq)
        assert err.max() <= TOL, err.max()
