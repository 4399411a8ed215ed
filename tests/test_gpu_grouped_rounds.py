"""Grouped decode launches for which eight-wave workgroups would be more than the CUs: re-planned with four waves, or,
where a row needs all eight for its activations, with more row blocks to a workgroup.  Against the oracle, and the
same launch twice."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = 2e-3


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("M,shapes", [
    (1, [(41600, 512), (64, 4352)]),                       # 326 eight-wave workgroups: four waves
    (2, [(20816, 1024), (16, 2432), (48, 4352)]),
    (4, [(41600, 512), (64, 8448)]),                       # eight waves needed: two row-block steps each
    (3, [(20816, 512), (20800, 512), (16, 9344)]),
])
def test_one_round_of_workgroups(bits, M, shapes):
    import oracle
    import torch
    import paper_2306_00978_amd as awq
    g = np.random.default_rng(M + bits)
    quantize = {4: oracle.quantize, 3: oracle.quantize_w3}[bits]
    pack = {4: awq.awq_quantize_pack, 3: awq.awq_quantize_pack_w3}[bits]
    multi = {4: awq.awq_w4a16_linear_multi, 3: awq.awq_w3a16_linear_multi}[bits]
    linears, expect = [], []
    for N, K in shapes:
        W = (g.standard_normal((N, K), dtype=np.float32) * 0.02).astype(np.float16)
        x = g.standard_normal((M, K)).astype(np.float16)
        s = g.uniform(0.5, 2.0, K).astype(np.float32)
        Wdq = oracle.dequant(*quantize(W, s))
        y = torch.full((M * N + 16,), float("nan"), dtype=torch.float16, device="cuda")
        packed = pack(torch.from_numpy(W).cuda(), torch.from_numpy(s).cuda())
        linears.append((torch.from_numpy(x).cuda(), *packed, y[:M * N].view(M, N), N))
        expect.append((x, Wdq, y))
    multi(linears)
    first = [y.cpu().numpy().copy() for _, _, y in expect]
    multi(linears)
    for (x, Wdq, y), got in zip(expect, first):
        n = M * Wdq.shape[0]
        assert np.all(np.isnan(got[n:]))                   # nothing written past the end
        assert np.array_equal(got[:n].view(np.uint16), y.cpu().numpy()[:n].view(np.uint16))
        err = oracle.norm_error(got[:n].reshape(M, -1), oracle.matmul(x, Wdq), x, Wdq)
        assert err.max() <= TOL, err.max()
