"""The K-split tile kernel (more than 16 tokens; 4- and 3-bit group 128, 2-bit group 64) against the oracle at the
sizes where it can go wrong: token tiles with a remainder (the last one moved back over its
neighbour), several token tiles and ragged weight tiles per workgroup, fewer runs of K than waves, waves with one
run more than others, and every pair of tile counts the planner picks on the way."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = 2e-3


def case(bits, N, K, M, seed):
    import oracle
    import torch
    import paper_2306_00978_amd as awq
    g = np.random.default_rng(seed)
    W = (g.standard_normal((N, K)) * 0.02).astype(np.float16)
    x = g.standard_normal((M, K)).astype(np.float16)
    s = g.uniform(0.5, 2.0, K).astype(np.float32)
    quantize = {4: oracle.quantize, 3: oracle.quantize_w3, 2: oracle.quantize_w2}[bits]
    Wdq = oracle.dequant(*quantize(W, s), group=64 if bits == 2 else 128)
    pack = {4: awq.awq_quantize_pack, 3: awq.awq_quantize_pack_w3, 2: awq.awq_quantize_pack_w2}[bits]
    packed = pack(torch.from_numpy(W).cuda(), torch.from_numpy(s).cuda())
    return x, Wdq, packed


@pytest.mark.parametrize("bits", [4, 3, 2])
@pytest.mark.parametrize("N,K", [(16, 256), (48, 768), (80, 1280), (208, 2304), (1040, 512), (4112, 1024)])
def test_tile_kernel_against_the_oracle(bits, N, K):
    import oracle
    import torch
    import paper_2306_00978_amd as awq
    linear = {4: awq.awq_w4a16_linear, 3: awq.awq_w3a16_linear, 2: awq.awq_w2a16_linear}[bits]
    x, Wdq, packed = case(bits, N, K, 300, N + K + bits)
    for M in (17, 31, 32, 33, 48, 77, 97, 128, 129, 300):
        buf = torch.full((M * N + 16,), float("nan"), dtype=torch.float16, device="cuda")
        y = buf[:M * N].view(M, N)
        linear(torch.from_numpy(x[:M]).cuda(), *packed, N, out=y)
        first = y.cpu().numpy().copy()
        assert bool(torch.isnan(buf[M * N:]).all())                     # nothing written past the end
        assert np.all(np.isfinite(first.astype(np.float32))), (M, "unwritten output")
        err = oracle.norm_error(first, oracle.matmul(x[:M], Wdq), x[:M], Wdq)
        assert err.max() <= TOL, (M, err.max())
        linear(torch.from_numpy(x[:M]).cuda(), *packed, N, out=y)
        assert np.array_equal(first.view(np.uint16), y.cpu().numpy().view(np.uint16))


def test_tile_kernel_keeps_infinities_and_nan_in_their_rows():
    """A token with an infinity or a NaN must not touch another token's outputs, also where a token
    tile is moved back over its neighbour."""
    import torch
    import paper_2306_00978_amd as awq
    N, K, M = 64, 512, 37
    x, _, packed = case(4, N, K, M, 5)
    clean = awq.awq_w4a16_linear(torch.from_numpy(x).cuda(), *packed, N).cpu().numpy()
    bad = x.copy()
    bad[20, 3], bad[30, 100] = np.inf, np.nan
    y = awq.awq_w4a16_linear(torch.from_numpy(bad).cuda(), *packed, N).cpu().numpy()
    others = [m for m in range(M) if m not in (20, 30)]
    assert np.array_equal(y[others].view(np.uint16), clean[others].view(np.uint16))
    assert not np.any(np.isfinite(y[20].astype(np.float32))) and np.all(np.isnan(y[30]))
