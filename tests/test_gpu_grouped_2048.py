"""Grouped calls at five to eight tokens with rows of 2048 columns beside longer ones: by the streaming kernel from 18 thousand weight tiles (as the tuning build
runs them with the batch and tile kernels left out, bit for bit), and against fp64 products on both sides of that line."""
import pytest

from tuning_build import tuning_build

pytestmark = pytest.mark.gpu

LAYER = [(2048, 2048), (512, 2048), (512, 2048), (2048, 2048), (5120, 2048), (5120, 2048), (2048, 5120)]      # 20 thousand tiles
SMALLER = [(2048, 2048), (2048, 2048), (4096, 2048), (2064, 5120)]                                             # 13 thousand


@pytest.mark.parametrize("bits,M", [(4, 5), (4, 6), (3, 5), (3, 7), (3, 8)])
@pytest.mark.parametrize("shapes", [LAYER, SMALLER])
def test_rows_of_2048_beside_longer_ones(bits, M, shapes):
    import torch
    import paper_2306_00978_amd as awq
    pack, unpack, multi = ((awq.awq_quantize_pack, awq.awq_unpack, awq.awq_w4a16_linear_multi) if bits == 4 else
                           (awq.awq_quantize_pack_w3, awq.awq_unpack_w3, awq.awq_w3a16_linear_multi))
    g = torch.Generator(device="cuda").manual_seed(10 * M + bits)
    packed = [pack((torch.randn((N, K), generator=g, device="cuda") * 0.02).half(), None) for N, K in shapes]
    xs = [torch.randn((M, K), generator=g, device="cuda").half() for N, K in shapes]
    results = []
    for few in (None, 0):
        ys = [torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda") for N, K in shapes]
        with tuning_build(AWQ_FEW=few):
            multi([(x, *p, y, N) for x, p, y, (N, K) in zip(xs, packed, ys, shapes)])
        results.append(ys)
    if shapes is LAYER:
        assert all(torch.equal(a, b) for a, b in zip(*results))
    for x, p, (N, K), outs in zip(xs, packed, shapes, zip(*results)):
        codes, scales, zeros = unpack(*p, N, K)
        w = ((codes.double().view(N, K // 128, 128) - zeros.double()[..., None]) * scales.double()[..., None]).view(N, K)
        ref = x.double() @ w.T
        # the rounding to fp16, products cut off 17 bits below the largest (codes as fp16 subnormals), fp32 sums
        bound = 2.0 ** -11 * ref.abs() + 2.0 ** -16 * (x.double().abs() @ w.abs().T) + 2.0 ** -24
        for y in outs:
            assert torch.all((y.double() - ref).abs() <= bound), (N, K)
