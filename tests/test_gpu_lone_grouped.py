"""One linear of many features through the grouped call at five tokens and more: the kernel that takes the activations through LDS, as
the tuning build runs it with the batch and tile kernels left out, bit for bit."""
import pytest

from tuning_build import tuning_build

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K", [(16400, 1024), (24576, 3584), (40960, 1024), (65552, 640)])
@pytest.mark.parametrize("M", [5, 9, 16])
def test_many_features_go_through_lds(M, N, K):
    import torch
    import paper_2306_00978_amd as awq
    g = torch.Generator(device="cuda").manual_seed(N + M)
    packed = awq.awq_quantize_pack((torch.randn((N, K), generator=g, device="cuda") * 0.02).half(), None)
    x = torch.randn((M, K), generator=g, device="cuda").half()
    ys = []
    for few in (None, 0):
        ys.append(torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda"))
        with tuning_build(AWQ_FEW=few):
            awq.awq_w4a16_linear_multi([(x, *packed, ys[-1], N)])
    assert torch.equal(*ys)
    codes, scales, zeros = awq.awq_unpack(*packed, N, K)
    w = ((codes.float().view(N, K // 128, 128) - zeros.float()[..., None]) * scales.float()[..., None]).view(N, K).double()
    ref = x.double() @ w.T
    # the rounding to fp16, products cut off 17 bits below the largest (codes as fp16 subnormals), fp32 sums
    assert torch.all((ys[0].double() - ref).abs() <= 2.0 ** -11 * ref.abs() + 2.0 ** -16 * (x.double().abs() @ w.abs().T) + 2.0 ** -24)
