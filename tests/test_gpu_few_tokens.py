"""Decode calls of one or several linears through the batch kernel and the tile kernel (up to 16 tokens) against fp64 products
of the unpacked weights: one row block, row blocks that no workgroup's share divides, fewer groups than waves, uneven shares of them,
one to sixteen tokens; each kernel by force (the tuning build) and as the library chooses."""
import pytest

from tuning_build import tuning_build

pytestmark = pytest.mark.gpu

SHAPES = [(16, 256), (48, 512), (272, 1280), (160, 3840), (1040, 256), (64, 2304), (80, 2048), (32, 10240)]
NAMES = {4: ("awq_quantize_pack", "awq_unpack", "prepare_linear_multi", "awq_w4a16_linear"),
         3: ("awq_quantize_pack_w3", "awq_unpack_w3", "prepare_linear_multi_w3", "awq_w3a16_linear"),
         2: ("awq_quantize_pack_w2", "awq_unpack_w2", "prepare_linear_multi_w2", "awq_w2a16_linear")}


@pytest.mark.parametrize("bits", [4, 3, 2])
@pytest.mark.parametrize("few", [None, 1, 2, 3, 4, 5])
def test_few_tokens(bits, few):
    import torch
    import paper_2306_00978_amd as awq
    pack, unpack, prepare, linear = (getattr(awq, n) for n in NAMES[bits])
    group = 64 if bits == 2 else 128
    g = torch.Generator(device="cuda").manual_seed(bits)
    packed, weights = [], []
    for N, K in SHAPES:
        packed.append(pack((torch.randn((N, K), generator=g, device="cuda") * 0.02).half(), None))
        codes, scales, zeros = unpack(*packed[-1], N, K)
        weights.append(((codes.double().view(N, K // group, group) - zeros.double()[..., None]) * scales.double()[..., None]).view(N, K))
    for M in (1, 2, 3, 4, 5, 7, 8, 9, 15, 16):
        xs = [torch.randn((M, K), generator=g, device="cuda").half() for N, K in SHAPES]
        ys = [torch.full((M + 1, N), 7.0, dtype=torch.float16, device="cuda") for N, K in SHAPES]
        single = [torch.full((M + 1, N), 7.0, dtype=torch.float16, device="cuda") for N, K in SHAPES]
        with tuning_build(AWQ_FEW=few):
            prepare([(x, *p, y[:M], N) for x, p, y, (N, K) in zip(xs, packed, ys, SHAPES)])()
            for x, p, y, (N, K) in zip(xs, packed, single, SHAPES):
                linear(x, *p, N, out=y[:M])
        for x, w, shape, outs in zip(xs, weights, SHAPES, zip(ys, single)):
            ref = x.double() @ w.T
            # the rounding to fp16; fp32 sums of at most 48 terms (10 of a wave's 32 columns at a time and its groups, eight waves), each
            # rounded to 2^-24 of sums of up to four times |x| |w| (codes up to 15, where weights are code less zero point)
            bound = 2.0 ** -11 * ref.abs() + 2.0 ** -16 * (x.double().abs() @ w.abs().T) + 2.0 ** -24
            for y in outs:
                assert torch.all((y[:M].double() - ref).abs() <= bound), (M, shape)
                assert torch.all(y[M:] == 7.0), (M, shape)


@pytest.mark.parametrize("N,K", [(272, 1280), (80, 2048), (32, 10240)])
def test_forced_lone_w2_is_the_tile_kernel(N, K):
    """A lone 2-bit linear forced to the tile kernel gives that kernel's result in a group, bit for bit, whether or not its prompts run
    as blocks of the decode kernel."""
    import torch
    import paper_2306_00978_amd as awq
    g = torch.Generator(device="cuda").manual_seed(N)
    packed = awq.awq_quantize_pack_w2((torch.randn((N, K), generator=g, device="cuda") * 0.02).half(), None)
    x = torch.randn((16, K), generator=g, device="cuda").half()
    pair = [torch.empty((16, N), dtype=torch.float16, device="cuda") for _ in range(2)]
    with tuning_build(AWQ_FEW=1):
        awq.prepare_linear_multi_w2([(x, *packed, y, N) for y in pair])()
        assert torch.equal(awq.awq_w2a16_linear(x, *packed, N), pair[0])
