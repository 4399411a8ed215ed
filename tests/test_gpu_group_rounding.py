"""The batch kernel for several linears rounds its outputs to fp16 where the fp64 product does: what comes before that rounding is
fp32 throughout, in the matrix core as well."""
import pytest

from tuning_build import tuning_build

pytestmark = pytest.mark.gpu

SHAPES = [(2048, 512), (1024, 1280), (1040, 2048), (512, 5632)]
NAMES = {4: ("awq_quantize_pack", "awq_unpack", "prepare_linear_multi"), 3: ("awq_quantize_pack_w3", "awq_unpack_w3", "prepare_linear_multi_w3")}


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("M", [1, 2, 3, 5, 8, 11, 16])
def test_outputs_are_rounded_once(bits, M):
    import torch
    import paper_2306_00978_amd as awq
    pack, unpack, prepare = (getattr(awq, n) for n in NAMES[bits])
    g = torch.Generator(device="cuda").manual_seed(17 * M + bits)
    linears, refs = [], []
    for N, K in SHAPES:
        packed = pack((torch.randn((N, K), generator=g, device="cuda") * 0.02).half(), None)
        codes, scales, zeros = unpack(*packed, N, K)
        w = ((codes.double().view(N, K // 128, 128) - zeros.double()[..., None]) * scales.double()[..., None]).view(N, K)
        x = torch.randn((M, K), generator=g, device="cuda").half()
        linears.append((x, *packed, torch.empty((M, N), dtype=torch.float16, device="cuda"), N))
        refs.append(x.double() @ w.T)
    with tuning_build(AWQ_FEW=5):
        prepare(linears)()
    other = sum(int((l[4] != r.half()).sum()) for l, r in zip(linears, refs))
    # An error e before the rounding moves an output to its neighbour with a probability of 2 |e| / ulp, ulp 2^-11 to 2^-10 of the
    # output.  Some 40 fp32 roundings, 2^-25 on average, of sums up to four times the output are 7e-7 of it, or 0.2 % of the
    # outputs (measured: 0.04 to 0.08 %); products cut off 17 bits below the largest are 15 to 25 %.
    assert other <= 0.01 * sum(r.numel() for r in refs), other
