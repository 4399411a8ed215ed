"""Grouped 2-bit calls at nine tokens and more that stay with the 2-bit decode kernel, small ones, lone linears of short rows and layers of rows of different lengths: as the tuning build runs them with the tile
kernel left out, bit for bit."""
import pytest

from tuning_build import tuning_build

pytestmark = pytest.mark.gpu


LAYER = [(2048, 2048), (512, 2048), (512, 2048), (2048, 2048), (7168, 2048), (7168, 2048), (2048, 7168)]


@pytest.mark.parametrize("M", [9, 12, 16])
@pytest.mark.parametrize("shapes", [[(1024, 1024), (128, 1024), (128, 1024)], [(2560, 1024), (2560, 1024)], [(1792, 1792), (224, 1792), (224, 1792)], [(9952, 1024)], [(7696, 1792)], LAYER])
def test_groups_by_the_decode_kernel(M, shapes):
    import torch
    import paper_2306_00978_amd as awq
    g = torch.Generator(device="cuda").manual_seed(M)
    packed = [awq.awq_quantize_pack_w2((torch.randn((N, K), generator=g, device="cuda") * 0.02).half(), None) for N, K in shapes]
    xs = [torch.randn((M, K), generator=g, device="cuda").half() for N, K in shapes]
    results = []
    for few in (None, 0):
        ys = [torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda") for N, K in shapes]
        with tuning_build(AWQ_FEW=few):
            awq.prepare_linear_multi_w2([(x, *p, y, N) for x, p, y, (N, K) in zip(xs, packed, ys, shapes)])()
        results.append(ys)
    assert all(torch.equal(a, b) for a, b in zip(*results))
