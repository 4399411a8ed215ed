"""The K-split tile kernel (more than 16 tokens; 4- and 3-bit group 128, 2-bit group 64) against the oracle at the
sizes where it can go wrong: token tiles with a remainder (the last one moved back over its
neighbour), several token tiles and ragged weight tiles per workgroup, fewer runs of K than waves, waves with one
run more than others; then every pair of tile counts that is built, through the tuning build, which can force it; the
prefill kernel at the ragged shapes that this one has taken over; and where the line between the kernels lies."""
import numpy as np
import pytest

from tuning_build import tuning_build

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


PLANS = [(mt, nt) for mt in (1, 2, 3, 4, 5, 6, 8) for nt in (1, 2, 3, 4) if (mt, nt) != (8, 4)]


@pytest.mark.parametrize("bits", [4, 3, 2])
@pytest.mark.parametrize("N,K", [(208, 2304), (16, 256), (48, 768)])
def test_every_built_shape_of_a_workgroup(bits, N, K):
    """Feature tiles that the count does not divide, waves with one run of K more than others and without any; a token
    tile that is full, one that is moved back, and more than one workgroup of them."""
    import oracle
    import torch
    import paper_2306_00978_amd as awq
    linear = {4: awq.awq_w4a16_linear, 3: awq.awq_w3a16_linear, 2: awq.awq_w2a16_linear}[bits]
    x, Wdq, packed = case(bits, N, K, 16 * 8 * 2 + 5, N + K + bits)
    ref = oracle.matmul(x, Wdq)
    for mt, nt in PLANS:
        for M in sorted({17, 16 * max(mt, 2), 16 * max(mt, 2) - 3, 32 * mt + 5}):
            buf = torch.full((M * N + 16,), float("nan"), dtype=torch.float16, device="cuda")
            y, xg = buf[:M * N].view(M, N), torch.from_numpy(x[:M]).cuda()
            with tuning_build(AWQ_TILE_PLAN=10 * mt + nt):
                linear(xg, *packed, N, out=y)
            got = y.cpu().numpy().copy()
            assert bool(torch.isnan(buf[M * N:]).all())                 # nothing written past the end
            assert np.all(np.isfinite(got.astype(np.float32))), (mt, nt, M, "unwritten output")
            err = oracle.norm_error(got, ref[:M], x[:M], Wdq)
            assert err.max() <= TOL, (mt, nt, M, err.max())
            with tuning_build(AWQ_TILE_PLAN=10 * mt + nt):
                linear(xg, *packed, N, out=y)
            assert np.array_equal(got.view(np.uint16), y.cpu().numpy().view(np.uint16)), (mt, nt, M)


def test_neighbouring_workgroups_start_a_run_apart():
    """The order in which a wave adds its runs, from where it starts: that of the workgroup before, and one run further on.
    Three runs of the first wave add 2^25, 1 and -2^25 to every output: 1 where it starts at the third, else 0."""
    import oracle
    import torch
    import paper_2306_00978_amd as awq
    tiles, K, M = 13, 24 * 128, 17                                       # 16 x 16 tiles of y: 26 workgroups
    N = 16 * tiles
    codes, zeros = np.zeros((N, K), np.uint8), np.zeros((N, K // 128), np.uint8)
    scales, x = np.ones((N, K // 128), np.float16), np.zeros((M, K), np.float16)
    for run, value in ((0, 32768), (8, 1), (16, -32768)):
        x[:, run * 128] = value
        codes[:, run * 128] = 1 if value == 1 else 8
        scales[:, run] = 1 if value == 1 else 128
    packed = [torch.from_numpy(a).cuda() for a in oracle.pack(codes, scales, zeros)]
    packed[1] = packed[1].view(torch.float16)
    with tuning_build(AWQ_TILE_PLAN=11):
        y = awq.awq_w4a16_linear(torch.from_numpy(x).cuda(), *packed, N, workspace=False).cpu().numpy()
    unit = np.arange(N)[None, :] // 16 + tiles * (np.arange(M)[:, None] // 16)
    assert np.array_equal(y, (unit % 3 == 2).astype(np.float16))


@pytest.mark.parametrize("plan", [0] + [10 * mt + nt for mt, nt in PLANS])
def test_loss_form_of_every_built_shape_and_of_the_prefill_kernel(plan):
    """The scale search against the same arithmetic in plain torch (fp64 products of the fp16 operands); 0: the prefill
    kernel's loss form, at a ragged shape that it does not get otherwise."""
    import torch
    import paper_2306_00978_amd as awq
    T, N, K, alphas = 165, 272, 1280, [0.0, 0.4, 0.7]
    g = torch.Generator(device="cuda").manual_seed(9)
    W = (torch.randn((N, K), generator=g, device="cuda") * 0.02).half()
    gain = torch.ones(K, device="cuda")
    gain[torch.randperm(K, generator=g, device="cuda")[:K // 100]] = 20.0
    X = (torch.randn((T, K), generator=g, device="cuda") * gain).half()
    with tuning_build(AWQ_TILE_PLAN=plan):
        best, losses, _ = awq.awq_search_scale(W, X, alphas)
    y = X.double() @ W.double().T
    for a, got in zip(alphas, losses.cpu().numpy()):
        s = awq.awq_act_scale(X, a)
        codes, scales, zeros = awq.awq_unpack(*awq.awq_quantize_pack(W, s), N, K)
        q = (codes.double().view(N, K // 128, 128) - zeros.double()[..., None]) * scales.double()[..., None]
        ref = float((awq.awq_apply_inv_scale(X, s).double() @ q.view(N, K).T - y).square().sum())
        # fp16 rounding of both outputs and of the dequantized weights: 1e-4 of the loss, and a cross term of
        # 2e-2 / sqrt(outputs) standard deviation
        assert abs(got / ref - 1) <= 2e-4 + 0.06 / np.sqrt(T * N), (a, got, ref)
    assert int(best) == int(losses.argmin())


@pytest.mark.parametrize("N,K,M", [(176, 1408, 17), (176, 1408, 300), (272, 256, 129), (1040, 512, 100), (2064, 1152, 257)])
def test_prefill_kernel_at_shapes_the_tile_kernel_took_over(N, K, M):
    """Token and feature tiles with a remainder, plain and with K in ranges (where the workspace call cuts it), 4 bits, and
    3 bits through the re-packed codes, whose workspace is then seen to be used."""
    import oracle
    import torch
    import paper_2306_00978_amd as awq
    for bits in (4, 3):
        x, Wdq, packed = case(bits, N, K, M, N + K + M)
        ref, xg = oracle.matmul(x, Wdq), torch.from_numpy(x).cuda()
        need = awq.awq_linear_workspace_bytes(M, N, K)
        codes = (N * K // 2 + 255) // 256 * 256 if bits == 3 else 0
        for ranges in (False, True) if need else (False,):
            size = codes + (need if ranges else 0)
            ws = torch.full((max(size, 16),), 0xA5, dtype=torch.uint8, device="cuda")
            buf = torch.full((M * N + 16,), float("nan"), dtype=torch.float16, device="cuda")
            y = buf[:M * N].view(M, N)
            with tuning_build(AWQ_TILE_PLAN=0):
                if bits == 4:
                    awq.awq_w4a16_linear(xg, *packed, N, out=y, workspace=ws if ranges else False)
                else:
                    st = awq.load().awq_w3a16_linear_prefill(
                        xg.data_ptr(), *(t.data_ptr() for t in packed), y.data_ptr(), M, N, K, 128, ws.data_ptr(),
                        size if ranges else N * K // 2, awq._stream())
                    assert st == 0
            got = y.cpu().numpy()
            assert bool(torch.isnan(buf[M * N:]).all()) and np.all(np.isfinite(got.astype(np.float32)))
            if bits == 3 or ranges:
                assert not bool((ws[:16] == 0xA5).all())
            if ranges:
                assert not bool((ws[size - 16:] == 0xA5).all())
            err = oracle.norm_error(got, ref, x, Wdq)
            assert err.max() <= TOL, (bits, ranges, err.max())


@pytest.mark.parametrize("bits,N,K,M,used", [
    (4, 11008, 4096, 128, False),                    # few tokens: the tile kernel, whatever the workspace
    (4, 28672, 8192, 128, True),                     # two rounds of its workgroups: K over ranges (69 us against 90)
    (4, 4096, 11008, 448, True),                     # us, tile kernel and ranges: 57.3, 50.5
    (3, 4096, 4096, 300, False),
    (3, 4096, 4096, 2048, True),                     # the prefill kernel, on re-packed codes
    (3, 8192, 28672, 512, False),                    # very long K: 297, re-packed 320
])
def test_line_between_the_tile_and_the_prefill_kernel(bits, N, K, M, used):
    """What the kernel that does not run would have left in the workspace tells the two apart."""
    import oracle
    import torch
    import paper_2306_00978_amd as awq
    g = torch.Generator(device="cuda").manual_seed(N + K + M)
    W = (torch.randn((N, K), generator=g, device="cuda") * 0.02).half()
    x = torch.randn((M, K), generator=g, device="cuda").half()
    packed = {4: awq.awq_quantize_pack, 3: awq.awq_quantize_pack_w3}[bits](W, torch.ones(K, device="cuda"))
    size = awq.awq_linear_workspace_bytes(M, N, K) if bits == 4 else N * K // 2
    ws = torch.full((size,), 0xA5, dtype=torch.uint8, device="cuda")
    if bits == 4:
        y = awq.awq_w4a16_linear(x, *packed, N, workspace=ws)
    else:
        y = torch.empty((M, N), dtype=torch.float16, device="cuda")
        assert awq.load().awq_w3a16_linear_prefill(x.data_ptr(), *(t.data_ptr() for t in packed), y.data_ptr(), M, N, K,
                                                   128, ws.data_ptr(), size, awq._stream()) == 0
    assert bool((ws == 0xA5).all()) != used
    codes, scales, zeros = (awq.awq_unpack if bits == 4 else awq.awq_unpack_w3)(*packed, N, K)
    rows = np.linspace(0, M - 1, 3).astype(int)
    cols = slice(0, N, max(1, N // 256))
    Wdq = oracle.dequant(*(t[cols].cpu().numpy() for t in (codes, scales, zeros)))
    xr = x[rows].cpu().numpy()
    err = oracle.norm_error(np.ascontiguousarray(y[rows][:, cols].cpu().numpy()), oracle.matmul(xr, Wdq), xr, Wdq)
    assert err.max() <= TOL, err.max()


@pytest.mark.parametrize("K", [128, 256, 384, 640])
@pytest.mark.parametrize("N", [16, 48, 80, 272])
def test_prefill_kernel_at_its_shortest_k(N, K):
    """One group of 128 columns (less than the loads ahead of the first product), two, three (the ring goes round once) and five;
    feature tiles of a wave with one, three and, in the second wave, one of four."""
    import oracle
    import torch
    import paper_2306_00978_amd as awq
    M = 145
    x, Wdq, packed = case(4, N, K, M, N + K)
    buf = torch.full((M * N + 16,), float("nan"), dtype=torch.float16, device="cuda")
    y = buf[:M * N].view(M, N)
    with tuning_build(AWQ_TILE_PLAN=0):
        awq.awq_w4a16_linear(torch.from_numpy(x).cuda(), *packed, N, out=y, workspace=False)
    got = y.cpu().numpy()
    assert bool(torch.isnan(buf[M * N:]).all()) and np.all(np.isfinite(got.astype(np.float32)))
    err = oracle.norm_error(got, oracle.matmul(x, Wdq), x, Wdq)
    assert err.max() <= TOL, err.max()


@pytest.mark.parametrize("bits,N,K,M,used", [
    (4, 4096, 4096, 400, False),                     # the estimates side by side (us, tile kernel and ranges: 24.7, 29.2)
    (4, 4096, 4096, 1000, True),                     # 51.2, 42.7
    (4, 4096, 11008, 129, False),                    # one rule for every token count above 128: 25.5, 31.6
    (4, 4096, 11008, 200, False),                    # long K: 31.4, 34.2
    (4, 4096, 11008, 256, False),                    # 31.6, 36.5
    (4, 4096, 11008, 500, True),                     # 57.3, 50.5 at 448 tokens
    (4, 4096, 14336, 300, False),                    # 46.6, 49.4
    (4, 1024, 28672, 256, False),                    # 33.2, 44.0
    (4, 1024, 14336, 500, False),                    # 28.2, 30.5
    (3, 4096, 4096, 160, False),                     # 12.9, re-packed 50.6
    (3, 28672, 256, 145, True),                      # many features, short K, just above the token counts without a look: 20.8, 16.5
])
def test_line_where_both_kernels_have_estimates(bits, N, K, M, used):
    test_line_between_the_tile_and_the_prefill_kernel(bits, N, K, M, used)


@pytest.mark.parametrize("N,K,M,tile", [
    (28672, 512, 128, True),                         # up to here without a look
    (28672, 512, 129, False),                        # us, tile kernel and K whole: 21.1, 13.9
    (57344, 512, 160, False),                        # 36.1, 24.9
    (4096, 4096, 160, True),                         # 13.9, 44
    (11008, 4096, 161, True),
    (4096, 14336, 960, True),                        # long K: 128, 144
    (5120, 13824, 700, True),                        # 121, 135
])
def test_line_without_a_workspace(N, K, M, tile):
    """Nothing but the bits of the result tells which kernel ran: the same call with the prefill kernel forced."""
    import torch
    import paper_2306_00978_amd as awq
    g = torch.Generator(device="cuda").manual_seed(N + K + M)
    W = (torch.randn((N, K), generator=g, device="cuda") * 0.02).half()
    x = torch.randn((M, K), generator=g, device="cuda").half()
    packed = awq.awq_quantize_pack(W, torch.ones(K, device="cuda"))
    y = awq.awq_w4a16_linear(x, *packed, N, workspace=False)
    with tuning_build(AWQ_TILE_PLAN=0):
        prefill = awq.awq_w4a16_linear(x, *packed, N, workspace=False)
    assert torch.equal(y, prefill) != tile


@pytest.mark.parametrize("N,K,M,shape,slower", [(1024, 28672, 700, 34, 43), (1536, 24576, 448, 34, 43), (512, 14336, 1300, 34, 43)])
def test_shape_of_a_workgroup_where_rows_are_long(N, K, M, shape, slower):
    """Where the token tiles of an XCD are more than its L2, workgroups of few tokens (10 * mt + nt): 67, 50 and 35 us; the slower
    shape takes 81, 58 and 43.  They show in the bits of the result, as a workgroup's waves start elsewhere."""
    import torch
    import paper_2306_00978_amd as awq
    g = torch.Generator(device="cuda").manual_seed(N + K + M)
    W = (torch.randn((N, K), generator=g, device="cuda") * 0.02).half()
    x = torch.randn((M, K), generator=g, device="cuda").half()
    packed = awq.awq_quantize_pack(W, torch.ones(K, device="cuda"))
    y = awq.awq_w4a16_linear(x, *packed, N, workspace=False)
    for plan in (shape, slower):
        with tuning_build(AWQ_TILE_PLAN=plan):
            assert torch.equal(y, awq.awq_w4a16_linear(x, *packed, N, workspace=False)) == (plan == shape)
