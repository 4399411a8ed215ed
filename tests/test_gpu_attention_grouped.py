"""Decode attention with several query heads to a key/value head (the kernel that runs both products on
the matrix cores) against the oracle: positions around its blocks of 16, waves and slices without
positions, 3 to 20 query heads to a kv head (partly filled and several head tiles), each of its three splits of the
value dimensions.  The library as it is takes few positions to the other kernel and picks the split; the tuning build runs
this one, with each split, at every size."""
import numpy as np
import pytest

from tuning_build import tuning_build

pytestmark = pytest.mark.gpu

TOL = 2e-3          # of max|v|: fp16 rounding of the output (2^-11) and fp32 sums / exponentials


@pytest.mark.parametrize("F", [None, 4, 2, 1])
@pytest.mark.parametrize("H,Hkv,positions", [
    (12, 4, (0, 1, 31, 32, 33, 63, 130)),
    (64, 8, (0, 15, 127, 128, 300, 4000)),
    (40, 2, (5, 64, 700)),
    (48, 16, (97, 1500)),
    (256, 32, (40, 1030)),
    (96, 32, (2, 513)),
])
def test_grouped_attention_against_the_oracle(H, Hkv, positions, F):
    import oracle
    import torch
    import paper_2306_00978_amd as awq
    for pos in positions:
        g = np.random.default_rng(1000 * H + pos)
        lmax = pos + 9
        q, k, v = (g.standard_normal((n, 128)).astype(np.float16) for n in (H, Hkv, Hkv))
        q[0] *= 30                                                       # one sharp head
        kc = np.full((Hkv, lmax, 128), np.nan, np.float16)               # rows past the token must not be read
        vc = kc.copy()
        kc[:, :pos] = g.standard_normal((Hkv, pos, 128))
        vc[:, :pos] = g.standard_normal((Hkv, pos, 128))
        ref, kc_ref, vc_ref = oracle.decode_attention(q, k, v, kc, vc, pos)
        kg, vg = torch.from_numpy(kc).cuda(), torch.from_numpy(vc).cuda()
        out = torch.full((H, 128), float("nan"), dtype=torch.float16, device="cuda")
        with tuning_build(AWQ_ATTENTION_F=F):
            awq.awq_decode_attention(*(torch.from_numpy(t).cuda() for t in (q, k, v)), kg, vg, pos, out=out)
        got = out.cpu().numpy().astype(np.float64)
        assert np.all(np.isfinite(got)), pos
        scale = np.abs(vc_ref[:, :pos + 1].astype(np.float64)).max()
        assert np.abs(got - ref.astype(np.float64)).max() <= TOL * scale, pos
        assert np.array_equal(vg.cpu().numpy().view(np.uint16), vc_ref.view(np.uint16))
        kn = kg.cpu().numpy()
        assert np.array_equal(np.delete(kn, pos, 1).view(np.uint16), np.delete(kc, pos, 1).view(np.uint16))
        a, b = kn[:, pos].astype(np.float64), kc_ref[:, pos].astype(np.float64)
        assert np.all(np.abs(a - b) <= np.abs(b) * 2.0 ** -10 + 1e-7)


# eight heads have a slice per 64 positions up to 64 of them: both sides of 16 slices, above which another kernel merges them, and
# the rows of its four waves
@pytest.mark.parametrize("slices", [1, 3, 4, 5, 8, 9, 16, 17, 61, 64])
@pytest.mark.parametrize("short", [0, 63])
def test_merge_of_every_number_of_slices(slices, short):
    import oracle
    import torch
    import paper_2306_00978_amd as awq
    H, pos = 8, 64 * slices - 1 - short
    assert awq.load().awq_decode_attention_workspace_bytes(H, 128, pos + 1) == H * slices * 130 * 4
    g = np.random.default_rng(100 * slices + short)
    q, k, v = (g.standard_normal((H, 128)).astype(np.float16) for _ in range(3))
    q[1] *= 30                                                           # one slice has nearly all the weight
    kc, vc = (g.standard_normal((H, pos + 1, 128)).astype(np.float16) for _ in range(2))
    ref = oracle.decode_attention(q, k, v, kc, vc, pos)[0].astype(np.float64)
    out = awq.awq_decode_attention(*(torch.from_numpy(t).cuda() for t in (q, k, v, kc, vc)), pos)
    assert np.abs(out.cpu().numpy().astype(np.float64) - ref).max() <= TOL * np.abs(vc.astype(np.float64)).max()


# a slice has whole blocks of 16 positions: the last ones have none, in both kernels, and their maximum is -Inf and their sum 0
@pytest.mark.parametrize("H,Hkv,pos,slices,filled", [(8, 8, 4096, 64, 52), (24, 24, 3999, 22, 21), (8, 1, 4096, 64, 52), (28, 4, 2000, 19, 18)])
def test_merge_of_slices_without_positions(H, Hkv, pos, slices, filled):
    import oracle
    import torch
    import paper_2306_00978_amd as awq
    need = awq.load().awq_decode_attention_workspace_bytes(H, 128, pos + 1)
    assert need == H * slices * 130 * 4
    chunk = (-(-(pos + 1) // slices) + 15) // 16 * 16
    assert -(-(pos + 1) // chunk) == filled < slices
    g = np.random.default_rng(H + pos)
    q, k, v = (g.standard_normal((n, 128)).astype(np.float16) for n in (H, Hkv, Hkv))
    kc, vc = (g.standard_normal((Hkv, pos + 1, 128)).astype(np.float16) for _ in range(2))
    ref = oracle.decode_attention(q, k, v, kc, vc, pos)[0].astype(np.float64)
    out = awq.awq_decode_attention(*(torch.from_numpy(t).cuda() for t in (q, k, v, kc, vc)), pos)
    assert np.abs(out.cpu().numpy().astype(np.float64) - ref).max() <= TOL * np.abs(vc.astype(np.float64)).max()


# the library's choice is F = 4, 2 and 1 workgroups to a slice of the positions (64, 128 and 256 items)
SPLITS = [(64, 8, 1000), (128, 32, 700), (384, 128, 700)]
MANY_SLICES = [(28, 4, 1100), (24, 3, 1200), (16, 2, 1400)]             # 18, 19 and 22 slices: the other merge


@pytest.mark.parametrize("H,Hkv,pos", SPLITS + MANY_SLICES)
@pytest.mark.parametrize("where", ["value of the last row", "keys", "key of the token", "key, positive", "key of the token, positive"])
def test_infinities_in_the_caches_have_the_weight_of_their_score(H, Hkv, pos, where):
    """An infinite value reaches its own output column only; a key whose score is -Inf has the weight 0, wherever it lies
    (alone, a whole block of 16 rows, the first row of a slice, the token itself); a score of +Inf gives NaN."""
    import torch
    import paper_2306_00978_amd as awq
    from oracle import rope_rotate
    g = np.random.default_rng(H + pos)
    lmax = pos + 3
    q, k, v = (g.standard_normal((n, 128)).astype(np.float16) for n in (H, Hkv, Hkv))
    q[:, 63] = 0.5 + np.abs(q[:, 63])                                    # the slowest pair: positive after the rotation
    q[:, 127] = 0.5 + np.abs(q[:, 127])
    q[1, 5], q[1, 63], q[1, 127] = 30000, 2.0 ** -22, 2.0 ** -24         # elements below the high halves of the head's largest
    kc, vc = np.full((2, Hkv, lmax, 128), np.nan, np.float16)
    kc[:, :pos], vc[:, :pos] = g.standard_normal((2, Hkv, pos, 128))
    kc[:, :, 5] = 0
    kc[:, :, 69] = 0
    k[:, 5] = k[:, 69] = 0
    if where == "value of the last row":
        vc[:, pos - 1, 7] = np.inf
        vc[:, pos - 1, 100] = -np.inf
    elif where == "keys":
        kc[:, 16:32, 63] = kc[:, 0, 63] = kc[:, 77, 63] = kc[:, pos - 1, 63] = -np.inf
    elif where == "key of the token":
        k[:, 63] = -np.inf
    elif where == "key, positive":
        kc[:, 3, 63] = np.inf
    else:
        k[:, 63] = np.inf
    qr, kr = rope_rotate(q.astype(np.float64), pos), rope_rotate(k.astype(np.float64), pos)
    assert (qr[:, 63] > 0).all() and (qr[:, 127] > 0).all()
    keys = np.concatenate([kc[:, :pos].astype(np.float64), kr[:, None]], 1)
    vals = np.concatenate([vc[:, :pos].astype(np.float64), v[:, None].astype(np.float64)], 1)
    G = H // Hkv
    with np.errstate(invalid="ignore"):
        score = np.einsum("gld,ghd->ghl", keys, qr.reshape(Hkv, G, 128)) / np.sqrt(128)
        weight = np.exp(score - score.max(-1, keepdims=True))
        weight /= weight.sum(-1, keepdims=True)
        want = np.einsum("ghl,gld->ghd", weight, np.where(np.isinf(vals), 0, vals))
        for g_, l, d in zip(*np.nonzero(np.isinf(vals))):
            want[g_, :, d] += weight[g_, :, l] * vals[g_, l, d]
    want = want.reshape(H, 128)
    out = torch.full((H, 128), 7.0, dtype=torch.float16, device="cuda")
    awq.awq_decode_attention(*(torch.from_numpy(t).cuda() for t in (q, k, v)), torch.from_numpy(kc).cuda(),
                             torch.from_numpy(vc).cuda(), pos, out=out)
    got = out.cpu().numpy().astype(np.float64)
    fine = np.isfinite(want)
    assert fine.all() == (where in ("keys", "key of the token"))
    assert np.array_equal(got[~fine], want[~fine], equal_nan=True)
    assert np.abs(got[fine] - want[fine]).max(initial=0) <= TOL * np.abs(vals[np.isfinite(vals)]).max()


@pytest.mark.parametrize("F", [None, 4, 2, 1])
@pytest.mark.parametrize("H,Hkv,pos", [(32, 4, 20), (96, 24, 20), (384, 64, 40)])
def test_small_elements_beside_a_large_one_keep_their_bits(H, Hkv, pos, F):
    """A head whose largest elements meet zeros in every key: the scores are those of the small ones, 2^-30 of the
    largest and multiplied by keys of 2^15, and need their fp32 bits."""
    import oracle
    import torch
    import paper_2306_00978_amd as awq
    g = np.random.default_rng(H)
    q = (g.standard_normal((H, 128)) * 6e-5).astype(np.float16)
    q[:, 63], q[:, 127] = 60000, -20000
    k, *rows = (np.where(g.random((Hkv, 128)) < 0.5, -32768, 32768).astype(np.float16) for _ in range(pos + 1))
    kc, vc = np.zeros((2, Hkv, pos + 5, 128), np.float16)
    kc[:, :pos] = np.stack(rows, 1)
    kc[:, :, [63, 127]] = k[:, [63, 127]] = 0
    vc[:, :pos] = g.standard_normal((Hkv, pos, 128))
    v = g.standard_normal((Hkv, 128)).astype(np.float16)
    ref, _, _ = oracle.decode_attention(q, k, v, kc, vc, pos)
    with tuning_build(AWQ_ATTENTION_F=F):
        out = awq.awq_decode_attention(*(torch.from_numpy(t).cuda() for t in (q, k, v, kc, vc)), pos)
    # the rounding of the output and of the reference, half a unit of 2^-10 each, and fp32 sums of 128 products of about 0.2
    # (scores off by 1e-5); with two halves to a query the scores were off by 2e-2 and the outputs by 6e-3
    scale = np.abs(vc.astype(np.float64)).max()
    assert np.abs(out.cpu().numpy().astype(np.float64) - ref.astype(np.float64)).max() <= 1.1e-3 * scale
