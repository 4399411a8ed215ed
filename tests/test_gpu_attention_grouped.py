"""Decode attention with several query heads to a key/value head (the kernel that runs both products on
the matrix cores) against the oracle: positions around its blocks of 16, waves and slices without
positions, 3 to 20 query heads to a kv head (partly filled and several head tiles), each of its three splits of the
value dimensions."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = 2e-3          # of max|v|: fp16 rounding of the output (2^-11) and fp32 sums / exponentials


@pytest.mark.parametrize("H,Hkv,positions", [
    (12, 4, (0, 1, 31, 32, 33, 63, 130)),
    (64, 8, (0, 15, 127, 128, 300, 4000)),
    (40, 2, (5, 64, 700)),
    (48, 16, (97, 1500)),
    (256, 32, (40, 1030)),
    (96, 32, (2, 513)),
])
def test_grouped_attention_against_the_oracle(H, Hkv, positions):
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
