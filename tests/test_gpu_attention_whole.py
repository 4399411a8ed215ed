"""Decode attention on short contexts: one launch for a head's whole context against the oracle, and the two launches beside it, at
the edges of a wave's batch of positions (4, 64, 256, 320) and with what lies behind the last row not a number."""
import numpy as np
import pytest

from tuning_build import tuning_build

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("whole", [None, 0, 1024])
@pytest.mark.parametrize("H,Hkv", [(1, 1), (4, 2), (24, 3)])
def test_short_contexts_against_the_oracle(H, Hkv, whole):
    import torch
    import oracle
    import paper_2306_00978_amd as awq
    g = np.random.default_rng(H)
    Lmax = 640
    q = g.standard_normal((H, 128)).astype(np.float16)
    k, v = (g.standard_normal((Hkv, 128)).astype(np.float16) for _ in range(2))
    kc, vc = (g.standard_normal((Hkv, Lmax, 128)).astype(np.float16) for _ in range(2))
    for pos in (0, 1, 3, 4, 5, 63, 64, 65, 255, 256, 257, 319, 320, 511, 513, 600):
        kp, vp = kc.copy(), vc.copy()
        kp[:, pos:], vp[:, pos:] = np.nan, np.nan
        kg, vg = torch.from_numpy(kp).cuda(), torch.from_numpy(vp).cuda()
        with tuning_build(AWQ_ATTENTION_WHOLE=whole):
            out = awq.awq_decode_attention(*(torch.from_numpy(t).cuda() for t in (q, k, v)), kg, vg, pos)
        ref, k_ref, v_ref = oracle.decode_attention(q, k, v, kc, vc, pos)
        # the bound of the other attention tests: 2e-3 of the largest value
        assert np.abs(out.cpu().numpy().astype(np.float64) - ref).max() <= 2e-3 * np.abs(vc[:, :pos + 1]).max(), pos
        assert np.array_equal(vg[:, pos].cpu().numpy().view(np.uint16), v.view(np.uint16))
        assert np.isnan(kg[:, pos + 1:].cpu().numpy()).all()


@pytest.mark.parametrize("pos", [300, 400])
def test_a_score_of_minus_infinity_has_no_weight(pos):
    """One launch and two: keys with an infinity against the query in the first rows of the lane groups, and in all rows."""
    import torch
    import paper_2306_00978_amd as awq
    q, k, v = (torch.ones((2, 128), dtype=torch.float16, device="cuda") for _ in range(3))
    for rows in ([0, 1, 2, 3, 64], list(range(pos))):
        kc = torch.zeros((2, 512, 128), dtype=torch.float16, device="cuda")
        vc = torch.ones((2, 512, 128), dtype=torch.float16, device="cuda")
        vc[:, rows] = 5.0
        kc[:, rows, 127] = -float("inf")             # the pair that this theta does not turn
        out = awq.awq_decode_attention(q, k, v, kc, vc, pos, rope_theta=1e30)
        assert torch.equal(out, torch.ones_like(out))
