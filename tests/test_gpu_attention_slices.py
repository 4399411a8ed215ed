"""Decode attention in slices that end within a batch of a wave's positions (64 of a workgroup): slices of 80, 96, 144 and 160 positions, a
last slice of a few, against the oracle and with what lies behind the last row not a number."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,Hkv,pos", [(40, 40, 1000), (24, 24, 1500), (48, 24, 1000), (48, 24, 1501), (20, 20, 2047), (40, 20, 2050), (64, 64, 705), (32, 32, 1457),
                                       (24, 24, 1762)])
def test_slices_that_end_within_a_batch(H, Hkv, pos):
    import torch
    import oracle
    import paper_2306_00978_amd as awq
    g = np.random.default_rng(H + pos)
    q = g.standard_normal((H, 128)).astype(np.float16)
    k, v = (g.standard_normal((Hkv, 128)).astype(np.float16) for _ in range(2))
    kc, vc = (g.standard_normal((Hkv, pos + 70, 128)).astype(np.float16) for _ in range(2))
    ref = oracle.decode_attention(q, k, v, kc, vc, pos)[0]
    # the bound of the other attention tests: 2e-3 of the largest value
    bound = 2e-3 * np.abs(vc[:, :pos + 1]).max()
    kc[:, pos:], vc[:, pos:] = np.nan, np.nan
    out = awq.awq_decode_attention(*(torch.from_numpy(t).cuda() for t in (q, k, v, kc, vc)), pos)
    assert np.abs(out.cpu().numpy().astype(np.float64) - ref).max() <= bound
