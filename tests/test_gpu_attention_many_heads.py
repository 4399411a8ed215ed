"""Decode attention on short contexts with as many heads as the chip has CUs, and more: from 257 heads on, and beyond 200 positions where 16 kv heads
and more are shared, by the two launches that the tuning build takes when told to, bit for bit; and against the oracle."""
import numpy as np
import pytest

from tuning_build import tuning_build

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,Hkv,pos,two", [(257, 257, 100, True), (272, 17, 20, True), (320, 8, 250, True), (256, 32, 219, True), (256, 32, 60, False),
                                           (192, 16, 319, False), (256, 256, 319, False), (256, 8, 300, False)])
def test_many_heads_on_short_contexts(H, Hkv, pos, two):
    import torch
    import oracle
    import paper_2306_00978_amd as awq
    g = np.random.default_rng(H + pos)
    q = g.standard_normal((H, 128)).astype(np.float16)
    k, v = (g.standard_normal((Hkv, 128)).astype(np.float16) for _ in range(2))
    kc, vc = (g.standard_normal((Hkv, 320, 128)).astype(np.float16) for _ in range(2))
    outs = {}
    for whole in (None, 0, 320):
        with tuning_build(AWQ_ATTENTION_WHOLE=whole):
            outs[whole] = awq.awq_decode_attention(*(torch.from_numpy(t).cuda() for t in (q, k, v, kc, vc)), pos)
    assert torch.equal(outs[None], outs[0 if two else 320])
    assert not torch.equal(outs[0], outs[320])               # what tells the two apart
    ref = oracle.decode_attention(q, k, v, kc, vc, pos)[0]
    # the bound of the other attention tests: 2e-3 of the largest value
    assert np.abs(outs[None].cpu().numpy().astype(np.float64) - ref).max() <= 2e-3 * np.abs(vc[:, :pos + 1]).max()
