"""The split merge at the sizes where it can go wrong: fewer splits than
waves, one more than a batch of row loads (8, then 16 more, per wave), more
than 64 splits a wave (several rounds of lanes), and both sides of the rule
that gives a row one wave or four (1024 rows); most splits empty in the large
plans.  The output is the oracle's within the decode bar, equal to that of
another split plan within the rounding of fp32 sums of the plans' partials
(1e-5 of a row's largest value; about a hundred terms of 2^-24 each), and the
fused step's, bit for bit."""
import numpy as np
import pytest

import oracle
from gpu_harness import Pair, rel_err, say

pytestmark = pytest.mark.gpu


def _bits(rng, *shape):
    return oracle.f32_to_bf16(rng.standard_normal(shape).astype(np.float32))


@pytest.mark.parametrize("batch,H,G,d,bits", [(2, 1, 4, 128, 2), (3, 2, 1, 64, 4), (2, 1, 8, 128, 4), (130, 1, 8, 64, 2),
                                              (257, 1, 4, 128, 2)])
def test_split_counts(gpu, batch, H, G, d, bits):
    rng = np.random.default_rng(batch + d + bits)
    p = Pair(gpu, batch, H, G, d, bits, 4, 32, 8, 0.96, 0.92, cap=420, seed=1, oracle_ref=False)
    counts = rng.integers(200, 400, batch).astype(np.int32)
    p.append(_bits(rng, batch, 400, H, d), _bits(rng, batch, 400, H, d), counts)
    q = _bits(rng, batch, H * G, d)
    outs = []
    # pages per wave 2 at least: 8 pages a split until the device is full
    for n_splits in (1, 4, 9, 33, 40, 97, 105, 257, 300):
        top = 4 + 64 * 8 * n_splits
        say("merge batch %d heads %d G %d d %d bits %d: plan for %d tokens" % (batch, H, G, d, bits, top))
        outs.append(p.decode(q, max_seq_len=top))
        assert rel_err(outs[-1], outs[0]) <= 1e-5
    want = p.mirror.decode(q, p.tinv, p.sm_scale)
    assert rel_err(outs[0], want) <= 2e-3
    # a step that appends nothing: the same attention by the fused step
    k1 = _bits(rng, batch, H, d)
    for top in (500, 4 + 64 * 8 * 40):
        got, _, _ = p.step(k1, k1, np.zeros(batch, np.int32), q, max_seq_len=top)
        assert np.array_equal(got, p.decode(q, max_seq_len=top))
