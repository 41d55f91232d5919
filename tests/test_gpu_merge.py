"""The split merge at the sizes where it can go wrong.

Plans: fewer splits than waves, one more than a batch of row loads (8, then 16
more, per wave), more than 64 splits a wave (several rounds of lanes), and
both sides of the rule that gives a row one wave or four (1024 rows).  The
output is the oracle's within the decode bar, equal to that of another split
plan within the rounding of fp32 sums of the plans' partials (1e-5 of a row's
largest value; about a hundred terms of 2^-24 each), and the fused step's, bit
for bit.

Those sequences are short: most splits of the large plans are empty.  The
tests of live splits hold sequences so long that every split, and so every row
of every batch of a wave, counts, up to and past the 64 splits of a pass:
decode, fused step and chunk, one wave a row and four, own runs and dealt out
ones.  They compare every head with Eq. (2) in fp64 over what the cache holds
(its reconstructed pages and bf16 windows), to the decode bar."""
import numpy as np
import pytest

import oracle
import paper_2609_38121_amd as wk
from gpu_harness import HeldCache, Pair, rel_err, say

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


@pytest.mark.parametrize("H,G,d,bits", [(1, 4, 128, 2), (2, 4, 128, 2), (1, 8, 64, 4)])
def test_long_sequence_of_few_heads(gpu, H, G, d, bits):
    say("merge 131072 tokens heads %d G %d d %d bits %d" % (H, G, d, bits))
    p = HeldCache(gpu, H, G, d, bits, [131072])
    p.check_decode_and_step()


def test_live_splits_around_a_pass(gpu):
    """Four waves a row: the counts around 56 and 64 splits a wave, each split
    holding four whole pages."""
    p = HeldCache(gpu, 1, 8, 64, 2, [100], cap=140000)
    for splits in (56, 221, 224, 225, 233, 240, 256, 257, 258, 300, 513):
        say("merge %d live splits" % splits)
        pages = 4 * (splits - 1)  # and the window's
        p.grow([4 + 64 * pages + 20])
        end = int(p.cache.quant_end[0])
        assert -(-(end - 4) // 64) == pages and p.splits(4 + 2 * 64 * pages) == splits
        p.check_decode_and_step(4 + 2 * 64 * pages)


def test_live_splits_dealt_out(gpu):
    """The longest sequence's runs take the other sequences' workgroups."""
    lengths = [300, 65536, 60, 200, 1, 420, 90, 330]
    say("merge dealt out %s" % lengths)
    p = HeldCache(gpu, 1, 4, 128, 2, lengths)
    assert p.splits(65600) < 225  # more only where they are dealt out
    p.check_decode_and_step()


def test_live_splits_one_wave_a_row(gpu):
    lengths = [150 + b for b in range(127)] + [262144]
    say("merge one wave a row, 262144 tokens")
    p = HeldCache(gpu, 1, 8, 64, 2, lengths)
    assert p.splits(p.cache.max_seq_len) > 64
    p.check_decode_and_step(rows=[0, 50, 126, 127])


def test_live_splits_of_a_chunk(gpu):
    say("merge chunk of 16 at 32768 tokens")
    p = HeldCache(gpu, 1, 4, 64, 2, [32768])
    (S, end), q = p.counters(), p.queries(16)
    out = wk.wushkv_chunk_attention(p.cache, q, p.tinv, sm_scale=p.sm_scale)
    for t in range(16):
        p.check(out[:, t], q[:, t].contiguous(), S - 15 + t, end)
