"""Page runs dealt out by the lengths found: ragged batches whose longest
sequence takes most of the workgroups, sequences with no pages and none at
all, lengths far below max_seq_len, the largest batch that is dealt (64) and
the first that is not (65), odd and single heads.  The output is the oracle's within the decode
bar and equals that of a plan that runs in rounds, where nothing is dealt
out, within the rounding of the partials' fp32 sums (1e-5 of a row's largest
value, as for any two split plans), and a chunk of one token has its bits.
Decode steps over the same batches keep
the cache bit-exact."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_38121_amd as wk
from gpu_harness import HeldCache, Pair, rel_err, say, to_dev_bf16

pytestmark = pytest.mark.gpu


def _bits(rng, *shape):
    return oracle.f32_to_bf16(rng.standard_normal(shape).astype(np.float32))


CASES = [
    (5, 2, 4, 128, 2, [3000, 60, 200, 0, 700]),
    (3, 1, 8, 128, 4, [10, 2500, 5]),
    (2, 3, 1, 64, 4, [1900, 1900]),
    (1, 2, 2, 64, 2, [900]),
    (8, 2, 8, 128, 2, [100, 3100, 90, 80, 2900, 40, 500, 1]),
    (64, 1, 4, 64, 2, [1200] * 3 + [150] * 61),
    (65, 1, 4, 64, 2, [1200] * 3 + [150] * 62),
]


@pytest.mark.parametrize("batch,H,G,d,bits,lengths", CASES)
def test_ragged_runs(gpu, batch, H, G, d, bits, lengths):
    rng = np.random.default_rng(batch + d + bits)
    top = max(lengths)
    cap = 4 * top
    p = Pair(gpu, batch, H, G, d, bits, 4, 32, 8, 0.96, 0.92, cap=cap, seed=2, oracle_ref=False,
             page_order="random", pool_factor=1.25)
    p.append(_bits(rng, batch, top, H, d), _bits(rng, batch, top, H, d), lengths)
    rounds = 4 + 64 * 8 * 4000 // (batch * H)  # more splits than the device holds at once
    for it in range(3):
        q = _bits(rng, batch, H * G, d)
        ref = p.decode(q, max_seq_len=rounds)
        for m in (top + 8, cap):
            say("runs batch %d heads %d G %d d %d bits %d max_seq_len %d" % (batch, H, G, d, bits, m))
            out, e, _ = p.decode_check(q, max_seq_len=m)
            assert rel_err(out, ref) <= 1e-5
        # a chunk of one token is the decode; rows without one are zero
        nt = (rng.random(batch) < 0.7).astype(np.int32)
        nt[int(np.argmax(lengths))] = 1
        live = (nt > 0) & (p.gpu.seq_len.cpu().numpy() > 0)
        one = wk.wushkv_chunk_attention(p.gpu, to_dev_bf16(q[:, None], p.dev), p.tinv_dev,
                                        n_tok=torch.from_numpy(nt).to(p.dev), sm_scale=p.sm_scale,
                                        max_seq_len=top + 8).cpu().numpy()[:, 0]
        dec = p.decode(q, max_seq_len=top + 8)
        assert np.array_equal(one[live], dec[live]) and not one[~live].any()
        n = (rng.random(batch) < 0.7).astype(np.int32)
        p.step(_bits(rng, batch, H, d), _bits(rng, batch, H, d), n, q, max_seq_len=top + 8)
        p.check_cache()


@pytest.mark.parametrize("pages,lengths", [(32, [100, 8000, 90, 300, 60, 40, 500, 70]), (16, [100, 60000]), (8, [5000])])
def test_sequences_longer_than_max_seq_len(gpu, pages, lengths):
    """max_seq_len is the caller's statement; a replayed graph's sequences may
    outgrow it.  A sequence's pages past those the grid was sized for are then
    left out, and every other one is attended to once."""
    say("runs of %s sized for %d pages" % (lengths, pages))
    p = HeldCache(gpu, 1, 4, 64, 2, lengths)
    (S, end), q = p.counters(), p.queries()
    # (two pages a wave: the grid holds these pages and no more)
    out = p.decode(q, 4 + 64 * pages)
    assert p.splits(4 + 64 * pages) == pages // 8 + 1
    p.check(out, q, S, end, most=pages)
