"""The exact selection behind Eq. (7)'s clip range (sorting and merging
networks over 16-bit magnitudes) at every list length it is built for, K =
d - floor(kappa (d - 1)) = 1 .. 16, and on both sides of the last one, where
ranks are counted instead: rows of one sign, of zeros of both signs, of ties,
of denormals, with magnitudes above 2^121 and infinities, against the oracle's
sort, bit for bit (the codes are integers: no tolerance).  A large append
(lane-pair tiles) and appends of eight tokens (16 lanes a group) must leave
the same bytes, NaNs included."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_38121_amd as wk
from gpu_harness import Pair, eye_bits, say, to_dev_bf16

pytestmark = pytest.mark.gpu


def _kappa(d, K):
    """A quantile whose lower order statistic is the K-th largest."""
    return 1.0 if K == 1 else (d - K + 0.37) / (d - 1)


def _rows(rng, n, d, huge, nan=False):
    """bf16 patterns [n][d]: every special row in turn, random rows between."""
    x = rng.standard_normal((n, d)).astype(np.float32)
    x[:, ::7] *= 9.0
    for i in range(0, n, 2):
        s = (i // 2) % 11
        if s == 0: x[i] = 0.0
        elif s == 1: x[i] = -0.0
        elif s == 2: x[i] = 1.5
        elif s == 3: x[i] = -np.abs(x[i])
        elif s == 4: x[i] = np.abs(x[i])
        elif s == 5: x[i] = np.where(x[i] > 0.5, 0.0, np.where(x[i] < -1.5, x[i], -0.0))
        elif s == 6 and huge: x[i, rng.integers(d)] = 1.5e38
        elif s == 7 and huge: x[i, rng.choice(d, 2, replace=False)] = [np.inf, -np.inf]
        elif s == 8: x[i] = rng.choice([-2.0, -1.0, 1.0, 2.0], d)
        elif s == 9: x[i] *= 1e-39
        elif s == 10 and nan: x[i, rng.choice(d, 3, replace=False)] = [np.nan, -np.nan, np.nan]
    return oracle.f32_to_bf16(x)


@pytest.mark.parametrize("d,bits", [(128, 2), (128, 4), (64, 2), (64, 3)])
def test_every_list_length_against_the_oracle(gpu, d, bits):
    for Kk, Kv in [(K, 18 - K) for K in range(1, 18)]:
        rng = np.random.default_rng(100 * d + 10 * bits + Kk)
        say("select d=%d bits=%d K keys %d values %d" % (d, bits, Kk, Kv))
        p = Pair(gpu, 1, 1, 1, d, bits, 4, 8, 8, _kappa(d, Kk), _kappa(d, Kv), cap=400, seed=Kk, oracle_ref=False)
        assert d - int(np.floor(np.float32(_kappa(d, Kv)).astype(np.float64) * (d - 1))) == Kv
        k = oracle.f32_to_bf16(rng.standard_normal((1, 200, 1, d)).astype(np.float32))
        v = _rows(rng, 200, d, huge=Kv > 4)[None, :, None]
        p.append(k, v, [200])
        p.check_cache()
        # a short flush: 16 lanes a group
        k, v = k[:, :8], _rows(rng, 8 * 11, d, huge=Kv > 4)[None, Kk % 8::11, None]
        p.append(k, np.ascontiguousarray(v[:, :8]), [8])
        p.check_cache()


@pytest.mark.parametrize("d,bits", [(128, 2), (64, 4)])
def test_large_and_short_appends_agree_on_any_rows(gpu, d, bits):
    for K in (4, 7, 12):
        rng = np.random.default_rng(7 * d + bits + K)
        say("select paths d=%d bits=%d K=%d" % (d, bits, K))
        n, eye = 176, to_dev_bf16(eye_bits(1, d), gpu)
        k = to_dev_bf16(_rows(rng, n, d, True, True)[None, :, None], gpu)
        v = to_dev_bf16(_rows(rng, n, d, True, True)[None, :, None], gpu)
        # (the transform spreads a NaN or an infinity over its row)
        pages = []
        for step in (n, 8):
            c = wk.WushKVCache(1, 1, d, bits, 4, 8, 8, _kappa(d, K), _kappa(d, K), max_seq_len=400, device=gpu)
            for at in range(0, n, step):
                wk.wushkv_append(c, k[:, at:at + step].contiguous(), v[:, at:at + step].contiguous(),
                                 torch.tensor([step], dtype=torch.int32, device=gpu), eye)
            torch.cuda.synchronize()
            pages.append(c.pages.cpu().numpy())
        assert np.array_equal(pages[0], pages[1])
