"""Whole histories of more tokens than two windows of block ids hold (a wave asks for 64 ids at a time: 4096 tokens of its
workgroup), and scores of -inf where whole histories are read.  Requests alias blocks freely past their first one, which keeps
the caches small and the batch one that shares nothing."""
import numpy as np
import pytest

import workloads as W
from gpu_harness import assert_close, run_hip, values
from oracle.attention import decode_attention

pytestmark = pytest.mark.gpu


def _aliased(Hq, Hkv, d, lens, seed, nblocks=1500):
    rng = np.random.default_rng(seed)
    B = len(lens)
    width = max(-(-n // 16) for n in lens) + 2
    bt = rng.integers(B, nblocks, size=(B, width)).astype(np.int32)
    bt[:, 0] = rng.permutation(B)
    draw = lambda *shape: W.f32_to_bf16_bits(rng.standard_normal(size=shape, dtype=np.float32))
    return draw(B, Hq, d), draw(nblocks, Hkv, 16, d), draw(nblocks, Hkv, 16, d), bt, np.array(lens, dtype=np.int32)


def _whole(info, B, Hkv):
    return info["variant"] == 1 and info["items"] == B * Hkv and info["partial_rows"] == 0 and info["overflow"] == 0


@pytest.mark.parametrize("Hq,Hkv,d,longest", [(8, 8, 64, [8191, 8192, 8193, 8321]), (24, 8, 128, [8200, 12289, 12500])])
def test_more_than_two_windows_of_ids(Hq, Hkv, d, longest):
    lens = [2900 + 37 * j % 500 for j in range(140 - len(longest))] + longest
    q, k, v, bt, L = _aliased(Hq, Hkv, d, lens, d)
    out, info = run_hip(q, k, v, bt, L, Hq, Hkv, d, "bf16", fused_max=-1)
    assert _whole(info, len(lens), Hkv)
    rows = [0, 70] + list(range(140 - len(longest), 140))
    want = decode_attention(values(q), values(k), values(v), bt, L, requests=rows)
    assert_close(out, want, "bf16", rows=rows, what=f"{Hq}/{Hkv}/{d} {longest}")


@pytest.mark.parametrize("Hq,Hkv,d", [(8, 8, 64), (24, 8, 128)])
def test_scores_of_minus_infinity(Hq, Hkv, d):
    """All of a wave's tiles, its first tile, everything but one token, and a history that scores nothing else."""
    B, G = 140, Hq // Hkv
    cases = [(1700, [t for t in range(1700) if t // 32 % 4 == 1]), (1700, range(32)), (1025, range(1024)), (1500, [t for t in range(1500) if t != 700]),
             (900, range(900))]
    lens = [n for n, _ in cases] + [1300 + 11 * j % 400 for j in range(B - len(cases))]
    q, k, v, bt, L = _aliased(Hq, Hkv, d, lens, d + 1)
    at = len(k)
    k, v = (np.concatenate([x] + [x[:120]] * len(cases)) for x in (k, v))
    for i, (n, _) in enumerate(cases):                 # blocks of their own
        nb = -(-n // 16)
        bt[i, 1:nb] = at + 120 * i + np.arange(nb - 1)
    finite = values(k).astype(np.float32).copy()
    for i, (n, tokens) in enumerate(cases):
        q[i, :G, 0] = W.f32_to_bf16_bits(np.ones(1, np.float32))[0]
        for t in tokens:
            k[bt[i, t // 16], 0, t % 16, 0] = 0xFF80
            finite[bt[i, t // 16], 0, t % 16, 0] = -1e30
    out, info = run_hip(q, k, v, bt, L, Hq, Hkv, d, "bf16", fused_max=-1)
    assert _whole(info, B, Hkv)
    none = len(cases) - 1
    assert np.isnan(out[none, :G]).all() and np.isfinite(out[none, G:]).all()
    rows = [i for i in range(len(cases) + 2) if i != none]
    want = decode_attention(values(q), finite, values(v), bt, L, requests=rows)
    assert_close(out, want, "bf16", rows=rows, what=f"{Hq}/{Hkv}/{d}")
