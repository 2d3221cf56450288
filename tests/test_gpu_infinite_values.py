"""Infinities and NaN in V: an output element is infinite where an infinity meets a positive weight, NaN where both infinities
or a NaN do, and what it was otherwise - whichever kernel reads the history, and wherever in it (first and later tiles, the
last one, waves and pieces of their own) the value lies.  The weights that meet them are well above zero."""
import numpy as np
import pytest

import workloads as W
from gpu_harness import assert_close, run_hip, values
from oracle.attention import decode_attention
from test_gpu_direct import _batch

pytestmark = pytest.mark.gpu

SHAPES = [("f32", 8, 2, 64), ("f32", 5, 1, 128), ("bf16", 14, 2, 128), ("bf16", 16, 1, 64), ("bf16", 4, 2, 256)]


def _put(v, bt, i, L, dtype):
    """Into request i's V, KV head 0: infinities of either sign, both in one dim, and a NaN; at dims of their own."""
    d = v.shape[3]
    bits = {"+": 0x7F80, "-": 0xFF80, "n": 0x7FC0}
    tokens = [0, L // 3, L // 2, L - 1]
    where = [(tokens[0], 1, "+"), (tokens[1], 17, "-"), (tokens[2], d // 2 + 3, "+"), (tokens[3], d - 1, "-"),
             (tokens[1], 5, "+"), (tokens[3], 5, "-"), (tokens[2], d - 8, "n"), (tokens[0], 33 % d, "+"), (tokens[3], 33 % d, "+")]
    for t, x, what in where:
        v[bt[i, t // 16], 0, t % 16, x] = bits[what] if dtype == "bf16" else np.float32({"+": np.inf, "-": -np.inf, "n": np.nan}[what])


def _check(out, want, dtype, rows, what):
    got, want = out[rows], want[rows]
    assert np.isinf(want).any() and np.isnan(want).any(), what
    assert np.array_equal(np.isnan(got), np.isnan(want)), what
    assert np.array_equal(np.where(np.isinf(want), want, 0), np.where(np.isinf(got), got, 0)), what
    fine = np.isfinite(want)
    assert_close(np.where(fine, got, 0), np.where(fine, want, 0), dtype, what=what)


@pytest.mark.parametrize("dtype,Hq,Hkv,d", SHAPES)
@pytest.mark.parametrize("lens", [[33, 300, 40], [1601, 900], [16], [4097]])
@pytest.mark.parametrize("planned", [False, True])
def test_small_batches(dtype, Hq, Hkv, d, lens, planned):
    q, k, v, bt, L = _batch(dtype, Hq, Hkv, d, lens, 31)
    for i in (0, len(lens) - 1):
        _put(v, bt, i, lens[i], dtype)
    out, info = run_hip(q, k, v, bt, L, Hq, Hkv, d, dtype, fused_max=-1 if planned else bt.shape[1])
    assert (info["variant"] != 2) == planned
    with np.errstate(invalid="ignore"):
        want = decode_attention(values(q), values(k), values(v), bt, L)
    _check(out, want, dtype, range(len(lens)), f"{dtype} {Hq}/{Hkv}/{d} {lens} planned {planned}")


@pytest.mark.parametrize("Hq,Hkv,d,B", [(8, 8, 64, 140), (14, 2, 128, 600)])
def test_whole_histories(Hq, Hkv, d, B):
    rng = np.random.default_rng(B)
    lens = rng.integers(500, 1800, size=B).tolist()
    q, k, v, bt, L = _batch("bf16", Hq, Hkv, d, lens, 32)
    rows = [0, 7, B // 2, B - 1]
    for i in rows[1:]:
        _put(v, bt, i, lens[i], "bf16")
    out, info = run_hip(q, k, v, bt, L, Hq, Hkv, d, "bf16", fused_max=-1)
    assert info["items"] == B * Hkv and info["partial_rows"] == 0
    with np.errstate(invalid="ignore"):
        want = decode_attention(values(q), values(k), values(v), bt, L, requests=rows)
    _check(out, want, "bf16", rows, f"{Hq}/{Hkv}/{d} {B}")
    assert np.isfinite(np.delete(out, rows[1:], axis=0)).all()


@pytest.mark.parametrize("dtype,Hq,Hkv,d,low", [("f32", 8, 2, 64, -752), ("bf16", 8, 2, 64, -752), ("bf16", 14, 2, 128, -1064), ("bf16", 4, 2, 256, -1504)])
@pytest.mark.parametrize("how", [dict(fused_max=-1, split_blocks=2), dict(fused_max=-1, split_blocks=2, merge_rows_min=-1), dict(fused_max=1 << 20)])
def test_a_piece_whose_weight_is_subnormal(dtype, Hq, Hkv, d, low, how):
    """The first 256 tokens weigh e^-94 (2^-136) of the others: a piece of their own that holds an infinity still makes the output
    infinite."""
    q, k, v, bt, L = _batch(dtype, Hq, Hkv, d, [1601], 33)
    bits = (lambda x: W.f32_to_bf16_bits(np.array([x], np.float32))[0]) if dtype == "bf16" else np.float32
    q[0, :Hq // Hkv, 0] = bits(1)
    for t in range(256):
        k[bt[0, t // 16], 0, t % 16, 0] = bits(low)
    v[bt[0, 0], 0, 3, 1] = bits(np.inf)
    out, info = run_hip(q, k, v, bt, L, Hq, Hkv, d, dtype, **how)
    want = decode_attention(values(q), values(k), values(v), bt, L)
    assert np.isposinf(want[0, :Hq // Hkv, 1]).all() and np.array_equal(np.isposinf(out), np.isposinf(want))
    assert_close(np.where(np.isinf(want), 0, out), np.where(np.isinf(want), 0, want), dtype, what=f"{dtype} {Hq}/{Hkv}/{d} {how}")
