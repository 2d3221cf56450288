"""Lines of the default route that keep one workgroup from reading a long history alone: float32 with two to sixteen query heads
per KV head up to 1.5 MB of a history to a workgroup, bfloat16 with more than eight up to twelve tiles to a wave.  The table's
width is all that the rule sees, so a batch with one long history among short ones goes the way of its longest."""
import numpy as np
import pytest

from gpu_harness import assert_close, run_hip, values
from oracle.attention import decode_attention
from test_gpu_direct import _batch
from test_gpu_routes import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,Hq,Hkv,d,B,T,planless", [
    ("f32", 32, 16, 32, 9, 5856, True), ("f32", 32, 16, 32, 9, 5872, False),        # 1.5 MB, whole histories
    ("f32", 16, 8, 32, 9, 17568, True), ("f32", 16, 8, 32, 9, 17584, False),          # ... in three pieces each
    ("bf16", 9, 1, 64, 160, 3072, True), ("bf16", 9, 1, 64, 160, 3088, False),      # twelve tiles to a wave
])
def test_either_side_of_the_lines_over_a_workgroup(dtype, Hq, Hkv, d, B, T, planless):
    _check(dtype, Hq, Hkv, d, B, T, planless)


@pytest.mark.parametrize("dtype,Hq,Hkv,d,B,longest,short", [
    ("f32", 2, 1, 64, 134, 46207, 34), ("f32", 16, 8, 32, 64, 100000, 500), ("bf16", 16, 1, 64, 70, 11373, 28),
])
def test_one_long_history_among_short_ones_is_planned(dtype, Hq, Hkv, d, B, longest, short):
    lens = [short + j % 7 for j in range(B)]
    lens[B // 3] = longest
    q, k, v, bt, L = _batch(dtype, Hq, Hkv, d, lens, 21)
    out, info = run_hip(q, k, v, bt, L, Hq, Hkv, d, dtype, fused_max=0)
    assert info["variant"] != 2
    rows = [0, B // 3, B - 1]
    want = decode_attention(values(q), values(k), values(v), bt, L, requests=rows)
    assert_close(out, want, dtype, rows=rows, what=f"{dtype} {Hq}/{Hkv}/{d} {B} x {longest}/{short}")
