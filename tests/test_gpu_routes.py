"""Which way a call goes by default, on either side of every line of the rule, and how many pieces the plan-free kernel cuts
histories into; the result is the other way's within the oracle's tolerance, and the oracle's for some requests."""
import numpy as np
import pytest

from gpu_harness import TOL, assert_close, run_hip, values
from oracle.attention import decode_attention
from test_gpu_direct import _batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,Hq,Hkv,d,B,below,above", [
    ("bf16", 28, 4, 128, 10, 4880, 4896),              # 100 MB of histories
    ("bf16", 65, 1, 64, 4, 1600, None),                # (query groups past the matrix-core sweep's: by the estimate, always here)
    ("bf16", 12, 4, 256, 13, 1312, None),              # 70 MB in few workgroups
    ("bf16", 32, 8, 128, 13, 2048, 2064),              # one round of workgroups, 1 MB each
    ("bf16", 16, 4, 256, 30, 1296, 1312),              # ... 1.33 MB each at head_dim 256
    ("bf16", 4, 4, 128, 100, 512, 528),                # two rounds, 256 KB each
    ("f32", 32, 32, 32, 5, 3008, 4096),                # one query head per KV head on the vector unit
    ("f32", 32, 8, 128, 16, 1024, None),
])
def test_either_side_of_the_lines_over_lengths(dtype, Hq, Hkv, d, B, below, above):
    for T, planless in ((below, True), (above, False)):
        if T is not None:
            _check(dtype, Hq, Hkv, d, B, T, planless)


@pytest.mark.parametrize("T,below,above", [(64, 960, 1000),        # two tiles: 128 MB
                                           (80, 384, 400),         # 64 MB where there are more than six workgroups to a compute unit
                                           (96, 384, 388)])        # 100 MB up to there
def test_either_side_of_the_lines_over_requests(T, below, above):
    for B, planless in ((below, True), (above, False)):
        _check("bf16", 28, 4, 128, B, T, planless)


def _check(dtype, Hq, Hkv, d, B, T, planless):
    lens = [T] + [max(1, T - (37 * j) % T) for j in range(1, B)]
    q, k, v, bt, L = _batch(dtype, Hq, Hkv, d, lens, B + T, stride_extra=0)
    out, info = run_hip(q, k, v, bt, L, Hq, Hkv, d, dtype, fused_max=0)
    what = f"{dtype} {Hq}/{Hkv}/{d} {B} x {T}"
    assert (info["variant"] == 2) == planless, what
    other, info = run_hip(q, k, v, bt, L, Hq, Hkv, d, dtype, fused_max=-1 if planless else 1 << 20)
    assert (info["variant"] == 2) != planless, what
    max_abs, rel = TOL[dtype]                          # (each is within this of the oracle)
    assert np.isfinite(out).all() and np.abs(out - other).max() <= 2 * max_abs
    assert np.linalg.norm(out - other) <= 2 * rel * np.linalg.norm(other)
    rows = [0, B // 2, B - 1]
    assert_close(out, decode_attention(values(q), values(k), values(v), bt, L, requests=rows), dtype, rows=rows, what=what)


@pytest.mark.parametrize("dtype,Hq,Hkv,d,B,T,pieces,waves", [
    ("bf16", 32, 8, 128, 1, 1600, 7, 8),               # as many as a wave has tiles
    ("f32", 32, 8, 128, 4, 2048, 8, 8),                # as many as fill the compute units
    ("bf16", 8, 2, 256, 3, 2000, 16, 4),
    ("bf16", 32, 8, 128, 16, 512, 1, 8),               # two tiles to a wave: not worth the merge
    ("bf16", 32, 8, 128, 16, 2048, 2, 8),
    ("bf16", 32, 8, 128, 17, 1600, 1, 8),              # more than half of the compute units taken as it is
])
def test_pieces_of_a_history(dtype, Hq, Hkv, d, B, T, pieces, waves):
    q, k, v, bt, L = _batch(dtype, Hq, Hkv, d, [T] * B, 9, stride_extra=0)
    out, info = run_hip(q, k, v, bt, L, Hq, Hkv, d, dtype, fused_max=bt.shape[1])
    assert info["variant"] == 2 and info["shares"] == B * Hkv * pieces * waves
    rows = [0, B - 1]
    assert_close(out, decode_attention(values(q), values(k), values(v), bt, L, requests=rows), dtype, rows=rows)
