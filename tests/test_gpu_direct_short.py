"""bfloat16 without a plan in narrow tables: K rows in neighbouring lanes up to 4 blocks at head_dim 128 and 16 at 256, in pieces beyond
(and at head_dim 64).  On both sides of every line, with one to sixteen query heads, ends inside a block, infinities in V."""
import numpy as np
import pytest

from gpu_harness import assert_close, run_hip, values
from oracle.attention import decode_attention
from test_gpu_direct import _batch
from test_gpu_infinite_values import _check, _put

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,width", [(64, 4), (64, 5), (128, 1), (128, 4), (128, 5), (256, 3), (256, 4), (256, 5), (256, 8), (256, 16), (256, 17)])
@pytest.mark.parametrize("Hq,Hkv", [(2, 2), (7, 1), (32, 2), (20, 1)])
def test_both_ways_to_lay_out_k(Hq, Hkv, d, width):
    top = 16 * width
    lens = [top, 1, top - 1, max(1, top - 16), 0, max(1, top - 33), top // 2 + 1, 15]
    q, k, v, bt, L = _batch("bf16", Hq, Hkv, d, lens, 41 + width)
    bt = np.ascontiguousarray(bt[:, :width])
    out, info = run_hip(q, k, v, bt, L, Hq, Hkv, d, "bf16", fused_max=width)
    assert info["variant"] == 2
    want = decode_attention(values(q), values(k), values(v), bt, L)
    assert_close(out, want, "bf16", what=f"{Hq}/{Hkv}/{d} width {width}")
    if width > 3:
        rows = [0, 3]
        for i in rows:
            _put(v, bt, i, lens[i], "bf16")
        out, _ = run_hip(q, k, v, bt, L, Hq, Hkv, d, "bf16", fused_max=width)
        with np.errstate(invalid="ignore"):
            want = decode_attention(values(q), values(k), values(v), bt, L)
        _check(out, want, "bf16", rows, f"{Hq}/{Hkv}/{d} width {width}")
