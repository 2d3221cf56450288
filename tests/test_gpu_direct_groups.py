"""The kernel that needs no plan, float32, at query groups around the four heads that its 4x4 products take: every head_dim,
histories that end at every row of a block, of two blocks (a tile at head_dim 32 and 64) and of the waves' first tiles, whole
and in pieces, against the float64 oracle; dead slots hold NaN."""
import numpy as np
import pytest

from gpu_harness import assert_close, run_hip, values
from oracle.attention import decode_attention
from test_gpu_direct import _batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [32, 64, 128, 256])
@pytest.mark.parametrize("group", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("lens", [list(range(0, 35)) + [127, 128, 129, 255, 257, 385], [3000]])
def test_query_groups_of_up_to_four_heads_and_one_more(d, group, lens):
    q, k, v, bt, L = _batch("f32", 2 * group, 2, d, lens, 11 * group + d + len(lens))
    out, info = run_hip(q, k, v, bt, L, 2 * group, 2, d, "f32", fused_max=bt.shape[1])
    assert info["variant"] == 2
    # assert_close's 1e-5: sums of up to d products and up to 3000 weighted rows, 2^-24 each, of outputs of about 1
    assert_close(out, decode_attention(values(q), values(k), values(v), bt, L), "f32", what=f"group {group} d {d} {lens[:3]}")
    assert (out[L == 0] == 0).all()
    again, _ = run_hip(q, k, v, bt, L, 2 * group, 2, d, "f32", fused_max=bt.shape[1])
    assert np.array_equal(out, again)
