"""Lines of the default route that go by the query heads of a KV head: bfloat16 with more than eight up to 225 MB of histories,
float32 with two to sixteen up to 1.5 MB of a history to a workgroup; on either side the other way's result and the oracle's."""
import pytest

from test_gpu_routes import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,Hq,Hkv,d,B,T,planless", [
    ("bf16", 32, 2, 128, 40, 5488, True), ("bf16", 32, 2, 128, 40, 5504, False),    # 225 MB
    ("bf16", 9, 1, 128, 80, 2800, True), ("bf16", 8, 1, 128, 80, 2800, False),      # 115 MB, nine heads and eight
    ("bf16", 9, 1, 64, 1025, 480, False),                                           # more than four workgroups to a compute unit
    ("f32", 32, 16, 32, 9, 5600, True), ("f32", 16, 16, 32, 9, 5600, False),        # two heads and one; the estimate has both planned
])
def test_either_side_of_the_lines_over_heads(dtype, Hq, Hkv, d, B, T, planless):
    _check(dtype, Hq, Hkv, d, B, T, planless)
