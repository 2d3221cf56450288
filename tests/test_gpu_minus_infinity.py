"""Scores of -inf (a key row that holds an infinity): weight 0 next to any finite score, wherever the tokens lie - also where
they are all that a wave, a piece or a first tile of 32 tokens holds - and an undefined row (0/0) where there is nothing else."""
import numpy as np
import pytest

import workloads as W
from gpu_harness import assert_close, run_hip, values
from oracle.attention import decode_attention
from test_gpu_direct import _batch

pytestmark = pytest.mark.gpu

SHAPES = [("f32", 8, 2, 64), ("f32", 4, 2, 128), ("bf16", 14, 2, 128), ("bf16", 8, 2, 64), ("bf16", 4, 2, 256)]


def _forbid(k, q, bt, tokens, dtype, requests=(0,)):
    """The score of KV head 0 with the given tokens of request 0 (and of whoever shares their blocks) becomes -inf: the key's
    element 0 is -inf, the query's is 1.  Returns the keys with -1e30 in its place, which the oracle gives weight 0."""
    one = W.f32_to_bf16_bits(np.ones(1, np.float32))[0] if dtype == "bf16" else np.float32(1)
    Hkv = k.shape[1]
    G = q.shape[1] // Hkv
    for i in requests:
        q[i, :G, 0] = one
    finite = values(k).astype(np.float32).copy()
    for t in tokens:
        b = bt[requests[0], t // 16]
        k[b, 0, t % 16, 0] = np.uint16(0xFF80) if dtype == "bf16" else np.float32(-np.inf)
        finite[b, 0, t % 16, 0] = -1e30
    return finite


@pytest.mark.parametrize("dtype,Hq,Hkv,d", SHAPES)
@pytest.mark.parametrize("lens,tokens", [
    ([33, 300, 33], [32]),                            # alone in the second wave's only tile
    ([290, 33], list(range(32))),                     # all of the first wave's first tile (and its second is finite or absent)
    ([257], list(range(16, 257))),                    # everything but the first block
    ([1601, 900], [1600]),                            # cut into pieces: alone in its piece's last tile
    ([1601, 900], list(range(0, 1568))),              # ... and whole pieces
])
def test_without_a_plan(dtype, Hq, Hkv, d, lens, tokens):
    q, k, v, bt, L = _batch(dtype, Hq, Hkv, d, lens, 11)
    finite = _forbid(k, q, bt, tokens, dtype)
    out, info = run_hip(q, k, v, bt, L, Hq, Hkv, d, dtype, fused_max=bt.shape[1])
    assert info["variant"] == 2
    assert_close(out, decode_attention(values(q), finite, values(v), bt, L), dtype, what=f"{dtype} {Hq}/{Hkv}/{d} {lens}")


@pytest.mark.parametrize("dtype,Hq,Hkv,d", SHAPES)
@pytest.mark.parametrize("lens", [[33, 0, 40], [1601, 0]])
def test_nothing_but_minus_infinity(dtype, Hq, Hkv, d, lens):
    q, k, v, bt, L = _batch(dtype, Hq, Hkv, d, lens, 12)
    _forbid(k, q, bt, range(lens[0]), dtype)
    out, info = run_hip(q, k, v, bt, L, Hq, Hkv, d, dtype, fused_max=bt.shape[1])
    assert info["variant"] == 2
    G = Hq // Hkv
    assert np.isnan(out[0, :G]).all() and np.isfinite(out[0, G:]).all()
    assert (out[1] == 0).all() and np.isfinite(out[2:]).all()


@pytest.mark.parametrize("dtype,Hq,Hkv,d", SHAPES)
@pytest.mark.parametrize("lens,tokens", [([33, 300, 33], [32]), ([290, 33], list(range(288))), ([1601, 900], list(range(0, 1568)))])
@pytest.mark.parametrize("split", [0, 2])
def test_own_columns_under_a_plan(dtype, Hq, Hkv, d, lens, tokens, split):
    """Pieces of a request's own columns whose first tile, or every tile, scores -inf."""
    q, k, v, bt, L = _batch(dtype, Hq, Hkv, d, lens, 13)
    finite = _forbid(k, q, bt, tokens, dtype)
    out, info = run_hip(q, k, v, bt, L, Hq, Hkv, d, dtype, fused_max=-1, split_blocks=split)
    assert info["variant"] == (1 if dtype == "bf16" else 0)
    assert_close(out, decode_attention(values(q), finite, values(v), bt, L), dtype, what=f"{dtype} {Hq}/{Hkv}/{d} {lens} split {split}")


@pytest.mark.parametrize("dtype,Hq,Hkv,d,members", [("f32", 8, 2, 64, 5), ("bf16", 8, 2, 64, 20), ("bf16", 4, 2, 256, 20),
                                                  ("bf16", 8, 2, 128, 9), ("bf16", 8, 2, 128, 20), ("bf16", 8, 2, 128, 40)])
@pytest.mark.parametrize("spared", [[], [511], [200]])
def test_a_shared_run_under_a_plan(dtype, Hq, Hkv, d, members, spared):
    """A run of 512 tokens that scores -inf for every member, but for the tokens spared (head_dim 128, bf16: one row tile,
    teams of two waves, teams of four); the members' own tokens are finite."""
    lens = [512 + 3 + 5 * j for j in range(members)]
    q, k, v, bt, L = _batch(dtype, Hq, Hkv, d, lens, 14)
    for i in range(1, members):
        bt[i, :32] = bt[0, :32]
    finite = _forbid(k, q, bt, [t for t in range(512) if t not in spared], dtype, requests=tuple(range(members)))
    out, info = run_hip(q, k, v, bt, L, Hq, Hkv, d, dtype, fused_max=-1)
    assert info["groups"] == 1 and info["grouped_requests"] == members
    assert_close(out, decode_attention(values(q), finite, values(v), bt, L), dtype, what=f"{dtype} {Hq}/{Hkv}/{d} x{members}")
    q, k, v, bt, L = _batch(dtype, Hq, Hkv, d, [512] * members, 15)       # and nothing else: undefined rows of KV head 0 alone
    for i in range(1, members):
        bt[i, :32] = bt[0, :32]
    _forbid(k, q, bt, range(512), dtype, requests=tuple(range(members)))
    out, _ = run_hip(q, k, v, bt, L, Hq, Hkv, d, dtype, fused_max=-1)
    G = Hq // Hkv
    assert np.isnan(out[:, :G]).all() and np.isfinite(out[:, G:]).all()
