"""The kernel that needs no plan (short or few histories): histories that end at every kind of edge of its tiles, waves and
pieces, query groups below, at and above a row tile, against the float64 oracle; dead slots hold NaN."""
import numpy as np
import pytest

import workloads as W
from gpu_harness import assert_close, oracle_for, run_hip, run_workload, values
from oracle.attention import decode_attention

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 15, 16, 17, 31, 32, 33, 63, 65, 127, 128, 129, 255, 256, 257, 300, 511, 513]
SHAPES = [("f32", 4, 4, 32), ("f32", 8, 2, 64), ("f32", 17, 1, 128), ("f32", 6, 2, 256), ("bf16", 16, 1, 64), ("bf16", 14, 2, 128),
          ("bf16", 33, 1, 128), ("bf16", 5, 1, 256), ("bf16", 65, 1, 64)]


def _batch(dtype, Hq, Hkv, d, lens, seed, stride_extra=3):
    rng = np.random.default_rng(seed)
    nbs = [-(-L // 16) for L in lens]
    nblocks = sum(nbs) + 2
    ids = rng.permutation(nblocks).astype(np.int32)
    bt = np.full((len(lens), max(max(nbs), 1) + stride_extra), -1, dtype=np.int32)
    at = 0
    for i, nb in enumerate(nbs):
        bt[i, :nb] = ids[at:at + nb]
        at += nb
    def draw(*shape):
        x = rng.standard_normal(size=shape, dtype=np.float32)
        return W.f32_to_bf16_bits(x) if dtype == "bf16" else x
    q, k, v = draw(len(lens), Hq, d), draw(nblocks, Hkv, 16, d), draw(nblocks, Hkv, 16, d)
    live = np.zeros(nblocks, dtype=np.int64)
    for i, L in enumerate(lens):
        for c in range(nbs[i]):
            live[bt[i, c]] = min(16, L - 16 * c)
    for c in (k, v):
        for b in range(nblocks):
            c[b, :, live[b]:] = W.BF16_NAN if dtype == "bf16" else np.float32(np.nan)
    return q, k, v, bt, np.array(lens, dtype=np.int32)


@pytest.mark.parametrize("dtype,Hq,Hkv,d", SHAPES)
@pytest.mark.parametrize("lens", [EDGES, [1600], [4095, 3], [777, 1601, 16]])
def test_edges_of_tiles_waves_and_pieces(dtype, Hq, Hkv, d, lens):
    """Many requests: whole histories.  One to three long ones: few workgroups, so histories are cut into pieces (an odd
    number of them, some without a tile of the short request) and merged."""
    q, k, v, bt, L = _batch(dtype, Hq, Hkv, d, lens, 7 * Hq + d + len(lens))
    out, info = run_hip(q, k, v, bt, L, Hq, Hkv, d, dtype, fused_max=bt.shape[1])
    assert info["variant"] == 2 and info["overflow"] == 0
    assert_close(out, decode_attention(values(q), values(k), values(v), bt, L), dtype, what=f"direct {dtype} {Hq}/{Hkv}/{d} {lens}")
    assert (out[L == 0] == 0).all()
    again, _ = run_hip(q, k, v, bt, L, Hq, Hkv, d, dtype, fused_max=bt.shape[1])
    assert np.array_equal(out, again)


@pytest.mark.parametrize("dtype,Hq,Hkv,d", SHAPES)
@pytest.mark.parametrize("blocks", [1, 2, 3, 4, 5])
def test_tables_of_up_to_two_tiles_and_just_more(dtype, Hq, Hkv, d, blocks):
    """Workgroups of two waves up to two tiles of the table's width (a tile: two blocks; one for float32 from head_dim 128 on)."""
    lens = sorted({0, 1, 15, 16, 17, 16 * blocks - 15, 16 * blocks - 1, 16 * blocks} & set(range(16 * blocks + 1)))
    q, k, v, bt, L = _batch(dtype, Hq, Hkv, d, lens, 3 * Hq + d + blocks, stride_extra=0)
    assert bt.shape[1] == blocks
    out, info = run_hip(q, k, v, bt, L, Hq, Hkv, d, dtype, fused_max=blocks)
    assert info["variant"] == 2
    waves = 2 if blocks <= (2 if dtype == "f32" and d >= 128 else 4) else 4 if d == 256 else 8
    assert info["shares"] == waves * len(lens) * Hkv * -(-Hq // Hkv // 16)
    assert_close(out, decode_attention(values(q), values(k), values(v), bt, L), dtype, what=f"direct {dtype} {Hq}/{Hkv}/{d} {lens}")
    assert (out[L == 0] == 0).all()


@pytest.mark.parametrize("dtype,Hq,Hkv,d", [("f32", 8, 2, 64), ("bf16", 14, 2, 128)])
@pytest.mark.parametrize("lens", [[40, 300, 33], [1600, 900]])
def test_nan_and_infinity_of_a_live_token_stay_with_their_request(dtype, Hq, Hkv, d, lens):
    """A NaN in one live K or V row, or an infinite score, reaches every query head that attends to it and no other request;
    scores of -inf next to finite ones of the same tile have weight 0 (for tiles of nothing else: test_gpu_minus_infinity)."""
    nan = W.BF16_NAN if dtype == "bf16" else np.float32(np.nan)
    inf = (lambda s: np.uint16(0x7F80 if s > 0 else 0xFF80)) if dtype == "bf16" else (lambda s: np.float32(s * np.inf))
    for where in ("k", "v", "+inf", "-inf"):
        q, k, v, bt, L = _batch(dtype, Hq, Hkv, d, lens, 5)
        t = lens[0] - 1                                    # the last token, in a tile that ends short
        blk = bt[0, t // 16]
        if where in ("k", "v"):
            (k if where == "k" else v)[blk, 0, t % 16, 3] = nan
        else:
            q[0, :, 0] = W.f32_to_bf16_bits(np.ones(Hq, np.float32)) if dtype == "bf16" else 1.0
            k[blk, 0, t % 16, 0] = inf(1 if where == "+inf" else -1)
        out, _ = run_hip(q, k, v, bt, L, Hq, Hkv, d, dtype, fused_max=bt.shape[1])
        G = Hq // Hkv
        if where == "k":
            assert np.isnan(out[0, :G]).all()
        elif where == "v":
            assert np.isnan(out[0, :G, 3]).all() and np.isfinite(np.delete(out[0, :G], 3, axis=1)).all()
        elif where == "+inf":
            assert np.isnan(out[0, :G]).all()
        else:
            kk = values(k).astype(np.float32).copy()
            kk[blk, 0, t % 16, 0] = -1e30                  # the oracle's weight 0
            want = decode_attention(values(q), kk, values(v), bt, L)
            assert_close(out, want, dtype, what="-inf score")
        assert np.isfinite(out[0, G:]).all() and np.isfinite(out[1:]).all()


def test_short_and_few_histories_need_no_plan_and_long_batches_do():
    small = W.generate(W.Spec("chats", 91, "bf16", 28, 4, 128, ((8, 0),), (90, 700)))
    out, bt, lens, info = run_workload(small, fused_max=0)
    assert info["variant"] == 2
    assert_close(out, oracle_for(small, bt, lens), "bf16", what="short chats by default")
    wide = W.generate(W.Spec("f32_layer", 92, "f32", 32, 8, 128, ((6, 512),), (100, 700)))
    out, bt, lens, info = run_workload(wide, fused_max=0)
    assert info["variant"] == 2
    assert_close(out, oracle_for(wide, bt, lens), "f32", what="float32 layer by default")
    big = W.generate(W.Spec("big", 93, "bf16", 32, 8, 128, ((40, 1024),), (5, 60)))
    out, bt, lens, info = run_workload(big, fused_max=0)
    assert info["variant"] == 1 and info["groups"] == 1
