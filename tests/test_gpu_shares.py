"""How a plan cuts the private columns into shares, where it can go wrong: shares that end just before, in and just behind a
segment's charge for the change of request, segments of one tile, empty histories, and tables far wider than any history."""
import numpy as np
import pytest

from gpu_harness import assert_close, run_hip, values
from oracle.attention import decode_attention
from test_gpu_direct import _batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv,d", [(10, 2, 64), (8, 8, 128), (6, 3, 256)])
@pytest.mark.parametrize("B,longest,seed", [(7, 200, 1), (160, 40, 2), (300, 97, 3), (91, 400, 4), (64, 161, 5), (1, 16000, 6), (3, 3000, 7)])
def test_shares_that_end_at_every_place_of_a_segment(Hq, Hkv, d, B, longest, seed):
    rng = np.random.default_rng(seed)
    lens = [int(x) for x in rng.integers(0, longest + 1, B)]
    lens[0] = longest
    q, k, v, bt, L = _batch("bf16", Hq, Hkv, d, lens, seed + d)
    out, info = run_hip(q, k, v, bt, L, Hq, Hkv, d, "bf16", fused_max=-1)
    assert info["variant"] == 1 and info["overflow"] == 0 and info["groups"] == 0
    assert_close(out, decode_attention(values(q), values(k), values(v), bt, L), "bf16", what=f"{Hq}/{Hkv}/{d} B={B} up to {longest}")
    assert (out[L == 0] == 0).all()
    fixed, _ = run_hip(q, k, v, bt, L, Hq, Hkv, d, "bf16", fused_max=-1, split_blocks=4)   # no charge, pieces of two tiles
    assert_close(fixed, decode_attention(values(q), values(k), values(v), bt, L), "bf16", what="fixed split")


@pytest.mark.parametrize("extra", [0, 1, 700, 5001])
def test_a_prefix_in_a_table_wider_than_its_histories(extra):
    """The longest history, not the table's width, bounds the search for common runs."""
    shared, lens = 9, [9 * 16 + 1, 9 * 16 + 33, 9 * 16, 300, 301, 12 * 16, 15, 4 * 16]
    q, k, v, bt, L = _batch("bf16", 8, 2, 128, lens, 31 + extra, stride_extra=extra)
    for i in (1, 2, 4, 5):
        bt[i, :shared] = bt[0, :shared]
    bt[7, :4] = bt[3, :4]
    k, v = values(k), values(v)
    k[np.isnan(k)], v[np.isnan(v)] = 0.25, -0.5          # (the blocks that changed hands hold live tokens of others)
    from workloads import f32_to_bf16_bits
    kb, vb = f32_to_bf16_bits(k.astype(np.float32)), f32_to_bf16_bits(v.astype(np.float32))
    out, info = run_hip(q, kb, vb, bt, L, 8, 2, 128, "bf16", fused_max=-1)
    assert info["variant"] == 1 and info["groups"] == 2 and info["grouped_requests"] == 7
    assert_close(out, decode_attention(values(q), values(kb), values(vb), bt, L), "bf16", what=f"{extra} columns more")


def _shared(dtype, Hq, Hkv, d, members, run, own, seed):
    """`members` requests on a common run of `run` columns, each with own[i] tokens after it (no dead slots: _batch's are refilled)."""
    lens = [16 * run + n for n in own]
    q, k, v, bt, L = _batch(dtype, Hq, Hkv, d, lens, seed)
    for i in range(1, members):
        bt[i, :run] = bt[0, :run]
    return q, k, v, bt, L


@pytest.mark.parametrize("dtype,Hq,Hkv,d", [("f32", 8, 2, 64), ("f32", 4, 2, 256), ("bf16", 65, 1, 64)])
@pytest.mark.parametrize("tokens", [2048, 16384])
def test_the_even_split_is_rounded_up_and_not_past_that(dtype, Hq, Hkv, d, tokens):
    """A batch whose shares are as short as they may be (four tiles of two blocks), and come out even."""
    q, k, v, bt, L = _batch(dtype, Hq, Hkv, d, [tokens], 51)
    out, info = run_hip(q, k, v, bt, L, Hq, Hkv, d, dtype, fused_max=-1)
    assert info["split_blocks"] == 8 and info["shares"] == Hkv * tokens // (8 * 16) and info["items"] == info["shares"]
    assert_close(out, decode_attention(values(q), values(k), values(v), bt, L), dtype, what=f"{dtype} {Hq}/{Hkv}/{d} {tokens}")


@pytest.mark.parametrize("Hq,Hkv,d", [(8, 8, 64), (8, 8, 128), (8, 8, 256)])
def test_no_more_shares_than_the_tiles_are_worth(Hq, Hkv, d):
    """A share holds four tiles or more on average, of tiles that are swept: what a segment is charged is none."""
    q, k, v, bt, L = _shared("bf16", Hq, Hkv, d, 24, 8, [20] * 24, 61)
    out, info = run_hip(q, k, v, bt, L, Hq, Hkv, d, "bf16", fused_max=-1)
    assert info["groups"] == 1 and info["grouped_requests"] == 24
    assert info["shares"] <= Hkv * (4 + 24) // 4         # one row tile of the run's four tiles, and each request's own one
    assert_close(out, decode_attention(values(q), values(k), values(v), bt, L), "bf16", what=f"{Hq}/{Hkv}/{d}")
