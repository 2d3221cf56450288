"""Columns that one item alone reads pass by the caches, others do not: batches of either kind, and both in one - nothing shared,
groups, groups that split off a larger one, members that go on sharing and stay together, grouping switched off - against the
oracle.  (Small ones, which stay in the caches whatever reads them: what is marked, and larger ones, are test_gpu_once_marks'.)"""
import numpy as np
import pytest

import workloads as W
from gpu_harness import assert_close, run_hip, values
from oracle.attention import decode_attention

pytestmark = pytest.mark.gpu

# (requests, blocks they share behind the system prompt) per group, and the system prompt's blocks
SHAPES = {
    "apart": (((7, 0),), 0),
    "groups": (((5, 12), (3, 5), (1, 0)), 0),
    "split_off": (((10, 32), (12, 33)), 16),
    "stay_together": (((2, 3), (2, 4), (2, 3), (2, 5)), 64),
}


@pytest.mark.parametrize("max_group", [0, 1])
@pytest.mark.parametrize("shape", sorted(SHAPES))
@pytest.mark.parametrize("Hq,Hkv,d", [(32, 8, 128), (8, 2, 64), (4, 2, 256), (6, 2, 128)])
def test_either_kind_of_columns(Hq, Hkv, d, shape, max_group):
    groups, system = SHAPES[shape]
    rng = np.random.default_rng(400 + d + Hq)
    B = sum(n for n, _ in groups)
    own = rng.integers(1, 300, size=B)
    ids = iter(rng.permutation(4096))
    take = lambda n: [next(ids) for _ in range(n)]
    top, rows, lens = take(system), [], []
    for n, shared in groups:
        run = top + take(shared)
        for _ in range(n):
            length = 16 * len(run) + int(own[len(rows)])
            rows.append(run + take(-(-length // 16) - len(run)))
            lens.append(length)
    used = {b: k for k, b in enumerate(sorted({b for r in rows for b in r}))}
    bt = np.full((B, max(map(len, rows)) + 3), -1, dtype=np.int32)
    for i, r in enumerate(rows):
        bt[i, :len(r)] = [used[b] for b in r]
    order = rng.permutation(B)
    bt, lens = bt[order], np.array(lens, dtype=np.int32)[order]
    draw = lambda *s: W.f32_to_bf16_bits(rng.standard_normal(s, dtype=np.float32))
    q, k, v = draw(B, Hq, d), draw(len(used), Hkv, 16, d), draw(len(used), Hkv, 16, d)
    out, info = run_hip(q, k, v, bt, lens, Hq, Hkv, d, "bf16", max_group=max_group)
    assert info["overflow"] == 0 and (info["groups"] > 0) == (shape != "apart" and max_group == 0)
    assert_close(out, decode_attention(values(q), values(k), values(v), bt, lens), "bf16", what=f"{shape} d={d} max_group={max_group}")
