"""What the planner marks as read once (the sweep has it pass by the caches), read from the plan itself: batches of 32 MB and more,
whatever one item alone reads and nothing else; smaller ones stay in the caches.  And results on both sides of that line."""
import numpy as np
import pytest

import workloads as W
from gpu_harness import assert_close, plan_items, to_device, values
from oracle.attention import decode_attention

pytestmark = pytest.mark.gpu

ONCE, TEAM = 1 << 24, 15 << 16


def _sweep(Hq, Hkv, d, groups, system, own, seed, max_group=0):
    """groups: (requests, blocks they share behind the system prompt's).  -> (items, plan info)"""
    import torch
    from paper_2605_06046_amd import AttnParams, FEA_DTYPE_BF16, fea_decode_attention, fea_decode_plan_info, fea_decode_workspace_bytes
    rng = np.random.default_rng(seed)
    ids = iter(range(1 << 20))
    take = lambda n: [next(ids) for _ in range(n)]
    top, rows, lens = take(system), [], []
    for n, shared in groups:
        run = top + take(shared)
        for _ in range(n):
            rows.append(run + take(own(len(rows))))
            lens.append(16 * len(rows[-1]) - int(rng.integers(0, 16)))
    bt = np.full((len(rows), max(map(len, rows)) + 3), -1, dtype=np.int32)
    for i, r in enumerate(rows):
        bt[i, :len(r)] = r
    lens = np.array(lens, dtype=np.int32)
    draw = lambda *s: W.f32_to_bf16_bits(rng.standard_normal(s, dtype=np.float32))
    n = next(ids)
    q, k, v = draw(len(rows), Hq, d), draw(n, Hkv, 16, d), draw(n, Hkv, 16, d)
    p = AttnParams(Hq, Hkv, d, FEA_DTYPE_BF16, fused_max=-1, max_group=max_group)
    ws = torch.zeros(fea_decode_workspace_bytes(p, *bt.shape), dtype=torch.uint8, device="cuda")
    dq = to_device(q)
    out = torch.full_like(dq, float("nan"))
    fea_decode_attention(p, dq, to_device(k), to_device(v), torch.from_numpy(bt).cuda(), torch.from_numpy(lens).cuda(), out, ws)
    info = fea_decode_plan_info(ws)
    torch.cuda.synchronize()
    some = list(range(0, len(rows), max(1, len(rows) // 6)))
    want = decode_attention(values(q), values(k), values(v), bt, lens, requests=some)
    assert_close(out.float().cpu().numpy().astype(np.float64), want, "bf16", rows=some, what=f"{Hq}/{Hkv}/{d}")
    return plan_items(ws, len(rows), Hkv), info


def _marks(items):
    """Of the items that sweep anything: (marked, all) of requests' own columns, of runs swept by waves on their own, of teams'."""
    live = items[items["nrows"] > 0]
    own, team = live["mlist_off"] < 0, (live["g"] & TEAM) != 0
    once = (live["g"] & ONCE) != 0
    return [(int((once & s).sum()), int(s.sum())) for s in (own, ~own & ~team, team)]


# A tile of 32 tokens has 128 head_dim bytes: 1954 of them are 32 MB at head_dim 128, 3907 at 64, 977 at 256.
@pytest.mark.parametrize("Hq,Hkv,d,tiles", [(32, 8, 128, 245), (8, 2, 64, 1954), (8, 4, 256, 245)])
@pytest.mark.parametrize("less", [0, 1])
def test_the_line(Hq, Hkv, d, tiles, less):
    own = lambda i: 2 * (tiles // 5 + (tiles % 5 if i == 0 else 0) - (less if i == 1 else 0))
    items, info = _sweep(Hq, Hkv, d, ((5, 0),), 0, own, 7 + d)
    assert info["groups"] == 0 and info["overflow"] == 0
    (marked, of), runs, teams = _marks(items)
    assert runs == teams == (0, 0) and of > 0 and marked == (0 if less else of)


@pytest.mark.parametrize("large", [False, True])
@pytest.mark.parametrize("Hq,Hkv,d", [(8, 2, 128), (8, 4, 64), (2, 1, 256)])
@pytest.mark.parametrize("shape,groups,system,own_marked,run_marked", [
    ("groups", ((5, 12), (3, 6), (1, 0)), 0, True, True),
    ("split_off", ((10, 32), (12, 34)), 16, True, False),                # both groups sweep the system prompt
    ("stay_together", ((2, 4), (2, 4), (2, 4), (2, 6)), 64, False, True),   # of their own columns some are the same
])
def test_what_is_marked(shape, groups, system, own_marked, run_marked, Hq, Hkv, d, large):
    items, info = _sweep(Hq, Hkv, d, groups, system, lambda i: (400 if large else 20) + i, 31)
    assert info["groups"] > 0 and info["overflow"] == 0
    own, runs, teams = _marks(items)
    assert own[1] > 0 and runs[1] > 0 and teams == (0, 0)
    assert own[0] == (own[1] if large and own_marked else 0) and runs[0] == (runs[1] if large and run_marked else 0)


def test_nothing_was_looked_for():
    items, info = _sweep(8, 2, 128, ((5, 40),), 0, lambda i: 500, 5, max_group=1)
    own, runs, _ = _marks(items)
    assert info["groups"] == 0 and own[1] > 0 and own[0] == runs[1] == 0
