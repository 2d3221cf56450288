"""The planner's launch with workgroups that read the ends of the histories ahead of the sweep: what they read is thrown away, so a
call gives what a plan alone (which has none of them) and a sweep over it give, bit for bit, and nothing outside the histories is
followed: dead columns hold -1, requests are empty, shorter than a block, or without a part of their own.  Whether they read is
seen in the plan's header, and goes by the rule restated here."""
import numpy as np
import pytest

import workloads as W
from gpu_harness import assert_close, library_tables, oracle_for, to_device

pytestmark = pytest.mark.gpu


def _ahead(bt, lens, Hkv, d, workgroups):
    """Tiles that the launch reads ahead: its workgroups do if half of those that share a run with a request of theirs, of 32 looked
    at, have 60 MB of their own behind it, were all alike."""
    B, stride = bt.shape
    column = B * Hkv * 2 * 16 * d * 2
    own, opens = int(60e6) // column, False
    for i in {b % B for b in range(1, workgroups)}:
        others = [(i + 1 + k % 32) % B for k in range(32)]
        shares = [o for o in others if o != i and bt[o, 0] == bt[i, 0]]
        last = {o: -(-int(lens[o]) // 16) - 1 - own for o in shares}
        apart = [o for o in shares if last[o] >= 1 and bt[o, last[o]] != bt[i, last[o]]]
        opens |= bool(shares) and 2 * len(apart) >= len(shares)
    return min(stride // 4, (int(28e6) + column) // (2 * column)) if opens and d != 256 else 0


# A column of 16 tokens holds 64 head_dim bytes of K and V per KV head: own parts of 60 MB and more in all turn the reading on.
@pytest.mark.parametrize("run_kernel_min", [0, -1])     # (-1: the planner's launch is the second one)
@pytest.mark.parametrize("B,Hq,Hkv,d,own,empty,reads", [
    (40, 32, 8, 128, (384, 700), 3, 5),    # 64 KB a column: 24 columns and more each
    (40, 32, 8, 128, (352, 380), 0, None),   # about the line
    (70, 8, 8, 128, (257, 500), 1, 3),
    (37, 6, 3, 64, (2160, 2600), 2, 31),
    (24, 4, 2, 256, (1300, 1500), 1, 0),   # (head_dim 256: never)
    (40, 32, 8, 128, (200, 300), 0, 0),    # less of their own
    (72, 32, 8, 64, (384, 700), 2, 6),
])
def test_same_result_as_a_plan_without_it(B, Hq, Hkv, d, own, empty, reads, run_kernel_min):
    import torch
    from paper_2605_06046_amd import (AttnParams, FEA_DTYPE_BF16, FEA_FLAG_PLAN_ONLY, FEA_FLAG_REUSE_PLAN,
                                      fea_decode_attention, fea_decode_workspace_bytes)
    wl = W.generate(W.Spec("ahead", 300 + B, "bf16", Hq, Hkv, d, ((B, 320),), own))
    bt, lens = library_tables(wl)
    bt, lens = bt.copy(), lens.copy()
    lens[1:1 + empty] = np.array([0, 1, 15], dtype=np.int32)[:empty]       # no history, and ones that end in the first block
    columns = (lens + 15) // 16
    bt[np.arange(bt.shape[1])[None, :] >= columns[:, None]] = -1
    mk = lambda flags: AttnParams(Hq, Hkv, d, FEA_DTYPE_BF16, flags=flags, fused_max=-1, run_kernel_min=run_kernel_min)
    q, k, v = to_device(wl.q), to_device(wl.k_cache), to_device(wl.v_cache)
    dbt, dl = torch.from_numpy(bt).cuda(), torch.from_numpy(lens).cuda()
    n = fea_decode_workspace_bytes(mk(0), *bt.shape)
    ws_a, ws_b = (torch.zeros(n, dtype=torch.uint8, device="cuda") for _ in range(2))
    out_a, out_b = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
    fea_decode_attention(mk(0), q, k, v, dbt, dl, out_a, ws_a)
    ahead = [int(ws[48:52].view(torch.int32)) for ws in (ws_a, ws_b)]      # (word 12)
    workgroups = torch.cuda.get_device_properties(0).multi_processor_count // 2
    assert ahead == [_ahead(bt, lens, Hkv, d, workgroups), 0] and reads in (None, ahead[0])
    fea_decode_attention(mk(FEA_FLAG_PLAN_ONLY), q, k, v, dbt, dl, out_b, ws_b)
    fea_decode_attention(mk(FEA_FLAG_REUSE_PLAN), q, k, v, dbt, dl, out_b, ws_b)
    torch.cuda.synchronize()
    assert torch.equal(out_a, out_b)
    rows = list(range(0, B, max(1, B // 12)))
    assert_close(out_a.float().cpu().numpy().astype(np.float64), oracle_for(wl, bt, lens, requests=rows), "bf16", rows=rows, what="read ahead")
