"""Where a shared run is cut for teams of four waves: weights are rounded to bfloat16 against the largest score of their piece, so an
output repeats bit for bit from one build to the next only while the cuts stay where they are."""
import pytest

import workloads as W
from gpu_harness import library_tables, to_device

pytestmark = pytest.mark.gpu


def test_cuts_of_a_shared_run():
    """64 requests on one prefix of 4096 tokens (four row tiles of 64 query rows to a team)."""
    import torch
    from paper_2605_06046_amd import (AttnParams, FEA_DTYPE_BF16, FEA_FLAG_PLAN_ONLY, fea_decode_attention, fea_decode_plan_info,
                                      fea_decode_workspace_bytes)
    wl = W.generate(W.CONFIGS["c2"])
    bt, lens = library_tables(wl)
    s = wl.spec
    p = AttnParams(s.num_q_heads, s.num_kv_heads, s.head_dim, FEA_DTYPE_BF16, flags=FEA_FLAG_PLAN_ONLY, fused_max=-1)
    ws = torch.zeros(fea_decode_workspace_bytes(p, *bt.shape), dtype=torch.uint8, device="cuda")
    q = to_device(wl.q)                 # (a plan alone reads neither q nor the caches)
    fea_decode_attention(p, q, q, q, torch.from_numpy(bt).cuda(), torch.from_numpy(lens).cuda(), torch.empty_like(q), ws)
    info = fea_decode_plan_info(ws)
    assert (info["groups"], info["items"], info["split_blocks"], info["partial_rows"]) == (1, 1410, 26, 21000)
