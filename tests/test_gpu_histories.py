"""Large batches that share nothing: the planner makes no plan, the sweep takes whole histories.  Lengths at the edges of tiles,
waves and id windows among long ones, one plan used again and stretched, captured, and the same batch with one shared block."""
import numpy as np
import pytest

from gpu_harness import assert_close, to_device, values
from oracle.attention import decode_attention
from test_gpu_direct import _batch

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 15, 16, 17, 31, 32, 33, 127, 128, 129, 255, 256, 257, 4095, 4096, 4097, 4129]


@pytest.mark.parametrize("Hq,Hkv,d,B,typical", [(8, 8, 64, 140, 900), (14, 2, 128, 600, 900), (16, 1, 64, 1030, 1000), (40, 8, 128, 130, 800)])
def test_whole_histories(Hq, Hkv, d, B, typical):
    import torch
    from paper_2605_06046_amd import (AttnParams, FEA_DTYPE_BF16, FEA_FLAG_REFRESH_PLAN, FEA_FLAG_REUSE_PLAN, fea_decode_attention,
                                      fea_decode_plan_info, fea_decode_workspace_bytes)
    rng = np.random.default_rng(Hq + B)
    lens = EDGES + rng.integers(typical // 2, typical * 2, size=B - len(EDGES)).tolist()
    rng.shuffle(lens)
    q, k, v, bt, L = _batch("bf16", Hq, Hkv, d, lens, B)
    dq, dk, dv = (to_device(x) for x in (q, k, v))
    dbt, dl = torch.from_numpy(bt).cuda(), torch.from_numpy(L).cuda()
    made = AttnParams(Hq, Hkv, d, FEA_DTYPE_BF16, fused_max=-1)
    ws = torch.full((fea_decode_workspace_bytes(made, B, bt.shape[1]),), 0x5A, dtype=torch.uint8, device="cuda")

    def call(flags=0, lengths=dl):
        p = AttnParams(Hq, Hkv, d, FEA_DTYPE_BF16, fused_max=-1, flags=flags)
        out = torch.full_like(dq, float("nan"))
        fea_decode_attention(p, dq, dk, dv, dbt, lengths, out, ws)
        return out

    out = call()
    info = fea_decode_plan_info(ws)
    assert info["variant"] == 1 and info["groups"] == 0 and info["overflow"] == 0
    assert info["items"] == B * Hkv and info["partial_rows"] == 0            # (no plan was made)
    rows = [i for i, n in enumerate(lens) if n in EDGES][:len(EDGES)] + [0, B - 1]
    want = decode_attention(values(q), values(k), values(v), bt, L, requests=rows)
    assert_close(out.float().cpu().numpy().astype(np.float64), want, "bf16", rows=rows, what=f"{Hq}/{Hkv}/{d} {B}")
    assert (out[torch.from_numpy(L == 0).cuda()] == 0).all()
    assert torch.isfinite(out.float()).all()
    for flags in (FEA_FLAG_REUSE_PLAN, FEA_FLAG_REFRESH_PLAN, 0, FEA_FLAG_REUSE_PLAN):
        assert torch.equal(call(flags), out)
    # shorter lengths: a plan of an earlier step
    earlier = torch.clamp(dl - 1, min=0)
    before = call(0, earlier)
    grown = call(FEA_FLAG_REFRESH_PLAN)
    assert torch.equal(grown, out) and not torch.equal(before, out)
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    p, r = (AttnParams(Hq, Hkv, d, FEA_DTYPE_BF16, fused_max=-1, flags=f) for f in (0, FEA_FLAG_REUSE_PLAN))
    o1, o2 = torch.empty_like(dq), torch.empty_like(dq)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        fea_decode_attention(p, dq, dk, dv, dbt, dl, o1, ws)
        fea_decode_attention(r, dq, dk, dv, dbt, dl, o2, ws)
    for _ in range(3):
        o1.fill_(float("nan"))
        o2.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(o1, out) and torch.equal(o2, out)
        call(0, earlier)
    # one request on another's first block: a plan again
    a, b = [i for i, n in enumerate(lens) if n > typical // 2][:2]
    shared = bt.copy()
    shared[b, :2] = shared[a, :2]
    dbt.copy_(torch.from_numpy(shared))
    out = call()
    info = fea_decode_plan_info(ws)
    assert info["groups"] == 1 and info["grouped_requests"] == 2 and info["partial_rows"] > 0
    want = decode_attention(values(q), values(k), values(v), shared, L, requests=[a, b, 0])
    assert_close(out.float().cpu().numpy().astype(np.float64), want, "bf16", rows=[a, b, 0], what="one shared run")


@pytest.mark.parametrize("Hq,Hkv,d,B,tokens,longest,whole", [
    (8, 8, 64, 128, 768, 768, True), (8, 8, 64, 128, 736, 736, False),          # 24 tiles a history
    (8, 8, 128, 128, 384, 384, True), (8, 8, 128, 128, 352, 352, False),        # 12 tiles
    (8, 8, 64, 128, 768, 3136, True), (8, 8, 64, 128, 768, 3264, False),        # 98 and 102 tiles, 252 workgroups for 24 800
    (16, 1, 128, 500, 1000, 1000, True), (16, 1, 128, 530, 1000, 1000, False),  # nearly two to a compute unit, and a few more
    (17, 1, 128, 512, 1000, 1000, False), (4, 4, 256, 300, 1000, 1000, False),
    (8, 8, 128, 2048, 400, 400, True), (8, 8, 128, 2049, 400, 400, False),
])
def test_which_batches_are_read_whole(Hq, Hkv, d, B, tokens, longest, whole):
    """By the plan alone: no caches are read."""
    import torch
    from paper_2605_06046_amd import AttnParams, FEA_DTYPE_BF16, FEA_FLAG_PLAN_ONLY, fea_decode_attention, fea_decode_plan_info, fea_decode_workspace_bytes
    lens = np.full(B, tokens, dtype=np.int32)
    lens[B // 2] = longest
    width = -(-longest // 16) + 1
    bt = np.arange(B * width, dtype=np.int32).reshape(B, width)
    p = AttnParams(Hq, Hkv, d, FEA_DTYPE_BF16, flags=FEA_FLAG_PLAN_ONLY)
    ws = torch.empty(fea_decode_workspace_bytes(p, B, width), dtype=torch.uint8, device="cuda")
    none = torch.empty(16, dtype=torch.bfloat16, device="cuda")
    q = torch.empty(B, Hq, d, dtype=torch.bfloat16, device="cuda")
    fea_decode_attention(p, q, none, none, torch.from_numpy(bt).cuda(), torch.from_numpy(lens).cuda(), q, ws)
    info = fea_decode_plan_info(ws)
    assert info["variant"] == 1 and info["groups"] == 0 and info["overflow"] == 0
    assert (info["partial_rows"] == 0) == whole
