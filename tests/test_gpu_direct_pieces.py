"""Histories that the kernel without a plan cuts into pieces: the workgroup that comes last folds them, counted by words of the
workspace that nobody clears.  Whatever the workspace holds, call after call with other piece counts, in a graph replayed
with other calls between: the rows of the float64 oracle, the same bits each time."""
import numpy as np
import pytest

from gpu_harness import assert_close, to_device, values
from oracle.attention import decode_attention
from test_gpu_direct import _batch

pytestmark = pytest.mark.gpu

KEY = 0xFEA5D1A2C37E6B00          # what marks a counter, and words that nearly are one


@pytest.mark.parametrize("dtype,Hq,Hkv,d", [("f32", 8, 2, 64), ("f32", 17, 1, 32), ("bf16", 14, 2, 128), ("bf16", 40, 1, 64), ("bf16", 6, 2, 256)])
@pytest.mark.parametrize("fill", [0, 0xFFFFFFFFFFFFFFFF, KEY, KEY ^ 0x100, "noise"])
def test_any_workspace_any_order_of_calls(dtype, Hq, Hkv, d, fill):
    import torch
    from paper_2605_06046_amd import AttnParams, FEA_DTYPE_BF16, FEA_DTYPE_F32, fea_decode_attention, fea_decode_workspace_bytes
    p = AttnParams(Hq, Hkv, d, FEA_DTYPE_BF16 if dtype == "bf16" else FEA_DTYPE_F32, fused_max=1 << 20)
    planned = AttnParams(Hq, Hkv, d, p.dtype, fused_max=-1)
    batches = [_batch(dtype, Hq, Hkv, d, lens, 31 + len(lens)) for lens in ([3100], [900, 1601, 16, 0], [5000, 37])]
    size = max(fea_decode_workspace_bytes(x, b[3].shape[0], b[3].shape[1]) for b in batches for x in (p, planned))
    ws = torch.empty((size + 7) // 8, dtype=torch.int64, device="cuda")
    if fill == "noise":
        ws.random_()
    else:
        ws.fill_(fill - (1 << 64) if fill >= 1 << 63 else fill)
    ws = ws.view(torch.uint8)
    dev = [[to_device(x) for x in b[:3]] + [torch.from_numpy(b[3]).cuda(), torch.from_numpy(b[4]).cuda()] for b in batches]
    first = [None] * len(batches)

    def call(j, params=p):
        q, k, v, bt, L = dev[j]
        out = torch.full_like(q, float("nan"))
        fea_decode_attention(params, q, k, v, bt, L, out, ws)
        return out

    for step, j in enumerate([0, 1, 2, 2, 0, 1]):
        if step == 3:
            call(1, planned)                  # a plan, partial rows and run search over the same memory
        out = call(j)
        torch.cuda.synchronize()
        if first[j] is None:
            first[j] = out.clone()
            q, k, v, bt, L = batches[j]
            assert_close(out.float().cpu().numpy().astype(np.float64), decode_attention(values(q), values(k), values(v), bt, L), dtype,
                         what=f"{dtype} {Hq}/{Hkv}/{d} batch {j}")
        assert torch.equal(out, first[j])
    st = torch.cuda.Stream()
    q, k, v, bt, L = dev[0]
    out = torch.full_like(q, float("nan"))
    st.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        fea_decode_attention(p, q, k, v, bt, L, out, ws)
    for between in (None, 1, 2):
        if between is not None:
            call(between)
            call(between, planned)
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, first[0])
