"""FEA_FLAG_REFRESH_PLAN across the line between calls that need no plan and calls that do: requests grow, their table gets
new columns, and the workspace holds what the plan-free kernel left in it (or, before any call, nothing but set bits)."""
import numpy as np
import pytest

from gpu_harness import assert_close, to_device, values
from oracle.attention import decode_attention
from paper_2605_06046_amd import (AttnParams, FEA_DTYPE_BF16, FEA_DTYPE_F32, FEA_FLAG_REFRESH_PLAN, FEA_FLAG_REUSE_PLAN,
                                  fea_decode_attention, fea_decode_plan_info, fea_decode_workspace_bytes)
from test_gpu_direct import _batch

pytestmark = pytest.mark.gpu


class Steps:
    """One batch over some decode steps: the final table and caches are drawn once, a step sees a prefix of them."""

    def __init__(self, dtype, Hq, Hkv, d, final_lens, seed, **pkw):
        import torch
        self.dtype, self.heads, self.d, self.pkw, self.torch = dtype, (Hq, Hkv), d, pkw, torch
        self.q, self.k, self.v, self.bt, _ = _batch(dtype, Hq, Hkv, d, final_lens, seed, stride_extra=0)
        self.dev = [to_device(x) for x in (self.q, self.k, self.v)]
        self.ws = torch.full((fea_decode_workspace_bytes(self.params(0), len(final_lens), self.bt.shape[1]),), 0xFF,
                             dtype=torch.uint8, device="cuda")

    def params(self, flags):
        return AttnParams(*self.heads, self.d, FEA_DTYPE_BF16 if self.dtype == "bf16" else FEA_DTYPE_F32, flags=flags, **self.pkw)

    def step(self, lens, width, flags, check=True):
        torch = self.torch
        bt = np.ascontiguousarray(self.bt[:, :width])
        lens = np.asarray(lens, dtype=np.int32)
        out = torch.full_like(self.dev[0], float("nan"))
        fea_decode_attention(self.params(flags), *self.dev, torch.from_numpy(bt).cuda(), torch.from_numpy(lens).cuda(), out, self.ws)
        info = fea_decode_plan_info(self.ws)
        got = out.float().cpu().numpy().astype(np.float64)
        if check:
            assert info["overflow"] == 0
            want = decode_attention(values(self.q), values(self.k), values(self.v), bt, lens)
            assert_close(got, want, self.dtype, what=f"{self.dtype} {self.heads}/{self.d} width {width} flags {flags}")
            assert (got[lens == 0] == 0).all()
        return got, info


@pytest.mark.parametrize("dtype,Hq,Hkv,d", [("f32", 8, 2, 64), ("bf16", 14, 2, 128), ("bf16", 8, 2, 64), ("bf16", 10, 2, 256), ("bf16", 65, 1, 64)])
@pytest.mark.parametrize("lens", [
    [640], [1600], [16000],                            # whole histories, and cut ones (the last left partial rows behind)
    [1, 16, 17, 640, 333, 0, 150, 65],                 # short next to long, one empty
    [1600, 5],
    [1 + 7 * j % 97 for j in range(1100)],             # more (request, KV head) pairs than the sweep has waves
])
def test_a_table_that_outgrows_the_plan_free_kernel(dtype, Hq, Hkv, d, lens):
    lens = np.array(lens)
    width = -(-int(lens.max()) // 16)
    grown = lens + np.where(lens > 0, 17, 0)
    later = grown + np.where(lens > 0, 40, 0)
    s = Steps(dtype, Hq, Hkv, d, [int(x) for x in later], 3, fused_max=width)
    _, info = s.step(lens, width, FEA_FLAG_REFRESH_PLAN)
    assert info["variant"] == 2
    for flag in (FEA_FLAG_REFRESH_PLAN, FEA_FLAG_REUSE_PLAN):   # the step that crosses, and its other layers
        _, info = s.step(grown, s.bt.shape[1] - 1, flag)
        assert info["variant"] == (1 if dtype == "bf16" and Hq < 65 else 0) and info["groups"] == 0
    s.step(later, s.bt.shape[1], FEA_FLAG_REFRESH_PLAN)
    s.step(grown, s.bt.shape[1], 0)                    # a plan of its own after all


@pytest.mark.parametrize("dtype,Hq,Hkv,d", [("f32", 8, 2, 64), ("bf16", 14, 2, 128)])
@pytest.mark.parametrize("lens,merge_rows_min", [([640, 33], 0), ([1600], -1)])
def test_a_reused_plan_that_is_none_is_reported(dtype, Hq, Hkv, d, lens, merge_rows_min):
    """(Outside the contract: nothing may have changed since the plan.  The rows must be NaN, not what is left in the workspace.)"""
    width = -(-max(lens) // 16)
    s = Steps(dtype, Hq, Hkv, d, [n + 32 for n in lens], 4, fused_max=width, merge_rows_min=merge_rows_min)
    s.step(lens, width, 0)
    got, info = s.step(lens, width + 1, FEA_FLAG_REUSE_PLAN, check=False)
    assert np.isnan(got).all() and info["overflow"] == 2 and info["variant"] == 2
    s.step(lens, width + 2, 0)


@pytest.mark.parametrize("dtype,Hq,Hkv,d", [("f32", 8, 2, 64), ("bf16", 14, 2, 128), ("bf16", 10, 2, 256)])
@pytest.mark.parametrize("split", [2, 7, 64])
def test_a_plan_of_fixed_pieces_under_a_wider_table(dtype, Hq, Hkv, d, split):
    """With a fixed split the workspace's sections follow from the table's width: a refresh under a wider table cannot stretch
    the plan where it lies.  (Fewer new columns than make a piece: it can, and does.)"""
    lens = np.array([640, 1000, 33, 7, 500])
    width = -(-int(lens.max()) // 16)
    steps = [lens + grown for grown in (0, 17, 400)]
    s = Steps(dtype, Hq, Hkv, d, [int(x) for x in steps[-1]], 5, fused_max=-1, split_blocks=split)
    s.step(steps[0], width, 0)
    s.step(steps[1], width + 2, FEA_FLAG_REFRESH_PLAN)
    s.step(steps[1], width + 2, FEA_FLAG_REUSE_PLAN)
    s.step(steps[2], s.bt.shape[1], FEA_FLAG_REFRESH_PLAN)
    s.step(steps[2], s.bt.shape[1], FEA_FLAG_REFRESH_PLAN)
