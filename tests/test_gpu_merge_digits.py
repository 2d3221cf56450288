"""The merge where query groups and KV heads are powers of two and where they are not (rows are taken apart by shifts or by
divisions), one wave per row and several rows per wave, with few and with many partials a row, at every head_dim."""
import pytest

import workloads as W
from gpu_harness import assert_close, oracle_for, run_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("bf16", 256), ("f32", 32), ("f32", 64), ("f32", 128), ("f32", 256)])
@pytest.mark.parametrize("Hq,Hkv", [(8, 2), (12, 4), (15, 3), (6, 6), (7, 1)])
@pytest.mark.parametrize("merge_rows_min", [-1, 1 << 30])
def test_rows_taken_apart(dtype, d, Hq, Hkv, merge_rows_min):
    wl = W.generate(W.Spec("digits", 5, dtype, Hq, Hkv, d, ((5, 640), (2, 0)), (1, 300), interleave=True))
    out, bt, lens, info = run_workload(wl, merge_rows_min=merge_rows_min, split_blocks=4)
    assert info["overflow"] == 0 and info["variant"] == (1 if dtype == "bf16" else 0)
    assert_close(out, oracle_for(wl, bt, lens), dtype, what=f"merge {dtype} {Hq}/{Hkv}/{d}")
