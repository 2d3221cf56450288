"""Pieces of a shared run that a team of waves sweeps, of as many tiles as its ring holds (4 for two waves, 8 for four), one less,
one more, the fewest a team takes, and odd and even numbers: what is asked for ahead, and read ahead, ends with the piece."""
import numpy as np
import pytest

import workloads as W
from gpu_harness import assert_close, oracle_for, run_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hq,Hkv", [(32, 4, 1), (64, 4, 1), (40, 4, 1), (700, 32, 8)])
@pytest.mark.parametrize("tiles", [4, 5, 6, 7, 8, 9, 13, 16, 17])
def test_tiles_around_the_ring(B, Hq, Hkv, tiles):
    wl = W.generate(W.Spec("rings", 90 + tiles, "bf16", Hq, Hkv, 128, ((B, 32 * tiles),), (1, 40)))
    out, bt, lens, info = run_workload(wl)
    assert info["groups"] == 1 and info["grouped_requests"] == B and info["overflow"] == 0 and info["shared_blocks"] == 2 * tiles
    rows = list(range(0, B, max(1, B // 64)))
    assert_close(out, oracle_for(wl, bt, lens, requests=rows), "bf16", rows=rows, what=f"B={B} {tiles} tiles")
    assert np.isfinite(out).all()
