"""Fixed-scratch batches near the limit: with grid windows up to the size where
their workspace still fits, without them from there to the form's own limit,
refused above; against the CPU oracle."""
import numpy as np
import pytest

import oracle
import paper_2509_03653_amd as nsgc
from gpu_util import assert_same, gpu_stats, say

pytestmark = pytest.mark.gpu

ROOM = nsgc.NOALLOC_SCRATCH_BYTES - nsgc.NOALLOC_PLAN_BYTES


# (windows, the most of them that fit one link bucket per hash range)
@pytest.mark.parametrize("window,before", [(9000, 599), (20000, 267), (1 << 17, 39), (1 << 20, 5)])
def test_up_to_the_limit(window, before):
    nsgc.set_tune(nsgc.default_tune())
    rng = np.random.default_rng(window)
    grid = max(n for n in range(4_900_000 // window, 5_700_000 // window)   # the most that fit the grid
               if nsgc.plan_sizes(np.arange(n + 1, dtype=np.int64) * window)["workspace_bytes"] <= ROOM)
    src = (rng.zipf(1.3, 6_400_000) % (1 << 26)).astype(np.uint32)
    dst = (rng.zipf(1.2, 6_400_000) % (1 << 26)).astype(np.uint32)
    for n in sorted({grid, min(grid + 1, max(grid, before)), max(grid, before)}):
        off = np.arange(n + 1, dtype=np.int64) * window
        say(f"[gpu] fixed scratch {n} x {window}: {nsgc.plan_sizes(off)['workspace_bytes']} of {ROOM}")
        assert_same(gpu_stats(src, dst, off, "noalloc"), oracle.window_stats(src, dst, off, threads=8),
                    f"{n} x {window}")
    with pytest.raises(nsgc.NsgcError, match="fit"):
        gpu_stats(src, dst, np.arange(5_700_000 // window + 2, dtype=np.int64) * window, "noalloc")
