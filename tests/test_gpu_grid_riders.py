"""Short windows that ride along with grid windows, at the edges of the rule,
against the CPU oracle; and that they cost no launch of their own."""
import time

import numpy as np
import pytest

import oracle
import paper_2509_03653_amd as nsgc
from gpu_util import assert_same, gpu_stats, say, to_gpu
from hashed_addresses import DESTINATION_MARKER, SOURCE_MARKER

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _default_tune():
    nsgc.set_tune(nsgc.default_tune())
    yield
    nsgc.set_tune(nsgc.default_tune())


def packets(rng, n):
    src, dst = (rng.zipf(1.3, n) % (1 << 30)).astype(np.uint32), rng.integers(0, 5000, n).astype(np.uint32)
    src[::61], dst[::43] = SOURCE_MARKER, DESTINATION_MARKER
    return src, dst


# all ride; a shorter or an empty window keeps the launch and the 4096 packets
# and less with it; as many as may ride and one more; beside larger cells
@pytest.mark.parametrize("sizes", [
    [1025, 8193], [8193, 2047, 2048, 2049, 4095, 4096, 4097, 8192], [1024, 8193, 1025, 4097],
    [0, 8193, 1025], [8193] + [1100] * 256, [8193] + [1100] * 257, [8193] + [4097] * 250 + [2000] * 7,
    [1500000, 1300, 3000], [1 << 21, 5000, 2000],
    # fewer row buckets than items for the dominant addresses
    [1 << 21, 9282, 17342, 40013],
])
@pytest.mark.parametrize("small_max", [1024, 2048])
def test_riders(sizes, small_max):
    t = nsgc.default_tune()
    t.small_max = small_max
    nsgc.set_tune(t)
    src, dst = packets(np.random.default_rng(len(sizes)), sum(sizes))
    off = np.cumsum([0] + sizes).astype(np.int64)
    want = oracle.window_stats(src, dst, off, threads=8)
    for form in ("batched", "graph", "noalloc", "plain"):
        say(f"[gpu] riders {sizes[:9]} {small_max} {form}")
        assert_same(gpu_stats(src, dst, off, form), want, f"{sizes[:9]}/{form}")


def test_time_of_a_mixed_batch():
    # Seven windows of 1947 .. 22721 packets took 60 us with a launch for the
    # shorter ones in front, 48 as link buckets and 42 with all on the grid; the
    # longer ones alone take about 40.
    import torch
    sizes = [9000, 12000, 22000, 2000, 2600, 5000, 6000]
    src, dst = packets(np.random.default_rng(7), sum(sizes))
    s, d = to_gpu(src), to_gpu(dst)
    out = torch.empty((7, 9), dtype=torch.int64, device="cuda")
    t = []
    for w in (3, 7):
        off = np.cumsum([0] + sizes[:w]).astype(np.int64)
        best = 1e9
        for _ in range(10):
            torch.cuda.synchronize()
            start = time.perf_counter()
            for _ in range(50):
                nsgc.window_stats(s, d, off, out=out[:w])
            torch.cuda.synchronize()
            best = min(best, (time.perf_counter() - start) / 50)
        say(f"[gpu] {w} windows: {best * 1e6:.1f} us")
        t.append(best)
    assert t[1] < 1.25 * t[0]
