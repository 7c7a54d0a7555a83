"""GPU parity of the windows that one workgroup takes whole, at the edges of
its three sizes, against the CPU oracle and against the partitioned kernels."""
import numpy as np
import pytest

import oracle
import paper_2509_03653_amd as nsgc
from gpu_util import assert_same, gpu_stats, say
from hashed_addresses import DESTINATION_MARKER, SOURCE_MARKER

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 2, 31, 32, 33, 63, 64, 65, 255, 256, 257, 511, 513, 2047, 2048, 2049, 4095, 4097,
         6143, 6144, 6145, 8191, 8192, 8193]


@pytest.fixture(autouse=True)
def _default_tune():
    nsgc.set_tune(nsgc.default_tune())
    yield
    nsgc.set_tune(nsgc.default_tune())


# distinct links (the fullest tables), one link, few addresses, the tables'
# markers, heavy-tailed
@pytest.mark.parametrize("kind", ["distinct", "one", "few", "markers", "zipf"])
@pytest.mark.parametrize("small_max", [1024, 2048, 1, 0])
def test_edges(kind, small_max):
    t = nsgc.default_tune()
    t.small_max = small_max
    nsgc.set_tune(t)
    rng = np.random.default_rng(7)
    off = np.cumsum([3] + EDGES + [700] * 300 + [100] * 300).astype(np.int64)
    n = int(off[-1])
    src, dst = {
        "distinct": lambda: (rng.permutation(n), rng.permutation(n)),
        "one": lambda: (np.full(n, 77), np.full(n, 78)),
        "few": lambda: (rng.integers(0, 9, n), rng.integers(0, 5, n)),
        "markers": lambda: (np.where(rng.random(n) < 0.5, SOURCE_MARKER, rng.integers(0, 40, n)),
                            np.where(rng.random(n) < 0.5, DESTINATION_MARKER, rng.integers(0, 3000, n))),
        "zipf": lambda: (rng.zipf(1.3, n) % (1 << 30), rng.zipf(1.2, n) % (1 << 30)),
    }[kind]()
    src, dst = src.astype(np.uint32), dst.astype(np.uint32)
    want = oracle.window_stats(src, dst, off, threads=8)
    for form in ("batched", "graph", "plain", "noalloc"):
        say(f"[gpu] whole windows {kind} small_max={small_max} {form}")
        assert_same(gpu_stats(src, dst, off, form), want, f"{kind}/{small_max}/{form}")


# plans around the sizes where their way to the device changes: windows in the
# launch's arguments (up to 224 of one size), plans of up to 3840 and 4 * 3840
# bytes and longer, with and without a grid window; one graph for all of them
@pytest.mark.parametrize("grid", [0, 8193, 140000])
def test_plan_sizes(grid):
    rng = np.random.default_rng(grid)
    g = nsgc.Graph(600000, 2600)
    for windows in (1, 2, 223, 224, 225, 120, 200, 215, 890, 940, 960, 1700, 2500):
        off = np.cumsum([0] + [grid] * (grid > 0) + rng.integers(0, 300, windows).tolist()).astype(np.int64)
        n = int(off[-1])
        src = (rng.zipf(1.3, n) % (1 << 30)).astype(np.uint32)
        dst = (rng.zipf(1.3, n) % (1 << 30)).astype(np.uint32)
        want = oracle.window_stats(src, dst, off, threads=8)
        say(f"[gpu] plan of {windows} windows beside {grid}: {nsgc.plan_sizes(off)['plan_bytes']} bytes")
        assert_same(gpu_stats(src, dst, off, "graph", graph=g), want, f"{windows}/{grid}/graph")
        for form in ("batched", "noalloc", "batched", "noalloc"):
            assert_same(gpu_stats(src, dst, off, form), want, f"{windows}/{grid}/{form}")
    g.close()
