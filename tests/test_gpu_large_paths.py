"""Which way the windows of the large tier take: hash partitioning for ordinary
traffic of every size it is made for, sorting for windows whose addresses were
chosen to crowd a cell or a bucket and for those out of its range."""
import numpy as np
import pytest

import oracle
import paper_2509_03653_amd as nsgc
from gpu_util import assert_same, gpu_stats, say
from hashed_addresses import COL, ROW, _unmix

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _tune():
    t = nsgc.default_tune()
    t.large_min_log2 = 20
    nsgc.set_tune(t)
    yield
    nsgc.set_tune(nsgc.default_tune())


def taken(src, dst, what, form="batched"):
    off = np.array([0, src.size], np.int64)
    before = nsgc.large_window_counts()
    say(f"[gpu] large window {what} {src.size} {form}")
    assert_same(gpu_stats(src, dst, off, form), oracle.window_stats(src, dst, off), what)
    after = nsgc.large_window_counts()
    return after["grid"] - before["grid"], after["sorting"] - before["sorting"]


def even(rng, n):
    return rng.integers(0, 1 << 32, n, dtype=np.uint64).astype(np.uint32)


def few(rng, n):
    return rng.integers(0, 4096, n).astype(np.uint32)


def heavy_tailed(rng, n):
    return (rng.zipf(1.3, n) % (1 << 26)).astype(np.uint32)


@pytest.mark.parametrize("draw", [even, few, heavy_tailed])
@pytest.mark.parametrize("n", [1 << 20, (1 << 20) + 16385, (2560 << 10) + 1, 5000011])
def test_ordinary_traffic_is_partitioned(n, draw):
    rng = np.random.default_rng(n)
    assert taken(draw(rng, n), draw(rng, n), draw.__name__) == (1, 0)


def test_links_of_many_packets():
    # a hundred links of 3.4 * 10^5 packets each, more of them than there are
    # dominant addresses: cells of a few links and very many keys
    n = (1 << 25) + 3
    i = (np.arange(n) % 100).astype(np.uint32)
    assert taken(i * np.uint32(7), i + np.uint32(5000), "a hundred links") == (1, 0)


def test_fixed_scratch_and_plain_forms():
    rng = np.random.default_rng(1)
    src, dst = heavy_tailed(rng, 1 << 20), heavy_tailed(rng, 1 << 20)
    for form in ("noalloc", "plain"):
        assert taken(src, dst, "heavy-tailed", form) == (1, 0)


# distinct links that share the top bits of their hashed forms
@pytest.mark.parametrize("n,rbits,cbits", [(1 << 20, 10, 10), (3000001, 12, 11), (1 << 20, 15, 0), (1 << 20, 0, 15)])
def test_crowded_windows_are_sorted(n, rbits, cbits):
    rng = np.random.default_rng(n + rbits)
    ids = lambda bits, view: _unmix(rng.integers(0, 1 << (32 - bits), n).astype(np.uint64), *view).astype(np.uint32)
    assert taken(ids(rbits, ROW), ids(cbits, COL), f"crowded {rbits}/{cbits}") == (0, 1)
