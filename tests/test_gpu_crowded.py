"""Windows whose traffic was made to fall into one cell of the grid: many links,
links of many packets, the tables' marker and a dominant address in it, against
the CPU oracle; and that such a window takes time in proportion to its packets."""
import time

import numpy as np
import pytest

import oracle
import paper_2509_03653_amd as nsgc
from gpu_util import assert_same, gpu_stats, say, to_gpu
from hashed_addresses import COL, DESTINATION_MARKER, ROW, SOURCE_MARKER, _unmix

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _default_tune():
    nsgc.set_tune(nsgc.default_tune())
    yield
    nsgc.set_tune(nsgc.default_tune())


def hashed(ids, view):
    return _unmix(np.asarray(ids, np.uint64).copy(), *view).astype(np.uint32)


def last_cell(rng, n):
    """Links whose hashed addresses' top nine bits are ones."""
    low = lambda: rng.integers(0, 1 << 23, n).astype(np.uint64) | np.uint64(0xFF800000)
    return hashed(low(), ROW), hashed(low(), COL)


def check(src, dst, what, forms=("batched",)):
    perm = np.random.default_rng(1).permutation(src.size)
    src, dst = src[perm], dst[perm]
    off = np.array([0, src.size], np.int64)
    want = oracle.window_stats(src, dst, off)
    for form in forms:
        say(f"[gpu] crowded {what} n={src.size} {form}")
        assert_same(gpu_stats(src, dst, off, form), want, f"{what}/{form}")


# from what the single passes and a few rounds take to what is sorted
@pytest.mark.parametrize("n", [9000, 12289, 30000, 40000, 65536, 65537, 70001, 300000, 1100000])
@pytest.mark.parametrize("repeat", [1, 3])
def test_links_of_one_cell(n, repeat):
    rng = np.random.default_rng(n)
    src, dst = last_cell(rng, n)
    pick = np.arange(n) // repeat
    check(src[pick], dst[pick], f"x{repeat}", ("batched", "graph"))


# a link of more packets than an entry holds, the link that equals the tables'
# marker, in a cell that is sorted
@pytest.mark.parametrize("packets", [1, 524287, 524288, 1048575])
def test_heavy_and_marker_links(packets):
    rng = np.random.default_rng(packets)
    src, dst = last_cell(rng, 100000)
    for s, d in ((SOURCE_MARKER, DESTINATION_MARKER), (SOURCE_MARKER, int(dst[0])), (int(src[1]), int(dst[1]))):
        check(np.concatenate([src, np.full(packets, s, np.uint32)]),
              np.concatenate([dst, np.full(packets, d, np.uint32)]), f"{packets} packets of a link")


# a dominant source (destination) whose links, moved off its strip, meet in one
# cell: the other address decides by how much, from its bits 3 .. 18
@pytest.mark.parametrize("view", [0, 1])
@pytest.mark.parametrize("n", [20000, 250000])
def test_dominant_address_in_one_cell(n, view):
    rng = np.random.default_rng(n + view)
    other = (np.uint64(0xF8000000) | (rng.integers(0, 256, n).astype(np.uint64) << np.uint64(19))
             | (rng.integers(0, 1000, n).astype(np.uint64) << np.uint64(3)) | rng.integers(0, 8, n).astype(np.uint64))
    hot = hashed([0x12345678], ROW if view == 0 else COL)[0]
    cols = [np.full(n, hot, np.uint32), hashed(other, COL if view == 0 else ROW)]
    more = rng.integers(0, 1 << 32, (2, n // 2), dtype=np.uint64).astype(np.uint32)
    check(np.concatenate([cols[view], more[0]]), np.concatenate([cols[1 - view], more[1]]),
          f"dominant {view}", ("batched", "graph"))


def test_entity_counts_of_one_cell():
    rng = np.random.default_rng(3)
    low = lambda: rng.integers(0, 1 << 23, 200000).astype(np.uint64) | np.uint64(0xFF800000)
    src, dst = hashed(low(), ROW), hashed(low(), ROW)   # (destinations are hashed like sources)
    e = oracle.window_entities(src, dst, 0, src.size)
    say("[gpu] entity counts of one cell")
    got = nsgc.window_entity_counts(to_gpu(src), to_gpu(dst), np.array([0, src.size], np.int64))
    assert got.cpu().numpy().tolist() == [[len(e["link_keys"]), len(e["row_ids"]), len(e["col_ids"]),
                                           e["unique_ips"]]]


def test_time_of_a_crowded_window():
    # 2 * 10^6 links in one of the window's 2048 cells, a thousand times what a
    # cell is made for: 0.41 s with one link bucket per hash range.  Reading the
    # cell once per table of links took 12.8 s.
    import torch
    n = 2000000
    rng = np.random.default_rng(9)
    src = hashed(rng.integers(0, 1 << 26, n).astype(np.uint64), ROW)
    dst = hashed(rng.integers(0, 1 << 27, n).astype(np.uint64), COL)
    s, d, off = to_gpu(src), to_gpu(dst), np.array([0, n], np.int64)
    say(f"[gpu] time of {n} links in one cell")
    out = nsgc.window_stats(s, d, off)
    torch.cuda.synchronize()
    t = time.perf_counter()
    nsgc.window_stats(s, d, off, out=out)
    torch.cuda.synchronize()
    t = time.perf_counter() - t
    say(f"[gpu] {t:.3f} s")
    assert_same(out.cpu().numpy().view(np.uint64), oracle.window_stats(src, dst, off), "timed")
    assert t < 0.41
