"""GPU parity of the grid windows (partitioned windows of more than 2^13
packets) at the sizes and traffic where their kernels change course, against
the CPU oracle and against the path of one link bucket per hash range.

Addresses with chosen hashed forms put packets into chosen cells and buckets.
"""
import numpy as np
import pytest

import oracle
import paper_2509_03653_amd as nsgc
from gpu_util import assert_same, gpu_stats, say
from hashed_addresses import COL, DESTINATION_MARKER, ROW, SOURCE_MARKER, _unmix

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _default_tune():
    nsgc.set_tune(nsgc.default_tune())
    yield
    nsgc.set_tune(nsgc.default_tune())


def hashed(ids, view):
    """The addresses whose hashed forms are `ids`."""
    return _unmix(np.asarray(ids, np.uint64).copy(), *view).astype(np.uint32)


def heavy_tailed(rng, n):
    return (rng.zipf(1.3, n) % (1 << 26)).astype(np.uint32)


def check(windows, what, forms):
    src = np.concatenate([s for s, _ in windows])
    dst = np.concatenate([d for _, d in windows])
    off = np.cumsum([0] + [s.size for s, _ in windows]).astype(np.int64)
    want = oracle.window_stats(src, dst, off, threads=8)
    for form in forms:
        say(f"[gpu] grid {what} form={form} sizes={np.diff(off).tolist()[:12]}")
        assert_same(gpu_stats(src, dst, off, form), want, f"{what}/{form}")


# the rule's first size; tiles of 2^11 .. 2^14 packets; one more strip, cell
# size and group of buckets; windows of big cells beside windows of small ones
@pytest.mark.parametrize("sizes", [
    [8192], [8193], [8193, 300, 8192, 9000],
    [3 * 2048 + 2048 + 1, 16384, 16385], [65535, 65536, 65537],
    [(1 << 18) - 1, 1 << 18], [1 << 19, (1 << 19) + 1], [(1 << 19) - 1, 12345],
    [1300000], [(1 << 20) + 1, 20001], [1800003, 8193, 70001], [1 << 21], [(1 << 22) + 5],
])
def test_sizes(sizes):
    rng = np.random.default_rng(sum(sizes))
    windows = [(heavy_tailed(rng, n), heavy_tailed(rng, n)) for n in sizes]
    check(windows, "heavy-tailed", ("batched", "graph", "noalloc") if sum(sizes) < 1 << 19 else ("batched",))
    few = [(rng.integers(0, 4096, n).astype(np.uint32), rng.integers(0, 4096, n).astype(np.uint32))
           for n in sizes]
    check(few, "even", ("batched",))


# n distinct links whose sources (destinations) share the top `rbits` (`cbits`)
# of their hashed form: overfull cells (the wide pass, rounds) and overfull row
# or column buckets (halved groups, sweeps)
@pytest.mark.parametrize("n,rbits,cbits", [
    (20000, 2, 2), (20000, 6, 0), (20000, 0, 6), (60000, 9, 0), (60000, 0, 9), (60000, 5, 5),
    (600000, 4, 4), (600000, 8, 0), (600000, 0, 8), (2000000, 3, 3),
])
def test_crowded_cells_and_buckets(n, rbits, cbits):
    rng = np.random.default_rng(n + 16 * rbits + cbits)
    r = (rng.integers(0, 1 << (32 - rbits), n)).astype(np.uint64)   # top bits zero
    c = (rng.integers(0, 1 << (32 - cbits), n)).astype(np.uint64)
    top = np.uint64(0xFFFFFFFF)
    check([(hashed(r, ROW), hashed(c, COL)), (hashed(top - r, ROW), hashed(top - c, COL))],
          f"crowded {rbits}/{cbits}", ("batched",))


# dominant addresses: one, fewer and more than are kept per view, one-sided and
# two-sided, of equal and of unequal weight; the tables' marker among them
@pytest.mark.parametrize("n", [9001, 50000, 1400000])
@pytest.mark.parametrize("rows,cols", [(1, 1), (1, 0), (0, 1), (3, 30), (31, 33), (65, 64), (200, 0)])
def test_dominant_addresses(n, rows, cols):
    rng = np.random.default_rng(n + 1000 * rows + cols)
    ids = rng.integers(0, 1 << 32, n, dtype=np.uint64).astype(np.uint32)

    def column(k, marker):
        x = rng.permutation(ids)
        if k:
            hot = rng.random(n) < 0.7
            x[hot] = ids[(rng.integers(0, k, n) * rng.integers(0, 2, n))[hot]]
        x[rng.random(n) < 0.1] = marker
        return x

    check([(column(rows, SOURCE_MARKER), column(cols, DESTINATION_MARKER)) for _ in range(2)],
          f"dominant {rows}x{cols}", ("batched", "graph"))


def test_same_as_one_bucket_per_hash_range():
    # wavefront targets of zero keep every window on the other path
    rng = np.random.default_rng(5)
    sizes = [8193, 10000, 40013, 131072, 700001]
    src = heavy_tailed(rng, sum(sizes))
    dst = heavy_tailed(rng, sum(sizes)) * np.uint32(7)
    off = np.cumsum([0] + sizes).astype(np.int64)
    got = {f: gpu_stats(src, dst, off, f) for f in ("batched", "graph", "plain", "noalloc")}
    t = nsgc.default_tune().to_dict()
    t["cls"] = [c[:3] + [0] for c in t["cls"]]
    nsgc.set_tune(nsgc.Tune.from_dict(t))
    want = gpu_stats(src, dst, off)
    for f, g in got.items():
        assert_same(g, want, f)


def test_graph_replays_between_other_work():
    # one graph, batches with and without grid windows in turn
    rng = np.random.default_rng(6)
    g = nsgc.Graph(400000, 8)
    for sizes in ([131072, 9000, 100], [500, 8192], [300000, 8193], [131072, 9000, 100]):
        src, dst = heavy_tailed(rng, sum(sizes)), heavy_tailed(rng, sum(sizes))
        off = np.cumsum([0] + sizes).astype(np.int64)
        want = oracle.window_stats(src, dst, off, threads=8)
        for k in range(3):
            assert_same(gpu_stats(src, dst, off, "graph", graph=g), want, f"{sizes} replay {k}")
            assert_same(gpu_stats(src, dst, off), want, f"{sizes} batched {k}")
    g.close()


# the large-window tier's two-level grid: its smallest sizes, one more tile,
# range, strip and cell size; what it gives up on is sorted
@pytest.mark.parametrize("n,rbits,cbits", [
    (1 << 20, 0, 0), ((1 << 20) + 1, 0, 0), ((1 << 21) - 3, 0, 0), (2560 << 10, 0, 0), ((2560 << 10) + 1, 0, 0),
    ((2560 << 11) + 16385, 0, 0), ((1 << 24) + 77, 0, 0),
    (1 << 20, 4, 4), ((1 << 20) + 5, 14, 0), (1 << 20, 0, 15), (1 << 20, 10, 10), (3000001, 12, 11),
])
def test_large_windows(n, rbits, cbits):
    t = nsgc.default_tune()
    t.large_min_log2 = 20
    nsgc.set_tune(t)
    rng = np.random.default_rng(n + rbits)
    if rbits or cbits:   # distinct links with shared top bits of their hashed forms
        src = hashed(rng.integers(0, 1 << (32 - rbits), n).astype(np.uint64), ROW)
        dst = hashed(rng.integers(0, 1 << (32 - cbits), n).astype(np.uint64), COL)
    else:
        src, dst = heavy_tailed(rng, n), heavy_tailed(rng, n)
        src[::97], dst[::89] = SOURCE_MARKER, DESTINATION_MARKER
    off = np.array([0, n], np.int64)
    assert int(nsgc.plan_inspect(off)["tier"][0]) == 3
    say(f"[gpu] large grid {n} {rbits}/{cbits}")
    assert_same(gpu_stats(src, dst, off), oracle.window_stats(src, dst, off), f"large {n} {rbits}/{cbits}")


# entity counts on the grid: links of an address with itself, ids that fill one
# bucket (sweeps) or one cell, dominant addresses in one view or both, the
# tables' marker
@pytest.mark.parametrize("n", [1025, 4096, 8193, 50000, 1100000])
@pytest.mark.parametrize("kind", ["loops", "zipf", "crowded", "dominant", "marker", "distinct"])
def test_entity_counts(n, kind):
    import torch
    rng = np.random.default_rng(n)
    ids = rng.integers(0, 1 << 32, n, dtype=np.uint64).astype(np.uint32)
    src, dst = heavy_tailed(rng, n), heavy_tailed(rng, n)
    if kind == "loops":
        dst = np.where(rng.random(n) < 0.7, src, dst)
        src[::3] = ids[::3]
        dst[::3] = ids[::3]
    elif kind == "crowded":
        few = rng.integers(0, 1 << 22, n).astype(np.uint64)   # top ten bits zero, or all ones
        src, dst = hashed(few, ROW), hashed(np.uint64(0xFFFFFFFF) - rng.permutation(few), ROW)
    elif kind == "dominant":
        src = np.where(rng.random(n) < 0.8, ids[rng.integers(0, 40, n)], ids)
        dst = np.where(rng.random(n) < 0.6, ids[20 + rng.integers(0, 90, n)], rng.permutation(ids))
    elif kind == "marker":
        src[::5], dst[::7] = SOURCE_MARKER, SOURCE_MARKER     # (destinations are hashed like sources)
        dst[1::50] = 0xFFFFFFFF
    elif kind == "distinct":
        src, dst = np.arange(n), n // 2 + np.arange(n)
    src, dst = src.astype(np.uint32), dst.astype(np.uint32)
    half = n // 2 + 1
    off = np.array([0, n, n + half], np.int64)
    src, dst = np.concatenate([src, dst[:half]]), np.concatenate([dst, src[:half]])
    want = []
    for a, b in zip(off[:-1], off[1:]):
        e = oracle.window_entities(src, dst, int(a), int(b))
        want.append([len(e["link_keys"]), len(e["row_ids"]), len(e["col_ids"]), e["unique_ips"]])
    say(f"[gpu] entity counts {kind} n={n}")
    s, d = (torch.from_numpy(x.view(np.int32)).cuda() for x in (src, dst))
    got = nsgc.window_entity_counts(s, d, off)
    torch.cuda.synchronize()
    assert got.cpu().numpy().tolist() == want
