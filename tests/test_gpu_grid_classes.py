"""Grid windows at the sizes where their phase B changes kernels: more packets per
cell than one kernel's threads hold, more tiles than it has threads.  Against the
CPU oracle, and in time."""
import time

import numpy as np
import pytest

import oracle
import paper_2509_03653_amd as nsgc
from gpu_util import assert_same, gpu_stats, say, to_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _default_tune():
    nsgc.set_tune(nsgc.default_tune())
    yield
    nsgc.set_tune(nsgc.default_tune())


def tuned(**knobs):
    nsgc.set_tune(nsgc.Tune.from_dict(dict(nsgc.default_tune().to_dict(), **knobs)))


def few(rng, n):
    return rng.integers(0, 4096, n).astype(np.uint32)


def heavy_tailed(rng, n):
    return (rng.zipf(1.3, n) % (1 << 26)).astype(np.uint32)


@pytest.mark.parametrize("sizes,form,knobs", [
    ([1 << 23], "batched", {}), ([(1 << 23) + 1, 9000], "batched", {}),
    ([(1 << 24) - 1], "batched", {}), ([(1 << 24) + 1], "graph", {}),
    ([1 << 22, (1 << 22) + 1, 1311744, 1311745], "batched", dict(max_link_buckets_log2=10)),
    ([(1 << 20) + 1, 1 << 19, (1 << 19) + 1], "batched", dict(tile_log2=11)),
    ([3000000, 200000], "batched", dict(max_link_buckets_log2=4)),
])
@pytest.mark.parametrize("draw", [few, heavy_tailed])
def test_classes(sizes, form, knobs, draw):
    rng = np.random.default_rng(sum(sizes))
    n = sum(sizes)
    src, dst = draw(rng, n), draw(rng, n)
    off = np.cumsum([0] + sizes).astype(np.int64)
    say(f"[gpu] grid classes {sizes} {form} {knobs} {draw.__name__}")
    tuned(**knobs)
    assert_same(gpu_stats(src, dst, off, form), oracle.window_stats(src, dst, off, threads=8), f"{sizes}")


@pytest.mark.parametrize("draw", [few, heavy_tailed])
def test_entity_counts_above_two_to_the_24(draw):
    rng = np.random.default_rng(24)
    n = (1 << 24) + 1
    src, dst = draw(rng, n), draw(rng, n)
    say(f"[gpu] entity counts {n} {draw.__name__}")
    got = nsgc.window_entity_counts(to_gpu(src), to_gpu(dst), np.array([0, n], np.int64))
    key = np.unique((src.astype(np.uint64) << np.uint64(32)) | dst)
    s, d = np.unique(src), np.unique(dst)
    assert got.cpu().numpy().tolist() == [[key.size, s.size, d.size, np.union1d(s, d).size]]


def seconds(call, repeat=5):
    import torch
    call()
    best = 1e9
    for _ in range(repeat):
        torch.cuda.synchronize()
        t = time.perf_counter()
        call()
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    return best


def test_time_of_small_tiles():
    # 512 tiles of 2^11 packets in each window, twice the threads of the kernel
    # for small cells: 2.2 times the time of 2^13-packet tiles when every cell was
    # left over for it, 1.0 with tiles that fit.
    rng = np.random.default_rng(1)
    s, d = to_gpu(heavy_tailed(rng, 1 << 23)), to_gpu(heavy_tailed(rng, 1 << 23))
    off = np.arange(9, dtype=np.int64) << 20
    t = {}
    for tile in (13, 11):
        tuned(tile_log2=tile)
        t[tile] = seconds(lambda: nsgc.window_stats(s, d, off))
        say(f"[gpu] tile_log2 {tile}: {t[tile] * 1e6:.0f} us")
    assert t[11] < 1.5 * t[13]


def test_time_per_packet_of_a_graph_window():
    # 2^24 + 1 packets are 1025 tiles: every cell was left over twice and took 2.5
    # times as long per packet as in a window of 2^23; 1.2 times in turns of 1024.
    rng = np.random.default_rng(2)
    n = (1 << 24) + 1
    s, d = to_gpu(few(rng, n)), to_gpu(few(rng, n))
    t = {}
    for m in (1 << 23, n):
        g = nsgc.Graph(m, 1)
        t[m] = seconds(lambda: g.launch(s, d, np.array([0, m], np.int64)))
        say(f"[gpu] graph window of {m} packets: {t[m] * 1e6:.0f} us")
        g.close()
    assert t[n] / n < 1.7 * t[1 << 23] / (1 << 23)
