"""The bounds that reservations and graphs are sized from: enough for every batch
of at most as many packets and windows, and not many times what a batch takes."""
import numpy as np
import pytest

import paper_2509_03653_amd as nsgc


@pytest.fixture(autouse=True)
def _default_tune():
    before = nsgc.get_tune()
    nsgc.set_tune(nsgc.default_tune())
    yield
    nsgc.set_tune(before)


def sizes_of(windows):
    return nsgc.plan_sizes(np.concatenate([[0], np.cumsum(windows)]).astype(np.int64))


@pytest.mark.parametrize("windows", [[8193], [40013], [1 << 17], [1 << 20], [1 << 22], [20000] * 10, [1 << 17] * 8])
def test_bounds_are_not_many_times_the_plan(windows):
    # (before the grid windows 1.02 to 1.2 and, for many equal windows, 4 times)
    s = sizes_of(windows)
    assert s["workspace_bound"] <= (2 if len(windows) == 1 else 5) * s["workspace_bytes"], s


@pytest.mark.parametrize("knobs", [
    {}, {"tile_log2": 11}, {"cls": [[16384, 16384, 16384, 64]] * 33, "max_link_buckets_log2": 12},
    {"cls": [[16384, 16384, 16384, 64]] * 33, "small_max": 0}, {"small_max": 2048, "max_link_buckets_log2": 10},
])
def test_bounds_cover_smaller_batches(knobs):
    nsgc.set_tune(nsgc.Tune.from_dict(dict(nsgc.default_tune().to_dict(), **knobs)))
    rng = np.random.default_rng(5)
    for trial in range(150):
        w = int(rng.choice([1, 2, 3, 4, 8, 30, 300]))
        windows = (np.floor(2.0 ** rng.uniform(9, 22, w)) if trial % 2 else
                   np.full(w, 2 ** int(rng.integers(11, 20)) + 1)).astype(np.int64)
        bound = sizes_of(windows)
        for _ in range(4):   # fewer windows, cut down or joined
            part = windows[rng.random(w) < rng.random()]
            part = part // int(rng.integers(1, 40))
            if trial % 3 == 0 and part.size:
                part = np.array([part.sum()], np.int64)
            s = sizes_of(part)
            assert s["plan_bytes"] <= bound["plan_bound"], (windows[:5], part[:5], s, bound)
            assert s["workspace_bytes"] <= bound["workspace_bound"], (windows[:5], part[:5], s, bound)
