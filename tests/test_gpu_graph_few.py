"""Graph launches of a few short windows, which take one kernel and no replay,
between replays and on two streams, against the CPU oracle."""
import numpy as np
import pytest

import oracle
import paper_2509_03653_amd as nsgc
from gpu_util import assert_same, say, to_gpu

pytestmark = pytest.mark.gpu


def test_few_windows_between_replays():
    import torch
    nsgc.set_tune(nsgc.default_tune())
    rng = np.random.default_rng(12)
    batches = [[7, 1, 21], [0, 0], [131072, 9000], [8192], [300] * 224, [300] * 225, [5, 20000], [1], [700, 90, 4000]]
    cols = []
    for sizes in batches:
        n = sum(sizes)
        cols.append((rng.integers(0, 700, n).astype(np.uint32), rng.integers(0, 90, n).astype(np.uint32),
                     np.cumsum([0] + sizes).astype(np.int64)))
    want = [oracle.window_stats(s, d, off) for s, d, off in cols]
    dev = [(to_gpu(s), to_gpu(d), off) for s, d, off in cols]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    g = nsgc.Graph(150000, 256)
    outs = []
    order = [int(x) for x in rng.integers(0, len(batches), 60)]
    say(f"[gpu] graph launches of few windows between replays: {order[:12]}")
    for k, i in enumerate(order):
        s, d, off = dev[i]
        outs.append(g.launch(s, d, off, stream=streams[(k // 3) % 2]))
    torch.cuda.synchronize()
    g.close()
    for k, (i, out) in enumerate(zip(order, outs)):
        assert_same(out.cpu().numpy().view(np.uint64), want[i], f"launch {k}: {batches[i][:4]}")
