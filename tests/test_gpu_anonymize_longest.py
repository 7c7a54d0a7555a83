"""The longest anonymization there is: 2^31 - 1 packets whose 2^32 - 2 addresses
are all distinct, so that the sorted list of the tiles' distinct addresses
reaches its greatest length.  Every address below 2^32 - 2 occurs, so an
address is its own rank and must come out as the permutation's value of it; the
values of both columns are checked to be a permutation by their sum and sum of
squares."""
import random

import pytest

import oracle
from gpu_util import say

pytestmark = pytest.mark.gpu


def test_all_addresses_distinct():
    import torch

    import paper_2509_03653_amd as nsgc
    n, seed = (1 << 31) - 1, 0x1234567
    say(f"[gpu] anonymize {n} packets, all addresses distinct")
    # sources 0 .. n - 1, destinations n .. 2 n - 1, as 32-bit patterns
    src = torch.arange(n, dtype=torch.int32, device="cuda")
    dst = torch.empty_like(src)
    dst[0] = n
    torch.arange(-(1 << 31), -(1 << 31) + n - 1, dtype=torch.int32, device="cuda", out=dst[1:])
    _, _, num = nsgc.anonymize(src, dst, seed, out_src=src, out_dst=dst)
    N = 2 * n
    assert int(num[0]) == N
    total = squares = 0
    for col in (src, dst):
        for i in range(0, n, 1 << 27):
            v = col[i:i + (1 << 27)].long() & 0xFFFFFFFF
            total += int(v.sum())
            squares += int((v * v).sum())
    assert total == N * (N - 1) // 2
    assert (squares - (N - 1) * N * (2 * N - 1) // 6) % (1 << 64) == 0
    rng = random.Random(4)
    for a in [0, 1, 511, 512, n - 1, n, n + 1, N - 512, N - 2, N - 1] + [rng.randrange(N) for _ in range(200)]:
        col, i = (src, a) if a < n else (dst, a - n)
        assert int(col[i]) & 0xFFFFFFFF == oracle.permute(a, N, seed), a
    del src, dst
    nsgc.release()
    torch.cuda.empty_cache()
