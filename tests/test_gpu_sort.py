"""GPU parity of the anonymization at the edges of its tiles (2^14 entries of a
column), of the sort's tiles and ranges (2048 and 8192 keys, 512 ranges) and of
its two scatter forms, against the CPU oracle."""
import numpy as np
import pytest

from test_gpu_anonymize import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["distinct", "few", "extreme"])
@pytest.mark.parametrize("n", [1, 63, 64, 1023, 1024, 1025, 2048, 4097, 16383, 16384, 16385, 40000,
                               (1 << 19) - 1, (1 << 19) + 1, 1300007])
def test_anonymize_edges(n, kind):
    rng = np.random.default_rng(n)
    if kind == "distinct":       # as many distinct addresses as entries: the fullest tables and lists
        x = rng.permutation(2 * n).astype(np.uint64) * np.uint64(2147483659 // (2 * n) + 1) & np.uint64(0xFFFFFFFF)
        src, dst = x[:n], x[n:]
    elif kind == "few":
        src, dst = rng.integers(0, 7, n), rng.integers(3, 3000, n)
    else:                        # the tables' free mark, zero, and neighbours that differ in one byte
        pool = np.array([0, 0xFFFFFFFF, 0xFFFFFFFE, 0xFFFFFF, 0x100, 0x10000, 0x1000000, 0x80000000])
        src, dst = pool[rng.integers(0, 8, n)], pool[rng.integers(1, 5, n)]
    src, dst = src.astype(np.uint32), dst.astype(np.uint32)
    check(src, dst, n, f"{kind} {n}")
    check(src, dst, n + 1, f"{kind} {n} in place", in_place=True)
