"""The ranges in which the device-wide sort and the anonymization deal a list to
workgroups (csrc/nsgc_ranges.hpp, compiled here for the CPU), up to the longest
list: every element of both columns of 2^31 - 1 packets distinct."""
import ctypes
import os
import subprocess

import pytest

from conftest import ROOT

CODE = """
#include "nsgc_ranges.hpp"
extern "C" void range_of(uint64_t n, uint32_t step, uint32_t parts, uint32_t part, uint64_t* out) {
  const nsgc::ListRange r = nsgc::list_range(n, step, parts, part);
  out[0] = r.beg;
  out[1] = r.end;
}
"""


@pytest.fixture(scope="module")
def range_of(tmp_path_factory):
    d = tmp_path_factory.mktemp("ranges")
    (d / "r.cpp").write_text(CODE)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I",
                           os.path.join(ROOT, "paper_2509_03653_amd", "csrc"),
                           str(d / "r.cpp"), "-o", str(d / "r.so")])
    lib = ctypes.CDLL(str(d / "r.so"))
    lib.range_of.argtypes = [ctypes.c_uint64] + [ctypes.c_uint32] * 3 + [ctypes.c_void_p]

    def call(n, step, parts, part):
        out = (ctypes.c_uint64 * 2)()
        lib.range_of(n, step, parts, part, out)
        return int(out[0]), int(out[1])
    return call


@pytest.mark.parametrize("step", [512, 2048, 8192])
@pytest.mark.parametrize("n", [1, 511, 512, 513, 512 * 512, 512 * 512 + 1, 10 ** 6 + 7, (1 << 31) - 1,
                               (1 << 32) - 8192, (1 << 32) - 513, (1 << 32) - 512, (1 << 32) - 511,
                               (1 << 32) - 2, (1 << 32) - 1])
def test_ranges_cover_the_list_in_order(range_of, n, step):
    parts = min(-(-n // step), 512)
    at, longest = 0, 0
    for part in range(parts):
        beg, end = range_of(n, step, parts, part)
        assert beg == at and end >= beg, (n, step, part)
        assert end == n or (end - beg) % step == 0
        at, longest = end, max(longest, end - beg)
    assert at == n
    assert longest <= (-(-n // step) + parts - 1) // parts * step   # no range above its share
