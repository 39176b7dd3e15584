"""Host only: the bins that the decode launch sorts scores into, compiled for the host from the kernels' header."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2408_07092_amd", "csrc")

SOURCE = r"""
#define __host__
#define __device__
#include "ds_bins.h"
using namespace ds;

// Walks all scores of one sign and magnitude of the label query in ascending order, 2^16 at a time: bins must not
// decrease, and the keys of a bin must begin and end where its scores do.  0, or the line that failed.
extern "C" int check(uint32_t magnitude, int neg)
{
    const BinScale s((int)magnitude);
    uint32_t last = 0, last_hi = 0;
    for (uint32_t i = 0; i < 0x8000; ++i) {
        const uint32_t x = neg ? 0x7fff - i : i, side = s.bin(x << 16 | 0x1234), bin = neg ? kSideBins - 1 - side : kSideBins + side;
        uint32_t lo, hi;
        if (side >= kSideBins) return __LINE__;
        s.keys(bin, lo, hi);
        const uint32_t k0 = neg ? ~(0x80000000u | x << 16 | 0xffff) : (0x80000000u | x << 16);
        const uint32_t k1 = neg ? ~(0x80000000u | x << 16) : (0x80000000u | x << 16 | 0xffff);
        if (k0 < lo || k1 > hi) return __LINE__;
        if (i == 0 && lo != k0) return __LINE__;
        if (i == 0x7fff && hi != k1) return __LINE__;
        if (i && bin != last && (bin < last || lo != last_hi + 1 || lo != k0)) return __LINE__;
        last = bin;
        last_hi = hi;
    }
    return 0;
}

extern "C" void bins(const uint32_t *scores, int n, uint32_t magnitude, uint32_t *out)
{
    const BinScale s((int)magnitude);
    for (int i = 0; i < n; ++i) out[i] = scores[i] >> 31 ? kSideBins - 1 - s.bin(scores[i]) : kSideBins + s.bin(scores[i]);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("bins")
    (d / "bins.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-O2", "-shared", "-fPIC", "-I", CSRC, "-o", str(d / "bins.so"), str(d / "bins.cpp")], check=True)
    lib = ctypes.CDLL(str(d / "bins.so"))
    lib.check.argtypes = [ctypes.c_uint32, ctypes.c_int]
    lib.bins.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_uint32, ctypes.c_void_p]
    return lib


def test_bins_are_ordered_and_hold_the_keys_that_they_say(lib):
    """For every exponent that the label query's largest value can have, and both signs."""
    for e in range(256):
        for neg in (0, 1):
            assert lib.check(e << 23 | 0x345678, neg) == 0, (e, neg)


@pytest.mark.parametrize("share", [8, 16, 32])
@pytest.mark.parametrize("scale", [2.0 ** e for e in range(-24, 17, 2)])
def test_few_keys_share_the_threshold_bin_whatever_their_scale(lib, scale, share):
    """Scores of normally distributed keys: the k-th largest one's bin holds less than a 400th of the tokens where the
    label channels of K are of ordinary size, and less than a 60th at any other scale that fp16 has."""
    n = 65536
    s = (np.random.default_rng(5).standard_normal(n) * scale * 2.0).astype(np.float32)
    out = np.empty(n, np.uint32)
    lib.bins(s.ctypes.data, n, int(np.float32(1.0).view(np.uint32)), out.ctypes.data)
    order = np.argsort(-s, kind="stable")
    assert (np.diff(out[order].astype(np.int64)) <= 0).all()
    held = int((out == out[order[n // share - 1]]).sum())
    assert held < n // (400 if 0.125 <= scale <= 32 else 60), held
