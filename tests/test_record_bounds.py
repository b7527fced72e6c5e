"""Which words of a record a receiver reads (csrc/record_bounds.h), whatever the ranks of a corrupt bitmap are: all of them lie in the
record.  On the host, with the records that the library itself lays out."""
import ctypes
import os
import subprocess

import pytest

from paper_1811_08596_amd import fftsp

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#include "%s/paper_1811_08596_amd/csrc/record_bounds.h"
// 0, or 1 + the first bit position whose reads leave the record of S bytes
extern "C" uint64_t outside(uint32_t S, uint32_t W, uint32_t k, const int* windows, int n, uint32_t most)
{
    const int last = fftsp::last_code_word(S, W), end = (int)(S / 4), codes = 4 + (int)W;
    auto in = [&](int word) { return codes + word >= 0 && codes + word < end; };
    for (uint64_t b = 0; b <= (uint64_t)most; ++b) {
        // every position around the codes' end, and steps through what lies beyond
        if (b > 64ull * (uint64_t)(last + 40) && (b %% 977)) continue;
        for (int i = 0; i < n; ++i) {
            const int first = fftsp::window_first((uint32_t)b, last, windows[i]);
            if (!in(first) || !in(first + windows[i] - 1)) return 1 + b;
        }
        if (k == 0) continue;
        const int word = fftsp::code_word((uint32_t)b, last);
        if (word < 0 || !in(word) || !in(fftsp::word_after(word, last))) return 1 + b;
        if ((b >> 5) <= (uint64_t)last && word != (int)(b >> 5)) return 1 + b;  // codes that are there are the ones read
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("bounds")
    (d / "bounds.cpp").write_text(SOURCE % ROOT)
    subprocess.run(["g++", "-O2", "-shared", "-fPIC", "-std=c++17", "-o", str(d / "bounds.so"), str(d / "bounds.cpp")], check=True)
    f = ctypes.CDLL(str(d / "bounds.so")).outside
    f.restype = ctypes.c_uint64
    f.argtypes = [ctypes.c_uint32] * 3 + [ctypes.POINTER(ctypes.c_int), ctypes.c_int, ctypes.c_uint32]
    return f


@pytest.mark.parametrize("bits", (3, 8, 9, 15, 16, 32))
@pytest.mark.parametrize("logL", (16, 17, 19, 22))
def test_reads_stay_in_the_record(lib, logL, bits):
    L, bins = 1 << logL, (1 << logL >> 1) + 1
    windows = [(8 * widest + 31 + 31) // 32 for widest in (16, 30)] + [4]  # Stretch<8, ...>::WORDS, and ByteWindow's
    for theta in (0.0, 1.0 / bins, 2.0 / bins, 40.0 / bins, 0.1, 1.0):
        k, S = fftsp.kept_per_chunk(L, theta), fftsp.packed_bytes(L, L, theta, bits) - 64
        W = (bins + 31) // 32
        assert S == (16 + 4 * W + (2 * bits * k + 31) // 32 * 4 + 15) // 16 * 16
        # all bins claimed by the bitmap, its padding bits too
        assert lib(S, W, k, (ctypes.c_int * 3)(*windows), 3, 2 * bits * 32 * W) == 0
