"""Where Top-k's long calls look for the threshold (csrc/sample.h and k_sample of csrc/codec.hip), followed on the host: that the window is as narrow as
the lists behind it where a gradient ends inside a chunk, and which of the three ways to the threshold the gradients of
test_gpu_topk_sampled.py take, so that none of the ways goes untested there."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_1811_08596_amd import workloads
from tests.test_gpu_topk_sampled import SAMPLES, misleading, sampled, stretch, with_zeros

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#include "%s/paper_1811_08596_amd/csrc/sample.h"
extern "C" uint32_t slot(uint32_t g, uint32_t slots) { return fftsp::sample_slot(g, slots); }
extern "C" float variance(float d, uint32_t k, uint32_t L, uint32_t present) { return fftsp::sample_variance(d, k, L, present); }
extern "C" float margin(uint32_t L, uint32_t present) { return fftsp::sample_margin(L, present); }
extern "C" int takes(uint32_t chunk_tiles, size_t tiles, int whole) { return fftsp::sampled(chunk_tiles, tiles, whole); }
extern "C" uint32_t samples(void) { return fftsp::kSamples; }
extern "C" uint32_t length(uint32_t L) { return fftsp::sample_stretch(L); }
extern "C" float deviations(void) { return fftsp::kSampleDeviations; }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("sample")
    (d / "sample.cpp").write_text(SOURCE % ROOT)
    subprocess.run(["g++", "-O2", "-ffp-contract=off", "-shared", "-fPIC", "-std=c++17", "-o", str(d / "sample.so"), str(d / "sample.cpp")], check=True)
    s = ctypes.CDLL(str(d / "sample.so"))
    s.variance.restype = s.margin.restype = s.deviations.restype = ctypes.c_float
    s.variance.argtypes = [ctypes.c_float] + [ctypes.c_uint32] * 3
    s.takes.argtypes = [ctypes.c_uint32, ctypes.c_size_t, ctypes.c_int]
    assert s.samples() == SAMPLES and all(s.length(1 << p) == stretch(1 << p) for p in range(18, 21))
    return s


def keys_of(x):
    return (np.ascontiguousarray(x, np.float32).view(np.uint32) & 0x7FFFFFFF).astype(np.int64)


def from_above(counts, rank):
    """The bucket that holds the rank-th largest, and how many lie above it; None where there are fewer."""
    run = np.cumsum(counts[::-1])
    at = int(np.searchsorted(run, rank))
    return None if at == len(run) else (len(run) - 1 - at, int(run[at - 1]) if at else 0, int(run[at]))


def window(lib, X, k, present):
    """The two keys between which k_sample has candidates lie, of a chunk with its padding."""
    f, L = np.float32, len(X)
    S = lib.samples()
    many, lanes = S // stretch(L), stretch(L) // 4
    keys = keys_of(X[sampled(L)]).reshape(many, 4 * lanes)
    share = f(k) / f(L)
    # a quarter by its top twelve bits: of four neighbours one, another one in every eighth of the stretches
    quarter = keys.reshape(many, lanes, 4)[np.arange(many), :, (np.arange(many) // (many // 8)) & 3].ravel()
    coarse, few = np.bincount(quarter >> 19, minlength=4096), S // 4
    at, wide = share * f(few), f(20) * np.sqrt(share * (f(1) - share) * f(few)) + f(20)
    clamp = lambda r, most: int(min(max(r, 1), most))
    top, bottom, middle = (from_above(coarse, clamp(r, few))[0] for r in (at - wide, at + wide, at))
    base, extent = bottom << 19, ((top - bottom + 1) << 19) - 1
    shift = extent.bit_length() - 10
    d = keys.ravel() - base
    fine, above = np.bincount(d[(d >= 0) & (d <= extent)] >> shift, minlength=1024), int((d > extent).sum())
    row = 16 // lanes
    rows = (keys >= middle << 19).sum(axis=1).reshape(-1, row)
    differences = f(lanes * int((np.diff(rows, axis=1) ** 2).sum())) * f(0.5 / lanes * row / (row - 1))
    wide = f(lib.deviations()) * np.sqrt(f(lib.variance(differences, k, L, present))) + f(lib.margin(L, present))
    at = share * f(S)
    r0, r1 = clamp(at - wide, S), clamp(at + wide, S)
    hi, lo = 0x7FFFFFFF, 1
    found = from_above(fine, r0 - above)
    if at - wide >= 1 and above < r0 and found:
        hi = min(base + (found[0] << shift) + (1 << shift) - 1, hi)
    if at + wide <= S:
        found = from_above(fine, r1 - above)
        lo = max(1, base) if above >= r1 else max(1, base + (found[0] << shift)) if found else 1
    return lo, hi


def chunks_of(g, L):
    for c in range(-(-g.size // L)):
        x = g[c * L:(c + 1) * L]
        yield np.pad(x, (0, L - x.size)), x.size


def outcome(lib, X, k, present):
    if k == 0:
        return "nothing kept", 0
    lo, hi = window(lib, X, k, present)
    keys = keys_of(X)
    kept, candidates = int((keys > hi).sum()), int(((keys >= lo) & (keys <= hi)).sum())
    return "inside" if kept < k <= kept + candidates else "zero" if kept < k and lo == 1 else "samples", candidates


def kept(theta, L):
    return int(np.floor(theta * L + 0.5))


@pytest.mark.parametrize("logL", (18, 20))
@pytest.mark.parametrize("theta", (0.15, 0.5))
def test_a_chunk_that_the_gradient_fills_in_part(lib, logL, theta):
    """Where it is hardly fuller than what is kept of it the candidates are no more than k_resolve's first rows hold, 128 a tile."""
    L = 1 << logL
    k = kept(theta, L)
    for fuller in (1.0001, 1.01, 1.04, 1.3, 2.0, 5.0, 100.0):
        present = min(L, int(k * fuller) + 1)
        for g in (workloads.small_mixed(present, seed=logL), np.random.default_rng(logL).normal(size=present).astype(np.float32)):
            X = np.pad(g, (0, L - present))
            way, candidates = outcome(lib, X, k, present)
            assert way == "inside" and (fuller > 1.1 or candidates <= 128 * -(-present // 2048)), (fuller, way, candidates)
    assert outcome(lib, np.pad(g[:k], (0, L - k)), k, k)[0] in ("inside", "zero")
    assert outcome(lib, np.pad(g[:k // 2], (0, L - k // 2)), k, k // 2)[0] == "zero"


def test_rows_with_a_scale_each(lib):
    """Neighbours that are alike: the window is no wider than k_resolve's first rows."""
    L, k = 1 << 20, kept(0.15, 1 << 20)
    for seed in range(4):
        rng = np.random.default_rng(seed)
        for row in (64, 1024):
            X = (rng.normal(size=(L // row, row)) * 10.0 ** rng.uniform(-4, 0, (L // row, 1))).astype(np.float32).ravel()
            way, candidates = outcome(lib, X, k, L)
            assert way == "inside" and candidates <= 128 * L // 2048, (row, candidates * 2048 / L)


@pytest.mark.parametrize("logL", (18, 19, 20))
def test_ways_to_the_threshold(lib, logL):
    L, ways = 1 << logL, {}
    for theta in (0.001, 0.15, 0.5, 0.97):
        for name, g in misleading(logL).items():
            for X, present in list(chunks_of(g, L))[:4]:
                ways.setdefault(name, []).append(outcome(lib, X, kept(theta, L), present)[0])
    assert set(ways["plain"]) == {"inside"}
    assert ways["scaled"].count("samples") >= 4 and ways["ties"].count("samples") >= 4


def test_ways_with_zeros(lib):
    L, ways = 1 << 18, []
    for theta in (0.1, 0.5, 0.9):
        for X, present in list(chunks_of(with_zeros(theta), L))[:10]:
            ways.append(outcome(lib, X, kept(theta, L), present)[0])
    assert ways.count("zero") >= 6 and ways.count("inside") >= 6


def test_which_calls_take_the_sample(lib):
    calls = [(64, 11000, 1), (128, 7168, 1), (128, 7169, 1), (256, 7169, 1), (512, 10240, 1), (512, 10241, 1), (512, 4096, 0), (512, 4097, 0), (128, 4097, 0), (1024, 11000, 0)]
    assert [lib.takes(*c) for c in calls] == [0, 0, 1, 1, 0, 1, 0, 1, 1, 0]
