"""Top-k's long chunks take the threshold from a sample: byte for byte the oracle's result, whatever the sample says.  Gradients whose
sampled places lie (csrc/codec.hip, sample_slot: the places are a fixed function of the chunk's length) send the selection to the
samples themselves; so do chunks that end before most of them."""
import numpy as np
import pytest

from paper_1811_08596_amd import workloads
from tests.gpu_harness import Device

pytestmark = pytest.mark.gpu
STRETCHES = 2048


@pytest.fixture(scope="module")
def dev():
    return Device()


def sampled(L):
    g, slots = np.arange(STRETCHES, dtype=np.uint64), L // (16 * STRETCHES)
    at = g * slots + ((g * 2654435761 & 0xFFFFFFFF) >> 15 & (slots - 1))
    return (16 * at[:, None] + np.arange(16, dtype=np.uint64)).astype(np.int64).ravel()


def check(dev, ref, g, L, theta, bits):
    assert np.array_equal(dev.topk_compress(g, L, theta, bits), ref.topk_compress(g, L, theta, bits, nthreads=16))


# more than 4096 tiles of 2048; k_resolve holds 288 of a chunk's summaries, or 513
@pytest.mark.parametrize("theta", [0.001, 0.15, 0.5, 0.97])
@pytest.mark.parametrize("logL", [18, 19, 20])
def test_a_sample_that_misleads(dev, ref, logL, theta):
    L = 1 << logL
    print(f"L=2^{logL} theta={theta}", flush=True)
    chunks = (4096 << 11) // L + 1
    n = chunks * L - L // 3
    g = workloads.small_mixed(n, seed=logL)
    check(dev, ref, g, L, theta, 10)
    at = (sampled(L)[None, :] + L * np.arange(1, chunks - 2, 3)[:, None]).ravel()  # of every third chunk
    h = g.copy()
    h[at] *= np.float32(2.0 ** -9)
    h[at + L] *= np.float32(2.0 ** 9)
    check(dev, ref, h, L, theta, 8)
    h = g.copy()
    h[:L] = 0.25  # nothing but ties among what the sample shows, and next to nothing of it elsewhere
    h[sampled(L)] = 0.5
    h[L:2 * L] = 0.5
    h[L + sampled(L)] = 0.25
    check(dev, ref, h, L, theta, 32)


@pytest.mark.parametrize("theta", [0.0, 0.3, 1.0])
def test_scales_that_differ_and_short_chunks(dev, ref, theta):
    L = 1 << 18
    scale = np.repeat(np.float32(10.0) ** np.arange(-6, 2, dtype=np.float32), L // 8)
    g = np.tile(scale, 34) * workloads.small_mixed(34 * L, seed=1)
    for n in (34 * L, 32 * L + 1, 32 * L + 15, 33 * L + 4 * 777 + 2):
        check(dev, ref, g[:n], L, theta, 8)
    g[::2] = np.inf
    g[1::64] = np.nan
    dev.topk_compress(g, L, theta, 8)  # what such a gradient gives is its bit patterns' order; it only has to come back


@pytest.mark.parametrize("theta", [0.0003, 0.1, 0.5, 0.9])
def test_zeros_are_no_candidates(dev, ref, theta):
    """The threshold at, just above and well below the smallest value that is not zero."""
    L = 1 << 18
    n = 33 * L + 3 * L // 8
    rng = np.random.default_rng(5)
    g = workloads.small_mixed(n, seed=2)
    g[g == 0.0] = np.float32(1e-3)
    k = int(np.floor(theta * L + 0.5))
    keep = [0, 1, 5, k - 1, k, k + 1, k + 300, L // 2, L // 2 + 100, L]  # of a chunk's samples, those that are not zero
    for c in range(33):
        zero = rng.permutation(L)[min(max(keep[c % len(keep)], 0), L):]
        g[c * L + zero] = np.float32(-0.0) if c % 2 else np.float32(0.0)
    g[7 * L:8 * L] *= np.float32(2.0 ** -130)  # subnormal
    check(dev, ref, g, L, theta, 8)
    check(dev, ref, g, L, theta, 32)
