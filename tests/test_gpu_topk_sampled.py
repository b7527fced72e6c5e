"""Top-k's long chunks take the threshold from a sample: byte for byte the oracle's result, whatever the sample says.  Gradients whose
sampled places lie (csrc/codec.hip, sample_slot: the places are a fixed function of the chunk's length) send the selection to the
samples themselves; so do chunks that end before most of them."""
import numpy as np
import pytest

from paper_1811_08596_amd import workloads
from tests.gpu_harness import Device

pytestmark = pytest.mark.gpu
SAMPLES = 1 << 15


@pytest.fixture(scope="module")
def dev():
    return Device()


def stretch(L):
    return 8 if L >= 1 << 20 else 16


def sampled(L):
    g, slots = np.arange(SAMPLES // stretch(L), dtype=np.uint64), L // SAMPLES
    at = g * slots + ((g * 2654435761 & 0xFFFFFFFF) >> 15 & (slots - 1))
    return (stretch(L) * at[:, None] + np.arange(stretch(L), dtype=np.uint64)).astype(np.int64).ravel()


def check(dev, ref, g, L, theta, bits):
    assert np.array_equal(dev.topk_compress(g, L, theta, bits), ref.topk_compress(g, L, theta, bits, nthreads=16))


def misleading(logL):
    """Gradients by name: what the sample shows is like the rest, smaller or larger than it, or ties that are not the rest's."""
    L = 1 << logL
    chunks = (4096 << 11) // L + 1
    g = workloads.small_mixed(chunks * L - L // 3, seed=logL)
    at = (sampled(L)[None, :] + L * np.arange(1, chunks - 2, 3)[:, None]).ravel()  # of every third chunk
    scaled = g.copy()
    scaled[at] *= np.float32(2.0 ** -9)
    scaled[at + L] *= np.float32(2.0 ** 9)
    ties = g.copy()
    ties[:L] = 0.25  # nothing but ties among what the sample shows, and next to nothing of it elsewhere
    ties[sampled(L)] = 0.5
    ties[L:2 * L] = 0.5
    ties[L + sampled(L)] = 0.25
    return {"plain": g, "scaled": scaled, "ties": ties}


def with_zeros(theta):
    """Thirty-three chunks of 2^18 and a part of one, with about as many samples that are not zero as are kept, or all but none or all of them."""
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
    return g


# more than 4096 tiles of 2048; k_resolve holds 288 of a chunk's summaries, or 513.  (Which way to the threshold each takes: test_topk_window.py.)
@pytest.mark.parametrize("theta", [0.001, 0.15, 0.5, 0.97])
@pytest.mark.parametrize("logL", [18, 19, 20])
def test_a_sample_that_misleads(dev, ref, logL, theta):
    L = 1 << logL
    print(f"L=2^{logL} theta={theta}", flush=True)
    for (name, g), bits in zip(misleading(logL).items(), (10, 8, 32)):
        check(dev, ref, g, L, theta, bits)


@pytest.mark.parametrize("fuller", [1.0001, 1.07, 1.3, 5.0])
@pytest.mark.parametrize("logL", [18, 20])
def test_a_gradient_that_ends_soon_after_what_is_kept(dev, ref, logL, fuller):
    L, theta = 1 << logL, 0.15
    print(f"L=2^{logL} {fuller}", flush=True)
    check(dev, ref, workloads.small_mixed((4096 << 11) + int(theta * L * fuller) + 1, seed=logL), L, theta, 32)


@pytest.mark.parametrize("theta", [0.0, 0.3, 1.0])
def test_scales_that_differ_and_short_chunks(dev, ref, theta):
    L = 1 << 18
    scale = np.repeat(np.float32(10.0) ** np.arange(-6, 2, dtype=np.float32), L // 8)
    g = np.tile(scale, 34) * workloads.small_mixed(34 * L, seed=1)
    for n in (34 * L, 32 * L + 1, 32 * L + 15, 33 * L + 4 * 777 + 2):
        check(dev, ref, g[:n], L, theta, 8)
    # Values that are no numbers are ranked by their bit patterns too: a chunk has the record that it has in a call of its own, which does not take the
    # sample, with just k samples kept
    g[::2] = np.inf
    g[1::64] = np.nan
    g[3 * L:3 * L + L // 3] = np.float32(1.0)
    n = 32 * L + 1
    record = dev.f.topk_packed_bytes(L, L, theta, 8) - 64
    many, k = dev.topk_compress(g[:n], L, theta, 8)[64:].reshape(33, record), int(np.floor(theta * L + 0.5))
    for c in (0, 3, 31, 32):
        alone = dev.topk_compress(g[c * L:min((c + 1) * L, n)], L, theta, 8)[64:]
        assert np.array_equal(many[c], alone) and int(np.unpackbits(many[c][16:16 + L // 8]).sum()) == k


@pytest.mark.parametrize("theta", [0.0003, 0.1, 0.5, 0.9])
def test_zeros_are_no_candidates(dev, ref, theta):
    """The threshold at, just above and well below the smallest value that is not zero."""
    g = with_zeros(theta)
    check(dev, ref, g, 1 << 18, theta, 8)
    check(dev, ref, g, 1 << 18, theta, 32)
