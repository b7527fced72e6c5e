"""The per-tile codec kernels (csrc/codec.hip) at their edges against the oracle, bit for bit, through the stage-level entry
points: chunks of part of a tile, of one tile and one bin, and of many tiles; every way codes are stored (bytes, bit-packed
in one and in two words, whole words); all, some and none of the bins kept; spectra without ties and with many."""
import numpy as np
import pytest

from tests.gpu_harness import Device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return Device()


@pytest.mark.parametrize("bits", (3, 8, 9, 16, 32))
@pytest.mark.parametrize("logL", (5, 10, 12, 13, 16, 17))
def test_tiles_match_the_oracle(dev, ref, logL, bits):
    L, chunks = 1 << logL, 3
    n = chunks * L - 7
    rng = np.random.default_rng(logL * 64 + bits)
    smooth = rng.standard_normal(chunks * (L + 2)).astype(np.float32)
    ties = np.round(smooth * 4.0) / 4.0
    for name, spec in (("smooth", smooth), ("ties", ties.astype(np.float32))):
        for theta in (1.0, 0.5, 0.01, 0.0):
            print(f"L=2^{logL} bits={bits} theta={theta} {name}", flush=True)
            want = ref.encode_spectrum(spec, n, L, theta, bits, nthreads=4)
            assert np.array_equal(dev.encode(spec, n, L, theta, bits), want)
            out, st = dev.decode(want, n, L, theta, bits, want_status=True)
            assert st == 0
            assert np.array_equal(out.view(np.uint32), ref.decode_spectrum(want, n, L, theta, bits, nthreads=4).view(np.uint32))
        streams = [ref.encode_spectrum(np.roll(spec, 2 * i), n, L, 0.4, bits, nthreads=4) for i in range(3)]
        out, st = dev.decode_accumulate(streams, n, L, 0.4, bits)
        assert st == 0
        assert np.array_equal(out, ref.decode_accumulate_spectrum(streams, n, L, 0.4, bits, nthreads=4))


@pytest.mark.parametrize("bits", (8, 32))
@pytest.mark.parametrize("tail", (1, 786, 2048, 3000, 70000))
def test_topk_chunk_of_nearly_only_zeros(dev, ref, tail, bits):
    """tiles whose candidates are all one value count as one candidate, beside tiles where they are not"""
    L = 1 << 17
    n = L + tail
    rng = np.random.default_rng(tail)
    g = rng.standard_normal(n).astype(np.float32)
    g[rng.random(n) < 0.01] = 0.0
    for theta in (0.9, 0.6, 0.001):
        print(f"tail={tail} bits={bits} theta={theta}", flush=True)
        assert np.array_equal(dev.topk_compress(g, L, theta, bits), ref.topk_compress(g, L, theta, bits))
