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
@pytest.mark.parametrize("logL, tail", ((17, 1), (17, 786), (17, 2048), (17, 3000), (17, 70000), (20, 786), (20, 70001)))
def test_topk_chunk_of_nearly_only_zeros(dev, ref, logL, tail, bits):
    """tiles whose candidates are all one value count as one candidate, beside tiles where they are not; in chunks that one
    workgroup resolves alone and in longer ones"""
    L = 1 << logL
    n = L + tail
    rng = np.random.default_rng(tail)
    g = rng.standard_normal(n).astype(np.float32)
    g[rng.random(n) < 0.01] = 0.0
    for theta in (0.9, 0.6, 0.001):
        print(f"L=2^{logL} tail={tail} bits={bits} theta={theta}", flush=True)
        assert np.array_equal(dev.topk_compress(g, L, theta, bits), ref.topk_compress(g, L, theta, bits, nthreads=8))


@pytest.mark.parametrize("logL, ties", ((21, False), (21, True), (22, False), (22, True)))
def test_chunks_resolved_by_several_workgroups(dev, ref, logL, ties):
    L = 1 << logL
    spec = np.random.default_rng(logL).standard_normal(2 * (L + 2)).astype(np.float32)
    if ties:
        spec = (np.round(spec * 4.0) / 4.0).astype(np.float32)
    for theta in (0.5, 0.001):
        print(f"L=2^{logL} ties={ties} theta={theta}", flush=True)
        want = ref.encode_spectrum(spec, 2 * L - 5, L, theta, 8, nthreads=8)
        assert np.array_equal(dev.encode(spec, 2 * L - 5, L, theta, 8), want)
