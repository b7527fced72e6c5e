"""Chunk-resident senders code a chunk's survivors row by row or, where few enough survive, next to each other: both sides of
that line, a handful of survivors and ties at the threshold, at widths whose codes straddle words and at stored ones."""
import numpy as np
import pytest

from tests.gpu_harness import Device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return Device()


def _gradient(n, seed, tied):
    g = np.random.default_rng(seed).standard_normal(n).astype(np.float32)
    return np.round(2 * g) / 2 if tied else g


@pytest.mark.parametrize("tied", (False, True))
@pytest.mark.parametrize("bits", (3, 8, 13, 16))
@pytest.mark.parametrize("logL", range(9, 16))
def test_either_side_of_the_line(dev, ref, logL, bits, tied):
    L = 1 << logL
    n = 3 * L - 9
    g = _gradient(n, logL + bits, tied)
    spec = dev.rfft(g, L)
    for theta in (2 / L, 0.1, 0.2, 0.21, 1 / 3, 0.35, 0.5, 0.52):
        print(f"L=2^{logL} bits={bits} theta={theta} tied={tied}", flush=True)
        assert np.array_equal(dev.compress(g, L, theta, bits), ref.encode_spectrum(spec, n, L, theta, bits, nthreads=4))
        assert np.array_equal(dev.topk_compress(g, L, theta, bits), ref.topk_compress(g, L, theta, bits, nthreads=4))
