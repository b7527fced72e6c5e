"""Chunk-resident kernels keep no twiddles that no stage wants, and a receiver's bitmap table where its data will be: every length
they take, sent and received alone and among others, at the widest codes (whose records leave the table least room)."""
import pytest

from tests.gpu_harness import Device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return Device()


@pytest.mark.parametrize("bits", (8, 16, 32))
@pytest.mark.parametrize("logL", range(5, 16))
def test_round_trip_and_the_spectrum_behind_it(dev, ref, logL, bits):
    import numpy as np
    L = 1 << logL
    n = max(3 * L, 4096 + L) - 5
    g = (np.random.default_rng(logL).standard_normal(n) * 1e-3).astype(np.float32)
    for theta in (1.0, 0.3):
        print(f"L=2^{logL} bits={bits} theta={theta}", flush=True)
        packed = dev.compress(g, L, theta, bits)
        spec = dev.rfft(g, L)
        assert np.array_equal(packed, ref.encode_spectrum(spec, n, L, theta, bits, nthreads=4))
        got, status = dev.decompress(packed, n, L, theta, bits, want_status=True)
        assert status == 0
        want = ref.decompress(packed, n, L, theta, bits)
        # two transforms of binary32, one of them rounded once: 2^-24 sqrt(log2 L) of the values, as test_gpu_parity derives it
        assert np.linalg.norm(got - want) <= 1e-5 * np.linalg.norm(want)
