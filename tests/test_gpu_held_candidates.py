"""The threshold search of chunks whose candidates a workgroup holds in registers, at the most tiles it holds (512 of samples, 513
of bins) and one step beyond: few candidates, tiles with more than a row of them, ties in bin order and a chunk that ends early."""
import numpy as np
import pytest

from tests.gpu_harness import Device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return Device()


def _values(kind, n):
    g = np.random.default_rng(n & 1023).standard_normal(n).astype(np.float32)
    return {"normal": g, "tied": np.round(8 * g) / 8, "crowded": 1.0 + 1e-3 * g, "alike": np.full(n, -0.25, np.float32)}[kind].astype(np.float32)


@pytest.mark.parametrize("kind", ("normal", "tied", "crowded", "alike"))
@pytest.mark.parametrize("logL", (20, 21))
def test_samples(dev, ref, logL, kind):
    L = 1 << logL
    g = _values(kind, L + L // 2 + 3)
    for theta in (0.003, 0.3):
        print(f"samples L=2^{logL} {kind} theta={theta}", flush=True)
        assert np.array_equal(dev.topk_compress(g, L, theta, 8), ref.topk_compress(g, L, theta, 8, nthreads=8))


@pytest.mark.parametrize("kind", ("normal", "tied", "crowded", "alike"))
@pytest.mark.parametrize("logL", (21, 22))
def test_bins(dev, ref, logL, kind):
    L = 1 << logL
    n = L
    spec = _values(kind, L + 2)
    spec[1] = spec[L + 1] = 0.0  # the DC and Nyquist bins are real
    for theta in (0.003, 0.3):
        print(f"bins L=2^{logL} {kind} theta={theta}", flush=True)
        assert np.array_equal(dev.encode(spec, n, L, theta, 8), ref.encode_spectrum(spec, n, L, theta, 8, nthreads=8))
