"""Short calls of two-pass chunk lengths: the sender's last kernel finds the threshold (csrc/codec.hip)."""
import numpy as np
import pytest

from tests.gpu_harness import Device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return Device()


@pytest.mark.parametrize("chunks", (1, 12))
@pytest.mark.parametrize("logL", (16, 17, 18, 19, 20))
def test_threshold_among_keys_that_share_their_digits(dev, ref, logL, chunks):
    """keys that agree in everything but their last bits, at the same place in many tiles, so that one lane meets several of
    them; and few and many equal ones (third digit, ties)"""
    L = 1 << logL
    B, n = L // 2 + 1, chunks * L
    rng = np.random.default_rng(logL)
    near = rng.standard_normal((chunks, B, 2)).astype(np.float32) * 1e-3
    for c in range(chunks):
        for t in range(0, B - 1, 2048):
            spots = t + rng.choice(2048, 150 * 2048 // L + 2, replace=False)
            near[c, spots, 0] = 1.0 + rng.integers(0, 1 << 6, spots.size) * np.float32(2.0 ** -23)
            near[c, spots, 1] = 0.0
    big = near.copy()
    big[:, ::3, 0] = 7.0   # kept outright
    equal = np.where(np.abs(near) < 0.5, near, np.float32(1.0))
    for name, spec in (("near", near), ("below larger ones", big), ("equal", equal)):
        ones = int((np.abs(spec[0, :, 0] - 1.0) < 0.1).sum()) + int((spec[0, :, 0] > 5).sum())
        base = int((spec[0, :, 0] > 5).sum())
        for k in (base + 1, (base + ones) // 2, ones):
            theta = float(np.float32(k / B))
            print(f"L=2^{logL} chunks={chunks} {name} k={k}", flush=True)
            want = ref.encode_spectrum(spec.reshape(-1), n, L, theta, 8, nthreads=8)
            assert np.array_equal(dev.encode(spec.reshape(-1), n, L, theta, 8), want)
