"""The peers' decoder at its edges: the narrowest and widest codes of both of its kernels, records shorter than a lane's
window, a tile's last bin, odd numbers of peers, and more words than one part of the prefix counts."""
import numpy as np
import pytest

from paper_1811_08596_amd import workloads
from tests.gpu_harness import Device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return Device()


@pytest.mark.parametrize("bits", [3, 8, 9, 15, 16])
@pytest.mark.parametrize("L,theta,peers", [(32, 0.97, 2), (32, 0.5, 1), (1024, 0.9, 3), (4096, 0.3, 2), (1 << 15, 0.99, 5),
                                           (1 << 16, 0.5, 2), (1 << 20, 0.5, 3)])
def test_sum_of_peers(dev, ref, L, theta, peers, bits):
    n = 2 * L - L // 4 - 1
    print(f"peers n={n} L={L} theta={theta} bits={bits} peers={peers}", flush=True)
    streams = [ref.compress(workloads.small_mixed(n, seed=7 * p + bits) * np.float32(1 + p), L, theta, bits, nthreads=8)
               for p in range(peers)]
    got, status = dev.decode_accumulate(streams, n, L, theta, bits)
    want = ref.decode_accumulate_spectrum(streams, n, L, theta, bits, nthreads=8)
    assert status == 0
    assert np.array_equal(got.view(np.uint32), want.view(np.uint32))  # the same sums in the same order
