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


@pytest.mark.parametrize("kind", ("normal", "alike", "crowded"))
def test_tensors_beside_a_longer_one(dev, kind):
    """A tensor of 2^22 has its candidates counted before the search, and with it those of 2^21, which are held where they are the
    longest.  The spectrum of an impulse has one magnitude, and noise beside it crowds one bucket."""
    torch, f = dev.torch, dev.f
    sizes, theta, bits = [(1 << 21) - 1, 1 << 20, 1 << 21, 1 << 22], 0.3, 8
    offs = [0, *(int(v) for v in np.cumsum(sizes))]
    g = torch.randn(offs[-1], device="cuda", generator=torch.Generator(device="cuda").manual_seed(5)) * {"normal": 1.0, "alike": 0.0, "crowded": 1e-6}[kind]
    if kind != "normal":
        g[offs[:-1]] = 1.0
    for last in (4, 3):  # with the longest and without
        at = offs[:last + 1]
        packed = torch.empty(f.packed_bytes_segments(at, theta, bits), dtype=torch.uint8, device="cuda")
        f.compress_segments(g[:at[-1]], at, theta, bits, packed, dev.workspace(f.workspace_bytes_segments(at, bits)))
        record = 64
        for i, n in enumerate(sizes[:last]):
            L = 1 << (n - 1).bit_length()
            one = torch.empty(f.packed_bytes(n, L, theta, bits), dtype=torch.uint8, device="cuda")
            f.compress(g[at[i]:at[i + 1]].clone(), L, theta, bits, one, dev.ws_for(n, L, bits))
            print(f"{kind} of {last} tensors: {i}", flush=True)
            got = packed[record:record + one.numel() - 64]
            assert torch.equal(got[:12], one[64:76]) and torch.equal(got[16:], one[80:])  # the fourth word is the tensor's length
            record += one.numel() - 64
