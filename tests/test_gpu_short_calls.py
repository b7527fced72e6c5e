"""Short calls of two-pass chunk lengths go through kernels of their own (csrc/short.hip): small tiles, the receiver's first pass
reading the records, the sender's last kernel finding the threshold.  What they compute is what the long calls' kernels compute, bit
for bit."""
import numpy as np
import pytest

from tests.gpu_harness import Device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return Device()


@pytest.mark.parametrize("logL", (16, 17, 18, 19, 20, 21))
@pytest.mark.parametrize("chunks, tail", ((1, 1), (1, 40003), (2, 6), (3, 65534)))
def test_ragged_short_call_and_the_same_chunks_in_a_long_one(dev, logL, chunks, tail):
    """the last chunk ends in it, after an odd or an even number of samples; the long call holds the zeros that follow"""
    torch, f, L, theta, bits = dev.torch, dev.f, 1 << logL, 0.4, 9
    n, many = (chunks - 1) * L + tail, chunks + (1 << 23) // L + 1
    gen = torch.Generator(device="cuda").manual_seed(logL * 8 + chunks)
    long = torch.randn(many * L, device="cuda", generator=gen) * 1e-3
    long[n:chunks * L] = 0.0

    def all_of(x, count):
        ws, c = dev.ws_for(count, L, bits), -(-count // L)
        spec, out, hout, back = torch.empty(c * (L + 2), device="cuda"), torch.empty_like(x), torch.empty_like(x), torch.empty_like(x)
        f.rfft(x, L, spec, ws)
        f.irfft(spec, count, L, back, ws)
        packed = torch.empty(f.packed_bytes(count, L, theta, bits), dtype=torch.uint8, device="cuda")
        half = torch.empty_like(packed)
        f.compress(x, L, theta, bits, packed, ws)
        f.decompress(packed, packed.numel(), out, L, theta, bits, ws)
        f.compress_h(x, L, theta, bits, 8, half, ws)
        f.decompress_h(half, half.numel(), hout, L, theta, bits, 8, ws)
        assert f.device_status(ws) == 0
        return (spec.view(torch.int32).view(c, -1), packed[64:].view(c, -1), half[64:].view(c, -1), back.view(torch.int32),
                out.view(torch.int32), hout.view(torch.int32))

    short, want = all_of(long[:n].clone(), n), all_of(long, many * L)
    for i, (what, a, b) in enumerate(zip(("spectra", "records", "half records", "inverse", "samples", "half samples"), short, want)):
        print(f"L=2^{logL} n={n}: {what}", flush=True)
        assert torch.equal(a, b[:chunks if i < 3 else n])


@pytest.mark.parametrize("bits", (3, 8, 9, 16, 32))
@pytest.mark.parametrize("logL", (16, 17, 18, 19))
def test_receiver_without_a_spectrum(dev, logL, bits):
    """decompress takes the bins from the records; decode_spectrum and irfft go through a spectrum"""
    torch, f, L = dev.torch, dev.f, 1 << logL
    n = 2 * L - 4099
    g = torch.randn(n, device="cuda", generator=torch.Generator(device="cuda").manual_seed(bits)) * 1e-2
    ws = dev.ws_for(n, L, bits)
    for theta in (1.0, 0.5, 0.003, 0.0):
        print(f"L=2^{logL} bits={bits} theta={theta}", flush=True)
        packed = torch.empty(f.packed_bytes(n, L, theta, bits), dtype=torch.uint8, device="cuda")
        f.compress(g, L, theta, bits, packed, ws)
        out, want, spec = torch.empty_like(g), torch.empty_like(g), torch.empty(2 * (L + 2), device="cuda")
        f.decompress(packed, packed.numel(), out, L, theta, bits, ws)
        assert f.device_status(ws) == 0
        f.decode_spectrum(packed, packed.numel(), n, L, theta, bits, spec, ws)
        f.irfft(spec, n, L, want, ws)
        assert torch.equal(out.view(torch.int32), want.view(torch.int32))
        # a bitmap that claims every bin is reported (test_record_bounds.py: what is read then)
        if theta < 1.0:
            packed[64 + 16:64 + 16 + L // 16] = 255
            f.decompress(packed, packed.numel(), out, L, theta, bits, ws)
            assert f.device_status(ws) != 0


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
