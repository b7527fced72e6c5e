"""Long receivers take the inverse's first pass straight from the records (csrc/receive.hip).  They give the bits that a decoded
spectrum (decode_spectrum) and its inverse give, at every chunk length, for windows of the record at its end and across bitmap words,
and a bitmap that claims more bins than there are is reported (test_record_bounds.py: what is read then)."""
import pytest

from tests.gpu_harness import Device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return Device()


@pytest.mark.parametrize("bits", (3, 6, 8, 9, 11, 15, 16, 32))
@pytest.mark.parametrize("logL", (16, 17, 18, 19, 20, 21, 22))
def test_receiver_and_the_spectrum_it_leaves_out(dev, logL, bits):
    torch, f, L = dev.torch, dev.f, 1 << logL
    chunks = max(2, (400 << 14) // L + 1)  # more tiles than short calls have, a number that does not divide by eight
    n = chunks * L - 4099
    g = torch.randn(n, device="cuda", generator=torch.Generator(device="cuda").manual_seed(bits)) * 1e-2
    ws = dev.ws_for(n, L, bits)
    for theta in (1.0, 0.5, 3.0 / L, 0.0):
        print(f"L=2^{logL} chunks={chunks} bits={bits} theta={theta}", flush=True)
        nb = f.packed_bytes(n, L, theta, bits)
        packed = torch.empty(nb, dtype=torch.uint8, device="cuda")
        f.compress(g, L, theta, bits, packed, ws)
        out, want, spec = torch.empty_like(g), torch.empty_like(g), torch.empty(chunks * (L + 2), device="cuda")
        f.decompress(packed, nb, out, L, theta, bits, ws)
        assert f.device_status(ws) == 0
        f.decode_spectrum(packed, nb, n, L, theta, bits, spec, ws)
        f.irfft(spec, n, L, want, ws)
        assert torch.equal(out.view(torch.int32), want.view(torch.int32))
        # a sum of one stream is that stream
        one = dev.workspace(f.workspace_bytes_accumulate(n, L, bits, 1))
        f.decompress_accumulate([packed], nb, 1.0, want, L, theta, bits, one)
        assert f.device_status(one) == 0
        assert torch.equal(out.view(torch.int32), want.view(torch.int32))
        if theta < 1.0:
            packed[64 + 16:64 + 16 + L // 16] = 255  # every bin, in the first record
            packed[-(nb - 64) // chunks + 16:][:L // 16] = 255  # and in the last one, at the end of the stream
            f.decompress(packed, nb, out, L, theta, bits, ws)
            assert f.device_status(ws) != 0


@pytest.mark.parametrize("half", (0, 1))
@pytest.mark.parametrize("bits", (8, 15))
def test_chunks_of_2_to_the_16_on_either_side_of_the_wave_count(dev, bits, half):
    """161 chunks of binary32 take the kernel with six waves a SIMD, their first 160 by themselves the one with eight."""
    torch, f, L = dev.torch, dev.f, 1 << 16
    g = torch.randn(161 * L, device="cuda", generator=torch.Generator(device="cuda").manual_seed(bits)) * 1e-2
    outs = []
    for chunks in (161, 160):
        n = chunks * L
        packed, out = torch.empty(f.packed_bytes(n, L, 0.4, bits), dtype=torch.uint8, device="cuda"), torch.empty(n, device="cuda")
        ws = dev.ws_for(n, L, bits)
        if half:
            f.compress_h(g[:n], L, 0.4, bits, 10, packed, ws)
            f.decompress_h(packed, packed.numel(), out, L, 0.4, bits, 10, ws)
        else:
            f.compress(g[:n], L, 0.4, bits, packed, ws)
            f.decompress(packed, packed.numel(), out, L, 0.4, bits, ws)
        assert f.device_status(ws) == 0
        outs.append(out)
    assert torch.equal(outs[0][:160 * L].view(torch.int32), outs[1].view(torch.int32))
