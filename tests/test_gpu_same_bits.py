"""A chunk's transform does not depend on the call it is part of: spectrum, record and samples are the same bits whether the
chunk is alone, one of many (other tile sizes, csrc/fft.hip), or a tensor of a per-tensor call (other kernels again)."""
import pytest

from tests.gpu_harness import Device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return Device()


@pytest.mark.parametrize("logL,chunks", [(16, 40), (17, 40), (18, 24), (19, 24), (20, 9), (20, 60), (21, 5), (21, 20), (22, 3), (22, 11)])
def test_a_chunk_alone_and_among_others(dev, logL, chunks):
    f, torch, L, theta, bits = dev.f, dev.torch, 1 << logL, 0.4, 12
    gen = torch.Generator(device="cuda").manual_seed(logL)
    g = torch.randn(chunks * L, device="cuda", generator=gen) * 1e-3

    def all_of(x):
        n = x.numel()
        ws = dev.ws_for(n, L, bits)
        spec = torch.empty(n // L * (L + 2), device="cuda")
        back = torch.empty_like(x)
        f.rfft(x, L, spec, ws)
        f.irfft(spec, n, L, back, ws)
        packed = torch.empty(f.packed_bytes(n, L, theta, bits), dtype=torch.uint8, device="cuda")
        out = torch.empty_like(x)
        f.compress(x, L, theta, bits, packed, ws)
        f.decompress(packed, packed.numel(), out, L, theta, bits, ws)
        ws = dev.workspace(f.workspace_bytes_accumulate(n, L, bits, 1))
        alone = torch.empty_like(x)
        f.decompress_accumulate([packed], packed.numel(), 1.0, alone, L, theta, bits, ws)
        assert torch.equal(out, alone)
        half, hout = torch.empty_like(packed), torch.empty_like(x)
        f.compress_h(x, L, theta, bits, 8, half, ws)
        f.decompress_h(half, half.numel(), hout, L, theta, bits, 8, ws)
        return spec.view(torch.int32), back.view(torch.int32), packed[64:], out.view(torch.int32), half[64:], hout.view(torch.int32)

    many = [t.view(chunks, -1) for t in all_of(g)]
    offs = [i * L for i in range(chunks + 1)]
    ws = dev.workspace(f.workspace_bytes_segments(offs, bits))
    packed = torch.empty(f.packed_bytes_segments(offs, theta, bits), dtype=torch.uint8, device="cuda")
    out = torch.empty_like(g)
    f.compress_segments(g, offs, theta, bits, packed, ws)
    f.decompress_segments(packed, packed.numel(), out, offs, theta, bits, ws)
    tensors = [packed[64:].view(chunks, -1), out.view(torch.int32).view(chunks, -1)]
    tensors[0][:, 12:16] = 0  # a per-tensor record carries its chunk length
    for c in (0, chunks // 2, chunks - 1):
        one = all_of(g[c * L:(c + 1) * L].clone())
        for what, a, b in zip(("spectrum", "inverse", "record", "samples", "half record", "half samples"), many, one):
            differ = int((a[c] != b).sum())
            print(f"L=2^{logL} chunk {c} of {chunks}: {what} differs in {differ}", flush=True)
            assert differ == 0
        assert torch.equal(tensors[0][c], one[2]) and torch.equal(tensors[1][c], one[3])
