"""Long receivers' kernel of half the LDS against the one of short launches: the same bits on either side of the rule that chooses
(csrc/receive.hip, kPairsFrom and the tensors' launches)."""
import pytest

from tests.gpu_harness import Device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return Device()


def first_long(log_l, half):
    rows = (log_l - 1) // 2
    tiles = {7: (3584, 4224), 8: (2177, 2305), 9: (257, 1025), 10: (257, 257)}[rows][half]
    return -(-tiles // (1 << (log_l - 1 - rows - 4)))


@pytest.mark.parametrize("half", (0, 1))
@pytest.mark.parametrize("theta,bits", [(0.4, 8), (1.0, 8), (0.002, 3), (0.4, 15), (1.0, 9)])
@pytest.mark.parametrize("log_l", (16, 17, 18, 19, 20, 21, 22))
def test_chunks(dev, log_l, theta, bits, half):
    torch, f, L = dev.torch, dev.f, 1 << log_l
    most = first_long(log_l, half)
    print(f"2^{log_l} theta={theta} bits={bits} half={half} chunks={most}", flush=True)
    g = torch.randn(most * L, device="cuda", generator=torch.Generator(device="cuda").manual_seed(log_l)) * 1e-2
    outs = []
    for chunks in (most, most - 1):
        n = chunks * L - (3 if chunks == most else 0)
        packed, out = torch.empty(f.packed_bytes(n, L, theta, bits), dtype=torch.uint8, device="cuda"), torch.empty(n, device="cuda")
        ws = dev.ws_for(n, L, bits)
        if half:
            f.compress_h(g[:n], L, theta, bits, 10, packed, ws)
            f.decompress_h(packed, packed.numel(), out, L, theta, bits, 10, ws)
        else:
            f.compress(g[:n], L, theta, bits, packed, ws)
            f.decompress(packed, packed.numel(), out, L, theta, bits, ws)
        assert f.device_status(ws) == 0
        outs.append(out)
    n = (most - 1) * L
    assert torch.equal(outs[0][:n].view(torch.int32), outs[1].view(torch.int32))


# short launches' sets first; the long ones have them in front: 1025 tiles of 2^13 points from 2^20 on downwards, 257 of 2^14 above
@pytest.mark.parametrize("bits", (6, 15))
@pytest.mark.parametrize("few,more", [
    ([1 << 20] * 3, [1 << 20] * 14),
    ([1 << 16, 3 << 15, (1 << 17) + 4, 1 << 18, 1 << 19, (1 << 20) - 8], [1 << 20] * 14 + [70000] * 5),
    ([1 << 21], [(1 << 21) - 12, 1 << 22, 1 << 22]),
    ([1 << 22, 1 << 16, 200000], [1 << 22, 1 << 21] + [1 << 20] * 15),
])
def test_tensors(dev, few, more, bits):
    torch, f = dev.torch, dev.f
    print(f"{len(few)} and {len(few) + len(more)} tensors, bits={bits}", flush=True)
    g = torch.randn(sum(few) + sum(more), device="cuda", generator=torch.Generator(device="cuda").manual_seed(bits)) * 1e-2
    outs = []
    for sizes in (few, few + more):
        offsets = [0]
        for s in sizes:
            offsets.append(offsets[-1] + s)
        packed = torch.empty(f.packed_bytes_segments(offsets, 0.3, bits), dtype=torch.uint8, device="cuda")
        ws = torch.empty(f.workspace_bytes_segments(offsets, bits), dtype=torch.uint8, device="cuda")
        out = torch.empty(offsets[-1], device="cuda")
        f.compress_segments(g[:offsets[-1]], offsets, 0.3, bits, packed, ws)
        f.decompress_segments(packed, packed.numel(), out, offsets, 0.3, bits, ws)
        assert f.device_status(ws) == 0
        outs.append(out)
    assert torch.equal(outs[0].view(torch.int32), outs[1][:sum(few)].view(torch.int32))
