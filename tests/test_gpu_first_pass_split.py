"""The transform's first passes with a tile in half of the LDS (csrc/fft.hip, fwd_a_split and inv_a_split): the bits of the small tiles and of the
persistent kernels, on either side of the rules that choose, with ends and starts of tensors that allow 16-byte accesses, 8-byte ones and none."""
import pytest

from tests.gpu_harness import Device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return Device()


# chunks of a call that takes the kernel in question; test_host_launches.py pins which one that is.  The last lines are receivers whose output
# passes the caches by, against chunks on their own, whose output does not
@pytest.mark.parametrize("half,log_l,chunks", [
    (0, 16, 512), (0, 18, 70), (0, 19, 40), (0, 20, 31), (0, 20, 32), (0, 21, 10), (0, 22, 4), (0, 22, 14), (0, 22, 22),
    (1, 18, 70), (1, 19, 40), (1, 20, 31), (1, 20, 33), (1, 21, 17), (1, 22, 4), (1, 22, 10),
    (0, 16, 513), (0, 18, 129), (0, 19, 65), (0, 20, 33), (0, 22, 9), (1, 15, 1025), (1, 16, 513), (1, 18, 129), (1, 19, 65), (1, 22, 9),
])
@pytest.mark.parametrize("short", (0, 8, 1, 6))
def test_chunks(dev, half, log_l, chunks, short):
    f, torch, L = dev.f, dev.torch, 1 << log_l
    theta, bits, n = 0.2, 8, chunks * L - short
    print(f"half={half} 2^{log_l} x {chunks}, {short} samples short", flush=True)
    g = torch.randn(chunks * L, device="cuda", generator=torch.Generator(device="cuda").manual_seed(log_l)) * 1e-3

    def both(x):
        n = x.numel()
        ws = dev.ws_for(n, L, bits)
        out = torch.full((n + 4,), 7.0, device="cuda")
        packed = torch.empty(f.packed_bytes(n, L, theta, bits), dtype=torch.uint8, device="cuda")
        to = out[:n]
        if half:
            f.compress_h(x, L, theta, bits, 8, packed, ws)
            f.decompress_h(packed, packed.numel(), to, L, theta, bits, 8, ws)
        else:
            f.compress(x, L, theta, bits, packed, ws)
            f.decompress(packed, packed.numel(), to, L, theta, bits, ws)
        assert f.device_status(ws) == 0
        assert bool((out[n:] == 7.0).all())  # nothing beside the samples
        return packed[64:].view(-(-n // L), -1), to.clone().view(torch.int32)

    many = both(g[:n])
    for c in (0, chunks // 2, chunks - 1):
        end = min((c + 1) * L, n)
        one = both(g[c * L:end].clone())
        assert torch.equal(many[0][c], one[0][0]) and torch.equal(many[1][c * L:end], one[1])


# every tensor alone (the small tiles) and among others: launches of columns of up to 2^9, up to 2^10, and up to 2^11; the last one has more than
# 1024 tiles of 2^14 points
@pytest.mark.parametrize("sizes", [
    [1 << 18, (1 << 18) - 3, 70001, 1 << 16, (1 << 17) + 2] + [1 << 18] * 24,
    [(1 << 19) + 1, 1 << 20, 70001, 1 << 16, 140002] + [(1 << 20) - 4] * 12,
    [(1 << 19) + 1, 1 << 20, 70001, 1 << 16, 140002, (1 << 21) + 5] + [(1 << 20) - 4] * 12,
    [(1 << 19) + 1, 1 << 20, 70001, 1 << 16, 140002] + [(1 << 20) - 4] * 34,
])
@pytest.mark.parametrize("shift", (0, 1, 2))
def test_tensors(dev, sizes, shift):
    f, torch = dev.f, dev.torch
    sizes = [32 + shift] + sizes  # where the others start
    print(f"{len(sizes)} tensors, {shift} off", flush=True)

    def receive(x, sizes):
        offsets = [0]
        for s in sizes:
            offsets.append(offsets[-1] + s)
        n = offsets[-1]
        packed = torch.empty(f.packed_bytes_segments(offsets, 0.3, 8), dtype=torch.uint8, device="cuda")
        ws = torch.empty(f.workspace_bytes_segments(offsets, 8), dtype=torch.uint8, device="cuda")
        out = torch.full((n + 4,), 7.0, device="cuda")
        f.compress_segments(x, offsets, 0.3, 8, packed, ws)
        f.decompress_segments(packed, packed.numel(), out[:n], offsets, 0.3, 8, ws)
        assert f.device_status(ws) == 0
        assert bool((out[n:] == 7.0).all())
        return out[:n].clone().view(torch.int32)

    g = torch.randn(sum(sizes), device="cuda", generator=torch.Generator(device="cuda").manual_seed(shift)) * 1e-2
    many, at = receive(g, sizes), 0
    for i, s in enumerate(sizes):
        if i < 8:
            assert torch.equal(many[at:at + s], receive(g[at:at + s].clone(), [s])), i
        at += s
