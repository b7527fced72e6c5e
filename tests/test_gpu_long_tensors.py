"""Per-tensor calls with tensors longer than one workgroup takes: all lengths share their launches, so every record must be
the one the uniform path makes of that tensor alone and every tensor come back as from the uniform receiver.  More tensors than
one table holds; every length, filling its chunk or not, at offsets and sizes that are and are not multiples of four; both
tile sizes of the transforms; beside short tensors on the side stream, also inside a captured graph."""
import numpy as np
import pytest

from tests.gpu_harness import Device

pytestmark = pytest.mark.gpu

SETS = {
    "more_than_a_table": [40000 + 361 * i for i in range(70)] + [65536, 40001, 9],
    "every_length": [50000, 1 << 16, 100004, 1 << 17, 200001, 1 << 18, 300000, 1 << 19, 700004, (1 << 20) - 3, 1 << 20, 1400000,
                     1 << 21, 3000000, 1 << 22, 12, 4096, 33],
    "large_tiles": [(1 << 22) - 5 * i for i in range(13)] + [70000, 1 << 18, 12345],
    "large_tiles_alone": [1 << 22, 3000004, (1 << 21) + 8],
    "large_and_short": [3000004, 2500000, 1 << 22, 3500000, 65540, 30000, 100, 7],
}


@pytest.fixture(scope="module")
def dev():
    return Device()


@pytest.mark.parametrize("name", SETS)
def test_long_tensors_match_the_uniform_path(dev, ref, name):
    torch, f = dev.torch, dev.f
    sizes, theta, bits = SETS[name], 0.3, 8
    offs = [int(v) for v in np.concatenate([[0], np.cumsum(sizes)])]
    rng = np.random.default_rng(len(sizes))
    g = dev.to_dev((rng.laplace(size=offs[-1]) * 1e-3).astype(np.float32))
    ws = dev.workspace(f.workspace_bytes_segments(offs, bits))
    nb = f.packed_bytes_segments(offs, theta, bits)
    packed = torch.full((nb,), 0xEE, dtype=torch.uint8, device=dev.dev)
    out = torch.full((offs[-1],), float("nan"), dtype=torch.float32, device=dev.dev)

    def step():
        f.compress_segments(g, offs, theta, bits, packed, ws)
        f.decompress_segments(packed, nb, out, offs, theta, bits, ws)

    step()
    assert f.device_status(ws) == 0
    pos = 64
    for i, s in enumerate(sizes):
        L = ref.segment_length(s)
        print(f"{name}: tensor {i} of {s}", flush=True)
        x = g[offs[i]:offs[i + 1]].clone()
        one = torch.empty(f.packed_bytes(s, L, theta, bits), dtype=torch.uint8, device=dev.dev)
        work = dev.ws_for(s, L, bits)
        back = torch.empty_like(x)
        f.compress(x, L, theta, bits, one, work)
        f.decompress(one, one.numel(), back, L, theta, bits, work)
        S = one.numel() - 64
        got, want = packed[pos:pos + S].clone(), one[64:].clone()
        assert int(got[12:16].view(torch.int32)[0]) == L
        got[12:16] = 0
        want[12:16] = 0
        assert torch.equal(got, want)
        assert torch.equal(out[offs[i]:offs[i + 1]].view(torch.int32), back.view(torch.int32))
        pos += S
    assert pos == nb

    bad = packed.clone()
    bad[64 + 16] ^= 1                                      # one bit too many or too few in the first tensor's bitmap
    f.decompress_segments(bad, nb, out, offs, theta, bits, ws)
    assert f.device_status(ws) == 6
    step()
    assert f.device_status(ws) == 0
    if name != "large_and_short":
        return
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            step()
    torch.cuda.synchronize()
    for replay in range(3):
        g.mul_(0.7)
        step()
        torch.cuda.synchronize()
        want_packed, want_out = packed.clone(), out.clone()
        packed.fill_(0xEE)
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(packed, want_packed) and torch.equal(out.view(torch.int32), want_out.view(torch.int32)), replay
