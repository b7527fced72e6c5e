"""Tensors that start and end anywhere: pieces of eight and sixteen bytes are read where they lie, and the piece that a tensor's end cuts
is read by samples (csrc/fft_core.h, csrc/split_tile.h).  Every record is that of the tensor alone in a chunk filled up with zeros, where no
piece is cut, and nothing of a neighbour gets in."""
import numpy as np
import pytest

from tests.gpu_harness import Device

pytestmark = pytest.mark.gpu

SETS = {
    "one_workgroup": [1, 2, 3, 5, 31, 33, 34, 63, 127, 1021, 1022, 4095, 8190, 16381, 16387, 32765],
    "small_tiles": [32769, 32771, 65534, 65537, 1 << 17, 131070, 262143, 262149, 7],          # columns of 2^8 to 2^9
    "columns_to_2^10": [3, 65537, 131069, 131075, 262142, 524287, 524285, (1 << 20) - 1, (1 << 20) + 6, 70001],
    "whole_tiles": [40001, 65537, 131069, 131075, 262142, 524287, 524285, (1 << 20) - 1, (1 << 20) + 6],  # no short ones: columns of 2^8 to 2^10
    "whole_tiles_of_2^11": [40001, 300002, (1 << 20) + 6, (1 << 22) - 3],
    "columns_of_2^11": [1, 40001, 131074, 600003, (1 << 21) + 5, (1 << 22) - 2, 50002],
}


@pytest.fixture(scope="module")
def dev():
    return Device()


@pytest.mark.parametrize("name", SETS)
def test_tensors_start_and_end_anywhere(dev, ref, name):
    torch, f, sizes, theta, bits = dev.torch, dev.f, SETS[name], 0.5, 12
    offs = [int(v) for v in np.concatenate([[0], np.cumsum(sizes)])]
    gen = torch.Generator(device="cuda").manual_seed(len(sizes))
    g = torch.randn(offs[-1], device="cuda", generator=gen)
    for i in range(1, len(sizes), 2):  # neighbours of another size altogether
        g[offs[i]:offs[i + 1]] *= 1e6
    packed = torch.full((f.packed_bytes_segments(offs, theta, bits),), 0xEE, dtype=torch.uint8, device="cuda")
    out = torch.full((offs[-1],), float("nan"), device="cuda")
    ws = dev.workspace(f.workspace_bytes_segments(offs, bits))
    f.compress_segments(g, offs, theta, bits, packed, ws)
    f.decompress_segments(packed, packed.numel(), out, offs, theta, bits, ws)
    assert f.device_status(ws) == 0
    pos = 64
    for i, s in enumerate(sizes):
        L = ref.segment_length(s)
        print(f"{name}: tensor {i} of {s} from {offs[i]}", flush=True)
        x = torch.zeros(L, device="cuda")
        x[:s] = g[offs[i]:offs[i + 1]]
        one, back = torch.empty(f.packed_bytes(L, L, theta, bits), dtype=torch.uint8, device="cuda"), torch.empty_like(x)
        work = dev.ws_for(L, L, bits)
        f.compress(x, L, theta, bits, one, work)
        f.decompress(one, one.numel(), back, L, theta, bits, work)
        S = one.numel() - 64
        got, want = packed[pos:pos + S].clone(), one[64:].clone()
        got[12:16] = 0  # a per-tensor record carries its chunk length
        want[12:16] = 0
        assert torch.equal(got, want)
        assert torch.equal(out[offs[i]:offs[i + 1]].view(torch.int32), back[:s].view(torch.int32))
        pos += S
    assert pos == packed.numel()
