"""Launch sets of tensors whose transforms have second passes of different row lengths: one launch for all of them (csrc/fft.hip, csrc/receive.hip).

A workgroup of that launch does one tile of rows of 2^10, two of 2^9, four of 2^8 or eight of 2^7.  Every record and every sample has to
be what a call with that tensor as its only chunk gives, bit for bit, on either side of the receivers' line (256 tiles of 2^13 points where
rows of 2^10 are among them)."""
import pytest
import torch

from paper_1811_08596_amd import fftsp

pytestmark = pytest.mark.gpu

# (samples, how many): the padded length is the next power of two; 2^16 has rows of 2^7, 2^17 and 2^18 of 2^8, 2^19 and 2^20 of 2^9, 2^21 and 2^22 of 2^10
SETS = {
    "rows of 2^7 and 2^10, odd": [(65535, 9), (1048577, 1), (2097151, 1)],
    "rows of every length": [(40001, 3), (131072, 1), (200003, 2), (524288, 1), (1000001, 1), (2000003, 1), (4000001, 1)],
    "below the receivers' line": [(65536, 3), (300000, 3), (1100000, 1)],
    "just below it, then at it": [(65536, 31), (2097152, 1), (33000, 1)],
    "at it": [(65536, 32), (2097152, 1), (33000, 1), (32, 1)],
    "one short tensor beside long ones": [(40000, 1), (1500000, 4)],
    "rows of every length, few tiles": [(40001, 1), (131072, 1), (200003, 1), (524288, 2), (1500000, 1)],
    "rows of 2^10 alone": [(1500000, 4), (3000001, 1)],
}


@pytest.mark.parametrize("theta,bits", [(0.3, 8), (0.15, 11), (0.6, 6)])
@pytest.mark.parametrize("name", list(SETS))
def test_every_tensor_is_what_it_is_alone(name, theta, bits):
    check_alone(name, [s for s, many in SETS[name] for _ in range(many)], theta, bits)


def check_alone(name, sizes, theta, bits):
    dev = torch.device("cuda")
    sizes = sizes[::2] + sizes[1::2]  # not in the order of their lengths
    offsets = [0]
    for s in sizes:
        offsets.append(offsets[-1] + s)
    gen = torch.Generator(device=dev)
    gen.manual_seed(7)
    grad = torch.randn(offsets[-1], device=dev, generator=gen)
    packed = torch.empty(fftsp.packed_bytes_segments(offsets, theta, bits), dtype=torch.uint8, device=dev)
    work = torch.empty(fftsp.workspace_bytes_segments(offsets, bits), dtype=torch.uint8, device=dev)
    out = torch.full_like(grad, float("nan"))
    fftsp.compress_segments(grad, offsets, theta, bits, packed, work)
    fftsp.decompress_segments(packed, packed.numel(), out, offsets, theta, bits, work)
    assert fftsp.device_status(work) == 0
    at = 64
    for i, n in enumerate(sizes):
        length = max(32, 1 << (n - 1).bit_length())
        g = grad[offsets[i]:offsets[i + 1]].clone()
        one = torch.empty(fftsp.packed_bytes(n, length, theta, bits), dtype=torch.uint8, device=dev)
        w = torch.empty(fftsp.workspace_bytes(n, length, bits), dtype=torch.uint8, device=dev)
        alone = torch.empty_like(g)
        fftsp.compress(g, length, theta, bits, one, w)
        fftsp.decompress(one, one.numel(), alone, length, theta, bits, w)
        size = one.numel() - 64
        here, there = packed[at:at + size].clone(), one[64:].clone()
        here[12:16] = 0  # a tensor's record says its length there
        there[12:16] = 0
        assert torch.equal(here, there), (name, i, n)
        assert torch.equal(out[offsets[i]:offsets[i + 1]], alone), (name, i, n)
        at += size
    assert at == packed.numel()
