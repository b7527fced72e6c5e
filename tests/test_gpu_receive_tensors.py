"""Per-tensor receivers take the inverse's first pass straight from the records as well (csrc/receive.hip): every row length, each
alone in its launch or beside others, at the narrowest and widest codes.  Every tensor comes back with the bits that its decoded
spectrum (decode_spectrum) and its inverse give, and a bitmap that claims too many bins is reported."""
import numpy as np
import pytest

from tests.gpu_harness import Device

pytestmark = pytest.mark.gpu

SETS = {
    "every_length": [50000, 1 << 16, 100004, 1 << 17, 200001, 1 << 18, 300000, 1 << 19, 700004, (1 << 20) - 3, 1 << 20, 1 << 21,
                     3000000, 1 << 22, 1 << 22, 12, 4096],
    "rows_of_up_to_2^9": [60000 + 91 * i for i in range(20)] + [(1 << 17) - 7, 1 << 18] * 8 + [(1 << 19) - 8, 1 << 20, (1 << 20) - 1, 9],
    "rows_of_2^9": [(1 << 19) - 8, 1 << 20, (1 << 20) - 1],
    "rows_of_2^10": [(1 << 21) - 9, 1 << 22],
}


@pytest.fixture(scope="module")
def dev():
    return Device()


# launch sets of few tiles, which go through csrc/short.hip wholly or in one pass
SHORT_SETS = {
    "one_of_2^21": [(1 << 21) - 9, 77],                                    # the tallest rows there
    "2^18_and_2^19": [(1 << 18) - 3] * 9 + [(1 << 19) - 8, 1 << 19],       # more than 192 tiles: the others' forward passes
    "2^21_and_short_ones": [1 << 21] + [(1 << 16) - 1] * 17,               # the same, and the tallest rows' inverse passes
    "2^16_and_a_tall_one": [1 << 16] * 20 + [(1 << 18) - 1],
}


@pytest.mark.parametrize("bits", (3, 8, 9, 15))
@pytest.mark.parametrize("name", SETS)
def test_tensors_and_the_spectra_they_leave_out(dev, ref, name, bits):
    check(dev, ref, name, SETS[name], bits)


@pytest.mark.parametrize("bits", (8, 16, 32))
@pytest.mark.parametrize("name", SHORT_SETS)
def test_short_launch_sets(dev, ref, name, bits):
    check(dev, ref, name, SHORT_SETS[name], bits)


def check(dev, ref, name, sizes, bits):
    torch, f = dev.torch, dev.f
    offs = [int(v) for v in np.concatenate([[0], np.cumsum(sizes)])]
    g = torch.randn(offs[-1], device="cuda", generator=torch.Generator(device="cuda").manual_seed(bits)) * 1e-2
    ws = dev.workspace(f.workspace_bytes_segments(offs, bits))
    out = torch.empty_like(g)
    for theta in (1.0, 0.4, 0.0):
        print(f"{name} bits={bits} theta={theta}", flush=True)
        nb = f.packed_bytes_segments(offs, theta, bits)
        packed = torch.empty(nb, dtype=torch.uint8, device="cuda")
        f.compress_segments(g, offs, theta, bits, packed, ws)
        f.decompress_segments(packed, nb, out, offs, theta, bits, ws)
        assert f.device_status(ws) == 0
        for i, n in enumerate(sizes):
            L = ref.segment_length(n)
            if L < 1 << 16:
                continue
            x, work = g[offs[i]:offs[i + 1]].clone(), dev.ws_for(n, L, bits)
            one = torch.empty(f.packed_bytes(n, L, theta, bits), dtype=torch.uint8, device="cuda")
            spec, want = torch.empty(L + 2, device="cuda"), torch.empty_like(x)
            f.compress(x, L, theta, bits, one, work)
            f.decode_spectrum(one, one.numel(), n, L, theta, bits, spec, work)
            f.irfft(spec, n, L, want, work)
            assert torch.equal(out[offs[i]:offs[i + 1]].view(torch.int32), want.view(torch.int32)), i
    last = ref.segment_length(sizes[0]) // 16
    packed[64 + 16:64 + 16 + last] = 255  # every bin, in the first record
    f.decompress_segments(packed, nb, out, offs, theta, bits, ws)
    assert f.device_status(ws) != 0
