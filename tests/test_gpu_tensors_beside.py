"""Sets of tensors: those of one workgroup each and the first kernel of a few longer ones, twenty-two at most, are one launch
(csrc/chunk.hip), whether every workgroup has a compute unit to itself or not.  Every record and every sample is what a call with that
tensor as its only chunk gives, bit for bit, on either side of that line; a bitmap that claims too many bins is reported."""
import pytest
import torch

from paper_1811_08596_amd import fftsp, workloads
from tests.test_gpu_tensor_rows import check_alone

pytestmark = pytest.mark.gpu

# A sender's longer tensor of 2^16 is 16 workgroups, a receiver's 32; a shorter one of 2^13 samples or more is one.
SETS = {
    "ResNet-20": workloads.resnet20_sizes(),
    "the shortest, and one of 2^18": [1, 200003],
    "shorter ones of 2^5 to 2^15, one of 2^17 and one of 2^18": [32768, 32767, 16385, 9000, 4097, 2049, 700, 300, 100, 64, 33, 7, 131072, 131075],
    "sender alone: one of 2^20": [20000, 5, 1000001],
    "sender, halves of the LDS: columns of 2^8 to 2^11": [20000, 5, 40001, 131072, 300001, 600003, 1048577, 2097155],
    "the same, as many as go": [9000] * 3 + [2097151] * 7 + [70001, 100003],
    "the same, one more": [9000] * 3 + [2097151] * 8,
    "beside brief ones, as many as go": [500, 4096] + [1048577] * 4,
    "beside brief ones, more": [500, 4096] + [1048577] * 4 + [40000],
    "a compute unit to every workgroup": [9000] * 32 + [60001] * 7,
    "more workgroups than compute units": [8193] * 65 + [40001] * 12,
    "as many of either as go": [20001] * 128 + [60001] * 9 + [100001] * 8 + [200001] * 2,
    "sender alone: many tiles of rows of 2^8": [300] * 20 + [150001] * 10,
    "two launches of shorter ones": [300] * 129 + [60001] * 2,
    "twenty long ones": [300] + [40001] * 20,
    "as many long ones as go": [300] + [40001] * 22,
    "one more of them": [300] + [40001] * 23,
    "twenty-two, halves of the LDS": [9000] * 20 + [70001] * 9 + [200001] * 6 + [300001] * 4 + [1100001] * 3,
    "nineteen, halves of the LDS": [9000] * 20 + [70001] * 6 + [200001] * 6 + [300001] * 4 + [1100001] * 3,
}


@pytest.mark.parametrize("theta,bits", [(0.3, 6), (0.5, 8), (0.1, 12), (0.2, 32), (0.0, 8)])
@pytest.mark.parametrize("name", list(SETS))
def test_every_tensor_is_what_it_is_alone(name, theta, bits):
    check_alone(name, SETS[name], theta, bits)


TABLES = [300, 9000, 300001, 600003, 1048577, 2097155]  # the bitmaps' table of the longer ones is beside the short ones


class Stream:
    def __init__(self, sizes, theta=0.3, bits=8):
        self.sizes, self.theta, self.bits, self.offsets = sizes, theta, bits, [0]
        for s in sizes:
            self.offsets.append(self.offsets[-1] + s)
        grad = torch.randn(self.offsets[-1], device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
        self.packed = torch.empty(fftsp.packed_bytes_segments(self.offsets, theta, bits), dtype=torch.uint8, device="cuda")
        self.work = torch.empty(fftsp.workspace_bytes_segments(self.offsets, bits), dtype=torch.uint8, device="cuda")
        self.out = torch.empty_like(grad)
        fftsp.compress_segments(grad, self.offsets, theta, bits, self.packed, self.work)

    def status(self, theta=None):
        fftsp.decompress_segments(self.packed, self.packed.numel(), self.out, self.offsets, theta or self.theta, self.bits, self.work)
        return fftsp.device_status(self.work)


# a short one of ResNet-20's tensors and one of 2^16; a short one and two long ones of a set whose bitmaps' table is beside the short ones
@pytest.mark.parametrize("name,tensor", [("ResNet-20", 1), ("ResNet-20", 21), ("tables", 0), ("tables", 2), ("tables", 5)])
def test_a_wrong_bitmap_is_reported(name, tensor):
    st = Stream(sorted(SETS.get(name, TABLES)))
    assert st.status() == 0
    at = 64
    for s in st.sizes[:tensor]:
        length = max(32, 1 << (s - 1).bit_length())
        at += fftsp.packed_bytes(s, length, st.theta, st.bits) - 64
    st.packed[at + 16:at + 18] = 255
    assert st.status() == 6


# Receivers whose first kernel has the shorter and the longer tensors, either kind of it; launches of their own; and sets of one kind of tensors.  The
# stream's header is looked at once, by whichever kernel is the call's first.
@pytest.mark.parametrize("name", ["ResNet-20", "tables", "two launches of shorter ones", "sender alone: many tiles of rows of 2^8", "shorter ones", "longer ones"])
def test_a_wrong_header_is_reported(name):
    st = Stream({"tables": TABLES, "shorter ones": [300, 9000], "longer ones": [60001] * 2}.get(name) or SETS[name])
    assert st.status() == 0
    for word in (0, 1, 2, 3, 5, 6, 7, 12):  # what it is, its version, samples, tensors, code bits, mantissa, scale
        st.packed[4 * word] ^= 1
        assert st.status() == 6, word
        st.packed[4 * word] ^= 1
        assert st.status() == 0, word
    assert st.status(theta=0.25) == 6  # a shorter stream, other numbers of kept bins
    assert st.status() == 0
