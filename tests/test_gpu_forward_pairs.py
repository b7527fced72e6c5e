"""The forward second pass with a tile in half of the LDS (csrc/fft.hip, fwd_b_pairs): in binary16 calls of more than the short kernels' tiles,
a chunk's record and its samples are the bits that the chunk has on its own.  (Tensors' launches: test_gpu_receive_pairs.py.)"""
import pytest

from tests.gpu_harness import Device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return Device()


@pytest.mark.parametrize("theta,bits", [(0.3, 8), (1.0, 32)])
@pytest.mark.parametrize("log_l", (17, 18, 19, 20, 21, 22))
def test_a_chunk_alone_and_among_others(dev, log_l, theta, bits):
    f, torch, L = dev.f, dev.torch, 1 << log_l
    chunks = max(3, 1100 >> (log_l - 14))  # tiles of 2^13
    g = torch.randn(chunks * L, device="cuda", generator=torch.Generator(device="cuda").manual_seed(log_l)) * 1e-3

    def records(x):
        n = x.numel()
        ws = dev.ws_for(n, L, bits)
        packed, out = torch.empty(f.packed_bytes(n, L, theta, bits), dtype=torch.uint8, device="cuda"), torch.empty(n, device="cuda")
        f.compress_h(x, L, theta, bits, 8, packed, ws)
        f.decompress_h(packed, packed.numel(), out, L, theta, bits, 8, ws)
        assert f.device_status(ws) == 0
        return packed[64:].view(n // L, -1), out.view(torch.int32).view(n // L, -1)

    print(f"2^{log_l}, {chunks} chunks, theta={theta} bits={bits}", flush=True)
    many = records(g)
    for c in (0, chunks - 1):
        one = records(g[c * L:(c + 1) * L].clone())
        assert torch.equal(many[0][c], one[0][0]) and torch.equal(many[1][c], one[1][0])
