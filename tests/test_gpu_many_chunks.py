"""Receivers of streams with more than 2^20 chunks: the per-record verdicts lie beyond 2^32 words of the workspace (16 KiB
of histogram a chunk; 34 GB here).  Every receiver against the oracle, and a fault in the last record is reported."""
import numpy as np
import pytest

from tests.gpu_harness import Device, rel_l2

pytestmark = pytest.mark.gpu

L, THETA, BITS = 32, 0.3, 8
N = ((1 << 20) + 1) * L - 9


@pytest.fixture(scope="module")
def dev():
    d = Device()
    yield d
    d.torch.cuda.empty_cache()


@pytest.fixture(scope="module")
def work(dev):
    return dev.workspace(dev.f.workspace_bytes_accumulate(N, L, BITS, 2))


@pytest.mark.parametrize("receiver", ["decompress", "decode_spectrum", "topk", "accumulate", "decode_accumulate"])
def test_receivers_of_many_chunks(dev, ref, work, receiver):
    print(f"many chunks: {receiver}", flush=True)
    f, torch = dev.f, dev.torch
    g = (np.random.default_rng(5).laplace(size=N) * 1e-3).astype(np.float32)
    make, stride = (ref.topk_compress, ref.topk_record_stride) if receiver == "topk" else (ref.compress, ref.record_stride)
    packed = make(g, L, THETA, BITS, nthreads=8)
    k = (ref.topk_kept_per_chunk if receiver == "topk" else ref.kept_per_chunk)(L, THETA)
    bad = packed.copy()
    bad[packed.size - stride(L, k, BITS) + 16] ^= 1    # one bit too many or too few in the last record's bitmap
    bins = receiver.startswith("decode")
    out = torch.empty(-(-N // L) * (L + 2) if bins else N, dtype=torch.float32, device=dev.dev)
    first = dev.to_dev(packed)
    for stream, status in ((packed, 0), (bad, 6)):
        last = dev.to_dev(stream)
        if receiver == "decompress":
            f.decompress(last, last.numel(), out, L, THETA, BITS, work)
        elif receiver == "decode_spectrum":
            f.decode_spectrum(last, last.numel(), N, L, THETA, BITS, out, work)
        elif receiver == "topk":
            f.topk_decompress(last, last.numel(), out, L, THETA, BITS, work)
        elif receiver == "accumulate":
            f.decompress_accumulate([first, last], last.numel(), 0.5, out, L, THETA, BITS, work)
        else:
            f.decode_accumulate_spectrum([first, last], last.numel(), N, L, THETA, BITS, out, work)
        assert f.device_status(work) == status
        if status:
            continue
        got = out.cpu().numpy()
        if receiver == "decode_spectrum":
            assert np.array_equal(got.view(np.uint32), ref.decode_spectrum(packed, N, L, THETA, BITS, nthreads=8).view(np.uint32))
        elif receiver == "decode_accumulate":
            want = ref.decode_accumulate_spectrum([packed, packed], N, L, THETA, BITS, nthreads=8)
            assert np.array_equal(got.view(np.uint32), want.view(np.uint32))
        elif receiver == "topk":
            assert np.array_equal(got.view(np.uint32), ref.topk_decompress(packed, N, L, THETA, BITS, nthreads=8).view(np.uint32))
        else:  # the same stream twice, halved, is the stream
            assert rel_l2(got, ref.decompress(packed, N, L, THETA, BITS, nthreads=8)) <= 1e-5
