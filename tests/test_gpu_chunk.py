"""Chunk-resident sender and receiver (csrc/chunk.hip; chunk lengths up to 2^15) against the stage-level entry points,
which run the per-tile kernels: the packed bytes must be those of rfft + encode_spectrum, and the receiver must give the
oracle's samples.  Every geometry of the kernels (lanes per chunk, chunks per workgroup), a last workgroup that is only
partly filled, every way codes are stored, and inputs whose threshold falls into a run of equal keys: an impulse
(all magnitudes equal up to rounding), zeros (one key for every bin), a period (few non-zero bins)."""
import numpy as np
import pytest

from paper_1811_08596_amd import workloads
from tests.gpu_harness import Device, rel_l2

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return Device()


def signals(L, chunks, tail):
    n = chunks * L - tail
    yield "laplace", workloads.small_mixed(n, seed=L % 89)
    g = np.zeros(n, np.float32)
    g[::L] = 1.0
    yield "impulses", g
    yield "zeros", np.zeros(n, np.float32)
    yield "period", np.tile(np.array([1, -2, 3, 0.5], np.float32), n // 4 + 1)[:n].copy()


@pytest.mark.parametrize("logL", range(5, 16))
def test_sender_equals_stages_and_receiver_matches_the_oracle(dev, ref, logL):
    L = 1 << logL
    chunks = max(3, (1 << 13 >> logL) + 2)                # more than one workgroup, the last one not full
    for name, g in signals(L, chunks, L // 3 + 1):
        spec = dev.rfft(g, L)
        for theta, bits in ((0.3, 8), (0.15, 10), (1.0, 16), (0.5, 32), (0.02, 3), (0.0, 8)):
            print(f"L=2^{logL} {name} theta={theta} bits={bits}", flush=True)
            got = dev.compress(g, L, theta, bits)
            assert np.array_equal(got, dev.encode(spec, g.size, L, theta, bits))
            out, st = dev.decompress(got, g.size, L, theta, bits, want_status=True)
            want = ref.decompress(got, g.size, L, theta, bits)
            assert st == 0 and np.isfinite(out).all()
            assert rel_l2(out, want) <= 1e-5 or np.abs(out - want).max() <= 1e-6 * max(np.abs(g).max(), 1e-30)


def test_status_is_per_call_and_per_record(dev, ref):
    L, n, theta, bits = 1 << 10, 37 * (1 << 10) - 5, 0.4, 8
    packed = ref.compress(workloads.small_mixed(n, seed=3), L, theta, bits)
    S = (packed.size - 64) // 37
    bad = packed.copy()
    bad[64 + 36 * S + 16] ^= 1                            # one bit too many or too few in the last record's bitmap
    t, f = dev.torch, dev.f
    ws = dev.ws_for(n, L, bits)
    out = t.empty(n, dtype=t.float32, device=dev.dev)
    for stream, want in ((packed, 0), (bad, 6), (packed, 0)):
        f.decompress(dev.to_dev(stream), packed.size, out, L, theta, bits, ws)
        assert f.device_status(ws) == want
    f.decompress(dev.to_dev(bad), packed.size, out, L, theta, bits, ws)
    f.compress(out, L, theta, bits, t.empty(packed.size, dtype=t.uint8, device=dev.dev), ws)
    assert f.device_status(ws) == 0                       # another call on the same workspace starts clean


@pytest.mark.parametrize("logL", range(5, 16))
def test_topk_sender_matches_the_oracle(dev, ref, logL):
    L = 1 << logL
    chunks = max(3, (1 << 13 >> logL) + 2)                # more than one workgroup, the last one not full
    for name, g in signals(L, chunks, L // 3 + 1):
        for theta, bits in ((0.3, 8), (0.15, 10), (1.0, 16), (0.5, 32), (0.02, 3), (0.0, 8)):
            print(f"topk L=2^{logL} {name} theta={theta} bits={bits}", flush=True)
            want = ref.topk_compress(g, L, theta, bits)
            assert np.array_equal(dev.topk_compress(g, L, theta, bits), want)
