"""What the entry points enqueue, without a GPU: a recording stand-in for the HIP runtime is loaded in front of the
library in a process of its own, so host-side decisions (which calls are taken, which launches they become) can be looked at
for sizes no CPU test could compute.  Device addresses are made up; nothing dereferences them."""
import json
import os
import re
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RUNTIME = r"""
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
typedef struct { uint32_t x, y, z; } dim3;
typedef int (*any)(void);
static struct { const void* f; char name[200]; } known[4096];
static int n_known;
static FILE* out;
static dim3 grid, block;
static size_t lds;
static void* stream;
static const char* name_of(const void* f)
{
    for (int i = 0; i < n_known; ++i) if (known[i].f == f) return known[i].name;
    return "?";
}
static void say(const char* what, const void* f, size_t a, size_t b)
{
    if (!out) out = fopen(getenv("LAUNCH_LOG"), "w");
    fprintf(out, "%s %s %zu %zu\n", what, name_of(f), a, b);
    fflush(out);
}
void** __hipRegisterFatBinary(const void* d) { static void* h; (void)d; return &h; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterFunction(void** m, const void* f, char* df, const char* name, unsigned t, void* a, void* b, void* c, void* d, int* w)
{
    if (n_known < 4096) { known[n_known].f = f; strncpy(known[n_known++].name, name, 199); say("has", f, 0, 0); }
}
void __hipRegisterVar(void** m, void* v, char* h, char* d, int e, size_t s, int c, int g) {}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t l, void* s) { grid = g; block = b; lds = l; stream = s; return 0; }
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* l, void** s) { *g = grid; *b = block; *l = lds; *s = stream; return 0; }
int hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t l, void* s) { say("launch", f, (size_t)g.x * b.x, l); return 0; }
int hipFuncSetAttribute(const void* f, int attr, int value) { say("lds", f, (size_t)value, (size_t)attr); return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetSymbolAddress(void** p, const void* s) { *p = (void*)(uintptr_t)0x10000; return 0; }
int hipGetLastError(void) { return 0; }
int hipStreamGetCaptureInfo(void* s, int* st, unsigned long long* id) { *st = 0; *id = 0; return 0; }
int hipStreamCreateWithFlags(void** s, unsigned f) { *s = (void*)(uintptr_t)0x20000; return 0; }
int hipStreamDestroy(void* s) { return 0; }
int hipStreamWaitEvent(void* s, void* e, unsigned f) { return 0; }
int hipEventCreateWithFlags(void** e, unsigned f) { *e = (void*)(uintptr_t)0x30000; return 0; }
int hipEventDestroy(void* e) { return 0; }
int hipEventRecord(void* e, void* s) { return 0; }
"""


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    d = tmp_path_factory.mktemp("runtime")
    src, so = d / "runtime.c", d / "runtime.so"
    src.write_text(RUNTIME)
    subprocess.run(["gcc", "-O1", "-w", "-shared", "-fPIC", "-o", str(so), str(src)], check=True)
    return str(so)


def calls_made(runtime, tmp_path, calls):
    """Runs the calls (entry point, arguments; "big" stands for a buffer that is large enough) in a process behind the
    recording runtime.  Returns their statuses and what was recorded: (what, kernel, number, number)."""
    log = tmp_path / "log"
    program = textwrap.dedent("""
        import ctypes, json, os, sys
        ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
        from paper_1811_08596_amd import fftsp
        lib, status = fftsp.load(), []
        for name, args in json.load(sys.stdin):
            f = getattr(lib, name)
            given = []
            for a, t in zip(args, f.argtypes):
                if a == "big":
                    a = 1 << 60 if t is ctypes.c_size_t else 1 << 40
                elif isinstance(a, list):
                    a = (t._type_ * len(a))(*a)
                given.append(a)
            status.append(f(*given))
        print(json.dumps(status))
    """)
    r = subprocess.run([sys.executable, "-c", program, runtime], input=json.dumps(calls), capture_output=True, text=True,
                       cwd=ROOT, env={**os.environ, "LAUNCH_LOG": str(log)}, timeout=120)
    assert r.returncode == 0, r.stderr
    rows = [line.split() for line in log.read_text().splitlines()] if log.exists() else []
    return json.loads(r.stdout), [(a, b, int(c), int(d)) for a, b, c, d in rows]


def decompress(n, L, theta=0.3, bits=8):
    return ["fftsp_decompress", ["big", "big", "big", n, L, theta, bits, "big", "big", None]]


def accumulate(n, L, peers=2):
    return ["fftsp_decompress_accumulate", [[1 << 40] * peers, peers, "big", 0.5, "big", n, L, 0.3, 8, "big", "big", None]]


def compress(n, L, theta=0.3, bits=8):
    return ["fftsp_compress", ["big", n, L, theta, bits, "big", "big", "big", "big", None]]


def segments(sizes, theta, bits):
    offs = [0]
    for s in sizes:
        offs.append(offs[-1] + s)
    return [["fftsp_compress_segments", ["big", offs, len(sizes), theta, bits, "big", "big", "big", "big", None]],
            ["fftsp_decompress_segments", ["big", "big", "big", offs, len(sizes), theta, bits, "big", "big", None]]]


def test_lds_limit_of_a_kernel_does_not_depend_on_the_call(runtime, tmp_path):
    """The limit belongs to the kernel on the device, so two threads' calls must set the same value, one that covers both."""
    calls = []
    for theta, bits in ((0.0, 8), (0.3, 8), (1.0, 16), (1.0, 32)):
        for logL in range(5, 23):
            L = 1 << logL
            calls += [compress(3 * L, L, theta, bits), decompress(3 * L, L, theta, bits), accumulate(3 * L, L)]
            if logL <= 21:
                calls += [["fftsp_topk_compress", ["big", 3 * L, L, theta, bits, "big", "big", "big", "big", None]],
                          ["fftsp_topk_decompress", ["big", "big", "big", 3 * L, L, theta, bits, "big", "big", None]]]
        for top in (50, 4096, 1 << 15, 1 << 17, 1 << 22):
            calls += segments([top // 2 + 1, top], theta, bits)
    status, rows = calls_made(runtime, tmp_path, calls)
    assert status == [0] * len(calls)
    limits = {}
    for what, kernel, a, b in rows:
        if what == "lds":
            limits.setdefault(kernel, set()).add(a)
    assert {k: v for k, v in limits.items() if len(v) > 1} == {}
    for what, kernel, threads, lds in rows:
        if what == "launch" and lds > 48 * 1024:
            assert lds <= min(limits[kernel]) <= 160 * 1024, kernel


def test_receivers_take_as_many_chunks_as_senders(runtime, tmp_path):
    """Short chunks of long gradients: the verdicts lie beyond 2^32 words of the workspace (16 KiB of histogram a chunk)."""
    n = 62378344
    calls = [decompress(n, 32), decompress(138357544, 128), accumulate(n, 64), accumulate(n, 32, 8),
             ["fftsp_topk_decompress", ["big", "big", "big", n, 32, 0.3, 8, "big", "big", None]],
             ["fftsp_decode_spectrum", ["big", "big", n, 32, 0.3, 8, "big", "big", "big", None]],
             ["fftsp_decode_accumulate_spectrum", [[1 << 40] * 2, 2, "big", n, 64, 0.3, 8, "big", "big", "big", None]],
             ["fftsp_compress", ["big", n, 32, 0.3, 8, "big", "big", "big", "big", None]]]
    status, _ = calls_made(runtime, tmp_path, calls)
    assert status == [0] * len(calls)


def kernels(runtime, tmp_path, calls):
    """names of the kernels each call launches"""
    made = []
    for i, call in enumerate(calls):
        d = tmp_path / str(i)
        d.mkdir()
        status, rows = calls_made(runtime, d, [call])
        assert status == [0]
        made.append([kernel for what, kernel, _, _ in rows if what == "launch"])
    return made


@pytest.mark.parametrize("logL, half, most", [(16, 0, 48), (17, 0, 24), (18, 0, 12), (19, 0, 6), (20, 0, 3), (21, 0, 1), (16, 1, 32), (18, 1, 8)])
def test_senders_leave_the_small_tiles_where_they_stop_paying(runtime, tmp_path, logL, half, most):
    L = 1 << logL
    calls = [["fftsp_compress_h", ["big", C * L, L, 0.5, 8, 0, "big", "big", "big", "big", None]] if half else compress(C * L, L, 0.5)
             for C in (most, most + 1)]
    small, large = kernels(runtime, tmp_path, calls)
    assert any("k_fwd_a_short" in k for k in small) and not any("short" in k for k in large)


@pytest.mark.parametrize("sizes, send, receive_a", [
    ([1 << 18] * 12, True, True), ([1 << 18] * 13, False, True), ([1 << 18] * 20, False, True), ([1 << 18] * 21, False, False),
    ([1 << 16] * 16 + [1 << 21], True, True), ([1 << 16] * 17 + [1 << 21], False, True), ([1 << 17] * 8 + [1 << 21] * 2, False, True),
    ([1 << 17] * 9 + [1 << 21] * 2, False, False)])
def test_tensors_leave_the_small_tiles_where_they_stop_paying(runtime, tmp_path, sizes, send, receive_a):
    sender, receiver = kernels(runtime, tmp_path, segments(sizes, 0.5, 8))
    assert any("k_fwd_a_long_short" in k for k in sender) == send
    assert any("k_inv_a_long_short" in k for k in receiver) == receive_a


# tiles of 2^14 points: a tensor of 2^18 is eight of them, of 2^21 64 and of 2^22 128
@pytest.mark.parametrize("sizes, kernel", [
    ([1 << 18] * 12, "short"), ([1 << 18] * 13, "long"), ([1 << 18] * 16, "long"), ([1 << 21] * 8, "long"), ([1 << 21] * 8 + [1 << 16], "split"), ([1 << 22], "long"),
    ([1 << 21] * 4, "long"), ([1 << 21] * 4 + [1 << 16], "split"), ([1 << 21] * 5 + [1 << 19], "long"), ([1 << 18] * 33, "long"), ([1 << 22, 1 << 21], "long"), ([1 << 22, 1 << 22], "split"), ([(1 << 19) - 5] * 32, "long"), ([(1 << 19) - 5] * 33, "split")])
def test_few_tensors_have_their_first_pass_whole_in_the_lds(runtime, tmp_path, sizes, kernel):
    sender, _ = kernels(runtime, tmp_path, segments(sizes, 0.5, 8))
    first, = [k for k in sender if "k_fwd_a" in k]
    assert kernel == ("short" if "long_short" in first else "split" if "split" in first else "long")


# the same tiles
@pytest.mark.parametrize("sizes, kernel", [
    ([1 << 21] + [1 << 18] * 4, "short"), ([1 << 21] + [1 << 18] * 5, "small"), ([1 << 21] + [1 << 20] * 2, "small"), ([1 << 21] * 2 + [1 << 16], "small"),
    ([1 << 21] * 2 + [1 << 16] * 2, "pairs"), ([1 << 21] * 2, "large"), ([1 << 18] * 16, "pairs")])
def test_few_tensors_of_both_rows_have_a_tile_for_every_compute_unit(runtime, tmp_path, sizes, kernel):
    sender, _ = kernels(runtime, tmp_path, segments(sizes, 0.5, 8))
    second, = [k for k in sender if "k_fwd_b" in k]
    assert kernel == ("short" if "long_short" in second else "pairs" if "pairs" in second else "small" if "ILi13E" in second else "large" if "ILi14E" in second else second)


# a tensor of 2^18 is 64 workgroups of a receiver's inverse pass B, of 2^17 and 2^16 32, with a quarter and an eighth of the lanes
@pytest.mark.parametrize("shorter, longer, beside", [
    ([300] * 128, [1 << 18] * 7, True), ([300] * 128, [1 << 18] * 8, False), ([300], [1 << 18] * 8, False), ([4096] * 20, [1 << 17] * 15, True),
    ([4096] * 20, [1 << 17] * 16, False), ([300] * 128, [1 << 16] * 19, True), ([300] * 20, [1 << 19] * 9, True), ([9000] * 128, [1 << 18] * 9, True),
    ([9000] * 128, [1 << 18] * 10, False), ([9000], [1 << 18] * 13, True), ([30000] * 64, [1 << 18] * 18, True), ([30000] * 65, [1 << 18] * 15, False), ([30000] * 128, [1 << 18] * 14, True)])
def test_receivers_leave_the_shorter_tensors_launch_where_its_workgroups_lie_idle(runtime, tmp_path, shorter, longer, beside):
    _, receiver = kernels(runtime, tmp_path, segments(shorter + longer, 0.3, 8))
    assert ("beside" in receiver[0]) == beside and any("k_decode_inv_b_long" in k for k in receiver) == (not beside)


# chunks of 2^20 and 2^22 hold 32 and 128 tiles of 2^14 points
@pytest.mark.parametrize("logL, half, C, forward, inverse", [
    (19, 0, 16, False, True), (19, 1, 120, False, True), (20, 0, 31, False, True), (20, 0, 32, False, True), (20, 1, 31, False, True), (20, 1, 32, True, True),
    (22, 0, 1, False, False), (22, 0, 2, False, True), (22, 0, 4, False, True), (22, 0, 5, False, False), (22, 0, 7, False, False), (22, 0, 8, False, True),
    (22, 0, 14, True, True), (22, 1, 7, False, True), (22, 1, 9, False, True), (22, 1, 10, True, True)])
def test_first_passes_with_half_of_the_lds(runtime, tmp_path, logL, half, C, forward, inverse):
    L = 1 << logL
    n = C * L
    if half:
        calls = [["fftsp_compress_h", ["big", n, L, 0.5, 8, 0, "big", "big", "big", "big", None]],
                 ["fftsp_decompress_h", ["big", "big", "big", n, L, 0.5, 8, 0, "big", "big", None]]]
    else:
        calls = [compress(n, L, 0.5), ["fftsp_decompress", ["big", "big", "big", n, L, 0.5, 8, "big", "big", None]]]
    sender, receiver = kernels(runtime, tmp_path, calls)
    assert any("k_fwd_a_split" in k for k in sender) == forward
    assert any("k_inv_a_split" in k for k in receiver) == inverse


@pytest.mark.parametrize("logL, C, kernel", [(17, 24, "short"), (17, 32, "pairs"), (20, 4, "pairs"), (21, 1, "short"), (21, 2, "k_fwd_bI"), (21, 3, "pairs"),
                                             (22, 1, "k_fwd_bI"), (22, 2, "pairs"), (16, 64, "k_fwd_bI")])
def test_binary16_senders_take_half_of_the_lds_where_it_pays(runtime, tmp_path, logL, C, kernel):
    made, = kernels(runtime, tmp_path, [["fftsp_compress_h", ["big", C << logL, 1 << logL, 0.5, 8, 0, "big", "big", "big", "big", None]]])
    second, = [k for k in made if "k_fwd_b" in k]
    assert kernel in second


# tiles of a receiver's second pass: chunks of 2^16 hold 16 of them (rows of 2^7), of 2^17 and 2^18 16 and 32 (2^8), of 2^19 and 2^20 32 and 64 (2^9)
@pytest.mark.parametrize("logL, half, C, kernel", [
    (16, 0, 160, "b"), (16, 0, 161, "six"), (16, 0, 223, "six"), (16, 0, 224, "pairs"), (16, 1, 239, "b"), (16, 1, 240, "six"), (16, 1, 263, "six"), (16, 1, 264, "pairs"),
    (17, 0, 136, "b"), (17, 0, 137, "pairs"), (18, 0, 68, "b"), (18, 0, 69, "pairs"), (17, 1, 144, "b"), (17, 1, 145, "pairs"), (18, 1, 72, "b"), (18, 1, 73, "pairs"),
    (19, 0, 20, "pairs"), (19, 1, 32, "b"), (19, 1, 33, "pairs"), (20, 0, 5, "pairs"), (20, 1, 16, "b"), (20, 1, 17, "pairs"),
    (21, 0, 4, "b"), (21, 0, 5, "pairs"), (21, 1, 5, "pairs"), (22, 1, 3, "pairs")])
def test_receivers_take_half_of_the_lds_where_it_pays(runtime, tmp_path, logL, half, C, kernel):
    n, L = C << logL, 1 << logL
    made, = kernels(runtime, tmp_path, [["fftsp_decompress_h", ["big", "big", "big", n, L, 0.5, 8, 0, "big", "big", None]] if half else decompress(n, L)])
    second, = [k for k in made if "k_receive" in k]
    assert kernel == ("pairs" if "k_receive_pairs" in second else "six" if "ELi6EE" in second else "b")


def test_every_form_of_the_inverse_first_pass_is_reached(runtime, tmp_path):
    """The forms that the library has are those that receivers of all lengths launch."""
    calls = []
    for logL in range(15, 23):
        L = 1 << logL
        for n in (1 << 22, 3 << 22, 5 << 22, (1 << 25) - 1, 1 << 25, 1 << 26):
            calls += [["fftsp_decompress_h", ["big", "big", "big", n, L, 0.5, 8, 0, "big", "big", None]], decompress(n, L), accumulate(n, L)]
    status, rows = calls_made(runtime, tmp_path, calls)
    assert status == [0] * len(calls)
    has, launched = ({form for w, name, _, _ in rows if w == what for form in re.findall(r"k_inv_a(?:_split)?ILi.*?EEv", name)} for what in ("has", "launch"))
    assert len(has) > 10 and has == launched


# samples of a receiver from which its output passes the caches by
@pytest.mark.parametrize("call, logL, n, by", [
    ("one", 16, (1 << 25) - 1, False), ("one", 16, 1 << 25, True), ("one", 20, 1 << 25, True), ("one", 22, 1 << 25, True),
    ("peers", 17, (1 << 25) - 1, False), ("peers", 16, 1 << 25, True), ("peers", 18, 1 << 25, True), ("raw", 16, 1 << 25, True), ("raw", 19, (1 << 25) - 1, False),
    ("half", 15, 1 << 25, True), ("half", 17, (1 << 25) - 1, False), ("half", 17, 1 << 25, True), ("half", 22, 1 << 25, True)])
def test_outputs_that_pass_the_caches_by(runtime, tmp_path, call, logL, n, by):
    L = 1 << logL
    made, = kernels(runtime, tmp_path, [
        {"one": decompress(n, L), "peers": accumulate(n, L, 8), "raw": decompress(n, L, bits=32),
         "half": ["fftsp_decompress_h", ["big", "big", "big", n, L, 0.5, 8, 0, "big", "big", None]]}[call]])
    last, = [re.search(r"k_inv_a(?:_split)?ILi\d+ELi\d+ELb(\d)ELb(\d)E", k) for k in made if "k_inv_a" in k]
    assert (last[1] == "1") == (call == "half") and (last[2] == "1") == by


@pytest.mark.parametrize("L, most", [(1 << 16, 16), (1 << 17, 4)])
def test_topk_finds_its_threshold_beside_the_codes_in_short_calls(runtime, tmp_path, L, most):
    calls = [["fftsp_topk_compress", ["big", C * L, L, 0.3, 8, "big", "big", "big", "big", None]] for C in (most, most + 1)]
    within, beyond = kernels(runtime, tmp_path, calls)
    assert not any("k_resolve" in k for k in within) and any("k_resolve" in k for k in beyond)


def test_the_benchmarks_traffic_is_that_of_the_kernels_it_launches(runtime, tmp_path):
    """bench.py quotes a kernel's measured traffic from profiles/; its names and the summary's rows are the kernels of the step."""
    import bench
    n, L = 62378344, 1 << 20
    made = kernels(runtime, tmp_path, [compress(n, L, 0.5), decompress(n, L, 0.5)])
    launched = {re.search(r"\d(k_[a-z_]+?)I?(?=[A-Z])", name)[1].rstrip("_") for call in made for name in call}
    assert set(bench.TRAFFIC_KERNELS.values()) == launched
    with open(os.path.join(ROOT, "profiles", "codec_config3_hbm_traffic.txt")) as f:
        rows = {line.split()[0] for line in f if line.startswith("k_")}
    assert rows == launched and all(bench.measured_traffic(k)[0] for k in bench.TRAFFIC_KERNELS)
    assert bench.topk_kernel_bytes("sample", n, L, 0.15, 32) > 0
