"""Which tile a workgroup does (csrc/stretches.h), on the host: every tile is some workgroup's and no other one's, and no XCD has more than its
eighth, rounded up, of the tiles of either kind."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#include "%s/paper_1811_08596_amd/csrc/stretches.h"
extern "C" uint32_t tile(uint32_t place, uint32_t total) { return fftsp::stretch_tile(place, total); }
extern "C" uint32_t tile_of_two(uint32_t place, uint32_t total, uint32_t few) { return fftsp::stretch_tile(place, total, few); }
extern "C" uint32_t apart(uint32_t total, uint32_t few) { return fftsp::few_apart(total, few); }
extern "C" uint32_t turned(uint32_t place, uint32_t total, uint32_t step) { return fftsp::turned_tile(place, total, step); }
extern "C" uint32_t places(uint32_t total, uint32_t few) { return fftsp::stretch_places(total, few); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("stretches")
    (d / "s.cpp").write_text(SOURCE % ROOT)
    subprocess.run(["g++", "-O2", "-shared", "-fPIC", "-std=c++17", "-o", str(d / "s.so"), str(d / "s.cpp")], check=True)
    return ctypes.CDLL(str(d / "s.so"))


def per_xcd(places, tile, total):
    """each XCD's tiles, in the order its workgroups come"""
    mine = [[tile(p) for p in range(x, places, 8)] for x in range(8)]
    mine = [[t for t in ts if t < total] for ts in mine]
    assert sorted(t for ts in mine for t in ts) == list(range(total))
    return mine


@pytest.mark.parametrize("total", [1, 7, 8, 9, 63, 64, 65, 1000, 1537, 4096])
def test_a_launch_of_one_kind(lib, total):
    for ts in per_xcd(lib.places(total, 0), lambda p: lib.tile(p, total), total):
        assert ts == list(range(ts[0], ts[0] + len(ts))) if ts else total < 8
        assert len(ts) <= -(-total // 8)
    assert [lib.tile_of_two(p, total, 0) for p in range(lib.places(total, 0))] == [lib.tile(p, total) for p in range(lib.places(total, 0))]


# thirty tensors of 2^17 beside thirty-two of 2^21 first, the set that had all of the former on one XCD
@pytest.mark.parametrize("few, others", [(120, 2048), (2, 1536), (1, 64), (7, 64), (8, 64), (9, 128), (383, 1024), (1000, 64)])
def test_a_launch_of_two_kinds(lib, few, others):
    total = few + others
    for ts in per_xcd(lib.places(total, few), lambda p: lib.tile_of_two(p, total, few), total):
        first, then = [t for t in ts if t < few], [t for t in ts if t >= few]
        assert ts == first + then and len(first) <= -(-few // 8) and len(then) <= -(-others // 8)
        assert all(b == a + 1 for part in (first, then) for a, b in zip(part, part[1:]))


@pytest.mark.parametrize("total", [1, 7, 8, 9, 64, 65, 1000, 1024, 1537, 2048, 4096])
def test_stretches_that_begin_at_different_columns(lib, total):
    """The same stretches, each gone round once from another place on: the XCDs begin in different eighths of a tensor of 128 tiles."""
    straight = per_xcd(lib.places(total, 0), lambda p: lib.tile(p, total), total)
    turned = per_xcd(lib.places(total, 0), lambda p: lib.turned(p, total, 16), total)
    assert per_xcd(lib.places(total, 0), lambda p: lib.turned(p, total, 0), total) == straight
    for a, b in zip(straight, turned):
        assert sorted(b) == a and (not b or b == a[a.index(b[0]):] + a[:a.index(b[0])])
    if total >= 1024:
        assert len({ts[0] % 128 // 16 for ts in turned}) == 8


@pytest.mark.parametrize("total, few, apart", [(2168, 120, 120), (1656, 120, 120), (1288, 584, 0), (1304, 472, 0), (1000, 299, 299), (1000, 300, 0), (64, 0, 0)])
def test_stretches_of_their_own_are_for_few_tiles(lib, total, few, apart):
    assert lib.apart(total, few) == apart
