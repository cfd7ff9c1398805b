"""How wide the tiles of a prefill launch are and in which order they start (csrc/prefill_rules.h, compiled here for the host)."""
import ctypes
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """
#include "prefill_rules.h"
using namespace lamps;
extern "C" {
void c_turn(int slot, int tiles, int pairs, int abreast, int *out)
{
    const rules::Turn at = rules::abreast_at(slot, tiles, pairs, abreast);
    out[0] = at.pair; out[1] = at.t;
}
void c_deal(int block, int pairs, int tiles, int abreast, int *out)
{
    const rules::Turn at = rules::deal(block, pairs, pairs / 8, tiles, abreast);
    out[0] = at.pair; out[1] = at.t;
}
int c_abreast(int heads, int dim, int batch, int total, int most, long long row, int bytes, int wt)
{
    const long long pairs = (long long)heads * batch, tiles = (most + wt - 1) / wt;
    const rules::Together w = rules::together({heads, 1, dim, batch, total, most, 0}, bytes, tiles,
                                              pairs / 8 * 8 * tiles + (pairs % 8 * tiles + 7) / 8 * 8, heads * ((long long)total / wt + batch), (int)(pairs / 8), 512);
    return rules::pairs_abreast(w, (int)row, (int)(pairs / 8));
}
int c_teams(int kv_heads, int group, int dim, int batch, int total, int most, long long row)
{
    return rules::teams({kv_heads, group, dim, batch, total, most, row});
}
int c_narrow(int kv_heads, int group, int dim, int batch, int total, int most, long long row, int tiled)
{
    return rules::narrow_tiles({kv_heads, group, dim, batch, total, most, row}, tiled);
}
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(SOURCE)
    so = str(d / "rules.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2410_18248_amd", "csrc"),
                           str(d / "rules.cpp"), "-o", so])
    return ctypes.CDLL(so)


def _turns(lib, tiles, pairs, abreast):
    out = (ctypes.c_int * 2)()
    for slot in range(tiles * pairs):
        lib.c_turn(slot, tiles, pairs, abreast, out)
        yield slot, out[0], out[1]


def test_every_tile_has_one_workgroup(lib):
    rng = random.Random(5)
    for _ in range(200):
        tiles, pairs = rng.choice([1, 2, 3, 5, 17, 130]), rng.choice([2, 3, 4, 5, 7, 8, 16, 23, 115])
        abreast = rng.randint(2, pairs)
        turns = [(p, t) for _, p, t in _turns(lib, tiles, pairs, abreast)]
        assert sorted(turns) == [(p, t) for p in range(pairs) for t in range(tiles)]
        for first in range(0, pairs, abreast):           # part by part, the longest tiles first
            part = [t for p, t in turns[first * tiles:(first + abreast) * tiles]]
            assert part == sorted(part)


@pytest.mark.parametrize("lengths", [[125, 118, 104, 94], [63, 47], [62, 60, 57, 55, 54, 52, 50, 47], [31, 16] * 4,
                                     [20, 18, 15, 12, 10, 9] * 2, [100, 20, 20, 20], [50, 41, 33, 30, 28, 27, 90]])
def test_work_is_even_over_shader_engines(lib, lengths):
    """An XCD's workgroups go to its four shader engines in turn.  Pairs of different lengths (in tiles, whose work
    grows with their place), all abreast: each engine's share of it."""
    tiles = max(lengths)
    work = [0, 0, 0, 0]
    for slot, pair, t in _turns(lib, tiles, len(lengths), len(lengths)):
        place = tiles - 1 - t
        if place < lengths[pair]:
            work[slot % 4] += place + 1
    assert max(work) <= 1.06 * sum(work) / 4, work


def test_the_largest_launches(lib):
    """Places of the last slots there may be, which a reciprocal has to find exactly."""
    rng = random.Random(6)
    out = (ctypes.c_int * 2)()
    for _ in range(3000):
        slots = rng.randint(1 << 18, (1 << 19) - 1)
        pairs = rng.choice([2, 3, 7, 64, 115, 600])
        tiles = slots // pairs
        abreast = rng.randint(2, pairs)
        slot = rng.randint(0, tiles * pairs - 1)
        if rng.random() < 0.5:
            slot = min(tiles * pairs - 1, slot // abreast * abreast + rng.choice([-1, 0]) % abreast)
        lib.c_turn(slot, tiles, pairs, abreast, out)
        first = slot // (abreast * tiles) * abreast
        n = min(abreast, pairs - first)
        assert out[1] == (slot - first * tiles) // n and first <= out[0] < first + n


@pytest.mark.parametrize("H,Hkv,D,batch,total,most,row,narrow", [
    # prompts, by their length on average
    (40, 40, 128, 24, 2950, 683, 688, True),             # an iteration's
    (32, 32, 128, 50, 2690, 128, 128, True),
    (32, 32, 128, 90, 11520, 250, 256, True),
    (32, 32, 128, 100, 13000, 250, 256, False),
    (8, 8, 64, 32, 11200, 500, 512, True),
    (32, 32, 64, 70, 9000, 250, 256, True),
    (32, 32, 64, 80, 10000, 250, 256, False),
    (32, 32, 128, 10, 4984, 600, 608, True),
    (32, 32, 128, 12, 6144, 512, 512, False),
    (40, 40, 128, 14, 4578, 362, 368, False),
    (32, 32, 128, 1, 1000, 1000, 1008, True),
    (32, 32, 128, 4, 16000, 4000, 4000, False),
    (32, 8, 128, 1, 1000, 1000, 1008, True),
    (32, 8, 128, 4, 16384, 4096, 4096, False),
    (8, 2, 64, 60, 8736, 250, 256, True),
    (8, 2, 64, 32, 11232, 500, 512, True),
    (16, 8, 64, 6, 6000, 1000, 1008, False),
    (16, 8, 64, 24, 4290, 683, 688, True),
    (32, 8, 64, 16, 3376, 272, 272, True),
    # half the tokens in half the columns: groups of 3, 5, 7; fewer: of 6, 9 and 10
    (12, 4, 128, 6, 1200, 300, 1300, True),
    (20, 4, 128, 6, 1200, 300, 1300, True),
    (28, 4, 128, 1, 1000, 1000, 1008, True),
    (24, 4, 128, 3, 1350, 600, 608, True),
    (48, 8, 128, 6, 1200, 300, 1300, False),
    (24, 4, 128, 20, 4000, 300, 304, True),
    (24, 4, 128, 6, 3600, 700, 704, False),
    (36, 4, 128, 3, 1350, 600, 608, False),
    (40, 4, 128, 4, 800, 300, 1300, False),
    (40, 4, 128, 1, 1000, 1000, 1008, True),
    (36, 4, 64, 30, 1700, 120, 128, False),
    (36, 4, 64, 1, 300, 300, 304, True),
    # cached positions: short rows, few new tokens to a tile of 128, more
    (32, 8, 128, 60, 1100, 64, 1040, True),
    (32, 8, 128, 10, 1750, 250, 1250, True),
    (32, 8, 128, 4, 800, 300, 2300, True),
    (32, 8, 128, 10, 1750, 250, 2250, False),
    (32, 8, 128, 40, 1360, 64, 2064, True),
    (32, 32, 128, 20, 340, 64, 2064, True),
    (32, 32, 128, 10, 1750, 250, 2250, True),
    (32, 32, 128, 17, 1260, 124, 2363, False),
    (32, 32, 128, 10, 1750, 250, 1250, True),
    (40, 40, 128, 20, 55, 5, 1568, False),               # a few tokens each
    (32, 32, 128, 30, 150, 8, 1008, False),
    (32, 8, 64, 20, 680, 64, 2064, True),
    (32, 8, 64, 50, 1400, 64, 2064, True),
    (32, 8, 64, 80, 2700, 64, 2064, False),
    (32, 32, 64, 24, 120, 8, 2008, True),
    (32, 32, 64, 30, 150, 8, 2008, False),
    # a row as long as the longest possible request
    (40, 40, 128, 24, 2950, 683, 32768, False),
    (32, 8, 128, 1, 1000, 1000, 32768, True),
    (64, 2, 128, 4, 400, 100, 112, False),               # groups above 16: no tiles of 64 columns
])
def test_width_of_tiles(lib, H, Hkv, D, batch, total, most, row, narrow):
    """On both sides of the lines."""
    row = ctypes.c_longlong(row)
    assert lib.c_narrow(Hkv, H // Hkv, D, batch, total, most, row, H > Hkv) == narrow


@pytest.mark.parametrize("heads,D,batch,total,most,row,bytes,wt,abreast", [
    # the launches whose rows are compared on the GPU, over their contexts and (test_contexts_decide) over long ones
    (40, 64, 5, 1518, 310, 640, 4, 128, 1),
    (40, 64, 5, 1518, 310, 608, 4, 128, 1),
    (40, 64, 5, 2148, 501, 608, 4, 128, 25),
    (9, 64, 3, 1790, 610, 2048, 4, 32, 1),
    (8, 256, 3, 2083, 700, 4096, 4, 16, 1),
    (16, 256, 2, 2054, 1030, 6144, 4, 64, 1),
    (9, 64, 3, 1190, 401, 512, 8, 16, 3),
    (9, 64, 3, 1790, 610, 1200, 4, 32, 3),
    (8, 256, 3, 4875, 1800, 3584, 4, 64, 2),
    (32, 128, 10, 1478, 250, 1100, 4, 128, 20),
    (9, 64, 3, 1790, 610, 610, 4, 32, 3),
    (9, 64, 3, 1790, 610, 1830, 4, 32, 1),
    (8, 256, 3, 2083, 700, 700, 4, 16, 3),
    (16, 256, 2, 2054, 1030, 1030, 4, 64, 4),
    (8, 256, 3, 4875, 1800, 3500, 4, 64, 2),
    (9, 64, 3, 1191, 401, 410, 8, 16, 3),
    (8, 64, 64, 7328, 130, 319, 8, 16, 64),
    # heads of 128, 128 columns: all of the groups of an XCD, parts of 20 MB, one by one where a pair has as much
    (32, 128, 4, 4000, 1000, 1008, 4, 128, 16),
    (40, 128, 4, 8192, 2048, 2048, 4, 128, 20),
    (32, 128, 4, 16384, 4096, 4096, 4, 128, 8),
    (16, 128, 1, 40000, 40000, 40000, 4, 128, 1),
    (8, 256, 3, 2100, 700, 4096, 4, 16, 1),              # a row of 4 096: mostly cached
    (8, 256, 3, 2100, 700, 1400, 4, 16, 3),
    (16, 256, 2, 4100, 2050, 4096, 4, 64, 2),            # parts of 10 MB: two, of the four groups
    (16, 256, 2, 12000, 6000, 6016, 4, 64, 2),           # three
    (16, 256, 2, 24000, 12000, 12000, 4, 64, 1),         # more than four, so four of one each
    # where the chip holds the launch at once, or many workgroups have no tile
    (32, 128, 2, 1000, 500, 512, 4, 128, 1),
    (32, 128, 24, 4200, 4000, 4000, 4, 128, 1),
    # few tiles, as many for every request
    (32, 128, 27, 8937, 362, 368, 4, 128, 1),
    (32, 128, 16, 8000, 500, 512, 4, 128, 64),
    (32, 128, 60, 10500, 250, 256, 4, 128, 120),
    # cached positions: twice the new ones and more, as many on heads that share an XCD, and few tiles of which many requests have fewer
    (32, 128, 10, 2000, 200, 1100, 4, 128, 1),
    (32, 128, 10, 1750, 250, 1375, 4, 128, 20),
    (32, 128, 10, 1750, 250, 1520, 4, 128, 1),
    (8, 64, 16, 8000, 500, 2750, 8, 16, 1),
    (8, 128, 10, 5000, 500, 1250, 4, 32, 10),
    (4, 128, 10, 5000, 500, 1250, 4, 16, 1),
    (4, 128, 10, 5000, 500, 900, 4, 16, 5),
    (8, 64, 16, 8000, 500, 750, 8, 16, 16),
])
def test_pairs_abreast(lib, heads, D, batch, total, most, row, bytes, wt, abreast):
    """row: the longest context, or its bound."""
    row = ctypes.c_longlong(row)
    assert lib.c_abreast(heads, D, batch, total, most, row, bytes, wt) == abreast


def test_pairs_left_over(lib):
    """Whole grids: every tile has one workgroup, eight pairs to a group, and the pairs that fill no group come in front of those
    that go abreast and behind those that do not."""
    out = (ctypes.c_int * 2)()
    for pairs, tiles in ((18, 27), (36, 42), (28, 8), (17, 5), (9, 3), (15, 130), (16, 7), (23, 1)):
        groups, rest = pairs // 8, pairs % 8
        spare = (rest * tiles + 7) // 8
        for abreast in sorted({1, 2, groups}):
            if abreast > groups:
                continue
            seen = {}
            for block in range(8 * (groups * tiles + spare)):
                lib.c_deal(block, pairs, tiles, abreast, out)
                if out[1] < tiles:
                    assert (out[0], out[1]) not in seen
                    seen[out[0], out[1]] = block
                    if out[0] < 8 * groups:
                        assert out[0] % 8 == block % 8
                else:
                    assert out[0] >= 8 * groups
            assert len(seen) == pairs * tiles
            left = [b for (p, _), b in seen.items() if p >= 8 * groups]
            others = [b for (p, _), b in seen.items() if p < 8 * groups]
            if rest:
                assert max(left) < min(others) if abreast > 1 else min(left) > max(others)


@pytest.mark.parametrize("H,Hkv,D,batch,total,most,row,two_teams", [
    (32, 8, 128, 4, 16384, 4096, 4096, True),
    (32, 8, 128, 4, 4000, 1000, 1008, True),
    (32, 8, 128, 1, 1000, 1000, 1008, False),
    (32, 4, 128, 41, 5371, 131, 144, False),              # short walks
    (28, 4, 128, 20, 1750, 103, 592, False),
    (32, 32, 128, 4, 16000, 4000, 4000, True),
    (32, 32, 128, 4, 4000, 1000, 1008, False),
    (40, 40, 128, 24, 2950, 683, 688, False),
    (32, 32, 128, 16, 4000, 250, 2256, True),             # full tiles
    (16, 16, 128, 25, 7150, 336, 1008, False),            # half-empty ones
    (32, 32, 128, 13, 2928, 321, 2480, False),            # some with a second one
    (32, 32, 128, 13, 2928, 256, 2480, True),
    (16, 16, 256, 37, 4148, 134, 1040, False),
    (16, 16, 256, 37, 4148, 128, 1040, True),
    (32, 8, 128, 4, 2048, 512, 2560, True),
    (16, 16, 256, 4, 2048, 512, 2560, True),
    (16, 16, 256, 1, 700, 700, 704, False),
    (16, 4, 256, 2, 40, 30, 48, True),                    # grouped heads of 256
    (32, 1, 256, 4, 4096, 1024, 1024, False),             # more heads than a wave has columns
    (64, 2, 128, 4, 4096, 1024, 1024, True),
    # a request among others and alone, as the test of equal bits has them
    (32, 8, 128, 4, 4000, 1002, 1008, True),
    (32, 8, 128, 1, 1002, 1002, 1008, False),
    (32, 32, 128, 4, 4120, 1036, 1040, True),
    (32, 32, 128, 1, 1036, 1036, 1040, False),
    (16, 16, 256, 4, 2048, 513, 928, True),
    (16, 16, 256, 1, 513, 513, 928, False),
])
def test_two_teams(lib, H, Hkv, D, batch, total, most, row, two_teams):
    lib.c_teams.argtypes = [ctypes.c_int] * 6 + [ctypes.c_longlong]
    assert lib.c_teams(Hkv, H // Hkv, D, batch, total, most, row) == two_teams
