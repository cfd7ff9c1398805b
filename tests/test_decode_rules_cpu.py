"""Which form a decode launch takes, and how the forms of long walks divide their ranges (csrc/decode_rules.h, compiled here for the host)."""
import ctypes
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """
#include "decode_rules.h"
using namespace lamps;
static rules::DecodeLaunch launch(int kv_heads, int group, int bf16, int dim, int batch, long long row, int bounded, long long capacity)
{
    const bool matrix = bf16 && group > 1;
    int gh = matrix ? 16 : 4;
    while (group % gh || (!matrix && gh == 3)) --gh;
    if (bf16 && !matrix) gh = 1;
    const int lpt = dim * (bf16 ? 2 : 4) / 16, chunk = matrix ? 16 : 64 / lpt * (lpt == 8 ? 2 : 4) * (gh == 4 ? 1 : 2);
    return {(long long)batch * kv_heads * (group / gh), batch, dim, row, 4 * chunk, matrix, bounded != 0, (size_t)gh * (dim + 2) * 4,
            (size_t)capacity};
}
extern "C" {
int c_form(int kv_heads, int group, int bf16, int dim, int batch, long long row, int bounded, long long capacity)
{
    return rules::decode_form(launch(kv_heads, group, bf16, dim, batch, row, bounded, capacity));
}
int c_cuts(int kv_heads, int group, int bf16, int dim, int batch, long long row, long long capacity, int *most)
{
    const rules::DecodeLaunch l = launch(kv_heads, group, bf16, dim, batch, row, 1, capacity);
    const int n = rules::decode_cuts(l);
    *most = n ? rules::decode_most_cuts(l) : 0;
    return n;
}
int c_spare(int matrix) { return rules::cut_spare(matrix); }
void c_cut(unsigned all, int spare, int round, int n, int chunk, int *out)
{
    const rules::CutSize c = rules::cut_size(all, spare, round);
    out[0] = c.size; out[1] = c.worth; out[2] = rules::cut_parts(n, c);
    out[3] = out[2] ? rules::cut_each(n, out[2], chunk) : 0;
}
int c_part(int sum, int longest, int batch, int even, int most, int chunk) { return rules::part_size(sum, longest, batch, even, most, 4, chunk); }
}
"""
PLAN, TWO, FOUR, EIGHT, CUT, PARTS = range(6)
ROOM = 64 << 20


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(SOURCE)
    so = str(d / "rules.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2410_18248_amd", "csrc"),
                           str(d / "rules.cpp"), "-o", so])
    lib = ctypes.CDLL(so)
    lib.c_form.argtypes = [ctypes.c_int] * 5 + [ctypes.c_longlong, ctypes.c_int, ctypes.c_longlong]
    lib.c_cuts.argtypes = [ctypes.c_int] * 5 + [ctypes.c_longlong, ctypes.c_longlong, ctypes.POINTER(ctypes.c_int)]
    lib.c_cut.argtypes = [ctypes.c_uint] + [ctypes.c_int] * 4 + [ctypes.POINTER(ctypes.c_int)]
    return lib


def form(lib, H, Hkv, dtype, D, batch, row, bounded=1, room=ROOM):
    return lib.c_form(Hkv, H // Hkv, dtype == "bf16", D, batch, row, bounded, room)


@pytest.mark.parametrize("H,Hkv,D,dtype,batch,row,want", [
    (32, 8, 128, "bf16", 1, 2000, PARTS), (32, 8, 128, "bf16", 1, 200, FOUR), (8, 8, 64, "bf16", 1, 4000, PARTS), (32, 8, 128, "bf16", 1, 32768, PARTS), (32, 8, 128, "bf16", 1, 65536, PARTS), (32, 8, 128, "bf16", 1, 65552, PLAN),
    # few ranges: parts on both sides of the lines
    (32, 8, 128, "bf16", 3, 8192, PARTS), (32, 8, 128, "bf16", 4, 8192, PARTS), (32, 8, 128, "bf16", 4, 8208, PARTS), (8, 1, 128, "bf16", 60, 65536, PARTS), (1, 1, 128, "bf16", 64, 131072, PLAN), (1, 1, 128, "bf16", 63, 131072, PARTS), (3, 3, 128, "bf16", 1, 51200, PARTS), (3, 3, 128, "bf16", 1, 51216, PLAN), (32, 8, 128, "bf16", 11, 2048, PARTS), (32, 8, 128, "bf16", 11, 2064, PLAN), (32, 8, 128, "bf16", 8, 2048, PARTS),
    (32, 8, 128, "bf16", 12, 2048, PLAN), (40, 40, 128, "bf16", 3, 2048, PARTS), (40, 40, 128, "bf16", 3, 2064, PARTS), (40, 40, 128, "bf16", 4, 2064, PLAN), (8, 1, 64, "bf16", 65, 1600, PLAN),
    # whole ranges
    (32, 8, 128, "bf16", 64, 304, FOUR), (40, 40, 128, "bf16", 40, 128, TWO), (40, 40, 128, "bf16", 40, 144, FOUR), (40, 40, 128, "bf16", 102, 256, FOUR), (40, 40, 128, "bf16", 103, 256, TWO), (40, 40, 128, "bf16", 103, 384, TWO),
    (32, 8, 128, "bf16", 200, 64, TWO), (32, 8, 128, "bf16", 200, 256, FOUR), (32, 8, 128, "bf16", 256, 512, FOUR), (32, 8, 128, "bf16", 257, 512, FOUR),
    (32, 8, 128, "bf16", 257, 784, PLAN), (32, 32, 128, "bf16", 6, 512, EIGHT), (32, 8, 128, "bf16", 10, 1024, EIGHT),
    # heads of 256: parts sooner, eight waves sooner, the plan and cuts in place of long walks by one workgroup
    (16, 8, 256, "bf16", 4, 256, FOUR), (16, 8, 256, "bf16", 4, 272, EIGHT), (16, 8, 256, "bf16", 4, 320, EIGHT), (16, 8, 256, "bf16", 4, 336, PARTS),
    (16, 8, 256, "bf16", 8, 576, EIGHT), (16, 8, 256, "bf16", 8, 592, PLAN), (16, 8, 256, "bf16", 16, 640, EIGHT), (16, 8, 256, "bf16", 16, 656, CUT),
    (16, 8, 256, "bf16", 127, 768, CUT), (16, 8, 256, "bf16", 128, 768, FOUR), (128, 8, 256, "bf16", 8, 576, FOUR), (10, 2, 256, "bf16", 257, 768, FOUR),
    # thousands of ranges by two waves
    (32, 8, 128, "bf16", 511, 256, FOUR), (32, 8, 128, "bf16", 512, 256, TWO), (32, 8, 128, "bf16", 512, 768, TWO), (32, 32, 128, "bf16", 300, 640, TWO),
    # looked at on the device
    (40, 40, 128, "bf16", 16, 1504, CUT), (40, 40, 128, "bf16", 16, 16384, CUT), (40, 40, 128, "bf16", 16, 16400, PLAN), (32, 32, 128, "bf16", 64, 4112, PLAN), (40, 40, 128, "bf16", 12, 4096, CUT), (40, 40, 128, "bf16", 12, 4112, PLAN), (32, 32, 128, "bf16", 64, 2048, CUT),
    (32, 8, 128, "bf16", 64, 1504, CUT), (32, 8, 128, "bf16", 256, 8192, CUT), (32, 8, 128, "bf16", 256, 16400, PLAN), (32, 8, 128, "bf16", 64, 16384, CUT), (32, 8, 128, "bf16", 32, 2048, CUT), (32, 8, 128, "bf16", 32, 2064, PLAN), (64, 32, 64, "bf16", 128, 4112, PLAN), (40, 40, 128, "bf16", 180, 1232, PLAN), (32, 32, 128, "bf16", 256, 512, PLAN),
    (32, 32, 128, "bf16", 257, 768, TWO), (31, 31, 128, "bf16", 257, 768, FOUR), (32, 32, 128, "bf16", 257, 784, PLAN), (32, 8, 128, "f32", 24, 2512, PLAN), (32, 8, 128, "f32", 40, 512, CUT),
    (10, 2, 256, "bf16", 129, 800, CUT),
    # what the GPU tests of skewed batches count on
    (32, 32, 64, "bf16", 17, 640, CUT), (8, 8, 64, "bf16", 70, 1504, CUT), (16, 16, 256, "bf16", 20, 912, CUT), (16, 8, 128, "bf16", 40, 2000, CUT),
    (16, 8, 64, "bf16", 66, 2048, CUT), (128, 4, 64, "bf16", 40, 1008, CUT), (8, 8, 32, "f32", 40, 912, CUT), (16, 2, 128, "f32", 130, 416, CUT),
    (6, 3, 64, "f32", 100, 704, CUT), (4, 4, 128, "bf16", 256, 512, CUT), (32, 32, 128, "bf16", 34, 800, CUT), (16, 8, 64, "bf16", 70, 1600, CUT),
    (8, 8, 64, "f32", 65, 1008, CUT),
    (3, 3, 64, "bf16", 343, 112, TWO), (16, 16, 64, "bf16", 260, 256, TWO), (8, 8, 128, "bf16", 513, 384, TWO), (8, 8, 64, "f32", 515, 144, TWO), (16, 8, 64, "bf16", 131, 64, TWO),
    (64, 32, 64, "bf16", 129, 512, TWO), (16, 8, 256, "bf16", 3, 400, PARTS), (16, 8, 256, "bf16", 9, 512, EIGHT), (16, 8, 256, "bf16", 20, 704, CUT),
    (128, 8, 256, "bf16", 9, 512, FOUR), (10, 2, 256, "bf16", 70, 304, EIGHT),
    (8, 2, 128, "bf16", 10, 2512, PARTS), (32, 1, 128, "bf16", 20, 1504, PARTS), (16, 4, 64, "bf16", 16, 1600, PARTS), (2, 1, 128, "bf16", 64, 1600, PARTS),
    (8, 8, 64, "bf16", 11, 1312, PARTS), (2, 2, 256, "bf16", 7, 2000, PARTS), (8, 2, 128, "f32", 30, 912, PARTS), (4, 4, 32, "f32", 16, 1120, PARTS),
    (10, 2, 256, "bf16", 3, 5008, PARTS), (8, 2, 128, "bf16", 4, 2000, PARTS),
])
def test_forms(lib, H, Hkv, D, dtype, batch, row, want):
    assert form(lib, H, Hkv, dtype, D, batch, row) == want
    assert form(lib, H, Hkv, dtype, D, batch, row, bounded=0) == PLAN


@pytest.mark.parametrize("H,Hkv,D,dtype", [(32, 32, 128, "bf16"), (32, 8, 128, "bf16"), (8, 8, 64, "f32")])
def test_no_more_is_refused_as_ranges_get_more(lib, H, Hkv, D, dtype):
    """Batches that a wave cannot sort go whole wherever that is the better form; nothing goes whole that fewer requests beside it would keep from it."""
    for row in (128, 256, 384, 496, 512, 640, 768):
        whole = [form(lib, H, Hkv, dtype, D, b, row) in (TWO, FOUR, EIGHT) for b in range(257, 700)]
        assert all(whole) or not any(whole), row


def test_room(lib):
    """What has no room for its partial states goes by the plan, which makes do with fewer shares."""
    assert form(lib, 40, 40, "bf16", 128, 16, 1504, room=(640 + 1024) * (130 * 4 + 8)) == CUT
    assert form(lib, 40, 40, "bf16", 128, 16, 1504, room=(640 + 1024) * (130 * 4 + 8) - 1) == PLAN
    assert form(lib, 32, 8, "bf16", 128, 1, 2000, room=8 * 32 * 4 * 130 * 4) == PARTS
    assert form(lib, 32, 8, "bf16", 128, 1, 2000, room=8 * 32 * 4 * 130 * 4 - 1) == PLAN


def _contexts(rng, batch, row):
    kind = rng.randrange(5)
    if kind == 0:
        n = [row] * batch
    elif kind == 1:
        n = [rng.randint(1, max(1, row // 20)) for _ in range(batch)]
        n[rng.randrange(batch)] = row
    elif kind == 2:
        n = [rng.randint(1, row) if rng.random() < 0.1 else 0 for _ in range(batch)]   # most wait
    elif kind == 3:
        n = [max(1, int(row ** rng.random())) for _ in range(batch)]
    else:
        n = [0] * batch
        n[rng.randrange(batch)] = row
    return n


def test_cut_launches(lib):
    """However long the contexts are against each other: the grid has a workgroup for every part, the parts are the range, and none is longer than one and a half
    even shares or three rounds."""
    rng, out = random.Random(7), (ctypes.c_int * 4)()
    for _ in range(4000):
        chunk = rng.choice([1, 2])
        round_, spare, batch, heads = 4 * chunk, rng.choice([512, 1024]), rng.randint(1, 256), rng.choice([1, 2, 8, 32, 40])
        n = _contexts(rng, batch, rng.randint(1, rng.choice([512, 2048])))
        all_ = sum(n) * heads
        items = 0
        for c in n:
            lib.c_cut(all_, spare, round_, c, chunk, out)
            size, worth, parts, each = out
            assert worth <= max(1.5 * (all_ / spare + round_ + 1), 3 * round_)
            if not parts:
                items += heads * (c > 0)
                assert c <= worth
                continue
            assert each <= worth and each % chunk == 0 and (parts - 1) * each < c + parts * chunk
            assert parts * each >= c
            items += parts * heads
        assert items <= batch * heads + spare


def test_parts(lib):
    """The same of launches of few ranges: `even` workgroups for each range there can be and one for each that runs, `most` parts of a range."""
    rng, most = random.Random(8), ctypes.c_int()
    done = 0
    while done < 4000:
        H, Hkv, D, dtype = rng.choice([(32, 8, 128, "bf16"), (40, 40, 128, "bf16"), (8, 2, 64, "bf16"), (8, 8, 64, "f32"), (8, 1, 128, "bf16"), (10, 2, 256, "bf16")])
        batch, row, room = rng.randint(1, 64), int(2 ** rng.uniform(6, 17.5)), rng.choice([ROOM, 31 << 20, 2 << 20])
        even = lib.c_cuts(Hkv, H // Hkv, dtype == "bf16", D, batch, row, room, ctypes.byref(most))
        if not even:
            continue
        done += 1
        gt, chunk = 16, 1 if H > Hkv else 2
        n = [(c + gt - 1) // gt for c in _contexts(rng, batch, row)]
        assert sum(n) + even * batch < 1 << 19             # what is divided
        size = lib.c_part(sum(n), max(n), batch, even, most.value, chunk)
        assert size % chunk == 0 and size < max(4 * chunk, sum(n) / (batch * even) + 1, max(n) / most.value + 1) + chunk
        for tries in range(9):
            own = [-(-c // size) for c in n]
            assert even <= most.value <= 64 and max(own) <= most.value
            assert sum(own) <= batch * even + sum(c > 0 for c in n)
            if sum(own) <= batch * even:
                break
            size += chunk
        if max(n) <= 1.02 * min(n):
            assert sum(own) <= batch * even
