"""How a split prefill launch divides its work (csrc/prefill_split.h, compiled here for the host): over random
batches, every (request, kv head, tile, run) has one workgroup, items stay within the partial slots, runs
cover the contexts, and the work is spread over all eight XCDs however little there is."""
import ctypes
import os
import random
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """
#include "prefill_split.h"
using namespace lamps::split;
extern "C" {
int c_tiles(int n, int wt, int tiles) { return tiles_of(n, wt, tiles); }
void c_cut(int stages, int tiles, int most, int head_slots, int heads, int group, int dim, int wide, int *out)
{
    const Cut c = cut_of({stages, tiles, most}, head_slots, heads, group, dim, wide);
    out[0] = c.per; out[1] = c.worth;
}
int c_runs(int stages, int per, int worth, int slots) { return runs_of(stages, {per, worth}, slots); }
int c_item(int block, int items, int slots) { return item_of(block, items, slots); }
void c_piece(int x, int tiles, int runs, int *out)
{
    const Piece p = piece_of(x, tiles, runs);
    out[0] = p.head; out[1] = p.run; out[2] = p.tile;
}
int c_div(int a, int b) { return small_div(a, b); }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("split")
    (d / "split.cpp").write_text(SOURCE)
    so = str(d / "split.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2410_18248_amd", "csrc"),
                           str(d / "split.cpp"), "-o", so])
    return ctypes.CDLL(so)


def _plan(lib, heads, new, ctx, wt, slots, group, wide, dim=128):
    """What the workgroups do: a list of (block, item, request, head, tile, run), per, and the requests' runs."""
    tiles = -(-max(new) // wt)
    nt = [lib.c_tiles(n, wt, tiles) if n else 0 for n in new]
    assert nt == [-(-n // wt) for n in new]
    stages = [(c - 1) // 32 + 1 if n else 0 for n, c in zip(new, ctx)]
    out = (ctypes.c_int * 3)()
    lib.c_cut(sum(a * b for a, b in zip(stages, nt)), sum(nt), max(stages), slots // heads, heads, group, dim, wide, out)
    per, worth = out[0], out[1]
    runs = [lib.c_runs(s, per, worth, slots) for s in stages]
    items = [a * b * heads for a, b in zip(nt, runs)]
    upto = np.cumsum(items)
    work = []
    for block in range(slots):
        item = lib.c_item(block, int(upto[-1]), slots)
        if item < 0 or item >= upto[-1]:
            continue
        r = int(np.searchsorted(upto, item, side="right"))
        lib.c_piece(int(item - (upto[r] - items[r])), nt[r], runs[r], out)
        work.append((block, item, r, out[0], out[2], out[1]))
    return work, per, runs, nt, stages


@pytest.mark.parametrize("wide,group,dim", [(False, 1, 128), (True, 1, 256), (True, 2, 128)])
def test_every_piece_has_one_workgroup(lib, wide, group, dim):
    rng = random.Random(3 + group)
    done = 0
    while done < 300:
        heads = rng.choice([1, 2, 3, 4, 5, 8, 16, 32, 40])
        wt = rng.choice([1, 2, 3, 4, 7, 8, 16, 32, 64])
        slots = rng.choice([512, 512, 504, 256, 64])
        n_req = rng.choice([1, 1, 2, 3, 7, 20, 64])
        new = [rng.choice([0, 1, 2, rng.randint(1, 64), int(2 ** rng.uniform(0, 10))]) for _ in range(n_req)]
        if not any(new):
            continue
        ctx = [max(n + rng.choice([0, 0, int(2 ** rng.uniform(0, 13)), rng.randint(0, 700)]), 1) for n in new]
        if sum(-(-n // wt) for n in new) * heads > slots // 2:      # the launcher does not split such a call
            continue
        done += 1
        work, per, runs, nt, stages = _plan(lib, heads, new, ctx, wt, slots, group, wide, dim)
        assert per % group == 0 and per >= 12
        total = sum(t * k * heads for t, k in zip(nt, runs))
        assert total <= slots                                        # a partial slot for each
        assert [w[1] for w in sorted(work, key=lambda w: w[1])] == list(range(total))
        want = {(r, g, t, k) for r in range(n_req) for g in range(heads) for t in range(nt[r]) for k in range(runs[r])}
        assert {w[2:] for w in work} == want and len(work) == len(want)
        for r, k in enumerate(runs):
            assert k == 1 or (k - 1) * per < stages[r] <= k * per    # the runs of the last tile cover it
        share = np.bincount([w[0] % 8 for w in work], minlength=8)   # workgroup b runs on XCD b mod 8
        assert share.max() <= -(-total // 8)
        if total >= 64:
            assert share.min() >= total // 8 - 7
        for r, g, t in {w[2:5] for w in work}:                       # a tile's items lie `tiles` apart, in run order
            at = sorted(w[1] for w in work if w[2:5] == (r, g, t))
            assert all(b - a == nt[r] for a, b in zip(at, at[1:]))


def test_empty_runs_do_not_gather_on_one_xcd(lib):
    """Tiles of a prompt that see half the context have half the runs: what is left to do is even over the XCDs."""
    work, per, runs, nt, stages = _plan(lib, 8, [200], [1300], 16, 512, 1, False)
    assert runs[0] > 2
    live = [w for w in work if w[5] * per < (1100 + min(200, 16 * (w[4] + 1)) - 1) // 32 + 1]
    share = np.bincount([w[0] % 8 for w in live], minlength=8)
    assert share.max() - share.min() <= 2, share


def test_requests_that_gain_nothing_are_not_cut(lib):
    for n, c, cut in [(400, 400, False), (16, 384, False), (16, 640, True), (16, 3000, True)]:
        assert (_plan(lib, 8, [n], [c], 16, 512, 1, False)[2][0] > 1) == cut, (n, c)
    for n, c, cut in [(400, 1000, False), (500, 500, False), (130, 3130, True), (400, 3400, True)]:
        assert (_plan(lib, 8, [n], [c], 32, 512, 2, True)[2][0] > 1) == cut, (n, c)
    for n, c, cut in [(500, 500, False), (900, 1600, False), (400, 1100, True), (700, 3700, True)]:
        assert (_plan(lib, 16, [n], [c], 64, 512, 1, True, 256)[2][0] > 1) == cut, (n, c)


def test_lying_arguments_stay_in_the_slots(lib):
    """More items than slots (device arguments that contradict the host's): no workgroup takes one past them."""
    for items in [513, 600, 4096, 1 << 24]:
        got = [lib.c_item(b, items, 512) for b in range(512)]
        assert min(got) >= 0 and max(got) < 512 and len(set(got)) == 512
    assert lib.c_runs(1 << 25, 12, 18, 512) == 512


def test_small_division(lib):
    rng = random.Random(1)
    for b in list(range(1, 300)) + [511, 512, 513, 4095, 32767, 1 << 18]:
        for a in {0, 1, b - 1, b, b + 1, 2 * b - 1, 2 * b, (1 << 19) - 1, (1 << 19) // b * b - 1} | {rng.randrange(1 << 19) for _ in range(50)}:
            if 0 <= a < 1 << 19:
                assert lib.c_div(a, b) == a // b, (a, b)
