"""lamps_decode_attn where workgroups take whole ranges, or ranges in parts, and on the other side of those lines: rows of few and of many rounds of
chunks, few ranges and many, two waves to a range, four, eight, and four with the longest contexts first and cut; contexts around a chunk, a part and at
the end of the row, paused and empty requests, equal lengths, a few long ones among many short ones, few that run, against the fp64 oracle; a call that
is replayed from a HIP graph with other lengths."""
import numpy as np
import pytest
import torch

import lamps_workloads as W
import oracle
from rig import Rig, n2t, to_f64, tol

pytestmark = pytest.mark.gpu

GEOMS = [("bf16", 8, 8, 64, 16), ("bf16", 6, 6, 128, 32), ("bf16", 2, 2, 256, 16), ("bf16", 16, 4, 64, 16), ("bf16", 16, 2, 128, 32),
         ("bf16", 32, 1, 128, 16), ("bf16", 10, 2, 256, 16), ("f32", 4, 4, 32, 16), ("f32", 6, 3, 64, 16), ("f32", 16, 2, 128, 32)]


def _check(dtype, H, Hkv, D, bs, batch, row, seed):
    rng = np.random.RandomState(seed)
    edges = [e for e in (0, 1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 257, row - 17, row - 1, row) if 0 <= e <= row]
    ctx = [int(x) for x in rng.choice(edges, batch)]
    ctx[0] = row
    ctx[batch // 2] = 0 if batch > 2 else ctx[batch // 2]
    running = [0 if batch > 1 and r % 6 == 1 else 1 for r in range(batch)]
    blocks = [(c + bs - 1) // bs for c in ctx]
    geom = W.Geometry(1, H, Hkv, D, bs, sum(blocks) + 4, (row + bs - 1) // bs, dtype)
    rig = Rig(geom, batch)
    table, _ = W.deal_block_table(W.permutation(3, geom.num_blocks), ctx, geom)
    K, V = zip(*[W.logical_kv(70 + 17 * r, geom, c) for r, c in enumerate(ctx)])
    rig.page_requests(0, table, K, V)
    q = W.queries(6, geom, batch)
    rig.workspace.fill_(255)                             # NaN where no part writes
    got = to_f64(rig.decode(0, q, table, ctx, running, sentinel=7.0))
    ref = oracle.decode_attn(q, K, V, ctx, running)
    on = np.asarray(running, dtype=bool)
    assert np.abs(got[on] - ref[on]).max() <= tol(geom), ctx
    assert (got[~on] == 7.0).all()
    assert np.array_equal(got, to_f64(rig.decode(0, q, table, ctx, running, sentinel=7.0)))
    rig.close()


@pytest.mark.parametrize("dtype,H,Hkv,D,bs", GEOMS)
def test_few_ranges(dtype, H, Hkv, D, bs):
    """Rows of one to thirteen rounds."""
    for batch, row in ((1, 16), (1, 100), (3, 130), (7, 260), (9, 400), (12, 520), (4, 800)):
        _check(dtype, H, Hkv, D, bs, batch, row, batch + row)


@pytest.mark.parametrize("dtype,H,Hkv,D,bs", GEOMS)
def test_parts(dtype, H, Hkv, D, bs):
    """Few ranges of longer rows."""
    for batch, row in ((1, 600), (1, 3001), (3, 1040), (4, 2080), (6, 1300)):
        _check(dtype, H, Hkv, D, bs, batch, row, batch + row)


@pytest.mark.parametrize("dtype,H,Hkv,D,bs,batch,row", [
    ("bf16", 8, 8, 64, 16, 130, 200), ("bf16", 8, 8, 64, 16, 300, 60), ("bf16", 32, 32, 128, 16, 33, 256), ("bf16", 32, 32, 128, 16, 33, 257),
    ("bf16", 32, 32, 128, 16, 34, 800), ("bf16", 32, 32, 128, 16, 65, 1600), ("bf16", 16, 8, 128, 16, 129, 190), ("bf16", 16, 8, 128, 16, 128, 400),
    ("bf16", 16, 8, 128, 16, 66, 1500), ("bf16", 16, 8, 64, 32, 257, 400), ("f32", 8, 8, 64, 16, 129, 600), ("f32", 12, 12, 32, 16, 100, 120),
    # cut by the lengths, the longest first: rows of 7 rounds to 24, 256 ranges and 1 536
    ("bf16", 32, 32, 128, 16, 17, 900), ("bf16", 32, 32, 128, 16, 48, 2900), ("bf16", 8, 8, 64, 32, 97, 2000), ("bf16", 16, 16, 256, 16, 33, 600),
    ("f32", 32, 8, 128, 16, 65, 300), ("f32", 8, 8, 32, 16, 65, 1500), ("bf16", 8, 2, 64, 16, 128, 1536), ("bf16", 16, 8, 128, 16, 33, 1000),
    ("bf16", 10, 2, 256, 16, 129, 800),
])
def test_many_ranges(dtype, H, Hkv, D, bs, batch, row):
    _check(dtype, H, Hkv, D, bs, batch, row, 5)


def _kinds(batch, row, rng):
    """Lengths and masks: one long among short ones, a few, few that run, none, all as long as can be, anything."""
    short = [int(x) for x in rng.randint(1, max(2, row // 20), batch)]
    few = [row - i if i % 7 == 3 else c for i, c in enumerate(short)]
    any_ = [int(x) for x in rng.randint(0, row + 1, batch)]
    yield [row if i == batch // 3 else c for i, c in enumerate(short)], [1] * batch
    yield few, [int(i % 5 != 1) for i in range(batch)]
    yield any_, [int(i in (1, batch - 1)) for i in range(batch)]
    yield any_, [0] * batch
    yield [row] * batch, [1] * batch
    yield any_, [int(x) for x in rng.rand(batch) < 0.7]
    yield [0] * batch, [1] * batch


def _skewed(dtype, H, Hkv, D, bs, batch, row):
    """All requests read the same blocks, each as far as its context."""
    rng = np.random.RandomState(batch + row)
    nblk = (row + bs - 1) // bs
    geom = W.Geometry(1, H, Hkv, D, bs, nblk + 2, nblk, dtype)
    rig = Rig(geom, batch)
    one, _ = W.deal_block_table(W.permutation(3, geom.num_blocks), [row], geom)
    table = np.repeat(one, batch, axis=0)
    K, V = W.logical_kv(70, geom, row)
    rig.page_requests(0, one, [K], [V])
    q = W.queries(6, geom, batch)
    for ctx, running in _kinds(batch, row, rng):
        rig.workspace.fill_(255)                         # NaN where no part writes
        got = to_f64(rig.decode(0, q, table, ctx, running, sentinel=7.0))
        on = np.asarray(running, dtype=bool)
        assert (got[~on] == 7.0).all()
        if on.any():
            ref = oracle.decode_attn(q[on], [K[:c] for c, r in zip(ctx, running) if r], [V[:c] for c, r in zip(ctx, running) if r],
                                     [c for c, r in zip(ctx, running) if r], [1] * int(on.sum()))
            assert np.abs(got[on] - ref).max() <= tol(geom), (ctx, running)
        assert np.array_equal(got, to_f64(rig.decode(0, q, table, ctx, running, sentinel=7.0)))
    rig.close()


@pytest.mark.parametrize("dtype,H,Hkv,D,bs,batch,row", [
    ("bf16", 32, 32, 64, 16, 17, 640), ("bf16", 8, 8, 64, 16, 70, 1500), ("bf16", 40, 40, 128, 16, 16, 1504), ("bf16", 16, 16, 256, 16, 20, 900),
    ("bf16", 16, 8, 128, 16, 40, 2000), ("bf16", 16, 8, 64, 32, 66, 2048), ("bf16", 128, 4, 64, 16, 40, 1000), ("bf16", 10, 2, 256, 16, 129, 800),
    ("f32", 8, 8, 32, 16, 40, 900), ("f32", 16, 2, 128, 32, 130, 400), ("f32", 6, 3, 64, 16, 100, 700), ("bf16", 4, 4, 128, 16, 256, 500),
])
def test_skewed_batches_of_many_ranges(dtype, H, Hkv, D, bs, batch, row):
    """Ranges that are cut by the lengths of the call, and whole ones behind them."""
    _skewed(dtype, H, Hkv, D, bs, batch, row)


@pytest.mark.parametrize("dtype,H,Hkv,D,bs,batch,row", [
    ("bf16", 8, 2, 128, 16, 10, 2500), ("bf16", 32, 1, 128, 16, 20, 1500), ("bf16", 16, 4, 64, 32, 16, 1600), ("bf16", 2, 1, 128, 16, 64, 1600), ("bf16", 8, 8, 64, 16, 11, 1300),
    ("bf16", 2, 2, 256, 16, 7, 2000), ("f32", 8, 2, 128, 16, 30, 900), ("f32", 4, 4, 32, 32, 16, 1100), ("bf16", 10, 2, 256, 16, 3, 5000),
    ("bf16", 8, 1, 128, 32, 9, 40000), ("bf16", 2, 2, 64, 16, 8, 30000), ("f32", 4, 2, 128, 16, 20, 9000), ("bf16", 4, 2, 128, 16, 40, 8000),
])
def test_skewed_batches_of_few_ranges(dtype, H, Hkv, D, bs, batch, row):
    """Ranges in parts of one size, which the lengths of the call decide."""
    _skewed(dtype, H, Hkv, D, bs, batch, row)


@pytest.mark.parametrize("dtype,H,Hkv,D,bs,batch,row", [
    ("bf16", 3, 3, 64, 16, 343, 100), ("bf16", 16, 16, 64, 16, 260, 250), ("bf16", 8, 8, 128, 32, 513, 380), ("f32", 8, 8, 64, 16, 515, 130), ("bf16", 16, 8, 64, 16, 131, 60),
    ("bf16", 64, 32, 64, 16, 129, 500),
])
def test_skewed_batches_of_ranges_in_pairs(dtype, H, Hkv, D, bs, batch, row):
    """Two waves to a range, and four to one whose neighbour waits; an odd number of ranges."""
    _skewed(dtype, H, Hkv, D, bs, batch, row)


@pytest.mark.parametrize("H,Hkv,batch,row", [(16, 8, 3, 400), (16, 8, 9, 500), (16, 8, 20, 700), (128, 8, 9, 500), (10, 2, 70, 300)])
def test_skewed_batches_of_heads_of_256(H, Hkv, batch, row):
    """In parts, by eight waves and four, cut by the lengths."""
    _skewed("bf16", H, Hkv, 256, 16, batch, row)


@pytest.mark.parametrize("dtype,H,Hkv,D,batch,row", [("bf16", 8, 2, 128, 4, 2000), ("bf16", 32, 32, 128, 34, 800), ("bf16", 8, 2, 128, 5, 300), ("bf16", 16, 8, 128, 130, 100),
                                                         ("bf16", 16, 8, 64, 70, 1600), ("f32", 8, 8, 64, 65, 1000)])
def test_replays_with_other_lengths(dtype, H, Hkv, D, batch, row):
    """The same graph over contexts that grow, shrink and trade places: order and stretches are worked out in the launch."""
    rng = np.random.RandomState(9)
    geom = W.Geometry(1, H, Hkv, D, 16, batch * ((row + 15) // 16) + 4, (row + 15) // 16, dtype)
    rig = Rig(geom, batch)
    full = [row] * batch
    table, _ = W.deal_block_table(W.permutation(3, geom.num_blocks), full, geom)
    K, V = zip(*[W.logical_kv(70 + 17 * r, geom, row) for r in range(batch)])
    rig.page_requests(0, table, K, V)
    q = W.queries(6, geom, batch)
    dq, dt = n2t(q, rig.dev), torch.as_tensor(table, device=rig.dev)
    dc = torch.zeros(batch, dtype=torch.int32, device=rig.dev)
    dm = torch.ones(batch, dtype=torch.uint8, device=rig.dev)
    out = torch.zeros(q.shape, device=rig.dev, dtype=rig.tdtype)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(rig.compute):
        rig.lamps.decode_attn(0, batch, dq, dt, dc, dm, out)
    rig.compute.synchronize()
    with torch.cuda.graph(graph, stream=rig.compute):
        rig.lamps.decode_attn(0, batch, dq, dt, dc, dm, out)
    for turn in range(3):
        ctx = [int(x) for x in rng.randint(0, (row if turn != 1 else row // 16) + 1, batch)]
        mask = [int(x) for x in rng.rand(batch) < 0.8]
        if turn == 1:
            ctx[0] = row
        mask[0] = 1
        dc.copy_(torch.as_tensor(np.asarray(ctx, dtype=np.int32)))
        dm.copy_(torch.as_tensor(np.asarray(mask, dtype=np.uint8)))
        out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        on = np.asarray(mask, dtype=bool)
        ref = oracle.decode_attn(q, [k[:c] for k, c in zip(K, ctx)], [v[:c] for v, c in zip(V, ctx)], ctx, mask)
        assert np.abs(to_f64(out)[on] - ref[on]).max() <= tol(geom)
        assert (to_f64(out)[~on] == 0.0).all()
    rig.close()
