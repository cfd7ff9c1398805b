"""lamps_prefill_attn with two teams of waves to a tile: launches over the line, lengths around a stage, a wave's columns and a tile,
tiles with waves that have no tokens, contexts that end inside a stage, both layouts, against the fp64 oracle; the rest of the pools is
NaN, and the launch is replayed from a HIP graph, bit for bit the same."""
import numpy as np
import pytest
import torch

import lamps_workloads as W
import oracle
from rig import Rig, n2t, to_f64, tol

pytestmark = pytest.mark.gpu

CASES = [
    # heads, block, new tokens, cached.  Tiles of 256 / G tokens (128 / G at 256), 32 / G (16 / G) to a wave
    (32, 2, 128, 16, [470, 464, 480, 481, 450, 455, 449], 0),             # 16 to a group: 16 tokens a tile, 2 a wave
    (56, 8, 128, 16, [470, 451, 449, 460], 0),                                # 7 to a group: 32 a tile, 4 columns of a wave empty
    (128, 4, 128, 32, [460, 451, 452], 5),                                    # 32 to a group
    (32, 32, 128, 16, [1024, 1023, 1057], 0),                                 # plain
    (40, 40, 128, 32, [255, 256, 240, 250, 256, 251, 256, 249, 256, 225], 700),    # one tile a request, over cached positions
    (32, 32, 256, 16, [512, 545, 497], 0),
    (32, 32, 256, 32, [128, 120, 127, 125, 113], 640),
    (8, 4, 256, 16, [1, 31, 32, 33, 64, 65, 130], 3),                         # grouped heads of 256: any size
    (12, 4, 256, 32, [2, 5, 40, 41, 170], 0),                                 # 3 to a group
]


@pytest.mark.parametrize("H,Hkv,D,bs,new,cached", CASES)
def test_rows(H, Hkv, D, bs, new, cached):
    B, ctx = len(new), [n + cached + (7 * i) % 31 * (cached > 0) for i, n in enumerate(new)]
    blocks = [(c + bs - 1) // bs for c in ctx]
    geom = W.Geometry(1, H, Hkv, D, bs, sum(blocks) + 4, max(blocks), "bf16")
    rig = Rig(geom, B)
    table, _ = W.deal_block_table(W.permutation(7, geom.num_blocks), ctx, geom)
    K, V = zip(*[W.logical_kv(70 + 17 * r, geom, c) for r, c in enumerate(ctx)])
    rig.page_requests(0, table, K, V)
    q = W.queries(13, geom, sum(new)) + np.uint16(0x80)   # (bf16 bits, doubled: scores that move the reference point now and then)
    q_start = np.concatenate([[0], np.cumsum(new)]).astype(np.int32)
    out = torch.full(q.shape, 7.0, device=rig.dev, dtype=rig.tdtype)
    dq = n2t(q, rig.dev)
    args = (torch.as_tensor(q_start, device=rig.dev), torch.as_tensor(table, device=rig.dev),
            torch.as_tensor(np.asarray(ctx, dtype=np.int32), device=rig.dev))

    def call():
        rig.lamps.prefill_attn(0, B, sum(new), dq, *args, out, max_new_tokens=max(new))

    with torch.cuda.stream(rig.compute):
        call()
    rig.compute.synchronize()
    got = to_f64(out)
    # sampled: the first and last tokens of each request and some between, each a prompt of one token over its prefix
    rng = np.random.RandomState(3)
    rows, Ks, Vs, ends = [], [], [], []
    for r, n in enumerate(new):
        for t in sorted({0, n - 1, n // 2, *rng.randint(0, n, 6).tolist()}):
            rows.append(int(q_start[r]) + t)
            ends.append(ctx[r] - n + t + 1)
            Ks.append(K[r][:ends[-1]])
            Vs.append(V[r][:ends[-1]])
    want = oracle.prefill_attn(q[rows], Ks, Vs, np.arange(len(rows) + 1, dtype=np.int32), ends, threads=8)
    assert np.abs(got[rows] - want).max() <= tol(geom)
    assert np.isfinite(got).all()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=rig.compute):
        call()
    for _ in range(3):
        out.fill_(5.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(to_f64(out), got)
    rig.close()


@pytest.mark.parametrize("H,Hkv,D,new,cached,double", [
    (32, 8, 128, [1000, 997, 1001, 1002], 0, 0), (32, 8, 128, [1000, 997, 1001, 1002], 0, 2), (32, 32, 128, [1030, 1025, 1029, 1036], 0, 2),
    (16, 16, 256, [512, 513, 511, 512], 400, 2),
])
def test_a_row_has_the_same_bits_by_either_kernel(H, Hkv, D, new, cached, double):
    """Together the requests go by two teams of waves, each alone by the kernel of four: a row does not depend on the requests beside it.
    Queries of N(0, 1), and doubled twice: there the reference point of the exponentials moves in most stages of some wave."""
    B, ctx = len(new), [n + cached for n in new]
    geom = W.Geometry(1, H, Hkv, D, 16, sum((c + 15) // 16 for c in ctx) + 4, (max(ctx) + 15) // 16, "bf16")
    rig = Rig(geom, B)
    table, _ = W.deal_block_table(W.permutation(7, geom.num_blocks), ctx, geom)
    g = torch.Generator(rig.dev).manual_seed(4)
    for pool in (rig.k_pool, rig.v_pool):
        pool.copy_(torch.randn(pool.shape, generator=g, device=rig.dev))
    dq = (torch.randn((sum(new), H, D), generator=g, device=rig.dev) * 2 ** double).to(rig.tdtype)
    out, alone = torch.full_like(dq, 7.0), torch.full_like(dq, 5.0)
    dt, dc = torch.as_tensor(table, device=rig.dev), torch.as_tensor(np.asarray(ctx, dtype=np.int32), device=rig.dev)
    first = np.concatenate([[0], np.cumsum(new)]).astype(np.int32)
    starts = [torch.as_tensor(np.asarray(x, dtype=np.int32), device=rig.dev) for x in [first] + [[0, n] for n in new]]
    torch.cuda.synchronize()
    with torch.cuda.stream(rig.compute):
        rig.lamps.prefill_attn(0, B, sum(new), dq, starts[0], dt, dc, out, max_new_tokens=max(new))
        for r, n in enumerate(new):
            rig.lamps.prefill_attn(0, 1, n, dq[first[r]:], starts[1 + r], dt[r:r + 1].contiguous(), dc[r:r + 1].contiguous(), alone[first[r]:],
                                   max_new_tokens=n)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), alone.view(torch.int16))
    rig.close()
