"""lamps_decode_attn on small launches -- shares that are pieces of one range each, shares of a whole
workgroup, and the two on either side of the rules that choose them -- against the fp64 oracle: single
requests around a chunk and a share, paused and empty requests in between, one long context among short
ones, more requests than threads, few and many ranges per resident wave.  With table rows that the longest context fills, by which most of these
go whole or in parts, and with rows longer than the pool, by which all of them go in shares."""
import numpy as np
import pytest
import torch

import lamps_workloads as W
import oracle
from rig import Rig, to_f64, tol

pytestmark = pytest.mark.gpu

ONE = [[1], [15], [16], [17], [63], [64], [65], [257], [1030]]
MIX = [[40, 0, 3, 900], [20, 33, 17, 64, 1, 128], [5000, 20, 20, 31], [100] * 40, [9] * 256, [7 + i % 50 for i in range(257)],
       [2500] + [25] * 60]
GEOMS = [("bf16", 4, 4, 128, 16), ("bf16", 8, 2, 128, 16), ("bf16", 2, 2, 256, 32), ("bf16", 4, 4, 64, 16), ("bf16", 16, 1, 64, 16),
         ("f32", 8, 2, 128, 16), ("f32", 4, 4, 32, 16)]


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("dtype,H,Hkv,D,bs", GEOMS)
def test_small_launches(dtype, H, Hkv, D, bs, wide):
    for ctx in ONE + MIX:
        blocks = [(c + bs - 1) // bs for c in ctx]
        geom = W.Geometry(1, H, Hkv, D, bs, sum(blocks) + 4, sum(blocks) + 5 if wide else max(max(blocks), 1), dtype)
        rig = Rig(geom, len(ctx))
        table, _ = W.deal_block_table(W.permutation(3, geom.num_blocks), ctx, geom)
        K, V = zip(*[W.logical_kv(70 + 17 * r, geom, c) for r, c in enumerate(ctx)])
        rig.page_requests(0, table, K, V)
        running = [0 if len(ctx) > 1 and r % 5 == 1 else 1 for r in range(len(ctx))]
        q = W.queries(6, geom, len(ctx))
        got = to_f64(rig.decode(0, q, table, ctx, running, sentinel=7.0))
        again = to_f64(rig.decode(0, q, table, ctx, running, sentinel=7.0))
        ref = oracle.decode_attn(q, K, V, ctx, running)
        on = np.asarray(running, dtype=bool)
        assert np.abs(got[on] - ref[on]).max() <= tol(geom), ctx
        assert (got[~on] == 7.0).all() and np.array_equal(got, again), ctx
        rig.close()
