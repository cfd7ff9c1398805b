"""lamps_prefill_attn on both sides of the line between tiles of 64 and of 128 columns: launches of a few rounds and of more, a stage
and two at a time, lengths at the edges of both tiles, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import lamps_workloads as W
import oracle
from rig import Rig, n2t, to_f64, tol

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,Hkv,D", [(24, 24, 128), (16, 8, 128), (8, 8, 64), (16, 8, 64), (6, 3, 64)])
@pytest.mark.parametrize("B,most", [(5, 30), (5, 150), (6, 390), (36, 129), (160, 28), (160, 140)])
def test_rows(H, Hkv, D, B, most):
    rng = np.random.RandomState(B + most)
    edges = [1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 150, 390]
    new = [int(x) for x in rng.choice([e for e in edges if e <= (most if B < 100 else 33)], B)]
    new[B // 2] = most
    ctx = [n + int(x) for n, x in zip(new, rng.choice([0, 0, 1, 17, 40], B))]
    blocks = [(c + 15) // 16 for c in ctx]
    geom = W.Geometry(1, H, Hkv, D, 16, sum(blocks) + 4, max(blocks), "bf16")
    rig = Rig(geom, B)
    table, _ = W.deal_block_table(W.permutation(7, geom.num_blocks), ctx, geom)
    K, V = zip(*[W.logical_kv(70 + 17 * r, geom, c) for r, c in enumerate(ctx)])
    rig.page_requests(0, table, K, V)
    q = W.queries(13, geom, sum(new))
    q_start = np.concatenate([[0], np.cumsum(new)]).astype(np.int32)
    want = oracle.prefill_attn(q, K, V, q_start, ctx, threads=8)
    for known in (max(new), 0):                         # the most new tokens known to the caller, or not
        out = torch.full(q.shape, 7.0, device=rig.dev, dtype=rig.tdtype)
        with torch.cuda.stream(rig.compute):
            rig.lamps.prefill_attn(0, B, sum(new), n2t(q, rig.dev), torch.as_tensor(q_start, device=rig.dev),
                                   torch.as_tensor(table, device=rig.dev), torch.as_tensor(np.asarray(ctx, dtype=np.int32), device=rig.dev),
                                   out, max_new_tokens=known)
        rig.compute.synchronize()
        assert np.abs(to_f64(out) - want).max() <= tol(geom)
    rig.close()


@pytest.mark.parametrize("H,Hkv,D", [(12, 2, 128), (18, 2, 64), (20, 2, 128)])
@pytest.mark.parametrize("B,most", [(5, 150), (36, 129)])
def test_groups_that_leave_columns_empty(H, Hkv, D, B, most):
    test_rows(H, Hkv, D, B, most)
