"""The reducers that keep a chunk's loads in flight while they work on the one before it: every number of chunks
that a wave can have at a time (an even number starts from the other set of registers), last ones full and
ragged, against the fp64 oracle.  Fixed partitions give a wave a whole range; fp32 prompts a quarter of its chunks."""
import numpy as np
import pytest
import torch

import lamps_workloads as W
import oracle
from rig import Rig, n2t, to_f64, tol

pytestmark = pytest.mark.gpu

LENGTHS = [1, 15, 16, 17, 32, 33, 48, 49, 64, 65, 80, 81, 96, 113, 128, 255, 256, 257, 400]


def _rig(H, Hkv, D, dtype, ctx, **kw):
    blocks = [(c + 15) // 16 for c in ctx]
    geom = W.Geometry(1, H, Hkv, D, 16, sum(blocks) + 4, max(blocks), dtype)
    rig = Rig(geom, len(ctx), **kw)
    table, _ = W.deal_block_table(W.permutation(8, geom.num_blocks), ctx, geom)
    K, V = zip(*[W.logical_kv(30 + 17 * r, geom, c) for r, c in enumerate(ctx)])
    rig.page_requests(0, table, K, V)
    return geom, rig, table, list(K), list(V)


@pytest.mark.parametrize("D", [64, 128, 256])
def test_decode(D):
    geom, rig, table, K, V = _rig(8, 2, D, "bf16", LENGTHS, part_tokens=256)
    q = W.queries(9, geom, len(LENGTHS))
    on = [1] * len(LENGTHS)
    got = to_f64(rig.decode(0, q, table, LENGTHS, on))
    assert np.abs(got - oracle.decode_attn(q, K, V, LENGTHS, on)).max() <= tol(geom)
    rig.close()


@pytest.mark.parametrize("D", [32, 64, 128])
def test_prefill(D):
    new = [min(c, 1 + 5 * r) for r, c in enumerate(LENGTHS)]
    geom, rig, table, K, V = _rig(4, 2, D, "f32", LENGTHS)
    q = W.queries(10, geom, sum(new))
    q_start = np.concatenate([[0], np.cumsum(new)]).astype(np.int32)
    out = torch.full(q.shape, 7.0, device=rig.dev)
    with torch.cuda.stream(rig.compute):
        rig.lamps.prefill_attn(0, len(new), sum(new), n2t(q, rig.dev), torch.as_tensor(q_start, device=rig.dev),
                               torch.as_tensor(table, device=rig.dev),
                               torch.as_tensor(np.asarray(LENGTHS, dtype=np.int32), device=rig.dev), out, max_new_tokens=max(new))
    rig.compute.synchronize()
    assert np.abs(to_f64(out) - oracle.prefill_attn(q, K, V, q_start, LENGTHS, threads=8)).max() <= tol(geom)
    rig.close()
