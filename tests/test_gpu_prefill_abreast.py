"""lamps_prefill_attn where a launch is several times what the chip holds and the (request, head) pairs of an XCD go abreast:
all together, in parts of which the last is smaller, with pairs left over that fill no group of 8; rows against the fp64 oracle."""
import numpy as np
import pytest
import torch

import lamps_workloads as W
import oracle
from rig import Rig, n2t, to_f64, tol

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,Hkv,D,dtype,row,reqs", [
    (40, 40, 64, "bf16", 640, [(300, 300), (320, 317), (290, 290), (305, 301), (310, 310)]),   # 25 groups, one part
    (18, 9, 64, "bf16", 2048, [(600, 600), (590, 580), (610, 610)]),                          # 3 groups, 3 pairs left over
    (32, 8, 256, "bf16", 4096, [(700, 700), (690, 688), (700, 695)]),                         # 3 groups in parts of 2 and 1
    (16, 16, 256, "bf16", 6144, [(1030, 1030), (1024, 1024)]),                                # 4 groups in parts of 1
    (9, 9, 64, "f32", 512, [(400, 400), (390, 390), (410, 401)]),
])
def test_rows(H, Hkv, D, dtype, row, reqs):
    ctx, new = [c for c, _ in reqs], [n for _, n in reqs]
    geom = W.Geometry(1, H, Hkv, D, 16, sum((c + 15) // 16 for c in ctx) + 4, row // 16, dtype)
    rig = Rig(geom, len(ctx))
    table, _ = W.deal_block_table(W.permutation(3, geom.num_blocks), ctx, geom)
    K, V = zip(*[W.logical_kv(50 + 17 * r, geom, c) for r, c in enumerate(ctx)])
    rig.page_requests(0, table, K, V)
    q = W.queries(11, geom, sum(new))
    q_start = np.concatenate([[0], np.cumsum(new)]).astype(np.int32)
    out = torch.full(q.shape, 7.0, device=rig.dev, dtype=rig.tdtype)
    with torch.cuda.stream(rig.compute):
        rig.lamps.prefill_attn(0, len(ctx), sum(new), n2t(q, rig.dev), torch.as_tensor(q_start, device=rig.dev),
                               torch.as_tensor(table, device=rig.dev), torch.as_tensor(np.asarray(ctx, dtype=np.int32), device=rig.dev),
                               out, max_new_tokens=max(new))
    rig.compute.synchronize()
    assert np.abs(to_f64(out) - oracle.prefill_attn(q, K, V, q_start, ctx, threads=8)).max() <= tol(geom)
    rig.close()
