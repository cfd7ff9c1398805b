"""lamps_prefill_attn where a launch is several times what the chip holds and the (request, head) pairs of an XCD go abreast:
all together, in parts of which the last is smaller, with pairs left over that fill no group of 8, and where they go one by one for
all that; rows against the fp64 oracle.  Which of these a launch does is asserted on the CPU (test_prefill_rules_cpu.py)."""
import numpy as np
import pytest
import torch

import lamps_workloads as W
import oracle
from rig import Rig, n2t, to_f64, tol

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,Hkv,D,dtype,row,reqs", [
    (40, 40, 64, "bf16", 640, [(300, 300), (320, 317), (290, 290), (305, 301), (310, 310)]),   # 25 groups, one by one
    (18, 9, 64, "bf16", 2048, [(600, 600), (590, 580), (610, 610)]),                          # 3 groups, 3 pairs left over, one part (the contexts decide)
    (32, 8, 256, "bf16", 4096, [(700, 700), (690, 688), (700, 695)]),                         # 3 groups, one part (the contexts decide)
    (16, 16, 256, "bf16", 6144, [(1030, 1030), (1024, 1024)]),                                # 4 groups, one part (the contexts decide)
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


@pytest.mark.parametrize("H,Hkv,D,dtype,row,reqs", [
    (40, 40, 64, "bf16", 608, [(400, 400), (420, 420), (440, 431), (505, 501), (410, 396)]),   # 25 groups, one part
    (18, 9, 64, "bf16", 1200, [(600, 600), (590, 580), (610, 610)]),                          # 3 groups, 3 pairs left over, one part
    (8, 8, 256, "bf16", 3584, [(1800, 1800), (1790, 1785), (1300, 1290)]),                    # 3 groups in parts of 2 and 1
    (32, 32, 128, "bf16", 1100, [(200 + 90 * r, 250 if r == 4 else 100 + 8 * r) for r in range(10)]),           # few tiles, 40 groups in two parts
])
def test_parts(H, Hkv, D, dtype, row, reqs):
    test_rows(H, Hkv, D, dtype, row, reqs)


@pytest.mark.parametrize("H,Hkv,D,dtype,row,reqs", [
    (18, 9, 64, "bf16", 8192, [(600, 600), (590, 580), (610, 610)]),                          # 3 groups, 3 pairs left over, one part
    (18, 9, 64, "bf16", 8192, [(600, 600), (1190, 580), (1830, 610)]),                        # a context of three times the new tokens: one by one
    (8, 8, 256, "bf16", 8192, [(3500, 1800), (1790, 1785), (1300, 1290)]),                    # in parts of 2 and 1
    (9, 9, 64, "f32", 4096, [(400, 400), (390, 390), (410, 401)]),
    (8, 8, 64, "f32", 8192, [(130 + 3 * r, 130 - r // 2) for r in range(64)]),                     # a request per lane
])
def test_contexts_decide(H, Hkv, D, dtype, row, reqs):
    """A table row that rules nothing in: the workgroups look at the contexts themselves."""
    test_rows(H, Hkv, D, dtype, row, reqs)
