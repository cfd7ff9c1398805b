"""lamps_prefill_attn on few new tokens over long contexts: the launches that cut a tile's cached
positions into runs and add them up in the workspace, against the fp64 oracle at the sizes where that
can go wrong (one position more or less than a run, the last run short, tiles of one request with
different numbers of runs, requests without new tokens, every head size, layout and tile width), with
the workspace full of NaN, replayed from a HIP graph, and bit for bit the same every time."""
import numpy as np
import pytest
import torch

import lamps_workloads as W
import oracle
from rig import Rig, n2t, to_f64, tol

pytestmark = pytest.mark.gpu

#        H  Hkv D    bs  (context, new tokens) per request
CASES = [
    (8, 2, 128, 16, [(1500, 20), (40, 3), (1200, 0), (1025, 64), (9, 9)]),
    (8, 2, 128, 32, [(1536, 16), (1537, 17), (1535, 1), (384, 16), (385, 16), (383, 16)]),
    (4, 4, 128, 16, [(2100, 65), (1030, 64), (700, 1)]),
    (4, 4, 64, 16, [(1024, 3), (3000, 70)]),
    (8, 2, 64, 64, [(1999, 40)]),
    (4, 4, 256, 16, [(1100, 70), (1700, 5)]),
    (8, 1, 256, 16, [(1300, 9), (2000, 17)]),
    (32, 1, 128, 16, [(1500, 5), (60, 2)]),                          # 32 heads per kv head: tiles of 128 columns
    (6, 2, 128, 16, [(1400, 30), (1100, 6)]),                        # group of 3: 15 of 16 columns in use
    (8, 2, 128, 16, [(2000, 300)]),                                  # many columns: tiles of 128
    (8, 1, 128, 16, [(1100 + 7 * i, 1 + i % 4) for i in range(64)]),   # the most requests
]


@pytest.mark.parametrize("H,Hkv,D,bs,reqs", CASES)
def test_split_contexts(H, Hkv, D, bs, reqs):
    ctx, new = [c for c, _ in reqs], [n for _, n in reqs]
    blocks = [(c + bs - 1) // bs for c in ctx]
    geom = W.Geometry(1, H, Hkv, D, bs, sum(blocks) + 4, max(blocks), "bf16")
    rig = Rig(geom, len(reqs))
    table, _ = W.deal_block_table(W.permutation(5, geom.num_blocks), ctx, geom)
    K, V = zip(*[W.logical_kv(600 + 17 * r, geom, c) for r, c in enumerate(ctx)])
    rig.page_requests(0, table, K, V)
    q_start = np.concatenate([[0], np.cumsum(new)]).astype(np.int32)
    total, dev = int(q_start[-1]), rig.dev
    q = W.queries(77 + D, geom, total)
    ref = oracle.prefill_attn(q, K, V, q_start, ctx, threads=8)
    qd, sd, td = n2t(q, dev), torch.as_tensor(q_start, device=dev), torch.as_tensor(table, device=dev)
    cd = torch.as_tensor(np.asarray(ctx, dtype=np.int32), device=dev)
    out = torch.full((total, H, D), 7.0, dtype=rig.tdtype, device=dev)

    def call():
        rig.lamps.prefill_attn(0, len(reqs), total, qd, sd, td, cd, out, max_new_tokens=max(new))

    rig.workspace.fill_(255)                             # NaN, and counts that no launch has left there
    torch.cuda.synchronize()
    with torch.cuda.stream(rig.compute):
        call()
    rig.compute.synchronize()
    first = out.clone()
    assert np.abs(to_f64(first) - ref).max() <= tol(geom)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=rig.compute):
        call()
    for k in range(4):                                   # replays (the same launch again) and eager calls in turn
        out.fill_(float("nan"))
        if k == 2:
            rig.workspace.fill_(0)
        torch.cuda.synchronize()
        if k % 2:
            with torch.cuda.stream(rig.compute):
                call()
        else:
            graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, first)
    rig.close()
