"""Recorded decode and prefill launches of one context, which share its workspace, replayed in one order on a stream
that is not the compute stream, with nothing but that order between them."""
import numpy as np
import pytest
import torch

import lamps_workloads as W
from rig import Rig, n2t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,Hkv,D", [(8, 2, 128), (4, 4, 64), (8, 1, 256)])
def test_replays_in_one_order(H, Hkv, D):
    ctx, new = [2000, 1300, 40], [20, 64, 7]
    blocks = [(c + 15) // 16 for c in ctx]
    geom = W.Geometry(1, H, Hkv, D, 16, sum(blocks) + 4, max(blocks), "bf16")
    rig = Rig(geom, 3)
    table, _ = W.deal_block_table(W.permutation(5, geom.num_blocks), ctx, geom)
    rig.page_requests(0, table, *zip(*[W.logical_kv(11 + 17 * r, geom, c) for r, c in enumerate(ctx)]))
    dev = rig.dev
    q_start = torch.as_tensor(np.concatenate([[0], np.cumsum(new)]).astype(np.int32), device=dev)
    td, cd = torch.as_tensor(table, device=dev), torch.as_tensor(np.asarray(ctx, dtype=np.int32), device=dev)
    mask = torch.ones(3, dtype=torch.uint8, device=dev)
    q1, q2 = n2t(W.queries(1, geom, 3), dev), n2t(W.queries(2, geom, sum(new)), dev)
    o1, o2 = torch.zeros_like(q1), torch.zeros_like(q2)

    def decode():
        rig.lamps.decode_attn(0, 3, q1, td, cd, mask, o1)

    def prefill():
        rig.lamps.prefill_attn(0, 3, sum(new), q2, q_start, td, cd, o2, max_new_tokens=max(new))

    torch.cuda.synchronize()
    graphs, want = [], []
    for call, out in ((decode, o1), (prefill, o2)):
        with torch.cuda.stream(rig.compute):
            call()
        rig.compute.synchronize()
        want.append(out.clone())
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=rig.compute):
            call()
        graphs.append(graph)
    side = torch.cuda.Stream(dev)
    torch.cuda.synchronize()
    got = []
    with torch.cuda.stream(side):
        for k in (0, 1, 1, 0, 1, 0, 0, 1):
            (o1, o2)[k].fill_(float("nan"))
            graphs[k].replay()
            got.append((k, (o1, o2)[k].clone()))
    torch.cuda.synchronize()
    for k, out in got:
        assert torch.equal(out, want[k])
    rig.close()
