"""fp32 lamps_prefill_attn, which workgroup takes which tile: launches with a workgroup per (request, head, tile), with one per
tile there is (one long prompt among short ones, the most new tokens unknown), and numbered by request (more
requests than a wave keeps track of), requests without new tokens in between; kv groups of more heads than a
tile has columns; and a batch whose full grid no launch could have."""
import numpy as np
import pytest
import torch

import lamps_workloads as W
import oracle
import paper_2410_18248_amd as P
from rig import Rig, n2t, to_f64, tol

pytestmark = pytest.mark.gpu

MANY = [(3 * i) % 7 for i in range(300)]
#        H   Hkv D    new tokens per request, cached, the bound is given
CASES = [
    (8, 8, 64, [17, 0, 64, 5], 30, True),
    (8, 8, 64, [600] + [3, 0, 9, 20] * 8, 20, True),
    (8, 2, 128, [200] + [1, 0, 7] * 15, 0, False),
    (4, 4, 32, [33] * 120, 0, False),
    (4, 1, 64, [25, 0, 1, 40], 50, False),
    (8, 8, 64, [700] + MANY, 5, True),                               # by request
    (8, 2, 128, MANY, 40, False),
    (2, 1, 32, [0, 0] + MANY + [90, 0], 0, False),
    (32, 1, 64, [40, 17, 0, 3], 60, True),                           # two passes of 16 heads
    (40, 2, 32, [21, 50], 20, True),                                 # two of 10: one token a tile, unused columns
    (17, 1, 128, [9, 30, 1], 20, True),                              # seventeen of one
    (34, 2, 64, [30] + [2, 5] * 20, 10, False),
]


@pytest.mark.parametrize("H,Hkv,D,new,cached,known", CASES)
def test_batches(H, Hkv, D, new, cached, known):
    rng = np.random.RandomState(len(new))
    ctx = [max(n + int(rng.randint(cached + 1)), 1) for n in new]
    blocks = [(c + 15) // 16 for c in ctx]
    geom = W.Geometry(1, H, Hkv, D, 16, sum(blocks) + 4, max(blocks), "f32")
    rig = Rig(geom, len(new))
    table, _ = W.deal_block_table(W.permutation(4, geom.num_blocks), ctx, geom)
    K, V = zip(*[W.logical_kv(50 + 17 * r, geom, c) for r, c in enumerate(ctx)])
    rig.page_requests(0, table, K, V)
    q_start = np.concatenate([[0], np.cumsum(new)]).astype(np.int32)
    total, dev = int(q_start[-1]), rig.dev
    q = W.queries(8 + D, geom, total)
    out = torch.full((total, H, D), 7.0, device=dev)
    with torch.cuda.stream(rig.compute):
        rig.lamps.prefill_attn(0, len(new), total, n2t(q, dev), torch.as_tensor(q_start, device=dev), torch.as_tensor(table, device=dev),
                               torch.as_tensor(np.asarray(ctx, dtype=np.int32), device=dev), out,
                               max_new_tokens=max(new) if known else 0)
    rig.compute.synchronize()
    assert np.abs(to_f64(out) - oracle.prefill_attn(q, K, V, q_start, ctx, threads=8)).max() <= tol(geom)
    rig.close()


def test_more_places_than_a_grid_has():
    """8 192 requests of four and five tokens on 128 heads, the most new tokens unknown: requests x heads x tiles of
    the batch's tokens are more than 2^31.  All requests read one block; expected values in float64."""
    H, D, B = 128, 32, 8192
    new = np.where(np.arange(B) % 2 == 0, 4, 5).astype(np.int32)
    start = np.concatenate([[0], np.cumsum(new)]).astype(np.int32)
    total, dev = int(start[-1]), torch.device("cuda:0")
    assert H * B * ((total + 15) // 16) > 0x7fffffff
    cfg = P.LampsConfig(1, H, H, D, 16, 1, 1, B, P.LAMPS_F32)
    g = torch.Generator(dev).manual_seed(2)
    kp, vp = (torch.randn(1, 1, H, 16 * D, generator=g, device=dev) for _ in range(2))
    q = torch.randn(total, H, D, generator=g, device=dev)
    out = torch.full_like(q, 7.0)
    ws = torch.empty(P.lamps_workspace_bytes(cfg), dtype=torch.uint8, device=dev)
    lam = P.Lamps(cfg, kp, vp, ws)
    lam.prefill_attn(0, B, total, q, torch.as_tensor(start, device=dev), torch.zeros(B, 1, dtype=torch.int32, device=dev),
                     torch.as_tensor(new, device=dev), out)
    torch.cuda.synchronize()
    at = torch.as_tensor(np.arange(total) - np.repeat(start[:-1], new), device=dev)
    seen = torch.arange(5, device=dev)[None, :] <= at[:, None]
    k, v = (x.view(H, 16, D)[:, :5].double() for x in (kp, vp))
    for h in range(0, H, 16):
        s = torch.stack([q[:, i].double() @ k[i].t() for i in range(h, h + 16)]) / D ** 0.5
        w = torch.softmax(s.masked_fill(~seen[None], -torch.inf), 2)
        ref = torch.stack([w[i] @ v[h + i] for i in range(16)], 1)
        assert (out[:, h:h + 16].double() - ref).abs().max() <= 1e-5
    lam.destroy()
