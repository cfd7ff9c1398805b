"""lamps_kv_append_tokens finds the request of a token (or of a 16-position sub-tile) 64 requests at a
time: batches around one, 64 and several times 64 requests, with requests that bring no tokens first,
last and in runs, byte for byte against the harness' pager."""
import numpy as np
import pytest
import torch

import lamps_workloads as W
from rig import Rig, n2t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,H,Hkv,D", [("bf16", 2, 2, 64), ("bf16", 4, 2, 128), ("bf16", 2, 1, 256), ("f32", 1, 1, 32)])
@pytest.mark.parametrize("n_req", [1, 2, 63, 64, 65, 130, 300])
def test_tokens_reach_their_requests(dtype, H, Hkv, D, n_req):
    rng = np.random.RandomState(n_req)
    new = rng.choice([0, 0, 1, 2, 15, 16, 17, 33], n_req)
    new[rng.randint(n_req)] = 5
    if n_req > 2:
        new[0] = new[-1] = 0
    old = rng.randint(0, 20, n_req)
    ctx = [int(a + b) for a, b in zip(old, new)]
    geom = W.Geometry(1, H, Hkv, D, 16, sum((c + 15) // 16 for c in ctx) + 4, max(max((c + 15) // 16 for c in ctx), 1), dtype)
    rig = Rig(geom, n_req)
    table, _ = W.deal_block_table(W.permutation(4, geom.num_blocks), ctx, geom)
    K, V = zip(*[W.logical_kv(30 + 17 * r, geom, c) for r, c in enumerate(ctx)])
    rig.page_requests(0, table, [k[:n] for k, n in zip(K, old)], [v[:n] for v, n in zip(V, old)])
    kn = np.concatenate([k[n:] for k, n in zip(K, old)])
    vn = np.concatenate([v[n:] for v, n in zip(V, old)])
    q_start = np.concatenate([[0], np.cumsum(new)]).astype(np.int32)
    dev = rig.dev
    with torch.cuda.stream(rig.compute):
        rig.lamps.kv_append_tokens(0, n_req, int(q_start[-1]), n2t(kn, dev), n2t(vn, dev), torch.as_tensor(q_start, device=dev),
                                   torch.as_tensor(table, device=dev), torch.as_tensor(np.asarray(ctx, dtype=np.int32), device=dev))
    rig.compute.synchronize()
    kp = np.full(geom.pool_shape, W.poison(geom), dtype=geom.np_dtype)
    vp = kp.copy()
    for r in range(n_req):
        W.page(kp, 0, table[r], K[r], rig.k_index)
        W.page(vp, 0, table[r], V[r], rig.v_index)
    got_k, got_v = rig.host_pools()
    assert got_k.tobytes() == kp.tobytes() and got_v.tobytes() == vp.tobytes()
    rig.close()


# around the number of requests that are told apart one by one, and around the size of a row whose
# vectors are asked for early (4 KiB)
@pytest.mark.parametrize("dtype,H,Hkv,D,n_req", [("bf16", 4, 2, 128, 15), ("bf16", 4, 2, 128, 16), ("bf16", 4, 1, 64, 17), ("bf16", 32, 32, 64, 5),
                                                 ("bf16", 33, 33, 64, 20), ("bf16", 16, 16, 256, 14), ("f32", 8, 8, 128, 9), ("f32", 9, 9, 128, 66)])
def test_few_requests_and_long_rows(dtype, H, Hkv, D, n_req):
    test_tokens_reach_their_requests(dtype, H, Hkv, D, n_req)
