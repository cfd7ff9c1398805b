"""lamps_prefill_attn: which workgroup takes which tile.  Batches whose requests bring very different
numbers of new tokens, where workgroups are started for the tiles there are only, against the fp64 oracle -- requests without new
tokens, one long prompt among short ones, up to and beyond the requests one wave keeps track of, head
counts that are no multiple of 8, every head size and layout."""
import numpy as np
import pytest
import torch

import lamps_workloads as W
import oracle
from rig import Rig, n2t, to_f64, tol

pytestmark = pytest.mark.gpu

#        H   Hkv D   requests, most new tokens, cached
CASES = [
    (4, 4, 128, 12, 900, 0),
    (16, 8, 128, 9, 700, 40),
    (6, 3, 64, 64, 300, 10),
    (2, 2, 64, 65, 500, 0),
    (2, 2, 256, 30, 300, 20),
    (4, 1, 256, 11, 200, 0),
    (2, 1, 64, 256, 200, 3),
    (1, 1, 64, 257, 300, 0),                          # one request too many for a wave
    (32, 1, 64, 20, 60, 5),
    (8, 8, 128, 3, 1100, 30),                         # one long prompt
]


@pytest.mark.parametrize("H,Hkv,D,n_req,most,cached", CASES)
def test_ragged_batches(H, Hkv, D, n_req, most, cached):
    rng = np.random.RandomState(n_req)
    new = [int(round(most ** u)) - 1 for u in rng.uniform(0, 0.7, n_req)]
    new[int(rng.randint(n_req))] = most
    _check(H, Hkv, D, new, cached, rng)


# the same for head counts that are no multiple of 8 where the full grid is larger than the chip and the
# longest request long enough for workgroups to be started for the tiles there are only, and just too short
@pytest.mark.parametrize("H,Hkv,D,n_req,most,cached", [(4, 4, 128, 24, 900, 0), (6, 3, 64, 64, 400, 10), (2, 1, 64, 256, 320, 3),
                                                       (2, 1, 64, 256, 319, 3), (32, 1, 64, 20, 330, 5), (4, 2, 128, 70, 100, 640)])
def test_ragged_batches_of_few_heads(H, Hkv, D, n_req, most, cached):
    test_ragged_batches(H, Hkv, D, n_req, most, cached)


#  launches that fit the chip at once, where half of the pairs take their tiles the other way round (4 and 8
#  tiles a pair), or not, as the second turn begins inside a pair's tiles (5, 12 and 7)
@pytest.mark.parametrize("H,Hkv,D,n_req,most,cached", [(8, 8, 64, 8, 640, 0), (8, 8, 64, 5, 1500, 0), (8, 8, 256, 5, 440, 70),
                                                       (16, 8, 128, 8, 512, 9), (8, 8, 128, 6, 500, 40)])
def test_even_batches(H, Hkv, D, n_req, most, cached):
    _check(H, Hkv, D, [most] * n_req, cached, np.random.RandomState(n_req))


def _check(H, Hkv, D, new, cached, rng):
    n_req = len(new)
    ctx = [max(n + int(rng.randint(cached + 1)), 1) for n in new]
    bs = 16
    blocks = [(c + bs - 1) // bs for c in ctx]
    geom = W.Geometry(1, H, Hkv, D, bs, sum(blocks) + 4, max(blocks), "bf16")
    rig = Rig(geom, n_req)
    table, _ = W.deal_block_table(W.permutation(8, geom.num_blocks), ctx, geom)
    K, V = zip(*[W.logical_kv(900 + 17 * r, geom, c) for r, c in enumerate(ctx)])
    rig.page_requests(0, table, K, V)
    q_start = np.concatenate([[0], np.cumsum(new)]).astype(np.int32)
    total, dev = int(q_start[-1]), rig.dev
    q = W.queries(78 + D, geom, total)
    out = torch.full((total, H, D), 7.0, dtype=rig.tdtype, device=dev)
    with torch.cuda.stream(rig.compute):
        rig.lamps.prefill_attn(0, n_req, total, n2t(q, dev), torch.as_tensor(q_start, device=dev), torch.as_tensor(table, device=dev),
                               torch.as_tensor(np.asarray(ctx, dtype=np.int32), device=dev), out, max_new_tokens=max(new))
    rig.compute.synchronize()
    assert np.abs(to_f64(out) - oracle.prefill_attn(q, K, V, q_start, ctx, threads=8)).max() <= tol(geom)
    rig.close()
