"""fp32 attention: many new tokens on the matrix cores, decode beside it
at the edges of its tiles and chunks of 16, against the fp64 oracle; and values that are no finite
numbers stay with the tokens that see them."""
import numpy as np
import pytest
import torch

import lamps_workloads as W
import oracle
from rig import Rig, n2t, to_f64, tol

pytestmark = pytest.mark.gpu

REQS = [(1, 1), (15, 15), (16, 16), (17, 17), (33, 33), (64, 1), (65, 5), (130, 0), (200, 48)]


def _rig(H, Hkv, D, bs, reqs, seed):
    ctx = [c for c, _ in reqs]
    blocks = [(c + bs - 1) // bs for c in ctx]
    geom = W.Geometry(1, H, Hkv, D, bs, sum(blocks) + 4, max(blocks), "f32")
    rig = Rig(geom, len(reqs))
    table, _ = W.deal_block_table(W.permutation(seed, geom.num_blocks), ctx, geom)
    K, V = zip(*[W.logical_kv(seed + 17 * r, geom, c) for r, c in enumerate(ctx)])
    return geom, rig, table, list(K), list(V), ctx


def _prefill(geom, rig, table, ctx, new, q):
    q_start = np.concatenate([[0], np.cumsum(new)]).astype(np.int32)
    dev = rig.dev
    out = torch.full(q.shape, 7.0, device=dev)
    with torch.cuda.stream(rig.compute):
        rig.lamps.prefill_attn(0, len(ctx), int(q_start[-1]), n2t(q, dev), torch.as_tensor(q_start, device=dev),
                               torch.as_tensor(table, device=dev), torch.as_tensor(np.asarray(ctx, dtype=np.int32), device=dev),
                               out, max_new_tokens=max(new))
    rig.compute.synchronize()
    return q_start, to_f64(out)


@pytest.mark.parametrize("H,Hkv,D,bs", [(8, 8, 64, 16), (8, 2, 32, 16), (6, 2, 128, 32), (16, 2, 64, 16), (32, 2, 128, 16),
                                        (5, 1, 64, 16), (3, 3, 32, 64), (2, 2, 128, 16)])
def test_prefill_and_decode(H, Hkv, D, bs):
    geom, rig, table, K, V, ctx = _rig(H, Hkv, D, bs, REQS, 40 + H + D)
    rig.page_requests(0, table, K, V)
    new = [n for _, n in REQS]
    q = W.queries(3, geom, sum(new))
    q_start, got = _prefill(geom, rig, table, ctx, new, q)
    assert np.abs(got - oracle.prefill_attn(q, K, V, q_start, ctx, threads=8)).max() <= tol(geom)
    q = W.queries(4, geom, len(ctx))
    out = rig.decode(0, q, table, ctx, [1] * len(ctx))
    assert np.abs(to_f64(out) - oracle.decode_attn(q, K, V, ctx, [1] * len(ctx))).max() <= tol(geom)
    rig.close()


def test_values_past_a_token_do_not_reach_it():
    """An infinite value of a later new token is no part of an earlier token's sum (0 * inf)."""
    reqs = [(40, 30), (90, 7)]
    geom, rig, table, K, V, ctx = _rig(4, 2, 64, 16, reqs, 9)
    V[0][25, 1, 3] = np.inf
    V[1][87, 0, 60] = np.nan
    rig.page_requests(0, table, K, V)
    q = W.queries(5, geom, 37)
    q_start, got = _prefill(geom, rig, table, ctx, [30, 7], q)
    ref = oracle.prefill_attn(q, K, V, q_start, ctx, threads=8)
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.isnan(ref).sum() == 2 * 3 and np.isinf(ref).sum() == 2 * 15
    fine = np.isfinite(ref)
    assert np.array_equal(got[~fine & ~np.isnan(ref)], ref[~fine & ~np.isnan(ref)])
    assert np.abs(got[fine] - ref[fine]).max() <= tol(geom)
    rig.close()


@pytest.mark.parametrize("H,Hkv,D", [(8, 8, 64), (8, 2, 32), (8, 2, 128)])
def test_a_chunk_is_summed_in_short_chains(H, Hkv, D):
    """Sixteen tokens of weight one (the queries are zero) whose values are one 1 and fifteen 2^-24:
    a chain that holds the 1 drops each 2^-24 it meets after it (half an ulp, ties to even).  Two
    chains of eight lose at most 7 of them, their sum and the division one each; a chain of sixteen
    loses up to 15 by itself.  Dim d has its 1 at token d % 16, so every place in a chain is met."""
    geom, rig, table, K, V, ctx = _rig(H, Hkv, D, 16, [(16, 16)], 5)
    V[0][:] = 2.0 ** -24
    for d in range(D):
        V[0][d % 16, :, d] = 1.0
    rig.page_requests(0, table, K, V)
    q = np.zeros((16, H, D), dtype=np.float32)
    _, got = _prefill(geom, rig, table, ctx, [16], q)
    want = (1 + 15 * 2.0 ** -24) / 16
    assert np.abs(got[15] - want).max() * 16 <= 9 * 2.0 ** -24
    rig.close()
