"""How a decode launch divides its work: one request per lane up to 64 of them, four per lane up to 256, by workgroups above;
pieces of one range each while there are enough shares, equal shares that straddle ranges otherwise, by waves and by
workgroups.  Batches on both sides of each line, with empty, paused and long requests among them, against the fp64 oracle.
Table rows are longer than the pool, so that no launch goes by what a row could hold (whole ranges, parts): those have tests of their own."""
import numpy as np
import pytest
import torch

import lamps_workloads as W
import oracle
from rig import Rig, to_f64, tol

pytestmark = pytest.mark.gpu


def _check(H, Hkv, D, dtype, ctx, running, shift=0):
    blocks = [(c + 15) // 16 for c in ctx]
    geom = W.Geometry(1, H, Hkv, D, 16, sum(blocks) + 4, sum(blocks) + 5, dtype)
    rig = Rig(geom, len(ctx))
    table, _ = W.deal_block_table(W.permutation(6, geom.num_blocks), ctx, geom)
    K, V = zip(*[W.logical_kv(20 + 17 * r, geom, c) for r, c in enumerate(ctx)])
    rig.page_requests(0, table, K, V)
    q = W.queries(9, geom, len(ctx))
    room = torch.full((len(ctx) * H * D + shift,), 7.0, dtype=rig.tdtype, device=rig.dev)
    out = room[shift:].view(len(ctx), H, D)
    got = to_f64(rig.decode(0, q, table, ctx, running, out=out))
    on = np.asarray(running, dtype=bool)
    assert (got[~on] == 7.0).all() and (room[:shift] == 7.0).all()
    if on.any():
        assert np.abs(got[on] - oracle.decode_attn(q, K, V, ctx, running)[on]).max() <= tol(geom)
    rig.close()


@pytest.mark.parametrize("H,Hkv,D,dtype", [(8, 2, 64, "bf16"), (2, 2, 128, "bf16"), (4, 2, 32, "f32")])
@pytest.mark.parametrize("B", [1, 5, 63, 64, 65, 200, 255, 256, 257, 300])
def test_batches(H, Hkv, D, dtype, B):
    rng = np.random.RandomState(B)
    ctx = [int(x) for x in np.exp(rng.uniform(0, np.log(400), B))]
    ctx[B // 2] = 0
    if B > 3:
        ctx[B - 2] = 3000
    _check(H, Hkv, D, dtype, ctx, [1] * B)
    _check(H, Hkv, D, dtype, ctx, [int(r % 7 != 3 and r < B - 1) if B > 1 else 0 for r in range(B)])


@pytest.mark.parametrize("n", [1, 2, 3, 5, 8, 13, 20, 33])
def test_sizes_of_pieces(n):
    """Equal ranges of n chunks and a few more: even cuts that pieces fit, that they fit with a chunk more, and that they don't."""
    for B, Hkv in ((40, 8), (64, 13), (90, 16)):
        ctx = [16 * n - (r % 5) * (r % 3) for r in range(B)]
        _check(2 * Hkv, Hkv, 64, "bf16", ctx, [int(r != 4) for r in range(B)])
    _check(24, 24, 64, "bf16", [16 * n - r % 7 for r in range(45)], [1] * 45)


@pytest.mark.parametrize("H,Hkv,D,dtype", [(8, 2, 64, "bf16"), (4, 4, 64, "bf16"), (4, 2, 64, "f32")])
@pytest.mark.parametrize("B", [3, 150])
def test_out_at_any_element(H, Hkv, D, dtype, B):
    _check(H, Hkv, D, dtype, [5 + 3 * r for r in range(B)], [1] * B, shift=1)


@pytest.mark.parametrize("n", [31, 34])
def test_by_waves_in_whole_chunks(n):
    """Shares of up to four chunks of 32 tokens, which are pieces, and of more, which straddle."""
    _check(24, 24, 64, "bf16", [16 * n - r % 7 for r in range(64)], [1] * 64)
