"""lamps_decode_attn about the line between cutting ranges by half-chunks and by whole ones (chunks of 32 tokens in
halves of 16, 8 heads of 64: one and a half chunks per resident wave), with lengths that end in either half of
a chunk, against the fp64 oracle; and the merge of ranges of up to eight pieces beside longer ones.  Table rows are longer than the
pool: by rows that the contexts fill, such launches are not planned."""
import numpy as np
import pytest

import lamps_workloads as W
import oracle
from rig import Rig, to_f64, tol

pytestmark = pytest.mark.gpu


def _check(geom_of, ctx, running):
    blocks = [(c + 15) // 16 for c in ctx]
    geom = geom_of(sum(blocks) + 4, sum(blocks) + 5)
    rig = Rig(geom, len(ctx))
    table, _ = W.deal_block_table(W.permutation(6, geom.num_blocks), ctx, geom)
    K, V = zip(*[W.logical_kv(20 + 17 * r, geom, c) for r, c in enumerate(ctx)])
    rig.page_requests(0, table, K, V)
    q = W.queries(9, geom, len(ctx))
    got = to_f64(rig.decode(0, q, table, ctx, running, sentinel=7.0))
    again = to_f64(rig.decode(0, q, table, ctx, running, sentinel=7.0))
    on = np.asarray(running, dtype=bool)
    assert np.abs(got[on] - oracle.decode_attn(q, K, V, ctx, running)[on]).max() <= tol(geom)
    assert (got[~on] == 7.0).all() and np.array_equal(got, again)
    rig.close()


@pytest.mark.parametrize("n", [60, 140, 144, 145, 150])
def test_cuts_on_both_sides_of_the_line(n):
    rng = np.random.RandomState(n)
    ctx = [int(x) for x in rng.randint(225, 257, n)]                  # 8 chunks each, 15 or 16 halves
    _check(lambda nb, mb: W.Geometry(1, 8, 8, 64, 16, nb, mb, "bf16"), ctx, [1] * n)
    _check(lambda nb, mb: W.Geometry(1, 8, 8, 64, 16, nb, mb, "bf16"), ctx[:n - 3] + [0, 1, 17], [int(r % 9 != 4) for r in range(n)])


@pytest.mark.parametrize("ctx", [[4000] + [30] * 40, [200] * 20 + [2500], [5000, 400, 300, 12, 900] * 3])
@pytest.mark.parametrize("dtype,H,Hkv,D", [("bf16", 8, 8, 64), ("bf16", 8, 2, 128), ("f32", 8, 4, 64), ("bf16", 32, 1, 64)])
def test_short_and_long_piece_lists(dtype, H, Hkv, D, ctx):
    _check(lambda nb, mb: W.Geometry(1, H, Hkv, D, 16, nb, mb, dtype), ctx, [1] * len(ctx))
