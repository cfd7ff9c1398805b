"""Contexts cut into more runs than are counted one by one: five and more to a tile, more than a wave looks at in one go, beside tiles of
few runs; the same checks as for the others (workspace of NaN, replays, bit for bit the same)."""
import pytest

import test_gpu_prefill_split as split

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,Hkv,D,bs,reqs", [
    (8, 2, 128, 16, [(6000, 2), (2500, 7), (1200, 3)]),
    (2, 1, 128, 16, [(30000, 1)]),
    (2, 2, 64, 32, [(9000, 70), (3000, 130)]),
    (2, 1, 256, 16, [(5000, 9)]),
    (1, 1, 256, 16, [(5000, 33)]),
])
def test_many_runs(H, Hkv, D, bs, reqs):
    split.test_split_contexts(H, Hkv, D, bs, reqs)


@pytest.mark.parametrize("reqs", [[(5000, 57)], [(5000, 9), (700, 11)], [(1500, 16), (1400, 13), (900, 5)]])
def test_blocks_of_a_tile(reqs):
    """Tiles with one to four blocks of 16 columns: added up by halves of their dims, or whole; few runs and many."""
    split.test_split_contexts(8, 2, 128, 16, reqs)
