"""Split prefill launches with tiles of 128 columns, which load two stages of 32 positions at a time: contexts
around a group and a run, cut and uncut requests in one call, both layouts, the checks of the 64-column
ones (against the fp64 oracle, workspace full of NaN, replayed from a HIP graph, bit for bit the same)."""
import pytest

from test_gpu_prefill_split import test_split_contexts as check

pytestmark = pytest.mark.gpu

#        H  Hkv D    bs  (context, new tokens) per request
CASES = [
    (8, 2, 64, 16, [(3000, 260), (700, 33), (64, 64)]),
    (8, 2, 128, 16, [(1537, 270), (1536, 1), (1535, 2), (1569, 31)]),
    (2, 2, 64, 32, [(2900, 1030)]),                                  # plain layout
    (2, 2, 128, 16, [(2600, 1025), (900, 3)]),
    (4, 1, 256, 16, [(2000, 300), (1400, 20)]),                      # one stage at a time
    (20, 1, 128, 16, [(1700, 13), (1025, 6)]),                       # 20 heads per kv head
]


@pytest.mark.parametrize("H,Hkv,D,bs,reqs", CASES)
def test_wide_tiles(H, Hkv, D, bs, reqs):
    check(H, Hkv, D, bs, reqs)
