"""Routing tables at the edges of the routing kernels: one launch or two (1024 tokens), logits held in 8 / 16 / 32 / 64
registers, rows that fill no wave or no whole step of the sort, tile heights that are no power of two, one expert, logits
of -inf, and rows whose logits are all the same."""
import numpy as np
import pytest

import paper_2503_20313_amd as tl
import tl_workloads as wl
from tests.gpu_util import make_ctx
from tests.test_gpu_moe import check_routing, route_on_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,E,k,R,C,tile_m", [(1, 1, 1, 1, 1, 256), (6, 3, 2, 2, 3, 1), (1023, 8, 5, 1, 1, 100), (1024, 64, 8, 8, 8, 128),
                                              (1025, 9, 3, 5, 1, 129), (1040, 17, 1, 8, 2, 64), (2100, 33, 7, 4, 5, 3), (16400, 16, 2, 16, 1, 256),
                                              (513, 32, 8, 1, 3, 2)])      # 513 x 8 rows in tiles of 2: more tiles than fit in LDS, one launch
def test_route_edges(T, E, k, R, C, tile_m):
    logits = wl.normal_f32((T, E), 1.0, 171, 0)
    logits[::3, : E // 2] = logits[::3, :1]     # ties
    logits[::11] = 0.25                         # all the same
    if E > k:
        logits[5::13, E - 1] = -np.inf          # never among the chosen, as E - 1 >= k others are finite
    ctx = make_ctx(world_size=R, rank=0, channels_per_rank=C)
    for renorm in (True, False):
        got = route_on_gpu(ctx, logits, T, E, k, tile_m, -(-T * k // tile_m) + E, renorm)
        check_routing(dict(T=T, E=E, topk=k, logits=logits), R, C, tile_m, got, renorm)
    tl.tl_ctx_destroy(ctx)
