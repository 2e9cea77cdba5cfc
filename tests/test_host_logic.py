"""Host-side logic of the library without a GPU: a context made by tl_ctx_create_host answers the geometry queries and
the schedule dump (paper: "Tile-Centric Mapping"), which are compared with the mapping oracle here as the GPU tests do
on the device context; shapes the mapping cannot serve are refused before anything could be enqueued."""
import random
import time

import pytest

import paper_2503_20313_amd as tl
from oracle import mapping as omap

CUS = 256


def host_ctx(**kw):
    base = dict(world_size=1, rank=0, channels_per_rank=1, comm_mode=tl.TL_COMM_WAVES, tile_order=tl.TL_ORDER_RING, xcd_swizzle=1)
    base.update(kw)
    return tl.tl_ctx_create_host(CUS, **base)


def test_more_than_64_channels_are_refused():
    """The consumer's wait set is a 64-bit mask over the global channel index: R*C = 128 must not get through."""
    ctx = host_ctx(world_size=8, channels_per_rank=16)
    with pytest.raises(tl.TileLinkError) as e:
        tl.tl_query_workspace(ctx, tl.TL_OP_AG_GEMM, [8192, 512, 512])
    assert e.value.status == tl.TL_ERR_UNSUPPORTED_SHAPE and "64" in str(e.value)
    tl.tl_ctx_destroy(ctx)
    ctx = host_ctx(world_size=8, channels_per_rank=8)      # exactly 64: fine
    assert tl.tl_query_workspace(ctx, tl.TL_OP_AG_GEMM, [8192, 512, 512]) == (256, 64)
    tl.tl_ctx_destroy(ctx)


def test_k_rules():
    ctx = host_ctx(world_size=4)
    for K in (1376, 3696, 8, 4104):                        # multiples of 8: accepted, a short last K step is zero-filled
        tl.tl_query_workspace(ctx, tl.TL_OP_AG_GEMM, [1024, 512, K])
        tl.tl_query_workspace(ctx, tl.TL_OP_GEMM_RS, [1024, 512, K])
    for K in (100, 3697, 4):
        with pytest.raises(tl.TileLinkError) as e:
            tl.tl_query_workspace(ctx, tl.TL_OP_GEMM_RS, [1024, 512, K])
        assert e.value.status == tl.TL_ERR_UNSUPPORTED_SHAPE
    tl.tl_ctx_destroy(ctx)


def test_host_context_cannot_launch():
    ctx = host_ctx(world_size=2)
    with pytest.raises(tl.TileLinkError) as e:
        tl.tl_ag_gemm(ctx, [0, 0], 0, 0, 0, 256, 512, 512, 0, 1, 0, 256)
    assert e.value.status == tl.TL_ERR_INVALID_ARG and "tl_ctx_create_host" in str(e.value)
    with pytest.raises(tl.TileLinkError):
        tl.tl_check_status(ctx, 0)
    tl.tl_ctx_destroy(ctx)
    with pytest.raises(tl.TileLinkError):
        tl.tl_ctx_create_host(0, world_size=2, rank=0, channels_per_rank=1)
    with pytest.raises(tl.TileLinkError):
        tl.tl_ctx_create_host(256, world_size=2, rank=2, channels_per_rank=1)


@pytest.mark.parametrize("rank,order,swz,gm", [(0, tl.TL_ORDER_RING, 1, 0), (5, tl.TL_ORDER_RING, 1, 8), (3, tl.TL_ORDER_NATURAL, 0, 1), (2, tl.TL_ORDER_RING, 0, 3)])
def test_ag_gemm_schedule_dump_matches_mapping_oracle(rank, order, swz, gm):
    M, N, K, R, C = 8192, 3584, 8192, 8, 4
    ctx = host_ctx(world_size=R, rank=rank, channels_per_rank=C, tile_order=order, xcd_swizzle=swz, group_m=gm)
    info = tl.tl_resolve(ctx, tl.TL_OP_AG_GEMM, [M, N, K])
    assert info["compute_workgroups"] == CUS
    got = tl.tl_dump_schedule(ctx, tl.TL_OP_AG_GEMM, [M, N, K])
    want = omap.ag_gemm_schedule_records(M, N, K, R, C, rank, info["tile_m"], info["tile_n"], info["compute_workgroups"],
                                         rotate=(order == tl.TL_ORDER_RING), swizzle=bool(swz), group_m=info["group_m"])
    assert got == [v for rec in want for v in rec]
    assert info["expected_per_channel"] == omap.channel_expected(M, K, R, C, info["comm_tile_m"], info["comm_tile_n"])
    tl.tl_ctx_destroy(ctx)


@pytest.mark.parametrize("rank,gm", [(5, 0), (0, 1)])
def test_arrival_order_schedule_matches_mapping_oracle(rank, gm):
    M, N, K, R, C = 8192, 3584, 8192, 8, 4
    ctx = host_ctx(world_size=R, rank=rank, channels_per_rank=C, tile_order=tl.TL_ORDER_ARRIVAL, group_m=gm)
    info = tl.tl_resolve(ctx, tl.TL_OP_AG_GEMM, [M, N, K])
    got = tl.tl_dump_schedule(ctx, tl.TL_OP_AG_GEMM, [M, N, K])
    want = omap.ag_gemm_schedule_records(M, N, K, R, C, rank, info["tile_m"], info["tile_n"], info["compute_workgroups"],
                                         rotate=True, swizzle=True, group_m=info["group_m"], arrival=True)
    assert got == [v for rec in want for v in rec]
    tl.tl_ctx_destroy(ctx)


@pytest.mark.parametrize("rank,order,swz", [(0, tl.TL_ORDER_RING, 1), (3, tl.TL_ORDER_NATURAL, 0), (5, tl.TL_ORDER_OWN_FIRST, 1)])
def test_gemm_rs_schedule_dump_matches_mapping_oracle(rank, order, swz):
    M, N, K, R = 8192, 8192, 3584, 8
    ctx = host_ctx(world_size=R, rank=rank, tile_order=order, xcd_swizzle=swz, comm_tile_m=128, comm_tile_n=512)
    info = tl.tl_resolve(ctx, tl.TL_OP_GEMM_RS, [M, N, K])
    got = tl.tl_dump_schedule(ctx, tl.TL_OP_GEMM_RS, [M, N, K])
    rot, own = order != tl.TL_ORDER_NATURAL, order == tl.TL_ORDER_OWN_FIRST
    gemm = omap.gemm_rs_schedule_records(M, N, K, R, rank, info["tile_m"], info["tile_n"], 128, 512, info["compute_workgroups"], rot, bool(swz),
                                         info["group_m"], own)
    table = omap.rs_tile_table(M, N, R, rank, info["tile_m"], info["tile_n"], 128, 512)
    want = [v for rec in gemm for v in rec]
    for t in omap.rs_consumer_order(M, N, R, rank, 128, 512, rot, own):
        cm, cn, rlo, rhi, clo, chi, dest, exp = table[t]
        want += [t, cm, cn, rlo, rhi, clo, chi, dest, exp]
    assert got == want
    tl.tl_ctx_destroy(ctx)


def test_moe_and_attention_geometry_queries():
    ctx = host_ctx(world_size=8, channels_per_rank=4, comm_mode=tl.TL_COMM_SIDE_KERNEL)
    q = tl.tl_moe_query(ctx, tl.TL_OP_MOE_AG_GATHER_GEMM, 8192, 4096, 1792, 32, 2)
    assert q["n_flags"] == 32 and q["tile_n"] in (128, 256) and q["max_row_tiles"] >= 16384 // q["tile_m"]
    tl.tl_ctx_destroy(ctx)
    ctx = host_ctx(world_size=8, rank=7, comm_mode=tl.TL_COMM_SIDE_KERNEL)
    a = tl.tl_attn_query(ctx, 32768, 32, 128, True)
    assert a["n_flags"] == 16 and a["shards_gathered"] == 8 and a["attention_workgroups"] == 16 * 32
    tl.tl_ctx_destroy(ctx)


def test_schedules_match_the_mapping_oracle_on_seeded_random_shapes():
    """200 seeded draws of (shape, world, channels, rank, tile, order, swizzle, group, grid size, compute units): every
    AllGather + GEMM and GEMM + ReduceScatter schedule the library dumps is the mapping oracle's, record by record -- whole
    and partial rounds, grids that are no multiple of the eight dies, ragged last tiles, every tile order."""
    import numpy as np
    rng = np.random.Generator(np.random.Philox(20313))
    tiles = [(256, 256), (256, 224), (128, 128)]
    checked = 0
    for _ in range(200):
        R = int(rng.choice([1, 2, 4, 8]))
        C = int(rng.choice([1, 2, 4]))
        tm, tn = tiles[int(rng.integers(len(tiles)))]
        rows_per_channel = int(rng.choice([64, 128, 256, 512]))
        M = R * C * rows_per_channel
        N = int(rng.integers(1, 40)) * 64 + int(rng.choice([0, 8, 200]))
        K = int(rng.integers(1, 64)) * 64
        rank = int(rng.integers(R))
        order = int(rng.choice([tl.TL_ORDER_NATURAL, tl.TL_ORDER_RING, tl.TL_ORDER_OWN_FIRST, tl.TL_ORDER_ARRIVAL]))
        swz, gm = int(rng.integers(2)), int(rng.choice([0, 1, 2, 3, 8]))
        cus = int(rng.choice([256, 64, 40, 304]))
        G = int(rng.choice([0, 0, 24, 100]))
        ctx = tl.tl_ctx_create_host(cus, world_size=R, rank=rank, channels_per_rank=C, comm_mode=tl.TL_COMM_SIDE_KERNEL, tile_order=order,
                                    xcd_swizzle=swz, group_m=gm, tile_m=tm, tile_n=tn, compute_workgroups=G)
        try:
            info = tl.tl_resolve(ctx, tl.TL_OP_AG_GEMM, [M, N, K])
        except tl.TileLinkError:
            tl.tl_ctx_destroy(ctx)
            continue
        got = tl.tl_dump_schedule(ctx, tl.TL_OP_AG_GEMM, [M, N, K])
        want = omap.ag_gemm_schedule_records(M, N, K, R, C, rank, info["tile_m"], info["tile_n"], info["compute_workgroups"],
                                             rotate=order != tl.TL_ORDER_NATURAL, swizzle=bool(swz), group_m=info["group_m"],
                                             arrival=order == tl.TL_ORDER_ARRIVAL)
        assert got == [v for rec in want for v in rec], (M, N, K, R, C, rank, tm, tn, order, swz, gm, cus, G)
        checked += 1
        if order != tl.TL_ORDER_ARRIVAL:
            try:
                info = tl.tl_resolve(ctx, tl.TL_OP_GEMM_RS, [M, N, K])
            except tl.TileLinkError:
                tl.tl_ctx_destroy(ctx)
                continue
            got = tl.tl_dump_schedule(ctx, tl.TL_OP_GEMM_RS, [M, N, K])
            rot, own = order != tl.TL_ORDER_NATURAL, order == tl.TL_ORDER_OWN_FIRST
            Tm_r, Tn_r = info["comm_tile_m"], info["comm_tile_n"]
            gemm = omap.gemm_rs_schedule_records(M, N, K, R, rank, info["tile_m"], info["tile_n"], Tm_r, Tn_r, info["compute_workgroups"], rot,
                                                 bool(swz), info["group_m"], own)
            table = omap.rs_tile_table(M, N, R, rank, info["tile_m"], info["tile_n"], Tm_r, Tn_r)
            want = [v for rec in gemm for v in rec]
            for t in omap.rs_consumer_order(M, N, R, rank, Tm_r, Tn_r, rot, own):
                cm, cn, rlo, rhi, clo, chi, dest, exp = table[t]
                want += [t, cm, cn, rlo, rhi, clo, chi, dest, exp]
            assert got == want, ("rs", M, N, K, R, C, rank, tm, tn, order, swz, gm, cus, G)
            checked += 1
        tl.tl_ctx_destroy(ctx)
    assert checked >= 150


@pytest.mark.parametrize("mode", [tl.TL_COMM_WAVES, tl.TL_COMM_SIDE_KERNEL])
@pytest.mark.parametrize("M,N,K", [(4096, 4096, 4096), (2048, 2048, 8192), (1024, 1024, 4096), (512, 3584, 8192), (256, 512, 512)])
def test_communication_alone_has_workgroups(mode, M, N, K):
    """Also where the tiles of the GEMM, which does not run, would fill the chip."""
    ctx = host_ctx(world_size=8, comm_mode=mode, comm_alone=1)
    assert tl.tl_resolve(ctx, tl.TL_OP_AG_GEMM, [M, N, K])["comm_workgroups"] >= 8
    tl.tl_ctx_destroy(ctx)


def producer_tile_by_every_divisor(rows, ld, total, workers):
    """The producer tile the library's comment asks for, over all divisors in ascending order."""
    want = total // workers
    if want > 65536:
        want = max(want // 2, 65536)
    want = min(max(want, 16384), 262144)
    best = None
    for tm in range(1, rows + 1):
        if rows % tm:
            continue
        tn, cost = ld, 1.0
        while True:
            size = 2 * tm * tn
            c = cost * (size / want if size > want else want / size)
            if best is None or c < best[0]:
                best = (c, tm, tn)
            if tn % 16 or tn // 2 < 64:
                break
            tn, cost = tn // 2, 1.5
    return best[1:]


def test_producer_tile_is_the_best_divisor():
    rng = random.Random(19)
    shapes = [(R, C, R * C * rng.choice([1, 2, 67, 128, 360, 1024, 1260, rng.randrange(1, 3000)]), 8 * rng.choice([1, 16, 125, 512, 1024, rng.randrange(1, 1200)]))
              for R, C in rng.choices([(1, 1), (2, 1), (4, 2), (8, 4), (7, 3)], k=150)]
    for R, C, M, K in shapes:
        ctx = host_ctx(world_size=R, channels_per_rank=C)
        info = tl.tl_resolve(ctx, tl.TL_OP_AG_GEMM, [M, 512, K])
        assert (info["comm_tile_m"], info["comm_tile_n"]) == producer_tile_by_every_divisor(M // (R * C), K, 2 * M * K, CUS), (R, C, M, K)
        tl.tl_ctx_destroy(ctx)


def test_geometry_does_not_take_longer_for_more_rows():
    """Every call works its geometry out: 2^20 rows per channel, where trying every number up to that takes a thousand times
    as long as for 2^10, in the time of the square root at most (32 times; the fixed part makes it far less)."""
    ctx = host_ctx()

    def best_of(M):
        times = []
        for _ in range(30):
            t0 = time.perf_counter()
            tl.tl_resolve(ctx, tl.TL_OP_AG_GEMM, [M, 512, 512])
            times.append(time.perf_counter() - t0)
        return min(times)

    small, large = best_of(1 << 10), best_of(1 << 20)
    assert large < 32 * small, (small, large)
    tl.tl_ctx_destroy(ctx)


@pytest.mark.parametrize("op,mode,dims,kw,tile", [
    # the reduce workgroups inside the launch take twice as long with the small tile's threads (measured, 128 against 256):
    (tl.TL_OP_GEMM_RS, tl.TL_COMM_WAVES, [2048, 2048, 768], dict(rs_direct_push=1), 256),      # 76 / 57 us
    (tl.TL_OP_GEMM_RS, tl.TL_COMM_WAVES, [1024, 8192, 256], dict(rs_direct_push=1), 256),      # 124 / 74
    (tl.TL_OP_GEMM_RS, tl.TL_COMM_WAVES, [4096, 4608, 1792], dict(rs_direct_push=1), 256),     # 286 / 182
    (tl.TL_OP_GEMM_RS, tl.TL_COMM_WAVES, [512, 4608, 3584], dict(rs_direct_push=1), 128),      # 74 / 93
    (tl.TL_OP_GEMM_RS, tl.TL_COMM_WAVES, [1024, 1024, 3584], dict(rs_direct_push=1), 128),     # 54 / 78
    (tl.TL_OP_GEMM_RS, tl.TL_COMM_WAVES, [1024, 2048, 3584], dict(), 128),                     # ring: 72 / 92
    # ... and not at all as a kernel of their own
    (tl.TL_OP_GEMM_RS, tl.TL_COMM_SIDE_KERNEL, [2048, 2048, 1792], dict(rs_direct_push=1), 128),
    (tl.TL_OP_GEMM_RS, tl.TL_COMM_SIDE_KERNEL, [4096, 2048, 1792], dict(rs_direct_push=1), 128),   # 56 / 74
    # a reduce side that moves every segment: one round of small tiles only (ring)
    (tl.TL_OP_GEMM_RS, tl.TL_COMM_SIDE_KERNEL, [2048, 2048, 1792], dict(), 128),               # 61 / 69
    (tl.TL_OP_GEMM_RS, tl.TL_COMM_SIDE_KERNEL, [4096, 2048, 1792], dict(), 256),               # 86 / 74
    (tl.TL_OP_GEMM_RS, tl.TL_COMM_SIDE_KERNEL, [4096, 4608, 1792], dict(), 256),               # 202 / 137
    # the GEMM has no more compute units than it is given
    (tl.TL_OP_AG_GEMM, tl.TL_COMM_SIDE_KERNEL, [2048, 2048, 8192], dict(), 128),
    (tl.TL_OP_AG_GEMM, tl.TL_COMM_SIDE_KERNEL, [2048, 2048, 8192], dict(compute_workgroups=64), 256),
])
def test_tile_shape_counts_what_else_the_call_does(op, mode, dims, kw, tile):
    ctx = host_ctx(world_size=8, comm_mode=mode, **kw)
    assert tl.tl_resolve(ctx, op, dims)["tile_m"] == tile
    tl.tl_ctx_destroy(ctx)


@pytest.mark.parametrize("segment,N,tile,reduce_tile", [
    (256, 1536, 128, (128, 128)), (64, 1536, 128, (64, 128)), (36, 1536, 128, (36, 128)),        # whole tiles, or less than one
    (251, 1536, 128, (251, 256)), (192, 512, 128, (192, 256)), (146, 520, 128, (146, 520)),      # the large tile's under the small one
    (443, 1536, 128, (1, 128)), (974, 1536, 128, (2, 128)), (443, 1536, 256, (1, 256)),          # thin under either
    (251, 1536, 256, (251, 256)), (320, 1536, 256, (160, 256))])
def test_reduce_tile_of_ragged_segments(segment, N, tile, reduce_tile):
    ctx = host_ctx(world_size=8, comm_mode=tl.TL_COMM_SIDE_KERNEL, tile_m=tile, tile_n=tile)
    info = tl.tl_resolve(ctx, tl.TL_OP_GEMM_RS, [8 * segment, N, 608])
    assert (info["comm_tile_m"], info["comm_tile_n"]) == reduce_tile
    tl.tl_ctx_destroy(ctx)


@pytest.mark.parametrize("mode", [tl.TL_COMM_WAVES, tl.TL_COMM_SIDE_KERNEL])
@pytest.mark.parametrize("direct", [0, 1])
def test_thin_reduce_tiles_take_the_large_tile(mode, direct):
    """443 rows a segment, a prime: reduce tiles of one row, twice as many under the small tile (125 / 86 us side kernel)."""
    ctx = host_ctx(world_size=8, comm_mode=mode, rs_direct_push=direct)
    assert tl.tl_resolve(ctx, tl.TL_OP_GEMM_RS, [8 * 443, 1536, 608])["tile_m"] == 256
    tl.tl_ctx_destroy(ctx)
