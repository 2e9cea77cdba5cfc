"""AllGather + GEMM where several workgroups share a tile along K and the gather is split over the launch by index: edges of
the 128x128 tile, K tails inside the last part, the smallest and largest number of parts, rows per channel without a
divisor to cut them by, and a gather whose notifications never arrive."""
import numpy as np
import pytest
import torch

import paper_2503_20313_amd as tl
import tl_workloads as wl
from oracle import ops
from tests.gpu_util import assert_close_bf16, dev, down, make_ctx, poison, up
from tests.test_gpu_ag_gemm import run_ag_gemm
from tests.test_gpu_ag_gemm_act import run_gated

pytestmark = pytest.mark.gpu
MODES = {"waves": tl.TL_COMM_WAVES, "side": tl.TL_COMM_SIDE_KERNEL, "none": tl.TL_COMM_NONE}


def shared(M, N, K, **kw):
    """Whether the call's workspace holds slots for tiles that are shared along K."""
    ctx = make_ctx(**kw)
    ws, _ = tl.tl_query_workspace(ctx, tl.TL_OP_AG_GEMM, [M, N, K])
    tl.tl_ctx_destroy(ctx)
    return ws > 256


@pytest.mark.parametrize("mode", ["waves", "side"])
@pytest.mark.parametrize("M,N,K,R,C", [(2, 8, 2048, 2, 1),            # one ragged tile, two parts
                                       (256, 264, 2056, 2, 2),        # two parts, the second with a K tail of 8
                                       (130, 392, 8200, 2, 1),        # seven parts, K tail, 65 rows per rank
                                       (130, 392, 16392, 2, 1),       # eight, the most
                                       (1024, 1152, 3144, 8, 4)])     # 72 tiles: three parts of a K that three does not divide
def test_shared_tiles(M, N, K, R, C, mode):
    w = wl.ag_gemm_inputs(M, N, K, R, config_id=161)
    assert shared(M, N, K, world_size=R, rank=1, channels_per_rank=C, comm_mode=MODES[mode])
    hs, g, c, flags, info = run_ag_gemm(w, 1, C, MODES[mode], epochs=3, tile_order=tl.TL_ORDER_OWN_FIRST)
    a_ref, _, c_ref = ops.ag_gemm(hs, w["b"])
    assert np.array_equal(g, a_ref)
    assert_close_bf16(c, c_ref, f"shared tiles {M}x{N}x{K} {mode}")
    assert flags.tolist() == [3 * info["expected_per_channel"]] * (R * C)


def test_shared_tiles_exact_small_integers():
    """Integer-valued inputs: every partial sum is exact in fp32, so the result must match bit for bit."""
    from oracle.bf16 import round_to_bf16
    rng = np.random.default_rng(6)
    R, M, N, K = 2, 256, 256, 4096
    shards = [round_to_bf16(rng.integers(-3, 4, size=(M // R, K)).astype(np.float64)) for _ in range(R)]
    w = dict(a_shards=shards, b=round_to_bf16(rng.integers(-2, 3, size=(K, N)).astype(np.float64)), M=M, N=N, K=K, world=R)
    assert shared(M, N, K, world_size=R)
    _, _, c, _, _ = run_ag_gemm(w, 1, 1, tl.TL_COMM_WAVES)
    _, _, c_ref = ops.ag_gemm(shards, w["b"])
    assert np.array_equal(c, c_ref)


@pytest.mark.parametrize("mode", ["waves", "none"])
def test_shared_tiles_do_not_depend_on_who_comes_last(mode):
    """Seven parts of N(0, 1) sums, whose fp32 rounding shows the order they are added in: the same call again and again gives
    the same bits, whichever workgroup comes last."""
    M, N, K, R = 512, 512, 8192, 2
    w = wl.ag_gemm_inputs(M, N, K, R, config_id=166)
    ctx = make_ctx(world_size=R, rank=1, comm_mode=MODES[mode])
    ws_bytes, n_flags = tl.tl_query_workspace(ctx, tl.TL_OP_AG_GEMM, [M, N, K])
    assert ws_bytes >= 256 + 16 * 7 * 128 * 128 * 4
    shards = [up(s) for s in w["a_shards"]]
    gathered, b = up(np.concatenate(w["a_shards"])), up(w["b"])
    flags, wsp = torch.zeros(n_flags, dtype=torch.int32, device=dev()), torch.zeros(ws_bytes // 4, dtype=torch.int32, device=dev())
    first = None
    for epoch in range(1, 31):
        c = poison((M, N))
        torch.cuda.synchronize()
        tl.tl_ag_gemm(ctx, shards, gathered, b, c, M, N, K, flags, epoch, wsp, ws_bytes)
        torch.cuda.synchronize()
        tl.tl_check_status(ctx, wsp)
        if first is None:
            first = c
            assert_close_bf16(down(c), ops.ag_gemm(w["a_shards"], w["b"])[2], "seven parts")
        assert torch.equal(c, first), epoch
    tl.tl_ctx_destroy(ctx)


@pytest.mark.parametrize("act", ["silu", "gelu"])
def test_shared_gated_tiles(act):
    w = wl.ag_gemm_gated_inputs(320, 96, 2312, 5, config_id=162)          # 2F = 192: a ragged column tile; K tail
    g, y, flags, info = run_gated(w, 1, 2, tl.TL_COMM_SIDE_KERNEL, act, epochs=2)
    a_ref, _, y_ref = ops.ag_gemm_act_mul(w["a_shards"], w["w_gate"], w["w_up"], act)
    assert_close_bf16(y, y_ref, f"shared gated {act}")


@pytest.mark.parametrize("mode", ["waves", "side"])
@pytest.mark.parametrize("M,K,R,C,kc", [(7 * 67, 1000, 7, 1, 0),        # 67 rows per channel: prime; rows of 2000 bytes
                                        (4 * 2 * 67, 8192, 4, 2, 0),    # ... cut along the columns
                                        (4096, 2048, 4, 2, 4)])         # four K chunks: the first by everybody, the rest in front
def test_gather_by_shares(M, K, R, C, kc, mode):
    w = wl.ag_gemm_inputs(M, 456, K, R, config_id=163)
    tile = dict(tile_m=256, tile_n=256, ag_k_chunks=kc) if kc else {}
    hs, g, c, flags, info = run_ag_gemm(w, 2, C, MODES[mode], epochs=2, tile_order=tl.TL_ORDER_OWN_FIRST, **tile)
    a_ref, _, c_ref = ops.ag_gemm(hs, w["b"])
    assert np.array_equal(g, a_ref)
    assert_close_bf16(c, c_ref, f"gather by shares {M}x{K} {mode}")
    assert flags.tolist() == [2 * info["expected_per_channel"]] * (R * C * info["k_chunks"])


def test_a_share_that_never_arrives_is_fetched_by_who_needs_it():
    """Flags that start far below zero never reach their target, as if no other workgroup of the launch had run yet: every
    workgroup copies the rows it needs itself after its patience, and the call completes."""
    M, N, K, R = 512, 264, 1024, 4
    w = wl.ag_gemm_inputs(M, N, K, R, config_id=164)
    ctx = make_ctx(world_size=R, rank=1, channels_per_rank=2, comm_mode=tl.TL_COMM_SIDE_KERNEL)
    ws_bytes, n_flags = tl.tl_query_workspace(ctx, tl.TL_OP_AG_GEMM, [M, N, K])
    shards = [up(s) for s in w["a_shards"]]
    gathered, b, c = poison((M, K)), up(w["b"]), poison((M, N))
    flags = torch.full((n_flags,), -(1 << 20), dtype=torch.int32, device=dev())
    wsp = torch.zeros(ws_bytes // 4, dtype=torch.int32, device=dev())
    torch.cuda.synchronize()
    tl.tl_ag_gemm(ctx, shards, gathered, b, c, M, N, K, flags, 1, wsp, ws_bytes)
    torch.cuda.synchronize()
    tl.tl_check_status(ctx, wsp)
    tl.tl_ctx_destroy(ctx)
    a_ref, _, c_ref = ops.ag_gemm(w["a_shards"], w["b"])
    assert np.array_equal(down(gathered), a_ref)
    assert_close_bf16(down(c), c_ref, "self-served gather")


def test_a_long_gather_by_shares_is_not_done_twice():
    """1 GiB in one round of workgroups, several times the patience a small gather gets: no slower than twice the same call
    with the producers' queue (if all workgroups lose patience together, it takes more than five times as long)."""
    M, N, K, R = 65536, 256, 8192, 8
    g = torch.Generator(device=dev())
    g.manual_seed(165)
    shards = [torch.randn(M // R, K, generator=g, device=dev(), dtype=torch.bfloat16) for _ in range(R)]
    b = torch.randn(K, N, generator=g, device=dev(), dtype=torch.bfloat16) * 0.02
    ref = torch.cat([s.float() @ b.float() for s in shards])
    best = {}
    for wg in (0, 64):
        ctx = make_ctx(world_size=R, rank=3, comm_mode=tl.TL_COMM_SIDE_KERNEL, comm_workgroups=wg)
        ws_bytes, n_flags = tl.tl_query_workspace(ctx, tl.TL_OP_AG_GEMM, [M, N, K])
        gathered, c = torch.zeros(M, K, device=dev(), dtype=torch.bfloat16), torch.zeros(M, N, device=dev(), dtype=torch.bfloat16)
        flags, wsp = torch.zeros(n_flags, dtype=torch.int32, device=dev()), torch.zeros(ws_bytes // 4, dtype=torch.int32, device=dev())
        comm = torch.cuda.Stream()
        times = []
        for epoch in range(1, 5):
            torch.cuda.synchronize()
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            tl.tl_ag_gemm(ctx, shards, gathered, b, c, M, N, K, flags, epoch, wsp, ws_bytes, torch.cuda.current_stream(), comm)
            torch.cuda.current_stream().wait_stream(comm)
            e1.record()
            torch.cuda.synchronize()
            tl.tl_check_status(ctx, wsp)
            times.append(e0.elapsed_time(e1))
        best[wg] = min(times)
        assert all(torch.equal(gathered[q * (M // R):(q + 1) * (M // R)], shards[q]) for q in range(R))
        assert float((c.float() - ref).norm() / ref.norm()) < 5e-3
        tl.tl_ctx_destroy(ctx)
    assert best[0] < 2 * best[64], best
