"""AllGather + GEMM tiles that several workgroups share along K, where calls repeat or follow one another on one workspace
in other ways than a growing epoch of one call: no part of the result may depend on what an earlier call left there."""
import numpy as np
import pytest
import torch

import paper_2503_20313_amd as tl
import tl_workloads as wl
from oracle import ops
from tests.gpu_util import assert_close_bf16, dev, down, make_ctx, poison, up
from tests.test_gpu_ag_gemm import check, run_ag_gemm

pytestmark = pytest.mark.gpu


class Call:
    """Buffers of one AllGather + GEMM shape; the workspace may be another call's."""

    def __init__(self, M, N, K, R, config_id, gathered=False):
        self.dims, self.R = (M, N, K), R
        self.w = wl.ag_gemm_inputs(M, N, K, R, config_id=config_id)
        self.shards = [up(s) for s in self.w["a_shards"]]
        self.gathered = up(np.concatenate(self.w["a_shards"])) if gathered else poison((M, K))
        self.b, self.c = up(self.w["b"]), poison((M, N))
        self.ref = ops.ag_gemm(self.w["a_shards"], self.w["b"])[2]

    def run(self, ctx, flags, epoch, ws, ws_bytes):
        self.c.copy_(poison(self.c.shape))
        torch.cuda.synchronize()
        tl.tl_ag_gemm(ctx, self.shards, self.gathered, self.b, self.c, *self.dims, flags, epoch, ws, ws_bytes)
        torch.cuda.synchronize()

    def check(self, what):
        assert_close_bf16(down(self.c), self.ref, what)


def scratch(ctx, *calls):
    """A zeroed workspace for the largest of the calls, and flags."""
    q = [tl.tl_query_workspace(ctx, tl.TL_OP_AG_GEMM, list(c.dims)) for c in calls]
    assert all(b > 256 for b, _ in q), "these calls are meant to share tiles along K"
    ws_bytes, n_flags = max(b for b, _ in q), max(f for _, f in q)
    return torch.zeros(ws_bytes // 4, dtype=torch.int32, device=dev()), ws_bytes, torch.zeros(n_flags, dtype=torch.int32, device=dev())


@pytest.mark.parametrize("epochs", [(1, 1, 1), (7, 7, 3)])
def test_without_communication_the_epoch_has_no_meaning(epochs):
    ctx = make_ctx(world_size=2, rank=0, comm_mode=tl.TL_COMM_NONE)
    call = Call(256, 264, 4096, 2, 171, gathered=True)
    ws, ws_bytes, flags = scratch(ctx, call)
    for i, epoch in enumerate(epochs):
        call.run(ctx, flags, epoch, ws, ws_bytes)
        call.check(f"call {i}, epoch {epoch}")
    tl.tl_ctx_destroy(ctx)


def test_two_shapes_on_one_workspace():
    """72 tiles and 2 tiles in turn: the counters of the one are not where the partial sums of the other go."""
    ctx = make_ctx(world_size=2, rank=0, comm_mode=tl.TL_COMM_NONE)
    calls = [Call(1024, 1152, 3072, 2, 172, gathered=True), Call(128, 200, 8192, 2, 173, gathered=True)]
    ws, ws_bytes, flags = scratch(ctx, *calls)
    for i in range(4):
        calls[i % 2].run(ctx, flags, i + 1, ws, ws_bytes)
        calls[i % 2].check(f"call {i}")
    tl.tl_ctx_destroy(ctx)


def test_retry_after_a_withheld_flag():
    ctx = make_ctx(world_size=2, rank=0, comm_mode=tl.TL_COMM_EXTERNAL, spin_timeout_us=20_000)
    call = Call(256, 128, 4096, 2, 174, gathered=True)
    ws, ws_bytes, flags = scratch(ctx, call)
    expected = tl.tl_resolve(ctx, tl.TL_OP_AG_GEMM, list(call.dims))["expected_per_channel"]
    flags[0] = expected
    call.run(ctx, flags, 1, ws, ws_bytes)
    with pytest.raises(tl.TileLinkError) as e:
        tl.tl_check_status(ctx, ws)
    assert e.value.status == tl.TL_ERR_TIMEOUT
    flags[1] = expected
    call.run(ctx, flags, 1, ws, ws_bytes)      # the same call again, now complete
    tl.tl_check_status(ctx, ws)
    call.check("retry")
    tl.tl_ctx_destroy(ctx)


def test_communication_alone_between_two_calls():
    cfg = dict(world_size=2, rank=1, comm_mode=tl.TL_COMM_SIDE_KERNEL)
    ctx, alone = make_ctx(**cfg), make_ctx(comm_alone=1, **cfg)
    call = Call(256, 264, 4096, 2, 175)
    ws, ws_bytes, flags = scratch(ctx, call)
    for epoch, c in ((1, ctx), (2, alone), (3, ctx)):
        call.run(c, flags, epoch, ws, ws_bytes)
        tl.tl_check_status(c, ws)
        if c is ctx:
            call.check(f"epoch {epoch}")
    for c in (ctx, alone):
        tl.tl_ctx_destroy(c)


def test_shared_tiles_behind_the_copy_engine():
    w = wl.ag_gemm_inputs(256, 264, 4104, 2, config_id=176)
    hs, g, c, flags, info = run_ag_gemm(w, 1, 2, tl.TL_COMM_COPY_ENGINE, epochs=3)
    check(w, hs, g, c, "copy engine")


@pytest.mark.parametrize("offset", [0, 32, 96])
def test_partial_sums_start_on_a_cache_line(offset):
    """A workspace that starts in the middle of a cache line: no line may hold partial sums of two tiles, and what the
    query asked for is enough.  Words in front of the partial sums are zero after the call, so the first one that is not
    tells where they start."""
    ctx = make_ctx(world_size=2, rank=0, comm_mode=tl.TL_COMM_NONE)
    call = Call(256, 264, 4096, 2, 177, gathered=True)
    ws_bytes, n_flags = tl.tl_query_workspace(ctx, tl.TL_OP_AG_GEMM, list(call.dims))
    guard = 64
    buf = torch.zeros(offset // 4 + ws_bytes // 4 + guard, dtype=torch.int32, device=dev())
    assert buf.data_ptr() % 128 == 0
    ws, flags = buf[offset // 4:], torch.zeros(n_flags, dtype=torch.int32, device=dev())
    for epoch in (1, 2):
        call.run(ctx, flags, epoch, ws, ws_bytes)
        call.check(f"workspace at {offset}, epoch {epoch}")
    words = buf.cpu().numpy()
    first = int(np.flatnonzero(words[(offset + 256) // 4:])[0]) + (offset + 256) // 4
    assert first * 4 % 128 < 16, first * 4            # (the first of N(0, 1) sums may itself be a zero)
    assert not words[(offset + ws_bytes) // 4:].any()
    tl.tl_ctx_destroy(ctx)


@pytest.mark.parametrize("mode", [tl.TL_COMM_WAVES, tl.TL_COMM_SIDE_KERNEL])
@pytest.mark.parametrize("M,N,K", [(1024, 1024, 2048), (2048, 2048, 512)])     # shared tiles / whole tiles that fill the chip
def test_communication_alone_gathers(mode, M, N, K):
    ctx = make_ctx(world_size=8, rank=3, channels_per_rank=2, comm_mode=mode, comm_alone=1)
    call = Call(M, N, K, 8, 178)
    ws_bytes, n_flags = tl.tl_query_workspace(ctx, tl.TL_OP_AG_GEMM, [M, N, K])
    expected = tl.tl_resolve(ctx, tl.TL_OP_AG_GEMM, [M, N, K])["expected_per_channel"]
    ws, flags = torch.zeros(ws_bytes // 4, dtype=torch.int32, device=dev()), torch.zeros(n_flags, dtype=torch.int32, device=dev())
    for epoch in (1, 2):
        call.gathered.copy_(poison((M, K)))
        call.run(ctx, flags, epoch, ws, ws_bytes)
        tl.tl_check_status(ctx, ws)
        assert np.array_equal(down(call.gathered), np.concatenate(call.w["a_shards"]))
        assert flags.tolist() == [epoch * expected] * 16
    tl.tl_ctx_destroy(ctx)


@pytest.mark.parametrize("mode", [tl.TL_COMM_WAVES, tl.TL_COMM_SIDE_KERNEL])
def test_gather_by_shares_and_by_the_queue_in_turn(mode):
    """Contexts of one shape on one workspace with a growing epoch: whoever comes next finds the queue where it expects it."""
    M, N, K, R = 512, 264, 1024, 4
    cfg = dict(world_size=R, rank=1, channels_per_rank=2, comm_mode=mode, spin_timeout_us=100_000)
    ctxs = dict(shares=make_ctx(**cfg), queue=make_ctx(comm_workgroups=8, **cfg), alone=make_ctx(comm_alone=1, **cfg))
    geometry = [tl.tl_resolve(c, tl.TL_OP_AG_GEMM, [M, N, K]) for c in ctxs.values()]
    assert len({(g["comm_tile_m"], g["comm_tile_n"], g["expected_per_channel"]) for g in geometry}) == 1
    call = Call(M, N, K, R, 179)
    ws_bytes, n_flags = tl.tl_query_workspace(ctxs["shares"], tl.TL_OP_AG_GEMM, [M, N, K])
    ws, flags = torch.zeros(ws_bytes // 4, dtype=torch.int32, device=dev()), torch.zeros(n_flags, dtype=torch.int32, device=dev())
    for epoch, name in enumerate(["shares", "queue", "shares", "alone", "queue", "shares"], 1):
        shards = [wl.normal_bf16((M // R, K), 1.0, 180, epoch, q) for q in range(R)]
        for q in range(R):
            call.shards[q].copy_(up(shards[q]))
        call.ref = ops.ag_gemm(shards, call.w["b"])[2]
        call.run(ctxs[name], flags, epoch, ws, ws_bytes)
        tl.tl_check_status(ctxs[name], ws)
        assert np.array_equal(down(call.gathered), np.concatenate(shards)), (epoch, name)
        if name != "alone":
            call.check(f"epoch {epoch}, {name}")
        assert flags.tolist() == [epoch * geometry[0]["expected_per_channel"]] * (R * 2)
        assert int(ws[1]) == epoch * geometry[0]["n_comm_tiles"]
    for c in ctxs.values():
        tl.tl_ctx_destroy(c)
