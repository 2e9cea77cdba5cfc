"""The calls whose time matters to a user of this library, as data: what is called, at which sizes, on which inputs.

Every case is one GPU's share of a tensor-parallel (or sequence-parallel) layer, called through the package's public entry
points the way bench.py and the tests call them: work goes to the current stream, the communication side to one side
stream that the program keeps, and the two streams are ordered against each other before and after the call.  Contexts,
flag arrays, workspaces, weights and output buffers are made once (prepare) and reused with a growing epoch (run).

Values follow tl_workloads.py: activations and attention inputs N(0, 1), weights N(0, 0.02), partial results that come
from other ranks scaled like a real partial product, gate logits N(0, 1).  bf16 everywhere, gate logits and weights fp32.
"""
import math

import torch

import paper_2503_20313_amd as tl

HEAD_DIM = 128
W_STD = 0.02
MODES = {"waves": tl.TL_COMM_WAVES, "side": tl.TL_COMM_SIDE_KERNEL}
ACTS = {"silu": tl.TL_ACT_SILU_MUL, "gelu": tl.TL_ACT_GELU_MUL}

_comm_stream = None


def _comm():
    """The program's one communication stream."""
    global _comm_stream
    if _comm_stream is None:
        _comm_stream = torch.cuda.Stream()
    return _comm_stream


# ---------------------------------------------------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------------------------------------------------
def listed():
    return [
        # The smallest configuration of the repository (two shards of [128, 512]), producers inside the fused kernel, one
        # stream: launch latency and the host path.
        dict(name="ag_gemm smallest", op="ag_gemm", M=256, N=512, K=512, R=2, rank=0, C=2, mode="waves", k_chunks=1),
        # A serving batch of 512 tokens through the first half of the MLP-5 layer: weights dominate the traffic, few tiles.
        dict(name="ag_gemm serving batch", op="ag_gemm", M=512, N=3584, K=8192, R=8, rank=3, C=1, mode="side", k_chunks=1),
        # MLP-1 prefill: a ragged N (11008 / 8) and one round of tiles, K chunks as bench.py chooses for it.
        dict(name="ag_gemm MLP-1", op="ag_gemm", M=8192, N=1376, K=4096, R=8, rank=0, C=4, mode="side", k_chunks=4),
        # MLP-5 prefill, the first half of bench.py's timed step.
        dict(name="ag_gemm MLP-5", op="ag_gemm", M=8192, N=3584, K=8192, R=8, rank=0, C=4, mode="side", k_chunks=1),
        # The same serving batch through the second half of the layer.
        dict(name="gemm_rs serving batch", op="gemm_rs", M=512, N=8192, K=3584, R=8, rank=3, mode="side"),
        # A short prompt batch whose rows divide by no tile size, with MLP-1's ragged K (a K tail).
        dict(name="gemm_rs ragged", op="gemm_rs", M=2000, N=4608, K=1376, R=8, rank=6, mode="side"),
        # The ring form at MLP-2's second half (14336 / 8).
        dict(name="gemm_ring_rs MLP-2", op="gemm_ring_rs", M=8192, N=4096, K=1792, R=8, rank=2, mode="side"),
        # The whole MLP-5 layer: gate/up GEMM with SiLUMul, then GEMM + ReduceScatter on its output.
        dict(name="mlp layer MLP-5", op="mlp_layer", M=8192, H=8192, F=3584, R=8, rank=0, C=4, mode="side", act="silu"),
        # A serving batch through a MoE layer with many small experts (MoE-3's share, top-5): routing and launches count.
        dict(name="moe layer serving batch", op="moe_layer", T=512, H=2048, F=192, E=32, topk=5, R=8, rank=5, C=1, mode="side", act="gelu"),
        # The MoE configuration of the benchmark, prefill.
        dict(name="moe layer prefill", op="moe_layer", T=8192, H=4096, F=1792, E=32, topk=2, R=8, rank=0, C=4, mode="side", act="silu"),
        # A short bidirectional sequence, query rows that fill no whole number of query blocks.
        dict(name="attention short", op="attention", S=3328, heads=16, R=4, rank=1, C=1, mode="side", causal=False),
        # The long-context configuration of the benchmark: causal, the rank with the most keys.
        dict(name="attention 32k causal", op="attention", S=32768, heads=32, R=8, rank=7, C=1, mode="side", causal=True),
    ]


def _log_int(rng, lo, hi, step=1):
    """An integer multiple of `step` in [lo, hi], spread over the logarithm."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)) * step
    return min(max(v, -(-lo // step) * step), hi // step * step)


def _world(rng):
    R = rng.choice([2, 4, 8, 8, 8])
    return R, rng.randrange(R)


def _mode(rng):
    return rng.choice(["side", "side", "side", "waves"])


def draw(rng):
    op = rng.choice(["ag_gemm", "ag_gemm", "gemm_rs", "gemm_rs", "gemm_ring_rs", "mlp_layer", "moe_layer", "moe_layer", "attention", "attention"])
    R, rank = _world(rng)
    C = rng.choice([1, 2, 4])
    if op == "ag_gemm":
        M = _log_int(rng, 128, 8192, R * C)
        N = _log_int(rng, 256, 3696, rng.choice([16, 64, 256]))
        K = _log_int(rng, 512, 8192, rng.choice([8, 64, 256]))
        chunked = K % 256 == 0 and K >= 2048 and -(-M // 256) * -(-N // 256) <= 256 and M * N > 1 << 20 and M >= 4096
        return dict(op=op, M=M, N=N, K=K, R=R, rank=rank, C=C, mode=_mode(rng), k_chunks=4 if chunked else 1)
    if op in ("gemm_rs", "gemm_ring_rs"):
        M = _log_int(rng, 128, 8192, R)
        N = _log_int(rng, 512, 8192, rng.choice([64, 256, 256]))
        K = _log_int(rng, 256, 3584, rng.choice([8, 32, 64]))
        return dict(op=op, M=M, N=N, K=K, R=R, rank=rank, mode=_mode(rng))
    if op == "mlp_layer":
        M = _log_int(rng, 128, 8192, R * C)
        H = _log_int(rng, 1024, 8192, 256)
        F = _log_int(rng, 256, 3584, 32)
        return dict(op=op, M=M, H=H, F=F, R=R, rank=rank, C=C, mode="side", act=rng.choice(["silu", "gelu"]))
    if op == "moe_layer":
        T = _log_int(rng, 128, 8192, R * C)
        H = _log_int(rng, 1024, 4096, 256)
        F = _log_int(rng, 128, 1792, 64)
        E = rng.choice([8, 16, 32])
        topk = rng.choice([1, 2, 2, 4, 5]) if T * H * F < 1 << 34 else 2
        return dict(op=op, T=T, H=H, F=F, E=E, topk=topk, R=R, rank=rank, C=C, mode="side", act=rng.choice(["silu", "gelu"]))
    S = _log_int(rng, 1024, 32768, R * C * 64)
    causal = rng.random() < 0.7
    n = S // R
    pairs = n * (rank * n + n / 2) if causal else n * S
    heads = rng.choice([h for h in (8, 12, 16, 32) if pairs * h <= 4e9])      # no more than the long-context case
    return dict(op="attention", S=S, heads=heads, R=R, rank=rank, C=C, mode=_mode(rng), causal=causal)


# ---------------------------------------------------------------------------------------------------------------------
# What a program has in hand before the call
# ---------------------------------------------------------------------------------------------------------------------
class _Draw:
    def __init__(self, seed):
        self.dev = torch.device("cuda", torch.cuda.current_device())
        self.g = torch.Generator(device=self.dev)
        self.g.manual_seed(seed)

    def normal(self, *shape, std=1.0, dtype=torch.bfloat16):
        t = torch.randn(shape, generator=self.g, device=self.dev, dtype=dtype)
        return t.mul_(std) if std != 1.0 else t

    def zeros(self, *shape, dtype=torch.bfloat16):
        return torch.zeros(shape, device=self.dev, dtype=dtype)


class _Op:
    """A context with its workspace, flags and call counter."""

    def __init__(self, d, op, dims, n_flags=None, **cfg):
        self.ctx = tl.tl_ctx_create(tile_order=tl.TL_ORDER_OWN_FIRST, xcd_swizzle=1, spin_timeout_us=10_000_000, **cfg)
        self.ws_bytes, flags = tl.tl_query_workspace(self.ctx, op, dims)
        self.flags = d.zeros(n_flags or flags, dtype=torch.int32)
        self.ws = d.zeros(self.ws_bytes // 4, dtype=torch.int32)
        self.epoch = 0

    def __del__(self):
        if getattr(self, "ctx", None) is not None:
            tl.tl_ctx_destroy(self.ctx)
            self.ctx = None

    def tail(self, cs, ms):
        self.epoch += 1
        return self.flags, self.epoch, self.ws, self.ws_bytes, cs, ms


def _gathered(d, rows, cols, R, rank):
    """R row shards of a [rows, cols] matrix; the local one lives at its place in the gathered buffer."""
    n = rows // R
    full = d.zeros(rows, cols)
    shards = [full[q * n:(q + 1) * n].copy_(d.normal(n, cols)) if q == rank else d.normal(n, cols) for q in range(R)]
    return shards, full


def _segments(d, case, rows, cols, std, ring=False):
    """What the other ranks hand to this one, and where this rank's rows of their segments land."""
    R, rank, n = case["R"], case["rank"], rows // case["R"]
    if ring:   # running sums: the one of segment q already holds (q - 1 - rank) mod R partial products
        recv = [d.normal(n, cols, std=std * math.sqrt((q - 1 - rank) % R)) if (q - 1 - rank) % R else 0 for q in range(R)]
    else:
        recv = [0 if q == rank else d.normal(n, cols, std=std) for q in range(R)]
    push = [0 if q == rank else d.zeros(n, cols) for q in range(R)]
    return recv, push


def _prepare_ag(d, case, s, N, K, gated=False):
    M = case["M"]
    s["shards"], s["gathered"] = _gathered(d, M, K, case["R"], case["rank"])
    s["b"] = d.normal(K, N, std=W_STD)                       # gated: the packed gate | up layout, drawn as it lies
    s["y"] = d.zeros(M, N // 2 if gated else N)
    s["ag"] = _Op(d, tl.TL_OP_AG_GEMM, [M, N, K], world_size=case["R"], rank=case["rank"], channels_per_rank=case["C"], comm_mode=MODES[case["mode"]],
                  ag_k_chunks=case.get("k_chunks", 1))


def _prepare_rs(d, case, s, N, K, ring=False):
    M, R, rank = case["M"], case["R"], case["rank"]
    s["w"] = d.normal(K, N, std=W_STD)
    s["partial"], s["out"] = d.zeros(M, N), d.zeros(M // R, N)
    s["recv"], s["push"] = _segments(d, case, M, N, math.sqrt(K) * W_STD, ring)
    s["rs"] = _Op(d, tl.TL_OP_GEMM_RS, [M, N, K], world_size=R, rank=rank, channels_per_rank=1, comm_mode=MODES[case["mode"]], rs_direct_push=0 if ring else 1)


def _prepare_moe(d, case, s):
    T, H, F, E, k, R, rank, C = (case[x] for x in ("T", "H", "F", "E", "topk", "R", "rank", "C"))
    s["logits"] = d.normal(T, E, dtype=torch.float32)
    s["shards"], s["gathered"] = _gathered(d, T, H, R, rank)
    s["w1"] = d.normal(E, H, 2 * F, std=W_STD)
    s["w2"] = d.normal(E, F, H, std=W_STD)
    cfg = dict(world_size=R, rank=rank, comm_mode=MODES[case["mode"]])
    s["p1"] = _Op(d, tl.TL_OP_MOE_AG_GATHER_GEMM, [T, H, 2 * F, E, k], channels_per_rank=C, **cfg)
    s["p2"] = _Op(d, tl.TL_OP_MOE_GEMM_SCATTER_RS, [T, H, F, E, k], channels_per_rank=1, rs_direct_push=1, **cfg)
    q1 = tl.tl_moe_query(s["p1"].ctx, tl.TL_OP_MOE_AG_GATHER_GEMM, T, H, 2 * F, E, k)
    q2 = tl.tl_moe_query(s["p2"].ctx, tl.TL_OP_MOE_GEMM_SCATTER_RS, T, H, F, E, k)
    # the two halves cut the sorted rows into tiles of their own height: one set of tables where the heights agree
    s["halves"] = [s["p1"], s["p2"]] if q1["tile_m"] != q2["tile_m"] else [s["p1"]]
    s["ids"], s["gate"] = d.zeros(T, k, dtype=torch.int32), d.zeros(T, k, dtype=torch.float32)
    s["offsets"], s["sorted"] = d.zeros(E + 1, dtype=torch.int32), d.zeros(T * k, dtype=torch.int32)
    for p, q in ((s["p1"], q1), (s["p2"], q2)):
        p.tile_m, p.tables, p.n_tiles = q["tile_m"], d.zeros(q["max_row_tiles"], 8, dtype=torch.int32), d.zeros(1, dtype=torch.int32)
    s["y1"], s["scatter"], s["partial"] = d.zeros(T * k, F), d.zeros(T * k, H), d.zeros(T, H)
    s["out"] = d.zeros(T // R, H)
    s["recv"], s["push"] = _segments(d, case, T, H, math.sqrt(F) * W_STD)


def _prepare_attention(d, case, s):
    S, heads, R, rank = case["S"], case["heads"], case["R"], case["rank"]
    n, ld = S // R, heads * HEAD_DIM
    s["q"], s["o"] = d.normal(n, ld), d.zeros(n, ld)
    s["k"], s["v"] = [d.normal(n, ld) for _ in range(R)], [d.normal(n, ld) for _ in range(R)]
    s["kg"], s["vg"] = d.zeros(S, ld), d.zeros(S, ld)
    s["at"] = _Op(d, tl.TL_OP_SP_AG_ATTENTION, [S, heads, HEAD_DIM], world_size=R, rank=rank, channels_per_rank=case["C"], comm_mode=MODES[case["mode"]])


def prepare(case, seed):
    d = _Draw(seed)
    s = {"case": case, "comm": _comm()}
    op = case["op"]
    if op == "ag_gemm":
        _prepare_ag(d, case, s, case["N"], case["K"])
    elif op in ("gemm_rs", "gemm_ring_rs"):
        s["a"] = d.normal(case["M"], case["K"])
        _prepare_rs(d, case, s, case["N"], case["K"], ring=op == "gemm_ring_rs")
    elif op == "mlp_layer":
        _prepare_ag(d, case, s, 2 * case["F"], case["H"], gated=True)
        _prepare_rs(d, case, s, case["H"], case["F"])
    elif op == "moe_layer":
        _prepare_moe(d, case, s)
    else:
        _prepare_attention(d, case, s)
    return s


# ---------------------------------------------------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------------------------------------------------
def _rs_outputs(s, rows):
    """The own segment's sum, the own rows of the partial product, and the rows pushed to the other ranks."""
    c = s["case"]
    n = rows // c["R"]
    return [s["out"], s["partial"][c["rank"] * n:(c["rank"] + 1) * n]] + [t for t in s["push"] if isinstance(t, torch.Tensor)]


def run(s):
    c = s["case"]
    op = c["op"]
    cs = torch.cuda.current_stream()
    ms = s["comm"]
    ms.wait_stream(cs)          # the inputs are complete, and so is the previous call
    if op == "ag_gemm":
        tl.tl_ag_gemm(s["ag"].ctx, s["shards"], s["gathered"], s["b"], s["y"], c["M"], c["N"], c["K"], *s["ag"].tail(cs, ms))
        out = [s["y"], s["gathered"]]
    elif op == "gemm_rs":
        tl.tl_gemm_rs(s["rs"].ctx, s["a"], s["w"], s["partial"], s["recv"], s["push"], s["out"], c["M"], c["N"], c["K"], *s["rs"].tail(cs, ms))
        out = _rs_outputs(s, c["M"])
    elif op == "gemm_ring_rs":
        tl.tl_gemm_ring_rs(s["rs"].ctx, s["a"], s["w"], s["partial"], s["recv"], s["push"], s["out"], c["M"], c["N"], c["K"], *s["rs"].tail(cs, ms))
        out = [s["out"], s["partial"]] + [t for t in s["push"] if isinstance(t, torch.Tensor)]
    elif op == "mlp_layer":
        tl.tl_ag_gemm_act_mul(s["ag"].ctx, s["shards"], s["gathered"], s["b"], s["y"], c["M"], c["F"], c["H"], ACTS[c["act"]], *s["ag"].tail(cs, ms))
        ms.wait_stream(cs)      # the reduce side of the second half may not run ahead into the first
        tl.tl_gemm_rs(s["rs"].ctx, s["y"], s["w"], s["partial"], s["recv"], s["push"], s["out"], c["M"], c["H"], c["F"], *s["rs"].tail(cs, ms))
        out = [s["gathered"], s["y"]] + _rs_outputs(s, c["M"])
    elif op == "moe_layer":
        T, H, F, E, k = c["T"], c["H"], c["F"], c["E"], c["topk"]
        p1, p2 = s["p1"], s["p2"]
        for p in s["halves"]:
            tl.tl_moe_route(p.ctx, s["logits"], T, E, k, True, p.tile_m, s["ids"], s["gate"], s["offsets"], s["sorted"], p.tables, p.n_tiles, cs)
        t2 = s["halves"][-1]
        tl.tl_moe_ag_gather_gemm_act_mul(p1.ctx, s["shards"], s["gathered"], s["w1"], s["sorted"], p1.tables, p1.n_tiles, s["y1"], T, H, F, E, k,
                                         ACTS[c["act"]], *p1.tail(cs, ms))
        ms.wait_stream(cs)
        tl.tl_moe_gemm_scatter_rs(p2.ctx, s["y1"], s["w2"], s["sorted"], t2.tables, t2.n_tiles, s["gate"], s["scatter"], s["partial"], s["recv"],
                                  s["push"], s["out"], T, H, F, E, k, *p2.tail(cs, ms))
        out = [s["ids"], s["gate"], s["gathered"], s["y1"]] + _rs_outputs(s, T)
    else:
        S, n = c["S"], c["S"] // c["R"]
        tl.tl_sp_ag_attention(s["at"].ctx, s["q"], s["k"], s["v"], s["kg"], s["vg"], s["o"], S, c["heads"], HEAD_DIM, c["causal"],
                              HEAD_DIM ** -0.5, *s["at"].tail(cs, ms))
        seen = (c["rank"] + 1) * n if c["causal"] else S
        out = [s["o"], s["kg"][:seen], s["vg"][:seen]]
    cs.wait_stream(ms)          # what follows on the current stream sees the communication side's results
    return out


# ---------------------------------------------------------------------------------------------------------------------
# What a pass cannot do without, and how far correct results may differ
# ---------------------------------------------------------------------------------------------------------------------
def _ag_bytes(M, N_in, N_out, K, R):
    return 2.0 * (M * K + (M - M // R) * K + K * N_in + M * N_out)


def _rs_bytes(M, N, R):
    """Peers' rows read, rows pushed, own rows of the partial product and the result written."""
    return 2.0 * (M // R) * N * (2 * (R - 1) + 2)


def work(case):
    op, R = case["op"], case["R"]
    if op == "ag_gemm":
        M, N, K = case["M"], case["N"], case["K"]
        return {"flops": 2.0 * M * N * K, "bytes": _ag_bytes(M, N, N, K, R)}
    if op in ("gemm_rs", "gemm_ring_rs"):
        M, N, K = case["M"], case["N"], case["K"]
        b = 2.0 * (M * K + K * N) + _rs_bytes(M, N, R)
        if op == "gemm_ring_rs":
            b += 2.0 * (M - M // R) * N          # the whole partial product is stored locally
        return {"flops": 2.0 * M * N * K, "bytes": b}
    if op == "mlp_layer":
        M, H, F = case["M"], case["H"], case["F"]
        return {"flops": 6.0 * M * H * F, "bytes": _ag_bytes(M, 2 * F, F, H, R) + 2.0 * (M * F + F * H) + _rs_bytes(M, H, R)}
    if op == "moe_layer":
        T, H, F, E, k = case["T"], case["H"], case["F"], case["E"], case["topk"]
        b = 4.0 * T * E + 2.0 * (T * H + (T - T // R) * H) + 2.0 * min(E, T * k) * 3 * H * F + 2.0 * 2 * T * k * F + _rs_bytes(T, H, R)
        return {"flops": 6.0 * T * k * H * F, "bytes": b}
    S, heads, n = case["S"], case["heads"], case["S"] // R
    lo = case["rank"] * n
    pairs = n * lo + n * (n + 1) / 2.0 if case["causal"] else float(n) * S
    seen = (case["rank"] + 1) * n if case["causal"] else S
    return {"flops": 4.0 * HEAD_DIM * heads * pairs, "bytes": 2.0 * heads * HEAD_DIM * (2 * n + 4 * seen)}


def tolerance(case):
    """bf16 results of fp32 sums: one rounding each, chains of two matrix products and the bf16 probabilities of attention
    a few; gathered rows, pushed bytes of equal sums and expert indices are the same."""
    return {"rel": 5e-3, "max": 5e-2, "differ": 0.0}
