"""Performance cases of the fused tensor-parallel GEMMs, through the binding's public entry points.

A case is ONE rank's view of an R-way tensor-parallel layer, all buffers in this GPU's memory:
`ag` = flux_ag_gemm (up projection / QKV), `rs` = flux_gemm_rs (down / output projection, peers reduced in the
epilogue), `a2a` = the Write-only flux_gemm_rs followed by flux_rs_reduce_slice of the own slice (what one rank
of a group executes when the partials travel as an AlltoAll).  `layers` weight matrices are walked per pass, as a
decode step walks its layers, so that few-row cases read their weights from memory and not from a cache.
"""
import torch

from paper_2406_06858_amd import binding as fb

DEV = "cuda:0"
TORCH = {"bf16": torch.bfloat16, "f32": torch.float32}
SIZE = {"bf16": 2, "f32": 4}


def _case(name, op, M, N, K, R, *, rank=3, layers=1, dtype="bf16", nk=False, in_place=True):
    c = {"op": op, "M": M, "N": N, "K": K, "R": R, "rank": rank, "layers": layers, "dtype": dtype, "nk": nk,
         "in_place": in_place}
    return c if name is None else {"name": name, **c}


def listed():
    return [
        # the small fp32 configuration: one call of a few microseconds, launch and host path
        _case("rs_small_f32", "rs", 128, 256, 256, 2, rank=1, dtype="f32"),
        # decode, batch 8, Llama-2-70B-like MLP at TP=8: up projection of four layers
        _case("ag_decode_m8", "ag", 8, 3584, 8192, 8, layers=4),
        # decode, batch 64: down projection of four layers
        _case("rs_decode_m64", "rs", 64, 8192, 3584, 8, layers=4),
        # decode with a batch that no tile divides, a linear layer's own weight layout, the local chunk handed over
        # in a buffer of its own
        _case("ag_decode_m200", "ag", 200, 3584, 8192, 8, layers=4, nk=True, in_place=False),
        # a short prompt through the MLP of the GPT-3-175B-like layer
        _case("rs_prompt_m512", "rs", 512, 12288, 6144, 8),
        # prefill, 4096 tokens, Llama-2-70B-like MLP: up and down projection
        _case("ag_prefill", "ag", 4096, 3584, 8192, 8),
        _case("rs_prefill", "rs", 4096, 8192, 3584, 8),
        # prefill of as many tokens as the prompts happen to have
        _case("ag_prefill_ragged", "ag", 3000, 3584, 8192, 8, in_place=False),
        # nothing is a multiple of a tile: rows, columns or inner dimension
        _case("rs_ragged", "rs", 1496, 5112, 3400, 8),
        # training, GPT-3-175B-like layer, 8192 tokens: QKV projection and attention output projection
        _case("ag_train", "ag", 8192, 4608, 12288, 8),
        _case("rs_train", "rs", 8192, 12288, 1536, 8),
        # backward of the QKV projection: the input gradient dY.W^T with W as the layer stores it, scattered to
        # its owners, and the sum of the own slice
        _case("a2a_backward", "a2a", 8192, 12288, 4608, 8, nk=True),
    ]


def draw(rng):
    """A case of the same ranges: 8 to 8192 rows, 256 to 12288 columns and inner dimension, 2 to 16 ranks."""
    while True:
        op = rng.choice(["ag", "ag", "rs", "rs", "a2a"])
        R = rng.choice([2, 4, 8, 8, 8, 16])
        M = int(round(8 * 1024 ** rng.random()))                # log-uniform, 8 .. 8192
        M = max(R, M // R * R)
        if rng.random() < 0.4:
            M = max(R, (M + 63) // 64 * 64)                     # (a multiple of every R)
        # widths: the layers' own, or any multiple of 8
        widths = [1536, 3584, 4608, 6144, 8192, 12288]
        N, K = (rng.choice(widths) if rng.random() < 0.6 else 8 * int(round(32 * 48 ** rng.random())) for _ in range(2))
        small = rng.random() < 0.15
        if small:                                               # the small calls' range
            M, N, K = min(M, 512) // R * R, min(N, 1024), min(K, 1024)
        dtype = "f32" if op == "rs" and rng.random() < 0.25 else "bf16"
        c = _case(None, op, M, N, K, R, rank=rng.randrange(R), layers=4 if M <= 256 and not small else 1, dtype=dtype,
                  nk=rng.random() < 0.4, in_place=rng.random() < 0.6)
        w = work(c)
        if w["flops"] <= 5e11 and w["bytes"] <= 1.2e9:
            return c


def _randn(gen, shape, dtype, std=1.0):
    return torch.randn(shape, generator=gen, device=DEV, dtype=torch.float32).mul_(std).to(TORCH[dtype])


def _workspace(op, p):
    n = fb.flux_workspace_bytes(op, p)
    return torch.zeros((n + 3) // 4, dtype=torch.int32, device=DEV) if n else None


def prepare(case, seed):
    """Activations N(0,1), weights N(0,0.02), as in a transformer layer; buffers, workspace and streams as a
    program keeps them."""
    op, M, N, K, R, rank, dtype = (case[k] for k in ("op", "M", "N", "K", "R", "rank", "dtype"))
    S = M // R
    gen = torch.Generator(device=DEV).manual_seed(seed)
    state = {"op": op, "calls": [], "stream": torch.cuda.current_stream()}
    nk = int(case["nk"])
    weights = [_randn(gen, (N, K) if nk else (K, N), "bf16", 0.02) for _ in range(case["layers"])]
    if op == "ag":
        p = fb.problem(M, N, K, R, rank, "bf16", dtype, b_is_nk=nk)
        remote = [r for r in range(R) if r != rank]
        order = torch.randperm(R - 1, generator=torch.Generator().manual_seed(seed)).tolist()
        state["arrival"] = [remote[i] for i in order]
        state["agg"] = torch.zeros((M, K), dtype=torch.bfloat16, device=DEV)
        state["signals"] = torch.zeros(R, dtype=torch.int32, device=DEV)
        state["copy_stream"] = torch.cuda.Stream()
        state["ws"] = _workspace(fb.FLUX_OP_AG, p)
        fb.flux_init_buffers(fb.FLUX_OP_AG, p, state["ws"], state["signals"])
        chunks = [_randn(gen, (S, K), "bf16") for _ in range(R)]
        if case["in_place"]:            # the rank's own activations were produced where they are gathered
            local = state["agg"][rank * S:(rank + 1) * S]
            local.copy_(chunks[rank])
            chunks[rank] = local
        state["chunks"] = chunks
        for B in weights:
            state["calls"].append((B, torch.zeros((M, N), dtype=TORCH[dtype], device=DEV)))
    else:
        wo = op == "a2a"
        p = fb.problem(M, N, K, R, rank, dtype, dtype, b_is_nk=nk, flags=fb.FLUX_FLAG_RS_WRITE_ONLY if wo else 0)
        state["ws"] = _workspace(fb.FLUX_OP_RS, p)
        if state["ws"] is not None:
            fb.flux_init_buffers(fb.FLUX_OP_RS, p, state["ws"])
        for B in weights:
            A = _randn(gen, (M, K), "bf16")
            outs = [torch.zeros((S, N), dtype=TORCH[dtype], device=DEV) for _ in range(R)]
            # a2a: the partials that the others have sent for this rank's slice; rs: theirs of the whole matrix
            peers = [None if r == rank else _randn(gen, (S if wo else M, N), dtype) for r in range(R)]
            own = torch.zeros((S, N), dtype=TORCH[dtype], device=DEV) if wo else None
            staged = [outs[rank] if r == rank else peers[r] for r in range(R)] if wo else None
            state["calls"].append((A, B, peers, outs, staged, own))
    state["p"] = p
    return state


def run(state):
    p = state["p"]
    if state["op"] == "ag":
        for B, C in state["calls"]:
            fb.flux_ag_gemm(p, state["chunks"], state["agg"], B, C, state["signals"], state["arrival"], state["ws"],
                            state["stream"], state["copy_stream"])
        return [C for _, C in state["calls"]] + [state["agg"]]
    outputs = []
    for A, B, peers, outs, staged, own in state["calls"]:
        if state["op"] == "a2a":
            fb.flux_gemm_rs(p, A, B, None, outs, state["ws"], state["stream"])
            fb.flux_rs_reduce_slice(p, staged, own, state["stream"])
            outputs.append(own)
        else:
            fb.flux_gemm_rs(p, A, B, peers, outs, state["ws"], state["stream"])
        outputs += outs
    return outputs


def work(case):
    """Each operand read once, each result written once.  (`ag`: the gathered matrix is a result; a local chunk
    that is in place already is read, not moved.)"""
    op, M, N, K, R, layers = (case[k] for k in ("op", "M", "N", "K", "R", "layers"))
    e = SIZE[case["dtype"]]
    S = M // R
    flops = 2.0 * M * N * K
    if op == "ag":
        moved = M - S if case["in_place"] else M
        nbytes = 2.0 * (M * K + K * N + moved * K) + e * M * N
    elif op == "rs":
        nbytes = 2.0 * (M * K + K * N) + e * R * M * N
        flops += (R - 1.0) * M * N
    else:
        nbytes = 2.0 * (M * K + K * N) + e * (M * N + R * S * N + S * N)
        flops += (R - 1.0) * S * N
    return {"bytes": layers * nbytes, "flops": layers * flops}


def tolerance(case):
    """About four times the distance from the same sums in fp64: bf16 results, one rounding to 8 significant bits
    (1.66e-3 in the 2-norm, 3.9e-3 at most; 4.4e-3 with the two roundings of `a2a`); fp32 results, sums in another
    order (4e-8 to 1.3e-7 in the 2-norm, up to 8e-7 at most over K = 8192)."""
    if case["dtype"] == "f32":
        return {"rel": 6e-7, "max": 4e-6}
    return {"rel": 7e-3, "max": 2e-2}
