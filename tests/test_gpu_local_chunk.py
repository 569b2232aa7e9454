"""A local chunk in a buffer of its own is moved by the GEMM grid, ahead of the remote chunks, or copied ahead of it; and the
slice reduction for every number of partials.  Integer inputs whose sums stay below 2^24: bit for bit."""
import pytest
import torch

from oracle import flux_oracle as fo
from paper_2406_06858_amd import binding as fb
from paper_2406_06858_amd import inputs as fi

import gpu_harness as gh
from test_gpu_strides import _say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,R,ctpc,cfg,pitch", [
    (8, 256, 512, 8, 1, 0, 0),            # a row per chunk, one piece per tile
    (200, 256, 1024, 8, 1, 0, 0),         # a tile over all chunks
    (200, 264, 1000, 8, 5, 3, 8),         # ragged, several signals per chunk, row pitch
    (512, 512, 512, 16, 2, 4, 0),         # the largest number of ranks: all sixteen places of the transfer order taken
    (64, 128, 256, 2, 1, 7, 0),
    (4096, 1280, 4096, 8, 1, 3, 0),       # several rounds of tiles, many pieces per owner
    (8192, 2560, 1536, 8, 1, 1, 0),       # the last chunks carried inside the main loops
    (768, 384, 8192, 2, 1, 3, 0),         # K-cut tiles, a chunk of 6 MiB: by the grid ...
    (770, 384, 8192, 2, 1, 3, 8),         # ... and above: a copy ahead of the grid
])
def test_local_chunk_moved_by_the_grid(M, N, K, R, ctpc, cfg, pitch):
    w = fi.Workload("local", "ag", M, N, K, R, a_dist=("int", 2), b_dist=("int", 2), seed=M + K + R)
    rank = R - 1
    chunks, B, arrival = fi.make_ag_inputs(w, rank)
    dB = B.to(gh.DEV)
    dchunks = [c.to(gh.DEV) for c in chunks]
    gathered = torch.cat(dchunks)
    want = (gathered.float() @ dB.float()).to(torch.bfloat16)           # exact in fp32: integers below 2^24
    store = torch.full((M, K + pitch), float("nan"), dtype=torch.bfloat16, device=gh.DEV)
    A_agg = store[:, :K]
    C = torch.empty((M, N), dtype=torch.bfloat16, device=gh.DEV)
    p = fb.problem(M, N, K, R, rank, "bf16", "bf16", cfg, comm_tiles_per_chunk=ctpc, spin_timeout_ticks=gh.TEST_TIMEOUT_TICKS,
                   lda=K + pitch if pitch else 0)
    signals = torch.zeros(R * ctpc, dtype=torch.int32, device=gh.DEV)
    ws = gh.workspace_for(fb.FLUX_OP_AG, p)
    ws.fill_(-1)
    fb.flux_init_buffers(fb.FLUX_OP_AG, p, ws, signals)
    preset = signals.clone()
    copy = torch.cuda.Stream()
    for call in range(4):                 # the third with the chunk in place: both forms on one workspace
        _say("local chunk", (M, N, K), "R", R, "cfg", cfg, "call", call)
        store.fill_(float("nan"))
        C.fill_(float("nan"))
        given = list(dchunks)
        if call == 2:
            given[rank] = A_agg[rank * w.S:(rank + 1) * w.S]
            given[rank].copy_(dchunks[rank])
        fb.flux_ag_gemm(p, given, A_agg, dB, C, signals, arrival, ws, torch.cuda.current_stream(), copy)
        torch.cuda.synchronize()
        assert fb.flux_query_status(ws) == (fb.FLUX_OK, 0)
        assert torch.equal(A_agg, gathered)
        assert torch.equal(signals, preset)
        assert torch.equal(C, want), f"call {call}"


@pytest.mark.parametrize("where", ["agg", "agg_across", "c"])
@pytest.mark.parametrize("M,N,K,R,cfg", [(64, 512, 512, 8, 0), (1024, 1024, 1024, 4, 3), (2048, 2560, 1536, 8, 1)])
def test_local_chunk_inside_what_the_call_writes(M, N, K, R, cfg, where):
    """The local chunk handed over in another chunk's rows of the gathered matrix, across two chunks' rows, or in the first
    rows of C: the call reads all of it before it writes there."""
    w = fi.Workload("local_inside", "ag", M, N, K, R, a_dist=("int", 2), b_dist=("int", 2), seed=M + K + R)
    rank = R - 1
    chunks, B, arrival = fi.make_ag_inputs(w, rank)
    dB = B.to(gh.DEV)
    dchunks = [c.to(gh.DEV) for c in chunks]
    gathered = torch.cat(dchunks)
    want = (gathered.float() @ dB.float()).to(torch.bfloat16)           # exact in fp32: integers below 2^24
    A_agg = torch.empty((M, K), dtype=torch.bfloat16, device=gh.DEV)
    C = torch.empty((M, N), dtype=torch.bfloat16, device=gh.DEV)
    at = {"agg": A_agg.flatten(), "agg_across": A_agg.flatten()[w.S // 2 * K:], "c": C.flatten()}[where][:w.S * K].view(w.S, K)
    p = fb.problem(M, N, K, R, rank, "bf16", "bf16", cfg, spin_timeout_ticks=gh.TEST_TIMEOUT_TICKS)
    signals = torch.zeros(R, dtype=torch.int32, device=gh.DEV)
    ws = gh.workspace_for(fb.FLUX_OP_AG, p)
    fb.flux_init_buffers(fb.FLUX_OP_AG, p, ws, signals)
    copy = torch.cuda.Stream()
    for call in range(3):
        _say("local inside", where, (M, N, K), "R", R, "call", call)
        A_agg.fill_(float("nan"))
        C.fill_(float("nan"))
        at.copy_(dchunks[rank])
        fb.flux_ag_gemm(p, dchunks[:rank] + [at] + dchunks[rank + 1:], A_agg, dB, C, signals, arrival, ws, torch.cuda.current_stream(), copy)
        torch.cuda.synchronize()
        assert fb.flux_query_status(ws) == (fb.FLUX_OK, 0)
        assert torch.equal(A_agg, gathered)
        assert torch.equal(C, want), f"call {call}"


@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("R", range(1, 17))
def test_slice_reduce_of_every_rank_count(R, dt):
    """Every number of partials from one to sixteen; one row of one vector, and a row count no workgroup divides."""
    td = torch.bfloat16 if dt == "bf16" else torch.float32
    for S, N in ((1, 8), (37, 136)):
        g = torch.Generator().manual_seed(R + S)
        staged = [torch.randint(-8, 9, (S, N), generator=g).to(td) for _ in range(R)]
        out = torch.full((S, N), float("nan"), dtype=td, device=gh.DEV)
        p = fb.problem(S * R, N, 64, R, R - 1, dt, dt)
        _say("slice reduce R", R, dt, (S, N))
        fb.flux_rs_reduce_slice(p, [t.to(gh.DEV) for t in staged], out)
        torch.cuda.synchronize()
        gh.assert_bits_equal(out, fo.reduce_slice([fi.to_numpy(t) for t in staged], dt, dt)[1], f"R {R} {(S, N)}")
