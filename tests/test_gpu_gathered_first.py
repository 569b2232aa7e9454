"""AllGather-GEMM calls that gather A first: everything moved up front (FLUX_FLAG_AG_COPY_UPFRONT), or the later chunks carried inside the first
round's main loops (several rounds of tiles in too few columns for the tiles to read A from the chunk sources, or a chunk inside what the call
writes).  The tile trace says that the tiles did wait.  Integer inputs whose sums stay below 2^24: bit for bit."""
import numpy as np
import pytest
import torch

from oracle import flux_oracle as fo
from paper_2406_06858_amd import binding as fb
from paper_2406_06858_amd import inputs as fi

import gpu_harness as gh
import test_gpu_graph_replay as replay
import test_gpu_strides as strides
import test_gpu_trace as tr
from test_gpu_strides import _say

pytestmark = pytest.mark.gpu

UPFRONT = fb.FLUX_FLAG_AG_COPY_UPFRONT


def _ints(M, N, K, R, seed=84):
    return fi.Workload("gathered_first", "ag", M, N, K, R, a_dist=("int", 2), b_dist=("int", 2), seed=seed)


NARROW = _ints(16384, 1792, 2048, 8)          # two rounds, seven columns of 256x256 tiles: three chunks are carried


def _trace(p):
    """The tile trace of the next AllGather call."""
    full, cut, k = fb.flux_split_plan(fb.FLUX_OP_AG, p)
    trace = torch.zeros((full + cut * k, 8), dtype=torch.int64, device=gh.DEV)
    fb.flux_trace_next_call(trace)
    return trace


def _waited(trace) -> bool:
    """Tiles that wait leave the time at which they were past their wait; those of a kernel without one leave their start's."""
    return bool((trace[:, 5] > trace[:, 4]).any())


def _check(w, rank, pads=(0, 0, 0), order="random", waits=True, **kw):
    """Two calls, each checked; the first one's trace."""
    chunks, B, arrival = fi.make_ag_inputs(w, rank)
    if order != "random":
        arrival = fo.default_order(rank, w.R) if order == "ring" else list(reversed(fo.default_order(rank, w.R)))
    dims = dict(kw)
    nk = dims.pop("nk", False)
    dims.pop("local_in_place", None)
    trace = _trace(fb.problem(w.M, w.N, w.K, w.R, rank, lda=w.K + pads[0] if pads[0] else 0, b_is_nk=int(nk), **dims))
    p, C, A_agg = strides._ag_call(w, rank, chunks, B, arrival, pads, **kw)
    assert _waited(trace) == waits
    gathered = torch.cat([c.to(gh.DEV) for c in chunks])
    assert torch.equal(A_agg, gathered)
    assert torch.equal(C, (gathered.float() @ B.to(gh.DEV).float()).to(C.dtype))
    return p


@pytest.mark.parametrize("w,order,carried,kw", [
    (NARROW, "ring", 3, dict()), (NARROW, "random", 3, dict()), (NARROW, "random", 0, dict(flags=UPFRONT)),
    (_ints(16384, 1792, 1536, 8), "random", 3, dict(nk=True)),
    (_ints(16384, 1792, 1536, 8), "random", 3, dict(tile_config=1, local_in_place=True)),
    (_ints(20480, 1792, 2048, 2), "random", 1, dict()),       # the first round is all local tiles
    (_ints(16384, 1792, 2048, 4), "random", 1, dict()),
    (_ints(12288, 1792, 1408, 16), "random", 3, dict()),      # fewer pieces per chunk than the first round has workgroups
])
def test_later_chunks_travel_inside_the_main_loops(w, order, carried, kw):
    _say("gathered first", (w.M, w.N, w.K, w.R), order, kw)
    p = _check(w, w.R - 1, order=order, **kw)
    assert fb.flux_ag_deferred_tiles(p) == carried


@pytest.mark.parametrize("M,N,K,R,ctpc,cfg,pitch", [
    (8, 256, 512, 8, 1, 0, 0),            # a row per chunk
    (64, 1024, 2048, 8, 4, 0, 0),
    (200, 264, 1000, 8, 5, 3, 8),         # ragged, several signals per chunk, row pitch
    (512, 512, 512, 16, 2, 4, 64),
    (4096, 2048, 512, 8, 1, 0, 0),
    (4096, 1280, 4096, 8, 4, 3, 0),       # several rounds of tiles
    (8192, 2560, 1536, 8, 1, 1, 0),
    (768, 384, 8192, 2, 1, 3, 0),         # K-cut tiles, a local chunk of 6 MiB: by the grid ...
    (770, 384, 8192, 2, 1, 3, 8),         # ... and above: a copy ahead of the grid
])
def test_everything_moved_up_front(M, N, K, R, ctpc, cfg, pitch):
    """... the local chunk in a buffer of its own and in its place; by default the same call reads the chunk sources and waits for nothing."""
    w = _ints(M, N, K, R, seed=M + K + R)
    kw = dict(comm_tiles_per_chunk=ctpc, tile_config=cfg)
    sh = fb.flux_tile_shape(fb.FLUX_OP_AG, fb.problem(M, N, K, R, 0, **kw))
    for order, flags, in_place in (("random", UPFRONT, False), ("reversed", UPFRONT, True), ("ring", 0, False)):
        _say("up front", (M, N, K), "R", R, "cfg", cfg, "flags", flags, "in place", in_place)
        few_columns = 32 * -(-N // sh.tile_n) < sh.tile_m
        _check(w, R - 1, (pitch, 0, 0), order, flags != 0 or few_columns, flags=flags, local_in_place=in_place, **kw)


@pytest.mark.parametrize("ctpc", [1, 2])
def test_up_front_into_rows_that_are_not_line_aligned(ctpc):
    """Base 16 bytes into a line: rows of two communication tiles can share one, and the wait drops stale lines from the die's L2."""
    w = _ints(2048, 512, 512, 8)
    chunks, B, arrival = fi.make_ag_inputs(w, 3)
    _, want = gh.oracle_ag(w, chunks, B)
    _say("up front, not line aligned", ctpc)
    C, A_agg, _, status = gh.run_ag(w, 3, chunks, B, arrival, flags=UPFRONT, comm_tiles_per_chunk=ctpc, repeat=2, agg_offset_elems=8)
    assert status == (fb.FLUX_OK, 0) and A_agg.data_ptr() % 128 == 16
    gh.assert_bits_equal(C, want, "C")
    gh.assert_bits_equal(A_agg, np.concatenate([fi.to_numpy(c) for c in chunks]), "A_agg")


@pytest.mark.parametrize("K,pitch,offset,N,waits", [
    (4104, 0, 0, 2048, True), (4104, 56, 0, 2048, False),                        # rows in parts of lines, a pitch of whole lines
    (4160, 0, 0, 2048, False), (4160, 8, 0, 2048, True), (4160, 0, 8, 2048, True),      # whole lines, a pitch of none, a base inside one
    (4104, 0, 0, 3592, False), (4088, 0, 0, 2048, False),                        # enough columns to hide it; below 32 MB
])
def test_large_gathered_matrix_of_partial_lines(K, pitch, offset, N, waits):
    w, rank = _ints(4096, N, K, 8), 5
    chunks, B, arrival = fi.make_ag_inputs(w, rank)
    dchunks, dB = [c.to(gh.DEV) for c in chunks], B.to(gh.DEV)
    gathered = torch.cat(dchunks)
    want = (gathered.float() @ dB.float()).to(torch.bfloat16)
    p = fb.problem(w.M, N, K, w.R, rank, tile_config=2, lda=K + pitch if pitch else 0, spin_timeout_ticks=gh.TEST_TIMEOUT_TICKS)
    store = torch.full((w.M * (K + pitch) + offset,), float("nan"), dtype=torch.bfloat16, device=gh.DEV)
    A_agg = store[offset:].view(w.M, K + pitch)[:, :K]
    C = torch.full((w.M, N), float("nan"), dtype=torch.bfloat16, device=gh.DEV)
    signals = torch.zeros(w.R, dtype=torch.int32, device=gh.DEV)
    ws = gh.workspace_for(fb.FLUX_OP_AG, p)
    fb.flux_init_buffers(fb.FLUX_OP_AG, p, ws, signals)
    for _ in range(2):
        store.fill_(float("nan"))
        C.fill_(float("nan"))
        _say("partial lines", (w.M, N, K), "pitch", pitch, "offset", offset)
        trace = _trace(p)
        fb.flux_ag_gemm(p, dchunks, A_agg, dB, C, signals, arrival, ws, torch.cuda.current_stream(), torch.cuda.Stream())
        torch.cuda.synchronize()
        assert fb.flux_query_status(ws) == (fb.FLUX_OK, 0)
        assert _waited(trace) == waits
        assert torch.equal(C, want) and torch.equal(A_agg, gathered)


def test_a_source_in_its_own_rows():
    """Eighteen columns of tiles, but a chunk lies in its own rows of the gathered matrix: A is gathered first, the later chunks travel inside the
    main loops, that one onto itself."""
    w, rank = _ints(8192, 4608, 2048, 8), 2
    chunks, B, arrival = fi.make_ag_inputs(w, rank)
    dchunks, dB = [c.to(gh.DEV) for c in chunks], B.to(gh.DEV)
    gathered = torch.cat(dchunks)
    want = (gathered.float() @ dB.float()).to(torch.bfloat16)
    p = fb.problem(w.M, w.N, w.K, w.R, rank, spin_timeout_ticks=gh.TEST_TIMEOUT_TICKS)
    assert fb.flux_ag_deferred_tiles(p) == 4
    signals = torch.zeros(w.R, dtype=torch.int32, device=gh.DEV)
    ws = gh.workspace_for(fb.FLUX_OP_AG, p)
    fb.flux_init_buffers(fb.FLUX_OP_AG, p, ws, signals)
    for far in (None, arrival[0], arrival[-1]):            # none, one that is moved up front, one that is carried
        A_agg = torch.full((w.M, w.K), float("nan"), dtype=torch.bfloat16, device=gh.DEV)
        C = torch.full((w.M, w.N), float("nan"), dtype=torch.bfloat16, device=gh.DEV)
        given = list(dchunks)
        if far is not None:
            given[far] = A_agg[far * w.S:(far + 1) * w.S]
            given[far].copy_(dchunks[far])
        _say("chunk in its own rows", far)
        trace = _trace(p)
        fb.flux_ag_gemm(p, given, A_agg, dB, C, signals, arrival, ws, torch.cuda.current_stream(), torch.cuda.Stream())
        torch.cuda.synchronize()
        assert fb.flux_query_status(ws) == (fb.FLUX_OK, 0)
        assert _waited(trace) == (far is not None)
        assert torch.equal(C, want) and torch.equal(A_agg, gathered)
        assert signals.tolist() == [1 if r == rank else 0 for r in range(w.R)]


def test_carried_pieces_are_moved_whatever_happens_to_the_tiles():
    """A spin limit of one tick: a workgroup whose signal is missing when it gets to its wait gives up; every kernel ends, every piece is moved."""
    rank = 1
    chunks, B, arrival = fi.make_ag_inputs(NARROW, rank)
    gathered = torch.cat([c.to(gh.DEV) for c in chunks])
    want = (gathered.float() @ B.to(gh.DEV).float()).to(torch.bfloat16)
    _say("carried, one tick")
    C, A_agg, _, (code, detail) = gh.run_ag(NARROW, rank, chunks, B, arrival, timeout_ticks=1)
    assert torch.equal(A_agg, gathered)
    own = slice(rank * NARROW.S, (rank + 1) * NARROW.S)
    assert torch.equal(C[own], want[own])
    assert code in (fb.FLUX_OK, fb.FLUX_ERR_TIMEOUT)
    if code == fb.FLUX_OK:
        assert torch.equal(C, want)
    else:
        assert 0 <= detail < NARROW.R and detail != rank


def test_carried_chunks_replay_from_a_graph():
    shape = dict(M=16384, N=1792, K=2048)
    trace = _trace(fb.problem(shape["M"], shape["N"], shape["K"], 8, 5))
    replay.test_ag_gemm_replays_from_a_graph(shape, 0)
    assert _waited(trace)


@pytest.mark.parametrize("cfg", [0, 1])
def test_trace_of_a_call_that_moves_everything_up_front(cfg):
    w, rank = _ints(4096, 5120, 512, 8, seed=92), 2
    chunks, B, arrival = fi.make_ag_inputs(w, rank)
    p = fb.problem(w.M, w.N, w.K, w.R, rank, tile_config=cfg, flags=UPFRONT, spin_timeout_ticks=gh.TEST_TIMEOUT_TICKS)
    grid, tile, _, coords, sh, _ = tr._expected_tiles("ag", p, w, rank, arrival, 8)
    trace = _trace(p)
    _say("trace, up front, cfg", cfg)
    _, _, _, status = gh.run_ag(w, rank, chunks, B, arrival, tile_config=cfg, flags=UPFRONT)
    assert status == (fb.FLUX_OK, 0) and _waited(trace)
    rec = tr._records(trace, grid)
    assert np.array_equal(rec["block"], np.arange(grid)) and np.array_equal(rec["tile"], tile)
    assert np.array_equal(np.stack([rec["m_tile"], rec["n_tile"]], axis=1), coords[tile])
    assert (rec["t_start"] <= rec["t_ready"]).all() and (rec["t_ready"] <= rec["t_main_end"]).all() and (rec["t_main_end"] <= rec["t_end"]).all()
    tr._check_dispatch_order(rec, tile, sh, w, "ag")
