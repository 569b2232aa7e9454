"""The pipelined main loop at the sizes where it can go wrong: shapes one row, one 8-column vector and one 8-deep K
vector to either side of the tile (masked loads and stores), and as few K slabs as the pipeline has stages, one less and
one more.  Every configuration, both layouts of B, NaN between the rows of the operands.  Integer inputs whose sums stay
below 2^24, so fp32 accumulation is exact in any order and the comparison is bit for bit."""
import pytest
import torch

from paper_2406_06858_amd import binding as fb
from paper_2406_06858_amd import inputs as fi

import gpu_harness as gh
from test_gpu_strides import _rs_call, _say

pytestmark = pytest.mark.gpu


def _shapes(bm, bn):
    yield from [(2, 8, 8), (bm + 2, bn + 8, 72), (2 * bm - 2, 2 * bn - 8, 184),      # all three ragged
                (bm + 2, bn, 64), (bm, bn + 8, 128), (bm, bn, 200)]                  # one of them
    yield from [(bm, bn, 64 * slabs) for slabs in (1, 2, 3, 4, 5, 6, 7)]             # pipeline barely filled


@pytest.mark.parametrize("nk", [False, True])
@pytest.mark.parametrize("cfg", range(1, 11))
def test_tile_edges_and_short_pipelines(cfg, nk):
    bm, bn, _ = fb.flux_tile_config_info(cfg)
    for M, N, K in _shapes(bm, bn):
        w = fi.Workload("edges", "rs", M, N, K, 2, a_dist=("int", 2), b_dist=("int", 2), peer_dist=("int", 8), seed=7 * M + K)
        A, B, peers = fi.make_rs_inputs(w, 1)
        _, want = gh.oracle_rs(w, 1, A, B, peers)
        _say("edges cfg", cfg, "nk", nk, (M, N, K))
        _, outs = _rs_call(w, 1, A, B, peers, (8, 16, 8), tile_config=cfg, nk=nk)
        for r in range(w.R):
            gh.assert_bits_equal(outs[r][1], want[r], f"{(M, N, K)} slice {r}")


@pytest.mark.parametrize("M,N,K", [(200, 520, 1000), (72, 264, 520), (40, 136, 4104), (1000, 776, 584)])
def test_all_gather_of_a_ragged_shape(M, N, K):
    """The signal-wait form of the masked kernels, whatever configuration the library picks."""
    w = fi.Workload("edges_ag", "ag", M, N, K, 8, a_dist=("int", 2), b_dist=("int", 2), seed=M + K)
    chunks, B, arrival = fi.make_ag_inputs(w, 5)
    _, want = gh.oracle_ag(w, chunks, B)
    _say("edges ag", (M, N, K))
    C, A_agg, _, status = gh.run_ag(w, 5, chunks, B, arrival, repeat=2)
    assert status == (fb.FLUX_OK, 0)
    assert torch.equal(A_agg.cpu(), torch.cat(chunks))
    gh.assert_bits_equal(C, want, f"{(M, N, K)}")


@pytest.mark.parametrize("op", ["ag", "rs"])
@pytest.mark.parametrize("M,N,K,tile", [(40, 1544, 2056, (64, 128)), (40, 1544, 2048, (64, 128)), (72, 1544, 2760, (64, 128)), (72, 1544, 2712, (64, 64)),
                                        (200, 4200, 1000, (64, 128)), (512, 584, 2056, (64, 128)), (328, 1032, 4104, (64, 128)), (520, 584, 2056, None)])
def test_tile_of_few_ragged_rows(op, M, N, K, tile):
    """The configuration the library takes to either side of its lines for few rows: K, size of the weights, rows."""
    p = fb.problem(M, N, K, 8, 5)
    got = fb.flux_tile_shape(fb.FLUX_OP_AG if op == "ag" else fb.FLUX_OP_RS, p)
    assert tile is None or (got.tile_m, got.tile_n) == tile
    w = fi.Workload("few_rows", op, M, N, K, 8, a_dist=("int", 2), b_dist=("int", 2), peer_dist=("int", 8), seed=M + K)
    _say("few rows", op, (M, N, K))
    if op == "ag":
        chunks, B, arrival = fi.make_ag_inputs(w, 5)
        _, want = gh.oracle_ag(w, chunks, B)
        C, _, _, status = gh.run_ag(w, 5, chunks, B, arrival, repeat=2)
        assert status == (fb.FLUX_OK, 0)
        gh.assert_bits_equal(C, want, f"{(M, N, K)}")
    else:
        A, B, peers = fi.make_rs_inputs(w, 5)
        _, want = gh.oracle_rs(w, 5, A, B, peers)
        _, outs = _rs_call(w, 5, A, B, peers, (8, 16, 8))
        for r in range(w.R):
            gh.assert_bits_equal(outs[r][1], want[r], f"{(M, N, K)} slice {r}")


@pytest.mark.parametrize("R,pd", [(1, "bf16"), (8, "bf16"), (8, "f32"), (16, "bf16"), (16, "f32")])
@pytest.mark.parametrize("cfg,M,N,K,split", [(9, 64, 256, 1024, 4), (8, 16, 256, 1024, 9), (9, 48, 264, 1000, 2), (2, 208, 264, 640, 3),
                                             (1, 256, 256, 1024, 16), (10, 128, 136, 520, 5), (9, 64, 128, 1088, 17)])
def test_k_cut_tile_finished_by_its_parts(cfg, M, N, K, split, R, pd):
    """All parts of a tile finish it together (up to 16 of them; 17 leave it to the last), also where every part but the
    last gives up waiting at once (a spin limit of one tick: its share falls to the last); the counters must be
    clear again after each call."""
    w = fi.Workload("parts", "rs", M, N, K, R, partial_dtype=pd, out_dtype=pd, a_dist=("int", 2), b_dist=("int", 2),
                    peer_dist=("int", 8), seed=M + K + R)
    rank = R - 1
    A, B, peers = fi.make_rs_inputs(w, rank)
    _, want = gh.oracle_rs(w, rank, A, B, peers)
    dA, dB = A.to(gh.DEV), B.to(gh.DEV)
    dpeers = [None if t is None else t.to(gh.DEV) for t in peers]
    ws = None
    for ticks in (0, 1, 0, 1):
        p = fb.problem(M, N, K, R, rank, pd, pd, cfg, split, spin_timeout_ticks=ticks)
        if ws is None:
            ws = gh.workspace_for(fb.FLUX_OP_RS, p)
            ws.fill_(-1)
            fb.flux_init_buffers(fb.FLUX_OP_RS, p, ws)
        outs = [torch.full((w.S, N), float("nan"), dtype=torch.bfloat16 if pd == "bf16" else torch.float32, device=gh.DEV) for _ in range(R)]
        _say("parts cfg", cfg, (M, N, K), "split", split, "R", R, pd, "ticks", ticks)
        fb.flux_gemm_rs(p, dA, dB, dpeers, outs, ws)
        torch.cuda.synchronize()
        for r in range(R):
            gh.assert_bits_equal(outs[r], want[r], f"ticks {ticks} slice {r}")


@pytest.mark.parametrize("M,N,K,cfg,split,R", [(64, 2048, 8192, 9, 16, 8), (64, 8192, 4096, 9, 4, 8), (256, 4096, 4096, 2, 8, 1), (64, 4096, 4096, 10, 16, 16)])
def test_k_parts_beside_a_kernel_that_holds_compute_units(M, N, K, cfg, split, R):
    """Half of the compute units belong to another stream's GEMM for longer than the K-cut call takes, so half of its parts
    start only when others leave: nobody may sit out the bound (100 us) waiting for them, and the sums are the same bit for
    bit, whoever takes over whose share.  Then two K-cut calls side by side."""
    held = fb.problem(4096, 2048, 32768, 1, 0, tile_config=1, split_k=1)               # 128 tiles, one per compute unit
    hA, hB = (torch.zeros(s, dtype=torch.bfloat16, device=gh.DEV) for s in ((4096, 32768), (32768, 2048)))
    hC = torch.empty((4096, 2048), dtype=torch.bfloat16, device=gh.DEV)
    w = fi.Workload("beside", "rs", M, N, K, R, a_dist=("int", 2), b_dist=("int", 2), peer_dist=("int", 8), seed=M + K + R)
    A, B, peers = fi.make_rs_inputs(w, 0)
    dA, dB = A.to(gh.DEV), B.to(gh.DEV)
    dpeers = [None if t is None else t.to(gh.DEV) for t in peers]
    total = dA.float() @ dB.float()                     # exact: integers whose sums stay below 2^24
    for t in dpeers[1:]:
        total += t.float()
    want = total.to(torch.bfloat16)
    p = fb.problem(M, N, K, R, 0, tile_config=cfg, split_k=split)
    grid = fb.flux_split_plan(fb.FLUX_OP_RS, p)[1] * split
    sides = []
    for _ in range(2):
        ws = gh.workspace_for(fb.FLUX_OP_RS, p)
        fb.flux_init_buffers(fb.FLUX_OP_RS, p, ws)
        sides.append((ws, [torch.empty((w.S, N), dtype=torch.bfloat16, device=gh.DEV) for _ in range(R)], torch.cuda.Stream()))
    rec = torch.zeros((grid, 8), dtype=torch.int64, device=gh.DEV)
    overlapped = False
    for attempt in range(6):
        _say("beside a kernel that holds units", (M, N, K), "cfg", cfg, "split", split, "R", R, "attempt", attempt)
        for _, outs, _ in sides:
            for o in outs:
                o.fill_(float("nan"))
        torch.cuda.synchronize()
        holder = torch.cuda.Stream()
        if attempt < 5:
            fb.flux_gemm_rs(held, hA, hB, [None], [hC], None, holder)
            fb.flux_trace_next_call(rec)
        for ws, outs, stream in sides[:1 if attempt < 5 else 2]:
            fb.flux_gemm_rs(p, dA, dB, dpeers, outs, ws, stream)
        torch.cuda.synchronize()
        for _, outs, _ in sides[:1 if attempt < 5 else 2]:
            assert torch.equal(torch.cat(outs), want)
        if attempt < 5:
            start, end_main, end = (rec[:, i].cpu() for i in (4, 6, 7))
            overlapped = overlapped or bool(start.max() > end_main.min())
            # (finishing a tile alone takes some tens of us; a part that sat out the bound is past it)
            assert int((end - end_main).max()) < 9000, f"a part waited {int((end - end_main).max()) / 100} us"
    if not overlapped:
        pytest.skip("the two kernels never ran at the same time")
