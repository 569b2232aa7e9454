"""AllGather calls whose grid reads A from the chunk sources and stores the gathered matrix out of its slabs in LDS, against the form that
gathers first and waits for signals (FLUX_FLAG_AG_COPY_UPFRONT, or what overlaps keep to it).  Integer inputs whose sums stay below
2^24: bit for bit."""
import pytest
import torch

from paper_2406_06858_amd import binding as fb
from paper_2406_06858_amd import inputs as fi

import gpu_harness as gh
from test_gpu_strides import _say

pytestmark = pytest.mark.gpu


def _case(M, N, K, R, seed=None):
    w = fi.Workload("chunk_sources", "ag", M, N, K, R, a_dist=("int", 2), b_dist=("int", 2), seed=seed or M + N + K + R)
    rank = (M + N) % R
    chunks, B, arrival = fi.make_ag_inputs(w, rank)
    dchunks = [c.to(gh.DEV) for c in chunks]
    gathered = torch.cat(dchunks)
    return w, rank, dchunks, B.to(gh.DEV), arrival, gathered


def _call(w, rank, given, dB, arrival, cfg, *, pitch=0, nk=False, flags=0, split=0, ctpc=1, in_place=False, dtype="bf16", agg=None, C=None):
    """One call on fresh buffers; the gathered matrix's rows, what lies between them, C."""
    p = fb.problem(w.M, w.N, w.K, w.R, rank, "bf16", dtype, cfg, split, flags, ctpc, spin_timeout_ticks=gh.TEST_TIMEOUT_TICKS,
                   lda=w.K + pitch if pitch else 0, b_is_nk=int(nk))
    store = torch.full((w.M, w.K + pitch), float("nan"), dtype=torch.bfloat16, device=gh.DEV) if agg is None else agg
    A_agg = store[:, :w.K]
    if C is None:
        C = torch.full((w.M, w.N), float("nan"), dtype=torch.float32 if dtype == "f32" else torch.bfloat16, device=gh.DEV)
    given = list(given)
    if in_place:
        local = A_agg[rank * w.S:(rank + 1) * w.S]
        local.copy_(given[rank])
        given[rank] = local
    signals = torch.zeros(w.R * ctpc, dtype=torch.int32, device=gh.DEV)
    ws = gh.workspace_for(fb.FLUX_OP_AG, p)
    ws.fill_(-1)
    fb.flux_init_buffers(fb.FLUX_OP_AG, p, ws, signals)
    preset = signals.clone()
    B = dB.t().contiguous() if nk else dB
    fb.flux_ag_gemm(p, given, A_agg, B, C, signals, arrival, ws, torch.cuda.current_stream(), torch.cuda.Stream())
    torch.cuda.synchronize()
    assert fb.flux_query_status(ws) == (fb.FLUX_OK, 0)
    assert torch.equal(signals, preset)
    return A_agg, store[:, w.K:], C


@pytest.mark.parametrize("cfg", range(1, 11))
@pytest.mark.parametrize("shape", [
    (1024, 2048, 512, 8),        # every tile divides it
    (200, 264, 200, 8),          # chunks of 25 rows; rows, columns and K with a remainder
    (16, 2056, 72, 16),          # a row per chunk
    (1036, 904, 328, 2),         # two long chunks, the border inside a tile
    (256, 1792, 64, 4),          # one slab; 256x256: the fewest columns of tiles that cover a tile's rows, less one
])
def test_chunk_sources_against_the_gathered_form(shape, cfg):
    w, rank, dchunks, dB, arrival, gathered = _case(*shape)
    want = gathered.float() @ dB.float()            # exact: integers below 2^24
    for nk, pitch, in_place, split, ctpc, dtype in ((False, 0, True, 0, 1, "bf16"), (True, 8, False, 0, 1, "bf16"), (False, 64, True, 3, 1, "f32"),
                                                    (True, 0, False, 2, next((d for d in (2, 5) if w.S % d == 0), 1), "f32")):
        _say("chunk sources", shape, "cfg", cfg, "nk", nk, "pitch", pitch, "in place", in_place, "split", split)
        for flags in (0, fb.FLUX_FLAG_AG_COPY_UPFRONT, fb.FLUX_FLAG_NO_SWIZZLE):
            agg, between, C = _call(w, rank, dchunks, dB, arrival, cfg, pitch=pitch, nk=nk, flags=flags, split=split, ctpc=ctpc, in_place=in_place, dtype=dtype)
            assert torch.equal(agg, gathered), flags
            assert between.isnan().all(), flags
            assert torch.equal(C, want.to(C.dtype)), flags


@pytest.mark.parametrize("shape", [(8, 384, 1024, 8), (64, 512, 2048, 8), (200, 512, 4096, 8), (3000, 1024, 512, 8), (2304, 4608, 320, 8)])
def test_chunk_sources_as_planned(shape):
    """The library's own tile and K cut, small N included (too few columns of tiles: the gathered form)."""
    for N in (shape[1], 128, 8):
        w, rank, dchunks, dB, arrival, gathered = _case(shape[0], N, shape[2], shape[3])
        _say("chunk sources as planned", (shape[0], N, shape[2]))
        agg, _, C = _call(w, rank, dchunks, dB, arrival, 0)
        assert torch.equal(agg, gathered)
        assert torch.equal(C, (gathered.float() @ dB.float()).to(C.dtype))


@pytest.mark.parametrize("where", ["its_rows", "c"])
def test_a_remote_chunk_inside_what_the_call_writes(where):
    """A remote chunk handed over in its own rows of the gathered matrix, or, every tile waiting for everything, inside C: as before."""
    w, rank, dchunks, dB, arrival, gathered = _case(32, 1024, 512, 4)
    far = (rank + 1) % w.R
    agg = torch.full((w.M, w.K), float("nan"), dtype=torch.bfloat16, device=gh.DEV)
    C = torch.full((w.M, w.N), float("nan"), dtype=torch.bfloat16, device=gh.DEV)
    at = {"its_rows": agg[far * w.S:(far + 1) * w.S], "c": C.flatten()[:w.S * w.K].view(w.S, w.K)}[where]
    at.copy_(dchunks[far])
    given = list(dchunks)
    given[far] = at
    out, _, C = _call(w, rank, given, dB, arrival, 0, agg=agg, C=C)
    assert torch.equal(out, gathered)
    assert torch.equal(C, (gathered.float() @ dB.float()).to(C.dtype))
