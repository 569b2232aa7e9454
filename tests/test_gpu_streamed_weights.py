"""Weights larger than all L2s under one or two rows of tiles are streamed by kernels of their own: every configuration that has them, both
layouts of B, both operations, whole and K-cut tiles, edges in rows and in K; and what keeps to the other kernels (rows of B that are no
whole lines, a second row of tiles that is far from full, three rows of tiles).  Integer inputs whose sums stay below 2^24: bit for bit."""
import pytest
import torch

from paper_2406_06858_amd import binding as fb

import gpu_harness as gh
from test_gpu_strides import _say

pytestmark = pytest.mark.gpu


def _ints(gen, shape, top=2):
    return torch.randint(-top, top + 1, shape, generator=gen, device=gh.DEV, dtype=torch.int32).to(torch.bfloat16)


@pytest.mark.parametrize("nk", [0, 1])
@pytest.mark.parametrize("M,cfg", [(8, 8), (32, 8), (48, 8), (64, 7), (128, 7), (40, 9), (64, 9), (128, 9), (192, 9), (200, 2), (304, 2), (496, 2)])
def test_streamed_weights(M, cfg, nk):
    R, rank = 8, 3
    for N, K in ((8192, 2304), (8192, 2312), (8200, 2304)):
        assert N * K * 2 > 32 << 20
        gen = torch.Generator(device=gh.DEV).manual_seed(M + K)
        A, B = _ints(gen, (M, K)), _ints(gen, (N, K) if nk else (K, N))
        product = A.float() @ (B.t() if nk else B).float()              # exact: integers below 2^24
        peers = [None if r == rank else _ints(gen, (M, N), 8) for r in range(R)]
        want = (product + sum(t.float() for t in peers if t is not None)).to(torch.bfloat16)
        chunks = [A[r * (M // R):(r + 1) * (M // R)].contiguous() for r in range(R)]
        for split in (1, 3):
            _say("streamed weights", (M, N, K), "nk", nk, "cfg", cfg, "split", split)
            p = fb.problem(M, N, K, R, rank, tile_config=cfg, split_k=split, b_is_nk=nk)
            ws = gh.workspace_for(fb.FLUX_OP_RS, p)
            if ws is not None:
                fb.flux_init_buffers(fb.FLUX_OP_RS, p, ws)
            outs = [torch.full((M // R, N), float("nan"), dtype=torch.bfloat16, device=gh.DEV) for _ in range(R)]
            fb.flux_gemm_rs(p, A, B, peers, outs, ws)
            torch.cuda.synchronize()
            assert torch.equal(torch.cat(outs), want)
            ws = gh.workspace_for(fb.FLUX_OP_AG, p)
            signals = torch.zeros(R, dtype=torch.int32, device=gh.DEV)
            fb.flux_init_buffers(fb.FLUX_OP_AG, p, ws, signals)
            agg = torch.full((M, K), float("nan"), dtype=torch.bfloat16, device=gh.DEV)
            C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=gh.DEV)
            fb.flux_ag_gemm(p, chunks, agg, B, C, signals, None, ws, torch.cuda.current_stream(), torch.cuda.Stream())
            torch.cuda.synchronize()
            assert torch.equal(agg, A)
            assert torch.equal(C, product.to(torch.bfloat16))
