"""Reduce-scatter tiles that add their peers ahead of the main loop (every second column, or row, of large tiles), and A asked for
ahead of it: whole and ragged tiles, up to eight ranks and more, both dtypes, both layouts of B, row pitches.
Where inputs are integers whose sums stay below 2^24, any order of an fp32 sum gives the same, and the comparison is bit for bit."""
import numpy as np
import pytest
import torch

from paper_2406_06858_amd import binding as fb
from paper_2406_06858_amd import inputs as fi

import gpu_harness as gh
from test_gpu_strides import _rs_call, _say

pytestmark = pytest.mark.gpu


def _check(M, N, K, R, dtype, cfg, nk, pads, rank):
    w = fi.Workload("peers_first", "rs", M, N, K, R, partial_dtype=dtype, out_dtype=dtype, a_dist=("int", 2), b_dist=("int", 2),
                    peer_dist=("int", 8), seed=M + N + K + R)
    A, B, peers = fi.make_rs_inputs(w, rank)
    _, want = gh.oracle_rs(w, rank, A, B, peers)
    _say("peers first", (M, N, K, R), dtype, "cfg", cfg, "nk", nk)
    _, outs = _rs_call(w, rank, A, B, peers, pads, tile_config=cfg, nk=nk)
    for r in range(R):
        gh.assert_bits_equal(outs[r][1], want[r], f"{(M, N, K, R)} slice {r}")


@pytest.mark.parametrize("R,dtype", [(2, "bf16"), (5, "bf16"), (8, "bf16"), (9, "bf16"), (16, "bf16"), (8, "f32")])
@pytest.mark.parametrize("cfg", [1, 2, 3])
def test_half_of_the_tiles_add_their_peers_first(cfg, R, dtype):
    bm, bn, _ = fb.flux_tile_config_info(cfg)
    for M, N, K in [(4 * bm, 5 * bn, 64), (4 * bm - 8, 5 * bn - 8, 136)]:          # 20 tiles: groups of eight, eight and four
        _check(M // R * R, N, K, R, dtype, cfg, R % 2 == 0, (8, 16, 8), R - 1)


@pytest.mark.parametrize("K,pad", [(5120, 0), (5112, 8), (4096, 1024)])
@pytest.mark.parametrize("nk", [False, True])
def test_a_asked_for_ahead_of_the_main_loop(K, pad, nk):
    """Rows of A a multiple of 2 KB apart, 256x128 tiles: rows and K that no batch of lines divides."""
    _check(264, 392, K, 2, "bf16", 2, nk, (pad, 0, 0), 1)


def test_a_asked_for_by_the_first_round_of_several():
    """Two rounds of 256x128 tiles, the second cut along K: 256 workgroups ask for all of A, the others for nothing."""
    p = fb.problem(2304, 4096, 5120, 2, 1, tile_config=2)
    full, cut, parts = fb.flux_split_plan(fb.FLUX_OP_RS, p)
    assert full == 256 and cut * parts > 0
    _check(2304, 4096, 5120, 2, "bf16", 2, False, (0, 0, 0), 1)


def _run(M, N, K, R, rank, cfg, A, B, others, flags=0):
    """The whole [M,N] result for `others`, the R-1 peers' partials in ascending rank."""
    p = fb.problem(M, N, K, R, rank, "bf16", "bf16", cfg, 1, flags)
    peers = list(others)
    peers.insert(rank, None)
    out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=gh.DEV)
    fb.flux_gemm_rs(p, A, B, peers, [out[r * (M // R):(r + 1) * (M // R)] for r in range(R)])
    torch.cuda.synchronize()
    return out


def _peers_come_first(M, N, R, bm, bn):
    """Per element: every second row of tiles where a slice is two tiles high or more, else every second column."""
    S = M // R
    rows, cols = torch.arange(M, device=gh.DEV) // bm, torch.arange(N, device=gh.DEV) // bn
    return (rows % 2 == 1)[:, None].expand(M, N) if S % bm == 0 and S >= 2 * bm else (cols % 2 == 1)[None, :].expand(M, N)


def _normal(gen, shape, std=1.0):
    return (torch.randn(shape, generator=gen) * std).bfloat16().to(gh.DEV)


@pytest.mark.parametrize("R", [2, 8])
@pytest.mark.parametrize("cfg", [1, 2, 3])
def test_results_do_not_depend_on_the_order_of_visits(cfg, R):
    """Which tiles add their peers first follows from where they lie in the result: the rank and the flags that change the
    order of visits change no bit."""
    bm, bn, _ = fb.flux_tile_config_info(cfg)
    M, N, K = 4 * bm, 6 * bn, 1024
    gen = torch.Generator().manual_seed(cfg * 10 + R)
    A, B, others = _normal(gen, (M, K)), _normal(gen, (K, N), 0.02), [_normal(gen, (M, N)) for _ in range(R - 1)]
    _say("order of visits", (M, N, K, R), "cfg", cfg)
    want = _run(M, N, K, R, 0, cfg, A, B, others)
    for rank, flags in [(0, fb.FLUX_FLAG_NO_SWIZZLE), (0, fb.FLUX_FLAG_NO_XCD_REMAP), (1, 0), (R - 1, 0), (R - 1, fb.FLUX_FLAG_NO_SWIZZLE)]:
        got = _run(M, N, K, R, rank, cfg, A, B, others, flags)
        assert torch.equal(got.view(torch.int16), want.view(torch.int16)), (rank, flags)


@pytest.mark.parametrize("R", [3, 9])
@pytest.mark.parametrize("cfg", [1, 2, 3])
def test_which_tiles_add_their_peers_first(cfg, R):
    """-v of the product, two peers of v each, v above half of the largest fp32: v where the product comes first, infinity where
    the peers do."""
    bm, bn, _ = fb.flux_tile_config_info(cfg)
    for S in (2 * bm, bm - 8):
        M, N, K = R * S, 4 * bn, 64
        v = 2.0 ** 127
        A, B = torch.zeros((M, K), dtype=torch.bfloat16, device=gh.DEV), torch.zeros((K, N), dtype=torch.bfloat16, device=gh.DEV)
        A[:, 5], B[5, :] = 1.0, -v
        others = [torch.full((M, N), v if j < 2 else 0.0, dtype=torch.bfloat16, device=gh.DEV) for j in range(R - 1)]
        _say("which tiles", (M, N, K, R), "cfg", cfg)
        got = _run(M, N, K, R, 1, cfg, A, B, others).double()
        first = _peers_come_first(M, N, R, bm, bn)
        assert torch.equal(got, torch.where(first, float("inf"), v).to(got)), (M, N)
        assert bool(first.any()) and not bool(first.all())


@pytest.mark.parametrize("R", [4, 12])
@pytest.mark.parametrize("cfg", [1, 2, 3])
def test_infinities_nan_and_denormals_among_peers_and_products(cfg, R):
    bm, bn, _ = fb.flux_tile_config_info(cfg)
    M, N, K = R * (bm // 4), 3 * bn, 192
    gen = torch.Generator().manual_seed(cfg + R)
    A, B, others = _normal(gen, (M, K)), _normal(gen, (K, N), 0.02), [_normal(gen, (M, N)) for _ in range(R - 1)]
    inf, nan = float("inf"), float("nan")
    A[3, 5], A[bm - 1, 7], B[11, 2], B[12, bn + 9] = inf, nan, -inf, inf
    for c in (0, bn, 2 * bn):
        others[0][17, c + 4], others[1][17, c + 5], others[R - 2][17, c + 6] = inf, -inf, nan
        others[0][18, c + 4], others[1][18, c + 4] = inf, -inf             # NaN
        others[0][3, c + 8], others[1][3, c + 9] = inf, -inf               # beside a row of infinite products
    _say("infinities", (M, N, K, R), "cfg", cfg)
    got = _run(M, N, K, R, R - 2, cfg, A, B, others).cpu().double()
    want = A.cpu().double() @ B.cpu().double()
    for t in others:
        want += t.cpu().double()
    assert torch.equal(got.isnan(), want.isnan()) and bool(want.isnan().any())
    assert torch.equal(torch.where(got.isinf(), got, 0.0), torch.where(want.isinf(), want, 0.0)) and bool(want.isinf().any())
    keep = want.isfinite()
    gh.assert_close(got[keep], want[keep].numpy(), "bf16")
    # peers below the smallest normal number, on their own: their sum, exactly
    tiny = 2.0 ** -133
    others = [torch.full((M, N), tiny * (j % 3 + 1), dtype=torch.bfloat16, device=gh.DEV) for j in range(R - 1)]
    got = _run(M, N, K, R, R - 2, cfg, torch.zeros_like(A), _normal(gen, (K, N), 0.02), others).cpu().double()
    assert torch.equal(got, torch.full_like(got, tiny * sum(j % 3 + 1 for j in range(R - 1))))


@pytest.mark.parametrize("cfg,R", [(1, 8), (2, 16), (3, 8)])
def test_peers_much_larger_than_products_over_a_long_k(cfg, R):
    """fp32 sums of peers around 100 and products around 1, K/32 steps: against fp64, both kinds of tiles within the rounding of the
    result and of (K / 32 + R) fp32 additions at the size of the peers' sum."""
    bm, bn, _ = fb.flux_tile_config_info(cfg)
    M, N, K = 2 * R * 8 * (bm // 64), 2 * bn, 8192
    gen = torch.Generator().manual_seed(cfg)
    A, B, others = _normal(gen, (M, K)), _normal(gen, (K, N), 0.011), [_normal(gen, (M, N), 100.0) for _ in range(R - 1)]
    _say("large peers", (M, N, K, R), "cfg", cfg)
    got = _run(M, N, K, R, 1, cfg, A, B, others).double().cpu()
    want = A.cpu().double() @ B.cpu().double()
    size = want.abs()
    for t in others:
        want += t.cpu().double()
        size += t.cpu().double().abs()
    bound = 2.0 ** -8 * want.abs() + (K / 32 + R) * 2.0 ** -24 * size * 2
    assert bool(((got - want).abs() <= bound).all())
    first = _peers_come_first(M, N, R, bm, bn).cpu()
    rel = [float((got - want)[k].norm() / want[k].norm()) for k in (first, ~first)]
    assert max(rel) < 2e-3, rel            # one rounding to bf16: 1.66e-3 in the 2-norm
