"""Reduce-scatter tiles that add their peers ahead of the main loop (every second group of eight large tiles), and A asked for
ahead of it: whole and ragged tiles, up to eight ranks and more, both dtypes, both layouts of B, row pitches.
Integer inputs whose sums stay below 2^24: any order of an fp32 sum gives the same, and the comparison is bit for bit."""
import pytest

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
