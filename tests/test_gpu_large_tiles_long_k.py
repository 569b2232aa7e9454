"""AllGather calls whose 256x256 tiles the library cuts along a long K by itself, with and without the transfer inside the main
loops, and transfers carried through an odd number of K slabs (the loop that carries takes them two at a time).
Integer inputs whose sums stay below 2^24: the comparison is bit for bit."""
import numpy as np
import pytest

from paper_2406_06858_amd import binding as fb
from paper_2406_06858_amd import inputs as fi

import gpu_harness as gh
from test_gpu_strides import _say

pytestmark = pytest.mark.gpu


def _check(w, rank, cfg=0, gbps=0, in_place=False):
    chunks, B, arrival = fi.make_ag_inputs(w, rank)
    _, want = gh.oracle_ag(w, chunks, B)
    Cg, A_agg, signals, status = gh.run_ag(w, rank, chunks, B, arrival, tile_config=cfg, link_gbps=gbps, local_in_place=in_place, repeat=2)
    assert status == (fb.FLUX_OK, 0)
    gh.assert_bits_equal(Cg, want, "C")
    gh.assert_bits_equal(A_agg, np.concatenate([fi.to_numpy(c) for c in chunks]), "A_agg")
    assert signals.tolist() == [int(r == rank) for r in range(w.R)]


@pytest.mark.parametrize("M,N,K,R,gbps,plan", [(768, 6144, 8192, 3, 0, (0, 72, 3)), (768, 6144, 8192, 3, 400, (0, 72, 3)), (264, 4240, 7400, 8, 0, (0, 34, 7)),
                                               (3256, 1264, 9224, 2, 0, (0, 65, 2))])
def test_tiles_cut_along_a_long_k(M, N, K, R, gbps, plan):
    p = fb.problem(M, N, K, R, 1, link_gbps=gbps)
    shape = fb.flux_tile_shape(fb.FLUX_OP_AG, p)
    assert (shape.tile_m, shape.tile_n) == (256, 256) and fb.flux_split_plan(fb.FLUX_OP_AG, p) == plan
    assert fb.flux_ag_deferred_tiles(p) == (R - 1 if gbps else 0)
    w = fi.Workload("long_k", "ag", M, N, K, R, a_dist=("int", 2), b_dist=("int", 2), seed=M + K)
    _say("ag long K", (M, N, K, R), "gbps", gbps)
    _check(w, 1, gbps=gbps, in_place=R == 8)


@pytest.mark.parametrize("K", [64, 192, 2112])
def test_transfer_carried_through_an_odd_number_of_slabs(K):
    p = fb.problem(1024, 512, K, 4, 2, tile_config=1, split_k=1, link_gbps=400)
    assert fb.flux_ag_deferred_tiles(p) == 3
    w = fi.Workload("odd_slabs", "ag", 1024, 512, K, 4, a_dist=("int", 2), b_dist=("int", 2), seed=K)
    _say("ag carried, K", K)
    chunks, B, arrival = fi.make_ag_inputs(w, 2)
    _, want = gh.oracle_ag(w, chunks, B)
    Cg, _, _, status = gh.run_ag(w, 2, chunks, B, arrival, tile_config=1, split_k=1, link_gbps=400, repeat=2)
    assert status == (fb.FLUX_OK, 0)
    gh.assert_bits_equal(Cg, want, "C")
