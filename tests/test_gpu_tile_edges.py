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
