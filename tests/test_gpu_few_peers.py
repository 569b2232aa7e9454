"""GEMM-ReduceScatter epilogues by number of ranks: built for 3, 7 and 15 peers, and for 1, 3 and 7 where small whole tiles ask for their
peers' rows ahead of the main loop.  Both sides of every border, whole and K-cut tiles, every configuration.  Integer inputs whose
sums stay below 2^24: bit for bit."""
import pytest
import torch

from paper_2406_06858_amd import binding as fb
from paper_2406_06858_amd import inputs as fi

import gpu_harness as gh
from test_gpu_strides import _say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg", range(1, 11))
@pytest.mark.parametrize("R", [1, 2, 3, 4, 5, 8, 9, 16])
def test_every_number_of_peers(R, cfg):
    for M, N, K in ((16 * R, 136, 200), (256 * R, 256, 128)):        # edges in every direction; tiles that divide it
        for split in (1, 3):
            for pd, od in (("bf16", "bf16"), ("f32", "f32"), ("bf16", "f32")):
                w = fi.Workload("few_peers", "rs", M, N, K, R, pd, od, a_dist=("int", 2), b_dist=("int", 2), peer_dist=("int", 4), seed=M + R + cfg)
                rank = (cfg + M) % R
                A, B, peers = fi.make_rs_inputs(w, rank)
                _say("few peers", (M, N, K), "R", R, "cfg", cfg, "split", split, pd, od)
                outs = gh.run_rs(w, rank, A, B, peers, tile_config=cfg, split_k=split)
                want = A.to(gh.DEV).float() @ B.to(gh.DEV).float()
                for t in peers:
                    if t is not None:
                        want += t.to(gh.DEV).float()
                assert torch.equal(torch.cat(outs), want.to(outs[0].dtype))


def test_many_short_tiles_of_few_ranks():
    """The resident kernel is built for up to 4 ranks and for more."""
    for R in (2, 4, 8):
        w = fi.Workload("few_peers_resident", "rs", 8192, 8192, 128, R, a_dist=("int", 2), b_dist=("int", 2), peer_dist=("int", 4), seed=R)
        p = fb.problem(w.M, w.N, w.K, R, 1)
        assert fb.flux_rs_resident_grid(p)[0] == 256
        A, B, peers = fi.make_rs_inputs(w, 1)
        _say("resident, ranks", R)
        outs = gh.run_rs(w, 1, A, B, peers)
        want = A.to(gh.DEV).float() @ B.to(gh.DEV).float()
        for t in peers:
            if t is not None:
                want += t.to(gh.DEV).float()
        assert torch.equal(torch.cat(outs), want.to(outs[0].dtype))
