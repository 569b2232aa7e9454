"""Reduce-scatter ends by type: fp32 partials with bf16 results (a lane's 8 columns stored as twice 4), and the resident kernel, which is built
for a type of the partials and for up to 4 ranks or for more.  Integer inputs whose sums stay below 2^24: bit for bit."""
import pytest
import torch

from paper_2406_06858_amd import binding as fb
from paper_2406_06858_amd import inputs as fi

import gpu_harness as gh
import test_gpu_strides as strides
from test_gpu_strides import _say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg", range(1, 11))
@pytest.mark.parametrize("R", [1, 2, 3, 4, 5, 8, 9, 16])
def test_fp32_partials_with_bf16_results(R, cfg):
    for M, N, K in ((16 * R, 136, 200), (256 * R, 256, 128)):        # edges in every direction; tiles that divide it
        for split in (1, 3):
            w = fi.Workload("f32_bf16", "rs", M, N, K, R, "f32", "bf16", a_dist=("int", 2), b_dist=("int", 2), peer_dist=("int", 4), seed=M + R + cfg)
            rank = (cfg + M) % R
            A, B, peers = fi.make_rs_inputs(w, rank)
            _say("fp32 partials, bf16 results", (M, N, K), "R", R, "cfg", cfg, "split", split)
            outs = gh.run_rs(w, rank, A, B, peers, tile_config=cfg, split_k=split)
            want = A.to(gh.DEV).float() @ B.to(gh.DEV).float()
            for t in peers:
                if t is not None:
                    want += t.to(gh.DEV).float()
            assert torch.equal(torch.cat(outs), want.to(outs[0].dtype))


@pytest.mark.parametrize("pads", [(8, 16, 24), (64, 0, 0), (0, 128, 0), (0, 0, 8)])
@pytest.mark.parametrize("shape", list(strides.RS_SHAPES))
def test_fp32_partials_with_bf16_results_and_row_pitches(shape, pads):
    strides.test_rs_with_row_pitches(shape, pads, "f32", "bf16")


@pytest.mark.parametrize("R,pd,od", [(2, "f32", "f32"), (4, "f32", "bf16"), (8, "f32", "f32"), (8, "f32", "bf16"), (16, "f32", "f32"), (16, "bf16", "f32")])
def test_resident_grid_by_type_of_the_partials(R, pd, od):
    w = fi.Workload("resident_by_type", "rs", 8192, 8192, 192, R, pd, od)
    assert fb.flux_rs_resident_grid(fb.problem(w.M, w.N, w.K, R, 1, pd, od))[0] == 256
    gen = torch.Generator(device=gh.DEV).manual_seed(R)
    draw = lambda shape, top, dt: torch.randint(-top, top + 1, shape, generator=gen, device=gh.DEV, dtype=torch.int32).to(dt)
    A, B = draw((w.M, w.K), 2, torch.bfloat16), draw((w.K, w.N), 2, torch.bfloat16)
    peers = [None if r == 1 else draw((w.M, w.N), 4, torch.float32 if pd == "f32" else torch.bfloat16) for r in range(R)]
    _say("resident, ranks", R, pd, od)
    outs = gh.run_rs(w, 1, A, B, peers)
    want = A.float() @ B.float()
    for t in peers:
        if t is not None:
            want += t.float()
    assert torch.equal(torch.cat(outs), want.to(outs[0].dtype))
