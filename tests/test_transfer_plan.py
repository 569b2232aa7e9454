"""Which transfer flux_ag_gemm plans where A has to be gathered first: grids of several rounds with fewer than eight columns of 256x256
tiles, too few for the tiles to read A from the chunk sources and store it on the way."""
from paper_2406_06858_amd import binding as fb

NARROW = (16384, 1792, 12288, 8, 2)              # 1.75 rounds of seven columns of tiles; the first covers 5 bands of 56


def test_deferred_transfer_of_narrow_grids():
    deferred = lambda *a, **kw: fb.flux_ag_deferred_tiles(fb.problem(*a, **kw))
    sh = fb.flux_tile_shape(fb.FLUX_OP_AG, fb.problem(*NARROW))
    assert 32 * -(-NARROW[1] // sh.tile_n) < sh.tile_m
    assert deferred(*NARROW) == 3
    assert deferred(12288, 1792, 12288, 8, 2) == 1                       # bands of 42 tiles
    for kw in (dict(flags=fb.FLUX_FLAG_AG_COPY_UPFRONT), dict(flags=fb.FLUX_FLAG_NO_SWIZZLE), dict(comm_tiles_per_chunk=2),
               dict(copy_workgroups=16), dict(tile_config=2), dict(lda=12288 + 64)):
        assert deferred(*NARROW, **kw) == 0, kw
    assert deferred(*NARROW, lda=12288, ldb=1792 + 64, ldc=1792 + 8) == 3
    assert deferred(9216, 1792, 12288, 8, 2, tile_config=1) == 0         # one round: every chunk is needed at once
    assert deferred(16384, 1792, 12288, 2, 0) == 0                       # the first round touches every chunk
    assert deferred(16384, 1792, 512, 8, 2) == 0                         # K too short to carry the vectors
    assert deferred(16384, 1792, 12288, 1, 0) == 0
