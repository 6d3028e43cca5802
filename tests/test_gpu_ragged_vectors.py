"""One iteration on vectors whose length sits at the edges of the kernels' pieces -- a tile of pass 1 (2^14 coordinates),
a tile of the update (1024), a workgroup of the tail (8192), groups of four --, so that most workers start off a 16-byte
boundary; with as many workers as the update shares out over workgroups, and with tiles in more than one group."""
import pytest

from tests.test_gpu_random_shapes import DEFAULTS, one_iteration

pytestmark = pytest.mark.gpu

SHAPES = [  # d, n, r, c, k
    (16_381, 3, 5, 40_000, 300), (16_383, 5, 4, 40_000, 16_383), (16_385, 4, 3, 40_000, 1), (16_386, 3, 2, 40_000, 4_000),
    (32_771, 5, 1, 33_000, 8_192), (49_155, 2, 6, 50_000, 49_155),
    (1_023, 17, 2, 20_000, 5), (1_025, 16, 3, 20_000, 1_025), (8_193, 33, 2, 17_000, 70), (7, 40, 2, 17_000, 3),
    (2_900_003, 2, 16, 70_001, 900),                                 # tiles of 2^12: two groups per XCD, the last a small one
]


@pytest.mark.parametrize("fuse_head", [0, 2], ids=["separate-head", "fused-head-per-worker"])
@pytest.mark.parametrize("d,n,r,c,k", SHAPES)
def test_lengths_at_the_edges_of_tiles(d, n, r, c, k, fuse_head):
    from paper_2210_07454_amd import sams
    sams.load()
    tun = dict(DEFAULTS, fuse_head=fuse_head, tile_log2=14 if 16_000 < d < 50_000 else 0)
    try:
        for key, val in tun.items():
            sams.sams_configure(key, val)
        assert one_iteration(sams, (d, n, r, c, k), seed=d % 97)
    finally:
        for key, val in DEFAULTS.items():
            sams.sams_configure(key, val)


def fused(d, n, r, c, pa):
    """whether the update also stages its vector, by the kernels that it launches"""
    import torch
    from paper_2210_07454_amd import inputs, sams
    sams.sams_configure("fuse_head", 2)
    try:
        with sams.Context(d, n, r, c, 4, inputs.hash_params(r)) as ctx:
            g, m, e = (torch.zeros(n, d, device="cuda") for _ in range(3))
            v, vhat = (torch.ones((n, d) if pa else (d,), device="cuda") for _ in range(2))
            update = ctx.amsgrad_ef_update_pa if pa else ctx.amsgrad_ef_update
            ctx.sams_profile_enable(True)
            update(g, m, e, v, vhat, torch.zeros(d, device="cuda"), None, None, 0, 0.9, 0.99, 1e-3)
            ctx.sams_profile_enable(False)
            return "k_head_scatter" in ctx.sams_profile_read()
    finally:
        sams.sams_configure("fuse_head", 0)


def test_ragged_vectors_fuse_the_head_only_where_that_is_faster():
    long = 1 << 24
    assert fused(300_000, 2, 3, 40_000, False) and fused(300_000, 2, 3, 40_000, True)
    assert fused(long + 1, 1, 2, 40_000, False) and fused(long + 4, 1, 2, 40_000, True)
    assert not fused(300_001, 2, 3, 40_000, False) and not fused(300_001, 2, 3, 40_000, True)
    assert not fused(long - 1, 1, 2, 40_000, False) and not fused(long + 1, 1, 2, 40_000, True)


@pytest.mark.parametrize("d,n,r,c,k,fuse_head", [
    ((1 << 24) + 1, 3, 2, 70_001, 20_000, 2), ((1 << 24) + 8_195, 2, 7, 200_003, 3_000, 2),
    ((1 << 24) + 1, 2, 1, 70_001, 20_000, 0), (1 << 23, 4, 1, 70_001, 20_000, 0), ((1 << 23) - 1, 4, 1, 70_001, 20_000, 0)])
def test_long_ragged_vectors(d, n, r, c, k, fuse_head):
    """the fused head: tiles of 2^14 and of 2^13 (half of its turns), a last tile of one coordinate and of three; the separate
    one: a worker per workgroup, and all workers"""
    from paper_2210_07454_amd import sams
    try:
        sams.sams_configure("fuse_head", fuse_head)
        assert one_iteration(sams, (d, n, r, c, k), seed=d % 97)
    finally:
        sams.sams_configure("fuse_head", 0)


@pytest.mark.parametrize("d,c,extra", [(60_000, 40_000, True), (60_000, 400, False), (60_001, 40_000, False), (6_000_000, 500, False)])
def test_room_for_the_compacted_gradients_only_where_the_head_fuses(d, c, extra):
    """g of every worker on the index set and the ranks of its bitmap words: not for a context that pulls, adds up rows in LDS
    or has its head apart"""
    from paper_2210_07454_amd import inputs, sams
    n, r, k = 3, 2, d // 10
    size = {}
    try:
        for fuse_head in (0, 2):
            sams.sams_configure("fuse_head", fuse_head)
            with sams.Context(d, n, r, c, k, inputs.hash_params(r)) as ctx:
                size[fuse_head] = ctx.scratch_bytes
    finally:
        sams.sams_configure("fuse_head", 0)
    assert size[2] - size[0] == (4 * n * k + (d + 31) // 32 * 4 if extra else 0)


@pytest.mark.parametrize("d,n,r,c,k,apart", [(300_001, 2, 3, 40_000, 700, True), (300_003, 2, 16, 40_000, 3_000, True),
                                             (1_100_001, 8, 4, 90_000, 11_000, False)])
def test_recovery_of_ragged_vectors(d, n, r, c, k, apart):
    """row estimates through memory where the tiles are many and small, in registers elsewhere: one iteration bit for bit"""
    import torch
    from paper_2210_07454_amd import inputs, sams
    try:
        sams.sams_configure("estimate_path", 2)
        assert one_iteration(sams, (d, n, r, c, k), seed=d % 97)
        with sams.Context(d, n, r, c, k, inputs.hash_params(r)) as ctx:
            ctx.sams_profile_enable(True)
            ctx.unsketch_estimates(torch.ones(r, c, device="cuda"), None, torch.empty(d, device="cuda"))
            ctx.sams_profile_enable(False)
            assert ("k_est_median" in ctx.sams_profile_read()) == apart
    finally:
        sams.sams_configure("estimate_path", 0)


@pytest.mark.parametrize("n", [1, 2, 3, 4, 9, 10, 17, 18, 33])
@pytest.mark.parametrize("r,c", [(3, 333), (3, 100_001), (4, 70_001)])
def test_mean_of_any_number_of_tables(n, r, c):
    import numpy as np
    import torch
    from oracle import Oracle
    from paper_2210_07454_amd import inputs, sams
    S = np.random.default_rng(n).standard_normal((n, r, c)).astype(np.float32)
    mean = torch.empty(r, c, device="cuda")
    with sams.Context(1_000, n, r, c, 1, inputs.hash_params(r)) as ctx:
        ctx.sketch_reduce(torch.from_numpy(S).cuda(), mean)
    assert np.array_equal(mean.cpu().numpy(), Oracle("f32").sketch_mean(S))


@pytest.mark.parametrize("d,n,r,c,k", [(300_001, 17, 2, 40_000, 4_687), (300_001, 17, 2, 40_000, 4_688), (261_121, 3, 1, 40_000, 261_121),
                                       (261_120, 3, 1, 40_000, 9_000), (2_200_000, 5, 1, 40_000, 500)])
def test_update_with_many_members(d, n, r, c, k):
    """the second moments on the index set by workgroups of their own, and (from 256 tiles on, more than 1 in 64 coordinates; or
    enough tiles for all workers of one to be together) by those that have all workers"""
    from paper_2210_07454_amd import sams
    assert one_iteration(sams, (d, n, r, c, k), seed=d % 97)
