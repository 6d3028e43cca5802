"""sketch_accumulate of narrow tables (128 to 2^14 buckets), where the workgroups pull their coordinates from tiles of the
vector: tables bit for bit those of a sequential loop, at the edges of tiles (13,308 coordinates), slices (64 buckets)
and windows, for workers that start off a 16-byte boundary, and where the path has to step back."""
import numpy as np
import pytest
import torch

from oracle import Oracle
from paper_2210_07454_amd import inputs

pytestmark = pytest.mark.gpu

SHAPES = [  # d, n, r, c
    (13_308, 2, 3, 128), (13_309, 3, 2, 129), (13_307, 3, 2, 191), (26_617, 5, 1, 16_384), (79_851, 3, 3, 10_007),
    (1, 5, 2, 128), (2, 4, 1, 200), (63, 5, 3, 4_096), (13_310, 90, 3, 400), (13_311, 130, 2, 1_999), (39_927, 67, 4, 2_040),
    (30_001, 70, 8, 9_000), (100_000, 2, 16, 5_000), (130_563, 1, 1, 16_383), (20_011, 300, 1, 700), (12_345, 150, 2, 16_000),
    (40_001, 20, 16, 3_457), (53_231, 100, 3, 8_003), (26_615, 87, 3, 14_337),   # several slices per wavefront, ragged ones too
]


def check(d, n, r, c, hp, seed):
    from paper_2210_07454_amd import sams
    rng = np.random.default_rng(seed)
    u = (rng.standard_normal((n, d)) * 10.0 ** rng.uniform(-3, 1, d)).astype(np.float32)
    u[:, ::7] *= np.float32(0.0)                                     # zeros of both signs
    S = torch.full((n, r, c), 9.0, device="cuda")
    with sams.Context(d, n, r, c, 1, hp) as ctx:
        assert ctx.sketch_mode == 2
        ctx.sketch_accumulate(torch.from_numpy(u).cuda(), S)
        got = S.cpu().numpy()
        ctx.sams_profile_enable(True)
        ctx.sketch_accumulate(torch.from_numpy(u).cuda(), S)
        ctx.sams_profile_enable(False)
        kernels = set(ctx.sams_profile_read())
    o = Oracle("f32")
    for i in range(n):
        assert np.array_equal(got[i].view(np.uint32), o.sketch(u[i], hp, c).view(np.uint32)), i
    return kernels


@pytest.mark.parametrize("d,n,r,c", SHAPES)
def test_narrow_tables_bit_exact(d, n, r, c):
    assert check(d, n, r, c, inputs.hash_params(r, seed=d % 89), d) == {"k_sketch_pull"}


def test_a_hash_that_crowds_the_buckets_takes_the_binned_path():
    """a = c: every coordinate whose product stays below the modulus falls into one bucket."""
    hp = inputs.hash_params(2, seed=1)
    hp[0, 0] = 1_000
    assert "k_sketch_pull" not in check(40_000, 2, 2, 1_000, hp, 3)


@pytest.mark.parametrize("c", [127, 16_385])
def test_tables_outside_the_range_take_the_binned_path(c):
    assert "k_sketch_pull" not in check(33_000, 2, 2, c, inputs.hash_params(2, seed=4), 5)


@pytest.mark.parametrize("d,n,r,c", [((1 << 22) + 1, 3, 2, 130), ((1 << 22) + 3, 1, 3, 4_097), (4_205_329, 2, 1, 16_384),
                                     (4_205_327, 5, 4, 10_007), (8_516_119, 1, 1, 897)])
def test_long_vectors_in_parts(d, n, r, c):
    """Above 2^22 coordinates the vector may be cut into parts: exact where the partial sums are, reproducible, and within
    the bound of sums in another order (a bucket of q terms: (q - 1) 2^-24 of the sum of their magnitudes, q about d / c)."""
    from paper_2210_07454_amd import sams
    rng = np.random.default_rng(d)
    hp = inputs.hash_params(r, seed=d % 89)
    whole = rng.integers(-3, 4, (n, d)).astype(np.float32)
    u = (rng.standard_normal((n, d)) * 10.0 ** rng.uniform(-3, 1, d)).astype(np.float32)
    S = torch.full((n, r, c), 9.0, device="cuda")
    with sams.Context(d, n, r, c, 1, hp) as ctx:
        ctx.sams_profile_enable(True)
        ctx.sketch_accumulate(torch.from_numpy(whole).cuda(), S)
        ctx.sams_profile_enable(False)
        assert "k_sketch_pull" in ctx.sams_profile_read()
        got = S.cpu().numpy()
        o = Oracle("f32")
        for i in range(n):
            assert np.array_equal(got[i], o.sketch(whole[i], hp, c)), i
        ctx.sketch_accumulate(torch.from_numpy(u).cuda(), S)
        got = S.cpu().numpy()
        ctx.sketch_accumulate(torch.from_numpy(u).cuda(), S)
        assert np.array_equal(got.view(np.uint32), S.cpu().numpy().view(np.uint32))
    o64 = Oracle("f64")
    plus = np.stack([hp[:, 0], hp[:, 1], np.full(r, 2, np.uint32), np.zeros(r, np.uint32)], axis=1).astype(np.uint32)   # every sign +1
    for i in range(n):
        mass = o64.sketch(np.abs(u[i]).astype(np.float64), plus, c)
        bound = 2.0 * d / c * 2.0 ** -24 * mass + 1e-37              # twice the average number of terms
        assert np.all(np.abs(got[i] - o64.sketch(u[i].astype(np.float64), hp, c)) <= bound), i


@pytest.mark.parametrize("d,c,pulls", [(40_000, 1_000, True), ((1 << 22) + 5, 500, True), (40_000, 127, False), (40_000, 40_000, False)])
def test_second_pass_variant_is_reported_where_there_is_one(d, c, pulls):
    """-1 from both where no second pass reads metadata: a context that pulls has no binned path."""
    from paper_2210_07454_amd import sams
    with sams.Context(d, 2, 2, c, 1, inputs.hash_params(2, seed=4)) as ctx:
        assert (ctx.accumulate_variant == -1) == pulls
        assert (ctx.record_rows == -1) == pulls


@pytest.mark.parametrize("d,n,r,c,pulls", [
    (4_000_000, 1, 1, 4_096, False), (1_000_000, 2, 3, 4_096, False), (4_000_000, 2, 3, 3_000, False), (4_000_000, 1, 1, 2_000, False),
    (4_000_000, 1, 1, 1_000, True), (431_003, 1, 1, 4_096, True), (4_000_000, 16, 5, 3_000, True), (4_000_000, 1, 1, 6_000, True),
    (4_300_000, 1, 1, 4_096, True),
    (4_000_000, 50, 5, 16_384, True), (5_000_000, 50, 5, 16_384, True), (4_000_000, 16, 5, 12_000, True), (5_000_000, 50, 5, 6_000, True)])
def test_shapes_that_pull(d, n, r, c, pulls):
    """Long vectors under a table that the binned path cuts into many windows for few pairs go the other way."""
    from paper_2210_07454_amd import sams
    u = torch.zeros(n, d, device="cuda")
    u[:, d // 2] = 1.0
    S = torch.empty(n, r, c, device="cuda")
    with sams.Context(d, n, r, c, 1, inputs.hash_params(r, seed=3)) as ctx:
        ctx.sams_profile_enable(True)
        ctx.sketch_accumulate(u, S)
        ctx.sams_profile_enable(False)
        assert ("k_sketch_pull" in ctx.sams_profile_read()) == pulls
    assert S.abs().sum(dim=2).eq(1.0).all()
