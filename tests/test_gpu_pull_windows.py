"""sketch_accumulate by lists of one and of four slices of 64 buckets, with up to two of the former and four of the latter per wavefront, rows
sharing the windows by the length of their lists: tables bit for bit those of a sequential loop (up to 2^22 coordinates; above, exact where partial sums are)."""
import numpy as np
import pytest
import torch

from oracle import Oracle
from paper_2210_07454_amd import inputs

pytestmark = pytest.mark.gpu


def sketch(u, hp, c, lists=0):
    """lists: the tunable "pull_lists"; with one, the context has to pull."""
    from paper_2210_07454_amd import sams
    n, d = u.shape
    S = torch.full((n, hp.shape[0], c), 9.0, device="cuda")
    sams.sams_configure("pull_lists", lists)
    try:
        ctx = sams.Context(d, n, hp.shape[0], c, 1, hp)
    finally:
        sams.sams_configure("pull_lists", 0)
    with ctx:
        ctx.sams_profile_enable(True)
        ctx.sketch_accumulate(torch.from_numpy(u).cuda(), S)
        ctx.sams_profile_enable(False)
        assert not lists or "k_sketch_pull" in ctx.sams_profile_read()
        return S.cpu().numpy()


def uneven(r, c, rows):
    """Hash parameters under which the given rows crowd a tile's coordinates into about a quarter of the buckets."""
    hp = inputs.hash_params(r, seed=3)
    for j in rows:
        hp[j, 0] = (2 ** 31 - 1) // 4 + 1                            # four coordinates on, almost the same hash value
    return hp


# buckets around whole lists (256; one list, one and a bit, five), whole windows (896, 1,792, 3,584: lists for every wavefront) and the widest;
# few and many pairs
@pytest.mark.parametrize("lists", [1, 2, 4])
@pytest.mark.parametrize("d,n,r,c", [(26_617, 80, 3, 255), (26_609, 90, 3, 257), (13_309, 3, 2, 128), (26_611, 2, 2, 1_100), (26_613, 256, 1, 896), (13_310, 86, 3, 897), (30_003, 128, 2, 1_792), (26_627, 64, 4, 1_793), (40_001, 30, 5, 1_025), (30_011, 60, 5, 3_583), (30_013, 60, 5, 3_585), (13_309, 130, 4, 7_169),
                                     (40_003, 75, 4, 10_753), (26_615, 64, 5, 14_336), (13_305, 256, 1, 16_384), (53_217, 32, 9, 8_191)])
def test_lists_of_one_and_of_four_slices(d, n, r, c, lists):
    rng = np.random.default_rng(d + c)
    u = (rng.standard_normal((n, d)) * 10.0 ** rng.uniform(-3, 1, d)).astype(np.float32)
    hp = inputs.hash_params(r, seed=c % 91)
    got = sketch(u, hp, c, lists)
    o = Oracle("f32")
    for i in range(n):
        assert np.array_equal(got[i].view(np.uint32), o.sketch(u[i], hp, c).view(np.uint32)), i


@pytest.mark.parametrize("lists", [0, 1, 2, 4])
@pytest.mark.parametrize("d,n,r,c,rows", [(40_001, 20, 4, 9_001, (1,)), (26_623, 40, 5, 6_000, (0, 4)), (30_001, 50, 3, 2_049, (2,)), (39_915, 7, 5, 12_345, (1, 2, 3))])
def test_rows_with_windows_of_their_own(d, n, r, c, rows, lists):
    rng = np.random.default_rng(d)
    u = rng.standard_normal((n, d)).astype(np.float32)
    hp = uneven(r, c, rows)
    got = sketch(u, hp, c, lists)
    o = Oracle("f32")
    for i in range(n):
        assert np.array_equal(got[i].view(np.uint32), o.sketch(u[i], hp, c).view(np.uint32)), i


@pytest.mark.parametrize("lists", [1, 2, 4])
@pytest.mark.parametrize("d,n,r,c,rows", [((1 << 22) + 7, 3, 4, 10_000, (2,)), (4_300_001, 2, 3, 16_384, ()), (4_194_311, 5, 2, 5_000, (0,))])
def test_parts_with_windows_of_their_own(d, n, r, c, rows, lists):
    rng = np.random.default_rng(d)
    u = rng.integers(-3, 4, (n, d)).astype(np.float32)               # every partial sum is a whole number below 2^24
    hp = uneven(r, c, rows)
    got = sketch(u, hp, c, lists)
    o = Oracle("f32")
    for i in range(n):
        assert np.array_equal(got[i], o.sketch(u[i], hp, c)), i


# tables around 2^14 and 2^15 buckets under vectors around 2^18 coordinates, where the choice between the paths changes: by either, the same bits
@pytest.mark.parametrize("d,n,r,c", [
    (262_144, 4, 3, 16_385), (262_143, 4, 3, 16_385), (300_001, 2, 2, 32_767), (300_007, 3, 5, 20_001), (280_001, 16, 2, 32_768),
    (280_003, 2, 2, 32_769), ((1 << 22) + 9, 2, 2, 32_768)])
@pytest.mark.parametrize("lists", [0, 1, 2, 4])
def test_wide_tables(d, n, r, c, lists):
    rng = np.random.default_rng(d + c)
    hp = inputs.hash_params(r, seed=8)                               # no row of long lists, for which none are made
    whole = d > 1 << 22                                              # the order of the additions is not promised
    u = rng.integers(-3, 4, (n, d)).astype(np.float32) if whole else rng.standard_normal((n, d)).astype(np.float32)
    got = sketch(u, hp, c, lists if c <= 1 << 15 else 0)
    o = Oracle("f32")
    for i in range(n):
        ref = o.sketch(u[i], hp, c)
        assert np.array_equal(got[i], ref) if whole else np.array_equal(got[i].view(np.uint32), ref.view(np.uint32)), i
