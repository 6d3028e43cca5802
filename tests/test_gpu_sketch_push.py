"""sketch_accumulate where workgroups pick their values out of the vectors, or out of sorted copies of them, by lists of words: tables bit for bit
those of a sequential loop, at the edges of phases (2,048 words; a multiple of 32 coordinates), windows and wavefronts."""
import numpy as np
import pytest
import torch

from oracle import Oracle
from paper_2210_07454_amd import inputs

pytestmark = pytest.mark.gpu

P31 = 2 ** 31 - 1


def context(d, n, r, c, hp, k=1, **tunables):
    from paper_2210_07454_amd import sams
    try:
        for key, val in tunables.items():
            sams.sams_configure(key, val)
        return sams.Context(d, n, r, c, k, hp)
    finally:
        for key in tunables:
            sams.sams_configure(key, 0)


def kernels(ctx, u, S):
    ctx.sams_profile_enable(True)
    ctx.sketch_accumulate(u, S)
    ctx.sams_profile_enable(False)
    return set(ctx.sams_profile_read())


def check(d, n, r, c, hp, windows, u=None):
    """windows: the tunable "push_windows"; returns the kernels of one sketch."""
    rng = np.random.default_rng(d + c)
    if u is None:
        u = (rng.standard_normal((n, d)) * 10.0 ** rng.uniform(-3, 1, d)).astype(np.float32)
        u[:, ::7] *= np.float32(0.0)                                 # zeros of both signs
    S = torch.full((n, r, c), 9.0, device="cuda")
    with context(d, n, r, c, hp, push_windows=windows) as ctx:
        assert ctx.sketch_mode == 2
        used = kernels(ctx, torch.from_numpy(u).cuda(), S)
        assert ctx.accumulate_variant == -1 or "k_sketch_push" not in used
    got = S.cpu().numpy()
    o = Oracle("f32")
    for i in range(n):
        ref = o.sketch(u[i], hp, c)
        assert np.array_equal(np.isnan(got[i]), np.isnan(ref))
        assert np.array_equal(got[i].view(np.uint32)[~np.isnan(ref)], ref.view(np.uint32)[~np.isnan(ref)]), i
    return used


# one window: 2,016 coordinates a phase; windows of up to and above 2^15 cells (where places have 14 bits); a vector of one coordinate, of one phase, one more
# and one less, the ring's eight phases and around; workers that do and do not fill an XCD's share
@pytest.mark.parametrize("d,n,r,c,windows", [
    (1, 2, 2, 40_800, 1), (2_016, 4, 2, 5_000, 1), (2_017, 3, 2, 4_999, 1), (2_015, 9, 1, 6_000, 1), (16_128, 2, 3, 40_800, 1), (16_129, 2, 3, 32_704, 1),
    (18_143, 1, 2, 32_705, 1), (4_033, 33, 5, 5_000, 1), (30_001, 3, 3, 65_409, 2), (40_003, 7, 2, 81_600, 2), (29_999, 2, 16, 3_000, 3), (100_003, 6, 4, 20_001, 5),
    (123_457, 4, 5, 100_000, 16), (60_000, 5, 2, 60_000, 7)])
def test_from_the_vectors(d, n, r, c, windows):
    assert check(d, n, r, c, inputs.hash_params(r, seed=d % 89), windows) == {"k_sketch_push"}


# tables so narrow that a phase has dozens of coordinates for a bucket (windows of a few buckets or none are all of this kind): the paths that they had
@pytest.mark.parametrize("d,n,r,c,windows", [
    (1, 1, 1, 1, 1), (3, 5, 2, 2, 2), (2_016, 4, 2, 64, 1), (2_017, 3, 2, 65, 1), (2_015, 9, 1, 63, 1), (250_001, 2, 3, 33, 16), (300_007, 2, 2, 17, 16),
    (5_000, 3, 2, 225, 16), (5_001, 2, 3, 241, 16)])
def test_lists_that_cannot_be_made(d, n, r, c, windows):
    assert "k_sketch_push" not in check(d, n, r, c, inputs.hash_params(r, seed=d % 89), windows)


@pytest.mark.parametrize("d,n,r,c,windows", [
    (1, 1, 1, 40_001, 102), (3_808, 4, 2, 30_000, 102), (3_809, 3, 5, 81_600, 102), (3_807, 5, 3, 9_001, 102), (100_001, 3, 10, 100_000, 103),
    (70_003, 2, 7, 50_001, 106), (200_000, 9, 5, 262_144, 109), (49_153, 2, 4, 3_000, 116), (49_152, 1, 16, 600_000, 116)])
def test_from_sorted_copies(d, n, r, c, windows):
    assert check(d, n, r, c, inputs.hash_params(r, seed=d % 83), windows) == {"k_sketch_push", "k_bin_scatter"}


# workers whose turns on an XCD are cut so that no compute unit has a workgroup more than it need have: 250, 245, 252, 243 and 510 workgroups
@pytest.mark.parametrize("d,n,r,c,windows,seed", [
    (40_003, 5, 10, 20_000, 5, 4), (40_003, 5, 10, 20_000, 105, 4), (50_001, 7, 5, 55_872, 107, 2), (45_001, 6, 14, 30_001, 3, 2), (45_002, 3, 9, 39_001, 9, 3),
    (30_001, 17, 15, 60_001, 102, 0)])
def test_workgroups_dealt_to_the_xcds(d, n, r, c, windows, seed):
    assert "k_sketch_push" in check(d, n, r, c, inputs.hash_params(r, seed=seed), windows)


def test_a_worker_more_takes_no_second_round():
    """245 workgroups fit the 256 compute units as 210 do: 1.8 times as long means that some units had two"""
    d, r, c, ms = 11_214_720, 5, 55_872, {}
    hp = inputs.hash_params(r, seed=46)
    for n in (6, 7):
        u, S = torch.randn(n, d, device="cuda"), torch.empty(n, r, c, device="cuda")
        with context(d, n, r, c, hp, push_windows=107) as ctx:
            ctx.sketch_accumulate(u, S)
            times = []
            for _ in range(7):
                ctx.sams_profile_enable(True)
                ctx.sketch_accumulate(u, S)
                ctx.sams_profile_enable(False)
                times.append(ctx.sams_profile_read()["k_sketch_push"][0])
            ms[n] = min(times)
    assert ms[7] < 1.4 * ms[6], ms


def repeating(r, c, dist, rows):
    """Hash parameters under which, in the given rows, most coordinates share the bucket with the one `dist` on."""
    hp = inputs.hash_params(r, seed=5)
    for z, j in enumerate(rows):
        hp[j, 0] = (3 + z) * c * pow(dist, -1, P31) % P31            # a * dist = (3 + z) c (mod p)
    return hp


# two to six coordinates of a phase in a bucket, for most of its buckets: with the windows for which a phase's shared buckets still find room (a bucket's
# words lie in one wavefront) by the lists, with the others by the paths that they had
@pytest.mark.parametrize("windows", [1, 3, 5, 103, 105])
@pytest.mark.parametrize("dist,rows,pushes", [
    (3_000, (1,), {1, 3, 5, 103, 105}), (1_500, (0, 2), {3, 103}), (601, (2,), {3, 5, 103, 105}), (200, (1,), set()), (97, (0,), set()), (40, (1,), set()),
    (5, (1,), set()), (1, (0, 1), set())])
def test_buckets_that_repeat_within_a_phase(dist, rows, pushes, windows):
    d, n, r, c = 50_021, 3, 3, 20_000
    used = check(d, n, r, c, repeating(r, c, dist, rows), windows)
    assert used == ({"k_sketch_push"} | ({"k_bin_scatter"} if windows > 100 else set()) if windows in pushes else {"k_bin_accumulate", "k_bin_scatter"})


@pytest.mark.parametrize("d,dist,windows", [(1_000, 97, 1), (1_000, 37, 1), (2_000, 101, 2), (3_000, 97, 3), (3_001, 97, 103), (5_000, 151, 105)])
def test_dozens_of_coordinates_of_a_phase_in_a_bucket(d, dist, windows):
    """half a phase, so that there is room: chains of 10 to 30 words that go on from lane to lane"""
    used = check(d, 3, 3, 20_000, repeating(3, 20_000, dist, (1,)), windows)
    assert used == {"k_sketch_push"} | ({"k_bin_scatter"} if windows > 100 else set())


@pytest.mark.parametrize("windows", [2, 104])
def test_infinities_and_nan_reach_their_cells_only(windows):
    d, n, r, c = 30_011, 3, 3, 20_011
    rng = np.random.default_rng(7)
    u = rng.standard_normal((n, d)).astype(np.float32)
    u[0, 5], u[1, 70], u[2, d - 1], u[2, 4_000] = np.inf, -np.inf, np.nan, np.float32(1e-44)
    check(d, n, r, c, inputs.hash_params(r, seed=8), windows, u)


# where the paths are chosen: by each of them the same bits, and the one that is meant
@pytest.mark.parametrize("d,n,r,c,kernel", [
    (262_144, 84, 5, 12_000, "k_sketch_push"), (262_143, 84, 5, 12_000, "k_sketch_pull"), (262_144, 84, 5, 10_000, "k_sketch_pull"),
    (400_009, 6, 3, 20_000, "k_sketch_pull"), (2 ** 22, 20, 5, 32_768, "k_sketch_push"), (300_001, 2, 2, 300_001, "k_bin_accumulate"), (400_003, 40, 5, 32_769, "k_sketch_push"), (1_000_001, 9, 5, 100_003, "k_sketch_push")])
def test_the_chosen_path(d, n, r, c, kernel):
    assert kernel in check(d, n, r, c, inputs.hash_params(r, seed=3), 0)


@pytest.mark.parametrize("d,n,r,c", [(997_358, 42, 3, 36_492), (538_297, 17, 5, 42_700), (609_463, 9, 3, 125_447), (886_797, 4, 4, 281_664)])
def test_a_head_that_does_not_fuse_changes_no_choice(d, n, r, c):
    """d no multiple of four: pass 1 writes the copies whatever "fuse_head" says, so the path and its windows are those of "fuse_head" 0"""
    hp = inputs.hash_params(r, seed=1)
    u, S = torch.randn(n, d, device="cuda"), torch.empty(n, r, c, device="cuda")
    seen = []
    for fuse_head in (0, 2):
        with context(d, n, r, c, hp, fuse_head=fuse_head) as ctx:
            seen.append((kernels(ctx, u, S), ctx.scratch_bytes, S.clone()))
    assert seen[0][:2] == seen[1][:2] and torch.equal(seen[0][2], seen[1][2])


def test_launches_of_a_fused_head_count_against_slices():
    """two workers of half a million coordinates: tail, head and second moments in launches of their own cost more than the sketch saves"""
    d, n, r, c = 531_384, 2, 10, 10_329
    u, S = torch.randn(n, d, device="cuda"), torch.empty(n, r, c, device="cuda")
    with context(d, n, r, c, inputs.hash_params(r, seed=26), fuse_head=2) as ctx:
        assert kernels(ctx, u, S) == {"k_sketch_pull"}


def kernels_of_an_iteration(d, n, r, c, k, seed, **tunables):
    """the kernels of a head and of the two sketches after it, of its vector and of another one"""
    g, m, e, other = (torch.zeros(n, d, device="cuda") for _ in range(4))
    v, vhat = (torch.ones(d, device="cuda") for _ in range(2))
    S = torch.empty(n, r, c, device="cuda")
    with context(d, n, r, c, inputs.hash_params(r, seed=seed), k, **tunables) as ctx:
        ctx.sams_profile_enable(True)
        ctx.amsgrad_ef_update(g, m, e, v, vhat, torch.zeros(d, device="cuda"), None, None, 0, 0.9, 0.99, 1e-3)
        ctx.sams_profile_enable(False)
        return set(ctx.sams_profile_read()), kernels(ctx, e, S), kernels(ctx, other, S)


def one_iteration_with(shape, seed, **tunables):
    from paper_2210_07454_amd import sams
    from tests.test_gpu_random_shapes import one_iteration
    try:
        for key, val in tunables.items():
            sams.sams_configure(key, val)
        assert one_iteration(sams, shape, seed=seed)
    finally:
        for key in tunables:
            sams.sams_configure(key, 0)


@pytest.mark.parametrize("windows,fuse_head", [(103, 2), (103, 0), (3, 2), (1, 0)])
@pytest.mark.parametrize("d", [40_000, 40_003])
def test_one_iteration(d, windows, fuse_head):
    """head, sketches, recovery and update; a second sketch of the same vector comes from what the head has staged"""
    shape, seed, tunables = (d, 5, 5, 33_003, 400), d % 97 + windows, dict(push_windows=windows, fuse_head=fuse_head)
    one_iteration_with(shape, seed, **tunables)
    head, sketch, another = kernels_of_an_iteration(*shape, seed, **tunables)
    fused = fuse_head == 2 and windows > 100 and d % 4 == 0
    assert ("k_head_scatter" in head) == fused
    assert sketch == {"k_sketch_push"} | ({"k_bin_scatter"} if windows > 100 and not fused else set())
    assert another == {"k_sketch_push"} | ({"k_bin_scatter"} if windows > 100 else set())


@pytest.mark.parametrize("d,windows", [((1 << 24) + 1, 103), ((1 << 24) + 3, 116)])
def test_copies_of_long_ragged_vectors_by_the_head(d, windows):
    """4-byte accesses: tiles that are no power of two, the last of a few coordinates; g compacted on the index set of the iteration before"""
    shape, seed, tunables = (d, 2, 2, 70_001, 20_000), 11, dict(push_windows=windows, fuse_head=2)
    one_iteration_with(shape, seed, **tunables)
    head, sketch, another = kernels_of_an_iteration(*shape, seed, **tunables)
    assert "k_head_scatter" in head and sketch == {"k_sketch_push"} and another == {"k_sketch_push", "k_bin_scatter"}


@pytest.mark.parametrize("pa", [False, True])
@pytest.mark.parametrize("tunables,kernel", [(dict(push_windows=104), "k_sketch_push"), (dict(sketch_path=2), "k_bin_accumulate")])
def test_copies_written_by_the_head_are_used_once_and_for_their_vector(tunables, kernel, pa):
    """A sketch of another vector, and a recovery, take the place of what the head staged: the next sketch of the head's vector sorts it again."""
    d, n, r, c, k = 50_004, 3, 5, 40_000, 200
    hp = inputs.hash_params(r, seed=6)
    gen = torch.Generator(device="cuda").manual_seed(1)
    g, other = torch.randn(n, d, device="cuda", generator=gen), torch.randn(n, d, device="cuda", generator=gen)
    m, e = torch.zeros(n, d, device="cuda"), torch.zeros(n, d, device="cuda")
    v, vhat = (torch.full((n, d) if pa else (d,), 1e-4, device="cuda") for _ in range(2))
    S = torch.empty(n, r, c, device="cuda")
    o = Oracle("f32")
    with context(d, n, r, c, hp, k, fuse_head=2, **tunables) as ctx:
        (ctx.amsgrad_ef_update_pa if pa else ctx.amsgrad_ef_update)(g, m, e, v, vhat, torch.zeros(d, device="cuda"), None, None, 0, 0.9, 0.99, 1e-3)
        want = np.stack([o.sketch(x, hp, c) for x in e.cpu().numpy()])
        sketches = [(kernel,), (kernel, "k_bin_scatter"), (kernel, "k_bin_scatter")]
        for u, expect in zip((e, other, e), sketches):
            assert kernels(ctx, u, S) == set(expect)
            assert np.array_equal(S.cpu().numpy(), want if u is e else np.stack([o.sketch(x, hp, c) for x in other.cpu().numpy()]))
        ctx.unsketch_topk(S.mean(0).contiguous(), None, torch.empty(k, device="cuda", dtype=torch.int32), None)
        assert kernels(ctx, e, S) == {kernel, "k_bin_scatter"}
        assert np.array_equal(S.cpu().numpy(), want)


@pytest.mark.parametrize("tunables", [dict(push_windows=104), dict(sketch_path=2)], ids=["copies", "bins"])
def test_a_sketch_that_fails_forgets_what_the_head_staged(tunables):
    """An error that an earlier HIP call of the thread has left behind is reported once pass 1 for another vector has been enqueued: what it
    overwrote is not taken for the head's vector afterwards."""
    from paper_2210_07454_amd import sams
    from tests.test_gpu_selection_recovers import hip
    d, n, r, c = 50_004, 3, 5, 40_000
    hp = inputs.hash_params(r, seed=6)
    gen = torch.Generator(device="cuda").manual_seed(2)
    g, other = torch.randn(n, d, device="cuda", generator=gen), torch.randn(n, d, device="cuda", generator=gen)
    m, e = torch.zeros(n, d, device="cuda"), torch.zeros(n, d, device="cuda")
    v, vhat = (torch.full((d,), 1e-4, device="cuda") for _ in range(2))
    S = torch.empty(n, r, c, device="cuda")
    o = Oracle("f32")
    lib = hip()
    with context(d, n, r, c, hp, fuse_head=2, **tunables) as ctx:
        ctx.amsgrad_ef_update(g, m, e, v, vhat, torch.zeros(d, device="cuda"), None, None, 0, 0.9, 0.99, 1e-3)
        torch.cuda.synchronize()
        assert lib.hipSetDevice(4096) != 0                               # no such device: leaves its error behind
        with pytest.raises(sams.SamsError):
            ctx.sketch_accumulate(other, S)
        lib.hipGetLastError()
        ctx.sketch_accumulate(e, S)
        assert np.array_equal(S.cpu().numpy(), np.stack([o.sketch(x, hp, c) for x in e.cpu().numpy()]))


def test_replayed_graph_equals_eager():
    d, n, r, c = 60_001, 4, 3, 50_000
    hp = inputs.hash_params(r, seed=2)
    u = torch.randn(n, d, device="cuda")
    for windows in (2, 103):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            with context(d, n, r, c, hp, push_windows=windows) as ctx:
                S, ref = torch.empty(n, r, c, device="cuda"), torch.empty(n, r, c, device="cuda")
                ctx.sketch_accumulate(u, ref)
                stream.synchronize()
                graph = torch.cuda.CUDAGraph()
                with torch.cuda.graph(graph, stream=stream):
                    ctx.sketch_accumulate(u, S)
                for _ in range(3):
                    S.fill_(3.0)
                    graph.replay()
                    stream.synchronize()
                    assert torch.equal(S, ref)
                    ctx.sketch_accumulate(u, ref)


def test_sums_in_parts_stay_in_parts():
    """above 2^22 coordinates a table of one LDS window is summed in parts, nearer to the exact sums than one after the other"""
    d, n, r, c = 2 ** 22 + 7, 9, 3, 32_768
    hp = inputs.hash_params(r, seed=4)
    u, S = torch.randn(n, d, device="cuda"), torch.empty(n, r, c, device="cuda")
    with context(d, n, r, c, hp) as ctx:
        assert ctx.sketch_mode == 1 and "k_sketch_push" not in kernels(ctx, u, S)


def test_without_room_for_the_copies():
    """the context sums lists of slices instead, as if the copies had not been asked for"""
    from tests.test_gpu_short_memory import hold_all_but
    d, n, r, c = 4_000_000, 30, 5, 32_000                               # copies of 960 MB
    hp = inputs.hash_params(r, seed=3)
    u, S, ref = torch.randn(n, d, device="cuda"), torch.empty(n, r, c, device="cuda"), torch.empty(n, r, c, device="cuda")
    with context(d, n, r, c, hp, push_windows=104) as ctx:
        assert kernels(ctx, u, ref) == {"k_sketch_push", "k_bin_scatter"}
    torch.cuda.empty_cache()
    held = hold_all_but(700 << 20)
    try:
        with context(d, n, r, c, hp, push_windows=104) as ctx:
            assert kernels(ctx, u, S) == {"k_sketch_pull"} and ctx.scratch_bytes < 700 << 20
            torch.cuda.synchronize()
    finally:
        del held
        torch.cuda.empty_cache()
    assert torch.equal(S, ref)


def test_without_room_for_what_the_head_compacts():
    """the copies find room, the gradients of the selected coordinates beside them do not: the context sums lists of slices, whose head compacts nothing"""
    from tests.test_gpu_short_memory import hold_all_but
    d, n, r, c, k = 4_000_000, 30, 5, 32_000, 2_000_000                 # lists and copies 1,081 MB, gradients 240 MB
    hp = inputs.hash_params(r, seed=3)
    u, S, ref = torch.randn(n, d, device="cuda"), torch.empty(n, r, c, device="cuda"), torch.empty(n, r, c, device="cuda")
    with context(d, n, r, c, hp, k, push_windows=104, fuse_head=2) as ctx:
        assert kernels(ctx, u, ref) == {"k_sketch_push", "k_bin_scatter"} and 1_310e6 < ctx.scratch_bytes < 1_340e6
    torch.cuda.empty_cache()
    held = hold_all_but(1150 << 20)
    try:
        with context(d, n, r, c, hp, k, push_windows=104, fuse_head=2) as ctx:
            assert kernels(ctx, u, S) == {"k_sketch_pull"} and ctx.scratch_bytes < 1_000e6
            torch.cuda.synchronize()
    finally:
        del held
        torch.cuda.empty_cache()
    assert torch.equal(S, ref)
