"""Selections that one workgroup finishes from up to 256 tiles' lists: around the entries its LDS holds (15,360) and writes in turns
(3,072), with the lists full of equal keys, and first histograms taken by the kernels that make the estimates."""
import numpy as np
import pytest
import torch

from oracle import Oracle
from paper_2210_07454_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k_in,listed,k_out", [(65_537, 15_360, 3_000), (100_003, 15_361, 3_000), (131_073, 3_071, 2_000), (131_073, 3_073, 1_999), (140_000, 7_168, 2_000), (140_000, 7_169, 2_000),
                                               (131_072, 7_168, 2_000), (300_001, 11_265, 17), (300_001, 60_000, 2_000), (1 << 20, 1 << 20, 1),
                                               ((1 << 20) - 4095, 7_167, 2_001), (40_000, 4_097, 4_000),
                                               (200_000, 15_360, 3_000), (200_000, 15_361, 2_999), (1 << 19, 19_457, 3_000), ((1 << 19) + 1, 15_361, 2_500),
                                               (1 << 20, 15_359, 2_500), (900_000, 40_000, 2_500)])
@pytest.mark.parametrize("equal", [False, True], ids=["distinct", "equal"])
def test_lists_around_what_lds_holds(k_in, listed, k_out, equal):
    """`listed` keys share the first digit of the threshold, all others lie below."""
    from paper_2210_07454_amd import sams
    rng = np.random.default_rng(k_in + listed)
    vals = rng.uniform(0.1, 0.4, k_in).astype(np.float32)
    at = rng.permutation(k_in)[:listed]
    vals[at] = np.float32(1.0625) if equal else rng.uniform(1.0, 1.1249, listed).astype(np.float32)
    vals *= rng.choice([-1.0, 1.0], k_in).astype(np.float32)
    cand = np.cumsum(rng.integers(1, 9, k_in)).astype(np.int32)
    io, do = torch.full((k_out,), -1, device="cuda", dtype=torch.int32), torch.full((k_out,), 7.0, device="cuda")
    idx, delta = Oracle("f32").refine(cand, vals, k_out)
    ci, vi = torch.from_numpy(cand).cuda(), torch.from_numpy(vals).cuda()
    for _ in range(2):
        sams.topk_refine_static(ci, vi, k_out, io, do)
        assert np.array_equal(io.cpu().numpy(), idx)
        assert np.array_equal(do.cpu().numpy().view(np.uint32), delta.view(np.uint32))


# estimates by gathers and from rows in LDS, where the filter and where the estimate kernel picks the first digit; k on either side of the routes
@pytest.mark.parametrize("d,r,c,k", [(65_537, 3, 2_000, 700), (262_143, 4, 5_000, 2_000), (262_145, 5, 9_001, 2_001), ((1 << 20) + 1, 3, 5_000, 2_000),
                                     (1_000_003, 5, 12_000, 90), (1_500_001, 2, 3_000, 30_000), (1 << 20, 5, 4_200, 2_000)])
def test_first_histogram_with_the_estimates(d, r, c, k):
    from paper_2210_07454_amd import sams
    rng = np.random.default_rng(d)
    hp = inputs.hash_params(r, seed=d % 87)
    S = (rng.standard_normal((r, c)) ** 3).astype(np.float32)
    vhat = rng.uniform(1e-4, 1.0, d).astype(np.float32)
    idx, est = torch.full((k,), -1, device="cuda", dtype=torch.int32), torch.full((k,), 7.0, device="cuda")
    o = Oracle("f32")
    e = o.unsketch(S, vhat, d, hp)
    ref = o.topk(e, k)
    with sams.Context(d, 2, r, c, k, hp) as ctx:
        Sd, vd = torch.from_numpy(S).cuda(), torch.from_numpy(vhat).cuda()
        for _ in range(2):
            ctx.unsketch_topk(Sd, vd, idx, est)
            assert np.array_equal(idx.cpu().numpy(), ref)
            assert np.array_equal(est.cpu().numpy().view(np.uint32), e[ref].view(np.uint32))


# the histogram pass: 128 workgroups of one, two and more turns of two tiles, then a workgroup per four tiles, 256 at most
@pytest.mark.parametrize("k_in,k_out", [(131_073, 9_000), (524_287, 70_000), (524_293, 70_000), (1_048_577, 9_000), (2_097_149, 1_500_000),
                                        (2_101_249, 300_001), (4_194_305, 100_000)])
def test_histogram_pass(k_in, k_out):
    from paper_2210_07454_amd import sams
    rng = np.random.default_rng(k_in)
    vals = (rng.standard_normal(k_in) / rng.random(k_in).clip(1e-6) ** 0.6).astype(np.float32)
    vals[-1] = np.float32(3e38)                                      # the last key counts
    cand = np.arange(k_in, dtype=np.int32)
    idx, delta = Oracle("f32").refine(cand, vals, k_out)
    io, do = torch.full((k_out,), -1, device="cuda", dtype=torch.int32), torch.full((k_out,), 7.0, device="cuda")
    ci, vi = torch.from_numpy(cand).cuda(), torch.from_numpy(vals).cuda()
    for _ in range(2):
        sams.topk_refine_static(ci, vi, k_out, io, do)
        assert np.array_equal(io.cpu().numpy(), idx)
        assert np.array_equal(do.cpu().numpy().view(np.uint32), delta.view(np.uint32))


# zeros of both signs and values below the first digit's range; fewer, as many and more keys that differ from zero than are kept
@pytest.mark.parametrize("k_in,k_out", [(5_000, 1_000), (60_000, 8_192), (65_536, 7_500), (65_537, 3_000), (131_072, 2_000), (140_000, 2_999), (431_003, 3_000), (1 << 20, 2_500)])
@pytest.mark.parametrize("nonzero", [0, 1, -1, -2, 0.5, 1.5, "front", "back"])
def test_mostly_zeros(k_in, k_out, nonzero):
    from paper_2210_07454_amd import sams
    rng = np.random.default_rng(k_in)
    vals = np.where(rng.random(k_in) < 0.5, np.float32(0.0), np.float32(-0.0)).astype(np.float32)
    if nonzero == "front":
        at = np.arange(k_out // 2)
    elif nonzero == "back":
        at = np.arange(k_in - k_out // 2, k_in)
    else:
        m = int(nonzero * k_out) if isinstance(nonzero, float) else (nonzero if nonzero >= 0 else k_out + 1 + nonzero)   # -1: k_out, -2: one fewer
        at = rng.permutation(k_in)[:m]
    vals[at] = rng.standard_normal(len(at)).astype(np.float32)
    vals[at[::3]] = np.float32(1e-41)                                # subnormal: differs from zero, shares its first digit
    vals[at[::5]] = np.float32(-3e-45)
    cand = np.cumsum(rng.integers(1, 9, k_in)).astype(np.int32)
    idx, delta = Oracle("f32").refine(cand, vals, k_out)
    io, do = torch.full((k_out,), -1, device="cuda", dtype=torch.int32), torch.full((k_out,), 7.0, device="cuda")
    ci, vi = torch.from_numpy(cand).cuda(), torch.from_numpy(vals).cuda()
    for _ in range(2):
        sams.topk_refine_static(ci, vi, k_out, io, do)
        assert np.array_equal(io.cpu().numpy(), idx)
        assert np.array_equal(do.cpu().numpy().view(np.uint32), delta.view(np.uint32))
