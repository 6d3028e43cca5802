"""The selection at the edges of its tiles (4096 keys) and of its routes (up to 2^16 keys, up to 2^20, more), with the
threshold inside a run of equal keys, inside a run of zeros of both signs, and with every key selected."""
import numpy as np
import pytest
import torch

from oracle import Oracle
from paper_2210_07454_amd import inputs

pytestmark = pytest.mark.gpu

EDGES = [1, 4095, 4096, 4097, 65_535, 65_536, 65_537, (1 << 20) - 1, 1 << 20, (1 << 20) + 1, 1_300_001]


@pytest.mark.parametrize("values", ["distinct", "few", "zeros"])
@pytest.mark.parametrize("k_in", EDGES)
def test_selection_at_tile_and_route_edges(k_in, values):
    from paper_2210_07454_amd import sams
    rng = np.random.default_rng(k_in)
    if values == "distinct":
        vals = rng.standard_normal(k_in).astype(np.float32)
    elif values == "few":                                            # long runs of equal keys: every list is full
        vals = (rng.integers(8, 12, k_in) / 8.0 * rng.choice([-1.0, 1.0], k_in)).astype(np.float32)
    else:                                                            # fewer keys differ from zero than are selected
        vals = np.where(rng.random(k_in) < 0.01, rng.standard_normal(k_in), rng.choice([-0.0, 0.0], k_in)).astype(np.float32)
    cand = np.cumsum(rng.integers(1, 9, k_in)).astype(np.int32)
    ci, vi = torch.from_numpy(cand).cuda(), torch.from_numpy(vals).cuda()
    for k_out in sorted({1, (k_in + 1) // 2, max(1, k_in // 50), k_in}):
        io = torch.full((k_out,), -1, device="cuda", dtype=torch.int32)
        do = torch.full((k_out,), 7.0, device="cuda")
        sams.topk_refine_static(ci, vi, k_out, io, do)
        idx, delta = Oracle("f32").refine(cand, vals, k_out)
        assert np.array_equal(io.cpu().numpy(), idx), k_out
        assert np.array_equal(do.cpu().numpy().view(np.uint32), delta.view(np.uint32)), k_out


@pytest.mark.parametrize("k_in,k_out", [(8_193, 8_193), (20_000, 8_192), (20_000, 8_193), (65_536, 8_192), (65_536, 65_536),
                                        (69_633, 60_001), (100_001, 6_501), (262_145, 43_000), (1_050_000, 1_049_999),
                                        (1_300_001, 220_000), (9_000_000, 1_000_000)])
@pytest.mark.parametrize("equal", [False, True], ids=["distinct", "half-equal"])
def test_selection_of_a_large_share(k_in, k_out, equal):
    """The largest k of the one-launch route and the one above it; lists in one, two, ... sixteen pieces a tile, with a last tile
    of one key, lists that end inside a piece, and ties that span pieces."""
    from paper_2210_07454_amd import sams
    rng = np.random.default_rng(k_in + k_out)
    vals = rng.standard_normal(k_in).astype(np.float32)
    if equal:
        vals[rng.random(k_in) < 0.5] = np.float32(-0.75)
    cand = np.cumsum(rng.integers(1, 9, k_in)).astype(np.int32)
    idx, delta = Oracle("f32").refine(cand, vals, k_out)
    ci, vi = torch.from_numpy(cand).cuda(), torch.from_numpy(vals).cuda()
    io, do = torch.full((k_out,), -1, device="cuda", dtype=torch.int32), torch.full((k_out,), 7.0, device="cuda")
    with sams.Context(k_in, 1, 1, 50, k_in, inputs.hash_params(1)) as ctx:
        ctx.topk_refine(ci, vi, k_out, io, do)
    assert np.array_equal(io.cpu().numpy(), idx)
    assert np.array_equal(do.cpu().numpy().view(np.uint32), delta.view(np.uint32))
