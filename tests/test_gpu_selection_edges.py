"""The selection at the edges of its tiles (4096 keys) and of its routes (up to 2^16 keys, up to 2^20, more), with the
threshold inside a run of equal keys, inside a run of zeros of both signs, and with every key selected."""
import numpy as np
import pytest
import torch

from oracle import Oracle

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
