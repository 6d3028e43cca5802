"""A context whose selection lists find no room on the device selects all the same, from the keys themselves."""
import numpy as np
import pytest
import torch

from oracle import Oracle
from paper_2210_07454_amd import inputs

pytestmark = pytest.mark.gpu


def hold_all_but(spare):
    """Takes device memory until `spare` bytes are left (to 64 MiB)."""
    held = []
    while True:
        free = torch.cuda.mem_get_info()[0] - spare
        if free < 64 << 20:
            return held
        held.append(torch.empty(min(free, 8 << 30) // (2 << 20) * (2 << 20), device="cuda", dtype=torch.uint8))


def test_selections_without_room_for_lists():
    from paper_2210_07454_amd import sams
    d, c, k, k_out = 200_000_003, 16_384, 3_000_001, 700_000             # more than 2^20 keys in both selections
    hp = inputs.hash_params(1, seed=3)
    rng = np.random.default_rng(7)
    S = torch.from_numpy(rng.standard_normal((1, c)).astype(np.float32)).cuda()      # c magnitudes: ties at the threshold
    vals = (rng.integers(-4000, 4001, k) / 8.0).astype(np.float32)
    cand = np.cumsum(rng.integers(1, 9, k)).astype(np.int32)
    vi, ci = torch.from_numpy(vals).cuda(), torch.from_numpy(cand).cuda()
    out = []
    for short in (True, False):
        idx, est = torch.full((k,), -1, device="cuda", dtype=torch.int32), torch.empty(k, device="cuda")
        io, do = torch.full((k_out,), -1, device="cuda", dtype=torch.int32), torch.empty(k_out, device="cuda")
        torch.cuda.empty_cache()
        held = hold_all_but(4 * d + d // 8 + (320 << 20)) if short else []
        try:
            sams.sams_configure("sketch_path", 1)
            with sams.Context(d, 1, 1, c, k, hp) as ctx:
                assert (ctx.scratch_bytes < 4 * d + d // 8 + (16 << 20)) == short    # lists of d keys: 6 d bytes
                ctx.unsketch_topk(S, None, idx, est)
                ctx.topk_refine(ci, vi, k_out, io, do)
                torch.cuda.synchronize()
        finally:
            sams.sams_configure("sketch_path", 0)
            del held
            torch.cuda.empty_cache()
        out.append([t.cpu().numpy() for t in (idx, est, io, do)])
    for a, b in zip(*out):
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))
    want_idx, want_delta = Oracle("f32").refine(cand, vals, k_out)
    assert np.array_equal(out[0][2], want_idx) and np.array_equal(out[0][3], want_delta)
