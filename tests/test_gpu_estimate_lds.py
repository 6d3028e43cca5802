"""Estimates of vectors of at least 2^20 coordinates from tables whose rows fit in LDS, bit for bit: all rows held there, some,
or just one; lengths around the kernel's step (256 workgroups of 1024 coordinates, four steps a turn); tables of few buckets, of
a power of two, and of exactly the LDS; hash parameters at the ends of their range."""
import numpy as np
import pytest
import torch

from oracle import Oracle
from paper_2210_07454_amd import inputs

pytestmark = pytest.mark.gpu
P31 = 2_147_483_647

M = 1 << 20
SHAPES = [  # d, r, c
    (M, 5, 128), (M - 1, 3, 400), (M + 1, 5, 10_000), (M + 262_143, 4, 8_192), (M + 262_145, 16, 3_001),
    (2 * M - 1, 10, 5_003), (M + 1_023, 2, 40_960), (1_300_001, 1, 40_961), (1_500_000, 7, 2), (2 * M + 1, 6, 3),
    (1_700_001, 3, 1), (M + 1_025, 12, 13_653), (1_200_003, 5, 40_959),
]


@pytest.mark.parametrize("extreme", [False, True], ids=["hashes", "extreme-hashes"])
@pytest.mark.parametrize("d,r,c", SHAPES)
def test_estimates_bit_exact(d, r, c, extreme):
    from paper_2210_07454_amd import sams
    rng = np.random.default_rng(d + r)
    hp = inputs.hash_params(r, seed=d % 83)
    if extreme:
        hp[0] = (P31 - 1, P31 - 1, P31 - 1, P31 - 1)
        hp[-1] = (1, 0, 1, P31 - 1)
    S = rng.standard_normal((r, c)).astype(np.float32)
    S.reshape(-1)[::5] = -0.0
    vhat = (10.0 ** rng.uniform(-6, 2, d)).astype(np.float32)
    o = Oracle("f32")
    with sams.Context(d, 1, r, c, 7, hp) as ctx:
        for vh in (vhat, None):
            est = torch.full((d,), 9.0, device="cuda")
            ctx.unsketch_estimates(torch.from_numpy(S).cuda(), None if vh is None else torch.from_numpy(vh).cuda(), est)
            want = o.unsketch(S, vh, d, hp)
            assert np.array_equal(est.cpu().numpy(), want)
