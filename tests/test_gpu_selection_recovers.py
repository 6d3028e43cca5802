"""A selection that ends half-way, or that another one runs into, spoils no later one: the histograms and counters that it
leaves are cleared before they are used again."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import Oracle
from paper_2210_07454_amd import inputs

pytestmark = pytest.mark.gpu


def candidates(k_in, seed):
    rng = np.random.default_rng(seed)
    vals = (rng.integers(-4000, 4001, k_in) / 8.0).astype(np.float32)
    return np.cumsum(rng.integers(1, 9, k_in)).astype(np.int32), vals


def hip():
    return ctypes.CDLL("libamdhip64.so.7")                           # the runtime that torch has loaded


def cut_chain(graph, keep):
    """Takes the nodes of a captured chain away behind the first `keep`; how many it had."""
    lib, raw = hip(), ctypes.c_void_p(graph.raw_cuda_graph())
    chain, cnt = [], ctypes.c_size_t(1)
    node = ctypes.c_void_p()
    assert lib.hipGraphGetRootNodes(raw, ctypes.byref(node), ctypes.byref(cnt)) == 0 and cnt.value == 1
    while True:
        chain.append(ctypes.c_void_p(node.value))
        cnt = ctypes.c_size_t(0)
        assert lib.hipGraphNodeGetDependentNodes(chain[-1], None, ctypes.byref(cnt)) == 0
        if cnt.value == 0:
            break
        assert cnt.value == 1
        assert lib.hipGraphNodeGetDependentNodes(chain[-1], ctypes.byref(node), ctypes.byref(cnt)) == 0
    for n in reversed(chain[keep:]):
        assert lib.hipGraphDestroyNode(n) == 0
    return len(chain)


@pytest.mark.parametrize("k_in", [5_000, 70_000, 300_000, 1_300_000])   # every route of the selection
def test_static_refine_after_one_that_ended_half_way(k_in):
    """The kernels of a call up to the first, second, ... one alone (a captured call whose later nodes are taken away), each
    time followed by a whole call."""
    from paper_2210_07454_amd import sams
    k_out = k_in // 3
    cand, vals = candidates(k_in, k_in)
    ci, vi = torch.from_numpy(cand).cuda(), torch.from_numpy(vals).cuda()
    io, do = torch.empty(k_out, device="cuda", dtype=torch.int32), torch.empty(k_out, device="cuda")
    want_idx, want_delta = Oracle("f32").refine(cand, vals, k_out)
    sams.topk_refine_static(ci, vi, k_out, io, do)
    torch.cuda.synchronize()
    keep, nodes = 1, 2
    while keep < nodes:
        graph = torch.cuda.CUDAGraph(keep_graph=True)
        with torch.cuda.graph(graph):
            sams.topk_refine_static(ci, vi, k_out, io, do)
        nodes = cut_chain(graph, keep)
        graph.instantiate()
        graph.replay()
        torch.cuda.synchronize()
        io.fill_(-1)
        sams.topk_refine_static(ci, vi, k_out, io, do)
        assert np.array_equal(io.cpu().numpy(), want_idx), (k_in, keep)
        assert np.array_equal(do.cpu().numpy(), want_delta), (k_in, keep)
        keep += 1


@pytest.mark.parametrize("sizes", [(5_000, 61_000), (70_001, 1_300_000), (3_000, 300_007)])
def test_static_refine_after_calls_that_overlapped(sizes):
    """Calls of two sizes on two streams: their own outputs are undefined, but no position that the larger one has listed may
    lead the smaller one past its candidates, and the next call by itself is right."""
    from paper_2210_07454_amd import sams
    calls = []
    for k_in in sizes:
        cand, vals = candidates(k_in, k_in)
        ci, vi = torch.from_numpy(cand).cuda(), torch.from_numpy(vals).cuda()
        k_out = k_in // 3
        io, do = torch.empty(k_out, device="cuda", dtype=torch.int32), torch.empty(k_out, device="cuda")
        calls.append((ci, vi, k_out, io, do, torch.cuda.Stream(), Oracle("f32").refine(cand, vals, k_out)))
    torch.cuda.synchronize()
    for _ in range(10):
        for ci, vi, k_out, io, do, stream, _ in calls:
            sams.topk_refine_static(ci, vi, k_out, io, do, stream)
    torch.cuda.synchronize()
    for ci, vi, k_out, io, do, _, want in calls:
        io.fill_(-1)
        sams.topk_refine_static(ci, vi, k_out, io, do)
        assert np.array_equal(io.cpu().numpy(), want[0]) and np.array_equal(do.cpu().numpy(), want[1])


# the first digit's histogram comes from the gathering estimates, from the plan's recovery below and above 2^20
# coordinates, or from a pass over the keys
@pytest.mark.parametrize("d,r,c", [(60_000, 5, 400), (300_001, 3, 120_000), (1_300_003, 3, 120_000), (431_003, 4, 9_001)])
def test_topk_after_a_call_that_failed_half_way(d, r, c):
    """An error that an earlier HIP call of the thread has left behind is reported by the first check of a call, after its
    estimates have been enqueued: the selection behind them never runs."""
    from paper_2210_07454_amd import sams
    k = d // 50
    rng = np.random.default_rng(d)
    hp = inputs.hash_params(r)
    S = rng.standard_normal((r, c)).astype(np.float32)
    vhat = (rng.random(d) + 0.1).astype(np.float32)
    o = Oracle("f32")
    want = o.topk(o.unsketch(S, vhat, d, hp), k)
    Sd, vd = torch.from_numpy(S).cuda(), torch.from_numpy(vhat).cuda()
    idx = torch.empty(k, device="cuda", dtype=torch.int32)
    lib = hip()
    with sams.Context(d, 2, r, c, k, hp) as ctx:
        for _ in range(2):
            assert lib.hipSetDevice(4096) != 0                       # no such device: leaves its error behind
            with pytest.raises(sams.SamsError):
                ctx.unsketch_topk(Sd, vd, idx)
            lib.hipGetLastError()
            idx.fill_(-1)
            for _ in range(2):
                ctx.unsketch_topk(Sd, vd, idx)
                assert np.array_equal(idx.cpu().numpy(), want)
