"""Split weights and device memory: an allocation of the context that fits only in their place takes
it, one that does not fit even there leaves them, a later call makes them again when there is
room; the bounds are the same bits throughout, replayed graphs included."""
import contextlib

import numpy as np
import pytest

from paper_2606_09377_amd.vcrown import OPT_GRAPH, VCR_ERR_OOM, VcrError
from tests.gpu_util import assert_close, gpu_ctx, to_dev
from workloads import Net, Node, random_mlp

pytestmark = pytest.mark.gpu

DIMS = [1024] + 5 * [4096] + [3]   # 0.86 GB of split weights; a workspace of 0.3 GB an input
FREE = 3 << 30                     # left free beside the copies and the first workspace


@contextlib.contextmanager
def free_memory(left):
    import torch
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    hold = torch.empty(max(torch.cuda.mem_get_info()[0] - left, 1), dtype=torch.uint8, device="cuda")
    try:
        yield
    finally:
        del hold
        torch.cuda.empty_cache()


@pytest.mark.parametrize("replay", [False, True])
def test_room_taken_and_regained(replay):
    import torch
    wl = random_mlp(991, DIMS, 1, 0.002)
    ctx = gpu_ctx(wl.net)
    if replay:
        ctx.set_option(OPT_GRAPH, 1)
    x0, C = to_dev(wl.x0), to_dev(wl.C)
    with_copies = ctx.stats()["net_bytes"]

    def one():
        got = []
        for _ in range(3):   # with replay: launched and recorded, then replayed twice
            lb, ub = ctx.crown_bounds(x0, wl.eps, C)
            torch.cuda.synchronize()
            got += [lb.cpu().numpy(), ub.cpu().numpy()]
        assert all(np.array_equal(g, got[k % 2]) for k, g in enumerate(got))
        return got[:2]

    want = one()
    copies = 12 * (1024 * 4096 + 4 * 4096 * 4096)
    xb, cb = x0.repeat(64, 1), C.repeat(64, 1, 1)
    assert ctx.workspace_bytes(64, 2) > 5 * FREE and ctx.workspace_bytes(8, 2) < FREE
    with free_memory(FREE):
        # not even in their place: the call fails, the copies stay
        with pytest.raises(VcrError) as e:
            ctx.crown_bounds(xb, wl.eps, cb)
        assert e.value.status == VCR_ERR_OOM
        assert ctx.stats()["net_bytes"] == with_copies
        assert all(np.array_equal(a, b) for a, b in zip(one(), want))
        # workspaces grown by less than the copies hold: one of them takes their place
        B = 8
        while ctx.stats()["net_bytes"] == with_copies:
            B += 1
            lb, ub = ctx.crown_bounds(xb[:B], wl.eps, cb[:B])
            torch.cuda.synchronize()
            for b in (0, B - 1):
                assert np.array_equal(lb[b].cpu().numpy(), want[0][0]) and np.array_equal(ub[b].cpu().numpy(), want[1][0])
        assert ctx.stats()["net_bytes"] == with_copies - copies
        assert all(np.array_equal(a, b) for a, b in zip(one(), want))
        assert ctx.stats()["net_bytes"] == with_copies - copies
    # room again
    assert all(np.array_equal(a, b) for a, b in zip(one(), want))
    assert ctx.stats()["net_bytes"] == with_copies


def test_a_recorded_graph_keeps_the_copies():
    """A caller's graph of an allocation-free call reads the copies: a workspace that fits only in
    their place fails, and the graph replays the same bits, with eager calls between."""
    import torch
    wl = random_mlp(992, [16384, 2048, 2048, 3], 1, 0.002)   # 0.45 GB of split weights
    ctx = gpu_ctx(wl.net)
    x0, C = to_dev(wl.x0), to_dev(wl.C)
    m = C.shape[1]
    lb, ub = torch.empty(1, m, device="cuda"), torch.empty(1, m, device="cuda")
    ctx.crown_bounds_noalloc(x0, wl.eps, C, (lb, ub))
    want = [lb.cpu().numpy(), ub.cpu().numpy()]
    with_copies = ctx.stats()["net_bytes"]
    copies = 12 * (16384 * 2048 + 2048 * 2048)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ctx.crown_bounds_noalloc(x0, wl.eps, C, (lb, ub))

    def replay():
        lb.zero_()
        ub.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(lb.cpu().numpy(), want[0]) and np.array_equal(ub.cpu().numpy(), want[1])

    replay()
    xb, cb = x0.repeat(200, 1), C.repeat(200, 1, 1)
    with free_memory(1 << 30):
        with pytest.raises(VcrError) as e:
            for B in range(2, 201):   # workspaces grown by less than the copies hold
                assert ctx.workspace_bytes(B, m) - ctx.workspace_bytes(B - 1, m) < copies
                ctx.crown_bounds(xb[:B], wl.eps, cb[:B])
                torch.cuda.synchronize()
                replay()
        assert e.value.status == VCR_ERR_OOM
        assert ctx.stats()["net_bytes"] == with_copies
        replay()
    replay()


def test_copies_made_again_are_whole_for_the_next_stream():
    """A request that fails in the copies' place too has them made again; the next call, on another
    stream and with nothing waited for, finds them whole."""
    import torch
    wl = random_mlp(993, DIMS, 1, 0.002)
    ctx = gpu_ctx(wl.net)
    x0, C = to_dev(wl.x0), to_dev(wl.C)
    want = [t.cpu().numpy() for t in ctx.crown_bounds(x0, wl.eps, C)]
    with_copies = ctx.stats()["net_bytes"]
    m, free = C.shape[1], 1 << 30
    side = torch.cuda.Stream()
    with free_memory(free):
        B = 2   # about 3 GB more than is free
        while ctx.workspace_bytes(B, m) < free + (3 << 30):
            B += 1
        xb, cb = x0.expand(B, -1).contiguous(), C.expand(B, -1, -1).contiguous()
        torch.cuda.synchronize()
        with pytest.raises(VcrError) as e:
            ctx.crown_bounds(xb, wl.eps, cb)
        assert e.value.status == VCR_ERR_OOM
        with torch.cuda.stream(side):
            lb, ub = ctx.crown_bounds(x0, wl.eps, C)
        side.synchronize()
        assert np.array_equal(lb.cpu().numpy(), want[0]) and np.array_equal(ub.cpu().numpy(), want[1])
    assert ctx.stats()["net_bytes"] == with_copies


def test_load_needs_the_layers_room_only():
    """2.1 GB of layer arrays load into 2.5 GB: no copy of the largest layer (1 GB) beside them."""
    import torch
    n = 16384
    rng = np.random.default_rng(5)
    W = np.zeros((n, n), np.float32)
    W[np.arange(n), rng.permutation(n)] = 1
    net = Net((n,), [Node("dense", -1, W=W, b=np.zeros(n, np.float32)), Node("relu", 0),
                     Node("dense", 1, W=rng.standard_normal((4, n)).astype(np.float32), b=np.ones(4, np.float32))])
    x0 = rng.random((1, n)).astype(np.float32)
    with free_memory(2500 << 20):
        ctx = gpu_ctx(net)
        assert 2 * 4 * n * n <= ctx.stats()["net_bytes"] < 2 * 4 * n * n + (32 << 20)
    lb, ub = ctx.crown_bounds(to_dev(x0), np.float32(0), to_dev(np.eye(4, dtype=np.float32)[None]))
    torch.cuda.synchronize()
    want = net.nodes[2].W.astype(np.float64) @ (W @ x0[0]) + 1
    assert_close(lb[0].cpu().numpy(), want, "lb")
    assert_close(ub[0].cpu().numpy(), want, "ub")
