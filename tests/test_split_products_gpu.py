"""The products on split bf16 operands: every tile shape at widths around its edges against the
oracle, and the same bits from every shape, with split weights in memory and without."""
import contextlib

import numpy as np
import pytest

from tests.gpu_util import assert_close, check_input, gpu_crown, gpu_ctx, to_dev
from tests.test_alpha_gpu import _assert_grad_close
from workloads import Workload, random_mlp
from workloads.gen import margin_spec, resnet_net

pytestmark = pytest.mark.gpu

# widths one below, at and above a block (16), a K step (32), a slab (64) and a tile (128): the
# rows of an intermediate pass are twice a width, so single inputs run the 32 x 64 tiles
EDGES = [[15, 16, 17, 2], [31, 33, 32, 3], [63, 64, 65, 5], [127, 129, 128, 10], [200, 257, 31, 100]]


@pytest.mark.parametrize("dims", EDGES, ids=lambda d: "x".join(map(str, d)))
def test_tile_edges(dims):
    wl = random_mlp(900 + dims[0], dims, 3, 0.02)
    lb, ub, layers = gpu_crown(gpu_ctx(wl.net), wl)
    for b in range(3):
        check_input(wl.net, wl.x0[b], wl.eps, wl.C[b], lb[b], ub[b], [(l[b], u[b]) for l, u in layers], what=f"input {b}")


# a chain's constant terms are summed per 64-column slab over its steps: slabs of one step that
# the next has not, and the other way round (widths going up and down again), one input and many
@pytest.mark.parametrize("dims", [[20, 700, 40, 260, 90, 3], [20, 30, 200, 500, 66, 64, 2]],
                         ids=lambda d: "x".join(map(str, d)))
def test_constants_over_changing_widths(dims):
    wl = random_mlp(920 + len(dims), dims, 40, 0.02)
    ctx = gpu_ctx(wl.net)
    lb, ub, layers = gpu_crown(ctx, wl)
    for b in (0, 39):
        l1, u1, _ = gpu_crown(ctx, wl, inputs=[b])
        assert np.array_equal(l1[0], lb[b]) and np.array_equal(u1[0], ub[b])
        check_input(wl.net, wl.x0[b], wl.eps, wl.C[b], lb[b], ub[b], [(l[b], u[b]) for l, u in layers], what=f"input {b}")


def test_every_tile_shape_gives_the_same_bits():
    """640 rows an input and six columns of 64: one input runs the 32 x 64 tiles, 8 inputs (480 tiles of
    64 x 64) the 64 x 64 ones and 64 inputs (960 of 128 x 128) the 128 x 128 ones."""
    wl = random_mlp(931, [300, 320, 320, 320, 11], 64, 0.01)
    ctx = gpu_ctx(wl.net)
    lb, ub, layers = gpu_crown(ctx, wl)
    for sel in ([0], [37], [63], [5, 9, 11, 20, 37, 41, 62, 63]):
        ls, us, lays = gpu_crown(ctx, wl, inputs=sel)
        assert np.array_equal(ls, lb[sel]) and np.array_equal(us, ub[sel])
        for (l, u), (lx, ux) in zip(layers, lays):
            assert np.array_equal(lx, l[sel]) and np.array_equal(ux, u[sel])
    check_input(wl.net, wl.x0[37], wl.eps, wl.C[37], lb[37], ub[37], [(l[37], u[37]) for l, u in layers])


def test_large_and_small_magnitudes():
    """Scaling a layer by 2^k and the next by 2^-k scales that layer's bounds by 2^k exactly and
    leaves the others as they are (2^-60 and 2^50: the ends of the range have their own tests)."""
    base = random_mlp(941, [40, 70, 60, 7], 2, 0.05)
    ref_lb, ref_ub, ref_layers = gpu_crown(gpu_ctx(base.net), base)
    for k in (-60, 50):
        wl = random_mlp(941, [40, 70, 60, 7], 2, 0.05)
        s = np.float32(2.0 ** k)
        wl.net.nodes[0].W, wl.net.nodes[0].b = wl.net.nodes[0].W * s, wl.net.nodes[0].b * s
        wl.net.nodes[2].W = wl.net.nodes[2].W / s
        lb, ub, layers = gpu_crown(gpu_ctx(wl.net), wl)
        assert np.array_equal(lb, ref_lb) and np.array_equal(ub, ref_ub)
        assert np.array_equal(layers[0][0], ref_layers[0][0] * s)
        assert np.array_equal(layers[1][1], ref_layers[1][1])


@contextlib.contextmanager
def short_memory():
    """A sixteenth of the device's memory left free: less than split weights are kept with."""
    import torch
    free, total = torch.cuda.mem_get_info()
    hold = torch.empty(max(free - total // 16, 1), dtype=torch.uint8, device="cuda")
    try:
        yield
    finally:
        del hold
        torch.cuda.empty_cache()


def same_bits(a, b):
    """Results as gpu_crown's (and what follows them) are equal bit for bit."""
    flat = lambda r: [x for v in r for x in (v if isinstance(v, (list, tuple)) else [v])]  # noqa: E731
    a, b = flat(flat(a)), flat(flat(b))
    assert len(a) == len(b) > 2
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


def test_same_bits_when_memory_is_short():
    """No split weights are kept then; the bounds are the same bits."""
    wl = random_mlp(951, [120, 200, 180, 77, 300, 9], 2, 0.03)
    with_split = gpu_ctx(wl.net)
    want = gpu_crown(with_split, wl)
    with short_memory():
        ctx = gpu_ctx(wl.net)
        assert ctx.stats()["net_bytes"] < with_split.stats()["net_bytes"]
        lb, ub, layers = gpu_crown(ctx, wl)
    for b in range(2):
        check_input(wl.net, wl.x0[b], wl.eps, wl.C[b], lb[b], ub[b], [(l[b], u[b]) for l, u in layers])
        assert_close(lb[b], want[0][b].astype(np.float64), "with and without split weights")
    same_bits((lb, ub, layers), want)


def odd_resnet(seed, hw, c1, c2, fc, n_out):
    """resnet_net on an odd image side (its stride-2 maps round up, and so do the dense columns)."""
    rng = np.random.default_rng(seed)
    net = resnet_net(rng, in_chw=(3, hw, hw), c1=c1, c2=c2, fc=fc, n_out=n_out)
    k = next(i for i, nd in enumerate(net.nodes) if nd.op == "flatten")
    n_flat = c2 * ((hw + 1) // 2) ** 2
    net.nodes[k + 1].W = (rng.standard_normal((fc, n_flat)) * np.sqrt(2 / n_flat)).astype(np.float32)
    x0 = rng.random((2, net.n_in)).astype(np.float32)
    return Workload(f"resnet{hw}", net, x0, np.float32(2 / 255), margin_spec(net, x0))


# an odd image side (window positions and rows that fill no 96- or 128-row tile), the 64-column
# blocks of 32 and 64 channels and the 128-column ones of 128, and stride 1 and 2
@pytest.mark.parametrize("hw,c1,c2,fc", [(7, 32, 64, 33), (5, 64, 128, 20)])
def test_convolutions_with_and_without_copies(hw, c1, c2, fc):
    """Bounds and slope gradients of a convolutional network with and, memory being short, without
    split dense weights: within the parity tolerance of the oracle, and the same bits."""
    import torch
    wl = odd_resnet(960 + hw, hw, c1, c2, fc, 5)
    with_split = gpu_ctx(wl.net)

    def run(ctx):
        lb, ub, layers = gpu_crown(ctx, wl)
        _, _, ex = ctx.alpha_crown_bounds(to_dev(wl.x0), wl.eps, to_dev(wl.C), iters=0, want_grad=True)
        torch.cuda.synchronize()
        return lb, ub, layers, ex["grad"].cpu().numpy()

    a = run(with_split)
    with short_memory():
        ctx = gpu_ctx(wl.net)
        assert ctx.stats()["net_bytes"] < with_split.stats()["net_bytes"]
        f = run(ctx)
    for lb, ub, layers, _ in (a, f):
        for b in range(2):
            check_input(wl.net, wl.x0[b], wl.eps, wl.C[b], lb[b], ub[b], [(l[b], u[b]) for l, u in layers])
    _assert_grad_close(a[3], f[3].astype(np.float64), "gradients")
    assert np.count_nonzero(f[3]) > 0
    same_bits(a, f)
