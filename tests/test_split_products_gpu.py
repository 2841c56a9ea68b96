"""The products on split bf16 operands: every tile shape at widths around its edges against the
oracle, the same bits from every shape, and the float32 kernels where the device has no room for
the split weights."""
import numpy as np
import pytest

from tests.gpu_util import assert_close, check_input, gpu_crown, gpu_ctx
from workloads import random_mlp

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


def test_every_tile_shape_gives_the_same_bits():
    """640 rows an input: one input runs the 32 x 64 and 64 x 64 tiles, 64 inputs (40960 rows)
    the 128 x 128 ones; the inputs are the same."""
    wl = random_mlp(931, [300, 320, 320, 320, 11], 64, 0.01)
    ctx = gpu_ctx(wl.net)
    lb, ub, layers = gpu_crown(ctx, wl)
    for b in (0, 37, 63):
        l1, u1, lay1 = gpu_crown(ctx, wl, inputs=[b])
        assert np.array_equal(l1[0], lb[b]) and np.array_equal(u1[0], ub[b])
        for (l, u), (lx, ux) in zip(layers, lay1):
            assert np.array_equal(lx[0], l[b]) and np.array_equal(ux[0], u[b])
    check_input(wl.net, wl.x0[37], wl.eps, wl.C[37], lb[37], ub[37], [(l[37], u[37]) for l, u in layers])


def test_large_and_small_magnitudes():
    """Scaling a layer by 2^k and the next by 2^-k scales that layer's bounds by 2^k exactly and
    leaves the others as they are, over most of float32's exponent range."""
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


def test_float32_kernels_when_memory_is_short():
    """With less than an eighth of the device's memory left no split weights are kept; the bounds
    come from the float32 kernels, within the parity tolerance."""
    import torch
    wl = random_mlp(951, [120, 200, 180, 9], 2, 0.03)
    with_split = gpu_ctx(wl.net)
    want = gpu_crown(with_split, wl)
    free, total = torch.cuda.mem_get_info()
    hold = torch.empty(max(free - total // 16, 1), dtype=torch.uint8, device="cuda")
    try:
        ctx = gpu_ctx(wl.net)
        assert ctx.stats()["net_bytes"] < with_split.stats()["net_bytes"]
        lb, ub, layers = gpu_crown(ctx, wl)
    finally:
        del hold
        torch.cuda.empty_cache()
    for b in range(2):
        check_input(wl.net, wl.x0[b], wl.eps, wl.C[b], lb[b], ub[b], [(l[b], u[b]) for l, u in layers])
        assert_close(lb[b], want[0][b].astype(np.float64), "float32 and split products")
