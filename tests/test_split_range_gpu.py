"""The products on split bf16 operands outside the range that three bf16 parts of the operands
themselves would cover: subnormal parts, values that round to infinity in bf16, sums that overflow."""
import copy

import numpy as np
import pytest

from tests.gpu_util import assert_close, check_input, gpu_crown, gpu_ctx, to_dev
from tests.test_alpha_gpu import _assert_grad_close
from tests.test_split_products_gpu import odd_resnet
from workloads import random_mlp

pytestmark = pytest.mark.gpu


def scaled(wl, at, s):
    """The network scaled by s from its `at`-th dense layer on: those weights times s, and every
    bias from there.  Bounds from there on are s times the original's."""
    out = copy.deepcopy(wl)
    dense = [nd for nd in out.net.nodes if nd.op == "dense"]
    dense[at].W = dense[at].W * np.float32(s)
    for nd in dense[at:]:
        nd.b = nd.b * np.float32(s)
    return out


def grid_mlp(seed, dims, batch, eps):
    """Weights and biases that are multiples of 2^-24: times 2^-118 they stay exact."""
    wl = random_mlp(seed, dims, batch, eps)
    for nd in wl.net.nodes:
        if nd.W is not None:
            nd.W = (np.round(nd.W * 2.0 ** 24) / 2.0 ** 24).astype(np.float32)
            nd.b = (np.round(nd.b * 2.0 ** 24) / 2.0 ** 24).astype(np.float32)
    return wl


# at = 0: the products' weights are tiny or huge; at = 1: their coefficient rows.  2^-118: the
# third part of the operands themselves is cut at 2^-133; 2^110: weights round to infinity.
# Tolerance: sums of 70 terms of about 1, each rounded by 2^-24 of itself (3e-5 of a bound would be
# lost if weights were split unscaled), and tiny coefficients by 2^-134, times their weights: below
# 2^-16 a unit of the column sums of the layer under them, 70 weights of 0.2.
@pytest.mark.parametrize("at", [0, 1])
@pytest.mark.parametrize("k", [-118, 110])
def test_bounds_scale_with_the_network(at, k):
    base = grid_mlp(961, [40, 70, 60, 7], 2, 0.05)
    lb, ub, layers = gpu_crown(gpu_ctx(base.net), base)
    slb, sub, slayers = gpu_crown(gpu_ctx(scaled(base, at, 2.0 ** k).net), base)
    tol = 70 * 2.0 ** -24
    if k < -110 and at == 1:
        tol += 2.0 ** -134 * 2.0 ** -k * np.abs(base.net.nodes[0].W).sum(0).max()
    got, want = [slb, sub], [lb, ub]
    for (l, u), (sl, su) in list(zip(layers, slayers))[at:]:
        got += [sl, su]
        want += [l, u]
    for g, w in zip(got, want):
        err = np.abs(g.astype(np.float64) * 2.0 ** -k - w)
        assert np.all(err <= tol * np.maximum(1, np.abs(w))), float(err.max())


def test_every_tile_shape_out_of_range():
    """640 rows an input, times 2^110: one input runs the two smaller tiles, 64 the largest."""
    base = random_mlp(931, [300, 320, 320, 320, 11], 64, 0.01)
    big = scaled(base, 0, 2.0 ** 110)
    lb, ub, _ = gpu_crown(gpu_ctx(base.net), base)
    ctx = gpu_ctx(big.net)
    blb, bub, _ = gpu_crown(ctx, base)
    for g, w in ((blb, lb), (bub, ub)):
        assert_close(g.astype(np.float64) * 2.0 ** -110, w.astype(np.float64), "scaled bounds")
    for sel in ([0], [63], [5, 9, 11, 20, 37, 41, 62, 63]):   # the 32 x 64 and the 64 x 64 tiles
        ls, us, _ = gpu_crown(ctx, base, inputs=sel)
        assert np.array_equal(ls, blb[sel]) and np.array_equal(us, bub[sel])


def test_the_largest_finite_weight_times_zero():
    """A weight of FLT_MAX into a neuron that nothing reads: every bound past it is finite."""
    wl = random_mlp(962, [40, 70, 60, 7], 2, 0.05)
    wl.net.nodes[0].W[3, 5] = np.finfo(np.float32).max
    wl.net.nodes[2].W[:, 3] = 0
    lb, ub, layers = gpu_crown(gpu_ctx(wl.net), wl)
    wl.net.nodes[0].W[3] = 0   # the same network for everything behind that neuron
    keep = np.arange(70) != 3
    ref = gpu_crown(gpu_ctx(wl.net), wl)
    for (l, u), (rl, ru) in zip(layers[1:], ref[2][1:]):
        assert_close(l, rl.astype(np.float64), "l")
        assert_close(u, ru.astype(np.float64), "u")
    assert np.array_equal(layers[0][0][:, keep], ref[2][0][0][:, keep])
    for b in range(2):
        check_input(wl.net, wl.x0[b], wl.eps, wl.C[b], lb[b], ub[b], ref[2] and [(l[b], u[b]) for l, u in ref[2]])


# a residual block's first convolution times s and its second over s: the block's values stay
@pytest.mark.parametrize("hw,c1,c2", [(7, 32, 64), (5, 64, 128)])
@pytest.mark.parametrize("k", [-112, 112])
def test_convolutions_out_of_range(hw, c1, c2, k):
    wl = odd_resnet(970 + hw, hw, c1, c2, 33, 5)

    def run(net):
        import torch
        ctx = gpu_ctx(net)
        lb, ub, layers = gpu_crown(ctx, wl)
        _, _, ex = ctx.alpha_crown_bounds(to_dev(wl.x0), wl.eps, to_dev(wl.C), iters=0, want_grad=True)
        torch.cuda.synchronize()
        return lb, ub, layers, ex["grad"].cpu().numpy()

    ref = run(wl.net)
    net = copy.deepcopy(wl.net)
    nodes = net.nodes
    scaled_relus = []
    for r, i in enumerate(k for k, nd in enumerate(nodes) if nd.op == "relu"):
        a = nodes[i].in0
        b = next((j for j, nd in enumerate(nodes) if nd.op == "conv2d" and nd.in0 == i), None)
        if b is None:
            continue
        nodes[a].W, nodes[a].b = nodes[a].W * np.float32(2.0 ** k), nodes[a].b * np.float32(2.0 ** k)
        nodes[b].W = nodes[b].W * np.float32(2.0 ** -k)
        scaled_relus.append(r)
    assert len(scaled_relus) == 3
    got = run(net)
    assert_close(got[0], ref[0].astype(np.float64), "lb")
    assert_close(got[1], ref[1].astype(np.float64), "ub")
    for r, ((l, u), (rl, ru)) in enumerate(zip(got[2], ref[2])):
        f = 2.0 ** -k if r in scaled_relus else 1.0
        assert_close(l.astype(np.float64) * f, rl.astype(np.float64), f"relu {r} l")
        assert_close(u.astype(np.float64) * f, ru.astype(np.float64), f"relu {r} u")
    _assert_grad_close(got[3], ref[3].astype(np.float64), "gradients")
