"""Split weights kept in memory save time only: without them (VCR_PRODUCTS_SPLIT_NO_COPIES, or no
room) every product has the same bits, at every tile shape and in every epilogue."""
import numpy as np
import pytest

from tests.gpu_util import gpu_crown, to_dev
from tests.test_float32_products_gpu import ctx_with
from tests.test_split_products_gpu import odd_resnet, same_bits
from workloads import random_mlp
from workloads.gen import draw_splits

import oracle

pytestmark = pytest.mark.gpu


def both(net):
    a, b = ctx_with("split")(net), ctx_with("split_no_copies")(net)
    assert b.stats()["net_bytes"] < a.stats()["net_bytes"]
    return a, b


# 640 rows an input: 1, 8 and 64 inputs run the 32 x 64, 64 x 64 and 128 x 128 tiles; ragged widths
@pytest.mark.parametrize("dims", [[300, 320, 320, 320, 11], [77, 300, 129, 333, 41, 3]],
                         ids=lambda d: "x".join(map(str, d)))
@pytest.mark.parametrize("inputs", [1, 8, 64])
def test_bounds(dims, inputs):
    wl = random_mlp(981, dims, 64, 0.01)
    a, b = both(wl.net)
    pick = list(range(inputs))
    same_bits(gpu_crown(a, wl, inputs=pick), gpu_crown(b, wl, inputs=pick))


@pytest.mark.parametrize("inputs", [1, 64])
def test_gradients_and_slopes(inputs):
    wl = random_mlp(982, [90, 200, 170, 150, 12], inputs, 0.03)

    def run(ctx):
        lb, ub, ex = ctx.alpha_crown_bounds(to_dev(wl.x0), wl.eps, to_dev(wl.C), iters=3, want_grad=True, want_alpha=True)
        return [t.cpu().numpy() for t in (lb, ub, ex["grad"], ex["alpha"])]

    same_bits(*map(run, both(wl.net)))


def test_subdomains_and_multipliers():
    wl = random_mlp(983, [60, 140, 300, 5], 1, 0.05)
    root = oracle.crown(wl.net, wl.x0[0], wl.eps, wl.C[0])
    sp = draw_splits(np.random.default_rng(3), oracle.unstable_pool(wl.net, root), 700, 5)
    dev = (to_dev(sp.relu_id), to_dev(sp.neuron), to_dev(sp.sign))

    def run(ctx):
        lb, ub, _ = gpu_crown(ctx, wl, splits=sp)
        bl, bu, _ = ctx.beta_crown_bounds(to_dev(wl.x0), wl.eps, to_dev(wl.C), dev, iters=3)
        return [lb, ub, bl.cpu().numpy(), bu.cpu().numpy()]

    same_bits(*map(run, both(wl.net)))


def test_large_layer_ibp():
    """|W| r of a layer of 2^24 weights: the sign is taken off the parts, or off the weights."""
    wl = random_mlp(984, [4096, 4100, 2], 3, 0.001)
    same_bits(*([t.cpu().numpy() for t in c.ibp_bounds(to_dev(wl.x0), wl.eps, to_dev(wl.C))] +
                [np.zeros(1)] for c in both(wl.net)))


def test_out_of_range():
    """The weights' products that overflow are taken again in float32 from the same weights."""
    wl = random_mlp(985, [40, 70, 60, 7], 2, 0.05)
    for nd in (wl.net.nodes[0], wl.net.nodes[2]):
        nd.W = nd.W * np.float32(2.0 ** 55)
    same_bits(*(gpu_crown(c, wl) for c in both(wl.net)))


def test_convolutional_network():
    wl = odd_resnet(986, 7, 32, 64, 75, 5)

    def run(ctx):
        lb, ub, layers = gpu_crown(ctx, wl)
        _, _, ex = ctx.alpha_crown_bounds(to_dev(wl.x0), wl.eps, to_dev(wl.C), iters=0, want_grad=True)
        return lb, ub, layers, ex["grad"].cpu().numpy()

    same_bits(*map(run, both(wl.net)))
