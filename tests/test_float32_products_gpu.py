"""VCR_OPT_PRODUCTS = float32: the kernels on the float32 matrix instructions, at every tile shape,
in every epilogue and with split neurons, multipliers and gradients, by the tests that the default
products pass."""
import numpy as np
import pytest

from paper_2606_09377_amd import Ctx
from paper_2606_09377_amd.vcrown import OPT_PRODUCTS, PRODUCTS
from tests import (gpu_util, test_alpha_conv_gpu, test_alpha_gpu, test_bab_gpu, test_beta_conv_gpu, test_beta_gpu,
                   test_conv_gpu, test_parity_gpu, test_split_products_gpu)
from tests.gpu_util import check_input, gpu_crown, to_dev
from workloads import random_mlp

pytestmark = pytest.mark.gpu


def ctx_with(products):
    def make(net):
        ctx = Ctx(0)
        ctx.set_option(OPT_PRODUCTS, PRODUCTS[products])
        ctx.load_net(net)
        return ctx
    return make


# (module, test, its arguments): slabs of changing widths; gradients and subdomains of dense
# chains; convolutions of 64 and 128 columns, clipped windows, gradients, split neurons
CASES = [
    (test_split_products_gpu, "test_tile_edges", ([127, 129, 128, 10],)),
    (test_split_products_gpu, "test_constants_over_changing_widths", ([20, 700, 40, 260, 90, 3],)),
    (test_split_products_gpu, "test_constants_over_changing_widths", ([20, 30, 200, 500, 66, 64, 2],)),
    (test_split_products_gpu, "test_every_tile_shape_gives_the_same_bits", ()),
    (test_alpha_gpu, "test_alpha_eval_and_gradient_match_oracle", ()),
    (test_alpha_gpu, "test_alpha_chunked_equals_whole", ()),
    (test_alpha_gpu, "test_alpha_mlp784x1024x6_full_batch", ()),
    (test_beta_gpu, "test_beta_subdomains_match_oracle", ()),
    (test_beta_gpu, "test_beta_deep_domains_one_layer", ()),
    (test_beta_gpu, "test_beta_bench_size_batches", ()),
    (test_bab_gpu, "test_bab_edge_cases", ()),
    (test_bab_gpu, "test_bab_many_splits_per_layer", ()),
    (test_bab_gpu, "test_bab_4096_domains_sampled", ()),
    (test_conv_gpu, "test_windows_larger_than_the_image", (6, 32, 128)),
    (test_alpha_conv_gpu, "test_alpha_conv_eval_and_gradient_match_oracle", (0,)),
    (test_alpha_conv_gpu, "test_alpha_conv_eval_and_gradient_match_oracle", (1,)),
    (test_beta_conv_gpu, "test_conv_subdomain_crown_matches_oracle", (0,)),
    (test_beta_conv_gpu, "test_conv_beta_subdomains_match_oracle", (1,)),
]


@pytest.mark.parametrize("module,name,args", CASES, ids=lambda v: v if isinstance(v, str) else
                         v.__name__.split(".")[-1] if hasattr(v, "__name__") else "-".join(map(str, v)))
def test_float32(module, name, args, monkeypatch):
    monkeypatch.setattr(module, "gpu_ctx", ctx_with("float32"))
    getattr(module, name)(*args)


def test_middle_tiles_and_large_layer_ibp():
    """5120 rows (the 64 x 64 tiles) against each input alone (the smallest ones), and the interval
    step of a layer of 2^24 weights as a float32 product."""
    wl = random_mlp(933, [300, 320, 320, 11], 8, 0.01)
    ctx = ctx_with("float32")(wl.net)
    lb, ub, layers = gpu_crown(ctx, wl)
    for b in (0, 7):
        l1, u1, _ = gpu_crown(ctx, wl, inputs=[b])
        assert np.array_equal(l1[0], lb[b]) and np.array_equal(u1[0], ub[b])
        check_input(wl.net, wl.x0[b], wl.eps, wl.C[b], lb[b], ub[b], [(l[b], u[b]) for l, u in layers])
    big = random_mlp(934, [4096, 4100, 2], 2, 0.001)
    a = [np.stack([t.cpu().numpy() for t in ctx_with(p)(big.net).ibp_bounds(to_dev(big.x0), big.eps, to_dev(big.C))])
         for p in ("float32", "split")]
    gpu_util.assert_close(a[0], a[1].astype(np.float64), "interval bounds")
    assert not np.array_equal(a[0], a[1])   # the two are different sums


def test_the_loaded_network_keeps_its_products():
    wl = random_mlp(935, [100, 150, 150, 5], 2, 0.02)
    runs = {p: gpu_crown(ctx_with(p)(wl.net), wl) for p in PRODUCTS}
    assert not np.array_equal(runs["split"][0], runs["float32"][0])
    ctx = ctx_with("split")(wl.net)
    ctx.set_option(OPT_PRODUCTS, PRODUCTS["float32"])
    assert np.array_equal(gpu_crown(ctx, wl)[0], runs["split"][0])
    ctx.load_net(wl.net)
    assert np.array_equal(gpu_crown(ctx, wl)[0], runs["float32"][0])
