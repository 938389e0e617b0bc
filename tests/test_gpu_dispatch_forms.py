"""Layers whose sizes send a product, the score kernel or the softmax to a form that the shapes of the other tests do
not reach: every tile of ragged products and gradient pairs with overhang, whole and cut contractions, last ranges of one
to four slabs, runs of several score tiles per workgroup, numbers of slices that are no multiple of 8.  Each form is
asserted on the host, so that another choice of tiles fails here instead of passing by it.  Against the fp64 oracle at
the suite's tolerance, under full recomputation with the same bits, and, where a contraction is cut, in the least
workspace, where one workgroup sums its ranges in series in tiles of 64 x 64, with the same bits too."""
import numpy as np
import pytest
import torch

import lynx_synth as synth
from oracle import lynx_oracle as orc
from oracle import policy_model as pm
from harness import GpuLayer, rel_err
from test_gpu_product_edges import TOL, run
from test_small_workspace import least_workspace

B = pytest.importorskip("paper_2406_08756_amd.binding")
import forms

MANY = "more than one range"

# name: (hidden, heads, head_dim, ffn, seq, micro_batch), {product or pair of gradients: its form}, bf16.  A form: rows and
# columns of the tile, ranges (pair: of the weight gradient, of the input gradient; GeLU backward in the latter).
# "residual" are products whose store pass adds bias, dropout and residual.
SHAPES = {
    "product_128_and_64": ((72, 2, 40, 2288, 944, 2), {"fc1": (128, 128, 1), "qkv": (64, 64, 1)}),
    "product_128_cut": ((2280, 1, 8, 12344, 24, 3), {"fc1": (128, 128, MANY), "fc1_grads": (128, 128, 1, MANY, 0)}),
    "product_128x64_cut": ((3176, 5, 40, 80, 1272, 2), {"qkv": (128, 64, MANY), "fc1_grads": (128, 128, MANY, 1, 0)}),
    "product_256": ((496, 1, 104, 3304, 1232, 2), {"fc1": (256, 256, 1)}),
    "product_256_cut": ((7712, 1, 72, 5648, 136, 1), {"fc1": (256, 256, MANY)}),
    "product_256x128": ((3152, 6, 104, 288, 1136, 2), {"qkv": (256, 128, 1), "qkv_grads": (256, 256, 1, 1, 0)}),
    "product_256x128_cut": ((3104, 2, 40, 2232, 912, 1), {"fc1": (256, 128, MANY)}),
    "residual_128_cut": ((72, 1, 8, 6680, 360, 8), {"fc2": (128, 128, MANY), "fc2_grads": (128, 128, MANY, 1, 1)}),
    "residual_128x64_cut": ((16, 1, 8, 4248, 208, 14), {"fc2": (128, 64, MANY)}),
    "residual_256": ((1808, 1, 40, 480, 968, 5), {"proj": (256, 256, 1), "fc2": (256, 256, 1)}),
    "residual_256_cut": ((5744, 1, 72, 7728, 72, 2), {"fc2": (256, 256, MANY)}),
    "residual_256x128": ((2792, 2, 80, 3104, 288, 5), {"fc2": (256, 128, 1), "fc2_grads": (256, 256, 1, 1, 1)}),
    "residual_256x128_cut": ((264, 2, 128, 3568, 1224, 4), {"fc2": (256, 128, MANY)}),
    "pair_64_weight_cut": ((1184, 2, 40, 720, 888, 4), {"proj_grads": (64, 64, MANY, 1, 0)}),
    "pair_128_gelu": ((1168, 2, 64, 3816, 240, 3), {"fc2_grads": (128, 128, 1, 1, 1)}),
    "pair_128_weight_cut_gelu": ((88, 1, 128, 2832, 976, 6), {"fc2_grads": (128, 128, MANY, 1, 1)}),
    "pair_128_input_cut": ((2936, 2, 40, 3944, 72, 2), {"fc1_grads": (128, 128, 1, MANY, 0)}),
    "pair_128_both_cut": ((72, 1, 8, 8024, 464, 3), {"fc1_grads": (128, 128, MANY, MANY, 0)}),
    "pair_256": ((3024, 5, 104, 448, 1192, 1), {"qkv_grads": (256, 256, 1, 1, 0)}),
    "pair_256_gelu": ((136, 1, 72, 14496, 136, 1), {"fc2_grads": (256, 256, 1, 1, 1)}),
    # (two heads of 64: with one of 8, nearly one-hot rows over 24 tokens, rounding to bf16 alone leaves an entry of the
    # query bias gradient off by 2.1 % of the largest of 24, the same in tiles of any size)
    "pair_256_input_cut": ((7080, 2, 64, 3096, 24, 1), {"fc2_grads": (256, 256, 1, MANY, 0)}),
    "pair_256_weight_cut": ((4704, 1, 8, 16, 232, 15), {"fc1_grads": (256, 256, MANY, 1, 0)}),
    "pair_256_weight_cut_gelu": ((728, 4, 64, 3264, 1128, 5), {"fc2_grads": (256, 256, MANY, 1, 1), "fc1_grads": (256, 128, 1, 1, 0)}),
    "pair_256_whole_tiles_weight_cut_gelu": ((1024, 2, 64, 4096, 1024, 4), {"fc2_grads": (256, 256, MANY, 1, 1)}),
    "pair_256x128_gelu": ((2896, 1, 8, 328, 360, 7), {"fc2_grads": (256, 128, 1, 1, 1)}),
    "pair_256x128_weight_cut_gelu": ((2728, 1, 8, 80, 560, 15), {"fc2_grads": (256, 128, MANY, 1, 1)}),
    "pair_256x128_weight_cut": ((264, 1, 8, 2696, 984, 12), {"fc1_grads": (256, 128, MANY, 1, 0)}),
    # the loop of the 256-row tiles with MN-major operands: contractions of one slab with a tail, of three with one (the
    # input gradient), last ranges of one slab and of five, each with a tail (the weight gradient)
    "pair_256_slab_of_16": ((16, 1, 8, 4032, 592, 7), {"fc2_grads": (256, 256, MANY, 1, 1)}),
    "pair_256_last_range_of_1": ((16, 1, 40, 4592, 1064, 4), {"fc2_grads": (256, 256, MANY, 1, 1)}),
    "pair_256_three_slabs": ((2440, 1, 8, 144, 840, 8), {"fc1_grads": (256, 256, MANY, 1, 0)}),
    "pair_256_tokens_392": ((3472, 3, 72, 4032, 56, 7), {"fc1_grads": (256, 256, 1, MANY, 0)}),
    # ... and the ring of three of 256 x 128: last ranges of one to four slabs
    "residual_256x128_last_1": ((72, 1, 8, 10624, 232, 12), {"fc2": (256, 128, 16)}),
    "residual_256x128_last_1_tail": ((72, 1, 8, 10568, 216, 13), {"fc2": (256, 128, 16)}),
    "residual_256x128_last_2_tail": ((72, 1, 40, 10664, 352, 8), {"fc2": (256, 128, 16)}),
    "residual_256x128_last_3": ((72, 1, 8, 10752, 264, 12), {"fc2": (256, 128, 16)}),
    "residual_256x128_last_4_tail": ((72, 1, 72, 9848, 296, 10), {"fc2": (256, 128, 16)}),
    # dQ and dK slice by slice: slices that are no multiple of 8, in each of the three tiles
    "slices_65": ((64, 13, 40, 64, 72, 5), {"slices": 65, "attention": forms.JOINT}),
    "slices_100": ((64, 25, 64, 64, 264, 4), {"slices": 100, "attention": forms.JOINT}),
    "slices_100_head72": ((64, 25, 72, 64, 264, 4), {"slices": 100, "attention": forms.JOINT}),
    # scores of more than 2048 tokens (formed alone, then the softmax), 64 lanes per row with eight vectors each; dPd in
    # runs of two and four tiles where the score gradient is not one launch
    "score_runs_of_2": ((64, 9, 8, 64, 2056, 1), {"run": 2}),
    "score_runs_of_4": ((64, 16, 40, 64, 2056, 1), {"run": 4}),
    "dpd_runs_of_4": ((64, 18, 8, 64, 1032, 2), {"run": 4}),
    "dpd_runs_of_4_head72": ((64, 18, 72, 64, 1032, 2), {"run": 4}),
    # many short slices
    "rows_200": ((64, 11, 8, 64, 200, 8), {}),
    "rows_328": ((64, 10, 8, 64, 328, 5), {}),
    "rows_1000": ((64, 17, 8, 64, 1000, 1), {}),
    "rows_1288": ((64, 13, 8, 64, 1288, 1), {}),
    "rows_520_head40": ((64, 15, 40, 64, 520, 4), {}),
    "rows_328_slices_176": ((64, 22, 8, 64, 328, 8), {}),
    "rows_328_head72": ((64, 22, 72, 64, 328, 8), {}),
    "rows_256_head64": ((64, 32, 64, 64, 256, 8), {}),
}

# So many values that the oracle would take long; the bits of the least workspace alone.
SERIES = {
    "pair_256_both_cut": ((136, 1, 8, 6744, 328, 15), {"fc1_grads": (256, 256, MANY, MANY, 0)}),
    "pair_256x128_input_cut": ((168, 1, 8, 14600, 376, 10), {"fc1_grads": (256, 128, 1, MANY, 0)}),
    "pair_256x128_both_cut": ((16, 1, 8, 9624, 1048, 15), {"fc1_grads": (256, 128, MANY, MANY, 0)}),
}


def config(shape):
    return synth.LayerConfig(synth.BF16, *shape, tp_size=2, tp_rank=1, seed=7, layer_id=3)


def is_cut(want):
    return any(r == MANY or r > 1 for form in want.values() if isinstance(form, tuple) for r in form[2:4 if len(form) > 3 else 3])


@pytest.mark.parametrize("name", list(SHAPES) + list(SERIES))
def test_form(name):
    shape, want = (SHAPES.get(name) or SERIES[name])
    h, a, d, f, s, b = shape
    for which, form in want.items():
        if which == "slices":
            assert a * b == form and form >= 64 and form % 8 != 0
        elif which == "attention":
            assert forms.attention(s, d, b, a) & form
        elif which == "run":
            assert forms.score_run(s, a * b) == form and not forms.attention(s, d, b, a) & forms.GRADIENT
        else:
            got = forms.of_layer(shape, which)
            assert len(got) == len(form) and all(g > 1 if w == MANY else g == w for g, w in zip(got, form)), (which, got, form)


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(SHAPES))
def test_layer(name):
    shape, want = SHAPES[name]
    cfg = config(shape)
    params = synth.make_params(cfg, random_ln=True)
    X, dOUT = synth.make_x(cfg), synth.make_dout(cfg)
    acts, grads = orc.layer_forward_backward(cfg, params, X, dOUT, step=2)
    layer = GpuLayer(cfg, params, workspace_bytes=max(B.lynx_workspace_bytes(cfg, m)
                                                      for m in (pm.STORE_ALL, pm.FULL_RECOMPUTE)))
    layer.workspace.fill_(0xFF)              # NaNs: nothing may be read that was not written
    first = run(layer, X, dOUT, pm.STORE_ALL)
    got = layer.results()
    assert rel_err(layer.out.float().cpu().numpy().astype(np.float64), acts["OUT"]) <= TOL[cfg.dtype]
    for k, ref in grads.items():
        assert rel_err(got[k], ref) <= TOL[cfg.dtype], (k, rel_err(got[k], ref))
    again = run(layer, X, dOUT, pm.FULL_RECOMPUTE)
    assert all((p == q).all() for p, q in zip(first, again))
    layer.close()
    if is_cut(want):
        assert_bits_of_the_least_workspace(cfg, params, X, dOUT, first)


def assert_bits_of_the_least_workspace(cfg, params, X, dOUT, first):
    layer = GpuLayer(cfg, params, workspace_bytes=least_workspace(cfg, pm.FULL_RECOMPUTE))
    layer.workspace.fill_(0xFF)
    least = run(layer, X, dOUT, pm.FULL_RECOMPUTE)
    layer.close()
    differing = [n for n, p, q in zip(("OUT", "dX") + synth.PARAM_NAMES, first, least) if not torch.equal(p, q)]
    assert not differing, differing


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(SERIES))
def test_bits_of_ranges_in_series(name):
    cfg = config(SERIES[name][0])
    gen = torch.Generator(device="cuda").manual_seed(3)
    params = synth.make_params(cfg, random_ln=True)
    X, dOUT = (torch.randn(cfg.tokens, cfg.hidden, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2))
    layer = GpuLayer(cfg, params, workspace_bytes=B.lynx_workspace_bytes(cfg, pm.FULL_RECOMPUTE))
    layer.workspace.fill_(0xFF)
    first = run(layer, X, dOUT, pm.FULL_RECOMPUTE)
    assert all(bool(torch.isfinite(t.float()).all()) for t in first)
    layer.close()
    assert_bits_of_the_least_workspace(cfg, params, X, dOUT, first)
