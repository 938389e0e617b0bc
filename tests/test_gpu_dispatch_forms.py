"""Layers whose sizes send a product, the score kernel or the softmax to a form that the shapes of the other tests do
not reach: every tile of ragged products and gradient pairs with overhang, whole and cut contractions, runs of several
score tiles per workgroup, 16 and 32 lanes per softmax row.  Against the fp64 oracle at the suite's tolerance, and
under full recomputation with the same bits."""
import numpy as np
import pytest

import lynx_synth as synth
from oracle import lynx_oracle as orc
from oracle import policy_model as pm
from harness import GpuLayer, rel_err
from test_gpu_product_edges import TOL, run

B = pytest.importorskip("paper_2406_08756_amd.binding")

pytestmark = pytest.mark.gpu

# name: (hidden, heads, head_dim, ffn, seq, micro_batch), bf16.  The products' names are what the cost model chooses
# for one of theirs; "residual" are those whose store pass adds bias, dropout and residual.
SHAPES = {
    "product_128_cut": (3104, 2, 40, 2232, 912, 1),
    "product_256": (496, 1, 104, 3304, 1232, 2),
    "product_256_cut": (3152, 6, 104, 288, 1136, 2),
    "product_256x128": (72, 2, 40, 2288, 944, 2),
    "product_128x64_cut": (3176, 5, 40, 80, 1272, 2),
    "residual_128_cut": (264, 2, 128, 3568, 1224, 4),
    "residual_256": (1808, 1, 40, 480, 968, 5),
    "residual_256_cut": (2792, 2, 80, 3104, 288, 5),
    "pair_128_both_cut": (88, 1, 128, 2832, 976, 6),
    "pair_256_input_cut": (2936, 2, 40, 3944, 72, 2),
    "pair_256_both_cut": (728, 4, 64, 3264, 1128, 5),
    "pair_256x128": (3024, 5, 104, 448, 1192, 1),
    "pair_256x128_weight_cut": (1184, 2, 40, 720, 888, 4),
    "pair_256x128_input_cut": (1168, 2, 64, 3816, 240, 3),
    # 16384 rows and more: 16 lanes per row with two, four and eight vectors each; 32 lanes, a ragged length
    "softmax_200": (64, 11, 8, 64, 200, 8),
    "softmax_328": (64, 10, 8, 64, 328, 5),
    "softmax_1000": (64, 17, 8, 64, 1000, 1),
    "softmax_1288": (64, 13, 8, 64, 1288, 1),
    # so many slices that a workgroup of the score kernel walks two or up to four tiles
    "score_runs_of_2": (64, 15, 40, 64, 520, 4),
    "score_runs_of_4": (64, 22, 8, 64, 328, 8),
    "score_runs_of_4_head72": (64, 22, 72, 64, 328, 8),
    "score_runs_of_4_whole": (64, 32, 64, 64, 256, 8),
}


@pytest.mark.parametrize("name", list(SHAPES))
def test_layer(name):
    cfg = synth.LayerConfig(synth.BF16, *SHAPES[name], tp_size=2, tp_rank=1, seed=7, layer_id=3)
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
