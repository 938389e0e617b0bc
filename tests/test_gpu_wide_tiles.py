"""The 256-row tiles of eight wavefronts in forward products: contractions of one to six slabs of 64 and one octet more or
less (prologue, steady loop and last slabs of the ring of 256 x 256), of nine and ten (256 x 128, which the cost model
gives nothing shorter), an output whose last tile is one octet wide (wavefronts with nothing to compute).  FC1 takes the
256 x 256 tile in the first kind of layer below and 256 x 128 in the second.  Against the fp64 oracle at the suite's
tolerance, and under full recomputation with the same bits."""
import numpy as np
import pytest

import lynx_synth as synth
from oracle import lynx_oracle as orc
from oracle import policy_model as pm
from harness import GpuLayer, rel_err
from test_gpu_product_edges import TOL, run

B = pytest.importorskip("paper_2406_08756_amd.binding")
import forms

# (hidden, heads, head_dim, ffn, seq, micro_batch), bf16; the last: rows of 2^22 elements and more, which the tile with
# 64-bit load offsets takes
SHAPES = ([(h, 8, 64, 1032, 128, 64) for h in (64, 72, 128, 136, 192, 200, 256, 264, 328, 392)] +
          [(h, 8, 64, 2656, 248, 12) for h in (520, 576, 584)] + [(8, 1, 8, (1 << 22) + 72, 24, 1)])


@pytest.mark.parametrize("shape", SHAPES[:-1], ids=lambda s: "h%d_f%d" % (s[0], s[3]))
def test_form(shape):
    assert forms.of_layer(shape, "fc1") == (256, 256 if shape[3] == 1032 else 128, 1)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "h%d_f%d" % (s[0], s[3]))
def test_layer(shape):
    cfg = synth.LayerConfig(synth.BF16, *shape, tp_size=2, tp_rank=1, seed=7, layer_id=3)
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
