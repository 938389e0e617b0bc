"""The gradient of the scores where a kernel of its own differentiates the stored dPd: the row dot products come from
the same rounded dPd and P, so what remains against 64 bits is the one rounding of dS."""
import math

import numpy as np
import pytest

import lynx_synth as synth
from oracle import lynx_oracle as orc
from harness import GpuLayer, to_host

B = pytest.importorskip("paper_2406_08756_amd.binding")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("a,d,s,b", [(2, 104, 328, 1), (1, 40, 136, 2), (3, 64, 256, 1), (2, 128, 392, 1), (1, 72, 1024, 1)])
def test_row_dot_products_are_those_of_the_stored_gradient(a, d, s, b):
    cfg = synth.LayerConfig(synth.BF16, 256, a, d, 128, s, b, tp_size=2, tp_rank=1, seed=7)
    layer = GpuLayer(cfg, synth.make_params(cfg, random_ln=True))
    taps = layer.tap_gradients(["dC", "dS"])
    layer.forward(synth.make_x(cfg), B.LYNX_RETAIN_STORE_ALL, step=2)
    qkv, P = layer.activation(2), np.tril(layer.activation(4))
    layer.backward(synth.make_dout(cfg))
    dC = to_host(taps["dC"]).reshape(cfg.tokens, cfg.proj)
    dS = np.tril(to_host(taps["dS"]).reshape(P.shape))
    layer.close()
    c = 1.0 / (1.0 - float(np.float32(cfg.dropout_p)))
    for bi in range(b):
        rows = slice(bi * s, (bi + 1) * s)
        for hd in range(a):
            v = qkv[rows, 2 * cfg.proj + hd * d:2 * cfg.proj + (hd + 1) * d]
            dPd = synth.round_to_bf16(dC[rows, hd * d:(hd + 1) * d] @ v.T).astype(np.float64)
            dP = orc.attention_mask_slice(cfg, 2, bi, hd) * dPd * c
            p = P[bi, hd]
            ref = p * (dP - (dP * p).sum(axis=1, keepdims=True)) / math.sqrt(d)
            # (one rounding to 8 bits is at most 2^-9 of every element.  A dPd that fp32 sums put on the other side
            # of a rounding boundary differs by 2^-8; one in some thousands does)
            assert np.linalg.norm(dS[bi, hd] - ref) <= 2.0 ** -9 * np.linalg.norm(ref), (bi, hd)
