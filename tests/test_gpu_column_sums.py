"""Bias gradients are sums over the tokens in one order, whatever the tile of the kernel that forms them: 32 rows as
four sums of every fourth row, ((0 + 1) + (2 + 3)); of those partial rows every sixteenth in turn, and the sixteen
sums in order.  Exactly that in numpy's fp32 is the expected result, bit for bit."""
import numpy as np
import pytest
import torch

import forms
import lynx_synth as synth
from harness import GpuLayer

B = pytest.importorskip("paper_2406_08756_amd.binding")

pytestmark = pytest.mark.gpu


def serial(rows):
    total = np.zeros(rows.shape[1:], dtype=np.float32)
    for r in rows:
        total = total + r
    return total


def column_sum(x, dtype):
    x = np.concatenate([x, np.zeros((-len(x) % 32, x.shape[1]), np.float32)]).reshape(-1, 32, x.shape[1])
    four = [serial(np.moveaxis(x[:, q::4], 1, 0)) for q in range(4)]
    partial = (four[0] + four[1]) + (four[2] + four[3])
    return synth._store(serial(np.stack([serial(partial[g::16]) for g in range(16)])), dtype)


# (hidden, seq, micro_batch): tiles of 16 vectors where tiles of 64 would be fewer than 512, of 64 elsewhere
@pytest.mark.parametrize("dtype", [synth.F32, synth.BF16])
@pytest.mark.parametrize("h,s,b", [(256, 128, 2), (264, 40, 5), (136, 1000, 1), (4088, 72, 28), (4104, 72, 28),
                                   (1024, 64, 128), (1032, 88, 93)])
def test_bias_gradients_are_summed_in_one_order(dtype, h, s, b):
    cfg = synth.LayerConfig(dtype, h, 1, 40, 8, s, b, dropout_p=0.0)
    layer = GpuLayer(cfg, synth.make_params(cfg))
    dQKV = layer.tap_gradients(["dQKV"])["dQKV"]
    dOUT = synth.make_dout(cfg)
    layer.forward(synth.make_x(cfg), B.LYNX_RETAIN_STORE_ALL)
    layer.backward(dOUT)
    torch.cuda.synchronize()
    got = {k: layer.grads[k].float().cpu().numpy() for k in ("b2", "bqkv")}
    layer.close()
    np.testing.assert_array_equal(got["b2"], column_sum(dOUT, dtype))
    dQKV = dQKV.float().cpu().numpy().reshape(cfg.tokens, 3 * cfg.proj)
    np.testing.assert_array_equal(got["bqkv"], column_sum(dQKV, dtype))


# (hidden, heads, head_dim, ffn, seq, micro_batch), side of the products' tile: the QKV bias gradient in the launch of the
# products (64) or behind it; whole and part tiles of 64 vectors, last blocks of less than 32 rows
@pytest.mark.parametrize("shape,side", [((264, 5, 104, 64, 72, 3), 64), ((512, 4, 128, 64, 384, 2), 64),
                                        ((3016, 7, 104, 64, 328, 3), 128), ((2048, 16, 128, 64, 1000, 4), 256)])
def test_qkv_bias_gradient_beside_the_products(shape, side):
    assert forms.of_layer(shape, "qkv_grads")[1] == side
    cfg = synth.LayerConfig(synth.BF16, *shape, dropout_p=0.0)
    layer = GpuLayer(cfg, synth.make_params(cfg))
    dQKV = layer.tap_gradients(["dQKV"])["dQKV"]
    layer.forward(synth.make_x(cfg), B.LYNX_RETAIN_STORE_ALL)
    layer.backward(synth.make_dout(cfg))
    torch.cuda.synchronize()
    got = layer.grads["bqkv"].float().cpu().numpy()
    layer.close()
    np.testing.assert_array_equal(got, column_sum(dQKV.float().cpu().numpy().reshape(cfg.tokens, 3 * cfg.proj), synth.BF16))


# a profile names the QKV bias gradient wherever it is a launch of its own, and the products' slot covers the products
@pytest.mark.parametrize("shape,side,apart", [((512, 4, 128, 64, 384, 2), 64, False), ((3016, 7, 104, 64, 328, 3), 128, True),
                                              ((2048, 16, 128, 64, 1000, 4), 256, True)])
def test_qkv_bias_gradient_in_the_profile(shape, side, apart):
    assert forms.of_layer(shape, "qkv_grads")[1] == side
    cfg = synth.LayerConfig(synth.BF16, *shape)
    layer = GpuLayer(cfg, synth.make_params(cfg))
    B.lynx_layer_set_profiling(layer.handle, True)
    layer.forward(synth.make_x(cfg), B.LYNX_RETAIN_STORE_ALL)
    layer.backward(synth.make_dout(cfg))
    slots = B.lynx_layer_profile_ms(layer.handle)
    layer.close()
    assert "b2_qkv_dgrad_wgrad" in slots and ("b2_bias_grad" in slots) == apart


# (hidden, heads, head_dim, ffn, seq, micro_batch), side of the products' tile: fp32, the guest between the products, and
# last where they have a unit each and it would not (248 and 256 of them)
@pytest.mark.parametrize("shape,side", [((640, 10, 64, 64, 432, 1), 32), ((512, 8, 64, 64, 400, 1), 64), ((512, 8, 64, 64, 512, 1), 64),
                                        ((520, 8, 64, 64, 392, 1), 32), ((1000, 15, 64, 64, 1000, 1), 64), ((1280, 10, 128, 64, 200, 1), 64)])
def test_qkv_bias_gradient_beside_fp32_products(shape, side):
    cfg = synth.LayerConfig(synth.F32, *shape, dropout_p=0.0)
    assert forms.f32(cfg.tokens, 3 * cfg.proj, cfg.hidden)[1][0] == side
    layer = GpuLayer(cfg, synth.make_params(cfg))
    layer.workspace.fill_(0xFF)
    taps = layer.tap_gradients(["dQKV", "dY1"])
    layer.forward(synth.make_x(cfg), B.LYNX_RETAIN_STORE_ALL)
    y1 = layer.activation_raw(1).view(cfg.tokens, -1).double()
    layer.backward(synth.make_dout(cfg))
    torch.cuda.synchronize()
    dQKV, dY1 = taps["dQKV"].view(cfg.tokens, -1), taps["dY1"].view(cfg.tokens, -1)
    got, w, dw = layer.grads["bqkv"].cpu().numpy(), layer.params["wqkv"].double(), layer.grads["wqkv"]
    layer.close()
    np.testing.assert_array_equal(got, column_sum(dQKV.cpu().numpy(), synth.F32))
    # (and no tile of the products is missing or done twice: a sum of K products in fp32 is within K 2^-24 sum |a b|)
    dQKV = dQKV.double()
    for out, a, b in ((dY1, dQKV, w), (dw, dQKV.t(), y1)):
        assert bool(((out - a @ b).abs() <= a.shape[1] * 2.0 ** -24 * (a.abs() @ b.abs())).all())
