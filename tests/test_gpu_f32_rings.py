"""fp32 products of linear layers in 64 x 64 tiles with a ring of three and of four stages, around the lines between
them, with contractions of fewer slabs than the ring has stages, of as many, and of more: FC1 and its gradients against
64 bits.  A sum of K products in fp32, in whatever order, is within K 2^-24 sum |a b| of the exact one to first order."""
import pytest
import torch

import forms
import lynx_synth as synth
from harness import GpuLayer

B = pytest.importorskip("paper_2406_08756_amd.binding")

pytestmark = pytest.mark.gpu

# (tokens, ffn, hidden), (tile, stages) of FC1's forward, of its gradients, of FC2's gradients
SHAPES = [((1000, 1016, 8), (64, 4), (32, 4), (32, 4)), ((1000, 1016, 72), (64, 4), (32, 4), (32, 4)),
          ((1000, 1016, 104), (64, 4), (32, 4), (32, 4)), ((1000, 2040, 32), (64, 3), (32, 4), (32, 4)),
          ((1000, 3064, 72), (64, 3), (32, 4), (32, 4)), ((1000, 4480, 136), (64, 3), (32, 4), (32, 4)),
          ((192, 5120, 1280), (64, 4), (64, 4), (64, 3)), ((2000, 4480, 264), (64, 3), (64, 4), (64, 3)),
          ((8, 4480, 4480), (32, 4), (64, 4), (64, 4)), ((1000, 2040, 1000), (64, 3), (64, 3), (64, 4))]


@pytest.mark.parametrize("shape,fc1,fc1_grads,fc2_grads", SHAPES, ids=lambda v: "x".join(map(str, v)))
def test_linear_layer(shape, fc1, fc1_grads, fc2_grads):
    T, f, h = shape
    assert forms.f32(T, f, h) == (fc1, fc1_grads) and forms.f32(T, h, f)[1] == fc2_grads
    cfg = synth.LayerConfig(synth.F32, h, 1, 8, f, 8, T // 8)
    layer = GpuLayer(cfg, synth.make_params(cfg, random_ln=True))
    taps = layer.tap_gradients(["dV2", "dU", "dY2"])
    layer.workspace.fill_(0xFF)
    layer.forward(synth.make_x(cfg), B.LYNX_RETAIN_STORE_ALL, step=2)
    y2, u, g = (layer.activation_raw(i).view(T, -1).double() for i in (9, 10, 11))
    layer.backward(synth.make_dout(cfg))
    torch.cuda.synchronize()
    dv2, du, dy2 = (taps[k].view(T, -1).double() for k in ("dV2", "dU", "dY2"))
    p, gr = {k: v.double() for k, v in layer.params.items()}, {k: v.double() for k, v in layer.grads.items()}
    layer.close()

    def check(got, a, b, bias=None):
        exact, room = a @ b, a.abs() @ b.abs()
        if bias is not None:
            exact, room = exact + bias, room + bias.abs()
        assert bool(((got - exact).abs() <= (a.shape[1] + 1) * 2.0 ** -24 * room).all())

    check(u, y2, p["w1"].t(), p["b1"])
    check(dy2, du, p["w1"])
    check(gr["w1"], du.t(), y2)
    check(gr["w2"], dv2.t(), g)
