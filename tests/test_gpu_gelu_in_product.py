"""Operators 10 and 11 in one launch and as two: the same bits of U and G, whether U is written or not, in every kind of
tile that carries GeLU, with and without cut contractions; OUT of a forward pass that keeps neither."""
import pytest
import torch

import forms
import lynx_synth as synth
from oracle import policy_model as pm
from paper_2406_08756_amd import binding as B
from harness import GpuLayer

pytestmark = pytest.mark.gpu

# name: (dtype, hidden, heads, head_dim, ffn, seq, micro_batch), (columns of FC1's tile, its ranges), in one launch where U and G are kept
SHAPES = {
    "f32_32": ((synth.F32, 72, 1, 40, 104, 40, 1), None, True),
    "f32_64": ((synth.F32, 264, 2, 72, 4104, 264, 2), None, True),
    "bf16_64": ((synth.BF16, 136, 1, 64, 200, 72, 3), (64, 1), True),
    "bf16_64_whole": ((synth.BF16, 256, 2, 64, 512, 128, 2), (64, 1), True),
    "bf16_cut": ((synth.BF16, 4104, 1, 64, 328, 24, 1), (64, 0), False),  # where G is kept, partial sums are in its way
    "bf16_128": ((synth.BF16, 264, 2, 64, 2056, 1000, 1), (0, 1), True),
    "bf16_256": ((synth.BF16, 1024, 2, 64, 4096, 1024, 4), (256, 1), False),
}


@pytest.mark.parametrize("name", list(SHAPES))
def test_u_and_g(name):
    shape, form, joint = SHAPES[name]
    if form is not None:
        _, columns, ranges = forms.of_layer(shape[1:], "fc1")
        assert columns == form[0] or form[0] == 0 and 64 <= columns <= 128
        assert ranges == form[1] or form[1] == 0 and ranges > 1
    carries = name != "bf16_256"
    cfg = synth.LayerConfig(*shape, tp_size=2, seed=11)
    params, X = synth.make_params(cfg, random_ln=True), synth.make_x(cfg)
    both, neither = pm.STORE_ALL, pm.STORE_ALL & ~0xC00
    layer = GpuLayer(cfg, params, workspace_bytes=max(B.lynx_workspace_bytes(cfg, m) for m in (both, neither, pm.FULL_RECOMPUTE)))
    B.lynx_layer_set_profiling(layer.handle, True)

    def forward(mask):
        layer.workspace.fill_(0xFF)
        layer.forward(X, mask)
        slots = B.lynx_layer_profile_ms(layer.handle)
        return layer.out.clone(), "op11_gelu" not in slots

    out, one_launch = forward(both)
    assert one_launch == joint
    u, g = layer.activation_raw(10), layer.activation_raw(11)
    B.lynx_layer_reset(layer.handle)
    for segments in ((1 << 10, 1 << 11), (0xC00,)):
        assert torch.equal(forward(neither)[0], out)
        assert layer.activation_raw(10) is None
        for s in segments:
            layer.recompute(s)
        assert ("op11_gelu" not in B.lynx_layer_profile_ms(layer.handle)) == (carries and len(segments) == 1)
        assert torch.equal(layer.activation_raw(10), u) and torch.equal(layer.activation_raw(11), g)
        B.lynx_layer_reset(layer.handle)
    again, one_launch = forward(pm.FULL_RECOMPUTE)   # U is not written, G lies wherever there is room
    assert one_launch == carries and torch.equal(again, out)
    layer.close()
