"""dS in one launch with its row sums from C (head dimension 128, whole tiles): the gradients of a layer have the bits of the
kernels that rebuild P and take the row sums from a launch of their own (the attention option, which runs where none
of S, P and Pd is kept), at one and several blocks per wavefront, few and many workgroups, both numbers of wavefronts."""
import pytest
import torch

import forms
import lynx_synth as synth
from oracle import policy_model as pm
from paper_2406_08756_amd import binding as B
from harness import GpuLayer

pytestmark = pytest.mark.gpu

# (heads, seq, micro_batch)
SHAPES = [(1, 128, 1), (3, 128, 2), (8, 256, 8), (9, 256, 9), (2, 384, 1), (16, 512, 2), (5, 640, 1), (2, 1024, 2), (1, 1920, 1), (4, 2048, 4),
          (1, 1536, 1), (2, 768, 3), (3, 2048, 1)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "a%d_s%d_b%d" % s)
def test_bits_of_the_kernels_with_row_sums_of_their_own(shape):
    a, s, b = shape
    assert forms.attention(s, 128, b, a) & forms.FROM_C
    cfg = synth.LayerConfig(synth.BF16, 64, a, 128, 64, s, b, tp_size=2, tp_rank=1, seed=11, layer_id=5,
                            flags=B.LYNX_FLAG_FUSED_ATTENTION)
    apart = pm.STORE_ALL & ~0x38
    layer = GpuLayer(cfg, synth.make_params(cfg, random_ln=True),
                     workspace_bytes=max(B.lynx_workspace_bytes(cfg, m) for m in (pm.STORE_ALL, apart)))
    layer.params["wqkv"].mul_(6.0)     # rows far from uniform
    X, dOUT = synth.make_x(cfg), synth.make_dout(cfg)
    runs = []
    for mask in (pm.STORE_ALL, apart, pm.STORE_ALL):
        layer.workspace.fill_(0xFF)
        layer.forward(X, mask, step=3)
        layer.backward(dOUT)
        torch.cuda.synchronize()
        runs.append([layer.dx.clone()] + [layer.grads[k].clone() for k in synth.PARAM_NAMES])
    assert all(bool(torch.isfinite(t).all()) for t in runs[0])
    for other in runs[1:]:
        assert all(torch.equal(p, q) for p, q in zip(runs[0], other))
    layer.close()


@pytest.mark.parametrize("seq,micro_batch,heads,from_c", [(2048, 4, 4, True), (2048, 17, 1, False), (1024, 8, 8, True),
                                                          (1024, 13, 5, False), (1000, 1, 1, False), (2176, 1, 1, False)])
def test_the_line(seq, micro_batch, heads, from_c):
    assert bool(forms.attention(seq, 128, micro_batch, heads) & forms.FROM_C) == from_c


# (many short rows)
@pytest.mark.parametrize("seq,micro_batch,heads,from_c", [(512, 4, 48, True), (512, 4, 64, False), (128, 48, 16, True), (128, 64, 16, False)])
def test_the_line_of_rows(seq, micro_batch, heads, from_c):
    assert bool(forms.attention(seq, 128, micro_batch, heads) & forms.FROM_C) == from_c


# (heads, seq, batches beyond the line, batches of them below it)
@pytest.mark.parametrize("a,s,more,fewer", [(3, 2048, 6, 5), (5, 1024, 13, 12), (8, 384, 57, 2), (1, 256, 1025, 3)])
def test_bits_of_the_two_launches_beyond_the_line(a, s, more, fewer):
    assert not forms.attention(s, 128, more, a) & forms.FROM_C and forms.attention(s, 128, fewer, a) & forms.FROM_C
    X = dOUT = None
    got = []
    for b in (more, fewer):
        shape = (64, a, 128, 64, s, b)
        for which in ("qkv", "proj", "fc1", "fc2"):     # (nothing ahead of dS is cut in one and not in the other)
            assert forms.of_layer(shape, which)[2] == 1 and (which == "qkv" or forms.of_layer(shape, which + "_grads")[3] == 1)
        cfg = synth.LayerConfig(synth.BF16, *shape, tp_size=2, tp_rank=1, seed=11, layer_id=5)
        layer = GpuLayer(cfg, synth.make_params(cfg, random_ln=True))
        layer.params["wqkv"].mul_(6.0)
        if X is None:
            X, dOUT = synth.make_x(cfg), synth.make_dout(cfg)
        tap = layer.tap_gradients(["dS"])["dS"]
        layer.workspace.fill_(0xFF)
        layer.forward(X[:cfg.tokens], pm.STORE_ALL, step=3)
        layer.backward(dOUT[:cfg.tokens])
        torch.cuda.synchronize()
        got.append(tap.view(b, a, s, s)[:fewer].tril())
        layer.close()
    assert torch.equal(got[0].view(torch.int16), got[1].view(torch.int16))
