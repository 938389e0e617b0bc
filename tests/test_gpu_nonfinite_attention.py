"""Infinities and NaN in the kernels that keep scores and their gradient in registers: an element of Q, K or V that is not
finite reaches the rows whose sums it stands in, and no other row changes by a bit; what a row of such scores gives is
what the separate kernels give."""
import pytest
import torch

import lynx_synth as synth
from oracle import policy_model as pm
from harness import GpuLayer

B = pytest.importorskip("paper_2406_08756_amd.binding")
import forms

pytestmark = pytest.mark.gpu

# (heads, head_dim, seq, micro_batch)
SHAPES = [(2, 64, 72, 1), (1, 128, 96, 2), (3, 40, 136, 1), (2, 64, 520, 1), (2, 104, 1000, 1), (1, 128, 1032, 1), (1, 64, 2048, 1)]
INF = float("inf")


def setup(shape, **kw):
    a, d, s, b = shape
    cfg = synth.LayerConfig(synth.BF16, 64, a, d, 64, s, b, tp_size=2, tp_rank=1, seed=11, layer_id=5, **kw)
    layer = GpuLayer(cfg, synth.make_params(cfg, random_ln=True), workspace_bytes=B.lynx_workspace_bytes(cfg, pm.STORE_ALL))
    layer.params["wqkv"].mul_(6.0)
    return cfg, layer


def qkv(layer, cfg):
    """The resident QKV itself: [batch, seq, 3, heads, head_dim]."""
    addr, nbytes = B.lynx_layer_activation(layer.handle, 2)
    off = addr - layer.workspace.data_ptr()
    return layer.workspace[off:off + nbytes].view(torch.bfloat16).view(cfg.micro_batch, cfg.seq, 3, cfg.local_heads, cfg.head_dim)


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "a%d_d%d_s%d_b%d" % s)
def test_scores(shape):
    a, d, s, b = shape
    cfg, layer = setup(shape)
    assert forms.attention(s, d, b, a) & forms.SCORES
    X = synth.make_x(cfg)
    lower = torch.tril(torch.ones(s, s, dtype=torch.bool, device="cuda"))

    def tensors():
        return [layer.activation_raw(act).view(b * a, s, s) for act in (4, 5)]

    def regenerated(segments, spoil):
        layer.workspace.fill_(0xFF)
        layer.forward(X, 0x2001 | 4, step=3)
        if spoil:
            t = qkv(layer, cfg)
            t[0, s // 3, 0, 0] = INF                  # a row of infinities and NaN
            t[0, s // 2, 0, 0] = 3e38                 # overflows to both signs
            t[0, 2 * s // 3, 1, 0, 0] = float("nan")  # a column of NaN, from its diagonal on
            t[0, 0, 0, 0] = -INF * torch.sign(t[0, 0, 1, 0].float())  # the one score of row 0: minus infinity
        for seg in segments:
            B.lynx_recompute(layer.handle, seg)
        torch.cuda.synchronize()
        out = tensors()
        B.lynx_layer_reset(layer.handle)
        return out

    clean, one, apart = regenerated((0x38,), False), regenerated((0x38,), True), regenerated((8, 16, 32), True)
    for got, want, act in zip(one, apart, (4, 5)):
        same = (got.view(torch.int16) == want.view(torch.int16)) | (got.isnan() & want.isnan())
        assert bool((same | ~lower).all()), act
        assert bool((got.isnan() & lower).any())
    # every row of the other slices, and of this one those that are neither spoilt nor reach the spoilt column
    untouched = torch.ones(b * a, s, dtype=torch.bool, device="cuda")
    untouched[0, 2 * s // 3:] = False
    untouched[0, [0, s // 3, s // 2]] = False
    for got, want in zip(one, clean):
        assert bool(((got.view(torch.int16) == want.view(torch.int16)) | ~lower).all(-1)[untouched].all())
    layer.close()


@pytest.mark.parametrize("shape", [s for s in SHAPES if s[2] <= 1024], ids=lambda s: "a%d_d%d_s%d_b%d" % s)
def test_score_gradient(shape):
    a, d, s, b = shape
    cfg, layer = setup(shape)
    assert forms.attention(s, d, b, a) & forms.GRADIENT
    X, dOUT = synth.make_x(cfg), synth.make_dout(cfg)
    keep = torch.empty(b, a, s, s, dtype=torch.uint8, device="cuda")
    B.lynx_dropout_mask(cfg, 3, 0, keep)
    tap = layer.tap_gradients(["dS"])["dS"]
    lower = torch.tril(torch.ones(s, s, dtype=torch.bool, device="cuda"))

    def gradient(j, value):
        layer.workspace.fill_(0xFF)
        layer.forward(X, pm.STORE_ALL, step=3)
        if j is not None:
            qkv(layer, cfg)[0, j, 2, 0] = value
        layer.backward(dOUT)
        torch.cuda.synchronize()
        return tap.view(b, a, s, s).clone()

    clean = gradient(None, 0.0)
    assert bool(torch.isfinite(clean.float()[..., lower]).all())
    # (3e38: a row's sum overflows or not by its own values)
    for j, value in ((0, INF), (s // 2, float("nan")), (s - 1, -INF), (s // 3, 3e38)):
        got = gradient(j, value)
        touched = torch.zeros(b, a, s, dtype=torch.bool, device="cuda")
        touched[0, 0, j:] = keep[0, 0, j:, j] != 0      # a dropped element is none of the row's terms
        unchanged = (got.view(torch.int16) == clean.view(torch.int16)) | ~lower
        assert bool(unchanged.all(-1)[~touched].all()), (j, value)
        spoilt = ~torch.isfinite(got.float())
        if value != 3e38:
            assert bool((spoilt | ~lower)[touched].all()), (j, value)
    layer.close()


# (head dimension 128 and whole tiles: the row sums come from C, so a row of V spoils its column only, a row of C its row;
# four and eight wavefronts, one and several blocks each)
@pytest.mark.parametrize("shape", [(2, 128, 128, 1), (9, 128, 256, 9), (1, 128, 640, 2), (1, 128, 1536, 1), (1, 128, 2048, 1)],
                         ids=lambda s: "a%d_d%d_s%d_b%d" % s)
def test_score_gradient_with_row_sums_from_c(shape):
    a, d, s, b = shape
    cfg, layer = setup(shape)
    assert forms.attention(s, d, b, a) & forms.FROM_C
    X, dOUT = synth.make_x(cfg), synth.make_dout(cfg)
    keep = torch.empty(b, a, s, s, dtype=torch.uint8, device="cuda")
    B.lynx_dropout_mask(cfg, 3, 0, keep)
    tap = layer.tap_gradients(["dS"])["dS"]
    lower = torch.tril(torch.ones(s, s, dtype=torch.bool, device="cuda"))

    def context():
        addr, _ = B.lynx_layer_activation(layer.handle, 6)
        off = addr - layer.workspace.data_ptr()
        return layer.workspace[off:off + cfg.tokens * cfg.proj * 2].view(torch.bfloat16).view(b, s, a, d)

    def gradient(spoil):
        layer.workspace.fill_(0xFF)
        layer.forward(X, pm.STORE_ALL, step=3)
        spoil()
        layer.backward(dOUT)
        torch.cuda.synchronize()
        return tap.view(b, a, s, s).clone()

    clean = gradient(lambda: None)
    assert bool(torch.isfinite(clean.float()[..., lower]).all())

    def check(got, touched, what, spoils=True):
        unchanged = (got.view(torch.int16) == clean.view(torch.int16)) | ~lower
        assert bool((unchanged | touched).all()), what
        if spoils:
            assert bool((~torch.isfinite(got.float()) | ~(touched & lower)).all()), what

    # (3e38: a product overflows or not by its own values)
    for j, value in ((0, INF), (s // 2, float("nan")), (s - 1, -INF), (s // 3, 3e38)):
        touched = torch.zeros(b, a, s, s, dtype=torch.bool, device="cuda")
        touched[0, 0, j:, j] = keep[0, 0, j:, j] != 0      # a dropped element has no part in the gradient
        check(gradient(lambda: qkv(layer, cfg)[0, j, 2, 0].fill_(value)), touched, ("V", j, value), value != 3e38)
        touched.zero_()
        touched[0, a - 1, j] = True
        check(gradient(lambda: context()[0, j, a - 1, 5].fill_(value)), touched, ("C", j, value), value != 3e38)
    layer.close()
