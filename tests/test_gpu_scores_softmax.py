"""Operators 3 to 5 in one launch against the kernels that form S, P and Pd one after the other, bit for bit: row
blocks of 32, column blocks of 64, wavefronts with and without a second or fourth block, head dimensions around 64 and
128, and the first lengths on both sides of every form (512, 1024 and 2048).  With 16384 rows and more the separate softmax
takes 16 or 32 lanes per row, with one to eight vectors each, and with many slices the separate scores run over two or four
tiles per workgroup."""
import numpy as np
import pytest
import torch

import lynx_synth as synth
from oracle import policy_model as pm
from harness import GpuLayer

B = pytest.importorskip("paper_2406_08756_amd.binding")
import forms

# (heads, head_dim, seq, micro_batch)
SHAPES = [(1, 64, 8, 1), (2, 40, 40, 2), (3, 64, 64, 1), (1, 72, 72, 3), (2, 128, 96, 2), (2, 128, 128, 1), (9, 56, 136, 1),
          (2, 64, 512, 2), (2, 64, 520, 1), (1, 128, 512, 1), (2, 104, 328, 1), (3, 64, 1000, 1), (2, 128, 1024, 1),
          (1, 128, 1032, 1), (2, 64, 1088, 1), (1, 96, 1992, 1), (2, 128, 2048, 1), (1, 64, 2048, 2)]
# 16384 rows and more, and tiles per workgroup of the separate scores
MANY_ROWS = {(16, 8, 128, 8): 1, (11, 8, 200, 8): 1, (10, 8, 328, 5): 1, (22, 8, 328, 8): 4, (22, 72, 328, 8): 4, (15, 40, 520, 4): 2,
             (32, 64, 512, 4): 4, (17, 8, 1000, 1): 1, (20, 64, 1024, 2): 2, (22, 64, 1024, 2): 4, (13, 8, 1288, 1): 1}


def test_forms():
    for (a, d, s, b), run in MANY_ROWS.items():
        assert a * b * s >= 16384 and forms.score_run(s, a * b) == run, (a, d, s, b, forms.score_run(s, a * b))
        assert forms.attention(s, d, b, a) & forms.SCORES


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES + list(MANY_ROWS), ids=lambda s: "a%d_d%d_s%d_b%d" % s)
def test_bits_of_the_separate_kernels(shape):
    a, d, s, b = shape
    cfg = synth.LayerConfig(synth.BF16, 64, a, d, 64, s, b, tp_size=2, tp_rank=1, seed=11, layer_id=5)
    layer = GpuLayer(cfg, synth.make_params(cfg, random_ln=True), workspace_bytes=B.lynx_workspace_bytes(cfg, pm.STORE_ALL))
    # (parameters of deviation 1/8 here: scores that spread, rows far from uniform)
    for k, v in layer.params.items():
        v.mul_(6.0) if k == "wqkv" else None
    X = synth.make_x(cfg)
    lower = torch.tril(torch.ones(s, s, dtype=torch.bool, device="cuda"))
    pad = torch.arange(s, device="cuda")[None, :] < (torch.arange(s, device="cuda")[:, None] // 128 + 1) * 128

    defined = {3: lower, 4: pad, 5: pad}

    def tensor(act):
        t = layer.activation_raw(act)
        return None if t is None else t.view(torch.int16).view(b * a, s, s).masked_fill(~defined[act], 0)

    layer.workspace.fill_(0xFF)              # NaNs: nothing may be read, or left, that was not written
    layer.forward(X, pm.STORE_ALL, step=3)
    one = {act: tensor(act) for act in defined}
    B.lynx_layer_reset(layer.handle)
    for segments in ((8, 16, 32), (8, 0x30), (0x18, 32), (0x38,)):
        layer.workspace.fill_(0xFF)
        # forward without any of the three, QKV kept, then the segments
        layer.forward(X, 0x2001 | 4, step=3)
        compared = set()
        for seg in segments:
            B.lynx_recompute(layer.handle, seg)
            torch.cuda.synchronize()
            for act in defined:
                if (seg >> act) & 1 and (got := tensor(act)) is not None:
                    assert torch.equal(got, one[act]), (segments, act)
                    compared.add(act)
        # (S goes when P is there: it is seen where it is regenerated alone)
        assert compared == ({3, 4, 5} if segments[0] == 8 else {4, 5}), segments
        B.lynx_layer_reset(layer.handle)
    # P and Pd from an S that the one launch has kept
    for segments in ((16, 32), (0x30,)):
        layer.workspace.fill_(0xFF)
        layer.forward(X, 0x2001 | 4 | 8, step=3)
        assert torch.equal(tensor(3), one[3])
        for seg in segments:
            B.lynx_recompute(layer.handle, seg)
        torch.cuda.synchronize()
        for act in defined:
            assert torch.equal(tensor(act), one[act]), (segments, act)
        B.lynx_layer_reset(layer.handle)
    p = one[4].view(torch.bfloat16).float().cpu().numpy().astype(np.float64)
    assert np.abs(p.sum(-1) - 1.0).max() <= 2.0 ** -8    # each term rounded once: at most 2^-9 of the sum
    layer.close()
