"""dS formed in the launch that forms dPd, at the edges of its row blocks of 32, column blocks of 64 and forms (up to 256
and 512 columns, few and many workgroups, 1024): against the same formula in float64 on the tensors that the layer itself
holds (rounded C gradient, V, P), dropout masks from the library.  Tolerance: dPd and dS are rounded once each (2^-9
relative), dPd's error enters scale P (dP - dot) by |P| |dP|, and the row sum carries that of all its terms: 2^-8 of the
largest |P| |dP| of the row plus 2^-8 of the value, one bit more for the sums in 32 bits."""
import numpy as np
import pytest
import torch

import lynx_synth as synth
from oracle import policy_model as pm
from harness import GpuLayer

B = pytest.importorskip("paper_2406_08756_amd.binding")

pytestmark = pytest.mark.gpu

# (heads, head_dim, seq, micro_batch)
SHAPES = [(1, 64, 8, 1), (2, 40, 40, 2), (3, 64, 64, 1), (1, 72, 72, 3), (2, 96, 96, 2), (9, 56, 136, 1), (3, 104, 256, 2),
          (2, 64, 264, 1), (2, 64, 512, 2), (40, 64, 512, 1), (40, 80, 328, 1), (2, 64, 520, 1), (3, 64, 1000, 1),
          (1, 128, 1000, 1), (2, 96, 1024, 1), (2, 64, 1024, 2)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "a%d_d%d_s%d_b%d" % s)
def test_against_the_formula(shape):
    a, d, s, b = shape
    cfg = synth.LayerConfig(synth.BF16, 64, a, d, 64, s, b, tp_size=2, tp_rank=1, seed=11, layer_id=5, dropout_p=0.1)
    layer = GpuLayer(cfg, synth.make_params(cfg, random_ln=True), workspace_bytes=B.lynx_workspace_bytes(cfg, pm.STORE_ALL))
    layer.params["wqkv"].mul_(6.0)     # rows far from uniform
    layer.workspace.fill_(0xFF)
    taps = layer.tap_gradients(["dC", "dS"])
    layer.forward(synth.make_x(cfg), pm.STORE_ALL, step=3)
    p = layer.activation_raw(4).view(b, a, s, s).double()
    v = layer.activation_raw(2).view(b, s, 3, a, d)[:, :, 2].permute(0, 2, 1, 3).double()
    layer.backward(synth.make_dout(cfg))
    torch.cuda.synchronize()
    dc = taps["dC"].view(b, s, a, d).permute(0, 2, 1, 3).double()
    keep = torch.empty(b, a, s, s, dtype=torch.uint8, device="cuda")
    B.lynx_dropout_mask(cfg, 3, 0, keep)
    lower = torch.tril(torch.ones(s, s, dtype=torch.bool, device="cuda"))
    dp = torch.where(lower & (keep != 0), dc @ v.transpose(-1, -2).contiguous() / (1.0 - np.float32(0.1)), 0.0)
    p = torch.where(lower, p, 0.0)
    want = (p * (dp - (dp * p).sum(-1, keepdim=True))) / np.sqrt(d)
    ds = taps["dS"].view(b, a, s, s).double()
    got = torch.where(lower, ds, 0.0)
    scale = (p * dp.abs()).amax(-1, keepdim=True) / np.sqrt(d)
    assert ((got - want).abs() <= 2.0 ** -8 * (want.abs() + 2.0 * scale) + 1e-30).all()
    # zeros up to the next multiple of 128 columns, which dQ and dK read
    pad = torch.arange(s, device="cuda")[None, :] < (torch.arange(s, device="cuda")[:, None] // 128 + 1) * 128
    assert (ds.masked_fill(~(pad & ~lower), 0.0) == 0).all()
    layer.close()
