"""A workspace that has room for the column sums' partial sums, each in a hole of its own, but neither for those of a
cut contraction (33 MB, for FC2's input gradient, at the named size) nor for the one larger scratch that serves the
column sums in turn.  It is accepted, and the bits are those of the named size."""
import pytest
import torch

import lynx_synth as synth
from harness import GpuLayer
from test_host_runtime import FAKE, FDOUT, FDX, FOUT, FX, dry_layer

B = pytest.importorskip("paper_2406_08756_amd.binding")

CFG = synth.LayerConfig(synth.BF16, 2304, 18, 128, 9216, 448, 4, seed=3)
MASK = 0x235D
SIZES = (256256000, 260384768)


@pytest.mark.parametrize("size", SIZES)
def test_accepted(size):
    assert B.lynx_workspace_bytes(CFG, MASK) > size
    h = dry_layer(CFG, ws_bytes=size)
    B.lynx_layer_forward(h, FX, FOUT, MASK, 0)
    B.lynx_recompute(h, B.LYNX_SEG_ALL_MISSING)
    B.lynx_layer_backward(h, FDOUT, FDX, FAKE)
    assert B.lynx_layer_peak_bytes(h) <= size
    B.lynx_layer_destroy(h)


@pytest.mark.gpu
def test_same_bits_as_in_the_named_size():
    params, X, dOUT = synth.make_params(CFG, random_ln=True), synth.make_x(CFG), synth.make_dout(CFG)
    runs = []
    for size in (B.lynx_workspace_bytes(CFG, MASK),) + SIZES:
        layer = GpuLayer(CFG, params, workspace_bytes=size)
        layer.workspace.fill_(0xFF)              # NaNs: nothing may be read that was not written
        layer.forward(X, MASK)
        layer.recompute(B.LYNX_SEG_ALL_MISSING)
        layer.backward(dOUT)
        torch.cuda.synchronize()
        end = layer.ws_base + size - layer.workspace.data_ptr()
        assert bool((layer.workspace[end:] == 0xFF).all())
        runs.append([layer.out.clone(), layer.dx.clone()] + [layer.grads[k].clone() for k in synth.PARAM_NAMES])
        layer.close()
    for run in runs[1:]:
        assert all(torch.equal(p, q) for p, q in zip(runs[0], run))
