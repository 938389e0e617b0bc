"""Workspaces that were named, or just large enough, when FC2's gradients were computed in tiles with fewer column
partials of the GeLU store pass (one row of f floats per 128 rows of the tile, now one per 64 or 32), or when the GeLU
backward was split from that launch elsewhere.  They are accepted, and the bits are those of a roomy workspace."""
import pytest
import torch

import lynx_synth as synth
from harness import GpuLayer
from test_host_runtime import FAKE, FDOUT, FDX, FOUT, FX, dry_layer

B = pytest.importorskip("paper_2406_08756_amd.binding")

# name: (dtype, hidden, heads, head_dim, ffn, seq, micro_batch), flags, retain mask, phases, bytes
CASES = {
    "store_all": ((synth.BF16, 896, 7, 128, 3584, 256, 6), 0, 0x3FFF, (), 77525248),
    "selective_but_s": ((synth.BF16, 896, 7, 128, 3584, 256, 6), 0, 0x37CF, (), 77525248),
    "partials_without_a_hole": ((synth.BF16, 1024, 16, 64, 4096, 128, 4), 0, 0x37CF, (), 29565184),
    "fused_attention": ((synth.BF16, 1024, 8, 128, 4096, 256, 1), 1, 0x2001, (), 10572032),
    "named_with_cut_pairs": ((synth.BF16, 1280, 10, 128, 5120, 128, 2), 0, 0x2001, (), 14524672),
    "gelu_apart": ((synth.BF16, 4096, 8, 128, 4096, 256, 1), 0, 0x3FC7, (), 28332032),
    "gelu_apart_ragged": ((synth.BF16, 896, 5, 96, 1792, 128, 4), 0, 0x2001, (), 13633536),
    "least_of_a_wide_layer": ((synth.BF16, 3840, 30, 128, 15360, 256, 1), 0, 0x37CF, (), 55361792),
    "one_phase": ((synth.BF16, 640, 5, 128, 2560, 256, 7), 0, 0x37CF, (0x2A78,), 64612608),
    "early_gradients_high": ((synth.BF16, 320, 1, 64, 128, 1280, 5), 1, 0x3E37, (0x28C6,), 76236800),
    "phase_f32": ((synth.F32, 512, 2, 64, 512, 80, 3), 0, 0x385B, (0x11A8,), 5506816),
}


def config(name):
    return synth.LayerConfig(*CASES[name][0], tp_size=2, flags=CASES[name][1], seed=7, layer_id=3)


@pytest.mark.parametrize("name", list(CASES))
def test_accepted(name):
    _, _, mask, phases, size = CASES[name]
    h = dry_layer(config(name), ws_bytes=size)
    for _ in range(2):
        B.lynx_layer_forward(h, FX, FOUT, mask, 0)
        for segment in phases:
            B.lynx_recompute(h, segment)
        B.lynx_layer_backward(h, FDOUT, FDX, FAKE)
        assert B.lynx_layer_peak_bytes(h) <= size
    B.lynx_layer_destroy(h)


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["store_all", "fused_attention", "gelu_apart", "gelu_apart_ragged", "early_gradients_high", "phase_f32"])
def test_same_bits_as_in_a_roomy_workspace(name):
    _, _, mask, phases, size = CASES[name]
    cfg = config(name)
    params, X, dOUT = synth.make_params(cfg, random_ln=True), synth.make_x(cfg), synth.make_dout(cfg)
    runs = []
    for nbytes in (2 * B.lynx_workspace_bytes(cfg, mask), size):
        layer = GpuLayer(cfg, params, workspace_bytes=nbytes)
        layer.workspace.fill_(0xFF)              # NaNs: nothing may be read that was not written
        layer.forward(X, mask, step=2)
        for segment in phases:
            layer.recompute(segment)
        layer.backward(dOUT)
        torch.cuda.synchronize()
        end = layer.ws_base + nbytes - layer.workspace.data_ptr()
        assert bool((layer.workspace[end:] == 0xFF).all())
        runs.append([layer.out.clone(), layer.dx.clone()] + [layer.grads[k].clone() for k in synth.PARAM_NAMES])
        layer.close()
    differing = [n for n, p, q in zip(("OUT", "dX") + synth.PARAM_NAMES, *runs) if not torch.equal(p, q)]
    assert not differing, differing
