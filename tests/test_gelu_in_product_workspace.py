"""Operators 10 and 11 in one launch take no more of a workspace than the two do, one after the other: the sizes named
for a policy, and the peaks that a rehearsal of any sequence reports, are those of the library that knew the two only."""
import pytest

import lynx_synth as synth
from test_host_runtime import FAKE, FDOUT, FDX, FOUT, FX, dry_layer

B = pytest.importorskip("paper_2406_08756_amd.binding")

# (dtype, hidden, heads, head_dim, ffn, seq, micro_batch), flags, retain mask, phases, bytes named for the two operators.
# FC1's contraction is cut and neither G nor V2 is kept: Y2, U, G and the partial sums at once are more than that.
NAMED = [((synth.BF16, 4168, 1, 40, 10240, 128, 2), 0, 0x2001, (), 44030208),
         ((synth.BF16, 6944, 1, 128, 21504, 80, 2), 0, 0x2001, (), 56838656),
         ((synth.BF16, 2888, 1, 64, 10384, 64, 2), 0, 0x21ED, (), 22356992),
         ((synth.BF16, 2240, 1, 40, 8704, 136, 1), 0, 0x269F, (), 19168256),      # U is kept
         ((synth.BF16, 5384, 1, 96, 12928, 48, 2), 1, 0x2615, (), 25497600),
         ((synth.BF16, 5168, 40, 128, 17280, 96, 2), 0, 0x27BF, (), 66368768),
         ((synth.BF16, 5632, 1, 64, 21184, 64, 2), 0, 0x27EB, (0x282C, 0, 0, 0), 43830272)]

# The peak of the forward pass alone in a workspace with room to spare; contractions that are cut and that are not.
FORWARD_PEAK = [((synth.F32, 128, 1, 104, 64, 192, 2), 0, 0x2457, 1665024),
                ((synth.BF16, 128, 1, 40, 128, 128, 1), 0, 0x2001, 110592),
                ((synth.BF16, 1408, 1, 40, 768, 512, 2), 0, 0x2001, 7438336),
                ((synth.BF16, 3392, 7, 64, 1408, 256, 3), 0, 0x2001, 13320192),
                ((synth.BF16, 1280, 10, 128, 1408, 192, 7), 0, 0x21C1, 24095232)]


def config(shape, flags):
    return synth.LayerConfig(*shape, tp_size=2, flags=flags)


@pytest.mark.parametrize("shape,flags,mask,phases,size", NAMED)
def test_named_sizes(shape, flags, mask, phases, size):
    cfg = config(shape, flags)
    assert B.lynx_workspace_bytes_for_schedule(cfg, mask, phases or (0, 0, 0, 0)) == size
    for room in (0, 1 << 30):
        h = dry_layer(cfg, ws_bytes=size + room)
        for _ in range(2):
            B.lynx_layer_forward(h, FX, FOUT, mask, 0)
            for segment in phases:
                if segment:
                    B.lynx_recompute(h, segment)
            B.lynx_layer_backward(h, FDOUT, FDX, FAKE)
            assert B.lynx_layer_peak_bytes(h) == size
        B.lynx_layer_destroy(h)


@pytest.mark.parametrize("shape,flags,mask,peak", FORWARD_PEAK)
def test_peak_of_a_forward_pass(shape, flags, mask, peak):
    h = dry_layer(config(shape, flags), ws_bytes=1 << 30)
    B.lynx_layer_forward(h, FX, FOUT, mask, 0)
    assert B.lynx_layer_peak_bytes(h) == peak
    B.lynx_layer_destroy(h)
