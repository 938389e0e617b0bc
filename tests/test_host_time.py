"""Time on the host of a pass that is only planned: placing operators 10 and 11 as one launch, which follows what the two
would take before it decides, costs little beside a pass of the same operators that leaves them two."""
import time

import pytest

import lynx_synth as synth
from oracle import policy_model as pm
from test_host_runtime import FOUT, FX, dry_layer

B = pytest.importorskip("paper_2406_08756_amd.binding")

ONE_LAUNCH = [(synth.BF16, 5120, 5, 128, 2560, 128, 1),    # and a cut contraction
              (synth.BF16, 512, 4, 128, 1024, 384, 2)]
TWO = (synth.BF16, 1024, 16, 64, 4096, 1024, 8)


def planner(shape, mask):
    cfg = synth.LayerConfig(*shape)
    h = dry_layer(cfg, ws_bytes=B.lynx_workspace_bytes(cfg, mask))

    def once():
        t = time.perf_counter()
        for _ in range(10):
            B.lynx_layer_forward(h, FX, FOUT, mask, 0)
            B.lynx_layer_reset(h)
        return time.perf_counter() - t
    return h, once


@pytest.mark.parametrize("shape", ONE_LAUNCH)
@pytest.mark.parametrize("mask", [pm.FULL_RECOMPUTE, pm.STORE_ALL])
def test_one_launch_is_planned_as_fast_as_two(shape, mask):
    layers = [planner(shape, mask), planner(TWO, mask)]
    best = [1e9, 1e9]
    for _ in range(300):     # (in turn, the least of many: what else the machine does falls on both)
        best = [min(b, once()) for b, (_, once) in zip(best, layers)]
    for h, _ in layers:
        B.lynx_layer_destroy(h)
    # 1.02 to 1.14; with an arena of ordered trees, copied up to three times for the decision, 1.28 to 1.67
    assert best[0] <= 1.25 * best[1], best
