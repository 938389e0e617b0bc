"""GeLU and its gradient where they are saturated: pre-activations up to 1e18, whose squares fp32 still holds.
FC1 is zero, so U is its bias, column by column, and the gradient with respect to U is dG or 0."""
import numpy as np
import pytest
import torch

import lynx_synth as synth
from oracle import lynx_oracle as orc
from harness import GpuLayer, rel_err, to_host

B = pytest.importorskip("paper_2406_08756_amd.binding")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [synth.F32, synth.BF16])
def test_saturated_columns(dtype):
    cfg = synth.LayerConfig(dtype, 64, 1, 64, 72, 64, 1, tp_size=2, seed=5)
    params = synth.make_params(cfg, random_ln=True)
    params["w1"][:] = 0.0
    big = [10.0 ** (1 + 0.5 * k) for k in range(35)]             # 10 .. 1e18
    u = np.array(big + [-v for v in big] + [0.0, 1.0])
    params["b1"] = synth._store(u, dtype)
    X, dOUT = synth.make_x(cfg), synth.make_dout(cfg)
    taps = {}
    acts = orc.layer_forward(cfg, params, X)
    grads = orc.layer_backward(cfg, params, acts, dOUT, taps=taps)
    layer = GpuLayer(cfg, params)
    dU = layer.tap_gradients(["dU"])["dU"]
    layer.forward(X, B.LYNX_RETAIN_STORE_ALL)
    G = layer.activation(11)
    layer.backward(dOUT)
    got = layer.results()
    layer.close()
    # (each column by its own largest value: they span eighteen orders of magnitude; one rounding of 2^-9 per
    # element and one in dV2 and dG before it, against fp32's few roundings of 2^-24 times the 64 terms of dG)
    tol = {synth.F32: 1e-5, synth.BF16: 2e-2}[dtype]
    for j in range(len(big)):
        assert rel_err(G[:, j], acts["G"][:, j]) <= tol, u[j]
    assert not G[:, 35:70][:, u[35:70] < -100.0].any()
    dU = to_host(dU).reshape(taps["dU"].shape)
    assert np.isfinite(dU).all()
    assert not dU[:, u < -100.0].any()
    positive = u > 0
    assert rel_err(dU[:, positive], taps["dU"][:, positive]) <= tol
    assert rel_err(got["b1"][positive], grads["b1"][positive]) <= tol
    assert not got["b1"][u < -100.0].any()
