"""Tile indices divided by the host's inverses: exact up to the largest index that the inverse is made for, and beyond
what an inverse can do by an ordinary division."""
import random

import numpy as np
import pytest
import torch

import forms
import lynx_synth as synth
from harness import GpuLayer


@pytest.mark.parametrize("d", [1, 2, 3, 5, 7, 8, 24, 96, 1000, 4095, 4096, 46339, 46341, 65535, (1 << 20) + 1, (1 << 30) - 1])
def test_quotients_are_exact(d):
    limit = ((1 << 31) - 1) // d           # the largest index an inverse of d is made for
    rng = random.Random(d)
    xs = {0, 1, d - 1, d, d + 1, limit - 1, limit} | {rng.randrange(limit + 1) for _ in range(2000)}
    xs |= {q * d + e for q in (1, 2, limit // d, rng.randrange(limit // d + 1)) for e in (-1, 0, 1)}
    for x in (x for x in xs if 0 <= x <= limit):
        assert forms.quotient(x, d, limit) == (x // d, True), x


@pytest.mark.parametrize("d", [2, 3, 1000, (1 << 20) + 1])
def test_larger_indices_are_divided(d):
    most = (1 << 31) // d + 1
    for x in (0, d, most - 1, most, (1 << 31) - 1):
        assert forms.quotient(x, d, most) == (x // d, False), x


# so many slices that the kernels of attention divide their tile indices: by the slices, by the heads, by both
@pytest.mark.gpu
@pytest.mark.parametrize("a,b", [(30, 1600), (40000, 2)])
def test_attention_of_indices_that_are_divided(a, b):
    s, d, period = 8, 8, 5
    assert not forms.quotient(a * b - 1, a * b, a * b - 1)[1]
    assert forms.quotient(a * b - 1, a, a * b - 1)[1] == (a < 40000)

    def layer_of(heads, batches):
        cfg = synth.LayerConfig(synth.BF16, 8, heads, d, 64, s, batches, dropout_p=0.0)
        of = synth.LayerConfig(synth.BF16, 8, period, d, 64, s, 2, dropout_p=0.0)   # ... and what it repeats
        params, n = synth.make_params(of, random_ln=True), heads // period
        params["wqkv"] = np.tile(params["wqkv"].reshape(3, -1, 8), (1, n, 1)).reshape(-1, 8)
        params["bqkv"] = np.tile(params["bqkv"].reshape(3, -1), (1, n)).reshape(-1)
        params["wo"] = np.tile(params["wo"], (1, n))
        layer = GpuLayer(cfg, params)
        taps = layer.tap_gradients(["dS", "dQKV"])
        layer.workspace.fill_(0xFF)
        layer.forward(np.tile(synth.make_x(of), (batches // 2, 1)), 0x3FFF, step=3)
        c = layer.activation_raw(6).view(batches, s, heads, d).transpose(1, 2)
        layer.backward(np.tile(synth.make_dout(of), (batches // 2, 1)))
        torch.cuda.synchronize()
        layer.close()
        dqkv = taps["dQKV"].view(batches, s, 3, heads, d).transpose(1, 3)
        return c, taps["dS"].view(batches, heads, s, s).tril(), dqkv

    large = layer_of(a, b)
    # (of many heads the projection is a longer sum, so what follows the context is compared with its own first heads)
    small = layer_of(a if b > 2 else period, 2)
    for i, (got, want) in enumerate(zip(large, small)):
        if b == 2 and i > 0:
            want = got[:, :period]
        assert bool(torch.isfinite(want.float()).all()) and bool((want != 0).any())
        n = got.shape[0] // want.shape[0], got.shape[1] // want.shape[1]
        assert torch.equal(got, want.repeat(*n, *[1] * (got.dim() - 2))), i
