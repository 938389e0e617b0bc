"""The work this library is asked to do, as cases that can be prepared, run and compared.

A case is one tensor-parallel shard of a GPT block (or a slice of several), a retain policy and a
direction.  One pass of a "step" case is what a training program does per micro-batch: forward under the
policy, regeneration of what backward will miss, backward.  One pass of a "forward" case is what an
evaluation program does: forward, then the layer is reset.  Everything goes through the C ABI's binding.

Sizes span the tiny fp32 block up to the six-layer slice of the 23B-shaped shard (lynx_synth.CONFIGS),
whole tiles and ragged shapes, sequences from 64 to 2048 tokens, every head dimension that is a multiple
of 8 from 40 to 128, both storage types, all preset policies, seeded policies and the attention option.
"""
from __future__ import annotations

import math
import weakref

import torch

import lynx_synth as synth
from paper_2406_08756_amd import binding as B

POLICIES = {"store_all": B.LYNX_RETAIN_STORE_ALL, "full": B.LYNX_RETAIN_FULL_RECOMPUTE,
            "attention_only": B.LYNX_RETAIN_ATTENTION_ONLY, "elementwise_only": B.LYNX_RETAIN_ELEMENTWISE_ONLY}

# The operators each operator reads, those whose outputs backward reads (operator 3..5 do not exist where
# the attention option applies), as the header lists them.
_PARENTS = {1: (0,), 2: (1,), 3: (2,), 4: (3,), 5: (4,), 6: (5, 2), 7: (6,), 8: (0, 7), 9: (8,), 10: (9,), 11: (10,),
            12: (11,), 13: (8, 12)}
_BACKWARD_READS = (1, 2, 4, 5, 6, 8, 9, 10, 11)


def _named(name, workload, **kw):
    c = synth.CONFIGS[workload]
    case = {"name": name, "dtype": "f32" if c.dtype == synth.F32 else "bf16", "h": c.hidden, "a": c.local_heads,
            "d": c.head_dim, "f": c.local_ffn, "s": c.seq, "b": c.micro_batch, "tp": c.tp_size, "fused": False,
            "layers": 1, "mode": "step"}
    case.update(kw)
    return case


def listed():
    return [
        # the tiny fp32 block of the parity runs, under full recomputation: nothing but launches and latency
        _named("block_f32_full", "C1", mask=POLICIES["full"]),
        # a small bf16 layer, a few tiles of every kernel: a debugging or fine-tuning size, nothing dropped
        {"name": "small_bf16_store_all", "dtype": "bf16", "h": 512, "a": 4, "d": 128, "f": 1024, "s": 384, "b": 2, "tp": 1,
         "mask": POLICIES["store_all"], "fused": False, "layers": 1, "mode": "step"},
        # evaluation of one short prompt on the 13B-shaped shard: few tokens against all of the weights
        _named("prompt_forward", "C4", s=128, b=1, mask=POLICIES["full"], mode="forward"),
        # a mid-sized block in fp32, as used to judge what bf16 costs in accuracy
        {"name": "mid_f32_store_all", "dtype": "f32", "h": 1024, "a": 16, "d": 64, "f": 4096, "s": 512, "b": 2, "tp": 1,
         "mask": POLICIES["store_all"], "fused": False, "layers": 1, "mode": "step"},
        # no dimension is a multiple of a tile: every size only the multiple of 8 that the header asks for
        {"name": "odd_bf16_full", "dtype": "bf16", "h": 3016, "a": 7, "d": 104, "f": 1544, "s": 328, "b": 3, "tp": 4,
         "mask": POLICIES["full"], "fused": False, "layers": 1, "mode": "step"},
        # a sequence cut at a round decimal number, hidden a multiple of 64 only, head dimension 64
        {"name": "seq1000_selective", "dtype": "bf16", "h": 1600, "a": 25, "d": 64, "f": 6400, "s": 1000, "b": 4, "tp": 1,
         "mask": POLICIES["attention_only"], "fused": False, "layers": 1, "mode": "step"},
        # whole tiles, head dimension 64, sequence 1024: an ordinary single-GPU layer with nothing dropped
        {"name": "d64_store_all", "dtype": "bf16", "h": 1024, "a": 16, "d": 64, "f": 4096, "s": 1024, "b": 8, "tp": 1,
         "mask": POLICIES["store_all"], "fused": False, "layers": 1, "mode": "step"},
        # the 1.3B-shaped layer on one GPU under Selective Recomputation
        _named("gpt_1b3_selective", "C2", mask=POLICIES["attention_only"]),
        # the 7B-shaped shard, elementwise operators regenerated
        _named("gpt_7b_elementwise", "C3", mask=POLICIES["elementwise_only"]),
        # the 13B-shaped shard under Full Recomputation: the headline workload
        _named("gpt_13b_full", "C4", mask=POLICIES["full"]),
        # the same with the attention option, which trades time for three seq x seq tensors
        _named("gpt_13b_full_lean", "C4", mask=POLICIES["full"], fused=True),
        # six layers of the 23B-shaped shard, each under its own seeded policy: one pipeline stage
        _named("gpt_23b_slice", "C5", mask=-1, layers=synth.C5_LAYERS),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _multiple(rng, value, lo):
    """`value` rounded to a multiple of 8 to 256: whole tiles more often than not."""
    g = rng.choice((8, 8, 64, 128, 128, 256))
    return max(lo, int(round(value / g)) * g) if value >= g else max(lo, int(round(value / 8)) * 8)


def draw(rng):
    largest = max(work(c)["flops"] for c in listed())
    while True:
        f32 = rng.random() < 0.12
        h = _multiple(rng, _log_uniform(rng, 128, 1280) if f32 else _log_uniform(rng, 256, 6144), 64)
        d = rng.choice((40, 64, 64, 80, 96, 104, 128, 128, 128, 128))
        tp = rng.choice((1, 1, 2, 4, 8))
        a = max(1, round(h / d / tp))
        f = _multiple(rng, 4 * h / tp, 64)
        s = _multiple(rng, _log_uniform(rng, 64, 512) if f32 else _log_uniform(rng, 64, 2048), 64)
        b = max(1, round(_log_uniform(rng, 1, 8)))
        policy = rng.choice(("store_all", "full", "full", "attention_only", "elementwise_only", "seeded", "seeded"))
        mask = (rng.getrandbits(14) | 0x2001) if policy == "seeded" else POLICIES[policy]
        case = {"dtype": "f32" if f32 else "bf16", "h": h, "a": a, "d": d, "f": f, "s": s, "b": b, "tp": tp, "mask": mask,
                "fused": rng.random() < 0.2, "layers": 1, "mode": "forward" if rng.random() < 0.2 else "step"}
        if work(case)["flops"] <= largest:
            return case


def _masks(case):
    return synth.c5_retain_masks(0, case["layers"]) if case["mask"] < 0 else [case["mask"]] * case["layers"]


def _config(case, layer=0):
    return synth.LayerConfig(synth.F32 if case["dtype"] == "f32" else synth.BF16, case["h"], case["a"], case["d"],
                             case["f"], case["s"], case["b"], tp_size=case["tp"], layer_id=layer,
                             flags=B.LYNX_FLAG_FUSED_ATTENTION if case["fused"] else 0)


class _Layer:
    """One layer as a training program holds it: parameters, gradients, workspace and handle."""

    def __init__(self, cfg, mask, gen, tdtype, grads):
        self.mask = mask
        self.grads = grads
        self.params = {}
        for name, shape in synth.param_shapes(cfg).items():
            if name in ("g1", "g2"):
                v = 1.0 + 0.1 * torch.randn(shape, generator=gen, device="cuda")
            elif name in ("be1", "be2"):
                v = 0.1 * torch.randn(shape, generator=gen, device="cuda")
            else:
                v = 0.02 * torch.randn(shape, generator=gen, device="cuda")
            self.params[name] = v.to(tdtype)
        self.out = torch.empty(cfg.tokens, cfg.hidden, dtype=tdtype, device="cuda")
        self.d_x = torch.empty_like(self.out)
        nbytes = B.lynx_workspace_bytes(cfg, mask)
        self.workspace = torch.empty(nbytes + 256, dtype=torch.uint8, device="cuda")
        self.handle = B.lynx_layer_create(cfg, (self.workspace.data_ptr() + 255) // 256 * 256, nbytes)
        weakref.finalize(self, B.lynx_layer_destroy, self.handle)
        B.lynx_layer_set_params(self.handle, self.params)


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    tdtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    cfg = _config(case)
    x = torch.randn(cfg.tokens, cfg.hidden, generator=gen, device="cuda").to(tdtype)
    d_out = torch.randn(cfg.tokens, cfg.hidden, generator=gen, device="cuda").to(tdtype)
    # a stage's gradients of one parameter lie in one block, as an optimizer that updates them together wants
    grads = {k: torch.empty(case["layers"], *shape, dtype=tdtype, device="cuda")
             for k, shape in synth.param_shapes(cfg).items()}
    layers = [_Layer(_config(case, i), m, gen, tdtype, {k: v[i] for k, v in grads.items()})
              for i, m in enumerate(_masks(case))]
    return {"x": x, "d_out": d_out, "layers": layers, "grads": grads, "mode": case["mode"], "step": seed & 0xFFFF}


def run(state):
    x, layers = state["x"], state["layers"]
    for layer in layers:
        B.lynx_layer_forward(layer.handle, x, layer.out, layer.mask, state["step"])
        x = layer.out
    if state["mode"] == "forward":
        for layer in layers:
            B.lynx_layer_reset(layer.handle)
        return {"out": x}
    g = state["d_out"]
    for layer in reversed(layers):
        B.lynx_recompute(layer.handle, B.LYNX_SEG_ALL_MISSING)
        B.lynx_layer_backward(layer.handle, g, layer.d_x, layer.grads)
        g = layer.d_x
    return {"out": x, "d_x": g, "grads": state["grads"]}


def _is_fused(case, mask):
    return (case["fused"] and not mask & 0x38 and case["dtype"] == "bf16" and case["d"] == 128 and case["s"] % 128 == 0)


def work(case):
    e = 4 if case["dtype"] == "f32" else 2
    h, p, f, s = case["h"], case["a"] * case["d"], case["f"], case["s"]
    T = case["b"] * s
    attention = 2.0 * case["b"] * case["a"] * (s * (s + 1) // 2) * case["d"]   # one product, j <= i only
    flops = {2: 2.0 * T * 3 * p * h, 3: attention, 6: attention, 7: 2.0 * T * h * p, 10: 2.0 * T * f * h,
             12: 2.0 * T * h * f}
    parameters = 3 * p * (h + 1) + h * (p + 1) + f * (h + 1) + h * (f + 1) + 4 * h
    total_flops, total_bytes = 0.0, 2.0 * T * h * e
    for mask in _masks(case):
        total_flops += sum(flops.values())
        total_bytes += parameters * e
        if case["mode"] == "forward":
            continue
        total_flops += 2 * sum(flops.values())
        total_bytes += parameters * e
        if _is_fused(case, mask):
            # scores come back wherever P is needed: with the context (regenerated or not) and in backward
            missing = {i for i in (1, 2, 6, 8, 9, 10, 11) if not (mask >> i) & 1}
            stack, parents = list(missing), {**_PARENTS, 6: (2,)}
            total_flops += flops[3] * (1 + (6 in missing))
        else:
            missing = {i for i in _BACKWARD_READS if not (mask >> i) & 1}
            stack, parents = list(missing), _PARENTS
        while stack:
            for j in parents[stack.pop()]:
                if j and not (mask >> j) & 1 and j not in missing:
                    missing.add(j)
                    stack.append(j)
        total_flops += sum(flops.get(i, 0.0) for i in missing)
    if case["mode"] == "step":
        total_bytes += 2.0 * T * h * e
    return {"bytes": total_bytes, "flops": total_flops}


def tolerance(case):
    # Measured against the same layer in 64 bits with the same dropout masks, worst output (dX, OUT and the
    # twelve gradients) of the cases above and of drawn ones: bf16 2-norm 4.2e-3 to 1.1e-2 (every named
    # activation and gradient is rounded to 8 bits, up to twelve roundings in a row), largest element 0.09 of
    # the root mean square; fp32 6e-7 to 1.4e-6 and 1.3e-5.
    if case["dtype"] == "f32":
        return {"rel": 6e-6, "max": 6e-5}
    return {"rel": 2e-2, "max": 0.36}
