"""The forms that the kernels of a layer take, asked of the library on the host, so that a test that means to reach one
asserts it."""
import ctypes

import torch  # noqa: F401  (first, so that the library shares its HIP runtime)

from paper_2406_08756_amd import binding as B

_lib = ctypes.CDLL(B.LIB_PATH)
_lib.lynx_form_attention.restype = ctypes.c_uint
_lib.lynx_form_attention.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_longlong, ctypes.c_int, ctypes.c_int]
SCORES, GRADIENT, JOINT, FROM_C = 1, 2, 4, 8


def attention(seq, head_dim, micro_batch, heads):
    """Bits SCORES, GRADIENT, JOINT, FROM_C: what runs as one launch."""
    return _lib.lynx_form_attention(seq, head_dim, 3 * heads * head_dim, micro_batch, heads)


def score_run(seq, slices):
    return _lib.lynx_form_score_run(seq, slices)


def quotient(x, d, most):
    """(x / d as tile indices are divided, by the inverse or not)"""
    by_inverse = ctypes.c_int()
    return _lib.lynx_form_quotient(x, d, ctypes.c_longlong(most), ctypes.byref(by_inverse)), bool(by_inverse.value)


def product(M, N, K):
    """(rows, columns of the tile, K ranges)"""
    out = (ctypes.c_int * 3)()
    _lib.lynx_form_product(M, N, K, out)
    return tuple(out)


def pair(tokens, outputs, inputs, gelu):
    """(rows, columns of the tile, ranges of the weight gradient, of the input gradient, GeLU backward in it)"""
    out = (ctypes.c_int * 5)()
    _lib.lynx_form_pair(tokens, outputs, inputs, gelu, out)
    return tuple(out)


def of_layer(shape, which):
    """`which`: a forward product, or the gradients of its layer; shape: hidden, heads, head_dim, ffn, seq, micro_batch."""
    h, a, d, f, s, b = shape
    T, p = s * b, a * d
    outputs, inputs = {"qkv": (3 * p, h), "proj": (h, p), "fc1": (f, h), "fc2": (h, f)}[which.split("_")[0]]
    if which.endswith("_grads"):
        return pair(T, outputs, inputs, which == "fc2_grads")
    return product(T, outputs, inputs)


def f32(tokens, outputs, inputs):
    """fp32, a linear layer: (side of the tile, ring stages) of the forward product, of the pair of gradients"""
    out = (ctypes.c_int * 4)()
    _lib.lynx_form_f32(tokens, outputs, inputs, out)
    return tuple(out[:2]), tuple(out[2:])
