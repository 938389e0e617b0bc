"""Tile indices divided by the host's inverses: exact up to the largest index that the inverse is made for, and beyond
what an inverse can do by an ordinary division."""
import random

import pytest

import forms


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
