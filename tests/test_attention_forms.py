"""Launches of attention with more threads than HIP takes (2^32 in a dimension): so many slices that a launch for two
products, or with a workgroup per 32 rows, has too many, go by the kernels that have fewer."""
import pytest
import torch  # noqa: F401  (first, so that the library shares its HIP runtime)

pytest.importorskip("paper_2406_08756_amd.binding")

from forms import GRADIENT, JOINT, SCORES
from forms import attention as form


def test_ordinary_sizes():
    assert form(8, 8, 1, 1) == SCORES | GRADIENT | JOINT
    assert form(1024, 64, 8, 16) == SCORES | GRADIENT | JOINT
    assert form(2048, 128, 8, 5) == SCORES | JOINT
    assert form(2056, 128, 1, 5) == JOINT
    assert form(512, 136, 1, 5) == JOINT


# a workgroup of 256 threads per slice and product: 2^24 of them are one too many
@pytest.mark.parametrize("heads,joint", [(3, True), (4, False)])
def test_two_products_in_one_launch(heads, joint):
    assert bool(form(8, 8, 1 << 21, heads) & JOINT) == joint


# two row blocks of 32 and up to 512 threads each: 2^22 slices are one too many
@pytest.mark.parametrize("micro_batch,fused", [((1 << 18) - 1, True), (1 << 18, False)])
def test_scores_of_32_rows_per_workgroup(micro_batch, fused):
    assert bool(form(64, 8, micro_batch, 16) & SCORES) == fused
    assert bool(form(64, 8, micro_batch, 16) & GRADIENT) == fused
