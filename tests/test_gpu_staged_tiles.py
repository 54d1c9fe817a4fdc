"""GPU parity of the products and convolutions whose second operand passes through registers, on each tile shape: 64 x 64 on up
to 256 of those, 32 x 128 and 64 x 128 past it (the criteria of test_gpu_parity.py and test_gpu_conv.py)."""
import pytest

from test_gpu_conv import run_case
from test_gpu_parity import run_mm_case

pytestmark = pytest.mark.gpu

# K a multiple of 16: a partial step alone, behind one and behind several
KMAJOR = [
    ("bf16", "f32", 65, 131, 16),
    ("f16", "f16", 130, 190, 592),
    ("bf16", "bf16", 31, 16450, 48),
    ("f16", "f32", 64, 16401, 80),
]
# odd columns; more than 64 tiles of 128 x 128
NMAJOR = [
    ("i8", "i32", 129, 4163, 96),
    ("bf16", "bf16", 32, 8197, 208),
    ("i8", "i32", 31, 16451, 160),
    ("f16", "f16", 64, 16397, 80),
]
# channels that are no whole 128-byte step: two taps to a step and fractions of one
CONVS = [
    ("f16", "f32", 70, 3, 9, 10, 96, 3, 3, (1, 1), (1, 1), "canonical"),
    ("i8", "i32", 64, 5, 11, 8, 64, 3, 1, (1, 0), (2, 1), "tiled"),
    ("i8", "i32", 32, 22, 28, 28, 32, 3, 3, (1, 1), (1, 1), "canonical"),
    ("bf16", "bf16", 64, 22, 28, 28, 32, 3, 3, (1, 1), (1, 1), "canonical"),
]


@pytest.mark.parametrize("case", KMAJOR)
def test_k_a_multiple_of_16(case):
    run_mm_case(*case, layout="canonical", b_order="k", sparse=True, seed=96)


@pytest.mark.parametrize("case", NMAJOR)
def test_odd_columns(case):
    run_mm_case(*case, layout="canonical", b_order="n", sparse=True, seed=97)


@pytest.mark.parametrize("case", CONVS)
def test_convolutions(case):
    run_case(*case, sparse=True, seed=98)
