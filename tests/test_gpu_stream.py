"""GPU parity of the sparse products with few columns: those that split K across a workgroup's wavefronts, each with an LDS
ring of its own, and the streaming kernel's (the criteria of test_gpu_parity.py)."""
import pytest

from test_gpu_parity import run_mm_case

pytestmark = pytest.mark.gpu

# K: less than a step, fewer steps than wavefronts, one more than a multiple of them, partial last steps that the first or
# another wavefront takes, rings that wrap; N around the tile widths; one row, ragged rows
CASES = [
    ("i8", "i32", 32, 1, 64),
    ("i8", "i32", 33, 16, 1056),
    ("i8", "i32", 64, 17, 1152),
    ("i8", "i32", 96, 32, 4224),
    ("i8", "i32", 1000, 3, 8224),
    ("bf16", "bf16", 1, 2, 32),
    ("bf16", "f32", 64, 15, 576),
    ("f16", "f16", 45, 31, 544),
    ("f16", "f32", 320, 16, 4160),
    ("bf16", "bf16", 129, 32, 2592),
]


@pytest.mark.parametrize("case", CASES)
def test_products_match_oracle(case):
    run_mm_case(*case, layout="canonical", b_order="k", sparse=True, seed=61)
    if case[2] % 32 == 0 and case[4] % 64 == 0:
        run_mm_case(*case, layout="tiled", b_order="k", sparse=True, seed=62)


# N <= 32 and more row blocks than compute units: 8-bit operands on the streaming kernel, fewer tiles than wavefronts, one row past
# a block; K ending in half a tile: the tiled kernels for 16-bit operands, and for 8-bit ones the streaming kernel's form for it but
# for a short K, or a long one on few tiles; in a quarter of one: B staged through registers or, with a longer K, that form; 16-bit
# operands in two rounds of workgroups and past them
MANY_ROWS = [
    ("i8", "i32", 8224, 1, 64),
    ("i8", "i32", 8225, 7, 1024),
    ("i8", "i32", 8224, 16, 96),
    ("i8", "i32", 8255, 3, 1184),
    ("i8", "i32", 8193, 31, 2080),
    ("i8", "i32", 9000, 7, 160),
    ("i8", "i32", 16385, 16, 544),
    ("i8", "i32", 49153, 1, 1056),
    ("f16", "f16", 8225, 3, 48),
    ("bf16", "bf16", 8200, 9, 1040),
    ("f16", "f32", 77, 5, 144),
    ("bf16", "f32", 9098, 17, 96),
    ("bf16", "bf16", 8250, 2, 1056),
    ("f16", "f16", 10880, 1, 128),
    ("f16", "f32", 10881, 16, 192),
]


@pytest.mark.parametrize("case", MANY_ROWS)
def test_more_row_blocks_than_compute_units(case):
    run_mm_case(*case, layout="canonical", b_order="k", sparse=True, seed=63)
    if case[2] % 32 == 0 and case[4] % 64 == 0:
        run_mm_case(*case, layout="tiled", b_order="k", sparse=True, seed=64)
