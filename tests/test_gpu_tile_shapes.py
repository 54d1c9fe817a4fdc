"""GPU parity of the sparse products that the tiled kernels keep beside the kernels for few columns and few tiles: more than
512 columns, or more than 256 workgroups of 32 rows (the criteria of test_gpu_parity.py, test_gpu_splitk.py, test_gpu_f8.py
and test_gpu_ragged_output.py), and of the wider forms of the kernels that split K inside a workgroup."""
import pytest
import torch

from paper_2104_08378_amd import sp24
from test_gpu_f8 import test_f8_products_against_the_oracle as run_f8
from test_gpu_parity import run_mm_case
from test_gpu_ragged_output import test_every_column_and_nothing_else as run_ragged
from test_gpu_splitk import test_split_products_match_oracle_and_the_unsplit_products as run_split

pytestmark = pytest.mark.gpu

# K ends in the middle of a step: a partial step alone, behind one and behind a ring that wraps; ragged M and N.  Tiles of
# 64 x 64 (few of them with not one whole step; 65 of 128 x 128, N <= 64) and 64 x 128 (few of them), 128 x 128 with six (144 of them) and three stages (306),
# 256 x 256 (144)
PARTIAL = [
    ("i8", "i32", 224, 60, 96),
    ("i8", "i32", 64, 64, 64),
    ("bf16", "f32", 100, 33, 32),
    ("i8", "i32", 8231, 50, 160),
    ("bf16", "bf16", 8256, 61, 352),
    ("i8", "i32", 224, 700, 960),
    ("f16", "f32", 333, 600, 608),
    ("bf16", "f32", 70, 1000, 32),
    ("i8", "i32", 1440, 1500, 192),
    ("f16", "f16", 1450, 1411, 480),
    ("bf16", "bf16", 2100, 2300, 96),
    ("i8", "i32", 2112, 2300, 448),
    ("i8", "i32", 2830, 3010, 160),
    ("f16", "f32", 2830, 3010, 96),
]


@pytest.mark.parametrize("case", PARTIAL)
def test_partial_last_step_on_every_tile(case):
    dtype, out, M, N, K = case
    run_mm_case(*case, layout="canonical", b_order="k", sparse=True, seed=71)
    run_mm_case(dtype, out, M, N // 16 * 16, K, layout="canonical", b_order="n", sparse=True, seed=72)
    if M % 32 == 0 and K % 64 == 0:
        run_mm_case(*case, layout="tiled", b_order="k", sparse=True, seed=73)


# N-major rows at odd addresses on more than 256 tiles of 32 x 64 and at most 64 of 128 x 128: two row blocks to a workgroup,
# wavefronts with one to three tiles of K, a partial last one; a last row block that does not exist
TWO_ROW_BLOCKS = [
    ("i8", "i32", 2048, 509, 1152),
    ("i8", "i32", 2017, 509, 1184),
    ("bf16", "f32", 2017, 509, 1104),
    ("f16", "f16", 2048, 511, 1088),
    ("bf16", "bf16", 4100, 67, 400),
]


@pytest.mark.parametrize("case", TWO_ROW_BLOCKS)
def test_n_major_at_any_address_on_two_row_blocks(case):
    run_mm_case(*case, layout="canonical", b_order="n", sparse=True, seed=74)
    if case[2] % 32 == 0 and case[4] % 64 == 0:
        run_mm_case(*case, layout="tiled", b_order="n", sparse=True, seed=75)


# 64 columns a tile, seven wavefronts of two stages: less than a step, a step for each wavefront, one more, rings that wrap,
# a partial step for the first and for another wavefront; columns around a tile; one row
WIDE_STREAM = [
    ("i8", "i32", 32, 66, 64),
    ("i8", "i32", 65, 64, 896),
    ("i8", "i32", 96, 65, 1056),
    ("i8", "i32", 160, 511, 2144),
    ("bf16", "bf16", 1, 127, 32),
    ("f16", "f32", 320, 129, 448),
    ("f16", "f16", 45, 200, 960),
    ("bf16", "f32", 64, 512, 1504),
    ("bf16", "bf16", 129, 100, 2592),
]


@pytest.mark.parametrize("case", WIDE_STREAM)
def test_few_tiles_of_64_columns(case):
    run_mm_case(*case, layout="canonical", b_order="k", sparse=True, seed=76)
    if case[2] % 32 == 0 and case[4] % 64 == 0:
        run_mm_case(*case, layout="tiled", b_order="k", sparse=True, seed=77)


F8 = [
    (224, 700, 352, "canonical", "k"),      # 64 x 128 tiles, a partial step
    (224, 700, 192, "tiled", "k"),
    (1440, 1500, 160, "canonical", "k"),    # 128 x 128
    (1440, 1504, 320, "tiled", "n"),
    (2830, 3010, 96, "canonical", "k"),     # 256 x 256
    (70, 133, 160, "canonical", "n"),       # N-major at odd addresses: one row block, two, and B staged through registers
    (2048, 509, 640, "tiled", "n"),
    (2100, 701, 160, "canonical", "n"),
    (45, 100, 1056, "canonical", "k"),      # few tiles of 64 columns
    (8225, 5, 96, "canonical", "k"),        # tiles of 64 x 64, a partial step
    (8225, 5, 288, "canonical", "k"),       # the streaming kernel, half a tile
]


@pytest.mark.parametrize("case", F8)
def test_8_bit_float_products(case):
    run_f8(case, torch.float32)


SPLIT = [
    # more than 512 columns: K-major slices on the 128 x 128 kernel
    ("i8", "i32", 200, 640, 6176, "canonical", "k"),
    ("bf16", "f32", 256, 1024, 3104, "canonical", "k"),
    ("f16", "f16", 130, 577, 4096, "canonical", "k"),
    ("bf16", "bf16", 256, 768, 4096, "tiled", "k"),
    ("i8", "i32", 96, 1030, 8256, "tiled", "k"),
]


@pytest.mark.parametrize("case", SPLIT)
def test_split_products_with_many_columns(case):
    run_split(case)


@pytest.mark.parametrize("out", ["i8", "f16", "bf16", "f32"])
@pytest.mark.parametrize("M,N", [(224, 701), (96, 1033), (32, 515), (1440, 1502)])
def test_quantised_results_with_odd_rows(out, M, N):
    run_ragged("i8", out, M, N)


# N-major rows at odd addresses on more than 256 tiles of 32 x 64 and at most 64 of 128 x 128, sparse: up to 16 steps in the tiled
# layout (canonical 4) with B staged through registers, from 17 (5) on wavefronts that split K over two row blocks; partial steps
FEW_STEPS = [
    ("i8", "i32", 2048, 509, 2112, "tiled"),
    ("i8", "i32", 2048, 509, 2176, "tiled"),
    ("bf16", "bf16", 1408, 333, 1024, "tiled"),
    ("f16", "f32", 8192, 65, 1088, "tiled"),
    ("i8", "i32", 2017, 509, 608, "canonical"),
    ("bf16", "f32", 1999, 511, 304, "canonical"),
    ("f16", "f16", 1153, 509, 320, "canonical"),
]


@pytest.mark.parametrize("case", FEW_STEPS)
def test_n_major_at_any_address_with_few_steps(case):
    dtype, out, M, N, K, layout = case
    run_mm_case(dtype, out, M, N, K, layout=layout, b_order="n", sparse=True, seed=78)


@pytest.mark.parametrize("K", [2048, 2240])
def test_8_bit_floats_n_major_at_any_address_with_few_steps(K):
    run_f8((1536, 509, K, "tiled", "n"), torch.float32)


@pytest.mark.parametrize("out", ["i8", "bf16"])
def test_quantised_results_n_major_at_any_address_with_few_steps(out):
    g = torch.Generator(device="cuda").manual_seed(79)
    M, N, K = 2048, 509, 1024
    dt = torch.int8 if out == "i8" else torch.bfloat16
    V, meta = sp24.sp24_compress(torch.randint(-127, 128, (M, K), generator=g, device="cuda", dtype=torch.int8), layout="tiled")
    B = torch.randint(-127, 128, (K, 512), generator=g, device="cuda", dtype=torch.int8)
    scale = torch.rand(M, generator=g, device="cuda") * 1e-3
    want = sp24.sp24_spmm_i8_scaled(V, meta, B, dt, scale, 0.1, b_order="n", layout="tiled")[:, :N]       # the tiled kernels
    got = sp24.sp24_spmm_i8_scaled(V, meta, B[:, :N].contiguous(), dt, scale, 0.1, b_order="n", layout="tiled")
    torch.cuda.synchronize()
    assert torch.equal(got, want)
