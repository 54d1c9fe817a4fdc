"""GPU parity of the tiled products on tiles of 192 and 256 rows by 128 columns (the criteria of test_gpu_parity.py and
test_gpu_conv.py): more than 256 tiles of 128 x 128 and at most 256 of these; and, at most 128 tiles of 128 x 128, on tiles of
128 x 64 and 64 x 128 with four wavefronts, and the dense ones and the convolutions on 128 x 128 with eight."""
import pytest
import torch

from paper_2104_08378_amd import sp24
from test_gpu_conv import run_case as run_conv_case
from test_gpu_f8 import test_f8_products_against_the_oracle as run_f8
from test_gpu_parity import run_mm_case
from test_gpu_scaled import test_float_outputs_match_the_double_epilogue as run_scaled_float
from test_gpu_scaled import test_int8_output_is_bit_exact as run_scaled_int8

pytestmark = pytest.mark.gpu

# one whole tile and one that ends inside each of its row blocks and columns; whole and partial last steps; for the sparse
# products the fewest steps that take these tiles (12; 16 and 24 for results of 32 bits)
SPARSE = [
    ("bf16", "bf16", 300, 11007, 800, "canonical"),     # 192 rows
    ("f16", "f32", 320, 11001, 1024, "tiled"),
    ("i8", "i32", 384, 10990, 2112, "tiled"),
    ("f16", "f16", 200, 16500, 800, "canonical"),       # 256 rows
    ("bf16", "bf16", 256, 16400, 832, "tiled"),
    ("f16", "f32", 160, 16401, 1536, "tiled"),
]
# a single step, fewer than the ring holds, a partial one alone and behind others
DENSE = [
    ("bf16", "f32", 300, 11007, 96),
    ("i8", "i32", 384, 10990, 128),
    ("i8", "i32", 300, 11000, 480),
    ("f16", "f16", 200, 16500, 32),
    ("bf16", "bf16", 256, 16400, 352),
    ("i8", "i32", 160, 16401, 640),
]
# strided ones: four steps and nine, ragged rows and pixels
CONVS = [
    ("bf16", "bf16", 200, 22, 55, 56, 256, 1, 1, (0, 0), (2, 2), "canonical"),
    ("i8", "i32", 256, 43, 40, 40, 128, 3, 3, (1, 1), (2, 2), "tiled"),
]


@pytest.mark.parametrize("case", SPARSE)
def test_sparse_products(case):
    dtype, out, M, N, K, layout = case
    run_mm_case(dtype, out, M, N, K, layout=layout, b_order="k", sparse=True, seed=81)
    run_mm_case(dtype, out, M, N // 16 * 16, K, layout=layout, b_order="n", sparse=True, seed=82)


@pytest.mark.parametrize("case", DENSE)
def test_dense_products(case):
    dtype, out, M, N, K = case
    run_mm_case(dtype, out, M, N, K, layout=None, b_order="k", sparse=False, seed=83)
    run_mm_case(dtype, out, M, N // 16 * 16, K, layout=None, b_order="n", sparse=False, seed=84)


@pytest.mark.parametrize("case", CONVS)
@pytest.mark.parametrize("sparse", [True, False])
def test_strided_convolutions(case, sparse):
    run_conv_case(*case, sparse=sparse, seed=85)


# 128 x 64 (a canonical or 8-bit N-major operand: 64 x 128): a step, as many as the ring holds, one and several more, a partial
# one alone and behind others; one row, a row and a column past a tile
FEW = [
    ("bf16", "bf16", 1, 601, 64, "canonical"),
    ("f16", "f32", 129, 577, 512, "canonical"),
    ("i8", "i32", 160, 515, 1024, "tiled"),
    ("bf16", "f32", 288, 530, 576, "tiled"),
    ("i8", "i32", 129, 700, 1184, "canonical"),
    ("f16", "f16", 96, 1000, 1152, "tiled"),
    ("i8", "i32", 416, 641, 32, "canonical"),
    ("bf16", "bf16", 65, 650, 1568, "canonical"),
    ("i8", "i32", 64, 515, 1216, "tiled"),
]


@pytest.mark.parametrize("case", FEW)
def test_few_tiles(case):
    dtype, out, M, N, K, layout = case
    for n, b_order in ((N, "k"), (N // 16 * 16, "n")):
        run_mm_case(dtype, out, M, n, K, layout=layout, b_order=b_order, sparse=True, seed=86)
        run_mm_case(dtype, out, M, n, K, layout=None, b_order=b_order, sparse=False, seed=87)
    run_mm_case(dtype, out, M, 80, K, layout=layout, b_order="n", sparse=True, seed=88)


# 129 - 176 tiles of 128 x 128 (8-bit types: to 160, N-major ones on four wavefronts; convolutions to 210): no whole step, one, as
# many as the ring holds, more, partial ones behind them
EIGHT_DENSE = [
    ("bf16", "f32", 1450, 1411, 32),
    ("f16", "f16", 1409, 1410, 96),
    ("i8", "i32", 1440, 1500, 512),
    ("bf16", "bf16", 2000, 1281, 352),
]
EIGHT_CONVS = [
    ("f16", "f32", 130, 13, 20, 32, 64, 5, 1, (2, 0), (1, 1), "canonical"),
    ("i8", "i32", 96, 43, 40, 40, 128, 3, 3, (1, 1), (2, 2), "tiled"),
]


@pytest.mark.parametrize("case", EIGHT_DENSE)
def test_dense_products_on_eight_wavefronts(case):
    dtype, out, M, N, K = case
    run_mm_case(dtype, out, M, N, K, layout=None, b_order="k", sparse=False, seed=89)
    run_mm_case(dtype, out, M, N // 16 * 16, K, layout=None, b_order="n", sparse=False, seed=90)


@pytest.mark.parametrize("case", EIGHT_CONVS)
@pytest.mark.parametrize("sparse", [True, False])
def test_convolutions_on_eight_wavefronts(case, sparse):
    run_conv_case(*case, sparse=sparse, seed=91)


# few tiles of 128 x 64: fewer steps than the ring holds and more, ragged rows and pixels, padding
FEW_CONVS = [
    ("f16", "f32", 130, 3, 20, 13, 64, 3, 3, (1, 1), (2, 1), "canonical"),
    ("i8", "i32", 96, 5, 11, 12, 128, 5, 1, (2, 0), (1, 1), "tiled"),
    ("bf16", "bf16", 257, 2, 9, 8, 192, 1, 1, (0, 0), (2, 2), "canonical"),
]


@pytest.mark.parametrize("case", FEW_CONVS)
@pytest.mark.parametrize("sparse", [True, False])
def test_convolutions_on_few_tiles(case, sparse):
    run_conv_case(*case, sparse=sparse, seed=92)


# sparse 8-bit convolutions on more than 192 tiles of 256 rows: eight steps, and seven on 128 x 128
MOST_UNITS_CONVS = [
    ("i8", "i32", 160, 10, 50, 51, 128, 4, 2, (2, 0), (1, 1), "tiled"),
    ("i8", "i32", 150, 10, 50, 51, 128, 7, 1, (3, 0), (1, 1), "canonical"),
]


@pytest.mark.parametrize("case", MOST_UNITS_CONVS)
def test_convolutions_on_most_units(case):
    run_conv_case(*case, sparse=True, seed=93)


# 16-bit canonical operands, N-major: 48 steps on two wavefronts, 47 on four, a partial one behind them
CANONICAL_N_MAJOR = [
    ("bf16", "f32", 130, 640, 3104),
    ("f16", "f16", 200, 592, 3040),
]


@pytest.mark.parametrize("case", CANONICAL_N_MAJOR)
def test_canonical_n_major_products(case):
    run_mm_case(*case, layout="canonical", b_order="n", sparse=True, seed=94)


# int8 with 32-bit results on 256 rows: 24 steps and a partial one, the fewest that a sparse product takes them with
def test_int8_products_on_256_rows():
    run_mm_case("i8", "i32", 256, 16400, 3104, layout="canonical", b_order="k", sparse=True, seed=97)
    run_mm_case("i8", "i32", 224, 16400, 3136, layout="tiled", b_order="n", sparse=True, seed=98)


# quantised results on 192 and 256 rows: the fewest steps of the sparse product (12; 16 and 24 for 32-bit results) and partial ones,
# whole and ragged tiles, even and odd columns
@pytest.mark.parametrize("case", [(384, 10990, 1632, "canonical"), (320, 11007, 1664, "tiled"), (256, 16400, 1632, "canonical"), (193, 16401, 1600, "canonical")])
@pytest.mark.parametrize("sparse", [True, False])
def test_quantised_products(case, sparse):
    run_scaled_int8(case, sparse)


@pytest.mark.parametrize("case,out", [((300, 11007, 1632, "canonical"), "bf16"), ((384, 10990, 2112, "tiled"), "f32"),
                                      ((256, 16401, 1600, "tiled"), "bf16"), ((200, 16400, 3104, "canonical"), "f32")])
def test_quantised_products_with_float_results(case, out):
    run_scaled_float(case, out)


# (half precision is subnormal near zero, where its rounding is absolute, up to 2^-25, and the bound above relative: against the
# results of 32 bits, whose epilogue is the same, rounded once)
@pytest.mark.parametrize("M,N", [(384, 10990), (256, 16401)])
def test_quantised_products_with_half_precision_results(M, N):
    g = torch.Generator(device="cuda").manual_seed(99)
    rand = lambda *s: torch.randint(-127, 128, s, generator=g, device="cuda", dtype=torch.int8)
    V, meta = sp24.sp24_compress(rand(M, 1600), layout="tiled")
    B, scale = rand(N, 1600), torch.rand(M, generator=g, device="cuda") * 1e-3
    half, single = [sp24.sp24_spmm_i8_scaled(V, meta, B, t, scale, 0.02, scale, True, layout="tiled") for t in (torch.float16, torch.float32)]
    torch.cuda.synchronize()
    assert torch.equal(half, single.to(torch.float16))


@pytest.mark.parametrize("case,out", [((384, 10990, 1632, "canonical", "k"), torch.bfloat16), ((288, 11008, 2112, "tiled", "n"), torch.float32),
                                      ((256, 16401, 1600, "tiled", "k"), torch.float16), ((200, 16400, 3104, "canonical", "n"), torch.float32)])
def test_8_bit_float_products(case, out):
    run_f8(case, out)
