"""GPU parity of the sparse 3x3 unit-stride convolutions on every tile and patch of the patch kernel (the criteria of
test_gpu_conv.py)."""
import pytest

from test_gpu_conv import run_case
from test_gpu_scaled import test_quantised_convolution_int8_output_is_bit_exact as run_scaled

pytestmark = pytest.mark.gpu

# dtype, out, M, n_img, H, W, C, pad: one chunk of channels (64 of 16 bits, 128 of 8) and more, narrow and wide images, ragged
# filters and pixels
CASES = [
    ("f16", "f32", 32, 1, 3, 3, 64, (1, 1)),          # 64 x 64 tiles, 128-pixel patch, a tile larger than the output
    ("i8", "i32", 96, 7, 9, 11, 128, (1, 1)),
    ("bf16", "bf16", 160, 3, 13, 14, 192, (1, 1)),    # three chunks
    ("i8", "i32", 64, 2, 17, 20, 256, (0, 0)),
    ("f16", "f16", 96, 2, 23, 47, 64, (1, 1)),        # 192-pixel patch
    ("i8", "i32", 128, 1, 40, 61, 256, (1, 0)),
    ("bf16", "f32", 64, 1, 21, 56, 320, (1, 1)),
    ("f16", "f16", 64, 99, 13, 13, 64, (1, 1)),       # 64 x 128, 192-pixel patch: up to 64 filters, one chunk
    ("bf16", "f32", 32, 33, 23, 23, 128, (1, 1)),     # two
    ("i8", "i32", 128, 51, 13, 13, 256, (1, 1)),      # at most 256 tiles
    ("f16", "f16", 128, 6, 37, 38, 64, (1, 1)),       # 256-pixel patch
    ("i8", "i32", 160, 3, 44, 45, 256, (1, 1)),
    ("f16", "f32", 96, 24, 27, 26, 64, (1, 1)),       # 128 x 128, one chunk: 192- and 256-pixel patches
    ("i8", "i32", 96, 11, 39, 40, 128, (1, 1)),
    ("f16", "f16", 96, 22, 55, 55, 64, (1, 1)),       # 64 x 128, one chunk and more than 512 tiles of 128 x 128
]


@pytest.mark.parametrize("case", CASES)
def test_patch_tiles(case):
    dtype, out, M, n_img, H, W, C, pad = case
    run_case(dtype, out, M, n_img, H, W, C, 3, 3, pad, (1, 1), "tiled", sparse=True, seed=95)


# 128 x 128 tiles with several chunks of channels: more than 256 tiles of 64 x 128
SEVERAL_CHUNKS = [
    ("bf16", "bf16", 128, 22, 28, 28, 128, (1, 1)),   # 192-pixel patch: two chunks
    ("f16", "f32", 96, 28, 25, 26, 192, (1, 1)),      # three, ragged filters and pixels
    ("i8", "i32", 160, 14, 28, 29, 256, (1, 1)),
    ("f16", "f16", 128, 6, 56, 56, 128, (1, 1)),      # 256-pixel patch
    ("bf16", "f32", 96, 6, 55, 57, 192, (1, 1)),
    ("i8", "i32", 128, 6, 55, 57, 384, (1, 1)),
]


@pytest.mark.parametrize("case", SEVERAL_CHUNKS)
def test_large_tiles_with_several_chunks(case):
    dtype, out, M, n_img, H, W, C, pad = case
    run_case(dtype, out, M, n_img, H, W, C, 3, 3, pad, (1, 1), "tiled", sparse=True, seed=96)


# quantised results: 64 x 128 tiles, and 128 x 128 with several chunks on both patches
@pytest.mark.parametrize("M,n_img,H,W,C", [(64, 30, 24, 24, 128), (128, 22, 28, 28, 256), (96, 6, 56, 56, 256)])
def test_quantised_results(M, n_img, H, W, C):
    run_scaled((M, n_img, H, W, C, 3, 3, (1, 1), (1, 1), "tiled"))
