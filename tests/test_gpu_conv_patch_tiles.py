"""GPU parity of the sparse 3x3 unit-stride convolutions on every tile and patch of the patch kernel (the criteria of
test_gpu_conv.py)."""
import pytest

from test_gpu_conv import run_case

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
