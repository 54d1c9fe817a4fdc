"""Results whose rows are not whole, aligned 16-byte chunks: the tiled kernels' stores start at any address and the last
chunk of a row is cut to its columns (2057 columns here, and test_gpu_tile_shapes.py), the kernels for few tiles store by
element.  Bit-exact against the same product into an aligned buffer, and nothing outside
the result is written."""
import pytest
import torch

from paper_2104_08378_amd import sp24
from util import OUT_DT

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,out", [("i8", "i8"), ("i8", "i32"), ("i8", "bf16"), ("f16", "f16"), ("bf16", "f32")])
@pytest.mark.parametrize("M,N", [(96, 33), (64, 47), (160, 129), (2176, 2057)])
def test_every_column_and_nothing_else(dtype, out, M, N):
    K = 128
    g = torch.Generator(device="cuda").manual_seed(M + N)
    dt = torch.int8 if dtype == "i8" else OUT_DT[dtype]
    rand = (lambda *s: torch.randint(-127, 128, s, generator=g, device="cuda", dtype=torch.int8)) if dtype == "i8" else \
           (lambda *s: torch.randn(s, generator=g, device="cuda").to(dt))
    V, meta = sp24.sp24_compress(rand(M, K), layout="tiled")
    wide = (N + 15) // 16 * 16
    B = rand(wide, K)
    scale = torch.rand(M, generator=g, device="cuda") * 1e-3
    odt = OUT_DT[out] if out != "i8" else torch.int8

    def product(b, o):
        if dtype == "i8" and out != "i32":
            return sp24.sp24_spmm_i8_scaled(V, meta, b, odt, scale, 1.0, layout="tiled", out=o)
        return sp24.sp24_spmm(V, meta, b, odt, layout="tiled", out=o)

    want = product(B, torch.empty(M, wide, dtype=odt, device="cuda"))[:, :N]     # whole chunks
    # a window with an odd pitch, at an odd place of a buffer of marks: every alignment of a row occurs
    pitch, off = N + 3, 5
    buf = torch.full((M * pitch + 64,), 77, dtype=odt, device="cuda")
    view = buf[off:off + M * pitch].view(M, pitch)[:, :N]
    product(B[:N], view)
    torch.cuda.synchronize()
    assert torch.equal(view, want)
    view.fill_(77)
    assert bool((buf == 77).all())
