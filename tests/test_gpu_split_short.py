"""Split sparse products on both sides of the line below which they are not split (40 whole 128-byte steps of K in the tiled
layout, 32 in the canonical one, more than 32 columns; fewer with few rows on more than 160 columns): int8 equal to the oracle, floats within the bound of K fp32 additions;
up to the line the call is the unsplit product bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2104_08378_amd import sp24
from test_gpu_splitk import IN_DT, operands
from util import OUT_DT, out_to_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,out,M,N,K,layout,unsplit", [
    ("bf16", "f32", 512, 128, 2560, "tiled", True),        # 40 steps
    ("bf16", "f32", 512, 128, 2624, "tiled", False),       # 41
    ("f16", "f32", 1000, 100, 2096, "canonical", True),    # 32 and a partial one
    ("f16", "f32", 1000, 100, 2112, "canonical", False),   # 33
    ("i8", "i32", 256, 65, 5120, "tiled", True),           # 40, odd N
    ("i8", "i32", 256, 500, 4096, "canonical", True),      # 32
    ("i8", "i32", 256, 500, 4224, "canonical", False),     # 33
    ("f16", "f32", 1000, 100, 2080, "canonical", True),    # 32 and half a one that the streaming kernel takes
    ("bf16", "f32", 224, 200, 1792, "tiled", True),        # fewer than 256 rows on more than 160 columns: 28
    ("bf16", "f32", 224, 200, 1856, "tiled", False),       # 29
    ("f16", "f32", 100, 300, 1408, "canonical", True),     # 22
    ("f16", "f32", 100, 300, 1472, "canonical", False),    # 23
    ("i8", "i32", 256, 161, 4736, "tiled", True),          # fewer than 512: 37
    ("i8", "i32", 256, 161, 4864, "tiled", False),         # 38
])
def test_line_below_which_products_are_not_split(dtype, out, M, N, K, layout, unsplit):
    need = sp24.sp24_splitk_workspace_bytes(M, N, K, IN_DT[dtype])
    assert need > 0                                        # what callers are told does not depend on the layout
    Pn, Bmath, Bd, V, meta = operands(dtype, M, N, K, layout, "k", seed=41)
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
    D = sp24.sp24_spmm_splitk(V, meta, Bd, OUT_DT[out], layout=layout, workspace=ws)
    U = sp24.sp24_spmm(V, meta, Bd, OUT_DT[out], layout=layout)
    torch.cuda.synchronize()
    assert bool((ws == 0xFF).all()) == unsplit
    if unsplit:
        assert torch.equal(D, U)
    ref = oracle.gemm(Pn, Bmath, dtype)
    if dtype == "i8":
        assert np.array_equal(D.cpu().numpy(), ref)
    else:
        scale = np.abs(oracle.to_double(Pn, dtype)) @ np.abs(oracle.to_double(Bmath, dtype))
        assert (np.abs(out_to_f64(D) - ref) <= K * 2.0 ** -24 * scale + 1e-30).all()
