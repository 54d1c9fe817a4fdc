"""GPU parity of the products with an N-major B whose rows are not 16-byte aligned (an odd number of columns, a view
with an odd pitch), where K is split across the wavefronts of a workgroup: the criterion of test_gpu_parity.py."""
import numpy as np
import pytest
import torch

import oracle
from paper_2104_08378_amd import sp24, synth
from test_gpu_parity import run_mm_case
from util import OUT_DT, out_to_f64, to_gpu

pytestmark = pytest.mark.gpu

CASES = [
    # dtype, out, M, N, K: fewer K tiles than wavefronts, a partial last tile of K, one column (pieces of 16 bytes that
    # span many rows of B), columns just before and past a tile of 64, several tiles with ragged edges
    ("i8", "i32", 33, 1, 32),
    ("i8", "i32", 64, 63, 96),
    ("i8", "i32", 130, 65, 1056),
    ("i8", "i32", 96, 509, 2048),
    ("bf16", "bf16", 1, 3, 16),
    ("bf16", "f32", 65, 1, 80),
    ("f16", "f16", 64, 71, 464),
    ("f16", "f32", 160, 129, 1104),
    ("bf16", "bf16", 256, 333, 1024),
]


@pytest.mark.parametrize("case", CASES)
def test_products_match_oracle(case):
    run_mm_case(*case, layout="canonical", b_order="n", sparse=True, seed=31)
    run_mm_case(*case, layout="canonical", b_order="n", sparse=False, seed=32)
    if case[2] % 32 == 0 and case[4] % 64 == 0:
        run_mm_case(*case, layout="tiled", b_order="n", sparse=True, seed=33)


@pytest.mark.parametrize("dtype,out", [("i8", "i32"), ("f16", "f32")])
def test_nothing_outside_the_operand_counts(dtype, out):
    """B as an odd-pitched window in the middle of a buffer of NaN patterns (int8: large values): every read past a
    row's columns, before the first or past the last element would show."""
    M, N, K, pitch, off = 64, 37, 192, 53, 19
    A, Bt = synth.make("square_i8" if dtype == "i8" else "tiny_f16", M=M, N=N, K=K, seed=5)
    Pn, Bmath = oracle.prune(A, dtype), np.ascontiguousarray(Bt.T)
    ref = oracle.gemm(Pn, Bmath, dtype)
    fill = 127 if dtype == "i8" else float("nan")
    buf = torch.full((K * pitch + 64,), fill, dtype=torch.int8 if dtype == "i8" else torch.float16, device="cuda")
    Bv = buf[off:off + K * pitch].view(K, pitch)[:, :N]
    Bv.copy_(to_gpu(Bmath, dtype))
    V, meta = sp24.sp24_compress(to_gpu(A, dtype), layout="tiled")
    for D in (sp24.sp24_spmm(V, meta, Bv, OUT_DT[out], b_order="n", layout="tiled"),
              sp24.sp24_gemm_dense(to_gpu(Pn, dtype), Bv, OUT_DT[out], b_order="n")):
        if dtype == "i8":
            assert np.array_equal(D.cpu().numpy(), ref)
        else:
            assert np.abs(out_to_f64(D) - ref).max() <= K * 2.0 ** -24 * (np.abs(oracle.to_double(Pn, dtype)) @ np.abs(oracle.to_double(Bmath, dtype))).max()
