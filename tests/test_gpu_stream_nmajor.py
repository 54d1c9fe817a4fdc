"""Sparse products with few tiles and an N-major second operand of whole 16-byte chunks (the streaming kernel up to 256 workgroups
of 32 rows, canonical 16-bit operands of many steps and a B of whole lines 512, the tiled ones past it): against the oracle at the edges of column tiles, steps of K and rows."""
import numpy as np
import pytest
import torch

import oracle
from paper_2104_08378_amd import sp24, synth
from test_gpu_parity import NAME_OF
from util import OUT_DT, out_to_f64, to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,out,M,N,K,layout,pad", [
    ("bf16", "f32", 96, 8, 128, "tiled", 0),             # two steps, one chunk of columns
    ("f16", "f32", 64, 16, 1088, "tiled", 0),            # 17 steps on eight wavefronts
    ("bf16", "bf16", 33, 24, 528, "canonical", 8),       # one row past a tile; 8 steps and a quarter; a pitched B
    ("f16", "f32", 160, 32, 2112, "canonical", 0),
    ("bf16", "f32", 224, 40, 1600, "tiled", 0),          # ragged 64-column tile
    ("f16", "f16", 100, 200, 1552, "canonical", 16),     # ragged rows and columns, a quarter of a step
    ("bf16", "f32", 2048, 256, 192, "tiled", 0),         # 256 workgroups
    ("bf16", "f32", 2080, 256, 192, "tiled", 0),         # 260: not here
    ("bf16", "f32", 64, 1032, 256, "tiled", 0),          # many columns
    ("bf16", "f32", 2080, 256, 2048, "canonical", 0),    # 260 workgroups in two rounds
    ("bf16", "f32", 2080, 256, 1984, "canonical", 0),    # 31 steps: not here
    ("f16", "f16", 2080, 240, 2048, "canonical", 16),    # 260 workgroups, a ragged column tile in whole lines
    ("bf16", "f32", 2080, 256, 2048, "canonical", 8),    # rows that begin inside a line: not here
    ("bf16", "f32", 128, 4160, 2048, "canonical", 0),    # 260 workgroups on few rows
    ("bf16", "f32", 96, 5568, 2048, "canonical", 0),     # 261 on fewer: not here
    ("i8", "i32", 32, 16, 256, "tiled", 0),
    ("i8", "i32", 96, 48, 1120, "canonical", 16),        # 8 steps and three quarters
    ("i8", "i32", 128, 32, 2112, "tiled", 0),            # 16 steps and a half
    ("i8", "i32", 1000, 80, 1024, "canonical", 0),
    ("f8", "f32", 64, 144, 2048, "tiled", 0),
])
def test_few_tiles_nmajor(dtype, out, M, N, K, layout, pad):
    if dtype == "f8": A, Bt = synth.normal_bits((M, K), 0.5, "f8", 51, 9, 0), synth.normal_bits((N, K), 1.0, "f8", 51, 9, 1)
    else: A, Bt = synth.make(NAME_OF[dtype], M=M, N=N, K=K, seed=51)
    Bmath = np.ascontiguousarray(Bt.T)
    wide = np.zeros((K, N + pad), dtype=Bmath.dtype)
    wide[:, :N] = Bmath
    Bd = to_gpu(wide, dtype)[:, :N]
    Pn = oracle.prune(A, dtype)
    V, meta = sp24.sp24_compress(to_gpu(A, dtype), layout=layout)
    D = sp24.sp24_spmm(V, meta, Bd, OUT_DT[out], b_order="n", layout=layout)
    torch.cuda.synchronize()
    ref = oracle.gemm(Pn, Bmath, dtype)
    if dtype == "i8":
        assert np.array_equal(D.cpu().numpy(), ref)
        return
    # K fp32 additions, one rounding to the output type; 8-bit floats: what the instruction drops below 2^-15 of a block's largest product
    scale = np.abs(oracle.to_double(Pn, dtype)) @ np.abs(oracle.to_double(Bmath, dtype))
    ulp = {"f32": 2.0 ** -24, "f16": 2.0 ** -11, "bf16": 2.0 ** -8}[out]
    bound = K * 2.0 ** -24 * scale + ulp * np.abs(ref) + 1e-30 + (2.0 ** -15 * scale if dtype == "f8" else 0.0)
    assert (np.abs(out_to_f64(D) - ref) <= bound).all()
