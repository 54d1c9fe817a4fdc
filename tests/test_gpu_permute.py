"""GPU parity of the channel-permutation operations (Sec. 4.1 Step 2, Fig. 6) against the CPU oracle: the column
gather bit-exact, the retained magnitude to 1e-12 relative (its terms are exact doubles, only their order of
addition differs: the sum of n non-negative terms is off by at most n * 2^-53 relative, n < 2^14 per partial sum
and 2^11 partial sums)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2104_08378_amd import sp24, synth
from util import to_bits, to_gpu
from test_gpu_parity import NAME_OF, adversarial

pytestmark = pytest.mark.gpu

# rows x columns: one wavefront pass, ragged passes, a row longer than one LDS region (> 16 KiB), many workgroups
SHAPES = [(1, 32), (5, 96), (37, 160), (130, 1056), (3, 16416), (9000, 64)]


def dev_perm(perm):
    return torch.from_numpy(np.ascontiguousarray(perm, dtype=np.int32)).cuda()


@pytest.mark.parametrize("dtype", ["f16", "bf16", "i8"])
def test_permute_columns_bit_exact(dtype):
    for i, (M, K) in enumerate(SHAPES):
        A = adversarial(dtype, M, K, 70 + i) if i == 2 else synth.make(NAME_OF[dtype], M=M, N=16, K=K, seed=60 + i)[0]
        rng = np.random.default_rng(80 + i)
        perm = rng.permutation(K).astype(np.int32)
        Ad = to_gpu(A, dtype)
        P = sp24.sp24_permute_columns(Ad, dev_perm(perm))
        back = sp24.sp24_permute_columns(P, dev_perm(np.argsort(perm)))
        torch.cuda.synchronize()
        assert np.array_equal(to_bits(P), oracle.permute_columns(A, perm, dtype)), (dtype, M, K)
        assert np.array_equal(to_bits(back), A)
    # rows with a pitch larger than K, on both sides; an entry outside 0..K-1 reads column 0
    M, K = 33, 96
    A = synth.make(NAME_OF[dtype], M=M, N=16, K=K, seed=66)[0]
    big = torch.zeros((M, K + 32), dtype=to_gpu(A, dtype).dtype, device="cuda")
    big[:, :K] = to_gpu(A, dtype)
    out = torch.zeros((M, K + 64), dtype=big.dtype, device="cuda")
    perm = np.random.default_rng(9).permutation(K).astype(np.int32)
    sp24.sp24_permute_columns(big[:, :K], dev_perm(perm), out=out[:, :K])
    torch.cuda.synchronize()
    assert np.array_equal(to_bits(out[:, :K]), A[:, perm])
    assert not to_bits(out[:, K:]).any()
    wild = perm.copy()
    wild[5], wild[17] = -3, K
    P = sp24.sp24_permute_columns(to_gpu(A, dtype), dev_perm(wild))
    torch.cuda.synchronize()
    safe = wild.copy()
    safe[[5, 17]] = 0
    assert np.array_equal(to_bits(P), A[:, safe])


@pytest.mark.parametrize("dtype", ["f16", "bf16", "i8"])
def test_permute_rows_bit_exact(dtype):
    for i, (M, K) in enumerate(SHAPES):
        A = synth.make(NAME_OF[dtype], M=M, N=16, K=K, seed=110 + i)[0]
        perm = np.random.default_rng(120 + i).permutation(M).astype(np.int32)
        P = sp24.sp24_permute_rows(to_gpu(A, dtype), dev_perm(perm))
        torch.cuda.synchronize()
        assert np.array_equal(to_bits(P), oracle.permute_rows(A, perm, dtype)), (dtype, M, K)
    # pitched rows on both sides; an entry outside 0..M-1 reads row 0
    M, K = 37, 96
    A = synth.make(NAME_OF[dtype], M=M, N=16, K=K, seed=116)[0]
    big = torch.zeros((M, K + 32), dtype=to_gpu(A, dtype).dtype, device="cuda")
    big[:, :K] = to_gpu(A, dtype)
    out = torch.zeros((M, K + 64), dtype=big.dtype, device="cuda")
    perm = np.random.default_rng(19).permutation(M).astype(np.int32)
    perm[4] = M + 3
    sp24.sp24_permute_rows(big[:, :K], dev_perm(perm), out=out[:, :K])
    torch.cuda.synchronize()
    safe = perm.copy()
    safe[4] = 0
    assert np.array_equal(to_bits(out[:, :K]), A[safe])
    assert not to_bits(out[:, K:]).any()


# results on both sides of 5 MiB, 32 MiB and 5120 rows, between which they are stored past the L2: read back at once by the pruning
@pytest.mark.parametrize("dtype,M,K", [("bf16", 1280, 2048), ("bf16", 1281, 2048), ("i8", 4967, 1056), ("f8", 5120, 1056), ("i8", 5121, 1056),
                                       ("f16", 1366, 6144), ("bf16", 2048, 8192), ("bf16", 2051, 8192)])
def test_permute_columns_of_results_on_both_sides_of_the_l2(dtype, M, K):
    words = {"f16": np.uint16, "bf16": np.uint16, "i8": np.int8, "f8": np.uint8}[dtype]
    A = np.frombuffer(np.random.default_rng(K).bytes(M * K * np.dtype(words).itemsize), words).reshape(M, K).copy()
    perm = np.random.default_rng(M).permutation(K).astype(np.int32)
    Ad = to_gpu(A, dtype)
    for _ in range(2):
        P = sp24.sp24_permute_columns(Ad, dev_perm(perm))
        kept = sp24.sp24_prune(P)
        torch.cuda.synchronize()
        assert np.array_equal(to_bits(P), A[:, perm])
        assert torch.equal(kept.view(torch.uint8), sp24.sp24_prune(to_gpu(np.ascontiguousarray(A[:, perm]), dtype)).view(torch.uint8))


@pytest.mark.parametrize("dtype", ["f16", "bf16", "i8"])
def test_retained_magnitude_matches_the_oracle(dtype):
    for i, (M, K) in enumerate(SHAPES):
        A = synth.make(NAME_OF[dtype], M=M, N=16, K=K, seed=90 + i)[0]
        if i == 2:   # ties, signed zeros, -128 (no NaN or infinity: a finite total to compare)
            A = adversarial(dtype, M, K, 75)
            if dtype != "i8":
                finite = (A & 0x7FFF) < (0x7C00 if dtype == "f16" else 0x7F80)
                A = np.where(finite, A, np.uint16(0x3C00 if dtype == "f16" else 0x3F80)).astype(np.uint16)
        rng = np.random.default_rng(100 + i)
        perm = rng.permutation(K).astype(np.int32)
        Ad = to_gpu(A, dtype)
        plain = sp24.sp24_retained_magnitude(Ad)
        ordered = sp24.sp24_retained_magnitude(Ad, dev_perm(perm))
        # the same number by another route on the GPU: prune the gathered matrix, add up |p| in float64
        via = sp24.sp24_prune(sp24.sp24_permute_columns(Ad, dev_perm(perm))).to(torch.float64).abs().sum()
        torch.cuda.synchronize()
        assert plain.item() == pytest.approx(oracle.retained_magnitude(A, dtype), rel=1e-12), (dtype, M, K)
        assert ordered.item() == pytest.approx(oracle.retained_magnitude(A, dtype, perm=perm), rel=1e-12), (dtype, M, K)
        assert ordered.item() == pytest.approx(via.item(), rel=1e-12)
    # int8 totals are integers below 2^53: exact whatever the order
    A = synth.make("square_i8", M=257, N=16, K=1056, seed=7)[0]
    got = sp24.sp24_retained_magnitude(to_gpu(A, "i8")).item()
    assert got == oracle.retained_magnitude(A, "i8")
    # a kept NaN makes the total NaN; an empty matrix gives 0 and overwrites what the cell held
    if dtype != "i8":
        N = synth.make(NAME_OF[dtype], M=8, N=16, K=64, seed=3)[0].copy()
        N[3, 10] = 0x7E00 if dtype == "f16" else 0x7FC0
        assert np.isnan(sp24.sp24_retained_magnitude(to_gpu(N, dtype)).item())
    cell = torch.full((1,), 5.0, dtype=torch.float64, device="cuda")
    sp24.sp24_retained_magnitude(to_gpu(A, "i8")[:0], out=cell)
    assert cell.item() == 0.0


@pytest.mark.parametrize("dtype,M,K", [("bf16", 37, 2400), ("f16", 37, 2416), ("i8", 100, 4544), ("i8", 100, 4576), ("bf16", 2051, 64),
                                       ("i8", 41, 15360), ("i8", 41, 15392), ("bf16", 1024, 160), ("f16", 1025, 160), ("bf16", 1040, 2400),
                                       ("bf16", 1040, 2416), ("i8", 1100, 4544), ("i8", 2100, 4576), ("i8", 4096, 96), ("f16", 4097, 96),
                                       ("bf16", 9000, 128)])
def test_retained_magnitude_on_both_sides_of_the_workgroup_sizes(dtype, M, K):
    """Rows that 16 (past 1024 rows), 8 or 4 wavefronts to a workgroup find room for, 128 and 256 workgroups, and more rows than one
    pass takes."""
    A = synth.make(NAME_OF[dtype], M=M, N=16, K=K, seed=K)[0]
    perm = np.random.default_rng(K).permutation(K).astype(np.int32)
    got = sp24.sp24_retained_magnitude(to_gpu(A, dtype), dev_perm(perm))
    assert got.item() == pytest.approx(oracle.retained_magnitude(A, dtype, perm=perm), rel=1e-12)      # exact terms, any order


def test_joint_permutation_leaves_the_dense_product_unchanged():
    """Sec. 4.1 Step 2: columns of A and rows of B (the columns of a K-major B) permuted alike -- same product.  Exact
    for int8; checked on the GPU's own dense product."""
    M, N, K = 96, 64, 256
    A, Bt = synth.make("square_i8", M=M, N=N, K=K, seed=12)
    perm = dev_perm(np.random.default_rng(13).permutation(K))
    Ad, Bd = to_gpu(A, "i8"), to_gpu(Bt, "i8")
    D0 = sp24.sp24_gemm_dense(Ad, Bd, torch.int32)
    D1 = sp24.sp24_gemm_dense(sp24.sp24_permute_columns(Ad, perm), sp24.sp24_permute_columns(Bd, perm), torch.int32)
    torch.cuda.synchronize()
    assert torch.equal(D0, D1)
    assert np.array_equal(D0.cpu().numpy(), oracle.gemm(A, np.ascontiguousarray(Bt.T), "i8"))


def search_on_a_copy(Ad, start, sweeps):
    """sp24_permute_search_workspace with a workspace of its own (the binding brings one where the copy is faster)."""
    lib, (M, K), dt = sp24.lib(), Ad.shape, sp24._DT[Ad.dtype]
    need, perm = lib.sp24_permute_search_workspace_bytes(M, K, dt), dev_perm(start)
    assert need > 0
    workspace = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
    assert lib.sp24_permute_search_workspace(Ad.data_ptr(), perm.data_ptr(), M, K, Ad.stride(0), dt, sweeps, workspace.data_ptr(), need, sp24._stream()) == 0
    torch.cuda.synchronize()
    return perm


# --- the search for a column order: the order found must equal the oracle's entry for entry -------------------
# rows x columns: K/4 a power of two and not (groups that sit out rounds); fewer rows than lanes, a ragged last pass
# over the rows, several passes
SEARCH_SHAPES = [(40, 32), (300, 48), (256, 64), (1000, 96), (17, 160), (2100, 128)]


@pytest.mark.parametrize("dtype", ["f16", "bf16", "i8"])
def test_permute_search_order_equals_the_oracle(dtype):
    for i, (M, K) in enumerate(SEARCH_SHAPES):
        if dtype == "i8" and K % 32:
            K += 16                                             # int8 needs K % 32 == 0; 48 -> 64 etc. keeps a mix of group counts
        A = adversarial(dtype, M, K, 170 + i) if i in (1, 4) else synth.make(NAME_OF[dtype], M=M, N=16, K=K, seed=160 + i)[0]
        Ad = to_gpu(A, dtype)
        for sweeps in (1, 2):
            got = sp24.sp24_permute_search(Ad, sweeps=sweeps)
            torch.cuda.synchronize()
            want = oracle.permute_search(A, dtype, sweeps=sweeps)
            assert np.array_equal(got.cpu().numpy(), want), (dtype, M, K, sweeps)
        # the figure of merit does not fall (both evaluated on the GPU), and the order is a permutation
        before = float(sp24.sp24_retained_magnitude(Ad).cpu()[0])
        after = float(sp24.sp24_retained_magnitude(Ad, got).cpu()[0])
        assert sorted(got.cpu().tolist()) == list(range(K))
        if not np.isnan(before):
            assert after >= before * (1 - 1e-12)


# K/4 = 4, 20, 28, 36, 44, 72, 132, 260, 304 groups: rounds of fewer than eight pairs, and of every remainder of a division by
# the eight XCDs, where the last round pairs few of the groups or most
@pytest.mark.parametrize("K", [16, 80, 112, 144, 176, 288, 528, 1040, 1216])
def test_permute_search_on_group_counts_that_are_no_power_of_two(K):
    dtype, M = "bf16", 70
    A = synth.make(NAME_OF[dtype], M=M, N=16, K=K, seed=190 + K)[0]
    got = sp24.sp24_permute_search(to_gpu(A, dtype), sweeps=2)
    torch.cuda.synchronize()
    want = oracle.permute_search(A, dtype, sweeps=2)
    assert np.array_equal(got.cpu().numpy(), want)
    if K > 32:
        assert np.array_equal(search_on_a_copy(to_gpu(A, dtype), np.arange(K, dtype=np.int32), 2).cpu().numpy(), want)


@pytest.mark.parametrize("dtype", ["f16", "bf16", "i8", "f8"])
@pytest.mark.parametrize("M,K", [(40, 64), (17, 160), (256, 64), (200, 96), (3, 288), (300, 32)])
def test_permute_search_of_small_matrices_on_a_copy(dtype, M, K):
    """Ties, infinities and NaN among them; pitched rows."""
    A = adversarial(dtype, M, K, 250) if dtype != "f8" else np.random.default_rng(250).choice(
        np.array([0x00, 0x80, 0x01, 0x81, 0x38, 0xB8, 0x39, 0x08, 0x7E, 0xFE, 0x7F, 0xFF], dtype=np.uint8), size=(M, K))
    Ad = to_gpu(A, dtype)
    big = torch.zeros((M, K + 32), dtype=torch.uint8 if dtype == "f8" else Ad.dtype, device="cuda")
    big[:, :K] = Ad.view(torch.uint8) if dtype == "f8" else Ad
    start = np.random.default_rng(251).permutation(K).astype(np.int32)
    got = search_on_a_copy((big.view(torch.float8_e4m3fn) if dtype == "f8" else big)[:, :K], start, 2)
    assert np.array_equal(got.cpu().numpy(), oracle.permute_search(A, dtype, sweeps=2, perm=start))


@pytest.mark.parametrize("dtype,K", [("bf16", 4096), ("f16", 4112), ("i8", 8192), ("f8", 8192)])
def test_permute_search_of_a_large_matrix_from_any_order(dtype, K):
    """On a copy, and in place with rows enough for the form of the kernel whose wavefronts go through them together, the last pass
    over the rows a partial one.  Rows of zeros add nothing to any sum: the oracle gets the others, each at its place modulo the 256 lanes."""
    M = 8200
    if dtype == "f8":
        A = synth.f64_to_f8_bits(np.random.default_rng(201).standard_normal((520, K)))
    else:
        A = synth.make(NAME_OF[dtype], M=520, N=16, K=K, seed=201)[0]
    Ad = to_gpu(A, dtype)
    big = torch.zeros((M, K), dtype=Ad.dtype, device="cuda")
    big.view(torch.uint8)[:512], big.view(torch.uint8)[8192:] = Ad.view(torch.uint8)[:512], Ad.view(torch.uint8)[512:]
    start = np.random.default_rng(202).permutation(K).astype(np.int32)
    got, placed = sp24.sp24_permute_search(big, perm=dev_perm(start)), dev_perm(start)
    assert sp24.lib().sp24_permute_search(big.data_ptr(), placed.data_ptr(), M, K, K, sp24._DT[big.dtype], 1, sp24._stream()) == 0
    torch.cuda.synchronize()
    want = oracle.permute_search(A, dtype, sweeps=1, perm=start)
    assert np.array_equal(got.cpu().numpy(), want)
    assert np.array_equal(placed.cpu().numpy(), want)


# four workgroups to a pair of groups (up to 64 pairs, 512 columns), two (up to 192, and floats past 256 with few pairs or 1024 rows) and one (the
# others), at the edges of the copy's blocks of 512 rows and of their halves; int8 sums past what 16 bits hold; the search in place and the one
# on a copy find the same order
@pytest.mark.parametrize("dtype,M,K", [("bf16", 256, 512), ("f16", 257, 528), ("f8", 513, 544), ("i8", 1024, 1024), ("bf16", 1537, 1040),
                                       ("f16", 2048, 1040), ("i8", 769, 1056), ("i8", 130_600, 32),
                                       ("bf16", 769, 1536), ("bf16", 513, 1552), ("f16", 300, 2048), ("f8", 1025, 2048), ("i8", 300, 2048),  # 192 | 194, 256, one
                                       ("f16", 600, 2064), ("f8", 513, 3584), ("bf16", 700, 3600), ("f16", 1023, 4096), ("bf16", 1024, 4096),  # 258, 448 | 450, one to 1023
                                       ("bf16", 513, 8192), ("i8", 513, 8192)])
def test_permute_search_in_place_and_on_a_copy(dtype, M, K):
    A = adversarial(dtype, M, K, 210) if dtype != "f8" else synth.f64_to_f8_bits(np.random.default_rng(210).standard_normal((M, K)))
    if M > 100_000:
        A = np.where(A % 3, np.int8(-128), A)                    # the largest magnitude in most places
    Ad, lib = to_gpu(A, dtype), sp24.lib()
    start = np.random.default_rng(211).permutation(K).astype(np.int32)
    copied, placed = search_on_a_copy(Ad, start, 2), dev_perm(start)
    assert lib.sp24_permute_search(Ad.data_ptr(), placed.data_ptr(), M, K, K, sp24._DT[Ad.dtype], 2, sp24._stream()) == 0
    torch.cuda.synchronize()
    assert torch.equal(copied, placed)
    assert np.array_equal(copied.cpu().numpy(), oracle.permute_search(A, dtype, sweeps=2, perm=start))


# few rows: in place from the order of memory, on a copy from a given one (floats, many columns), in place both ways (two or three rounds; int8 from 193
# pairs on; small matrices, unless a graph is recorded)
@pytest.mark.parametrize("dtype,M,K,default,given", [("bf16", 300, 4096, False, True), ("f16", 401, 4096, True, True), ("bf16", 600, 8192, False, True),
                                                     ("i8", 300, 4096, True, True), ("i8", 255, 2048, False, False), ("i8", 256, 2048, True, True),
                                                     ("bf16", 255, 32, False, False), ("f16", 257, 32, True, True),
                                                     ("f8", 256, 512, False, False), ("bf16", 257, 512, True, True), ("f16", 128, 1024, False, False),
                                                     ("f16", 129, 1024, True, True)])
def test_permute_search_of_few_rows_by_either_route(dtype, M, K, default, given):
    A = synth.make(NAME_OF[dtype], M=M, N=16, K=K, seed=220)[0] if dtype != "f8" else synth.f64_to_f8_bits(np.random.default_rng(220).standard_normal((M, K)))
    Ad = to_gpu(A, dtype)
    assert (sp24._search_workspace(Ad, True) is not None, sp24._search_workspace(Ad, False) is not None) == (default, given)
    first = sp24.sp24_permute_search(Ad)
    again = sp24.sp24_permute_search(Ad, perm=dev_perm(np.arange(K)))
    torch.cuda.synchronize()
    assert torch.equal(first, again)
    assert np.array_equal(first.cpu().numpy(), oracle.permute_search(A, dtype, sweeps=1))


def test_permute_search_without_memory_for_the_copy(monkeypatch):
    dtype, M, K = "bf16", 300, 1024
    A = synth.make(NAME_OF[dtype], M=M, N=16, K=K, seed=230)[0]
    Ad, start = to_gpu(A, dtype), np.random.default_rng(231).permutation(K).astype(np.int32)
    perm = dev_perm(start)
    asked = []

    def no_memory(*args, **kwargs):
        asked.append(args)
        raise torch.cuda.OutOfMemoryError("none left")

    monkeypatch.setattr(torch, "empty", no_memory)
    sp24.sp24_permute_search(Ad, sweeps=2, perm=perm)
    monkeypatch.undo()
    torch.cuda.synchronize()
    assert asked and np.array_equal(perm.cpu().numpy(), oracle.permute_search(A, dtype, sweeps=2, perm=start))


def test_permute_search_on_a_copy_replays_from_a_graph():
    """The copy's memory is the graph's own; each replay on other weights, with eager searches in between."""
    dtype, M, K = "bf16", 700, 1024
    sets = [synth.make(NAME_OF[dtype], M=M, N=16, K=K, seed=240 + i)[0] for i in range(3)]
    A, perm, start = to_gpu(sets[0], dtype).clone(), dev_perm(np.arange(K)), dev_perm(np.random.default_rng(241).permutation(K))
    assert sp24._search_workspace(A, False) is not None

    def path():
        perm.copy_(start)
        sp24.sp24_permute_search(A, sweeps=2, perm=perm)

    path()
    torch.cuda.synchronize()
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side):
        path()
    torch.cuda.synchronize()
    for bits in sets[1:] + sets[:1]:
        A.copy_(to_gpu(bits, dtype))
        graph.replay()
        torch.cuda.synchronize()
        replayed = perm.clone()
        path()
        torch.cuda.synchronize()
        assert torch.equal(replayed, perm)
        assert np.array_equal(perm.cpu().numpy(), oracle.permute_search(bits, dtype, sweeps=2, perm=start.cpu().numpy()))


def test_permute_search_starts_from_a_given_order_and_takes_pitched_rows():
    dtype, M, K = "bf16", 500, 96
    A = synth.make(NAME_OF[dtype], M=M, N=16, K=K, seed=181)[0]
    rng = np.random.default_rng(182)
    start = rng.permutation(K).astype(np.int32)
    big = torch.zeros((M, K + 40), dtype=torch.bfloat16, device="cuda")
    big[:, :K] = to_gpu(A, dtype)
    perm = dev_perm(start)
    out = sp24.sp24_permute_search(big[:, :K], sweeps=2, perm=perm)
    torch.cuda.synchronize()
    assert out.data_ptr() == perm.data_ptr()                    # refined in place
    assert np.array_equal(out.cpu().numpy(), oracle.permute_search(A, dtype, sweeps=2, perm=start))
    # zero sweeps and an empty matrix leave the order alone
    perm2 = dev_perm(start)
    sp24.sp24_permute_search(to_gpu(A, dtype), sweeps=0, perm=perm2)
    sp24.sp24_permute_search(to_gpu(A, dtype)[:0], sweeps=3, perm=perm2)
    torch.cuda.synchronize()
    assert np.array_equal(perm2.cpu().numpy(), start)


def test_permute_search_ties_heavy_int8_and_equal_columns():
    # few distinct magnitudes: most ways tie and the first must win; all columns equal: nothing moves
    rng = np.random.default_rng(183)
    A = rng.integers(-2, 3, size=(700, 128)).astype(np.int8)
    got = sp24.sp24_permute_search(to_gpu(A, "i8"), sweeps=2)
    E = np.full((64, 64), 7, dtype=np.int8)
    same = sp24.sp24_permute_search(to_gpu(E, "i8"), sweeps=1)
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), oracle.permute_search(A, "i8", sweeps=2))
    assert np.array_equal(same.cpu().numpy(), np.arange(64))


def test_permute_search_leaves_the_sparse_product_path_consistent():
    # the order found, applied to the weights' columns and to the K-major second operand alike, gives a pruned
    # product that the oracle reproduces from the same permuted operands (Sec. 4.1: the result of the layer is kept)
    dtype, M, K, N = "i8", 128, 256, 64
    A, Bt = synth.make(NAME_OF[dtype], M=M, N=N, K=K, seed=184)
    Ad, Bd = to_gpu(A, dtype), to_gpu(Bt, dtype)
    perm = sp24.sp24_permute_search(Ad, sweeps=1)
    Ap, Bp = sp24.sp24_permute_columns(Ad, perm), sp24.sp24_permute_columns(Bd, perm)
    V, meta = sp24.sp24_compress(Ap, layout="tiled")
    D = sp24.sp24_spmm(V, meta, Bp, torch.int32, layout="tiled")
    torch.cuda.synchronize()
    p = perm.cpu().numpy()
    ref = oracle.gemm(oracle.prune(np.ascontiguousarray(A[:, p]), dtype), np.ascontiguousarray(Bt[:, p].T), dtype)
    assert np.array_equal(D.cpu().numpy(), ref)
