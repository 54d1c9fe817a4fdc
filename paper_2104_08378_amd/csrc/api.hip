// C ABI of libsp24: argument validation on the host, then kernel selection.
// Nothing here allocates, synchronises or touches the current device.
#include <algorithm>
#include <atomic>

#include "common.hpp"
#include "launch.hpp"

using namespace sp24;

// Memory of the library's own for sp24_spmm_splitk_static, whose callers cannot allocate or pass a workspace: the
// partial products of the split product live here instead.  Every GPU the library runs on holds its own copy of
// the array until the process ends.  In host code the array's name stands for the symbol, it is not a device
// address: the address on the current device comes from hipGetSymbolAddress (static_scratch() below), and only
// that pointer is handed to kernels.
static __device__ __align__(256) unsigned char scratch[SP24_STATIC_SCRATCH_BYTES];

namespace {

bool is_input_type(sp24_dtype t) { return t == SP24_F16 || t == SP24_BF16 || t == SP24_I8 || t == SP24_F8; }
bool is_layout(sp24_layout l) { return l == SP24_LAYOUT_CANONICAL || l == SP24_LAYOUT_TILED; }
bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Dimension rule of Sec. 3.2 / Sec. 4.2 on the inner dimension.
bool k_legal(int64_t K, sp24_dtype t) { return K > 0 && K % (esize_of(t) == 1 ? 32 : 16) == 0; }

bool layout_fits(int64_t M, int64_t K, sp24_layout l)
{
    return l == SP24_LAYOUT_CANONICAL || (M % 32 == 0 && K % 64 == 0);
}

bool out_legal(sp24_dtype in, sp24_dtype out, bool scaled)
{
    if (scaled) return in == SP24_I8 && (out == SP24_I8 || out == SP24_F32 || out == SP24_F16 || out == SP24_BF16);
    if (in == SP24_I8) return out == SP24_I32;
    return out == SP24_F32 || out == SP24_F16 || out == SP24_BF16;
}

// a matrix of `rows` rows, `cols` used columns, leading dimension ld (elements of size es);
// vec16: rows must start on 16-byte boundaries (the streaming kernels use 16-byte accesses),
// otherwise natural element alignment is enough.
sp24_status check_matrix(const void* p, int64_t rows, int64_t cols, int64_t ld, int es, bool vec16 = true)
{
    if (rows == 0) return SP24_OK;
    if (!p) return SP24_ERR_NULL;
    if (ld < cols) return SP24_ERR_SHAPE;
    if (vec16 ? (!aligned16(p) || (ld * es) % 16 != 0) : (reinterpret_cast<uintptr_t>(p) % es != 0)) return SP24_ERR_ALIGN;
    return SP24_OK;
}

bool ranges_overlap(const void* a, size_t na, const void* b, size_t nb)
{
    uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return x < y + nb && y < x + na;
}

} // namespace

extern "C" {

size_t sp24_values_bytes(int64_t M, int64_t K, sp24_dtype t)
{
    if (!is_input_type(t) || M < 0 || !k_legal(K, t)) return 0;
    return (size_t)M * (size_t)(K / 2) * (size_t)esize_of(t);
}

size_t sp24_meta_bytes(int64_t M, int64_t K, sp24_dtype t, sp24_layout l)
{
    if (!is_input_type(t) || !is_layout(l) || M < 0 || !k_legal(K, t) || !layout_fits(M, K, l)) return 0;
    return (size_t)M * (size_t)(K / 8);
}

sp24_status sp24_prune(const void* A, void* P, int64_t M, int64_t K, int64_t lda, int64_t ldp, sp24_dtype t, void* stream)
{
    if (!is_input_type(t)) return SP24_ERR_DTYPE;
    if (M < 0 || !k_legal(K, t)) return SP24_ERR_SHAPE;
    int es = esize_of(t);
    sp24_status s = check_matrix(A, M, K, lda, es);
    if (s != SP24_OK) return s;
    s = check_matrix(P, M, K, ldp, es);
    if (s != SP24_OK) return s;
    if (M > 0 && A == P && lda != ldp) return SP24_ERR_SHAPE;
    if (M > 0 && A != P) {
        size_t na = ((size_t)(M - 1) * lda + K) * es, np = ((size_t)(M - 1) * ldp + K) * es;
        if (ranges_overlap(A, na, P, np)) return SP24_ERR_SHAPE;
    }
    return launch_prune(A, P, M, K, lda, ldp, t, static_cast<hipStream_t>(stream));
}

sp24_status sp24_compress(const void* A, void* V, void* meta, int64_t M, int64_t K, int64_t lda, sp24_dtype t,
                          sp24_layout l, void* stream)
{
    if (!is_input_type(t)) return SP24_ERR_DTYPE;
    if (!is_layout(l)) return SP24_ERR_LAYOUT;
    if (M < 0 || !k_legal(K, t)) return SP24_ERR_SHAPE;
    if (!layout_fits(M, K, l)) return SP24_ERR_LAYOUT;
    int es = esize_of(t);
    sp24_status s = check_matrix(A, M, K, lda, es);
    if (s != SP24_OK) return s;
    if (M == 0) return SP24_OK;
    if (!V || !meta) return SP24_ERR_NULL;
    if (!aligned16(V) || !aligned16(meta)) return SP24_ERR_ALIGN;
    size_t na = ((size_t)(M - 1) * lda + K) * es;
    if (ranges_overlap(A, na, V, sp24_values_bytes(M, K, t)) || ranges_overlap(A, na, meta, sp24_meta_bytes(M, K, t, l)))
        return SP24_ERR_SHAPE;
    return launch_compress(A, V, meta, M, K, lda, t, l, static_cast<hipStream_t>(stream));
}

sp24_status sp24_decompress(const void* V, const void* meta, void* P, int64_t M, int64_t K, int64_t ldp, sp24_dtype t,
                            sp24_layout l, void* stream)
{
    if (!is_input_type(t)) return SP24_ERR_DTYPE;
    if (!is_layout(l)) return SP24_ERR_LAYOUT;
    if (M < 0 || !k_legal(K, t)) return SP24_ERR_SHAPE;
    if (!layout_fits(M, K, l)) return SP24_ERR_LAYOUT;
    int es = esize_of(t);
    sp24_status s = check_matrix(P, M, K, ldp, es);
    if (s != SP24_OK) return s;
    if (M == 0) return SP24_OK;
    if (!V || !meta) return SP24_ERR_NULL;
    if (!aligned16(V) || !aligned16(meta)) return SP24_ERR_ALIGN;
    size_t np = ((size_t)(M - 1) * ldp + K) * es;
    if (ranges_overlap(P, np, V, sp24_values_bytes(M, K, t)) || ranges_overlap(P, np, meta, sp24_meta_bytes(M, K, t, l)))
        return SP24_ERR_SHAPE;
    return launch_decompress(V, meta, P, M, K, ldp, t, l, static_cast<hipStream_t>(stream));
}

sp24_status sp24_prune_transposable(const void* A, void* P, int64_t M, int64_t K, int64_t lda, int64_t ldp, sp24_dtype t, void* stream)
{
    if (!is_input_type(t)) return SP24_ERR_DTYPE;
    if (M < 0 || M % 4 != 0 || !k_legal(K, t)) return SP24_ERR_SHAPE;
    int es = esize_of(t);
    sp24_status s = check_matrix(A, M, K, lda, es);
    if (s != SP24_OK) return s;
    s = check_matrix(P, M, K, ldp, es);
    if (s != SP24_OK) return s;
    if (M > 0 && A == P && lda != ldp) return SP24_ERR_SHAPE;
    if (M > 0 && A != P) {
        size_t na = ((size_t)(M - 1) * lda + K) * es, np = ((size_t)(M - 1) * ldp + K) * es;
        if (ranges_overlap(A, na, P, np)) return SP24_ERR_SHAPE;
    }
    return launch_prune_transposable(A, P, M, K, lda, ldp, t, static_cast<hipStream_t>(stream));
}

sp24_status sp24_mask_apply(const void* W, const void* meta, void* P, int64_t M, int64_t K, int64_t ldw, int64_t ldp, sp24_dtype t,
                            sp24_layout l, void* stream)
{
    if (!is_input_type(t)) return SP24_ERR_DTYPE;
    if (!is_layout(l)) return SP24_ERR_LAYOUT;
    if (M < 0 || !k_legal(K, t)) return SP24_ERR_SHAPE;
    if (!layout_fits(M, K, l)) return SP24_ERR_LAYOUT;
    int es = esize_of(t);
    sp24_status s = check_matrix(W, M, K, ldw, es);
    if (s != SP24_OK) return s;
    s = check_matrix(P, M, K, ldp, es);
    if (s != SP24_OK) return s;
    if (M == 0) return SP24_OK;
    if (!meta) return SP24_ERR_NULL;
    if (!aligned16(meta)) return SP24_ERR_ALIGN;
    if (W == P && ldw != ldp) return SP24_ERR_SHAPE;
    size_t nw = ((size_t)(M - 1) * ldw + K) * es, np = ((size_t)(M - 1) * ldp + K) * es;
    if (W != P && ranges_overlap(W, nw, P, np)) return SP24_ERR_SHAPE;
    if (ranges_overlap(P, np, meta, sp24_meta_bytes(M, K, t, l))) return SP24_ERR_SHAPE;
    return launch_mask_apply(W, meta, P, M, K, ldw, ldp, t, l, static_cast<hipStream_t>(stream));
}

sp24_status sp24_compress_masked(const void* W, const void* meta, void* V, int64_t M, int64_t K, int64_t ldw, sp24_dtype t,
                                 sp24_layout l, void* stream)
{
    if (!is_input_type(t)) return SP24_ERR_DTYPE;
    if (!is_layout(l)) return SP24_ERR_LAYOUT;
    if (M < 0 || !k_legal(K, t)) return SP24_ERR_SHAPE;
    if (!layout_fits(M, K, l)) return SP24_ERR_LAYOUT;
    int es = esize_of(t);
    sp24_status s = check_matrix(W, M, K, ldw, es);
    if (s != SP24_OK) return s;
    if (M == 0) return SP24_OK;
    if (!V || !meta) return SP24_ERR_NULL;
    if (!aligned16(V) || !aligned16(meta)) return SP24_ERR_ALIGN;
    size_t nw = ((size_t)(M - 1) * ldw + K) * es, nv = sp24_values_bytes(M, K, t);
    if (ranges_overlap(W, nw, V, nv) || ranges_overlap(V, nv, meta, sp24_meta_bytes(M, K, t, l))) return SP24_ERR_SHAPE;
    return launch_compress_masked(W, meta, V, M, K, ldw, t, l, static_cast<hipStream_t>(stream));
}

sp24_status sp24_permute_columns(const void* A, const int32_t* perm, void* P, int64_t M, int64_t K, int64_t lda, int64_t ldp,
                                 sp24_dtype t, void* stream)
{
    if (!is_input_type(t)) return SP24_ERR_DTYPE;
    if (M < 0 || !k_legal(K, t) || K > 0x7FFFFFFF) return SP24_ERR_SHAPE;
    int es = esize_of(t);
    sp24_status s = check_matrix(A, M, K, lda, es);
    if (s != SP24_OK) return s;
    s = check_matrix(P, M, K, ldp, es);
    if (s != SP24_OK) return s;
    if (M == 0) return SP24_OK;
    if (!perm) return SP24_ERR_NULL;
    if (reinterpret_cast<uintptr_t>(perm) % 4 != 0) return SP24_ERR_ALIGN;
    size_t na = ((size_t)(M - 1) * lda + K) * es, np = ((size_t)(M - 1) * ldp + K) * es;
    if (ranges_overlap(A, na, P, np) || ranges_overlap(P, np, perm, (size_t)K * 4)) return SP24_ERR_SHAPE;
    return launch_permute_columns(A, perm, P, M, K, lda, ldp, t, static_cast<hipStream_t>(stream));
}

sp24_status sp24_permute_rows(const void* A, const int32_t* perm, void* P, int64_t M, int64_t K, int64_t lda, int64_t ldp, sp24_dtype t,
                              void* stream)
{
    if (!is_input_type(t)) return SP24_ERR_DTYPE;
    if (M < 0 || M > 0x7FFFFFFF || !k_legal(K, t)) return SP24_ERR_SHAPE;
    int es = esize_of(t);
    sp24_status s = check_matrix(A, M, K, lda, es);
    if (s != SP24_OK) return s;
    s = check_matrix(P, M, K, ldp, es);
    if (s != SP24_OK) return s;
    if (M == 0) return SP24_OK;
    if (!perm) return SP24_ERR_NULL;
    if (reinterpret_cast<uintptr_t>(perm) % 4 != 0) return SP24_ERR_ALIGN;
    size_t na = ((size_t)(M - 1) * lda + K) * es, np = ((size_t)(M - 1) * ldp + K) * es;
    if (ranges_overlap(A, na, P, np) || ranges_overlap(P, np, perm, (size_t)M * 4)) return SP24_ERR_SHAPE;
    return launch_permute_rows(A, perm, P, M, K, lda, ldp, t, static_cast<hipStream_t>(stream));
}

sp24_status sp24_retained_magnitude(const void* A, const int32_t* perm, double* total, int64_t M, int64_t K, int64_t lda,
                                    sp24_dtype t, void* stream)
{
    if (!is_input_type(t)) return SP24_ERR_DTYPE;
    if (M < 0 || !k_legal(K, t) || K > 0x7FFFFFFF) return SP24_ERR_SHAPE;
    int es = esize_of(t);
    sp24_status s = check_matrix(A, M, K, lda, es);
    if (s != SP24_OK) return s;
    if (!total) return SP24_ERR_NULL;
    if (reinterpret_cast<uintptr_t>(total) % 8 != 0 || reinterpret_cast<uintptr_t>(perm) % 4 != 0) return SP24_ERR_ALIGN;
    if (M > 0) {
        size_t na = ((size_t)(M - 1) * lda + K) * es;
        if (ranges_overlap(A, na, total, 8) || (perm && ranges_overlap(perm, (size_t)K * 4, total, 8))) return SP24_ERR_SHAPE;
    }
    return launch_retained_magnitude(A, perm, total, M, K, lda, t, static_cast<hipStream_t>(stream));
}

static sp24_status check_permute_search(const void* A, const int32_t* perm, int64_t M, int64_t K, int64_t lda, sp24_dtype t, int sweeps)
{
    if (!is_input_type(t)) return SP24_ERR_DTYPE;
    if (M < 0 || !k_legal(K, t) || K > 0x7FFFFFFF || sweeps < 0 || sweeps > 64) return SP24_ERR_SHAPE;
    int es = esize_of(t);
    sp24_status s = check_matrix(A, M, K, lda, es);
    if (s != SP24_OK) return s;
    if (!perm) return SP24_ERR_NULL;
    if (reinterpret_cast<uintptr_t>(perm) % 4 != 0) return SP24_ERR_ALIGN;
    if (M > 0 && ranges_overlap(A, ((size_t)(M - 1) * lda + K) * es, perm, (size_t)K * 4)) return SP24_ERR_SHAPE;
    return SP24_OK;
}

sp24_status sp24_permute_search(const void* A, int32_t* perm, int64_t M, int64_t K, int64_t lda, sp24_dtype t, int sweeps, void* stream)
{
    const sp24_status s = check_permute_search(A, perm, M, K, lda, t, sweeps);
    return s != SP24_OK ? s : launch_permute_search(A, perm, M, K, lda, t, sweeps, static_cast<hipStream_t>(stream));
}

size_t sp24_permute_search_workspace_bytes(int64_t M, int64_t K, sp24_dtype t)
{
    return is_input_type(t) && M >= 0 && k_legal(K, t) && K <= 0x7FFFFFFF ? permute_search_workspace(M, K, t) : 0;
}

sp24_status sp24_permute_search_workspace(const void* A, int32_t* perm, int64_t M, int64_t K, int64_t lda, sp24_dtype t, int sweeps,
                                          void* workspace, size_t workspace_bytes, void* stream)
{
    const sp24_status s = check_permute_search(A, perm, M, K, lda, t, sweeps);
    if (s != SP24_OK) return s;
    const size_t need = permute_search_workspace(M, K, t);
    if (!workspace || need == 0) return launch_permute_search(A, perm, M, K, lda, t, sweeps, static_cast<hipStream_t>(stream));
    if (reinterpret_cast<uintptr_t>(workspace) % 16 != 0) return SP24_ERR_ALIGN;
    if (workspace_bytes < need || ranges_overlap(workspace, need, A, ((size_t)(M - 1) * lda + K) * esize_of(t)) ||
        ranges_overlap(workspace, need, perm, (size_t)K * 4))
        return SP24_ERR_SHAPE;
    return launch_permute_search_columns(A, perm, M, K, lda, t, sweeps, workspace, static_cast<hipStream_t>(stream));
}

// Argument checks of every product entry point.  *empty: nothing to compute (M or N is 0).
// x_bytes: extent of the NHWC input when a.conv.on (a.B then points at it), else unused
static sp24_status mm_validate(const MmArgs& a, size_t x_bytes, bool* empty)
{
    *empty = false;
    if (!is_input_type(a.in) || !out_legal(a.in, a.out, a.epi.on != 0)) return SP24_ERR_DTYPE;
    if (a.bo != SP24_B_KMAJOR && a.bo != SP24_B_NMAJOR) return SP24_ERR_LAYOUT;
    if (a.M < 0 || a.N < 0 || !k_legal(a.K, a.in)) return SP24_ERR_SHAPE;
    if (a.sparse) {
        if (!is_layout(a.layout)) return SP24_ERR_LAYOUT;
        if (!layout_fits(a.M, a.K, a.layout)) return SP24_ERR_LAYOUT;
    }
    if (a.M == 0 || a.N == 0) {
        *empty = true;
        return SP24_OK;
    }
    int es = esize_of(a.in), os = esize_of(a.out);
    sp24_status s;
    if (a.epi.on) {
        if (!a.epi.w_scale) return SP24_ERR_NULL;
        if (reinterpret_cast<uintptr_t>(a.epi.w_scale) % 4 != 0 || reinterpret_cast<uintptr_t>(a.epi.bias) % 4 != 0) return SP24_ERR_ALIGN;
    }
    if (a.sparse) {
        if (!a.A || !a.meta) return SP24_ERR_NULL;
        if (!aligned16(a.A) || !aligned16(a.meta)) return SP24_ERR_ALIGN;
    } else {
        s = check_matrix(a.A, a.M, a.K, a.lda, es);
        if (s != SP24_OK) return s;
    }
    if (a.conv.on) {
        if (!a.B) return SP24_ERR_NULL;
        if (reinterpret_cast<uintptr_t>(a.B) % es != 0) return SP24_ERR_ALIGN;
    } else {
        s = (a.bo == SP24_B_KMAJOR) ? check_matrix(a.B, a.N, a.K, a.ldb, es, false) : check_matrix(a.B, a.K, a.N, a.ldb, es, false);
        if (s != SP24_OK) return s;
    }
    s = check_matrix(a.D, a.M, a.N, a.ldd, os, false);
    if (s != SP24_OK) return s;
    size_t nd = ((size_t)(a.M - 1) * a.ldd + a.N) * os;
    size_t nb = a.conv.on ? x_bytes
                          : (a.bo == SP24_B_KMAJOR) ? ((size_t)(a.N - 1) * a.ldb + a.K) * es : ((size_t)(a.K - 1) * a.ldb + a.N) * es;
    size_t nA = a.sparse ? sp24_values_bytes(a.M, a.K, a.in) : ((size_t)(a.M - 1) * a.lda + a.K) * es;
    if (ranges_overlap(a.D, nd, a.B, nb) || ranges_overlap(a.D, nd, a.A, nA)) return SP24_ERR_SHAPE;
    if (a.sparse && ranges_overlap(a.D, nd, a.meta, sp24_meta_bytes(a.M, a.K, a.in, a.layout))) return SP24_ERR_SHAPE;
    if (a.epi.on && (ranges_overlap(a.D, nd, a.epi.w_scale, (size_t)a.M * 4) ||
                     (a.epi.bias && ranges_overlap(a.D, nd, a.epi.bias, (size_t)a.M * 4))))
        return SP24_ERR_SHAPE;
    return SP24_OK;
}

// N <= 32: where the tiled kernels (tiles of 64 or 128 rows, most of their columns unused) overtake the streaming
// kernel, whose workgroups of 32 rows each re-read all of B and run in more than one round past 256 row blocks.
// Measured at K = 4096 and 8192, M = 2048 .. 128256, operands from HBM, in tiles = ceil(M / 128):
//  * N > 16: the dense product always (M = 4096, K = 8192, N = 32: 40.6 -> 32.6 us), the sparse one from 86 tiles on
//    (11008 rows; below that it depends on M, within 15 % either way);
//  * N <= 16, 16-bit: from 86 tiles on, sparse 3 - 10 % faster up to 128 tiles (of 64 x 64 then), level to 191, then
//    ahead for good (32000 x 4096, N = 1: 36.4 -> 31.5 us; 128256 rows: 133 -> 117 us); dense 15 - 30 % faster
//    at 86 - 256 tiles, past that only for N > 8;
//  * N <= 16, 8-bit: the dense product for N > 8 from 86 tiles on; the sparse one stays with the streaming kernel
//    (10 - 20 % ahead at N <= 8 up to 128256 rows, level at N = 16).
static bool tiled_before_streaming(const MmArgs& a)
{
    if (a.N > 32) return true;                             // the streaming kernel does not take it anyway
    const int64_t tiles = (a.M + 127) / 128;
    if (a.N > 16) return !a.sparse || tiles >= 86;
    if (esize_of(a.in) == 2) return tiles >= 86 && (a.sparse || tiles <= 256 || a.N > 8);
    return !a.sparse && a.N > 8 && tiles >= 86;
}

// Sparse products whose tiles of 32 rows and 16, 32 or 64 columns each find a compute unit of their own: the kernel that
// splits K across a workgroup's wavefronts.  One workgroup's rings fill a unit's LDS, so a second round costs the whole
// time again: measured against the streaming and the tiled kernels, up to 256 workgroups 1.0 - 2.7 times as fast with 65 - 512
// columns (averages from the L2 / the last-level cache / HBM, K 512 - 8192: tiled layout bf16 1.28 / 1.3 / 1.41, int8 1.2 / 1.23 / 1.29,
// canonical 1.6 / 1.71 / 1.91 and 1.25 / 1.42 / 1.54; 1024 x 128 x 4096 bf16 11.3 -> 8.3 us, from HBM 20.8 -> 13.0) and 1.05 - 2.4 with fewer
// (8192 x 32 x 8192 25.1 -> 14.0, 8192 x 16 x 8192 18.1 -> 13.3; 4096 x 1 x 1024
// level; with the compressed operand from HBM 8192 x 16 x 8192 19.3 -> 16.4, 8192 x 64 x 8192 32.3 -> 27.8), past that 0.7 -
// 1.05 times in the tiled layout and 0.7 - 1.46 in the canonical one (averages 0.7 - 0.88 and 0.8 - 1.16) -- except for 16-bit inputs with N <= 32
// up to the 86 tiles of 128 rows from which the tiled kernels take them
// (9216 x 16 x 4096 17.0 -> 12.3 us in two rounds; 10976 x 16 x 1024, 86 tiles, 5.7 us on the tiled kernels against 6.6).  Where
// K has few steps and a partial one behind them, two rounds are 5 - 20 % behind the tiled kernels too (9098 x 17 x 288 4.8 us
// against 5.6).
// The limit of 512 columns is not one of speed: 32 - 512 rows on 513 - 2048 columns, up to 256 workgroups, would run 1.0 - 1.8 times as
// fast here in the tiled layout and 1.0 - 2.7 in the canonical one (128 x 1000 x 4096 bf16 11.7 -> 8.2 us, 17.3 -> 9.9 canonical).
// It keeps wide products of 16-bit types with few rows, convolutions written out
// among them, on the kernel that adds K in the order of the implicit convolution with one chunk of channels, so that the two
// agree bit for bit; narrower ones have not agreed since this kernel takes them, and the interface promises neither.
static bool stream_first(const MmArgs& a)
{
    if (!a.sparse || a.conv.on) return false;
    // An N-major B whose rows the transfers can fetch: the same rule without the limit of 512 columns.  Against the tiled kernels, times as fast
    // from the caches / from HBM, 32 - 8192 rows and 16 - 16384 columns, 2 - 128 steps: tiled layout bf16 1.13 - 2.9 / 1.1 - 2.6 (1024 x 512 x
    // 4096 15.4 -> 11.7 us, 512 x 128 x 8192 from HBM 37.4 -> 21.0), int8 1.0 - 3.0 / 1.02 - 2.5 (1024 x 512 x 4096 11.2 -> 9.4); canonical
    // from 8 steps on 0.95 - 2.1 / 1.0 - 2.6 and 1.04 - 2.5 / 1.02 - 2.2, with fewer 0.92 - 1.09; past 4096 columns 0.98 and more throughout.
    // On 257 - 512 workgroups 0.63 - 1.04, except for canonical 16-bit operands, past 32 columns and from 32 steps on: 0.98 - 1.20 / 1.04 - 1.54
    // (4096 x 192 x 2048 14.1 -> 13.0, from HBM 16.7 -> 13.9) with 128 rows and more and rows of B that are whole cache lines.  Rows that begin
    // inside a line 0.83 - 1.0 from the caches (1024 x 784 x 2048 14.1 -> 15.6), 64 - 96 rows 0.83 - 1.04 / 0.90 - 1.02 (96 x 10624 x 3072 from HBM 27.7 -> 30.2).
    if (a.bo == SP24_B_NMAJOR) {
        const int64_t es = esize_of(a.in), steps = a.K * es / 128;
        const bool whole_chunks = reinterpret_cast<uintptr_t>(a.B) % 16 == 0 && a.ldb * es % 16 == 0 && a.N * es % 16 == 0;
        const bool whole_lines = reinterpret_cast<uintptr_t>(a.B) % 128 == 0 && a.ldb * es % 128 == 0;
        const bool canonical = a.layout == SP24_LAYOUT_CANONICAL;
        const int most = canonical && es == 2 && a.N > 32 && a.M >= 128 && steps >= 32 && whole_lines ? 512 : 256;
        return whole_chunks && steps >= (canonical ? 8 : 2) && stream_workgroups(a) <= most;
    }
    if (a.N > 512) return false;
    // Few steps of an 8-bit operand: a wavefront has one at most, and the partial step at the end of K comes behind it.  With
    // N <= 32 the streaming kernel is 5 - 17 % ahead below four whole steps, and below eight where the last is a partial one
    // (33 - 8192 rows, replayed: K = 64 2.6 - 3.0 us against 3.0 - 3.5, 192 2.7 - 3.1 against 3.0 - 3.4, 576 2.9 - 3.6 against
    // 3.3 - 3.7; at 512 level in the tiled layout, 10 % behind in the canonical one).  Half a tile of 64 columns at the end costs
    // it more (32 x 16 x 288 3.2 here against 2.9).  16-bit types are level or behind there, and wider products within 5 %.
    if (a.N <= 32 && esize_of(a.in) == 1 && a.K % 64 == 0 && a.K < (a.K % 128 == 0 ? 512 : 1024)) return false;
    // Not one whole step, up to 64 columns: tiles of 64 x 64, one to a workgroup of two wavefronts (33 - 64 columns, 64 - 4096 rows
    // 2.8 - 3.5 us against 3.2 - 4.4; fewer 2.7 - 3.1 against 3.0 - 3.4; wider products are level or up to 12 % behind).
    if (a.N <= 64 && a.K * esize_of(a.in) < 128) return false;
    return stream_workgroups(a) <= 256 || (a.N <= 32 && esize_of(a.in) == 2 && (a.M + 127) / 128 < 86 && (a.K % 64 == 0 || a.K >= 1024));
}

// Sparse products that the tiled kernels do not take: tiles of their shape with B staged through registers, or (N-major,
// few tiles) K split across the wavefronts of a workgroup, which the former leaves idle.  Measured on N-major products
// with an odd N: up to 64 tiles of 128 x 128 the K-splitting kernel is ahead with many steps, from 72 on the staged one throughout
// (1.0 - 1.6 times as fast; 2560 x 509 x 2048 bf16 12.6 us against 16.3, 4096 x 257 x 4096 21.1 against 30.5).
// Between 257 workgroups of 32 x 64, past which the K-splitting kernel takes two row blocks to a workgroup, and 64 tiles the staged
// one is ahead with few steps.  Its time over the other's from the L2 / the last-level cache / HBM: tiled layout 0.73 - 0.87 /
// 0.72 - 0.86 / 0.72 - 0.87 up to 4 steps, 0.82 - 0.93 / 0.87 - 0.99 / 0.93 - 1.02 at 16, 0.87 - 0.94 / 0.91 - 1.04 / 0.96 - 1.07 at 20;
// canonical 0.9 - 1.0 / 0.91 - 1.03 / 0.91 - 1.03 at 4, 1.0 - 1.1 at 8.  (2048 x 509 x 1024 int8 6.3 us against 7.8.)
static bool staged_before_ksplit(const MmArgs& a)
{
    if (a.conv.on || a.bo == SP24_B_KMAJOR) return true;      // the K-splitting kernel does not take them anyway
    if (((a.M + 127) / 128) * ((a.N + 127) / 128) > 64) return true;
    const int64_t steps = a.K * esize_of(a.in) / 128;
    return ((a.M + 31) / 32) * ((a.N + 63) / 64) > 256 && steps <= (a.layout == SP24_LAYOUT_TILED ? 16 : 4);
}

// The kernel for a checked product: few columns or few tiles (K split across wavefronts), streaming (N <= 32), tiled, and for
// operands those cannot fetch the staged and the K-splitting ones; the general kernel takes what is left.
static sp24_status mm_dispatch(const MmArgs& a, hipStream_t st)
{
    bool handled = false;
    sp24_status s;
    const bool tiled_first = a.conv.on || tiled_before_streaming(a);
    if (stream_first(a)) {
        s = launch_mm_stream(a, st, &handled);
        if (handled) return s;
    }
    if (!tiled_first) {
        s = launch_mm_skinny(a, st, &handled);
        if (handled) return s;
    }
    s = launch_conv_narrow(a, st, &handled);
    if (handled) return s;
    s = launch_mm_tiled(a, st, &handled);
    if (handled) return s;
    if (tiled_first && !a.conv.on) {
        s = launch_mm_skinny(a, st, &handled);
        if (handled) return s;
    }
    if (staged_before_ksplit(a)) {
        s = launch_mm_staged(a, st, &handled);
        if (handled) return s;
    }
    s = launch_mm_ksplit(a, st, &handled);
    if (handled) return s;
    return launch_mm_simple(a, st);
}

static sp24_status mm_common(const MmArgs& a, hipStream_t st, size_t x_bytes = 0)
{
    bool empty;
    const sp24_status s = mm_validate(a, x_bytes, &empty);
    if (s != SP24_OK || empty) return s;
    return mm_dispatch(a, st);
}

// K split across workgroups.  The number of slices is a function of the shape and the input type alone: the one
// with the least estimated time among the candidates, where splitting costs 3 us (8 us for the streaming kernel:
// the second kernel and the shorter pipelines) plus the partial images written and read once at 4 TB/s, and must
// win by a tenth.
//  * N > 32 (tiled kernels, 128x128 tiles; rows past M are computed on a valid row and never stored): 1 .. min(8, compute units / tiles, steps / 4) slices of whole
//    128-byte steps; a launch takes 5 us plus 400 ns per step of its workgroups (fitted to measurements of both
//    types at 16 - 128 steps, operands from HBM); the unsplit product it is compared with runs shorter steps when it
//    has at most 128 tiles (smaller ones are taken then).
//  * N <= 32, M >= 32 (streaming kernel, one workgroup per 32 rows): 1 .. min(8, compute units / row blocks,
//    tiles / 32) slices of whole 64-column tiles; a workgroup takes 130 ns (16-bit) or 80 ns (8-bit) per tile of
//    its 32 rows (measured at K = 16384: latency-bound, the same whether 16 or 128 workgroups run).
//  * N <= 32, M < 32: not split (the general kernel).
struct SplitPlan {
    int slices, slice_steps;    // slice_steps in the kernel's own unit: 128-byte steps, or 64-column tiles
    bool streaming;             // the N <= 32 kernel
    int64_t ldw;                // values per row of a partial image
    size_t bytes;               // workspace: slices images of M x ldw accumulator values
};
static SplitPlan split_plan(int64_t M, int64_t N, int64_t K, sp24_dtype in)
{
    SplitPlan p = {1, 0, N <= 32, 0, 0};
    if (N <= 32 && M < 32) return p;
    const int es = esize_of(in);
    const int64_t ldw = (N + 3) / 4 * 4;
    int64_t units, most, unit_ns, base_ns, fixed_ns;         // K in the kernel's units; slices at most; time per unit; per launch; cost of splitting
    if (p.streaming) {
        units = (K + 63) / 64;
        most = 256 / ((M + 31) / 32);
        if (most > units / 32) most = units / 32;
        unit_ns = es == 2 ? 130 : 80;
        base_ns = 0;
        fixed_ns = 8000;
    } else {
        units = K * es / 128;
        most = 256 / (((M + 127) / 128) * ((N + 127) / 128));
        if (most > units / 4) most = units / 4;
        unit_ns = 400;
        base_ns = 5000;
        fixed_ns = 3000;
    }
    if (most > 8) most = 8;
    // The unsplit tiled product on at most 128 tiles runs on smaller ones, with shorter steps: 215 ns where they are 64 columns
    // wide, else 325 ns, which is 64x128 on two wavefronts (both fitted to the sparse products of both types at 64 and 128 steps).
    // Most operands now take 128x64 on four wavefronts, 1.07 - 1.38 times as fast.  From HBM the plan is right all the same
    // (against the unsplit product 1.0 - 3.4 times as fast dense, 1.1 - 4 canonical, 0.93 - 3 in the tiled layout), and
    // callers have been told its workspace; where a sparse operand in the tiled layout is better off unsplit, mm_splitk does not split.
    int64_t unsplit_unit_ns = unit_ns;
    if (!p.streaming && ((M + 127) / 128) * ((N + 127) / 128) <= 128) unsplit_unit_ns = N <= 64 ? 215 : 325;
    int64_t best_ns = (base_ns + units * unsplit_unit_ns) * 9 / 10, best = 1, best_per = units;
    for (int64_t want = 2; want <= most; ++want) {
        const int64_t per = (units + want - 1) / want;
        const int64_t slices = (units + per - 1) / per;      // no slice is empty
        const int64_t ns = base_ns + per * unit_ns + fixed_ns + slices * M * ldw / 500;
        if (ns < best_ns) {
            best_ns = ns;
            best = slices;
            best_per = per;
        }
    }
    if (best <= 1) return p;
    p.slices = (int)best;
    p.slice_steps = (int)best_per;
    p.ldw = ldw;
    p.bytes = (size_t)p.slices * (size_t)M * (size_t)ldw * 4;
    return p;
}

// Address of `scratch` on the current device, looked up once per device (with that device current) and kept.
static sp24_status static_scratch(void** out)
{
    constexpr int kMaxDevices = 64;
    static std::atomic<void*> ptr_of_device[kMaxDevices];
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SP24_ERR_LAUNCH;
    void* p = ptr_of_device[dev].load(std::memory_order_acquire);
    if (!p) {
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return SP24_ERR_LAUNCH;
        ptr_of_device[dev].store(p, std::memory_order_release);   // two first callers store the same address
    }
    *out = p;
    return SP24_OK;
}

// use_static: the partial products go to the library's own scratch array instead of a caller's workspace
static sp24_status mm_splitk(const MmArgs& a, void* workspace, size_t workspace_bytes, hipStream_t st, bool use_static = false)
{
    bool empty;
    sp24_status s = mm_validate(a, 0, &empty);
    if (s != SP24_OK || empty) return s;
    const SplitPlan plan = split_plan(a.M, a.N, a.K, a.in);
    if (plan.slices <= 1) return mm_dispatch(a, st);
    if (use_static) {
        if (plan.bytes > (size_t)SP24_STATIC_SCRATCH_BYTES) return SP24_ERR_WORKSPACE;
        s = static_scratch(&workspace);
        if (s != SP24_OK) return s;
        workspace_bytes = SP24_STATIC_SCRATCH_BYTES;
    }
    if (!workspace) return SP24_ERR_NULL;
    if (!aligned16(workspace)) return SP24_ERR_ALIGN;
    if (workspace_bytes < plan.bytes) return SP24_ERR_SHAPE;
    const int es = esize_of(a.in);
    const size_t nd = ((size_t)(a.M - 1) * a.ldd + a.N) * esize_of(a.out);
    const size_t nb = (a.bo == SP24_B_KMAJOR) ? ((size_t)(a.N - 1) * a.ldb + a.K) * es : ((size_t)(a.K - 1) * a.ldb + a.N) * es;
    const size_t nA = a.sparse ? sp24_values_bytes(a.M, a.K, a.in) : ((size_t)(a.M - 1) * a.lda + a.K) * es;
    if (ranges_overlap(workspace, plan.bytes, a.D, nd) || ranges_overlap(workspace, plan.bytes, a.B, nb) ||
        ranges_overlap(workspace, plan.bytes, a.A, nA))
        return SP24_ERR_SHAPE;
    if (a.sparse && ranges_overlap(workspace, plan.bytes, a.meta, sp24_meta_bytes(a.M, a.K, a.in, a.layout))) return SP24_ERR_SHAPE;
    MmArgs part = a;
    part.D = workspace;
    part.ldd = plan.ldw;
    part.out = (a.in == SP24_I8) ? SP24_I32 : SP24_F32;
    part.k_slices = plan.slices;
    part.slice_steps = plan.slice_steps;
    bool handled = false;
    if (stream_first(a) && (a.bo == SP24_B_KMAJOR || stream_workgroups(a) <= 256)) {
        // The unsplit product has one workgroup on each tile of 32 rows already, which takes 40 ns (N <= 32) or 100 ns per
        // 128-byte step whatever their number; of the plan's slices as many as find a unit of their own and as the
        // images are worth (written and read at 4 TB/s).  Against the plan's slices on the tiled or the streaming kernel:
        // 512 x 16 x 16384 bf16 10.1 -> 9.1 us, 1024 x 128 x 4096 12.5 -> 9.3.
        const int64_t steps = a.K * es / 128, steps_ns = steps * (a.N <= 32 ? 40 : 100), image_ns = a.M * plan.ldw / 500;
        const int most = (int)std::min<int64_t>(plan.slices, 256 / stream_workgroups(a));
        int n = most <= 1 ? 1 : 2;
        for (int x = 3; x <= most; ++x)
            if (steps_ns / x + x * image_ns < steps_ns / n + n * image_ns) n = x;
        // With more than 32 columns the plan's eight slices, which tiles of 128 x 128 leave room for, win where a slice is
        // long.  Measured over 16 - 512 steps a slice, operands from HBM: one slice (an unsplit product) is 3 - 40 % ahead until
        // 80 steps, 9 % behind to 3 % ahead at 96 and 5 - 20 % behind at 128 (8192 x 64 x 8192 bf16 26.8 against 23.5 us); two
        // slices are level until 64 or up to 15 % ahead, at 96 13 % behind to 5 % ahead (4096 x 64 x 12288 24.9 against 21.6), with
        // up to 64 columns 9 - 11 % behind at 80 already; three stay ahead with more than 64 columns (144 - 320 steps a slice: 4 - 18
        // %), with fewer until 80 (2400 x 64 x 15360 21.6 against 22.0, x 18432 24.4 against 23.9, x 24576 29.8 against 27.7); four
        // and more always (256 x 500 x 40960 1.41 times as fast, 128 x 512 2.1 times).
        // Operands in the last-level cache favour the kernel at one and two slices by some 10 % more.  The tiled kernels are slower
        // on a canonical operand: one slice of it is level at 128 steps, and two stay 9 % and more ahead as far as measured
        // (1000 x 200 x 20480 bf16 29.8 against 37.6).  An 8-bit N-major B in two slices of the tiled layout: 48 steps each 3 - 5 % ahead, 64 2 - 5 %
        // behind (1024 x 192 x 16384).
        // Few steps are not worth the second kernel and the images: past 32 columns the unsplit product is ahead up to 40 steps, of a
        // canonical operand up to 32, as long as its few workgroups bring in what HBM would give the split one's many: with fewer than 256 rows on more
        // than 160 columns up to 28 and 22, below 512 rows there, tiled, up to 37.  Times as fast as split, operands in the caches / from HBM (64 -
        // 1024 rows, 40 - 500 columns, three types): tiled up to 26 steps 1.3 - 1.4 / 1.0 - 1.3; 30 - 37 1.2 - 1.4 / 0.95 - 1.3, at 40 1.15 - 1.28 / 0.85 - 1.15
        // (512 x 64 x 2560 bf16 the least), and on the other side of the line 1.2 - 1.35 / 0.81 - 1.0 (64 x 400 x 2560); canonical up to 20 1.3 - 1.4 / 1.0 - 1.2, 30 - 32
        // 1.17 - 1.36 / 0.92 - 1.17, on the other side 1.2 - 1.3 / 0.84 - 1.0.  48 steps are level (tiled 6.9 - 8.6 / 8.3 - 9.3 us unsplit / split, from HBM 8.2 - 11.4 /
        // 9.1 - 10.4).  1000 x 64 x 2048 f16, canonical: 8.3 -> 6.6.  N-major: the line of the tiled kernels below, past which HBM
        // favours the cut (33 steps 1.22 - 1.35 / 0.81 - 1.11, 48 1.02 - 1.22 / 0.63 - 1.0; 8-bit, 32 steps, 1.24 - 1.37 / 0.70 - 1.04).
        const bool canonical = a.layout == SP24_LAYOUT_CANONICAL;
        const bool few_rows = a.N > 160 && a.M < 256, some_rows = a.N > 160 && a.M < 512;
        const int64_t kmajor_line = canonical ? (few_rows ? 22 : 32) : few_rows ? 28 : some_rows ? 37 : 40;
        if (a.N > 32 && steps <= (a.bo == SP24_B_NMAJOR ? (es == 2 ? 32 : 31) : kmajor_line)) n = 1;
        int64_t longest = steps;
        if (a.N > 32 && n <= (a.N <= 64 ? 3 : 2)) {
            if (n == 1) longest = canonical ? 128 : 104;
            else if (canonical) longest = 256;
            else longest = n == 3 ? 96 : a.N <= 64 ? 72 : a.bo == SP24_B_NMAJOR && es == 1 ? 56 : 88;
        }
        if (steps <= longest * n) {
            if (n == 1) return mm_dispatch(a, st);
            part.k_slices = n;
            s = launch_mm_stream(part, st, &handled);
            if (handled && s != SP24_OK) return s;
            if (handled) return launch_splitk_reduce(workspace, part.k_slices, a.M, a.N, plan.ldw, a.D, a.ldd, a.in == SP24_I8, a.out, st);
            part.k_slices = plan.slices;
        }
    } else if (a.sparse && a.layout == SP24_LAYOUT_TILED && a.N > 64 && (es == 2 || a.bo == SP24_B_KMAJOR)) {
        // The tiled layout has the shortest steps unsplit (128x64 tiles on four wavefronts).  The plan's cut against it, time over time
        // from the L2 / the last-level cache / HBM: K-major, both types, 1.5 / 1.37 / 1.04 at 32 steps, 1.4 / 1.17 / 0.9 at 40, 1.3 / 1.13 /
        // 0.85 at 48, 1.16 / 1.06 / 0.79 at 64; in two slices 1.12 / 1.12 / 1.05 at 96, 1.1 / 1.1 / 1.0 at 128, 1.02 / 1.02 / 0.95 at 160.
        // N-major bf16 1.36 / 1.33 / 1.05 at 32 and 1.24 / 1.2 / 0.9 at 40; int8 (tiles of 64x128) 1.29 / 1.11 / 0.82 at 32 already.
        const int64_t steps = a.K * es / 128;
        if (steps <= (a.bo == SP24_B_KMAJOR && plan.slices == 2 ? 128 : 32)) return mm_dispatch(a, st);
    }
    s = plan.streaming ? launch_mm_skinny(part, st, &handled) : launch_mm_tiled(part, st, &handled);
    if (!handled) return mm_dispatch(a, st);             // operands that kernel does not take: not split
    if (s != SP24_OK) return s;
    return launch_splitk_reduce(workspace, plan.slices, a.M, a.N, plan.ldw, a.D, a.ldd, a.in == SP24_I8, a.out, st);
}

size_t sp24_splitk_workspace_bytes(int64_t M, int64_t N, int64_t K, sp24_dtype in)
{
    if (!is_input_type(in) || M <= 0 || N <= 0 || !k_legal(K, in)) return 0;
    return split_plan(M, N, K, in).bytes;
}

sp24_status sp24_spmm_splitk(const void* V, const void* meta, const void* B, void* D, int64_t M, int64_t N, int64_t K, int64_t ldb,
                             int64_t ldd, sp24_dtype in, sp24_dtype out, sp24_border bo, sp24_layout l, void* workspace,
                             size_t workspace_bytes, void* stream)
{
    MmArgs a{V, meta, B, D, M, N, K, 0, ldb, ldd, in, out, bo, l, true};
    return mm_splitk(a, workspace, workspace_bytes, static_cast<hipStream_t>(stream));
}

sp24_status sp24_spmm_splitk_static(const void* V, const void* meta, const void* B, void* D, int64_t M, int64_t N, int64_t K,
                                    int64_t ldb, int64_t ldd, sp24_dtype in, sp24_dtype out, sp24_border bo, sp24_layout l,
                                    void* stream)
{
    MmArgs a{V, meta, B, D, M, N, K, 0, ldb, ldd, in, out, bo, l, true};
    return mm_splitk(a, nullptr, 0, static_cast<hipStream_t>(stream), true);
}

sp24_status sp24_gemm_dense_splitk(const void* A, const void* B, void* D, int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb,
                                   int64_t ldd, sp24_dtype in, sp24_dtype out, sp24_border bo, void* workspace,
                                   size_t workspace_bytes, void* stream)
{
    MmArgs a{A, nullptr, B, D, M, N, K, lda, ldb, ldd, in, out, bo, SP24_LAYOUT_CANONICAL, false};
    return mm_splitk(a, workspace, workspace_bytes, static_cast<hipStream_t>(stream));
}

sp24_status sp24_spmm(const void* V, const void* meta, const void* B, void* D, int64_t M, int64_t N, int64_t K, int64_t ldb,
                      int64_t ldd, sp24_dtype in, sp24_dtype out, sp24_border bo, sp24_layout l, void* stream)
{
    MmArgs a{V, meta, B, D, M, N, K, 0, ldb, ldd, in, out, bo, l, true};
    return mm_common(a, static_cast<hipStream_t>(stream));
}

sp24_status sp24_gemm_dense(const void* A, const void* B, void* D, int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb,
                            int64_t ldd, sp24_dtype in, sp24_dtype out, sp24_border bo, void* stream)
{
    MmArgs a{A, nullptr, B, D, M, N, K, lda, ldb, ldd, in, out, bo, SP24_LAYOUT_CANONICAL, false};
    return mm_common(a, static_cast<hipStream_t>(stream));
}

sp24_status sp24_spmm_i8_scaled(const void* V, const void* meta, const void* B, void* D, int64_t M, int64_t N, int64_t K,
                                int64_t ldb, int64_t ldd, const float* w_scale, float x_scale, const float* bias, int relu,
                                float inv_y_scale, sp24_dtype out, sp24_border bo, sp24_layout l, void* stream)
{
    MmArgs a{V, meta, B, D, M, N, K, 0, ldb, ldd, SP24_I8, out, bo, l, true};
    a.epi = Epilogue{w_scale, bias, x_scale, inv_y_scale, relu != 0, 1};
    return mm_common(a, static_cast<hipStream_t>(stream));
}

sp24_status sp24_gemm_dense_i8_scaled(const void* A, const void* B, void* D, int64_t M, int64_t N, int64_t K, int64_t lda,
                                      int64_t ldb, int64_t ldd, const float* w_scale, float x_scale, const float* bias, int relu,
                                      float inv_y_scale, sp24_dtype out, sp24_border bo, void* stream)
{
    MmArgs a{A, nullptr, B, D, M, N, K, lda, ldb, ldd, SP24_I8, out, bo, SP24_LAYOUT_CANONICAL, false};
    a.epi = Epilogue{w_scale, bias, x_scale, inv_y_scale, relu != 0, 1};
    return mm_common(a, static_cast<hipStream_t>(stream));
}

// Shared front end of the two convolution entry points: geometry checks, then the product path with B = X.
static sp24_status conv_common(MmArgs& a, int64_t n_img, int64_t H, int64_t W, int64_t C, int R, int S, int pad_h, int pad_w,
                               int stride_h, int stride_w, hipStream_t st)
{
    if (!is_input_type(a.in) || !out_legal(a.in, a.out, a.epi.on != 0)) return SP24_ERR_DTYPE;
    const int64_t lim = (int64_t)1 << 20;
    if (a.M < 0 || n_img < 0 || H < 1 || W < 1 || C < 1 || R < 1 || S < 1 || pad_h < 0 || pad_w < 0 || stride_h < 1 || stride_w < 1 ||
        H > lim || W > lim || C > lim || R > 4096 || S > 4096 || pad_h > 4096 || pad_w > 4096 || stride_h > 4096 || stride_w > 4096 ||
        H + 2 * pad_h < R || W + 2 * pad_w < S)
        return SP24_ERR_SHAPE;
    const int es = esize_of(a.in);
    if ((C * es) % 16 != 0) return SP24_ERR_SHAPE;      // 16 consecutive bytes of K never straddle a filter tap
    const int64_t OH = (H + 2 * pad_h - R) / stride_h + 1, OW = (W + 2 * pad_w - S) / stride_w + 1;
    const int64_t K = (int64_t)R * S * C;
    if (K > ((int64_t)1 << 30) || (n_img > 0 && OH * OW > (((int64_t)1 << 31) - 1) / n_img)) return SP24_ERR_SHAPE;
    if (n_img > 0 && H * W * C > (((int64_t)1 << 46) / n_img)) return SP24_ERR_SHAPE;
    a.N = n_img * OH * OW;
    a.K = K;
    a.bo = SP24_B_KMAJOR;
    a.ldb = K;
    if (R == 1 && S == 1 && pad_h == 0 && pad_w == 0 && stride_h == 1 && stride_w == 1) {
        // a pointwise convolution is the plain product with the NHWC input as the K-major second operand, one row
        // per pixel: it takes the product kernels as they are (the streaming one for few pixels included)
        a.conv = ConvGeom{};
        a.ldb = C;
        return mm_common(a, st);
    }
    a.conv = ConvGeom{1, (int)H, (int)W, (int)C, R, S, pad_h, pad_w, stride_h, stride_w, (int)OH, (int)OW};
    return mm_common(a, st, (size_t)n_img * H * W * C * es);
}

sp24_status sp24_spmm_conv2d(const void* V, const void* meta, const void* X, void* D, int64_t M, int64_t n_img, int64_t H,
                             int64_t W, int64_t C, int R, int S, int pad_h, int pad_w, int stride_h, int stride_w, int64_t ldd,
                             sp24_dtype in, sp24_dtype out, sp24_layout l, void* stream)
{
    MmArgs a{V, meta, X, D, M, 0, 0, 0, 0, ldd, in, out, SP24_B_KMAJOR, l, true};
    return conv_common(a, n_img, H, W, C, R, S, pad_h, pad_w, stride_h, stride_w, static_cast<hipStream_t>(stream));
}

sp24_status sp24_conv2d_dense(const void* A, const void* X, void* D, int64_t M, int64_t n_img, int64_t H, int64_t W, int64_t C,
                              int R, int S, int pad_h, int pad_w, int stride_h, int stride_w, int64_t lda, int64_t ldd,
                              sp24_dtype in, sp24_dtype out, void* stream)
{
    MmArgs a{A, nullptr, X, D, M, 0, 0, lda, 0, ldd, in, out, SP24_B_KMAJOR, SP24_LAYOUT_CANONICAL, false};
    return conv_common(a, n_img, H, W, C, R, S, pad_h, pad_w, stride_h, stride_w, static_cast<hipStream_t>(stream));
}

sp24_status sp24_spmm_conv2d_i8_scaled(const void* V, const void* meta, const void* X, void* D, int64_t M, int64_t n_img,
                                       int64_t H, int64_t W, int64_t C, int R, int S, int pad_h, int pad_w, int stride_h,
                                       int stride_w, int64_t ldd, const float* w_scale, float x_scale, const float* bias,
                                       int relu, float inv_y_scale, sp24_dtype out, sp24_layout l, void* stream)
{
    MmArgs a{V, meta, X, D, M, 0, 0, 0, 0, ldd, SP24_I8, out, SP24_B_KMAJOR, l, true};
    a.epi = Epilogue{w_scale, bias, x_scale, inv_y_scale, relu != 0, 1};
    return conv_common(a, n_img, H, W, C, R, S, pad_h, pad_w, stride_h, stride_w, static_cast<hipStream_t>(stream));
}

sp24_status sp24_conv2d_dense_i8_scaled(const void* A, const void* X, void* D, int64_t M, int64_t n_img, int64_t H, int64_t W,
                                        int64_t C, int R, int S, int pad_h, int pad_w, int stride_h, int stride_w, int64_t lda,
                                        int64_t ldd, const float* w_scale, float x_scale, const float* bias, int relu,
                                        float inv_y_scale, sp24_dtype out, void* stream)
{
    MmArgs a{A, nullptr, X, D, M, 0, 0, lda, 0, ldd, SP24_I8, out, SP24_B_KMAJOR, SP24_LAYOUT_CANONICAL, false};
    a.epi = Epilogue{w_scale, bias, x_scale, inv_y_scale, relu != 0, 1};
    return conv_common(a, n_img, H, W, C, R, S, pad_h, pad_w, stride_h, stride_w, static_cast<hipStream_t>(stream));
}

const char* sp24_status_string(sp24_status s)
{
    switch (s) {
    case SP24_OK: return "ok";
    case SP24_ERR_NULL: return "a required pointer is NULL";
    case SP24_ERR_SHAPE: return "illegal shape, leading dimension or overlapping buffers";
    case SP24_ERR_ALIGN: return "pointer or leading dimension not 16-byte aligned";
    case SP24_ERR_DTYPE: return "unknown or unsupported element type";
    case SP24_ERR_LAYOUT: return "unknown layout or shape not legal for the layout";
    case SP24_ERR_LAUNCH: return "HIP launch failed";
    case SP24_ERR_WORKSPACE: return "the shape needs more scratch memory than the library's static buffer holds";
    }
    return "unknown status";
}

} // extern "C"
