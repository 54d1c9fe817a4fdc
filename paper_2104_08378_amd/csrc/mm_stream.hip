// Sparse products with few columns (N <= 32) or few tiles: the decode-like shapes, bound by how fast a compute unit can
// bring its operands in.
//
// One workgroup per 32 rows and BR (16, 32 or 64) columns of D; its wavefronts split K among themselves (128-byte step s
// goes to wavefront s % NW, so that the workgroup reads A front to back).  Every wavefront has an LDS ring of its
// own, filled by direct transfers NS - 1 steps ahead: it awaits its own transfers and never a barrier.  The NW
// partial tiles are added through LDS, always in the same order.
//
// Why through LDS: the matrix instruction wants 16 bytes of each of 32 rows of B per half wavefront, and a load of that
// shape touches 32 cache lines for 1 KiB -- the address path, not the memory, then sets the pace.  A transfer has
// eight lanes to a row (a whole line), and for a canonical A four lanes to a row's 64 bytes of a step.
// 8192 x 64 x 8192 bf16: 76.5 MB of operands in 27.8 us from HBM (2.8 TB/s), in 18.4 us where they are still in the last-level
// cache (4.2 TB/s); every workgroup reads all of B besides, 268 MB from the L2, so that a unit brings in 48 and 73 GB/s.
// 8192 x 16 x 8192: 76 MB in 16.4 us from HBM (4.6 TB/s).  Measured and not kept: the compressed operand marked as passing once (nt), which
// helps loads into registers, costs these transfers 10 - 60 % (512 x 16 x 16384: 13.2 -> 21.2 us).
//
// NMAJ: B N-major, rows of whole 16-byte chunks: a transfer takes the tile's columns of as many K rows as 1 KiB holds, and fragments
// come through the transposing LDS reads of the tiled kernels.  Those had these products on 32 x 64 to 128 x 64 tiles before, a step
// behind a barrier each and fewer than half of the units at work: 1024 x 512 x 4096 bf16 15.4 -> 11.7 us, int8 11.2 -> 9.4, 1024 x 16 x 8192
// bf16 20.0 -> 7.8 (K-major 6.8), 512 x 128 x 8192 from HBM 37.4 -> 21.0.
#include "mm_operands.hpp"

namespace sp24 {

namespace {

// f(integral_constant<int, D>{}) for D, D - 1, ..., 0
template <int D, class F>
__device__ __forceinline__ void count_down(F&& f)
{
    if constexpr (D >= 0) {
        f(std::integral_constant<int, D>{});
        count_down<D - 1>(f);
    }
}

} // namespace

template <int DT, int BR, int NW, int NS, bool NMAJ>
__global__ __launch_bounds__(64 * NW) void k_spmm_stream(MmArgs a, int tiles_m, int tiles_n)
{
    constexpr int ES = is8<DT> ? 1 : 2;
    constexpr int T64 = is8<DT> ? 2 : 1;              // 64-column tiles of A per step
    constexpr int TN = BR == 64 ? 2 : 1;
    constexpr int NB = BR / 8, NV = NB + 2 + T64;     // transfers of a step: B (8 rows each), values (2 x 1 KiB), codes (256 B each)
    constexpr int kVOff = BR * kRowBytes, kMOff = kVOff + 2048, kStage = kMOff + T64 * 256;
    constexpr int kRing = NW * NS * kStage, kRed = NW * TN * 16 * 64 * 4;
    static_assert(kRing <= 160 * 1024 && (NS - 2) * NV <= 63, "LDS of a compute unit; vmcnt is a 6-bit counter");
    using acc_t = typename acc_of<DT>::type;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[kRing > kRed ? kRing : kRed];

    int tm, tn;
    tile_of_workgroup(tiles_m, tiles_n, tm, tn);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 31, q = lane >> 5;
    // this workgroup's share of K in whole steps, and the bytes of a partial step after them (0: none)
    int first = 0, end = (int)(a.K / (kRowBytes / ES)), tail = (int)((a.K * ES) % kRowBytes);
    if (a.k_slices > 1) {
        const int per = (end + a.k_slices - 1) / a.k_slices;
        first = min((int)blockIdx.y * per, end);
        if ((int)blockIdx.y < a.k_slices - 1) {
            end = min(first + per, end);
            tail = 0;
        }
        a.D = reinterpret_cast<uint8_t*>(a.D) + (int64_t)blockIdx.y * a.M * a.ldd * 4;
    }

    // ---- transfers: base address of the tile (the same in all lanes), the lane's offset ----
    const int64_t ldb = a.ldb * ES, n0 = (int64_t)tn * BR;
    const uint8_t* const b_base = reinterpret_cast<const uint8_t*>(a.B) + (NMAJ ? n0 * ES : n0 * ldb);
    const int64_t b_step = NMAJ ? (kRowBytes / ES) * ldb : (int64_t)kRowBytes;
    uint32_t b_off[NB];
    if constexpr (NMAJ) dma_offsets_nmajor<BR, 1, ES>(n0, a.N, ldb, 0, lane, b_off);
    else dma_offsets<BR, 1>(n0, a.N, ldb, 0, lane, b_off);
    const bool canonical = a.layout == SP24_LAYOUT_CANONICAL;
    const int64_t vrow = a.K / 2 * ES, mrow = a.K / 8, KB64 = a.K / 64;
    const uint8_t* v_base = reinterpret_cast<const uint8_t*>(a.A) + (canonical ? (int64_t)tm * 32 * vrow : tm * KB64 * (1024 * ES));
    const uint8_t* m_base = reinterpret_cast<const uint8_t*>(a.meta) + (canonical ? (int64_t)tm * 32 * mrow : tm * KB64 * 256);
    const int v_step = canonical ? 64 : 2048, m_step = canonical ? 8 * T64 : 256 * T64;
    uint32_t v_off[2], m_off[T64];
    int v_piece[2];                                   // canonical: 16-byte piece of the row's 64 bytes of values
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        const int row = x * 16 + (lane >> 2);
        v_piece[x] = canonical_piece(row, lane & 3);
        const int64_t rows_left = a.M - 1 - (int64_t)tm * 32;       // ragged M: a valid row, never stored
        v_off[x] = canonical ? (uint32_t)(min((int64_t)row, rows_left) * vrow) + v_piece[x] * 16 : x * 1024 + lane * 16;
    }
#pragma unroll
    for (int t = 0; t < T64; ++t) {
        const int64_t rows_left = a.M - 1 - (int64_t)tm * 32;
        m_off[t] = canonical ? (uint32_t)(min((int64_t)(t * 16 + lane / (2 * T64)), rows_left) * mrow) + (lane % (2 * T64)) * 4 : t * 256 + lane * 4;
    }
    uint8_t* const ring = lds + wave * (NS * kStage);
    auto fetch = [&](int step, int u) {
        uint8_t* const stage = ring + u * kStage;
#pragma unroll
        for (int x = 0; x < 2; ++x) lds_dma16(v_base + (int64_t)step * v_step, v_off[x], stage + kVOff + x * 1024);
#pragma unroll
        for (int t = 0; t < T64; ++t) lds_dma4(m_base + (int64_t)step * m_step, m_off[t], stage + kMOff + t * 256);
#pragma unroll
        for (int j = 0; j < NB; ++j) lds_dma16(b_base + step * b_step, b_off[j], stage + j * 1024);
    };
    // the partial step: what lies past K comes from the row of zeros
    auto fetch_tail = [&](int step) {
#pragma unroll
        for (int x = 0; x < 2; ++x)
            lds_dma_tail<false>(v_base + (int64_t)step * v_step, v_off[x], canonical ? v_piece[x] * 16 >= tail / 2 : ES == 1 && 64 * x >= tail,
                                ring + kVOff + x * 1024);
#pragma unroll
        for (int t = 0; t < T64; ++t)
            lds_dma_tail<true>(m_base + (int64_t)step * m_step, m_off[t], (canonical ? (lane % (2 * T64)) * 32 * ES : 64 * ES * t) >= tail,
                               ring + kMOff + t * 256);
#pragma unroll
        for (int j = 0; j < NB; ++j)
            lds_dma_tail<false>(b_base + step * b_step, b_off[j],
                                NMAJ ? past_k_nmajor<BR, 1, ES>(j, 0, lane, tail) : past_k_kmajor<BR, 1>(j, 0, lane, tail), ring + j * 1024);
    };

    // ---- operand reads: values of instruction j, and the two pieces of B (as in the tiled kernels) ----
    int a_off[2], frag_off[4];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int piece = is8<DT> ? 2 * j + q : 2 * q + j;
        a_off[j] = kVOff + (canonical ? r * 64 + canonical_piece(r, piece) * 16 : j * 1024 + lane * 16);
    }
    int m_read[T64];
#pragma unroll
    for (int t = 0; t < T64; ++t) m_read[t] = kMOff + (canonical ? r * (8 * T64) + (2 * t + q) * 4 : t * 256 + lane * 4);
    const int br = BR == 16 ? r & 15 : r;             // 16 columns: the upper half computes them again, never stored
#pragma unroll
    for (int c2 = 0; c2 < 4; ++c2) frag_off[c2] = br * kRowBytes + ((((2 * c2) | q) ^ ((br >> 1) & 7)) << 4);
    nmajor_frags<BR, TN, ES> b_nm;
    if constexpr (NMAJ) b_nm.init(0, BR == 16 ? lane & ~16 : lane);

    // 16-bit floats: two sums of each element, one per half of a step, added at the end, which leaves half the roundings in each (with the sums
    // in pairs below, 1000 x 64 x 2048 f16: relative error 9.7e-8 -> 8.0e-8, split in four slices 8.1e-8; up to 0.1 us).  8-bit floats, whose error is
    // what the instruction drops, have the same with one (5.7e-6 on normal values, 5.3e-5 on every bit pattern, 512 - 16384 columns of A), and
    // lose by the second: 288 x 316 x 1472, canonical, from HBM 5.5 -> 6.0 us, 634 x 52 x 3168 9.2 -> 9.9.
    constexpr bool kTwo = !is8<DT>;
    acc_t acc[TN], acc_second[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[j] = acc_second[j] = acc_t{};
    auto compute = [&](const uint8_t* stage) {
        int4v va[2];
        int code[T64];
        uint4v lo[2][TN], hi[2][TN];
#pragma unroll
        for (int j = 0; j < 2; ++j) va[j] = *reinterpret_cast<const int4v*>(stage + a_off[j]);
#pragma unroll
        for (int t = 0; t < T64; ++t) code[t] = *reinterpret_cast<const int*>(stage + m_read[t]);
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int nj = 0; nj < TN; ++nj) {
                const int c2lo = is8<DT> ? 2 * j : j, c2hi = is8<DT> ? 2 * j + 1 : 2 + j;
                if constexpr (NMAJ) {
                    lo[j][nj] = b_nm.piece(stage, c2lo, nj);
                    hi[j][nj] = b_nm.piece(stage, c2hi, nj);
                } else {
                    lo[j][nj] = *reinterpret_cast<const uint4v*>(stage + frag_off[c2lo] + nj * 32 * kRowBytes);
                    hi[j][nj] = *reinterpret_cast<const uint4v*>(stage + frag_off[c2hi] + nj * 32 * kRowBytes);
                }
            }
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int nj = 0; nj < TN; ++nj) {
                int8v f;
                f[0] = lo[j][nj][0]; f[1] = lo[j][nj][1]; f[2] = lo[j][nj][2]; f[3] = lo[j][nj][3];
                f[4] = hi[j][nj][0]; f[5] = hi[j][nj][1]; f[6] = hi[j][nj][2]; f[7] = hi[j][nj][3];
                if constexpr (is8<DT>) acc[nj] = smfmac32<DT, 0>(va[j], f, acc[nj], code[j]);
                else if (j == 0) acc[nj] = smfmac32<DT, 0>(va[0], f, acc[nj], code[0]);
                else acc_second[nj] = smfmac32<DT, 1>(va[1], f, acc_second[nj], code[0]);
            }
    };

    // This wavefront's steps first + wave, + NW, ...  A step is fetched into the stage whose reads have returned one
    // step earlier; the last NS - 1 have nothing to fetch and wait for what is left.
    const int mine = first + wave < end ? (end - first - wave + NW - 1) / NW : 0;
    const int ahead = min(mine, NS - 1);
    int next = first + wave;
    for (int u = 0; u < ahead; ++u, next += NW) fetch(next, u);
    int u = 0;
    auto consume = [&]() {
        compute(ring + u * kStage);
        u = u + 1 == NS ? 0 : u + 1;
    };
    int into = NS - 1;
    for (int i = NS - 1; i < mine; ++i, next += NW) {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(waitcnt_vm((NS - 2) * NV) & ~(15 << 8));       // the oldest step has landed; the reads of the one before have returned
        __builtin_amdgcn_sched_barrier(0);
        fetch(next, into);
        consume();
        into = into + 1 == NS ? 0 : into + 1;
    }
    count_down<NS - 2>([&](auto d_c) {
        constexpr int d = decltype(d_c)::value;              // steps fetched after this one
        if (ahead > d) {
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt(waitcnt_vm(d * NV));
            __builtin_amdgcn_sched_barrier(0);
            consume();
        }
    });
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0) & ~(15 << 8));                       // the last reads have returned
    __builtin_amdgcn_sched_barrier(0);
    if (tail != 0 && wave == (end - first) % NW) {
        fetch_tail(end);
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
        __builtin_amdgcn_sched_barrier(0);
        compute(ring);
    }

    // the partial tiles, added in pairs, pairs of pairs and so on in wavefront order (fewer roundings on the way of each)
    uint32_t (*red)[TN * 16][64] = reinterpret_cast<uint32_t (*)[TN * 16][64]>(lds);
    __syncthreads();                                  // the rings are done with
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            auto v = kTwo ? acc[j][e] + acc_second[j][e] : acc[j][e];
            red[wave][j * 16 + e][lane] = __builtin_bit_cast(uint32_t, v);
        }
    __syncthreads();
    for (int id = wave; id < TN * 16; id += NW) {
        const int j = id >> 4, e = id & 15;
        using val_t = typename std::conditional<DT == SP24_I8, int, float>::type;
        val_t part[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w) part[w] = __builtin_bit_cast(val_t, red[w][id][lane]);
#pragma unroll
        for (int d = 1; d < NW; d *= 2)
#pragma unroll
            for (int w = 0; w + d < NW; w += 2 * d) part[w] += part[w + d];
        const val_t sum = part[0];
        const int64_t m = (int64_t)tm * 32 + 8 * (e / 4) + 4 * q + (e % 4), n = n0 + j * 32 + r;
        if (m < a.M && n < a.N && j * 32 + r < BR) put<DT>(a, m, n, sum);
    }
}

template <int DT, bool NMAJ>
static sp24_status run_stream(const MmArgs& a, hipStream_t st)
{
    const int br = stream_columns(a);
    auto run = [&](auto kernel, int nw) {
        const int tiles_m = (int)((a.M + 31) / 32), tiles_n = (int)((a.N + br - 1) / br);
        kernel<<<dim3((unsigned)(tiles_m * tiles_n), (unsigned)(a.k_slices > 1 ? a.k_slices : 1)), dim3(64 * nw), 0, st>>>(a, tiles_m, tiles_n);
        return hipGetLastError() == hipSuccess ? SP24_OK : SP24_ERR_LAUNCH;
    };
    // As many wavefronts as the LDS holds with two or more stages each.  Eight of 4 (N <= 16) and 3 stages (N <= 32) are
    // ahead of 16 x 2, 10 x 3, 12 x 2, 6 x 4 and 4 x 8 by 1 - 20 %; for 64 columns 7 x 2 of 5 x 3, 4 x 3 and 3 x 5 by 1 - 15 %
    if (br == 16) return run(k_spmm_stream<DT, 16, 8, 4, NMAJ>, 8);
    if (br == 32) return run(k_spmm_stream<DT, 32, 8, 3, NMAJ>, 8);
    return run(k_spmm_stream<DT, 64, 7, 2, NMAJ>, 7);
}

sp24_status launch_mm_stream(const MmArgs& a, hipStream_t st, bool* handled)
{
    *handled = false;
    const int es = esize_of(a.in);
    const bool nmajor = a.bo == SP24_B_NMAJOR;
    bool ok = a.sparse && !a.conv.on && (reinterpret_cast<uintptr_t>(a.B) & 15u) == 0 && (a.ldb * es) % 16 == 0 && (!nmajor || a.N * es % 16 == 0) &&
              a.M <= ((int64_t)1 << 30) && a.N <= ((int64_t)1 << 30) && ((a.M + 31) / 32) * ((a.N + 15) / 16) < ((int64_t)1 << 30) &&
              a.K <= ((int64_t)1 << 24);                   // 32-bit offsets inside a tile: 64 rows of B (N-major: up to 128), 32 rows of values
    ok = ok && a.ldb * es < (nmajor ? (int64_t)1 << 24 : (int64_t)1 << 25);
    if (a.layout == SP24_LAYOUT_CANONICAL) ok = ok && a.K % 32 == 0;      // codes as 4-byte words
    if (!ok) return SP24_OK;
    *handled = true;
    auto run = [&](auto dt) {
        constexpr int DT = decltype(dt)::value;
        return nmajor ? run_stream<DT, true>(a, st) : run_stream<DT, false>(a, st);
    };
    if (a.in == SP24_I8) return run(std::integral_constant<int, SP24_I8>{});
    if (a.in == SP24_F8) return run(std::integral_constant<int, SP24_F8>{});
    if (a.in == SP24_F16) return run(std::integral_constant<int, SP24_F16>{});
    return run(std::integral_constant<int, SP24_BF16>{});
}

} // namespace sp24
