// Operands brought into registers, for the kernels whose operands the LDS transfers of the tiled kernels cannot take:
// an N-major B with rows at any address, a compressed first operand in either layout and with any legal K.
#pragma once
#include "mm_tiled.hpp"

namespace sp24 {

// A value of global memory at any address.  (An address chosen between an operand and the row of zeros no longer shows
// the compiler that it is global, and a flat load would be waited for with the LDS accesses.)
template <typename T>
__device__ __forceinline__ T load_any(const uint8_t* p)
{
    struct __attribute__((packed, aligned(1))) any_t { T v; };
    return reinterpret_cast<const __attribute__((address_space(1))) any_t*>(reinterpret_cast<uintptr_t>(p))->v;
}
// the same from an address that is a multiple of 16
__device__ __forceinline__ uint4v load16_aligned(const uint8_t* p)
{
    return *reinterpret_cast<const __attribute__((address_space(1))) uint4v*>(reinterpret_cast<uintptr_t>(p));
}
// 16 bytes from any address (one dwordx4 load)
__device__ __forceinline__ uint4v load16_any(const uint8_t* p) { return load_any<uint4v>(p); }

// The value's bytes moved down by `bytes` (0 .. 15), zeros on top.  Not as a 128-bit shift: its 64-bit shifts, with the
// amount in the last vector register of the kernel's allocation, were seen to take the amount from register 0 now and
// then (int8 1999 x 2177 x 416, N-major: tiles with the last rows' upper halves shifted by the lane's number).
__device__ __forceinline__ uint4v shift_down(uint4v v, int bytes)
{
    if (bytes & 4) v = uint4v{v[1], v[2], v[3], 0u};
    if (bytes & 8) v = uint4v{v[2], v[3], 0u, 0u};
    const uint32_t n = bytes & 3;
    return uint4v{__builtin_amdgcn_alignbyte(v[1], v[0], n), __builtin_amdgcn_alignbyte(v[2], v[1], n), __builtin_amdgcn_alignbyte(v[3], v[2], n),
                  __builtin_amdgcn_alignbyte(0u, v[3], n)};
}

// result element (m, n) from the accumulated value
template <int DT, typename ACC>
__device__ __forceinline__ void put(const MmArgs& a, int64_t m, int64_t n, ACC v)
{
    const int64_t at = m * a.ldd + n;
    if constexpr (DT == SP24_I8) {
        float s = 0.0f, b = 0.0f;
        if (a.out != SP24_I32) epilogue_row(a.epi, m, s, b);
        if (a.out == SP24_I32) store_bits<SP24_I32>(a.D, at, (uint32_t)v);
        else if (a.out == SP24_I8) store_bits<SP24_I8>(a.D, at, output_bits<SP24_I8>(v, s, b, a.epi));
        else if (a.out == SP24_F32) store_bits<SP24_F32>(a.D, at, output_bits<SP24_F32>(v, s, b, a.epi));
        else if (a.out == SP24_F16) store_bits<SP24_F16>(a.D, at, output_bits<SP24_F16>(v, s, b, a.epi));
        else store_bits<SP24_BF16>(a.D, at, output_bits<SP24_BF16>(v, s, b, a.epi));
    } else {
        if (a.out == SP24_F32) store_out<SP24_F32>(a.D, at, v);
        else if (a.out == SP24_F16) store_out<SP24_F16>(a.D, at, v);
        else store_out<SP24_BF16>(a.D, at, v);
    }
}

// The pieces (16 bytes) of ROWS K rows x BN columns of an N-major B that one of NT threads carries into an LDS image
// of the layout that nmajor_frags reads: rows row0, row0 + kRowsPerPiece, ..., chunk c of each.
template <int BN, int ES, int ROWS, int NT>
struct nmajor_pieces {
    static constexpr int kRowB = BN * ES, kChunks = kRowB / 16;
    static constexpr int NJ = ROWS * kChunks / NT;
    static constexpr int kRowsPerPiece = NT / kChunks;
    static_assert(ROWS * kChunks % NT == 0 && kRowsPerPiece % 8 == 0, "the swizzle is the same for all of a thread's pieces");
    const uint8_t* B;
    int64_t K, ldb, b_bytes, src0, reach;                     // ldb in bytes; from B to its last element's end
    int row0, dst0;
    __device__ __forceinline__ void init(const MmArgs& a, int64_t tn, int id)
    {
        B = reinterpret_cast<const uint8_t*>(a.B);
        K = a.K;
        ldb = a.ldb * ES;
        const int64_t col0 = tn * BN * ES;
        b_bytes = (K - 1) * ldb + a.N * ES;
        row0 = id / kChunks;
        const int c = id % kChunks;
        const int valid = (int)min((int64_t)kChunks, (a.N * ES - col0 + 15) / 16);   // chunks that hold columns of the matrix
        src0 = col0 + min(c, valid - 1) * 16;                 // byte of a row; past the last chunk: never stored
        reach = (ROWS - 1) * ldb + col0 + (valid - 1) * 16 + 16;   // end of the last piece, from the first row
        dst0 = row0 * kRowB + ((c ^ nmajor_swizzle<ES>(row0, kChunks)) << 4);
    }
    // groups of ROWS K rows, from the first on, all of whose pieces lie inside B
    __device__ __forceinline__ int64_t whole_groups() const
    {
        return b_bytes < reach ? 0 : min(K / ROWS, (b_bytes - reach) / (ROWS * ldb) + 1);
    }
    // such a group.  (A kernel keeps the loads of several groups in flight, and only a loop without branches lets the
    // compiler count them: the groups past these are a phase of their own.)
    __device__ __forceinline__ void load_whole(int64_t group, uint4v (&v)[NJ]) const
    {
        const uint8_t* p = B + group * ROWS * ldb + row0 * ldb + src0;
#pragma unroll
        for (int j = 0; j < NJ; ++j) v[j] = load16_any(p + j * kRowsPerPiece * ldb);
    }
    // the last rows: pieces that would end past the last element are read up to it and moved into place (B has 32
    // bytes at least), rows past K are zeros
    __device__ __forceinline__ void load_edge(int64_t group, uint4v (&v)[NJ]) const
    {
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int64_t k = group * ROWS + row0 + j * kRowsPerPiece;
            const int64_t at = min(k, K - 1) * ldb + src0;
            const int64_t over = max((int64_t)0, at + 16 - b_bytes);
            const uint4v x = shift_down(load16_any(B + at - over), (int)over);
            v[j] = k < K ? x : uint4v{0u, 0u, 0u, 0u};
        }
    }
    __device__ __forceinline__ void store(uint8_t* image, const uint4v (&v)[NJ]) const
    {
#pragma unroll
        for (int j = 0; j < NJ; ++j) *reinterpret_cast<uint4v*>(image + dst0 + j * kRowsPerPiece * kRowB) = v[j];
    }
};

// The compressed first operand of TM blocks of 32 rows, straight from memory in the matrix instruction's lane order:
// per 64-column tile one (8-bit) or two (16-bit) 16-byte pieces and one word of codes per lane.  Rows past M are a
// valid row (never stored), columns past K are zeros.
template <int DT, int TM>
struct compressed_rows {
    static constexpr int ES = is8<DT> ? 1 : 2;
    static constexpr int NA = ES;
    const uint8_t* v_src[TM];
    const uint8_t* m_src[TM];
    int64_t K;
    int v_step, m_step, piece_step;                            // bytes per 64-column tile; from a lane's piece of a tile to its next
    int q;
    // block0: the first row block
    __device__ __forceinline__ void init(const MmArgs& a, int64_t block0, int lane)
    {
        K = a.K;
        q = lane >> 5;
        const bool canonical = a.layout == SP24_LAYOUT_CANONICAL;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            if (canonical) {
                const int64_t m = min((block0 + i) * 32 + (lane & 31), a.M - 1);
                v_src[i] = reinterpret_cast<const uint8_t*>(a.A) + m * (K / 2 * ES) + 16 * ES * q;
                m_src[i] = reinterpret_cast<const uint8_t*>(a.meta) + m * (K / 8) + 4 * q;
            } else {
                const int64_t rb = min(block0 + i, a.M / 32 - 1);
                v_src[i] = reinterpret_cast<const uint8_t*>(a.A) + rb * (K / 64) * (1024 * ES) + lane * 16;
                m_src[i] = reinterpret_cast<const uint8_t*>(a.meta) + rb * (K / 64) * 256 + lane * 4;
            }
        }
        v_step = canonical ? 32 * ES : 1024 * ES;
        m_step = canonical ? 8 : 256;
        piece_step = canonical ? 16 : 1024;
    }
    // 64-column tile kb, all of it before K
    __device__ __forceinline__ void load_whole(int64_t kb, int4v (&v)[TM][NA], uint32_t (&code)[TM]) const
    {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
#pragma unroll
            for (int s = 0; s < NA; ++s) v[i][s] = __builtin_bit_cast(int4v, load16_aligned(v_src[i] + kb * v_step + s * piece_step));
            code[i] = load_any<uint32_t>(m_src[i] + kb * m_step);
        }
    }
    // any tile: what lies past K comes from a row of zeros (K may end in the middle of a word of codes)
    __device__ __forceinline__ void load_edge(int64_t kb, int4v (&v)[TM][NA], uint32_t (&code)[TM]) const
    {
        const int left = (int)min(max(K - kb * 64, (int64_t)0), (int64_t)64);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
#pragma unroll
            for (int s = 0; s < NA; ++s) {                      // a piece is all before K or all past it
                const uint8_t* p = v_src[i] + kb * v_step + s * piece_step;
                v[i][s] = __builtin_bit_cast(int4v, load16_aligned(32 * q + 16 * s < left ? p : k_zero_row));
            }
            const uint8_t* p = m_src[i] + kb * m_step;
            const uint16_t lo = load_any<uint16_t>(32 * q < left ? p : k_zero_row);          // the codes of 16 columns each
            const uint16_t hi = load_any<uint16_t>(32 * q + 16 < left ? p + 2 : k_zero_row);
            code[i] = lo | (uint32_t)hi << 16;
        }
    }
};

} // namespace sp24
