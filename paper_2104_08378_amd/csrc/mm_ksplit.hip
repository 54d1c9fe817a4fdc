// Products with an N-major B whose rows start at any address (an odd number of columns, or a view with an odd
// pitch): the activations that a previous product left as [features, tokens] for a prompt of arbitrary length.
// The tiled kernels' transfers go straight from memory to LDS and need 16-byte aligned rows; here B passes through
// registers, loaded 16 bytes per lane from wherever the row starts, and is written to LDS aligned.
//
// One workgroup per 32 x 64 or 64 x 64 tile of D, eight wavefronts that split K among themselves: 64-column tile kb goes to
// wavefront kb % 8, each accumulates a whole partial tile, and the eight are added through LDS in wavefront
// order.  Such products have few tiles (1024 x 509: 128) and would be bound by the latency of their loads; with K
// split eight ways every compute unit keeps eight times the bytes in flight, and a wavefront's LDS image of B is
// its own, so the loop has no barrier at all.  The compressed (or dense) first operand goes from memory into
// registers in the matrix instruction's own lane order.
//
// Measured against the general kernel that took these before (us, operands rotating): 1024 x 509 x 4096 int8 482 -> 12.7;
// 8192 x 17 x 8192 bf16 443 -> 30; 2048 x 509 x 2048 bf16 12.3.  Products with many tiles, or few steps of K, go to mm_staged.hpp.
#include "mm_operands.hpp"

namespace sp24 {

namespace {

constexpr int kSplitWaves = 8;
constexpr int TN = 2;                               // 32 x 32 accumulator tiles of a wavefront side by side

// between a wavefront's own LDS writes and reads: the LDS serves them in order, only the compiler must keep it
__device__ __forceinline__ void wave_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The dense first operand of TM blocks of 32 rows in the dense instruction's lane order, as compressed_rows
template <int DT, int TM>
struct dense_rows {
    static constexpr int ES = is8<DT> ? 1 : 2;
    static constexpr int NA = 2 * ES;
    const uint8_t* src[TM];
    int64_t row_bytes;
    int q;
    __device__ __forceinline__ void init(const MmArgs& a, int64_t block0, int lane)
    {
        q = lane >> 5;
        row_bytes = a.K * ES;
#pragma unroll
        for (int i = 0; i < TM; ++i)
            src[i] = reinterpret_cast<const uint8_t*>(a.A) + min((block0 + i) * 32 + (lane & 31), a.M - 1) * a.lda * ES + 16 * q;
    }
    __device__ __forceinline__ void load_whole(int64_t kb, int4v (&v)[TM][NA], uint32_t (&code)[TM]) const { load_edge(kb, v, code); }
    __device__ __forceinline__ void load_edge(int64_t kb, int4v (&v)[TM][NA], uint32_t (&code)[TM]) const
    {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
#pragma unroll
            for (int s = 0; s < NA; ++s) {
                const int64_t at = kb * (64 * ES) + 32 * s;
                v[i][s] = __builtin_bit_cast(int4v, load16_aligned(at + 16 * q < row_bytes ? src[i] + at : k_zero_row));
            }
            code[i] = 0;
        }
    }
};

} // namespace

template <int DT, bool SPARSE, int TM>
__global__ __launch_bounds__(64 * kSplitWaves) void k_mm_ksplit(MmArgs a, int tiles_m, int tiles_n)
{
    constexpr int ES = is8<DT> ? 1 : 2;
    constexpr int BN = 32 * TN;
    constexpr int kImage = 64 * BN * ES;                      // 64 K rows of B in LDS
    using acc_t = typename acc_of<DT>::type;
    constexpr int kRedBytes = kSplitWaves * TN * 16 * 64 * 4;
    constexpr int kLds = kSplitWaves * kImage > kRedBytes ? kSplitWaves * kImage : kRedBytes;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[kLds];

    int tm, tn;
    tile_of_workgroup(tiles_m, tiles_n, tm, tn);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 31, q = lane >> 5;
    const int tiles_k = (int)((a.K + 63) / 64);

    using pieces_t = nmajor_pieces<BN, ES, 64, 64>;
    using rows_t = typename std::conditional<SPARSE, compressed_rows<DT, TM>, dense_rows<DT, TM>>::type;
    constexpr int NA = rows_t::NA;
    pieces_t pieces;
    pieces.init(a, tn, lane);
    rows_t rows;
    rows.init(a, (int64_t)tm * TM, lane);
    uint8_t* const image = lds + wave * kImage;
    nmajor_frags<BN, TN, ES> frags;
    frags.init(0, lane);

    acc_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = acc_t{};

    struct Tile {
        uint4v b[pieces_t::NJ];
        int4v v[TM][NA];
        uint32_t code[TM];
    };
    auto compute = [&](const Tile& t) {
        wave_order();                                         // behind the reads of the previous tile
        pieces.store(image, t.b);
        wave_order();
        if constexpr (SPARSE) {
            constexpr int NI = ES;                            // instructions per tile: 8-bit one of 64 columns, 16-bit two of 32
#pragma unroll
            for (int s = 0; s < NI; ++s)
#pragma unroll
                for (int nj = 0; nj < TN; ++nj) {
                    const uint4v lo = frags.piece(image, s, nj), hi = frags.piece(image, s + NI, nj);
                    int8v b;
                    b[0] = lo[0]; b[1] = lo[1]; b[2] = lo[2]; b[3] = lo[3];
                    b[4] = hi[0]; b[5] = hi[1]; b[6] = hi[2]; b[7] = hi[3];
#pragma unroll
                    for (int i = 0; i < TM; ++i) {
                        if (s == 0) acc[i][nj] = smfmac32<DT, 0>(t.v[i][0], b, acc[i][nj], (int)t.code[i]);
                        else acc[i][nj] = smfmac32<DT, 1>(t.v[i][NA - 1], b, acc[i][nj], (int)t.code[i]);
                    }
                }
        } else {
#pragma unroll
            for (int s = 0; s < NA; ++s)
#pragma unroll
                for (int nj = 0; nj < TN; ++nj) {
                    const int4v b = __builtin_bit_cast(int4v, frags.piece(image, s, nj));
#pragma unroll
                    for (int i = 0; i < TM; ++i) acc[i][nj] = mfma32<DT>(t.v[i][s], b, acc[i][nj]);
                }
        }
    };
    // The tiles whose pieces all lie inside B: this wavefront's are wave, wave + 8, ..., the next one's loads under way
    // while a tile is computed.  (No branch around a load in the loop: the compiler then leaves them in flight.  More of
    // them, two to four tiles ahead, cost registers and time: 1024 x 509 x 4096 int8 12.7 us with one, 13.1 with three.)
    const int whole = (int)pieces.whole_groups();
    Tile tile;
    auto load = [&](int kb) {
        pieces.load_whole(kb, tile.b);
        rows.load_whole(kb, tile.v, tile.code);
    };
    if (wave < whole) {
        load(wave);
        int kb = wave;
        for (; kb + kSplitWaves < whole; kb += kSplitWaves) {
            if constexpr (TM == 1) {
                const Tile now = tile;
                load(kb + kSplitWaves);
                compute(now);
            } else {                                          // two workgroups to a unit hide more than a second set of registers
                compute(tile);
                load(kb + kSplitWaves);
            }
        }
        compute(tile);
    }
    for (int kb = whole; kb < tiles_k; ++kb)
        if (kb % kSplitWaves == wave) {
            pieces.load_edge(kb, tile.b);
            rows.load_edge(kb, tile.v, tile.code);
            compute(tile);
        }

    // the eight partial tiles, added in wavefront order, 32 rows at a time
    uint32_t (*red)[TN * 16][64] = reinterpret_cast<uint32_t (*)[TN * 16][64]>(lds);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        __syncthreads();                                      // the images, or the previous rows, are done with
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                auto v = acc[i][j][e];
                red[wave][j * 16 + e][lane] = __builtin_bit_cast(uint32_t, v);
            }
        __syncthreads();
#pragma unroll
        for (int x = 0; x < TN * 16 / kSplitWaves; ++x) {
            const int id = wave + x * kSplitWaves, j = id >> 4, e = id & 15;
            using val_t = typename std::conditional<DT == SP24_I8, int, float>::type;
            val_t sum = 0;
#pragma unroll
            for (int w = 0; w < kSplitWaves; ++w) sum += __builtin_bit_cast(val_t, red[w][id][lane]);
            const int64_t m = ((int64_t)tm * TM + i) * 32 + 8 * (e / 4) + 4 * q + (e % 4);
            const int64_t n = (int64_t)tn * BN + j * 32 + r;
            if (m < a.M && n < a.N) put<DT>(a, m, n, sum);
        }
    }
}

template <int DT>
static sp24_status run_ksplit(const MmArgs& a, hipStream_t st)
{
    auto run = [&](auto kernel, int bm) {
        const int tiles_m = (int)((a.M + bm - 1) / bm), tiles_n = (int)((a.N + 32 * TN - 1) / (32 * TN));
        kernel<<<dim3((unsigned)(tiles_m * tiles_n)), dim3(64 * kSplitWaves), 0, st>>>(a, tiles_m, tiles_n);
        return hipGetLastError() == hipSuccess ? SP24_OK : SP24_ERR_LAUNCH;
    };
    // Tiles of 32 rows while that gives no more than one workgroup a compute unit (1024 x 509 x 4096 int8 16.2 -> 12.7 us,
    // 8192 x 17 x 2048 bf16 13.1 -> 9.6); past that the 64-row tile, whose B serves twice the rows.
    const bool low = ((a.M + 31) / 32) * ((a.N + 63) / 64) <= 256;
    if (a.sparse) return low ? run(k_mm_ksplit<DT, true, 1>, 32) : run(k_mm_ksplit<DT, true, 2>, 64);
    return low ? run(k_mm_ksplit<DT, false, 1>, 32) : run(k_mm_ksplit<DT, false, 2>, 64);
}

sp24_status launch_mm_ksplit(const MmArgs& a, hipStream_t st, bool* handled)
{
    *handled = false;
    if (a.conv.on || a.bo != SP24_B_NMAJOR || a.k_slices > 1 || a.K > ((int64_t)1 << 30)) return SP24_OK;
    if (a.M > ((int64_t)1 << 30) || a.N > ((int64_t)1 << 30) || ((a.M + 31) / 32) * ((a.N + 63) / 64) >= ((int64_t)1 << 30)) return SP24_OK;
    *handled = true;
    if (a.in == SP24_I8) return run_ksplit<SP24_I8>(a, st);
    if (a.in == SP24_F8) return run_ksplit<SP24_F8>(a, st);
    if (a.in == SP24_F16) return run_ksplit<SP24_F16>(a, st);
    return run_ksplit<SP24_BF16>(a, st);
}

} // namespace sp24
