// Sparse products whose second operand passes through registers on its way to LDS: what the tiled kernels' direct
// transfers cannot fetch, on tiles of the same shape.
//
//   BSRC 0  K-major rows (with a compressed operand whose K is no multiple of 32, or rows that are not 16-byte aligned)
//   BSRC 1  a convolution's input, any channel count the library takes: a 128-byte step of K may lie across several
//           filter taps, so every 16-byte piece finds its own (a piece never straddles one)
//   BSRC 2  N-major rows at any address (an odd number of columns)
//
// A workgroup of four wavefronts computes 32*TM*WM x 32*TN*WN; a step is 128 bytes of K.  B: each thread loads its
// 16-byte pieces of the step two steps ahead into registers and writes them into one of two LDS images (swizzled as in
// the tiled kernels, so that fragment reads have no bank conflicts); A goes from memory into registers in the matrix
// instruction's own lane order, also two steps ahead.  One barrier per step, which waits for LDS only: the
// loads of the next steps stay in flight across it.  Past the barrier of step s nobody reads the image of step s - 1
// any more, which is the one that step s + 1 writes.  All waits for loads are the compiler's own, and the loop has no
// branch around a load, so that it can leave the younger ones in flight: it covers the steps that lie wholly inside both
// operands, and the last ones follow as a phase of their own.
//
// Bound by the latency and the issue of those loads: a tile moves the same bytes per product as a 128 x 128 tile of the
// tiled kernels.  Measured against the general and the K-splitting kernels that took these before (us): sparse 3x3
// convolution, 43 images of 28x28, 96 -> 192 channels, bf16 417 -> 32; 93 images of 15x15, 96 -> 96, 121 -> 15;
// 18624 x 552 x 5392 bf16 canonical 4667 -> 245 (217 with an earlier form of the loop, slower for N-major B); 2304 x 1411 x 400 f16 canonical 135 -> 11; N-major 6784 x 939 x 6464 bf16
// 193 -> 90, 4096 x 4095 x 4096 bf16 125, int8 83.
#pragma once
#include "mm_operands.hpp"

namespace sp24 {

// B of one thread: NJ pieces of each step
template <int DT, int BSRC, int BN>
struct staged_b;

template <int DT, int BN>
struct staged_b<DT, 0, BN> {
    static constexpr int ES = is8<DT> ? 1 : 2, NJ = BN * 8 / 256;
    const uint8_t* src[NJ];
    int64_t row_bytes;
    int at, dst0;                                              // byte of the row; place in the image
    __device__ __forceinline__ void init(const MmArgs& a, int64_t tn, int tid)
    {
        row_bytes = a.K * ES;
        at = (tid & 7) * 16;
        const int row = tid >> 3;
        dst0 = row * kRowBytes + (((tid & 7) ^ ((row >> 1) & 7)) << 4);
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int64_t n = min(tn * BN + row + j * 32, a.N - 1);   // past the last column: a valid row, never stored
            src[j] = reinterpret_cast<const uint8_t*>(a.B) + n * a.ldb * ES + at;
        }
    }
    // the pieces of step `step`; steps are asked for in order
    __device__ __forceinline__ void load(int step, uint4v (&v)[NJ])
    {
        const bool inside = (int64_t)step * kRowBytes + at < row_bytes;
#pragma unroll
        for (int j = 0; j < NJ; ++j) v[j] = load16_any(inside ? src[j] + (int64_t)step * kRowBytes : k_zero_row);
    }
    __device__ __forceinline__ void store(uint8_t* image, const uint4v (&v)[NJ]) const
    {
#pragma unroll
        for (int j = 0; j < NJ; ++j) *reinterpret_cast<uint4v*>(image + dst0 + j * 32 * kRowBytes) = v[j];
    }
};

template <int DT, int BN>
struct staged_b<DT, 1, BN> {
    static constexpr int ES = is8<DT> ? 1 : 2, NJ = BN * 8 / 256;
    const uint8_t* src[NJ];                                    // the (possibly virtual) pixel of tap (0, 0)
    int iy0[NJ], ix0[NJ];
    int r, s, c, cb;                                           // tap and byte of the pixel of this thread's next pieces; bytes of a pixel
    int H, W, R, S, dst0;
    __device__ __forceinline__ void init(const MmArgs& a, int64_t tn, int tid)
    {
        const ConvGeom& g = a.conv;
        H = g.H; W = g.W; R = g.R; S = g.S;
        cb = g.C * ES;
        r = s = 0;
        c = (tid & 7) * 16;
        wrap();
        const int row = tid >> 3;
        dst0 = row * kRowBytes + (((tid & 7) ^ ((row >> 1) & 7)) << 4);
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int64_t n = tn * BN + row + j * 32;
            const int64_t t = n / g.OW;
            const int ox = (int)(n - t * g.OW);
            const int64_t img = t / g.OH;
            const int oy = (int)(t - img * g.OH);
            iy0[j] = n < a.N ? oy * g.stride_h - g.pad_h : -(1 << 28);   // past the last pixel: zeros, never stored
            ix0[j] = ox * g.stride_w - g.pad_w;
            src[j] = reinterpret_cast<const uint8_t*>(a.B) + ((img * g.H + oy * g.stride_h - g.pad_h) * (int64_t)g.W + ix0[j]) * cb;
        }
    }
    __device__ __forceinline__ void wrap()
    {
        while (c >= cb) {
            c -= cb;
            if (++s == S) { s = 0; ++r; }
        }
    }
    __device__ __forceinline__ void load(int, uint4v (&v)[NJ])
    {
        const int64_t tap = ((int64_t)r * W + s) * cb + c;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const bool inside = r < R && (unsigned)(iy0[j] + r) < (unsigned)H && (unsigned)(ix0[j] + s) < (unsigned)W;
            v[j] = load16_any(inside ? src[j] + tap : k_zero_row);
        }
        c += kRowBytes;
        wrap();
    }
    __device__ __forceinline__ void store(uint8_t* image, const uint4v (&v)[NJ]) const
    {
#pragma unroll
        for (int j = 0; j < NJ; ++j) *reinterpret_cast<uint4v*>(image + dst0 + j * 32 * kRowBytes) = v[j];
    }
};

template <int DT, int BN>
struct staged_b<DT, 2, BN> : nmajor_pieces<BN, is8<DT> ? 1 : 2, is8<DT> ? 128 : 64, 256> {
    using base = nmajor_pieces<BN, is8<DT> ? 1 : 2, is8<DT> ? 128 : 64, 256>;
    __device__ __forceinline__ void load(int step, uint4v (&v)[base::NJ]) { base::load_whole(step, v); }
};

// every LDS access of this wavefront is done, then the workgroup's barrier; loads stay in flight
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int DT, int BSRC, int WM, int WN, int TM, int TN>
__global__ __launch_bounds__(256, 2) void k_spmm_staged(MmArgs a, int tiles_m, int tiles_n)
{
    static_assert(WM * WN == 4, "four wavefronts");
    constexpr int T64 = is8<DT> ? 2 : 1;                      // 64-column tiles of A per step
    constexpr int BN = 32 * TN * WN;
    constexpr int kImage = BN * kRowBytes;
    constexpr int kOutWide = DT == SP24_I8 ? SP24_I32 : SP24_F32;
    constexpr int kEpi = 4 * epilogue_geometry<kOutWide, TN>::kWaveBytes;
    constexpr int kLds = 2 * kImage > kEpi ? 2 * kImage : kEpi;
    using acc_t = typename acc_of<DT>::type;
    using b_t = staged_b<DT, BSRC, BN>;
    using a_t = compressed_rows<DT, TM>;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[kLds];

    int tm, tn;
    tile_of_workgroup(tiles_m, tiles_n, tm, tn);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int r = lane & 31, q = lane >> 5;
    const int nsteps = (int)((a.K + 64 * T64 - 1) / (64 * T64));

    b_t b;
    b.init(a, tn, tid);
    a_t rows;
    rows.init(a, (int64_t)tm * (WM * TM) + wm * TM, lane);
    struct A {
        int4v v[T64][TM][a_t::NA];
        uint32_t code[T64][TM];
    };

    // fragment reads: as in the tiled kernels
    int frag_off[4];
#pragma unroll
    for (int c2 = 0; c2 < 4; ++c2) frag_off[c2] = (wn * 32 * TN + r) * kRowBytes + ((((2 * c2) | q) ^ ((r >> 1) & 7)) << 4);
    nmajor_frags<BN, TN, is8<DT> ? 1 : 2> b_nm;
    if constexpr (BSRC == 2) b_nm.init(wn, lane);
    acc_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = acc_t{};

    uint4v bv[2][b_t::NJ];
    A av[2];
    auto compute = [&](const A& va, const uint8_t* image) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int nj = 0; nj < TN; ++nj) {
                const int c2lo = is8<DT> ? 2 * j : j, c2hi = is8<DT> ? 2 * j + 1 : 2 + j;
                uint4v lo, hi;
                if constexpr (BSRC == 2) {
                    lo = b_nm.piece(image, c2lo, nj);
                    hi = b_nm.piece(image, c2hi, nj);
                } else {
                    lo = *reinterpret_cast<const uint4v*>(image + frag_off[c2lo] + nj * 32 * kRowBytes);
                    hi = *reinterpret_cast<const uint4v*>(image + frag_off[c2hi] + nj * 32 * kRowBytes);
                }
                int8v f;
                f[0] = lo[0]; f[1] = lo[1]; f[2] = lo[2]; f[3] = lo[3];
                f[4] = hi[0]; f[5] = hi[1]; f[6] = hi[2]; f[7] = hi[3];
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    if constexpr (is8<DT>) acc[i][nj] = smfmac32<DT, 0>(va.v[j][i][0], f, acc[i][nj], (int)va.code[j][i]);
                    else if (j == 0) acc[i][nj] = smfmac32<DT, 0>(va.v[0][i][0], f, acc[i][nj], (int)va.code[0][i]);
                    else acc[i][nj] = smfmac32<DT, 1>(va.v[0][i][a_t::NA - 1], f, acc[i][nj], (int)va.code[0][i]);
                }
            }
    };
    // the steps that lie wholly inside both operands; past the last one the next (N-major: the last again), unused
    auto sweep = [&](int n) {
        auto load_b = [&](int step, uint4v (&v)[b_t::NJ]) { b.load(BSRC == 2 ? min(step, n - 1) : step, v); };
        auto load_a = [&](int step, A& x) {
#pragma unroll
            for (int t = 0; t < T64; ++t) rows.load_whole((int64_t)min(step, n - 1) * T64 + t, x.v[t], x.code[t]);
        };
        auto do_step = [&](int step, uint4v (&vb)[b_t::NJ], A& va, uint8_t* image) {
            b.store(image, vb);
            load_b(step + 2, vb);
            lds_barrier();
            // the loads stay where they are written: dealt out among the arithmetic they took 8 - 15 % longer (not so the
            // convolution's, which are 2 - 4 % faster that way)
            if constexpr (BSRC != 1) __builtin_amdgcn_sched_barrier(0);
            compute(va, image);
            if constexpr (BSRC != 1) __builtin_amdgcn_sched_barrier(0);
            load_a(step + 2, va);
            if constexpr (BSRC != 1) __builtin_amdgcn_sched_barrier(0);
        };
        load_b(0, bv[0]);
        load_a(0, av[0]);
        load_b(1, bv[1]);
        load_a(1, av[1]);
        int step = 0;
        for (; step + 2 <= n; step += 2) {
            do_step(step, bv[0], av[0], lds);
            do_step(step + 1, bv[1], av[1], lds + kImage);
        }
        if (step < n) do_step(step, bv[0], av[0], lds);
        lds_barrier();                                        // LDS is free
    };
    int whole = (int)(a.K / (64 * T64));
    if constexpr (BSRC == 2) whole = (int)b.whole_groups();
    if (whole > 0) sweep(whole);
    auto edge = [&](int step, const uint4v (&vb)[b_t::NJ]) {
        b.store(lds, vb);
#pragma unroll
        for (int t = 0; t < T64; ++t) rows.load_edge((int64_t)step * T64 + t, av[0].v[t], av[0].code[t]);
        lds_barrier();
        compute(av[0], lds);
        lds_barrier();
    };
    if constexpr (BSRC == 2) {
        for (int step = whole; step < nsteps; ++step) {
            b.load_edge(step, bv[0]);
            edge(step, bv[0]);
        }
    } else if (whole < nsteps) {                              // its pieces of B are under way already
        if (whole == 0) b.load(0, bv[0]);
        if (whole % 2 == 0) edge(whole, bv[0]);
        else edge(whole, bv[1]);
    }

    const int64_t row_base = ((int64_t)tm * WM + wm) * TM * 32, col_base = (int64_t)tn * BN + wn * TN * 32;
    auto put = [&](auto out_c) {
        constexpr int OUT = decltype(out_c)::value;
        store_wave_tile<DT, OUT, TM, TN>(a, acc, lds + wave * epilogue_geometry<OUT, TN>::kWaveBytes, row_base, col_base, lane);
    };
    using std::integral_constant;
    if constexpr (DT == SP24_I8) {
        if (a.out == SP24_I32) put(integral_constant<int, SP24_I32>{});
        else if (a.out == SP24_I8) put(integral_constant<int, SP24_I8>{});
        else if (a.out == SP24_F32) put(integral_constant<int, SP24_F32>{});
        else if (a.out == SP24_F16) put(integral_constant<int, SP24_F16>{});
        else put(integral_constant<int, SP24_BF16>{});
    } else {
        if (a.out == SP24_F32) put(integral_constant<int, SP24_F32>{});
        else if (a.out == SP24_F16) put(integral_constant<int, SP24_F16>{});
        else put(integral_constant<int, SP24_BF16>{});
    }
}

template <int DT, int BSRC>
static sp24_status run_staged_from(const MmArgs& a, hipStream_t st)
{
    auto run = [&](auto kernel, int bm, int bn) {
        const int tiles_m = (int)((a.M + bm - 1) / bm), tiles_n = (int)((a.N + bn - 1) / bn);
        kernel<<<dim3((unsigned)(tiles_m * tiles_n)), dim3(256), 0, st>>>(a, tiles_m, tiles_n);
        return hipGetLastError() == hipSuccess ? SP24_OK : SP24_ERR_LAUNCH;
    };
    // The smallest tile whose workgroups find a unit each, 64 x 64 on up to 256 of them: against 64 x 128 (32 x 128 up to 32 rows),
    // times as fast, convolutions 1.12 - 1.52 (96 -> 96 channels, 5x5, 4 images of 7x7 f16 24.5 -> 16.1 us, int8 15.4 -> 11.7), K a multiple of
    // 16 1.15 - 1.43 (1024 x 509 x 1040 bf16 9.4 -> 7.1), N-major 1.18 - 1.22 (3000 x 301 x 4096 bf16 42.9 -> 35.1); on 392 of
    // them 0.92 - 1.09, and 0.8 - 0.92 for products.  Past that as many rows as there are; tiles of 64 rows also while the large ones
    // would not give every compute unit one.  Two by two wavefronts also there: side by side (1 x 4), each would load
    // the same rows of A again, and the address path is the bound (4096 x 509 x 4096 N-major bf16 34 -> 27 us, 4096 x 509 x 1024
    // 12.8 -> 10.6).  From 256 tiles on the large ones are 20 - 50 % faster (4096 x 4095 x 4096: 185 -> 125), convolutions and
    // 8-bit gathers within 15 % either way.
    const int64_t large = ((a.M + 127) / 128) * ((a.N + 127) / 128);
    if (((a.M + 63) / 64) * ((a.N + 63) / 64) <= 256) return run(k_spmm_staged<DT, BSRC, 2, 2, 1, 1>, 64, 64);
    if (a.M <= 32) return run(k_spmm_staged<DT, BSRC, 1, 4, 1, 1>, 32, 128);
    if (a.M <= 64 || large < 256) return run(k_spmm_staged<DT, BSRC, 2, 2, 1, 2>, 64, 128);
    return run(k_spmm_staged<DT, BSRC, 2, 2, 2, 2>, 128, 128);
}

template <int DT>
static sp24_status run_staged(const MmArgs& a, hipStream_t st)
{
    if (a.conv.on) return run_staged_from<DT, 1>(a, st);
    if (a.bo == SP24_B_NMAJOR) return run_staged_from<DT, 2>(a, st);
    return run_staged_from<DT, 0>(a, st);
}

} // namespace sp24
