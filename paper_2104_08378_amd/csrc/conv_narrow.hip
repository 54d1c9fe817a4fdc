// Sparse 3 x 3 convolution of 8-bit inputs whose channel count is a multiple of 64 and not of 128 (the 64-channel
// layers of a network's first stage): the patch scheme of conv_patch.hpp -- all taps of a tile read one patch of the
// input in LDS, A goes straight into registers -- with chunks of 64 channels, so that a K step, one matrix instruction
// per accumulator tile, is one tap of one chunk, and K step (tap, chunk) is 64-column tile tap * chunks + chunk of the
// compressed rows.
//
// Such layers have few filters and large images: a tile is 64 filters x 128 pixels (a 128-row tile would be half
// padding), four wavefronts of 32 x 64.  With one chunk, nine steps of two instructions are all the arithmetic a
// wavefront has; the time is the latency of one patch in and one tile out, so what counts is how many workgroups
// share a compute unit.  A of a whole chunk (nine steps, 45 registers) is loaded ahead of the barrier, under the patch's own
// latency.  ONE: inputs with one chunk, which need one patch buffer and no registers for a next one: four workgroups to a
// unit with either size of patch, where two buffers of 256 pixels leave room for three (56 x 56, 64 -> 64, 32 images, int8: 784
// tiles on 768 places took 11.2 us, 8.7 on 1024; one image 5.0 -> 4.5, 28 x 28, 64 -> 128, 64 images 8.5 -> 8.2; 8-bit floats 7 -
// 29 % faster throughout).  With several chunks four with the 192-pixel patch, three with the 256-pixel one.
// (Four workgroups mean 128 registers: the 192-pixel instances for several chunks that need more keep 20 bytes a lane, int8
// to int8, or 24 - 84, 8-bit floats, in scratch memory.)
// Patch rows are 80 bytes apart: sixteen consecutive rows fall into sixteen different 16-byte columns of LDS.
//
// Measured with the quantised epilogue to int8, against the general kernel that took these layers before (us, operands
// rotating): 56 x 56, 64 -> 64 channels, 32 images 188 -> 8.7; 28 x 28, 64 -> 128, 32 images 107 -> 9.8; 14 x 14,
// 192 -> 192, 64 images 183 -> 10.5.  (Below 10 us it is the rate of the calls that is measured.)
#include "conv_patch.hpp"

namespace sp24 {

constexpr int kNarrowPitch = 80;

template <int DT, int OUT, int kPatchRows, bool ONE>
__global__ __launch_bounds__(256, ONE || kPatchRows <= kPatchRowsSmall ? 4 : 3) void k_conv_patch_narrow(MmArgs a, int tiles_m, int tiles_n)
{
    static_assert(is8<DT>, "a step is one instruction of 64 one-byte columns");
    constexpr int CB = 64;                             // channels (bytes) of a chunk
    constexpr int WN = 2, TM = 1, TN = 2, BN = 128, TAPS = 9;
    constexpr int kPitch = kNarrowPitch;
    constexpr int XP = kPatchRows * (CB / 16) / 256;   // 16-byte pieces of a patch per lane
    constexpr int kPatchBytes = (kPatchRows + 1) * kPitch, kZeroOff = kPatchRows * kPitch;
    constexpr int kEpiBytes = 4 * epilogue_geometry<OUT, TN>::kWaveBytes;
    constexpr int kBuffers = ONE ? 1 : 2;
    constexpr int kLdsBytes = kBuffers * kPatchBytes > kEpiBytes ? kBuffers * kPatchBytes : kEpiBytes;
    using acc_t = typename acc_of<DT>::type;
    __shared__ __attribute__((aligned(1024))) uint8_t lds_all[kLdsBytes];

    int tm, tn;
    tile_of_workgroup(tiles_m, tiles_n, tm, tn);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int r = lane & 31, q = lane >> 5;
    const ConvGeom g = a.conv;
    const int nchunks = ONE ? 1 : g.C / CB;
    const uint8_t* X = reinterpret_cast<const uint8_t*>(a.B);
    const int64_t n_pixels = (a.N / ((int64_t)g.OH * g.OW)) * g.H * g.W;      // input pixels in all images

    // linear index of the input pixel that tap (0, 0) meets for output pixel n (may lie before the image: padding)
    auto lin0_of = [&](int64_t n, int& iy, int& ix) -> int64_t {
        const int t = (int)n / g.OW;
        const int ox = (int)n - t * g.OW;
        const int img = t / g.OH;
        const int oy = t - img * g.OH;
        iy = oy - g.pad_h;
        ix = ox - g.pad_w;
        return (int64_t)(img * g.H + iy) * g.W + ix;
    };
    const int64_t n0 = (int64_t)tn * BN;
    int unused_y, unused_x;
    int64_t patch_first = lin0_of(n0, unused_y, unused_x);                     // wave-uniform
    if (patch_first < 0) patch_first = 0;

    // ---- the patch: piece x of this lane is patch row x * 64 + tid / 4, 16-byte column tid % 4.  Rows past the input
    // fetch the last pixel (no tap inside the image reads them) ----
    const int64_t last_rel = n_pixels - 1 - patch_first;
    const uint8_t* patch_base = X + patch_first * g.C;
    uint32_t piece_src[XP];
#pragma unroll
    for (int x = 0; x < XP; ++x) {
        const int row = x * 64 + (tid >> 2);
        piece_src[x] = (uint32_t)((row < last_rel ? row : last_rel) * g.C) + (tid & 3) * 16;
    }
    const uint32_t piece_dst = (uint32_t)((tid >> 2) * kPitch + (tid & 3) * 16);
    uint4v patch[XP];
    auto load_patch = [&](int chunk) {
#pragma unroll
        for (int x = 0; x < XP; ++x) patch[x] = *reinterpret_cast<const uint4v*>(patch_base + (int64_t)chunk * CB + piece_src[x]);
    };
    auto store_patch = [&](int buf) {
#pragma unroll
        for (int x = 0; x < XP; ++x) *reinterpret_cast<uint4v*>(lds_all + buf * kPatchBytes + piece_dst + x * 64 * kPitch) = patch[x];
    };
    load_patch(0);

    // ---- A: this wavefront's row block, straight from the tiled layout ----
    const int64_t KB64 = a.K / 64, rb_total = a.M / 32;
    int64_t rb = (int64_t)tm * 2 + wm;
    if (rb >= rb_total) rb = rb_total - 1;              // ragged M: a valid row block, never stored
    const uint8_t* v_base = reinterpret_cast<const uint8_t*>(a.A) + rb * KB64 * 1024;
    const uint8_t* m_base = reinterpret_cast<const uint8_t*>(a.meta) + rb * KB64 * 256;
    const __amdgpu_buffer_rsrc_t v_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(wave_uniform(v_base)), 0, __builtin_amdgcn_readfirstlane((int)(KB64 * 1024)), 0x00020000);
    const __amdgpu_buffer_rsrc_t m_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(wave_uniform(m_base)), 0, __builtin_amdgcn_readfirstlane((int)(KB64 * 256)), 0x00020000);
    int4v av[TAPS];
    int mv[TAPS];
    auto load_a = [&](int t, int chunk) {
        const int kt = t * nchunks + chunk;
        av[t] = __builtin_bit_cast(int4v, __builtin_amdgcn_raw_buffer_load_b128(v_rsrc, lane * 16, kt * 1024, 0));
        mv[t] = __builtin_amdgcn_raw_buffer_load_b32(m_rsrc, lane * 4, kt * 256, 0);
    };
#pragma unroll
    for (int t = 0; t < TAPS; ++t) load_a(t, 0);

    // LDS address (in buffer 0) of this lane's row of B for each tap and output pixel, as in k_conv_patch
    uint32_t b_row[TAPS][TN];
#pragma unroll
    for (int nj = 0; nj < TN; ++nj) {
        const int64_t n = n0 + wn * 32 * TN + nj * 32 + r;
        int iy0 = 0, ix0 = 0;
        const int prow = n < a.N ? (int)(lin0_of(n, iy0, ix0) - patch_first) : 0;
#pragma unroll
        for (int t = 0; t < TAPS; ++t) {
            const int tr = t / 3, ts = t % 3;
            const bool in = n < a.N && (unsigned)(iy0 + tr) < (unsigned)g.H && (unsigned)(ix0 + ts) < (unsigned)g.W;
            b_row[t][nj] = (uint32_t)(in ? (prow + tr * g.W + ts) * kPitch : kZeroOff) + q * 16;
        }
    }

    acc_t acc[TM][TN];
#pragma unroll
    for (int nj = 0; nj < TN; ++nj) acc[0][nj] = acc_t{};

    if (tid < kBuffers * (kPitch / 4)) reinterpret_cast<uint32_t*>(lds_all + kZeroOff + (tid / (kPitch / 4)) * kPatchBytes)[tid % (kPitch / 4)] = 0u;
    store_patch(0);
    if (nchunks > 1) load_patch(1);
    __syncthreads();
    for (int c = 0; c < nchunks; ++c) {
        // the patch of the next chunk goes into the other buffer, whose readers have passed the last barrier
        if (c + 1 < nchunks) store_patch((c + 1) & 1);
        if (c + 2 < nchunks) load_patch(c + 2);
        const uint8_t* buf = lds_all + (c & 1) * kPatchBytes;
#pragma unroll
        for (int t = 0; t < TAPS; ++t) {
#pragma unroll
            for (int nj = 0; nj < TN; ++nj) {
                const uint4v lo = *reinterpret_cast<const uint4v*>(buf + b_row[t][nj]);
                const uint4v hi = *reinterpret_cast<const uint4v*>(buf + b_row[t][nj] + 32);
                int8v b;
                b[0] = lo[0]; b[1] = lo[1]; b[2] = lo[2]; b[3] = lo[3];
                b[4] = hi[0]; b[5] = hi[1]; b[6] = hi[2]; b[7] = hi[3];
                acc[0][nj] = smfmac32<DT, 0>(av[t], b, acc[0][nj], mv[t]);
            }
            if (c + 1 < nchunks) load_a(t, c + 1);
        }
        __syncthreads();
    }
    // LDS becomes store scratch
    store_wave_tile<DT, OUT, TM, TN>(a, acc, lds_all + wave * epilogue_geometry<OUT, TN>::kWaveBytes,
                                     (int64_t)tm * 64 + wm * 32, (int64_t)tn * BN + wn * TN * 32, lane);
}

template <int DT, int OUT>
static sp24_status run_narrow(const MmArgs& a, hipStream_t st)
{
    const int tiles_m = (int)((a.M + 63) / 64), tiles_n = (int)((a.N + 127) / 128);
    const dim3 grid((unsigned)(tiles_m * tiles_n)), block(256);
    auto run = [&](auto kernel) { kernel<<<grid, block, 0, st>>>(a, tiles_m, tiles_n); };
    const bool small = conv_patch_span(a) <= kPatchRowsSmall;
    if (a.conv.C == 64) small ? run(k_conv_patch_narrow<DT, OUT, kPatchRowsSmall, true>) : run(k_conv_patch_narrow<DT, OUT, kPatchRowsLarge, true>);
    else small ? run(k_conv_patch_narrow<DT, OUT, kPatchRowsSmall, false>) : run(k_conv_patch_narrow<DT, OUT, kPatchRowsLarge, false>);
    return hipGetLastError() == hipSuccess ? SP24_OK : SP24_ERR_LAUNCH;
}

sp24_status launch_conv_narrow(const MmArgs& a, hipStream_t st, bool* handled)
{
    *handled = false;
    const bool ok = a.conv.on && esize_of(a.in) == 1 && a.conv.C % 64 == 0 && a.conv.C % 128 != 0 && conv_patch_span(a) > 0 &&
                    (reinterpret_cast<uintptr_t>(a.B) & 15u) == 0 && a.M <= ((int64_t)1 << 30) &&
                    ((a.M + 63) / 64) * ((a.N + 127) / 128) < ((int64_t)1 << 30);
    if (!ok) return SP24_OK;
    *handled = true;
    if (a.in == SP24_I8) {
        if (a.out == SP24_I32) return run_narrow<SP24_I8, SP24_I32>(a, st);
        if (a.out == SP24_I8) return run_narrow<SP24_I8, SP24_I8>(a, st);
        if (a.out == SP24_F32) return run_narrow<SP24_I8, SP24_F32>(a, st);
        if (a.out == SP24_F16) return run_narrow<SP24_I8, SP24_F16>(a, st);
        return run_narrow<SP24_I8, SP24_BF16>(a, st);
    }
    if (a.out == SP24_F32) return run_narrow<SP24_F8, SP24_F32>(a, st);
    if (a.out == SP24_F16) return run_narrow<SP24_F8, SP24_F16>(a, st);
    return run_narrow<SP24_F8, SP24_BF16>(a, st);
}

} // namespace sp24
