// Search for a column order under which 2:4 pruning keeps more magnitude (Sec. 4.1, Step 2; Fig. 6).
//
// The paper states the aim and leaves the method to a later publication; the method here is this library's own,
// chosen so that every step is independent work for a whole chip and the result is unique:
//
//   * the order is read as K/4 groups of four columns; the score of a group is the magnitude pruning keeps in it,
//     the sum over the rows of the row's two largest magnitudes among its four columns (NaN counts as +infinity);
//   * a step takes two groups g < h -- eight columns, positions 0..3 those of g -- and tries the 35 ways of dealing
//     them out as two groups of four: a way is the three positions a < b < c that share a group with position 0,
//     ways are visited in lexicographic order of (a, b, c), the first being the present arrangement, and a later
//     way wins only with a strictly higher sum of its two scores.  The winner is written back with position 0's
//     group in g and the other in h, each in ascending position;
//   * round r pairs every group whose bit r is clear with the group 2^r further on (where that exists): the pairs
//     of a round are disjoint, one workgroup takes one pair, and a round is one launch.  A sweep is the rounds
//     r = 0 .. ceil(log2(K/4)) - 1.
//
// Arithmetic (fixed, so that the order found does not depend on the machine): binary64 throughout; a row
// contributes the sum of its two largest magnitudes; the 256 lanes of the workgroup add the rows m = lane, lane +
// 256, ... in row order, and the 256 partial sums are added as a balanced binary tree over neighbours -- the
// butterfly below inside a wavefront (both partners form the same sum: addition commutes), then wavefronts 0 + 1,
// 2 + 3, and those two.  The two scores of a way are added last.  For int8 every sum is an exact integer.
//
// A row's two largest magnitudes among four columns are the largest of the six pair sums of those columns (the
// rounding of a sum is monotone, so the largest rounded pair sum is the rounded sum of the two largest): the
// kernel forms the 28 pair sums of the eight columns once per row and takes 70 maxima of six, one per group of
// four that can be formed.  What four columns a < b < c < d share with others is taken once -- the largest pair sum
// of (a, b, c), and the larger of (a, d) and (b, d) -- so that the 70 maxima cost 245 operations instead of 350.
//
// What bounds a round: those operations in binary64 (four cycles each per wavefront), and the eight single-element
// column loads per row, each touching 64 cache lines; the loads of the next row are issued before the arithmetic of
// the current one.  The 256 partial sums of the 70 scores are added by recursive halving (a lane passes on the half of
// the scores that its partner keeps): 72 exchanges instead of 420, in the same tree.  Measured on 4096 x 1024 bf16 (128 workgroups):
// 93 -> 24 us a round (8-bit: 40 -> 20); 4096 x 4096 bf16, where the workgroups outnumber the compute units, 130 -> 53.
#include <algorithm>

#include "common.hpp"
#include "launch.hpp"
#include "permute_search.hpp"

namespace sp24 {

namespace {

// magnitude of element `bits` as the type the row sums are formed in
template <int DT>
__device__ __forceinline__ auto search_magnitude(uint32_t bits)
{
    if constexpr (DT == SP24_I8) {
        const int v = (int)(int8_t)bits;
        return v < 0 ? -v : v;
    } else if constexpr (DT == SP24_F8) {
        return (double)magnitude_f8(bits);
    } else {
        float f;
        if constexpr (DT == SP24_F16) f = (float)__builtin_bit_cast(_Float16, (uint16_t)(bits & 0x7FFFu));
        else f = __uint_as_float((bits & 0x7FFFu) << 16);
        return (f != f) ? (double)__builtin_inff() : (double)f;
    }
}

// One step of the halving: of L scores held, a lane with bit W of its number clear keeps the first half and adds its
// partner's, the other keeps the second half; first, n: the number of the first score held, and how many are scores (the
// rest is padding: the halves of an odd number differ by one).
template <int L, int W>
__device__ __forceinline__ void halve(double (&v)[L], double (&kept)[(L + 1) / 2], int lane, int& first, int& n)
{
    constexpr int H = (L + 1) / 2;
    const bool up = (lane & W) != 0;
#pragma unroll
    for (int k = 0; k < H; ++k) {
        const double lower = v[k], upper = k + H < L ? v[k + H] : 0.0;
        kept[k] = (up ? upper : lower) + __shfl_xor(up ? lower : upper, W, 64);
    }
    first += up ? H : 0;
    n = up ? max(n - H, 0) : min(n, H);
}

} // namespace

// TOGETHER: a barrier every 256 rows, for matrices whose rows fill an L2 with the lines of few such blocks.  Once the order
// is no longer that of memory every workgroup reads lines all over the matrix, which it shares with the others only
// while they are at the same rows; with the arithmetic as short as it is the wavefronts drift apart, and each line is
// then fetched again (an arbitrary start order, us a sweep: 8192 x 4096 bf16 3006 -> 2273, 8192 x 8192 8-bit floats 8892 ->
// 5284, bf16, whose 256 rows are the whole L2, 10907 -> 11100; four sweeps from the order of memory 6899 -> 6408, 15251 ->
// 12894 and 18940 -> 17480; the first of them 1037 -> 1069, 2073 -> 2211 and 2541 -> 2455).
template <int DT, bool TOGETHER>
__global__ __launch_bounds__(256) void k_permute_search_round(const uint8_t* __restrict__ A, int32_t* perm, int64_t M, int64_t K,
                                                              int64_t lda_bytes, int bit)
{
    constexpr int ES = is8<DT> ? 1 : 2;
    using sum_t = typename std::conditional<DT == SP24_I8, int, double>::type;
    __shared__ double part[4][70];
    __shared__ int winner;

    // pair number -> g (bit `bit` clear) and h = g + 2^bit
    // (ids congruent mod 8 run on one XCD: each gets its eighth of the round's pairs, consecutive ones, whose columns share
    // cache lines in its L2)
    const uint32_t xcd = blockIdx.x & 7, share = gridDim.x / 8, rest = gridDim.x % 8;
    const int64_t p = (int64_t)xcd * share + min(xcd, rest) + (blockIdx.x >> 3), step = (int64_t)1 << bit;
    const int64_t g = ((p >> bit) << (bit + 1)) | (p & (step - 1)), h = g | step;
    int64_t off[8];                                            // byte offsets of the eight columns in a row
    int32_t col[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const uint32_t c = (uint32_t)perm[4 * (i < 4 ? g : h) + (i & 3)];
        col[i] = c < (uint64_t)K ? (int32_t)c : 0;            // an entry outside 0 .. K-1 reads column 0, never out of bounds
        off[i] = (int64_t)col[i] * ES;
    }

    sum_t acc[70];
#pragma unroll
    for (int s = 0; s < 70; ++s) acc[s] = 0;
    uint32_t bits[8];
    auto load_row = [&](int64_t m) {
        const uint8_t* row = A + m * lda_bytes;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if constexpr (ES == 1) bits[i] = row[off[i]];
            else bits[i] = *reinterpret_cast<const uint16_t*>(row + off[i]);
        }
    };
    if (threadIdx.x < M) load_row(threadIdx.x);
    for (int64_t m = threadIdx.x; m < M; m += 256) {
        sum_t x[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = search_magnitude<DT>(bits[i]);
        if (TOGETHER && m - threadIdx.x + 256 <= M) __syncthreads();      // (every lane has such a row)
        if (m + 256 < M) load_row(m + 256);
        // the arithmetic is 343 instructions of eight bytes: a row took 5 - 13 % longer where they lay across eight-byte
        // boundaries (32768 x 64 8-bit floats 563 against 637 us a sweep)
        __builtin_amdgcn_sched_barrier(0);
        asm volatile(".p2align 3");
        __builtin_amdgcn_sched_barrier(0);
        sum_t pair[8][8];
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = i + 1; j < 8; ++j) pair[i][j] = x[i] + x[j];
        // the larger of (a, d) and (b, d), shared by the sets that differ in c
        sum_t to_d[8][8][8];
#pragma unroll
        for (int a = 0; a < 8; ++a)
#pragma unroll
            for (int b = a + 1; b < 8; ++b)
#pragma unroll
                for (int d = b + 2; d < 8; ++d) to_d[a][b][d] = larger(pair[a][d], pair[b][d]);
        int s = 0;
#pragma unroll
        for (int a = 0; a < 8; ++a)
#pragma unroll
            for (int b = a + 1; b < 8; ++b)
#pragma unroll
                for (int c = b + 1; c < 7; ++c) {
                    const sum_t abc = larger(larger(pair[a][b], pair[a][c]), pair[b][c]);
#pragma unroll
                    for (int d = c + 1; d < 8; ++d) acc[s++] += larger(larger(abc, pair[c][d]), to_d[a][b][d]);   // lexicographic order of (a, b, c, d)
                }
    }

    // the 256 partial sums as a binary tree over neighbours: inside a wavefront by halving, which leaves two scores to a lane
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int first = 0, n = 70;
    double v70[70], v35[35], v18[18], v9[9], v5[5], v3[3], v2[2];
#pragma unroll
    for (int s = 0; s < 70; ++s) v70[s] = (double)acc[s];
    halve<70, 1>(v70, v35, lane, first, n);
    halve<35, 2>(v35, v18, lane, first, n);
    halve<18, 4>(v18, v9, lane, first, n);
    halve<9, 8>(v9, v5, lane, first, n);
    halve<5, 16>(v5, v3, lane, first, n);
    halve<3, 32>(v3, v2, lane, first, n);
    for (int k = 0; k < 2; ++k)
        if (k < n) part[wave][first + k] = v2[k];
    __syncthreads();
    // lane k of the first wavefront: the sum of way k -- sets of four in lexicographic order, 0 .. 34 hold position 0 and
    // the complement of set k is set 69 - k; then the largest sum, the lowest way among equals
    if (wave == 0) {
        double sum = -1.0;
        if (lane < 35) {
            const int o = 69 - lane;
            const double mine = (part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]);
            const double other = (part[0][o] + part[1][o]) + (part[2][o] + part[3][o]);
            sum = mine + other;
        }
        double best = sum;
#pragma unroll
        for (int w = 1; w < 64; w *= 2) best = __builtin_fmax(best, __shfl_xor(best, w, 64));
        const uint64_t at = __ballot(sum == best);
        if (lane == 0) winner = __builtin_ctzll(at);
    }
    __syncthreads();
    const int arg = __builtin_amdgcn_readfirstlane(winner);
    if (arg != 0 && threadIdx.x < 8) {
        // position threadIdx.x of the new arrangement: the winner's four positions, then the other four, ascending
        const int i = threadIdx.x;
        const uint32_t mine = way_mask(arg);
        const int src = nth_bit(i < 4 ? mine : mine ^ 0xFFu, i & 3);
        int32_t c = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) c = (src == j) ? col[j] : c;
        perm[4 * (i < 4 ? g : h) + (i & 3)] = c;
    }
}

sp24_status launch_permute_search(const void* A, int32_t* perm, int64_t M, int64_t K, int64_t lda, sp24_dtype t, int sweeps, hipStream_t st)
{
    const int64_t G = K / 4;
    int rounds = 0;
    while (((int64_t)1 << rounds) < G) ++rounds;
    if (M == 0 || rounds == 0) return SP24_OK;
    const int es = esize_of(t);
    const dim3 block(256);
    const uint8_t* a = static_cast<const uint8_t*>(A);
    // 256 rows of 8 KiB are half an L2; with fewer rows, or shorter ones, the barrier costs a sweep from the order of memory
    // more than it gives the others (4096 x 11008 bf16 1788 -> 1961 us, 8192 x 4096 8-bit floats 886 -> 1044).  Not for int8,
    // whose sums are 32-bit (8192 x 8192 from an arbitrary order 6430 -> 7255).
    const bool together = M >= 8192 && K * es >= 8192;
    for (int sweep = 0; sweep < sweeps; ++sweep)
        for (int r = 0; r < rounds; ++r) {
            // the pairs of the round, one for each group below G with bit r set.  No more workgroups than that: each XCD has an
            // eighth of the ids, in order, so that ids without a pair left the last XCDs idle where G is no power of two
            // (4096 x 11008 int8 2066 -> 1402 us a sweep, bf16 2836 -> 1788)
            const int64_t pairs = ((G >> (r + 1)) << r) + std::max<int64_t>(0, (G & (((int64_t)2 << r) - 1)) - ((int64_t)1 << r));
            const dim3 grid((unsigned)pairs);
            auto run = [&](auto kernel) { kernel<<<grid, block, 0, st>>>(a, perm, M, K, lda * es, r); };
            if (t == SP24_F16) together ? run(k_permute_search_round<SP24_F16, true>) : run(k_permute_search_round<SP24_F16, false>);
            else if (t == SP24_BF16) together ? run(k_permute_search_round<SP24_BF16, true>) : run(k_permute_search_round<SP24_BF16, false>);
            else if (t == SP24_F8) together ? run(k_permute_search_round<SP24_F8, true>) : run(k_permute_search_round<SP24_F8, false>);
            else run(k_permute_search_round<SP24_I8, false>);
            if (hipGetLastError() != hipSuccess) return SP24_ERR_LAUNCH;
        }
    return SP24_OK;
}

} // namespace sp24
