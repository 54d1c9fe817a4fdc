// The search for a column order (permute_search.hip states the method and the order of every sum) on a copy of the
// matrix that lies column by column, in a workspace of the caller's.
//
// What bounded a round in place (4096 x 1024 bf16: 20.8 us, 128 workgroups): a lane is a row, so that each load of a
// column's 64 values touched 64 cache lines, and 343 binary64 instructions a row on half of the compute units.  Here
//
//   * one pass lays the magnitudes out as [column][pair of row blocks][256 lanes][2 rows], 16 bits each (int8 as the
//     magnitude, 8-bit floats as the bf16 of the same value, NaN as infinity): a wavefront's load is 256 consecutive
//     bytes and brings two rows.  8 MB in, 8 MB out, once a call;
//   * a group of four's two largest magnitudes are taken from triples: with two(abc) the sum of the two largest of three
//     and one(abc) the largest, it is max(two(abc), one(abc) + d).  Twenty triples, three operations each, cover the 70
//     groups (as few as can: the Turan number T(8, 4, 3)), seven pairs the triples: 284 operations a row;
//   * the 35 ways of a pair are shared out to one, two or four workgroups (Deal below), each of which adds all rows for
//     its own ways, so that few pairs occupy the chip; no sum is split, and every sum keeps its order;
//   * no workgroup waits for the others of its pair: each leaves its best way and that way's sum behind, and
//     the next round's workgroups, which need the outcome of two pairs, pick the better of the records when they start;
//   * the lanes are numbered so that the first, longest steps of the tree are gfx950's v_permlane32_swap and
//     v_permlane16_swap, which exchange exactly the halves that the halving keeps.
//
// Measured (us a sweep, in place -> here): 4096 x 1024 bf16 179 -> 96 (a round 20.8 -> 10.9, of which the arithmetic is 4.3), int8 162 -> 76;
// 8192 x 8192 bf16 2405 -> 1030, from an arbitrary order 10446 -> 1030; 1024 x 512 68 -> 45; 64 x 128 level.
//
// int8 magnitudes are summed two rows at a time in packed 16-bit arithmetic (exact; moved to 32 bits every 254 rows of a lane).
#include <algorithm>

#include "common.hpp"
#include "launch.hpp"
#include "permute_search.hpp"

namespace sp24 {

namespace {

// The workgroups of a pair: their ways, and the triples and pairs of positions that their sums are made from.  Found by
// a search for the fewest operations: 284 a row in one part, 146 and 145 in two, 74 - 81 in each of four.
struct Part {
    uint64_t ways;            // bit w: way w is this part's
    int triples, pairs;
    uint8_t triple[20], pair[7];
};
template <int PARTS> struct Deal;
template <> struct Deal<1> {
    static constexpr Part part[1] = {
        {(1ull << 35) - 1, 20, 7,
         {0x85, 0x1a, 0xc8, 0xa2, 0x64, 0x51, 0x29, 0x34, 0x07, 0x4a, 0x98, 0x70, 0x92, 0x54, 0xc2, 0x61, 0x0d, 0x2c, 0x8a, 0x31},
         {0x82, 0x05, 0x21, 0x24, 0x50, 0x0a, 0x88}}};
};
constexpr uint64_t ways_of(std::initializer_list<int> list)
{
    uint64_t mask = 0;
    for (int w : list) mask |= 1ull << w;
    return mask;
}
template <> struct Deal<2> {
    static constexpr Part part[2] = {
        {ways_of({0, 1, 2, 3, 4, 7, 11, 16, 17, 19, 21, 23, 26, 27, 28, 30, 32, 33}), 10, 4,
         {0x68, 0x07, 0x91, 0x26, 0xb0, 0x49, 0x25, 0x4a, 0xd0, 0x86}, {0x06, 0x48, 0x90, 0x05}},
        {ways_of({5, 6, 8, 9, 10, 12, 13, 14, 15, 18, 20, 22, 24, 25, 29, 31, 34}), 11, 5,
         {0xc4, 0x1c, 0x61, 0x8a, 0x29, 0x54, 0x32, 0x8c, 0x83, 0x13, 0xc2}, {0x82, 0x21, 0x12, 0x0c, 0x44}}};
};
template <> struct Deal<4> {
    static constexpr Part part[4] = {
        {ways_of({0, 3, 7, 8, 14, 16, 18, 27, 29}), 7, 3, {0x89, 0xb0, 0x52, 0x43, 0x34, 0x0d, 0x46}, {0x42, 0x09, 0x30}},
        {ways_of({1, 4, 5, 11, 25, 26, 28, 31, 32}), 7, 3, {0x86, 0x68, 0x31, 0x13, 0x19, 0x4c, 0xa4}, {0x11, 0x84, 0x48}},
        {ways_of({6, 13, 15, 17, 20, 21, 24, 33, 34}), 6, 3, {0x2a, 0x1c, 0xa2, 0x45, 0x94, 0xc1}, {0x41, 0x22, 0x14}},
        {ways_of({2, 9, 10, 12, 19, 22, 23, 30}), 6, 4, {0xc8, 0x25, 0x8c, 0x43, 0x32, 0x1a}, {0x12, 0x88, 0x03, 0x05}}};
};

// Score s of a part: its s / 2-th way's group with position 0 (s even) or the other group
constexpr int score_count(const Part& p) { return 2 * __builtin_popcountll(p.ways); }
constexpr uint32_t score_mask(const Part& p, int s)
{
    uint64_t ways = p.ways;
    for (int i = 0; i < s / 2; ++i) ways &= ways - 1;
    const uint32_t mask = way_mask(__builtin_ctzll(ways));
    return s % 2 ? mask ^ 0xFFu : mask;
}
// the first triple (pair) of the part that lies in the mask, or -1
constexpr int triple_in(const Part& p, uint32_t mask)
{
    for (int t = 0; t < p.triples; ++t)
        if ((p.triple[t] & mask) == p.triple[t]) return t;
    return -1;
}
constexpr int pair_in(const Part& p, uint32_t mask)
{
    for (int t = 0; t < p.pairs; ++t)
        if ((p.pair[t] & mask) == p.pair[t]) return t;
    return -1;
}
template <int PARTS>
constexpr bool deal_is_complete()
{
    uint64_t all = 0;
    for (const Part& p : Deal<PARTS>::part) {
        if (all & p.ways) return false;
        all |= p.ways;
        for (int s = 0; s < score_count(p); ++s)
            if (triple_in(p, score_mask(p, s)) < 0) return false;
        for (int t = 0; t < p.triples; ++t)
            if (pair_in(p, p.triple[t]) < 0) return false;
    }
    return all == (1ull << 35) - 1;
}
static_assert(deal_is_complete<1>() && deal_is_complete<2>() && deal_is_complete<4>(), "every way once, every group from a triple, every triple from a pair");

template <typename F, int... I>
__device__ __forceinline__ void each_of(F f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void each(F f) { each_of(f, std::make_integer_sequence<int, N>{}); }

// the scores of one row (of two, packed) added to the part's sums
template <int PARTS, int PART, typename V, int N>
__device__ __forceinline__ void add_row(const V (&x)[8], V (&acc)[N])
{
    constexpr Part p = Deal<PARTS>::part[PART];
    V sum[p.pairs], most[p.pairs], two[p.triples], one[p.triples];
    each<p.pairs>([&](auto i) {
        constexpr int a = __builtin_ctz(p.pair[i]), b = 31 - __builtin_clz(p.pair[i]);
        sum[i] = x[a] + x[b];
        most[i] = larger(x[a], x[b]);
    });
    each<p.triples>([&](auto i) {
        constexpr int base = pair_in(p, p.triple[i]), c = __builtin_ctz(p.triple[i] ^ p.pair[base]);
        two[i] = larger(sum[base], most[base] + x[c]);
        one[i] = larger(most[base], x[c]);
    });
    each<N>([&](auto i) {
        constexpr int base = triple_in(p, score_mask(p, i)), d = __builtin_ctz(score_mask(p, i) ^ p.triple[base]);
        acc[i] += larger(two[base], one[base] + x[d]);
    });
}

// ---- the layout ----------------------------------------------------------------------------------------------

// Row of the 64 of a wavefront that hardware lane s holds: the tree's neighbours (bit 0, 1, ..) are 32, 16, 2, 1, 8 and 4
// lanes apart
__device__ __forceinline__ int row_of_lane(int s)
{
    return (s >> 5 & 1) | (s >> 4 & 1) << 1 | (s >> 1 & 1) << 2 | (s & 1) << 3 | (s >> 3 & 1) << 4 | (s >> 2 & 1) << 5;
}

// 16 bits that stand for the magnitude of an element
template <int DT>
__device__ __forceinline__ uint32_t stored_magnitude(uint32_t bits)
{
    if constexpr (DT == SP24_I8) return mag_key8(bits);
    else if constexpr (DT == SP24_F8) return __float_as_uint(magnitude_f8(bits)) >> 16;
    else return min(bits & 0x7FFFu, DT == SP24_F16 ? 0x7C00u : 0x7F80u);
}

} // namespace

// T[column][block][lane slot] = rows m (low half) and m + 256 (high half), m = 512 block + 64 wavefront + row_of_lane; rows
// past M are zeros.  One workgroup: 64 columns of the 128 rows that one wavefront's slots hold of a block.  Bound by the
// bytes (rows of 128 bytes in, 256 out).
template <int DT>
__global__ __launch_bounds__(256) void k_search_magnitudes(const uint8_t* __restrict__ A, uint32_t* __restrict__ T, int64_t M, int64_t K,
                                                           int64_t lda_bytes, int64_t blocks, uint32_t column_blocks)
{
    constexpr int ES = is8<DT> ? 1 : 2;
    __shared__ uint32_t tile[64][65];
    const int64_t col0 = (int64_t)(blockIdx.x % column_blocks) * 64, rest = blockIdx.x / column_blocks;
    const int64_t block = rest >> 2, row0 = 512 * block + 64 * (rest & 3);
    const int c = threadIdx.x & 7;                             // eight columns; all of them before K, or none
    const bool inside = col0 + 8 * c < K;
    uint32_t raw[2][2][2 * ES];
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int hi = 0; hi < 2; ++hi) {
            const int64_t m = row0 + 32 * p + (threadIdx.x >> 3) + 256 * hi;
            using piece_t = typename std::conditional<ES == 2, uint4v, uint2v>::type;
            piece_t v{};
            if (inside && m < M) v = *reinterpret_cast<const piece_t*>(A + m * lda_bytes + (col0 + 8 * c) * ES);
#pragma unroll
            for (int i = 0; i < 2 * ES; ++i) raw[p][hi][i] = v[i];
        }
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int word = e * ES / 4, shift = 8 * ((e * ES) % 4);
            constexpr uint32_t element = ES == 2 ? 0xFFFFu : 0xFFu;
            tile[8 * c + e][32 * p + (threadIdx.x >> 3)] =
                stored_magnitude<DT>(raw[p][0][word] >> shift & element) | stored_magnitude<DT>(raw[p][1][word] >> shift & element) << 16;
        }
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, from = row_of_lane(lane);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int64_t col = col0 + 16 * wave + i;
        if (col < K) T[(col * blocks + block) * 256 + 64 * (rest & 3) + lane] = tile[16 * wave + i][from];
    }
}

// ---- the rounds ----------------------------------------------------------------------------------------------

namespace {

// What a workgroup leaves for the next round: the best of its ways (the lowest among equals) and its sum
struct Record {
    double sum;
    int64_t way;
};

// The rounds before the present one, `now` of them (all sweeps counted).  Round q pairs by bit q % rounds; it kept the
// columns that it started from and its records in slot q % (rounds + 1).  Every group is paired in round 0 or the last
// round of a sweep (only group G - 1 can miss round 0, and it has the top bit), so no one looks back further than `rounds`.
struct History {
    const int32_t* first;                                      // the order the search starts from
    int32_t* columns;                                          // [rounds + 1][K]
    Record* records;                                           // [rounds + 1][pairs][PARTS]
    int64_t K, G, pairs;                                       // pairs: room for a round's
    int rounds, now;
    __device__ __forceinline__ int slot(int q) const { return q % (rounds + 1); }
};

// The columns of group g, after all earlier rounds.  (An entry outside 0 .. K-1 is one of column 0 once it has been moved.)
template <int PARTS>
__device__ __forceinline__ void columns_of(const History& h, int64_t g, int32_t (&col)[4])
{
    for (int q = h.now - 1; q >= 0 && q >= h.now - h.rounds; --q) {
        const int64_t step = (int64_t)1 << (q % h.rounds), low = g & ~step, high = g | step;
        if (high >= h.G) continue;                             // not paired in that round
        const int64_t pair = (low >> 1 & -step) | (low & (step - 1));
        const int32_t* kept = h.columns + h.slot(q) * h.K;
        int32_t was[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) was[i] = kept[4 * (i < 4 ? low : high) + (i & 3)];
        const Record* rec = h.records + (h.slot(q) * h.pairs + pair) * PARTS;
        double best = rec[0].sum;
        int way = (int)rec[0].way;
#pragma unroll
        for (int p = 1; p < PARTS; ++p) {
            const double sum = rec[p].sum;
            const int other = (int)rec[p].way;
            const bool wins = sum > best || (sum == best && other < way);
            best = wins ? sum : best;
            way = wins ? other : way;
        }
        way = __builtin_amdgcn_readfirstlane(way);
        if (way == 0) {
#pragma unroll
            for (int i = 0; i < 4; ++i) col[i] = g == low ? was[i] : was[4 + i];
            return;
        }
        const uint32_t four = g == low ? way_mask(way) : way_mask(way) ^ 0xFFu;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int from = nth_bit(four, i);
            int32_t c = 0;
#pragma unroll
            for (int j = 0; j < 8; ++j) c = from == j ? was[j] : c;
            col[i] = (uint64_t)(uint32_t)c < (uint64_t)h.K ? c : 0;
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) col[i] = h.first[4 * g + i];
}

// x of the lane W away (1, 2, 4 or 8)
template <int W>
__device__ __forceinline__ double partner(double x)
{
    if constexpr (W == 4) return __shfl_xor(x, 4, 64);
    else {
        constexpr int ctrl = W == 1 ? 0xB1 : W == 2 ? 0x4E : 0x128;      // quad_perm [1,0,3,2], [2,3,0,1]; row_ror:8
        const uint2v v = __builtin_bit_cast(uint2v, x);
        const uint2v r = {(uint32_t)__builtin_amdgcn_mov_dpp((int)v[0], ctrl, 0xF, 0xF, true), (uint32_t)__builtin_amdgcn_mov_dpp((int)v[1], ctrl, 0xF, 0xF, true)};
        return __builtin_bit_cast(double, r);
    }
}

// One step of the halving: of L scores held, a lane with bit W of its number clear keeps the first half and adds its
// partner's, the other keeps the second half; first, n: the number of the first score held, and how many are scores (the
// rest is padding: the halves of an odd number differ by one).
template <int L, int W>
__device__ __forceinline__ void halve(const double (&v)[L], double (&kept)[(L + 1) / 2], int lane, int& first, int& n)
{
    constexpr int H = (L + 1) / 2;
    const bool up = (lane & W) != 0;
#pragma unroll
    for (int k = 0; k < H; ++k) {
        const double lower = v[k], upper = k + H < L ? v[k + H] : 0.0;
        if constexpr (W >= 16) {
            // the swap leaves the lower score of both partners in the lanes that keep it, and the upper one's in the others
            const uint2v a = __builtin_bit_cast(uint2v, lower), b = __builtin_bit_cast(uint2v, upper);
            uint2v mine, theirs;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const auto s = W == 32 ? __builtin_amdgcn_permlane32_swap(a[i], b[i], false, false) : __builtin_amdgcn_permlane16_swap(a[i], b[i], false, false);
                mine[i] = s[0];
                theirs[i] = s[1];
            }
            kept[k] = __builtin_bit_cast(double, mine) + __builtin_bit_cast(double, theirs);
        } else
            kept[k] = (up ? upper : lower) + partner<W>(up ? lower : upper);
    }
    first += up ? H : 0;
    n = up ? max(n - H, 0) : min(n, H);
}

} // namespace

// A part of a pair's ways over all rows.  DT: SP24_BF16, SP24_F16 or SP24_I8, how the magnitudes are stored.
template <int DT, int PARTS, int PART>
__device__ __forceinline__ void search_part(const uint32_t* T, const int32_t (&col)[8], int64_t M, int64_t blocks, Record* record, double (*sums)[72])
{
    constexpr Part P = Deal<PARTS>::part[PART];
    constexpr int N = score_count(P);
    const uint32_t* src[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) src[i] = T + col[i] * blocks * 256 + threadIdx.x;

    double total[N];
    uint32_t row[2][8];
    auto load = [&](uint32_t (&r)[8], int64_t block) {
#pragma unroll
        for (int i = 0; i < 8; ++i) r[i] = src[i][block * 256];
    };
    // two blocks ahead: a block's arithmetic is 0.6 us, a load that misses the L2 takes longer
    load(row[0], 0);
    load(row[1], min((int64_t)1, blocks - 1));
    if constexpr (DT == SP24_I8) {
        // packed halves hold 255 rows of at most 256; an even number of them, because of the two rows of `row`
        constexpr int kPacked = 254;
        static_assert(kPacked * 256 < 65536 && kPacked % 2 == 0, "no carry into the upper half; blocks b0, b0 + 2, .. lie in row[0]");
        int wide[N];
#pragma unroll
        for (int s = 0; s < N; ++s) wide[s] = 0;
        for (int64_t b0 = 0; b0 < blocks; b0 += kPacked) {
            ushort2v acc[N];
#pragma unroll
            for (int s = 0; s < N; ++s) acc[s] = ushort2v{0, 0};
            const int64_t end = min(b0 + kPacked, blocks);
            for (int64_t b = b0; b < end; b += 2) {
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    if (b + u < end) {
                        ushort2v x[8];
#pragma unroll
                        for (int i = 0; i < 8; ++i) x[i] = __builtin_bit_cast(ushort2v, row[u][i]);
                        load(row[u], min(b + u + 2, blocks - 1));
                        add_row<PARTS, PART>(x, acc);
                    }
                }
            }
#pragma unroll
            for (int s = 0; s < N; ++s) wide[s] += (int)acc[s][0] + (int)acc[s][1];
        }
#pragma unroll
        for (int s = 0; s < N; ++s) total[s] = (double)wide[s];
    } else {
#pragma unroll
        for (int s = 0; s < N; ++s) total[s] = 0.0;
        for (int64_t b = 0; b < blocks; b += 2) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (b + u < blocks) {
                    uint32_t now[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) now[i] = row[u][i];
                    load(row[u], min(b + u + 2, blocks - 1));
#pragma unroll
                    for (int half = 0; half < 2; ++half) {
                        if (half == 1 && 512 * (b + u) + 256 >= M) break;        // no row in the upper halves
                        double x[8];
#pragma unroll
                        for (int i = 0; i < 8; ++i) {
                            if constexpr (DT == SP24_F16) x[i] = (double)(float)__builtin_bit_cast(_Float16, (uint16_t)(half ? now[i] >> 16 : now[i]));
                            else x[i] = (double)__uint_as_float(half ? now[i] & 0xFFFF0000u : now[i] << 16);
                        }
                        add_row<PARTS, PART>(x, total);
                    }
                }
            }
        }
    }

    // the partial sums as a binary tree over neighbours: inside a wavefront by halving, which leaves a score or two to a lane
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int first = 0, n = N;
    constexpr int N1 = (N + 1) / 2, N2 = (N1 + 1) / 2, N3 = (N2 + 1) / 2, N4 = (N3 + 1) / 2, N5 = (N4 + 1) / 2, N6 = (N5 + 1) / 2;
    double v1[N1], v2[N2], v3[N3], v4[N4], v5[N5], v6[N6];
    halve<N, 32>(total, v1, lane, first, n);
    halve<N1, 16>(v1, v2, lane, first, n);
    halve<N2, 2>(v2, v3, lane, first, n);
    halve<N3, 1>(v3, v4, lane, first, n);
    halve<N4, 8>(v4, v5, lane, first, n);
    halve<N5, 4>(v5, v6, lane, first, n);
#pragma unroll
    for (int k = 0; k < N6; ++k)
        if (k < n) sums[wave][first + k] = v6[k];
    __syncthreads();
    // lane w of the first wavefront: the sum of way w; then the largest, the lowest way among equals
    if (wave == 0) {
        double sum = -1.0;
        if (lane < 35 && (P.ways >> lane & 1)) {
            const int s = 2 * __builtin_popcountll(P.ways & ((1ull << lane) - 1));
            const double mine = (sums[0][s] + sums[1][s]) + (sums[2][s] + sums[3][s]);
            const double other = (sums[0][s + 1] + sums[1][s + 1]) + (sums[2][s + 1] + sums[3][s + 1]);
            sum = mine + other;
        }
        double best = sum;
#pragma unroll
        for (int w = 1; w < 64; w *= 2) best = __builtin_fmax(best, __shfl_xor(best, w, 64));
        const uint64_t at = __ballot(sum == best);
        if (lane == 0) *record = Record{best, __builtin_ctzll(at)};
    }
}

template <int DT, int PARTS>
__global__ __launch_bounds__(256) void k_search_round(const uint32_t* __restrict__ T, History h, int64_t M, int64_t blocks)
{
    __shared__ double sums[4][72];
    // (ids congruent mod 8 run on one XCD: each gets its eighth of the round's pairs, consecutive ones, the parts of a pair
    // behind each other, so that what they read together stays in its L2)
    const uint32_t xcd = blockIdx.x & 7, share = gridDim.x / 8, rest = gridDim.x % 8;
    const int64_t id = (int64_t)xcd * share + min(xcd, rest) + (blockIdx.x >> 3);
    const int64_t pair = id / PARTS;
    const int part = (int)(id % PARTS);
    const int bit = h.now % h.rounds;
    const int64_t step = (int64_t)1 << bit, low = (pair & -step) << 1 | (pair & (step - 1)), high = low | step;

    int32_t was[8], col[8];
    {
        int32_t four[4];
        columns_of<PARTS>(h, low, four);
#pragma unroll
        for (int i = 0; i < 4; ++i) was[i] = four[i];
        columns_of<PARTS>(h, high, four);
#pragma unroll
        for (int i = 0; i < 4; ++i) was[4 + i] = four[i];
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        was[i] = __builtin_amdgcn_readfirstlane(was[i]);
        col[i] = (uint64_t)(uint32_t)was[i] < (uint64_t)h.K ? was[i] : 0;      // never out of bounds
    }
    if (part == 0 && threadIdx.x == 0) {
        int32_t* kept = h.columns + h.slot(h.now) * h.K;
#pragma unroll
        for (int i = 0; i < 8; ++i) kept[4 * (i < 4 ? low : high) + (i & 3)] = was[i];
    }
    Record* record = h.records + (h.slot(h.now) * h.pairs + pair) * PARTS + part;
    each<PARTS>([&](auto p) {
        if (part == p) search_part<DT, PARTS, p>(T, col, M, blocks, record, sums);
    });
}

// the order found
template <int PARTS>
__global__ __launch_bounds__(64) void k_search_result(History h, int32_t* perm)
{
    const int64_t g = blockIdx.x;                              // (a wavefront to a group: columns_of is uniform)
    int32_t col[4];
    columns_of<PARTS>(h, g, col);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) perm[4 * g + i] = col[i];
    }
}

static int search_rounds(int64_t G)
{
    int rounds = 0;
    while (((int64_t)1 << rounds) < G) ++rounds;
    return rounds;
}
// pairs of the round of bit r: one for each group below G with that bit set
static int64_t round_pairs(int64_t G, int r)
{
    return ((G >> (r + 1)) << r) + std::max<int64_t>(0, (G & (((int64_t)2 << r) - 1)) - ((int64_t)1 << r));
}
constexpr int kMostParts = 4;

// the copy, then the rounds' columns, then their records
static size_t columns_offset(int64_t M, int64_t K) { return (size_t)K * ((M + 511) / 512) * 1024; }
static size_t records_offset(int64_t M, int64_t K) { return columns_offset(M, K) + (size_t)((search_rounds(K / 4) + 1) * K) * sizeof(int32_t); }

size_t permute_search_workspace(int64_t M, int64_t K, sp24_dtype t)
{
    if (M == 0 || search_rounds(K / 4) == 0) return 0;
    // a launch is less than 2^32 threads: the copy's 1024 to 64 columns and a block of 512 rows, and 512 to a pair
    const int64_t blocks = M / 512 + (M % 512 != 0), column_blocks = (K + 63) / 64;
    if (K >= (int64_t)1 << 26 || blocks > (((int64_t)1 << 22) - 1) / column_blocks) return 0;
    // Many pairs of few rows: a workgroup's start and end count, which are longer here (in place -> copy, from the order of memory: 64 x 4096
    // bf16 83 -> 102 us, 256 x 16384 334 -> 405, 512 x 16384 396 -> 443; 512 x 4096 122 -> 110, 1024 x 16384 583 -> 532).  int8 of fewer than 256 rows from 193 pairs
    // on, too (128 x 2048 57 -> 64; 256 x 2048 65 -> 64, 128 x 1024 51 -> 49), and two or three rounds, beside which the copy's two other launches
    // count (128 x 16 bf16 16.4 -> 17.5, 128 x 32 int8 21.9 -> 23.0; 256 x 32 25.0 -> 23.3)
    if (K / 8 > 256 && M <= (K / 8 > 1024 ? 512 : 256)) return 0;
    if (M < 256 && (K <= 32 || (t == SP24_I8 && K / 8 > 192))) return 0;
    return records_offset(M, K) + (size_t)(search_rounds(K / 4) + 1) * ((K / 4 + 1) / 2) * kMostParts * sizeof(Record);
}

template <int DT, int PARTS>
static sp24_status run_rounds(const uint32_t* T, History h, int32_t* perm, int64_t M, int64_t blocks, int sweeps, hipStream_t st)
{
    const int total = sweeps * h.rounds;
    for (; h.now < total; ++h.now) {
        k_search_round<DT, PARTS><<<dim3((unsigned)(round_pairs(h.G, h.now % h.rounds) * PARTS)), dim3(256), 0, st>>>(T, h, M, blocks);
        if (hipGetLastError() != hipSuccess) return SP24_ERR_LAUNCH;
    }
    k_search_result<PARTS><<<dim3((unsigned)h.G), dim3(64), 0, st>>>(h, perm);
    return hipGetLastError() == hipSuccess ? SP24_OK : SP24_ERR_LAUNCH;
}

sp24_status launch_permute_search_columns(const void* A, int32_t* perm, int64_t M, int64_t K, int64_t lda, sp24_dtype t, int sweeps, void* workspace,
                                          hipStream_t st)
{
    const int64_t G = K / 4, blocks = (M + 511) / 512, column_blocks = (K + 63) / 64;
    const int rounds = search_rounds(G);
    if (M == 0 || rounds == 0 || sweeps == 0) return SP24_OK;
    uint8_t* ws = static_cast<uint8_t*>(workspace);
    uint32_t* T = reinterpret_cast<uint32_t*>(ws);
    const dim3 grid((unsigned)(column_blocks * blocks * 4)), block(256);
    auto copy = [&](auto kernel) {
        kernel<<<grid, block, 0, st>>>(static_cast<const uint8_t*>(A), T, M, K, lda * esize_of(t), blocks, (uint32_t)column_blocks);
    };
    if (t == SP24_F16) copy(k_search_magnitudes<SP24_F16>);
    else if (t == SP24_BF16) copy(k_search_magnitudes<SP24_BF16>);
    else if (t == SP24_F8) copy(k_search_magnitudes<SP24_F8>);
    else copy(k_search_magnitudes<SP24_I8>);
    if (hipGetLastError() != hipSuccess) return SP24_ERR_LAUNCH;
    const History h{perm, reinterpret_cast<int32_t*>(ws + columns_offset(M, K)), reinterpret_cast<Record*>(ws + records_offset(M, K)), K, G, (G + 1) / 2, rounds, 0};
    // As many parts as leave the workgroups of a round room on the chip at once (4096 x 512 bf16 in one, two and four parts: 116, 81 and
    // 70 us a sweep, 4096 x 1024: 133, 96 and 106; 2048 x 2048, 256 pairs: 103, 107 and 126, with 16 rows 57, 63 and 77), and two again where float workgroups
    // outnumber the units: one holds 276 registers, which leaves a wavefront to a SIMD, each of two 178 (4096 x 11008: 945 -> 789; 300 x 2560
    // 97 -> 89, 600 x 16384 529 -> 497; 512 x 4096 115 and 119, 768 x 4096 132 and 135, 512 x 6144 168 and 171, 1024 x 4096 level; int8 501 and 498)
    const int64_t pairs = G / 2;
    const bool two_again = t != SP24_I8 && pairs > 256 && (M >= 1024 || pairs <= 448 || (pairs >= 1024 && M > 512));
    const int parts = pairs <= 64 ? 4 : pairs <= 192 || two_again ? 2 : 1;
    auto run = [&](auto dt) {
        constexpr int DT = decltype(dt)::value;
        if (parts == 4) return run_rounds<DT, 4>(T, h, perm, M, blocks, sweeps, st);
        if (parts == 2) return run_rounds<DT, 2>(T, h, perm, M, blocks, sweeps, st);
        return run_rounds<DT, 1>(T, h, perm, M, blocks, sweeps, st);
    };
    if (t == SP24_F16) return run(std::integral_constant<int, SP24_F16>{});
    if (t == SP24_I8) return run(std::integral_constant<int, SP24_I8>{});
    return run(std::integral_constant<int, SP24_BF16>{});
}

} // namespace sp24
