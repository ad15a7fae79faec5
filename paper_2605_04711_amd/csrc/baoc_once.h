// Finalize with one read of v and theta.  Included by baoc_profile.hip, whose helpers it uses.
#pragma once

namespace baoc {

// ---------------------------------------------------------------------------
// Finalize in one pass
//   k_bracket:     per block of several tasks, an interval of keys around each quantile and a typical p, from a sample of v
//   k_once:        the pass; a block of one task is finished by it
//   k_once_select: the order statistics from the keys that lay in the intervals, the sums; leaves the records
// What the passes above read v twice for, and how it is had from one read:
//   Eq. 4  The quantiles' first digits are not known in advance, but a sample of 16,384 coordinates places them within 1.2 % of the
//          ranks: keys inside the two intervals are listed, those below are counted.  Equal keys: zeros lie below every interval; an
//          interval of at most 512 keys is counted key by key and not listed; of more keys in a rank's bins than can be ordered, k_once_select
//          counts those of 256 to 1,024 cells of the bins, and a cell of one value gives the rank, one of several another walk over the lists.
//          Where a rank turns out to lie outside its interval, the lists are too short, or a sum is not finite, the block is marked and goes through
//          the passes above.
//          (Which keys are listed where is not the same from run to run; what is taken from them is, and so is what is marked.)
//   Eq. 6  With q = p / p0 - 1 for a fixed p0, sum ((p/p-bar - 1) theta)^2 = k^2 sum (q theta)^2 + 2 k (k-1) sum q theta^2 +
//          (k-1)^2 sum theta^2, k = p0 / p-bar.  For k well above 1 the terms are k^2 times their sum, so a rare large p (v = 0 at a
//          coordinate or two) must not raise p0: it is the median of the means of 16 parts of the sample, and the mean of all p where one
//          workgroup has the block.  Where the terms cancel all the same (distortion_cancels) the block is marked.
//   Eq. 7  |S - r c^T / mu|^2 = |S|^2 - (2/mu) sum_j c_j t_j + |r|^2 |c|^2 / mu^2 with t = S^T r.  A workgroup reads whole rows, so
//          that r_i is there while the row still is in registers; everything is summed in fp64, products of fp32 numbers being exact
//          there, since for a rank-one S the three terms cancel.
// ---------------------------------------------------------------------------

constexpr uint32_t kOnceBins = 2048;                      // most bins of an interval's keys; both intervals' fill a block's histogram
static_assert(2 * kOnceBins == kHistWords, "two intervals");
constexpr uint32_t kOnceStage = 1280;                     // words per wavefront in which listed keys gather: what is there before a batch of 1,024
constexpr uint32_t kOnceKeys = 4096;                      // keys of an interval that k_once_select orders at most
constexpr float kLeastP0 = 1e-30f;                        // where every p is zero

typedef f4 f4_any __attribute__((aligned(4)));            // four elements at any alignment

struct OnceSums {                                         // of a task
    double q, a, b, d, s2, rho, r2, all;                  // rho = sum r^2 / sum r; all = sum v
    uint32_t n[2];                                        // keys below the two intervals
    uint32_t n_list, pad_;
};

struct OnceUnit { double cross, c2; };                    // of 64 columns: sum of c t, c^2

struct OnceMem {
    char* base;                                           // the region
    OnceSums* sums;
    OnceUnit* units;
    const OnceRow* rows;
    uint32_t n_blocks, narrow_tasks;                      // tasks of 8 wavefronts; those of 16 come after them
    uint32_t* line;
    uint32_t* hist;
    const double* rec;
    double* out;
};

__host__ __device__ __forceinline__ uint64_t once_cols_units(uint32_t tasks, uint32_t cols) { return ((uint64_t)tasks * cols * 8 + 63) / 64; }
constexpr uint32_t kOncePart = 8192;                      // words of a list that a wavefront of k_once_select takes
__host__ __device__ __forceinline__ uint32_t once_parts(uint32_t cap) { return (cap + kOncePart - 1) / kOncePart; }
__host__ __device__ __forceinline__ uint32_t once_spill(const OnceRow& o) { return o.n_tasks * o.list_cap / 32 * 16; }   // words of the common list: half of the tasks'
__host__ __device__ __forceinline__ uint32_t once_list_units(const OnceRow& o) { return (uint32_t)(((uint64_t)o.n_tasks * once_parts(o.list_cap) + once_parts(once_spill(o)) + 3) / 4); }
__host__ __device__ __forceinline__ uint32_t once_col_units(uint32_t rows, uint32_t cols) { return rows ? (cols + 63) / 64 : 0u; }
__host__ __device__ __forceinline__ uint32_t once_keys_cap(uint64_t numel) { return (uint32_t)max((uint64_t)1024, min((uint64_t)kOnceKeys, numel >> 10)); }

// Pieces of four coordinates that a thread of k_bracket samples: 8,192 to 65,536 coordinates of a block; and the share of a block's keys
// that then lies in its two intervals, 5 standard deviations of the sample's rank to either side of a quantile.
// (Each piece is a cache line: with 16,384 coordinates of blocks of 2.4 M the sample moves a twentieth of v, 400 of them 55 us instead of 34, and
// the lists are a third shorter, which is worth less.)
__host__ __device__ __forceinline__ uint32_t sample_pieces(uint64_t numel)
{
    return numel >= (1u << 27) ? 16u : numel >= (1u << 26) ? 8u : numel >= (1u << 22) ? 4u : 2u;
}
constexpr float kListSlack = 1.2f;                        // a block's lists have at least this much more room
inline double listed_share(uint64_t numel) { return 2.0 * 2.0 * 1.5 / std::sqrt(4096.0 * sample_pieces(numel)); }

// Where a load of 1 << rpl rows starts that wants `row` and those after it, and a lane that wants four columns from `col` on: rows past the
// matrix are its last ones again, columns past a row likewise, so that no load is left out and none leaves its row.  What is read twice is skipped:
// the first once_skip() of the lane's four elements.  (Host code as well, for the tests.)
__host__ __device__ __forceinline__ uint32_t once_first_row(uint32_t row, uint32_t rpl, uint32_t rows) { return min(row, rows - (1u << rpl)); }
__host__ __device__ __forceinline__ uint32_t once_first_col(uint32_t col, uint32_t cols) { return min(col, cols - 4); }
__host__ __device__ __forceinline__ uint32_t once_skip(uint32_t row, uint32_t lrow, uint32_t rpl, uint32_t rows, uint32_t col, uint32_t cols)
{
    return once_first_row(row, rpl, rows) + lrow < row ? 4u : col - once_first_col(col, cols);
}

// The block that owns task or unit `id`: the last with first(block) <= id.  A wavefront looks at 64 blocks at a time.
template <typename Fn> __device__ __forceinline__ uint32_t find_owner(uint32_t n, uint32_t id, uint32_t lane, Fn first)
{
    uint32_t lo = 0, len = n;
    while (len > 1) {
        const uint32_t step = (len + 63) / 64, at = lane * step;
        const uint64_t below = __builtin_amdgcn_ballot_w64(at < len && first(lo + min(at, len - 1)) <= id);
        const uint32_t j = (uint32_t)__builtin_popcountll(below) - 1u;
        lo += j * step; len = min(step, len - j * step);
    }
    return scalar_u32(lo);
}

// An interval of a small block has fewer bins, since every task adds all of its own to the block's: a bin is left with about a hundred keys.
__host__ __device__ __forceinline__ uint32_t once_bins_log(uint32_t numel) { return min(11u, max(7u, 19u - (uint32_t)__builtin_clz(numel))); }
__host__ __device__ __forceinline__ uint32_t once_slots_log(uint32_t bins_log) { return max(9u, bins_log); }   // words of an interval in the histogram
static_assert(kOnceBins == 1u << 11, "once_bins_log");

// Shift that leaves 1 << n_log of `width` keys; and that of an interval, none where it has the keys of one prefix of two digits.
__host__ __device__ __forceinline__ uint32_t width_shift(uint32_t width, uint32_t n_log)
{
    const uint32_t bits = width > 1 ? 32u - (uint32_t)__builtin_clz(width - 1) : 0u;
    return bits > n_log ? bits - n_log : 0u;
}
__host__ __device__ __forceinline__ uint32_t once_shift(uint32_t width, uint32_t bins_log) { return width <= 1u << kBits3 ? 0u : width_shift(width, bins_log); }

// Where k_once_select collects a block's keys: those of the lower interval, then those of the upper one.  Of more keys than can be ordered, the
// range's cells: counts, largest keys and complements of the smallest ones, 1 << once_cells_log() words each.
__device__ __forceinline__ uint32_t* once_found(const OnceMem& mem, const OnceRow& o, uint32_t cols)
{
    return reinterpret_cast<uint32_t*>(mem.base + ((uint64_t)o.off_cols + once_cols_units(o.n_tasks, cols)) * 64);
}
__host__ __device__ __forceinline__ uint32_t once_cells_log(uint32_t keys_cap) { return 29u - (uint32_t)__builtin_clz(keys_cap); }
static_assert(kOnceKeys == 1u << 12, "1,024 cells at most");

// The intervals of a block from the two-digit prefixes at the ends of its quantiles' ranks: [end[0], end[1]) and [end[2], end[3]).  Zeros are
// below.  Where they overlap most of the block has one prefix; both quantiles then are in one interval, the second is empty, and that interval
// must leave zeros out or hold one prefix: false if not, or if there are values without order.
__host__ __device__ __forceinline__ bool once_intervals(const uint32_t (&prefix)[4], uint32_t (&end)[4])
{
    end[0] = max(prefix[0] << kBits3, 1u); end[1] = (prefix[1] + 1) << kBits3;
    end[2] = max(prefix[2] << kBits3, 1u); end[3] = (prefix[3] + 1) << kBits3;
    if (end[3] > 0x7f800000u) return false;
    if (end[1] <= end[2]) return true;
    end[1] = end[2] = end[3];
    return prefix[2] == 0 || prefix[0] == prefix[3];
}

// The keys at four ranks of what `walk` hands out, exactly.  h: kHistWords words of LDS; sel: eight words of LDS, of which the first
// four hold the keys' patterns in the end, or their first two digits.  Called by a whole workgroup of at least 256.
template <uint32_t THREADS, bool WHOLE, typename W>
__device__ __forceinline__ void order_stats(W walk, const uint32_t (&rank)[4], uint32_t* h, uint32_t* sel, uint32_t* sums, uint32_t lane, uint32_t wave)
{
    const uint32_t tid = threadIdx.x;
    auto clear = [&](uint32_t n) {
        __syncthreads();
        for (uint32_t i = tid; i < n; i += THREADS) h[i] = 0;
        __syncthreads();
    };
    clear(kBins1);
    walk([&](uint32_t key) { atomicAdd(&h[key >> kShift1], 1u); });
    __syncthreads();
    {
        uint32_t c[kBinsPerLane], mine = 0, incl = 0;
        if (tid < 256) {
            load_bins(c, h + tid * kBinsPerLane);
#pragma unroll
            for (uint32_t i = 0; i < kBinsPerLane; ++i) mine += c[i];
            incl = wave_scan(mine);
            if (lane == 63) sums[wave] = incl;
        }
        __syncthreads();
        if (tid < 256) {
            uint32_t at = incl - mine;
            for (uint32_t w = 0; w < wave; ++w) at += sums[w];
#pragma unroll
            for (uint32_t t = 0; t < 4; ++t)
                if (rank[t] >= at && rank[t] - at < mine) {
                    const Digit f = bin_of(c, tid * kBinsPerLane, at, rank[t]);
                    sel[t] = f.bin; sel[4 + t] = f.rank;
                }
        }
    }
    auto next = [&](auto last) {
        constexpr bool LAST = decltype(last)::value;
        constexpr uint32_t NB = LAST ? kBins3 : kBins2, BITS = LAST ? kBits3 : kBits2, SHIFT = LAST ? 0 : kShift2, N = NB / 64;
        clear(4 * NB);
        const Prefixes d = distinct_prefixes(sel, 0);
        walk([&](uint32_t key) { count_match(h, d, NB, key >> (SHIFT + BITS), (key >> SHIFT) & (NB - 1)); });
        __syncthreads();
        uint32_t key = 0, rank_in = 0;
        bool found = false;
        if (wave < 4) {
            const uint32_t slot = wave == 0 ? d.slot_of[0] : (wave == 1 ? d.slot_of[1] : (wave == 2 ? d.slot_of[2] : d.slot_of[3]));
            const uint32_t want = sel[4 + wave], prefix = sel[wave];
            uint32_t c[N], mine = 0;
            load_bins(c, h + slot * NB + lane * N);
#pragma unroll
            for (uint32_t i = 0; i < N; ++i) mine += c[i];
            const uint32_t at = wave_scan(mine) - mine;
            if (want >= at && want - at < mine) {
                const Digit f = bin_of(c, lane * N, at, want);
                key = (prefix << BITS) | f.bin; rank_in = f.rank; found = true;
            }
        }
        __syncthreads();
        if (found) { sel[wave] = key; sel[4 + wave] = rank_in; }
    };
    next(std::false_type());
    if (WHOLE) next(std::true_type());
    __syncthreads();
}

// ---------------------------------------------------------------------------

__device__ __forceinline__ double wave_total(double x)
{
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) x += __shfl_xor(x, d);
    return x;
}

// The pieces are drawn one from each of equal shares of the block, independently.  An interval reaches 5 standard deviations of the sample's rank to
// either side, at the resolution of two digits.  The four coordinates of a piece are neighbours and may be alike (kernels, rows, neurons of different
// scale), which gives a rank up to twice the deviation that independent coordinates would: it is estimated from how the counts differ from piece
// to piece, and where it is more than a tenth above the latter the intervals are taken again, at most as wide as the lists have room for.  (240
// blocks of 1 M, 9 neighbours of one scale: 2 of them were marked without that, finalize 511 us, 460 so.)
// Zeros are left out of an interval and counted as below: a quantile of a block with untouched coordinates is then known to be 0 however many there are.
// Bound by latency (loads, two rounds of counting) up to about 100 blocks, 23 us, then by the lines.
__global__ __launch_bounds__(1024) void k_bracket(const float* __restrict__ v_all, const TileRow* __restrict__ tiles, OnceMem mem, float eps)
{
    __shared__ alignas(16) uint32_t h[kHistWords];
    __shared__ uint32_t sel[8], sums[4], moment[4];
    __shared__ float sh[16];
    const uint32_t block = blockIdx.x, lane = threadIdx.x & 63u, wave = scalar_wave_index();
    if (mem.rows[block].n_tasks < 2) return;
    const TileRow& m = tiles[block];
    const uint32_t mine = sample_pieces(m.numel), pieces = 1024 * mine, n = 4 * pieces;
    const float* src = v_all + m.state_start;
    const uint32_t share = (uint32_t)(m.numel / pieces);
    f4 x[16];
    float psum = 0.f;
#pragma unroll
    for (uint32_t q = 0; q < 16; ++q) {
        x[q] = f4{0.f, 0.f, 0.f, 0.f};
        if (q < mine) {
            const uint32_t piece = q * 1024 + lane * 16 + wave;   // a wavefront's lie all over the block
            uint32_t z = (piece + 1) * 0x9E3779B9u;
            z ^= z >> 16; z *= 0x85EBCA6Bu; z ^= z >> 13; z *= 0xC2B2AE35u; z ^= z >> 16;
            uint32_t at = piece * share + (uint32_t)(((uint64_t)z * share) >> 32);
            at = min(at, (uint32_t)m.numel - 4) & ~3u;
            x[q] = *reinterpret_cast<const f4*>(src + at);
        }
    }
#pragma unroll
    for (uint32_t q = 0; q < 16; ++q)
        if (q < mine) psum += (preconditioner(x[q].x, eps) + preconditioner(x[q].y, eps)) + (preconditioner(x[q].z, eps) + preconditioner(x[q].w, eps));
    const float wave_p = wave_sum(psum);
    if (lane == 0) sh[wave] = wave_p;                         // order_stats has barriers
    auto of_piece = [&](uint32_t q, auto f) {
        const float e[4] = {x[q].x, x[q].y, x[q].z, x[q].w};   // (a bit cast of a vector's element takes the first one)
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) f(__builtin_bit_cast(uint32_t, e[k]) & 0x7fffffffu);
    };
    auto walk = [&](auto f) {
#pragma unroll
        for (uint32_t q = 0; q < 16; ++q)
            if (q < mine) of_piece(q, f);
    };
    const OnceRow& o = mem.rows[block];
    const uint32_t lo = n / 10, hi = n - 1 - n / 10;
    const float spread = 1.5f * __builtin_amdgcn_sqrtf((float)n);           // 5 sqrt(0.1 * 0.9 n)
    if (threadIdx.x < 4) moment[threadIdx.x] = 0;
    auto ends = [&](float reach) {
        const uint32_t d = (uint32_t)reach + 1, rank[4] = {lo - d, lo + d, hi - d, hi + d};
        order_stats<1024, false>(walk, rank, h, sel, sums, lane, wave);
    };
    ends(spread);
    // Keys below the inner ends, of all pieces: their number and the sum of the squares of a piece's.
    const uint32_t inner[2] = {(sel[1] + 1) << kBits3, sel[2] << kBits3};
#pragma unroll
    for (uint32_t t = 0; t < 2; ++t) {
        uint32_t first = 0, second = 0;
#pragma unroll
        for (uint32_t q = 0; q < 16; ++q)
            if (q < mine) {
                uint32_t c = 0;
                of_piece(q, [&](uint32_t key) { c += key < inner[t]; });
                first += c; second += c * c;
            }
        first = wave_scan(first); second = wave_scan(second);
        if (lane == 63) { atomicAdd(&moment[2 * t], first); atomicAdd(&moment[2 * t + 1], second); }
    }
    __syncthreads();
    float more = 0.f;                                         // times the variance of independent coordinates
#pragma unroll
    for (uint32_t t = 0; t < 2; ++t) {
        const float first = (float)moment[2 * t], second = (float)moment[2 * t + 1];
        if (first > 0.f && first < (float)n) more = fmaxf(more, (second - first * (first / (float)pieces)) / (first * (1.0f - first / (float)n)));
    }
    // as wide as the lists have room for: two intervals, two sides, a quarter to spare (the share of alike neighbours between two ranks varies, too)
    const float room = (float)o.list_cap * (float)o.n_tasks * 1.5f / (float)m.numel * (float)n * 0.2f;
    const float wide = fminf(spread * __builtin_amdgcn_sqrtf(more), room);
    if (wide > 1.1f * spread) ends(wide);
    uint32_t* line = mem.line + block * kArriveStride;
    if (threadIdx.x < 16) {
        // the patterns' order is the values'
        const uint32_t own = __builtin_bit_cast(uint32_t, sh[threadIdx.x]);
        uint32_t below = 0;
        for (uint32_t w = 0; w < 16; ++w) {
            const uint32_t x = __builtin_bit_cast(uint32_t, sh[w]);
            below += x < own || (x == own && w < threadIdx.x);
        }
        if (below == 7) line[L_INV_P0] = __builtin_bit_cast(uint32_t, 1.0f / fmaxf(sh[threadIdx.x] / (float)(n / 16), kLeastP0));
    }
    if (threadIdx.x == 0) {
        const uint32_t prefix[4] = {sel[0], sel[1], sel[2], sel[3]};
        uint32_t end[4];
        line[L_REDO] = !once_intervals(prefix, end);
        line[L_SPILL] = 0;
        for (uint32_t i = 0; i < 4; ++i) line[L_BRACKET + i] = end[i];
    }
    const uint32_t keys_cap = once_keys_cap(m.numel), words = 3u << once_cells_log(keys_cap);
    uint32_t* found = once_found(mem, mem.rows[block], m.rows ? m.cols : 0u);
    for (uint32_t i = threadIdx.x; i < words; i += 1024) found[i] = found[keys_cap + i] = 0;
}

// ---------------------------------------------------------------------------

// The same value, formed anew where it stands: what is cheap to form from it is not kept over a loop.
__device__ __forceinline__ uint32_t here(uint32_t x) { asm volatile("" : "+v"(x)); return x; }

// Sums of Q values over rows of 16 lanes by a halving exchange: a lane is left with the sum number lane / (16 / Q) of its row.
__device__ __forceinline__ float rows_sum(const float (&s)[4], uint32_t lane)
{
    const bool b3 = lane & 8u, b2 = lane & 4u;
    float h[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) h[q] = (b3 ? s[q + 2] : s[q]) + dpp<0x128, 0xf>(0.f, b3 ? s[q] : s[q + 2]);
    float a = (b2 ? h[1] : h[0]) + dpp<0x141, 0xf>(0.f, b2 ? h[0] : h[1]);
    a += dpp<0x4E, 0xf>(0.f, a);
    return a + dpp<0xB1, 0xf>(0.f, a);
}
__device__ __forceinline__ float rows_sum(const float (&s)[2], uint32_t lane)
{
    const bool b3 = lane & 8u;
    float a = (b3 ? s[1] : s[0]) + dpp<0x128, 0xf>(0.f, b3 ? s[0] : s[1]);
    a += dpp<0xB1, 0xf>(0.f, a);
    a += dpp<0x4E, 0xf>(0.f, a);
    return a + dpp<0x141, 0xf>(0.f, a);
}
__device__ __forceinline__ float rows_sum(const float (&s)[1], uint32_t)
{
    float a = s[0] + dpp<0xB1, 0xf>(0.f, s[0]);
    a += dpp<0x4E, 0xf>(0.f, a);
    a += dpp<0x141, 0xf>(0.f, a);
    return a + dpp<0x128, 0xf>(0.f, a);
}
__device__ __forceinline__ double scalar_f64(double x)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, x);
    return __builtin_bit_cast(double, (uint64_t)scalar_u32((uint32_t)(b >> 32)) << 32 | scalar_u32((uint32_t)b));
}
template <int CTRL> __device__ __forceinline__ double add_lane(double x)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = dpp_u32<CTRL, 0xf>(0u, (uint32_t)b), hi = dpp_u32<CTRL, 0xf>(0u, (uint32_t)(b >> 32));
    return x + __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
// Sum over 4, 8 or 16 lanes.
template <uint32_t LANES> __device__ __forceinline__ double part_sum(double x)
{
    x = add_lane<0xB1>(x);
    x = add_lane<0x4E>(x);
    if (LANES >= 8) x = add_lane<0x141>(x);
    if (LANES == 16) x = add_lane<0x128>(x);
    return x;
}
// A lane's value and that of the lane 16, or 32, away.  (The halves are copied out first: a bit cast of a vector's element takes the first.)
__device__ __forceinline__ float add_rows16(float x)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, x), false, false);
    const uint32_t a = r[0], b = r[1];
    return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
}
__device__ __forceinline__ float add_rows32(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, x), false, false);
    const uint32_t a = r[0], b = r[1];
    return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
}
// All Q sums for every lane of a row.
__device__ __forceinline__ void share_rows(float (&r)[4], float a)
{
    r[0] = dpp<0x150, 0xf>(0.f, a); r[1] = dpp<0x154, 0xf>(0.f, a); r[2] = dpp<0x158, 0xf>(0.f, a); r[3] = dpp<0x15C, 0xf>(0.f, a);
}
__device__ __forceinline__ void share_rows(float (&r)[2], float a) { r[0] = dpp<0x150, 0xf>(0.f, a); r[1] = dpp<0x158, 0xf>(0.f, a); }
__device__ __forceinline__ void share_rows(float (&r)[1], float a) { r[0] = a; }

// h[i] += 1; lanes that agree with the first one there are added together (all keys of a block may be equal).
__device__ __forceinline__ void count_alike(uint32_t* h, uint32_t i)
{
    const bool like_first = i == scalar_u32(i);
    const uint64_t alike = __builtin_amdgcn_ballot_w64(like_first);
    if (!like_first) atomicAdd(&h[i], 1u);
    else if (__builtin_amdgcn_mbcnt_hi((uint32_t)(alike >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)alike, 0u)) == 0)
        atomicAdd(&h[i], (uint32_t)__builtin_popcountll(alike));
}

// Barrier for what passes through LDS: loads from memory stay in flight.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Threads 0 .. 31 leave a block's record in host memory (or where it is); res, num, den and bad are known to thread 0.
__device__ __forceinline__ void leave_record(const double* rec, double* out, double res, double num, double den, bool bad, uint32_t* redo)
{
    const uint32_t i = threadIdx.x;
    if (out != rec && i < R_PSUM) out[i] = rec[i];
    if (i == 0) {
        out[R_CNUM] = num; out[R_CDEN] = den; out[R_FRES] = res;
        out[R_REDO] = bad ? 1.0 : 0.0;
        *redo = bad;
    }
}

__device__ __forceinline__ double once_residual(double s2, double cross, double mu, double r2, double c2)
{
    const double res = mu != 0.0 ? s2 - 2.0 * (cross / mu) + (r2 / mu) * (c2 / mu) : s2;
    return res < 0.0 ? 0.0 : res;
}

struct Distortion { double num; bool bad; };

// a, b and d have relative errors of about 1e-7 (groups of up to 256 terms in fp32).  Up to eight times the result the terms leave it within
// 1e-6; and what is below 1e-7 of d, C below 3e-4, within an error of C of 1e-7, which is that of q.
__host__ __device__ __forceinline__ bool distortion_cancels(double terms, double num, double d) { return terms > 8.0 * num && terms > 1e-7 * d; }

__host__ __device__ __forceinline__ Distortion once_distortion(double a, double b, double d, double q, double numel)
{
    const double k = numel / (numel + q);                 // p0 / p-bar
    const double ka = k * k * a, kb = 2.0 * k * (k - 1.0) * b, kd = (k - 1.0) * (k - 1.0) * d;
    const double num = ka + kb + kd;
    const bool bad = !(fabs(num) < INFINITY) || distortion_cancels(ka + fabs(kb) + kd, num, d);
    return Distortion{num < 0.0 ? 0.0 : num, bad};
}

// The pass.  A workgroup of NW wavefronts takes a task: of a matrix every n_tasks-th batch of whole rows, of another block every
// n_tasks-th round of coordinates.  Wavefronts stand `across` side by side and `down` below each other; a load takes 64, 128 or 256 columns
// of 4, 2 or 1 rows, a wavefront has `strips` of them side by side and 4 loads (3 of three strips) a batch.  A lane keeps fp64 sums of c and t for
// its four columns of every strip, which with the loads fill the 128 registers of four wavefronts per SIMD: a workgroup of 8 wavefronts has at
// most 6,144 columns and two are on a CU, one of 16 has 12,288.  All loads are unconditional (those past an edge read again what is there): with
// a branch around them they were waited for where they were issued, and the pass over 60 matrices of 4,096 x 4,096 took 1,450 us instead of
// 1,140.  Loads of v are a batch ahead of their use, those of theta most of one.  Tasks have total / 1,024 coordinates, 524,288 at most: a
// workgroup's start and end take 25 us, its rounds of 512 at a time leave the last one short (24 of 11,008 x 4,096 with 1 M a task 1,430 us, 1,292
// so).  LINES: rows of most matrices are whole cache lines, and loads carry the nontemporal hint (see whole_lines).
// Bound by HBM with the vector ALUs behind it: 60 matrices of 4,096 x 4,096, bf16 theta, 6.04 GB, 1,200 us, 5.0 TB/s; 30 vector instructions
// per coordinate (36 with 16 wavefronts), ALUs busy 83 % of the time; 16 wavefronts, 24 of 4,096 x 11,008, 6.5 GB, 1,575 us, 4.1 TB/s (a barrier for 12 loads of
// every wavefront).  The passes read 10.07 GB for the first of these in 1,590 us.
template <uint32_t NW, int TT, bool F, bool C, bool LINES>
__global__ __launch_bounds__(64 * NW, 4) void k_once(const float* __restrict__ v_all, const typename GradIO<TT>::elem* __restrict__ theta,
                                                     const TileRow* __restrict__ tiles, OnceMem mem, float eps, float eps_low)
{
    typedef GradIO<TT> IO;
    typedef typename IO::elem E;
    typedef typename IO::vec4 TV;
    __shared__ alignas(16) uint32_t hist[kHistWords];
    __shared__ alignas(16) uint32_t staged[NW * kOnceStage];
    __shared__ alignas(16) float rowsum[2][NW * 32];
    __shared__ double settled_sums[C ? 3 : 1][C ? 64 * NW : 1];
    __shared__ double part[NW][10], total[10];
    __shared__ uint32_t n_listed, below[NW][2], sel[8], scans[4];
    constexpr uint32_t THREADS = 64 * NW;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = scalar_wave_index();
    const uint32_t block = find_owner(mem.n_blocks, blockIdx.x, lane, [&](uint32_t i) { return NW == 8 ? mem.rows[i].first_task : mem.rows[i].first_wide; });
    const OnceRow& o = mem.rows[block];
    const TileRow& m = tiles[block];
    const uint32_t n_tasks = scalar_u32(o.n_tasks), local = blockIdx.x - scalar_u32(NW == 8 ? o.first_task : o.first_wide);
    const uint32_t rows = scalar_u32(m.rows), cols = scalar_u32(m.cols);
    const bool single = NW == 8 && n_tasks == 1;              // see plan_once
    uint32_t* line = mem.line + block * kArriveStride;
    const float* src = v_all + m.state_start;
    const E* tsrc = theta + m.grad_start;
    if (tid == 0) n_listed = 0;
    const uint32_t bins_log = scalar_u32(once_bins_log((uint32_t)m.numel)), slots = 1u << once_slots_log(bins_log);
    uint32_t end[4] = {0, 0, 0, 0}, shift[2] = {0, 0};
    float inv_p0 = 0.f;
    if (!single) {
        for (uint32_t i = tid; i < 2 * slots; i += THREADS) hist[i] = 0;
        const bool none = scalar_u32(line[L_REDO]) != 0;      // nothing is listed
#pragma unroll
        for (int i = 0; i < 4; ++i) end[i] = none ? 0u : scalar_u32(line[L_BRACKET + i]);
#pragma unroll
        for (int i = 0; i < 2; ++i) shift[i] = once_shift(end[2 * i + 1] - end[2 * i], bins_log);
        inv_p0 = __builtin_bit_cast(float, scalar_u32(line[L_INV_P0]));
    } else if (C) {
        // the mean of all p: the pass below and the quantiles read these lines from the L2
        const uint32_t numel = (uint32_t)m.numel;
        double psum = 0.0;
        for (uint32_t first = tid * 4; first < numel; first += THREADS * 16) {
            f4 x[4];
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q) x[q] = *reinterpret_cast<const f4*>(src + min(first + q * (THREADS * 4), (numel - 1) & ~3u));
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q) {
                const uint32_t at = first + q * (THREADS * 4);
                const float e[4] = {x[q].x, x[q].y, x[q].z, x[q].w};
                float p = 0.f;
#pragma unroll
                for (uint32_t k = 0; k < 4; ++k) p += at + k < numel ? preconditioner(e[k], eps) : 0.f;
                psum += (double)p;
            }
        }
        psum = wave_total(psum);
        if (lane == 0) part[wave][0] = psum;
        __syncthreads();
        psum = 0.0;
        for (uint32_t w = 0; w < NW; ++w) psum += part[w][0];
        inv_p0 = (float)((double)numel / fmax(psum, (double)numel * (double)kLeastP0));
    }
    const float eps_p0 = -eps * inv_p0;
    __syncthreads();

    double s2 = 0.0, r2 = 0.0;
    float fa = 0.f, fb = 0.f, fd = 0.f;
    // A lane adds at most 256 terms in fp32 before they go to fp64, in LDS: there are no registers to spare.  q, whose sum makes p-bar, four.
    double sum_q = 0.0;
    if (C) settled_sums[0][tid] = settled_sums[1][tid] = settled_sums[2][tid] = 0.0;
    auto settle = [&]() {
        if (!C) return;
        const uint32_t at = wave * 64 + here(lane);
        settled_sums[0][at] += (double)fa; settled_sums[1][at] += (double)fb; settled_sums[2][at] += (double)fd;
        fa = fb = fd = 0.f;
    };
    uint32_t n_below[2] = {0, 0}, n_stage = 0;
    uint32_t* stage = staged + wave * kOnceStage;
    const uint32_t cap = scalar_u32(o.list_cap);
    uint32_t* list = reinterpret_cast<uint32_t*>(mem.base + (uint64_t)o.off_list * 64) + (uint64_t)local * cap;
    // Room for n keys of the wavefront; from `cap` on, which stands after the tasks' lists, it is the block's common list: tasks may have very
    // different shares of the keys.
    struct Slots { uint32_t first, spilled, at; };
    auto reserve = [&](uint32_t n) {
        uint32_t x = 0;
        if (lane == 0) x = atomicAdd(&n_listed, n);
        Slots r{scalar_u32(x), 0, 0};
        if (r.first + n > cap) {
            r.spilled = max(r.first, cap);
            if (lane == 0) x = atomicAdd(&line[L_SPILL], r.first + n - r.spilled);
            r.at = scalar_u32(x);
        }
        return r;
    };
    auto put = [&](const Slots& r, uint32_t i, uint32_t key) {
        const uint32_t slot = r.first + i, common = r.at + (slot - r.spilled);
        if (slot < cap) st_device(&list[slot], key);
        else if (common < once_spill(o)) st_device(&list[(n_tasks - local) * cap + common], key);
    };
    auto flush = [&](bool all) {
        const uint32_t n = all ? n_stage : n_stage & ~63u;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        auto bin_of_key = [&](uint32_t key) { return key >= end[2] ? slots + ((key - end[2]) >> shift[1]) : (key - end[0]) >> shift[0]; };
        // (next to zeros, or empty, an interval has hardly a key)
        const bool counted = (shift[0] == 0 && end[0] > 1) || (shift[1] == 0 && end[2] > 1 && end[2] != end[3]);
        if (!counted) {
            const Slots r = reserve(n);
            const bool fits = r.first + n <= cap;
            for (uint32_t i = lane; i < n; i += 64) {
                const uint32_t key = stage[i];
                if (fits) st_device(&list[r.first + i], key); else put(r, i, key);
                atomicAdd(&hist[bin_of_key(key)], 1u);
            }
        } else {
            // An interval that is counted key by key is not listed.  Most keys may be equal: they are added together.  (503 M coordinates,
            // finalize, us: the sign of the gradient 5,440 by the passes, 1,000 so; clipped at 1.2 standard deviations 1,480 and 776.)
            for (uint32_t i = lane; i < n; i += 64) {
                const uint32_t key = stage[i];
                const bool listed = shift[key >= end[2]] != 0;
                const uint64_t to_list = __builtin_amdgcn_ballot_w64(listed);
                if (to_list) {
                    const Slots r = reserve((uint32_t)__builtin_popcountll(to_list));
                    const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(to_list >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)to_list, 0u));
                    if (listed) put(r, at, key);
                }
                count_alike(hist, bin_of_key(key));
            }
        }
        n_stage -= n;
        const uint32_t rest = lane < n_stage ? stage[n + lane] : 0u;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (lane < n_stage) stage[lane] = rest;
    };
    auto scan = [&](const uint32_t (&key)[4]) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint64_t m0 = __builtin_amdgcn_ballot_w64(key[e] < end[0]), m2 = __builtin_amdgcn_ballot_w64(key[e] < end[2]);
            const uint64_t hits = (__builtin_amdgcn_ballot_w64(key[e] < end[1]) & ~m0) | (__builtin_amdgcn_ballot_w64(key[e] < end[3]) & ~m2);
            n_below[0] += (uint32_t)__builtin_popcountll(m0); n_below[1] += (uint32_t)__builtin_popcountll(m2);
            const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(hits >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)hits, n_stage));
            if (__builtin_amdgcn_inverse_ballot_w64(hits)) stage[at] = key[e];
            n_stage += (uint32_t)__builtin_popcountll(hits);
            // counted now: left for later the masks would be kept in vector registers, lane by lane
            asm("" : "+s"(n_below[0]), "+s"(n_below[1]), "+s"(n_stage));
        }
    };
    static_assert(kOnceStage >= 63 + 1024, "what a flush leaves and the keys of a batch");
    auto batch_done = [&](uint32_t i) {
        if (n_stage > kOnceStage - 1024) flush(false);
        if (i % 16 == 15) settle();
    };
    // q = p / p0 - 1, by the series for p where eps is small against sqrt(v)
    auto series = [&](float v) {
        const float r = __builtin_amdgcn_rsqf(v);
        return __builtin_fmaf(r, __builtin_fmaf(eps_p0, r, inv_p0), -1.0f);
    };
    auto general = [&](float v) { return __builtin_fmaf(preconditioner(v, eps), inv_p0, -1.0f); };
    auto distort = [&](const float (&x)[4], const float (&th)[4], auto q_of, auto ok) {
        float four = 0.f;
#pragma unroll
        for (uint32_t e = 0; e < 4; ++e) {
            const float q = ok(e) ? q_of(x[e]) : 0.f, z = q * th[e];
            four += q;
            fa = __builtin_fmaf(z, z, fa);
            fb = __builtin_fmaf(z, th[e], fb);
            fd = __builtin_fmaf(th[e], th[e], fd);
        }
        sum_q += (double)four;
    };
    // Four elements of which the first `skip` do not count: lanes past the end of a row, or of a block, read its last four again.
    auto masked = [&](float (&x)[4], TV vt, uint32_t skip) {
        auto ok = [&](uint32_t e) { return e >= skip; };
        uint32_t key[4];
        float th[4];
        IO::unpack(vt, th);
#pragma unroll
        for (uint32_t e = 0; e < 4; ++e) {
            key[e] = ok(e) ? __builtin_bit_cast(uint32_t, x[e]) : ~0u;
            th[e] = ok(e) ? th[e] : 0.f;
        }
        if (!single) scan(key);
        if (C) distort(x, th, general, ok);
#pragma unroll
        for (uint32_t e = 0; e < 4; ++e) x[e] = ok(e) ? x[e] : 0.f;
    };
    auto whole = [&](const float (&x)[4], TV vt, auto q_of) {
        float th[4];
        IO::unpack(vt, th);
        distort(x, th, q_of, [](uint32_t) { return true; });
    };
    auto scan_whole = [&](const float (&x)[4]) {
        uint32_t key[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) key[e] = __builtin_bit_cast(uint32_t, x[e]);
        scan(key);
    };

    if (!rows) {
        // a round is 16 coordinates of every thread
        constexpr uint32_t kRound = THREADS * 16;
        const uint32_t numel = (uint32_t)m.numel, n_rounds = (numel + kRound - 1) / kRound;
        auto at = [&](uint32_t round, uint32_t q) { return round * kRound + q * (THREADS * 4) + here(tid) * 4; };
        f4 nx[4]; TV nt[4];
        auto issue = [&](uint32_t round) {
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q) {
                const float* from = src + min(at(round, q), numel - 4);
                nx[q] = LINES ? ld_stream<f4_any>(from) : *reinterpret_cast<const f4_any*>(from);
            }
        };
        auto issue_theta = [&](uint32_t round) {
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q) if (C) nt[q] = IO::loadv_shared(tsrc + min(at(round, q), numel - 4));
        };
        issue(local); issue_theta(local);
        for (uint32_t round = local, i = 0; round < n_rounds; round += n_tasks, ++i) {
            float x[4][4];
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q) { x[q][0] = nx[q].x; x[q][1] = nx[q].y; x[q][2] = nx[q].z; x[q][3] = nx[q].w; }
            const uint32_t next = min(round + n_tasks, n_rounds - 1);
            issue(next);
            if ((round + 1) * kRound <= numel) {
                if (!single) {
#pragma unroll
                    for (uint32_t q = 0; q < 4; ++q) scan_whole(x[q]);
                }
                if (C) {
#pragma unroll
                    for (uint32_t q = 0; q < 4; ++q) whole(x[q], nt[q], general);
                }
            } else {
#pragma unroll
                for (uint32_t q = 0; q < 4; ++q) masked(x[q], nt[q], at(round, q) - min(at(round, q), numel - 4));
            }
            issue_theta(next);
            batch_done(i);
        }
        flush(true);
    }
    double cross = 0.0, c2 = 0.0;
    auto walk = [&](auto strips, auto quads) {
        constexpr uint32_t K = decltype(strips)::value, Q = decltype(quads)::value;
        const uint32_t geom = scalar_u32(o.geom), lanes_log = geom & 15u, across = (geom >> 8) & 31u, down = (geom >> 16) & 255u;
        const uint32_t wrow = wave / across, wcol = wave - wrow * across, rpl = 6 - lanes_log;
        const uint32_t my_rows = Q << rpl, batch = down * my_rows, stride = batch * n_tasks;
        auto lcol = [&]() { return here(lane) & ((1u << lanes_log) - 1u); };
        auto lrow = [&]() { return here(lane) >> lanes_log; };
        auto first_col = [&](uint32_t k) { return (wcol * K + k) << (lanes_log + 2); };          // of a strip
        auto all_cols = [&](uint32_t k) { return first_col(k) + (4u << lanes_log) <= cols; };
        uint32_t at[K];                                       // the lane's first element of a load, from the load's first row
#pragma unroll
        for (uint32_t k = 0; k < K; ++k) at[k] = lrow() * cols + once_first_col(first_col(k) + 4 * lcol(), cols);
        uint32_t wide = 1; while (wide < across) wide *= 2;
        const double inv_cols = scalar_f64(1.0 / (double)cols);
        auto first_row = [&](uint32_t row, uint32_t q) { return once_first_row(row + (q << rpl), rpl, rows); };
        f4 nx[Q][K]; TV nt[Q][K];
        auto issue = [&](uint32_t row) {
#pragma unroll
            for (uint32_t q = 0; q < Q; ++q) {
                const char* p = reinterpret_cast<const char*>(src) + (uint64_t)first_row(row, q) * cols * 4;
#pragma unroll
                for (uint32_t k = 0; k < K; ++k) {
                    const float* from = reinterpret_cast<const float*>(p + here(at[k]) * 4u);
                    nx[q][k] = LINES ? ld_stream<f4_any>(from) : *reinterpret_cast<const f4_any*>(from);
                }
            }
        };
        // theta has registers for one batch: the next one's is asked for when this one's has been used
        auto issue_theta = [&](uint32_t row) {
            if (!C) return;
#pragma unroll
            for (uint32_t q = 0; q < Q; ++q) {
                const char* p = reinterpret_cast<const char*>(tsrc) + (uint64_t)first_row(row, q) * cols * sizeof(E);
#pragma unroll
                for (uint32_t k = 0; k < K; ++k) {
                    const E* from = reinterpret_cast<const E*>(p + here(at[k]) * (uint32_t)sizeof(E));
                    nt[q][k] = LINES ? IO::loadv_any(from) : IO::loadv_shared(from);
                }
            }
        };
        double cs[K][4], ts[K][4];
#pragma unroll
        for (uint32_t k = 0; k < K; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e) cs[k][e] = ts[k][e] = 0.0;
        const uint32_t batch0 = local * batch;
        uint32_t row = wrow < down ? batch0 + wrow * my_rows : rows, i = 0;                      // `rows`: a wavefront without work
        issue(row); issue_theta(row);
        for (uint32_t first = batch0; first < rows; first += stride, ++i) {
            float x[Q][K][4];
#pragma unroll
            for (uint32_t q = 0; q < Q; ++q)
#pragma unroll
                for (uint32_t k = 0; k < K; ++k) { x[q][k][0] = nx[q][k].x; x[q][k][1] = nx[q][k].y; x[q][k][2] = nx[q][k].z; x[q][k][3] = nx[q][k].w; }
            const uint32_t next = min(row + stride, rows);
            issue(next);
            const bool all_rows = row + my_rows <= rows;
#pragma unroll
            for (uint32_t k = 0; k < K; ++k) {
                if (all_rows && all_cols(k)) {
                    if (!single) {
#pragma unroll
                        for (uint32_t q = 0; q < Q; ++q) scan_whole(x[q][k]);
                    }
                    if (C) {
                        float low = x[0][k][0];
#pragma unroll
                        for (uint32_t q = 0; q < Q; ++q) low = fminf(fminf(fminf(low, x[q][k][0]), fminf(x[q][k][1], x[q][k][2])), x[q][k][3]);
                        const bool small = __builtin_amdgcn_ballot_w64(!(low > eps_low)) != 0;
                        if (!small) {
#pragma unroll
                            for (uint32_t q = 0; q < Q; ++q) whole(x[q][k], nt[q][k], series);
                        } else {
#pragma unroll
                            for (uint32_t q = 0; q < Q; ++q) whole(x[q][k], nt[q][k], general);
                        }
                    }
                } else {
#pragma unroll
                    for (uint32_t q = 0; q < Q; ++q) {
                        masked(x[q][k], nt[q][k], once_skip(row + (q << rpl), lrow(), rpl, rows, first_col(k) + 4 * lcol(), cols));
                    }
                }
            }
            issue_theta(next);
            batch_done(i);
            if (F) {
                // A row's sum: over 16 to 64 lanes, 256 columns at most, in fp32; the rest in fp64 through LDS, where each of a row's loads has 16 / Q
                // lanes.  One strip: [row of a load][wavefront][load].  Several: 16 lanes leave one number, [row of a load][load][wavefront][lanes].
                float* rs = rowsum[i & 1] + wrow * (wide * 16);
                const uint32_t l = here(lane), groups_log = lanes_log - 4, in_row = l >> lanes_log;
                auto of_lane = [&](uint32_t q, uint32_t k) { return (x[q][k][0] + x[q][k][1]) + (x[q][k][2] + x[q][k][3]); };
                auto meet = [&]() { if (across > 1) lds_barrier(); else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); };
                constexpr uint32_t kLanes = Q == 1 ? NW : 16 / Q;           // that have numbers of their own
                double row_sum = 0.0;
                auto gather = [&](auto of_wave) {
#pragma unroll
                    for (uint32_t w0 = 0; w0 < NW; w0 += kLanes) {
                        const uint32_t w = w0 + (l & (kLanes - 1));
                        if (w < across && wrow < down) row_sum += of_wave(w);
                    }
                };
                float sums[Q];
#pragma unroll
                for (uint32_t q = 0; q < Q; ++q) {
                    sums[q] = of_lane(q, 0);
#pragma unroll
                    for (uint32_t k = 1; k < K; ++k) sums[q] += of_lane(q, k);
                }
                float mine = rows_sum(sums, lane);
                if constexpr (K == 1) {
                    if (lanes_log > 4) mine = add_rows16(mine);
                    if (lanes_log > 5) mine = add_rows32(mine);
                    if ((l & ((1u << lanes_log) - 16u + 3u)) == 0 && wrow < down) rs[(in_row * wide + wcol) * 4 + ((l >> 2) & 3u)] = mine;
                    meet();
                    const float* from = rs + in_row * wide * 4 + ((l >> 2) & 3u);
                    gather([&](uint32_t w) { return (double)from[w * 4]; });
                } else {
                    const uint32_t load = Q == 2 ? (l >> 3) & 1u : 0u;
                    float* to = rs + (((in_row * Q + load) * wide) << groups_log);
                    if ((l & (16u / Q - 1u)) == 0 && wrow < down) to[(wcol << groups_log) + ((l >> 4) & ((1u << groups_log) - 1u))] = mine;
                    meet();
                    if (groups_log == 2) gather([&](uint32_t w) { const f4 y = reinterpret_cast<const f4*>(to)[w]; return ((double)y.x + (double)y.y) + ((double)y.z + (double)y.w); });
                    else if (groups_log == 1) gather([&](uint32_t w) { const float2 y = reinterpret_cast<const float2*>(to)[w]; return (double)y.x + (double)y.y; });
                    else gather([&](uint32_t w) { return (double)to[w]; });
                }
                float r[Q];
                share_rows(r, (float)(part_sum<kLanes>(row_sum) * inv_cols));
#pragma unroll
                for (uint32_t q = 0; q < Q; ++q) {
                    const double rd = (double)r[q];
                    r2 = __builtin_fma(rd, rd, r2);
#pragma unroll
                    for (uint32_t k = 0; k < K; ++k)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const double xd = (double)x[q][k][e];
                            cs[k][e] += xd;
                            s2 = __builtin_fma(xd, xd, s2);
                            ts[k][e] = __builtin_fma(rd, xd, ts[k][e]);
                        }
                }
            }
            row = next;
        }
        flush(true);
        if (!F) return;
        if (lcol() != 0 || wcol != 0) r2 = 0.0;               // all lanes of a row hold its sum
        // rho = sum r^2 / sum r of the task; columns leave as c and t / rho - c: of a rank-one S the latter is zero
        double rho = 0.0, t2 = wave_total(r2);
#pragma unroll
        for (uint32_t k = 0; k < K; ++k) rho += (cs[k][0] + cs[k][1]) + (cs[k][2] + cs[k][3]);
        rho = wave_total(rho);
        if (lane == 0) { part[wave][0] = rho; part[wave][1] = t2; }
        __syncthreads();                                      // and the last keys have left `staged`
        double all = 0.0;
        t2 = 0.0;
#pragma unroll 1
        for (uint32_t w = 0; w < NW; ++w) { all += part[w][0]; t2 += part[w][1]; }
        rho = all > 0.0 ? t2 / all * (double)cols : 0.0;
        if (tid == 0) { total[5] = rho; total[7] = all; }
        float2* to = reinterpret_cast<float2*>(mem.base + (uint64_t)o.off_cols * 64) + (uint64_t)local * cols;
        double* sh = reinterpret_cast<double*>(staged);       // 256 per wavefront
        static_assert(sizeof(staged) >= NW * 256 * sizeof(double), "a strip of every wavefront");
        const uint32_t width = 4u << lanes_log;               // columns of a strip
#pragma unroll
        for (uint32_t k = 0; k < K; ++k) {
            // sums over the rows of a wavefront's loads, then over the wavefronts below each other
            auto sum_down = [&](double (&y)[4]) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (lanes_log < 6) y[e] += __shfl_xor(y[e], 32);
                    if (lanes_log < 5) y[e] += __shfl_xor(y[e], 16);
                }
                if (down == 1) return;
                __syncthreads();
                if (lrow() == 0) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) sh[wave * width + 4 * lcol() + e] = y[e];
                }
                __syncthreads();
                if (wrow == 0 && lrow() == 0) {
#pragma unroll 1
                    for (uint32_t w = 1; w < down; ++w) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) y[e] += sh[(w * across + wcol) * width + 4 * lcol() + e];
                    }
                }
            };
            sum_down(cs[k]);
            sum_down(ts[k]);
            if (wrow == 0 && lrow() == 0) {
                const uint32_t col = first_col(k) + 4 * lcol(), base = once_first_col(col, cols);
#pragma unroll
                for (uint32_t e = 0; e < 4; ++e) {
                    if (base + e < col) continue;             // another lane's column
                    if (single) {
                        const double mean = (double)(float)(cs[k][e] / (double)rows);
                        cross = __builtin_fma(mean, ts[k][e], cross);
                        c2 = __builtin_fma(mean, mean, c2);
                    } else {
                        const float cf = (float)cs[k][e];
                        to[base + e] = float2{cf, rho != 0.0 ? (float)(ts[k][e] / rho - (double)cf) : 0.f};
                    }
                }
            }
        }
    };
    if (rows) {
        const uint32_t strips = (scalar_u32(o.geom) >> 4) & 15u;
        const std::integral_constant<uint32_t, 1> one; const std::integral_constant<uint32_t, 2> two;
        const std::integral_constant<uint32_t, 3> three; const std::integral_constant<uint32_t, 4> four;
        if (strips == 1) { walk(one, four); }
        else if (strips == 2) { walk(two, two); }
        else { walk(three, one); }
    }
    settle();
    const double mine[10] = {sum_q, C ? settled_sums[0][tid] : 0.0, C ? settled_sums[1][tid] : 0.0, C ? settled_sums[2][tid] : 0.0,
                             s2, 0.0, r2, 0.0, cross, c2};
    __syncthreads();                                          // `part` has been read
#pragma unroll
    for (int j = 0; j < 10; ++j) {
        const double w = j != 5 && j != 7 && (j < 7 || single) ? wave_total(mine[j]) : 0.0;
        if (lane == 0) part[wave][j] = w;
    }
    if (lane == 0) {
        below[wave][0] = n_below[0]; below[wave][1] = n_below[1];
    }
    __syncthreads();
    if (tid < 10) {
        double x = 0.0;
#pragma unroll 1
        for (uint32_t w = 0; w < NW; ++w) x += part[w][tid];
        if (tid != 5 && tid != 7) total[tid] = x;
    }
    __syncthreads();
    if (!single) {
        OnceSums* sums = mem.sums + (NW == 8 ? blockIdx.x : mem.narrow_tasks + blockIdx.x);
        if (tid < 8) reinterpret_cast<double*>(sums)[tid] = total[tid];
        if (tid >= 64 && tid < 66) {
            uint32_t n = 0;
            for (uint32_t w = 0; w < NW; ++w) n += below[w][tid - 64];
            sums->n[tid - 64] = n;
        }
        if (tid == 128) sums->n_list = n_listed;
        uint32_t* to = mem.hist + (uint64_t)block * kHistWords;
        for (uint32_t i = tid; i < 2 * slots; i += THREADS)
            if (hist[i]) atomicAdd(&to[i], hist[i]);
        return;
    }
    const uint32_t numel = (uint32_t)m.numel, rank[4] = {m.rank[0], m.rank[1], m.rank[2], m.rank[3]};
    order_stats<THREADS, true>([&](auto f) {
        for (uint32_t first = tid * 4; first < numel; first += THREADS * 16) {
            f4 x[4];
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q) x[q] = *reinterpret_cast<const f4*>(src + min(first + q * (THREADS * 4), (numel - 1) & ~3u));
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q) {
                const float e[4] = {x[q].x, x[q].y, x[q].z, x[q].w};
#pragma unroll
                for (uint32_t k = 0; k < 4; ++k)
                    if (first + q * (THREADS * 4) + k < numel) f(__builtin_bit_cast(uint32_t, e[k]) & 0x7fffffffu);
            }
        }
    }, rank, hist, sel, scans, lane, wave);
    const double* rec = mem.rec + (uint64_t)block * kRecDoubles;
    double* out = mem.out + (uint64_t)block * kRecDoubles;
    if (tid < 32) {
        const double res = F && rows ? once_residual(total[4], total[8], total[7] / ((double)rows * (double)cols), total[6], total[9]) : 0.0;
        const Distortion c = C ? once_distortion(total[1], total[2], total[3], total[0], (double)numel) : Distortion{0.0, false};
        leave_record(rec, out, res, c.num, total[3], !(fabs(res) < INFINITY) || c.bad, line + L_REDO);
        if (tid < 4) out[R_ORDER + tid] = (double)__builtin_bit_cast(float, sel[tid]);
    }
}

// Units of a block: the first walk its tasks' lists for the keys that share the ranks' bins, the others sum 64 columns over its tasks. The
// last to arrive orders the keys, adds the sums and leaves the record.  A chain of dependent loads for a small layout (8 blocks of 16.8 M 27 us),
// HBM for the lists and the column sums of large ones (3.5 G coordinates, 0.9 GB, 305 us).  Keys are collected in LDS first, since an atomic on
// the block's counter is a round trip of more than a microsecond (148 blocks, 124 M: 110 us with one for each key, 43 so), and counted eight
// reads at a time (8 blocks of 131 M, 2,000 keys each: 122 us with one read after another, 63 so).
template <bool F, bool C>
__global__ __launch_bounds__(256, 4) void k_once_select(const TileRow* __restrict__ tiles, OnceMem mem)
{
    __shared__ alignas(16) uint32_t keys[2 * kOnceKeys];      // a unit's of either interval; then the block's of one, 512 more than there are at most
    __shared__ double red[4][10];
    __shared__ uint32_t n_below[2], n_in[2], n_mine[2], first_mine[2], bin[4], bin_at[4], bin_n[4], scans[4], near_key[4], near_rank[4], open;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = scalar_wave_index();
    const uint32_t block = find_owner(mem.n_blocks, blockIdx.x, lane, [&](uint32_t i) { return mem.rows[i].first_unit; });
    const OnceRow& o = mem.rows[block];
    const TileRow& m = tiles[block];
    const uint32_t n_tasks = scalar_u32(o.n_tasks), rows = scalar_u32(m.rows), cols = scalar_u32(m.cols);
    const uint32_t unit = blockIdx.x - scalar_u32(o.first_unit), lists = once_list_units(o), units = lists + once_col_units(rows, cols);
    const OnceSums* sums = mem.sums + (o.geom >> 24 ? mem.narrow_tasks + o.first_wide : o.first_task);
    uint32_t* line = mem.line + block * kArriveStride;
    uint32_t* hist = mem.hist + (uint64_t)block * kHistWords;
    const uint32_t keys_cap = once_keys_cap(m.numel), cells_log = once_cells_log(keys_cap);
    uint32_t* found = once_found(mem, o, rows ? cols : 0u);
    const uint32_t bins_log = scalar_u32(once_bins_log((uint32_t)m.numel)), slots = 1u << once_slots_log(bins_log);
    bool bad = scalar_u32(line[L_REDO]) != 0;             // then there are no intervals
    uint32_t end[4], shift[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) end[i] = bad ? 0u : scalar_u32(line[L_BRACKET + i]);
#pragma unroll
    for (int i = 0; i < 2; ++i) shift[i] = once_shift(end[2 * i + 1] - end[2 * i], bins_log);

    const bool one_interval = end[2] == end[3];               // both quantiles are in the first
    auto interval_of = [&](uint32_t t) { return one_interval ? 0u : t >> 1; };

    // Keys below and in the intervals, the bins that hold the ranks, the keys before these and in them.
    auto digits = [&]() {
        if (tid < 2) n_below[tid] = n_mine[tid] = 0;
        if (tid < 4) { bin[tid] = ~0u; bin_at[tid] = bin_n[tid] = near_key[tid] = near_rank[tid] = 0; }
        if (tid == 4) open = 0;
        __syncthreads();
        uint32_t n[2] = {0, 0};
        for (uint32_t i = tid; i < n_tasks; i += 256) { n[0] += sums[i].n[0]; n[1] += sums[i].n[1]; }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const uint32_t all = wave_scan(n[j]);
            if (lane == 63) atomicAdd(&n_below[j], all);
        }
        const uint32_t q = wave >> 1, mine_at = (tid & 127u) * kBinsPerLane;
        uint32_t c[kBinsPerLane], mine = 0;
#pragma unroll
        for (uint32_t i = 0; i < kBinsPerLane; ++i) c[i] = 0;
        if (mine_at < slots) load_bins(c, hist + q * slots + mine_at);
#pragma unroll
        for (uint32_t i = 0; i < kBinsPerLane; ++i) mine += c[i];
        const uint32_t incl = wave_scan(mine);
        if (lane == 63) scans[wave] = incl;
        __syncthreads();
        const uint32_t at = incl - mine + (wave & 1u ? scans[wave - 1] : 0u);
        if (tid < 2) n_in[tid] = scans[2 * tid] + scans[2 * tid + 1];
#pragma unroll
        for (uint32_t t = 0; t < 4; ++t) {
            const uint32_t rank = m.rank[t] - n_below[q];
            if (interval_of(t) == q && rank >= at && rank - at < mine) {       // a rank below the interval wraps around
                const Digit f = bin_of(c, mine_at, at, rank);
                bin[t] = f.bin; bin_at[t] = rank - f.rank; bin_n[t] = f.count;
            }
        }
        __syncthreads();
    };
    static_assert(kOnceBins == 128 * kBinsPerLane && kBinsPerLane <= 1u << 7, "two wavefronts an interval");
    // The bins of an interval's ranks, and those between them, are one range of keys.
    struct Range { uint32_t first, width, before, n, shift; bool crowded; };
    auto range_of = [&](uint32_t q) {
        uint32_t lo = ~0u, hi = 0, before = 0, end_at = 0;
#pragma unroll
        for (uint32_t t = 0; t < 4; ++t)
            if (interval_of(t) == q && bin[t] != ~0u) {        // ~0: a zero, below the interval
                if (lo == ~0u) { lo = bin[t]; before = bin_at[t]; }
                hi = bin[t]; end_at = bin_at[t] + bin_n[t];
            }
        const uint32_t n = scalar_u32(end_at - before), sh = q ? shift[1] : shift[0];
        // nothing is wanted of keys that have a bin each
        const uint32_t width = scalar_u32(lo == ~0u || sh == 0 ? 0u : (hi - lo + 1) << sh);
        return Range{(q ? end[2] : end[0]) + (scalar_u32(lo) << sh), width, scalar_u32(before), n, width_shift(width, cells_log), n > keys_cap && width != 0};
    };

    // a wavefront's part of a task's list, or of the common one that stands after these
    const uint32_t cap = scalar_u32(o.list_cap), spilled = scalar_u32(line[L_SPILL]), parts = once_parts(cap), id = unit * 4 + wave;
    struct Part { uint32_t* from; uint32_t n, room; };
    auto part_of = [&](uint32_t id) {
        const uint32_t task = min(id / max(parts, 1u), n_tasks), at = (id - task * parts) * kOncePart, whole = task < n_tasks ? cap : once_spill(o);
        const uint32_t all = min(whole, task < n_tasks ? sums[task].n_list : spilled);
        return Part{reinterpret_cast<uint32_t*>(mem.base + (uint64_t)o.off_list * 64) + ((uint64_t)task * cap + at), all > at ? (uint32_t)min(all - at, kOncePart) : 0u,
                    (uint32_t)min(whole - at, kOncePart)};
    };
    Part own = unit < lists ? part_of(id) : Part{nullptr, 0u, 0u};
    own.n = scalar_u32(own.n);
    bool have = false;
    if (unit < lists && __syncthreads_or(own.n != 0)) {
        have = true;
        digits();
        const Range r[2] = {range_of(0), range_of(1)};
        auto keep = [&](uint32_t key, bool high) {
            const uint32_t at = atomicAdd(&n_mine[high], 1u);
            if (at < kOnceKeys) keys[high * kOnceKeys + at] = key;
        };
        // a part starts on a multiple of 16 words, as cap is one
        auto walk = [&](auto f) {
            for (uint32_t i = 4 * lane; i < own.n; i += 1024) {
                uint4 quad[4];
#pragma unroll
                for (uint32_t q = 0; q < 4; ++q) quad[q] = *reinterpret_cast<const uint4*>(own.from + min(i + 256 * q, (own.n - 1) & ~3u));
#pragma unroll
                for (uint32_t q = 0; q < 4; ++q) {
                    const uint32_t at = i + 256 * q;
                    f(quad[q].x, at < own.n); f(quad[q].y, at + 1 < own.n); f(quad[q].z, at + 2 < own.n); f(quad[q].w, at + 3 < own.n);
                }
            }
        };
        if (!r[0].crowded && !r[1].crowded) {
            walk([&](uint32_t key, bool there) {
                const bool low = key - r[0].first < r[0].width, high = key - r[1].first < r[1].width;
                if ((low || high) && there) keep(key, high);
            });
        } else {
            for (uint32_t i = tid; i < 3u << cells_log; i += 256) {
                if (r[0].crowded) keys[i] = 0;
                if (r[1].crowded) keys[kOnceKeys + i] = 0;
            }
            __syncthreads();
            uint32_t kept = 0;
            walk([&](uint32_t key, bool there) {
                const bool low = key - r[0].first < r[0].width, high = key - r[1].first < r[1].width;
                const bool to_cell = there && ((low && r[0].crowded) || (high && r[1].crowded));
                // the part keeps these keys, in front, for the case that their cell has several values
                const uint64_t hits = __builtin_amdgcn_ballot_w64(to_cell);
                if (to_cell) {
                    st_device(&own.from[__builtin_amdgcn_mbcnt_hi((uint32_t)(hits >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)hits, kept))], key);
                    uint32_t* cell = keys + high * kOnceKeys + (high ? (key - r[1].first) >> r[1].shift : (key - r[0].first) >> r[0].shift);
                    count_alike(keys, (uint32_t)(cell - keys));
                    if (cell[1u << cells_log] < key) atomicMax(cell + (1u << cells_log), key);
                    if (cell[2u << cells_log] < ~key) atomicMax(cell + (2u << cells_log), ~key);
                } else if ((low || high) && there) keep(key, high);
                kept += (uint32_t)__builtin_popcountll(hits);
            });
            // how many, in the part's last word; a key there (keys are below 2^31) if it is full
            if (own.n && lane == 0 && kept < own.room) st_device(&own.from[own.room - 1], kept | 1u << 31);
        }
        // the unit's keys go to the block's in one piece: an atomic for each would be a round trip for each
        __syncthreads();
        if (tid < 2 && n_mine[tid]) first_mine[tid] = atomicAdd(&line[L_KEYS + tid], n_mine[tid]);
        __syncthreads();
#pragma unroll
        for (uint32_t q = 0; q < 2; ++q) {
            for (uint32_t i = tid; i < min(n_mine[q], kOnceKeys) && first_mine[q] + i < keys_cap; i += 256)
                st_device(&found[q * keys_cap + first_mine[q] + i], keys[q * kOnceKeys + i]);
            if (!r[q].crowded) continue;
            for (uint32_t i = tid; i < 1u << cells_log; i += 256) {
                const uint32_t* cell = keys + q * kOnceKeys + i;
                uint32_t* to = found + q * keys_cap + i;
                if (cell[0] == 0) continue;
                atomicAdd(to, cell[0]);
                atomicMax(to + (1u << cells_log), cell[1u << cells_log]);
                atomicMax(to + (2u << cells_log), cell[2u << cells_log]);
            }
        }
    } else if (F && unit >= lists) {
        // 64 columns, a quarter of the tasks to each wavefront
        const uint32_t at = (unit - lists) * 64 + lane;
        const float2* from = reinterpret_cast<const float2*>(mem.base + (uint64_t)o.off_cols * 64) + min(at, cols - 1);
        double c = 0.0, t = 0.0;
#pragma unroll 8
        for (uint32_t i = wave; i < n_tasks; i += 4) {
            const float2 x = from[(uint64_t)i * cols];
            const double rho = sums[i].rho;
            c += (double)x.x;
            t = __builtin_fma(rho, (double)x.y + (double)x.x, t);
        }
        double* sh = reinterpret_cast<double*>(keys);
        sh[tid] = c; sh[256 + tid] = t;
        __syncthreads();
        if (wave == 0) {
            c = (sh[lane] + sh[64 + lane]) + (sh[128 + lane] + sh[192 + lane]);
            t = (sh[256 + lane] + sh[320 + lane]) + (sh[384 + lane] + sh[448 + lane]);
            const double mean = at < cols ? (double)(float)(c / (double)rows) : 0.0;
            const double cross = wave_total(mean * t), c2 = wave_total(mean * mean);
            if (lane == 0) { OnceUnit* u = mem.units + blockIdx.x; st_device(&u->cross, cross); st_device(&u->c2, c2); }
        }
    }
    if (!arrive_last(line + L_ARRIVED, units)) return;

    if (!have) digits();
    {
        double x[10] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        for (uint32_t i = tid; i < n_tasks; i += 256) {
            const double* s = reinterpret_cast<const double*>(sums + i);
#pragma unroll
            for (int j = 0; j < 8; ++j) x[j] += s[j];
        }
        if (F)
            for (uint32_t u = lists + tid; u < units; u += 256) {
                const OnceUnit* from = mem.units + (blockIdx.x - unit + u);
                x[8] += ld_device(&from->cross); x[9] += ld_device(&from->c2);
            }
#pragma unroll
        for (int d = 32; d > 0; d >>= 1)
#pragma unroll
            for (int j = 0; j < 10; ++j) x[j] += __shfl_xor(x[j], d);
        if (lane == 0) {
#pragma unroll
            for (int j = 0; j < 10; ++j) red[wave][j] = x[j];
        }
    }
    // a wavefront per rank
    const double* rec = mem.rec + (uint64_t)block * kRecDoubles;
    double* out = mem.out + (uint64_t)block * kRecDoubles;
    const uint32_t q = interval_of(wave), rank = wave == 0 ? m.rank[0] : wave == 1 ? m.rank[1] : wave == 2 ? m.rank[2] : m.rank[3];
    bad |= spilled > once_spill(o);
    uint32_t value = 0;
    bool near = false;                                        // of a crowded interval: the value, or the first key of its cell
#pragma unroll
    for (uint32_t half = 0; half < 2; ++half) {                // one interval after the other: its keys to LDS, then its ranks
        const Range r = range_of(half);
        const uint32_t n_keys = ld_device(line + L_KEYS + half), n = min(n_keys, keys_cap), first = end[2 * half], sh = shift[half];
        const uint32_t* from = found + half * keys_cap;
        __syncthreads();
        if (r.crowded)
            for (uint32_t i = tid; i < 1024; i += 256)
                for (uint32_t k = 0; k < 3; ++k) keys[k * 1024 + i] = i < 1u << cells_log ? ld_device(from + (k << cells_log) + i) : 0u;
        else
            for (uint32_t i = tid; i < n + 512; i += 256) keys[i] = i < n ? ld_device(from + i) : ~0u;
        __syncthreads();
        if (q != half) continue;
        const uint32_t b = bin[wave], want = rank - n_below[half] - r.before;
        if (rank < n_below[half]) bad |= first != 1;           // 0 is the only key below 1
        else if (rank - n_below[half] >= n_in[half] || b == ~0u) bad = true;
        else if (sh == 0) value = first + b;
        else if (r.crowded) {
            uint32_t c[16], mine = 0;
            load_bins(c, keys + lane * 16);
#pragma unroll
            for (uint32_t i = 0; i < 16; ++i) mine += c[i];
            const uint32_t at = wave_scan(mine) - mine;
            if (want >= at && want - at < mine) {
                const Digit f = bin_of(c, lane * 16, at, want);
                const uint32_t least = ~keys[2048 + f.bin], most = keys[1024 + f.bin];
                near_key[wave] = least == most ? most : r.first + (f.bin << r.shift);
                near_rank[wave] = f.rank;
                if (least != most) atomicOr(&open, 1u << wave);
            }
            near = true;
        } else if (n_keys > keys_cap) bad = true;
        else {
            uint32_t lo = first + (b << sh), hi = lo + (1u << sh) - 1;                       // the least key with `want` + 1 keys up to it
            while (lo < hi) {
                const uint32_t mid = lo + ((hi - lo) >> 1);
                uint32_t upto = 0;
                for (uint32_t i = 0; i < n; i += 512) {        // eight reads at a time, the last ones past the end
                    uint32_t key[8];
#pragma unroll
                    for (uint32_t k = 0; k < 8; ++k) key[k] = keys[i + 64 * k + lane];
#pragma unroll
                    for (uint32_t k = 0; k < 8; ++k) upto += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(key[k] <= mid));
                }
                if (upto > want) hi = mid; else lo = mid + 1;
            }
            value = lo;
        }
    }
    __syncthreads();
    // Ranks whose cell has several values: 11 bits at a time from what the parts have kept.
    const uint32_t n_parts = n_tasks * parts + once_parts(once_spill(o)), share = max(1u, 256 / max(n_parts, 1u));      // threads a part
#pragma unroll 1
    for (uint32_t half = 0; half < 2; ++half) {
        const uint32_t mine = scalar_u32(open) & (one_interval ? (half ? 0u : 15u) : 3u << (2 * half));
        if (mine == 0) continue;
        uint32_t left = range_of(half).shift;
        while (left > 0) {
            const uint32_t bits = min(left, 11u);
            __syncthreads();
            for (uint32_t i = tid; i < 2 * kOnceKeys; i += 256) keys[i] = 0;
            __syncthreads();
            const uint32_t from_key[4] = {near_key[0], near_key[1], near_key[2], near_key[3]};
            for (uint32_t i = tid / share; i < n_parts; i += 256 / share) {
                const Part p = part_of(i);
                if (p.n == 0) continue;
                const uint32_t word = ld_device(&p.from[p.room - 1]), n = word >> 31 ? word & 0x7fffffffu : p.room;
                for (uint32_t k = tid % share; k < n; k += 8 * share) {
                    uint32_t key[8];
#pragma unroll
                    for (uint32_t e = 0; e < 8; ++e) key[e] = ld_device(&p.from[min(k + e * share, n - 1)]);
#pragma unroll
                    for (uint32_t e = 0; e < 8; ++e)
#pragma unroll
                        for (uint32_t t = 0; t < 4; ++t) {
                            const uint32_t off = key[e] - from_key[t];
                            if (k + e * share < n && (mine >> t & 1u) && off < 1u << left) count_alike(keys, 2048 * t + (off >> (left - bits)));
                        }
                }
            }
            __syncthreads();
            left -= bits;
            if (mine >> wave & 1u) {
                const uint32_t want = near_rank[wave];
                uint32_t c[32], mine_n = 0;
                load_bins(c, keys + 2048 * wave + 32 * lane);
#pragma unroll
                for (uint32_t i = 0; i < 32; ++i) mine_n += c[i];
                const uint32_t at = wave_scan(mine_n) - mine_n;
                if (want >= at && want - at < mine_n) {
                    const Digit f = bin_of(c, 32 * lane, at, want);
                    near_key[wave] += f.bin << left; near_rank[wave] = f.rank;
                }
            }
            __syncthreads();
        }
    }
    if (near) value = near_key[wave];
    if (lane == 0) out[R_ORDER + wave] = (double)__builtin_bit_cast(float, value);
    if (tid == 0) scans[0] = 0;
    __syncthreads();
    if (bad && lane == 0) scans[0] = 1;
    __syncthreads();
    if (tid < 32) {
        double x[10];
#pragma unroll
        for (int j = 0; j < 10; ++j) x[j] = (red[0][j] + red[1][j]) + (red[2][j] + red[3][j]);
        const double res = F && rows ? once_residual(x[4], x[8], x[7] / ((double)rows * (double)cols), x[6], x[9]) : 0.0;
        const Distortion c = C ? once_distortion(x[1], x[2], x[3], x[0], (double)m.numel) : Distortion{0.0, false};
        leave_record(rec, out, res, c.num, x[3], scans[0] != 0 || !(fabs(res) < INFINITY) || c.bad, line + L_REDO);
    }
    if (tid >= 64 && tid < 66) st_device(line + L_KEYS + (tid - 64), 0u);
    for (uint32_t i = tid; i < 2 * slots; i += 256) hist[i] = 0;
}

}  // namespace baoc
