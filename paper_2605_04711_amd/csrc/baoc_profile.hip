// Gradient-stream profiler of BAOC for gfx950 (MI355X): kernels and the
// baoc_profile_* entry points.
//
// One sampled step is one streaming pass: every coordinate's gradient, previous
// gradient and fp32 EMA states are read once and written once (28 B per
// coordinate with fp32 gradients, 22 B with bf16), and everything Sec. 3.3 needs
// from that coordinate is accumulated in registers on the way:
//   Eq. 3  m <- beta_m m + (1-beta_m) g,  v <- beta_v v + (1-beta_v) g*g
//   Eq. 5  <g_t, g_{t-1}>, |g_t|^2, |m|^2, |v|_1
//   Eq. 8  update directions u = m/(sqrt(v)+eps_u) from the fp32 state and from
//          the state after a bf16 or a block-wise absmax 8-bit round trip.
// Work is cut into chunks that never straddle a parameter block; the step kernel cuts a chunk into
// slices, one workgroup (1, 2 or 4 wavefronts, a launch-shape parameter) and one partial row each.  A
// wavefront owns whole 256-coordinate quantisation groups (4 coordinates per lane, one or two groups
// next to each other), so a group's absmax is a DPP reduction inside the wavefront.  Sums go wavefront
// (DPP) -> workgroup (LDS) -> one partial row per workgroup -> per parameter block in fp64 (by the block's last
// workgroup on small layouts, by a second kernel on others).
// No float atomics anywhere: two runs give identical bits.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <limits>
#include <mutex>
#include <new>
#include <type_traits>
#include <vector>

#include "baoc_internal.h"

namespace baoc {

struct alignas(8) Chunk {
    uint64_t grad_start;    // element index into the caller's flat gradient buffer
    uint64_t state_start;   // element index into m / v / g_prev (multiple of 256)
    uint32_t count;         // coordinates in the chunk (only a block's last chunk may end off a multiple of 256)
    uint32_t block;
};

struct alignas(8) BlockRow {
    uint64_t grad_start;    // the block's offset in the caller's flat gradient buffer
    uint64_t state_start;
    uint64_t numel;
    uint32_t first_chunk, n_chunks;
    uint32_t groups_per_chunk;
    uint32_t first_prow, n_prows;   // the block's partial rows of the step kernel (one per workgroup: chunk x slice)
    uint32_t pad_;
};

struct StepConsts {
    float beta_m, beta_v, om_m, om_v, eps_u;
};

struct FoldArgs {
    const BlockRow* rows;
    uint32_t* arrived;
    double* rec_all;
    double beta_rho, eps;
};

typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint32_t u2 __attribute__((ext_vector_type(2)));

// ---------------------------------------------------------------------------
// wavefront reductions on the DPP crossbar (64 lanes = 4 rows of 16)
// ---------------------------------------------------------------------------

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp(float old, float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
        __builtin_bit_cast(int, old), __builtin_bit_cast(int, x), CTRL, ROW_MASK, 0xf, false));
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t old, uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)x, CTRL, ROW_MASK, 0xf, false);
}

// quad_perm[1,0,3,2]=0xB1, quad_perm[2,3,0,1]=0x4E, row_ror:4=0x124, row_ror:8=0x128 leave every
// lane of a row with the row's total; row_bcast:15 (0x142, rows 1 and 3) and row_bcast:31
// (0x143, rows 2 and 3) carry the totals upwards so that lane 63 ends with the wavefront's.
//
// Largest of the lanes' non-negative binary32 values.  Among non-negative values the order of the
// bit patterns as unsigned integers is the order of the values, so the reduction runs on integers
// (one v_max_u32 with a DPP operand per level).  A NaN pattern ranks above +inf, so a NaN anywhere
// in the group comes out as the maximum; such a group's sums are NaN whatever its scale is.
__device__ __forceinline__ float wave_max_nonneg(float v)
{
    uint32_t x = __builtin_bit_cast(uint32_t, v);
    x = max(x, dpp_u32<0xB1, 0xf>(0u, x));
    x = max(x, dpp_u32<0x4E, 0xf>(0u, x));
    x = max(x, dpp_u32<0x124, 0xf>(0u, x));
    x = max(x, dpp_u32<0x128, 0xf>(0u, x));
    x = max(x, dpp_u32<0x142, 0xa>(0u, x));
    x = max(x, dpp_u32<0x143, 0xc>(0u, x));
    return __builtin_bit_cast(float, (uint32_t)__builtin_amdgcn_readlane((int)x, 63));
}

__device__ __forceinline__ float wave_sum(float x)
{
    x += dpp<0xB1, 0xf>(0.f, x);
    x += dpp<0x4E, 0xf>(0.f, x);
    x += dpp<0x124, 0xf>(0.f, x);
    x += dpp<0x128, 0xf>(0.f, x);
    x += dpp<0x142, 0xa>(0.f, x);
    x += dpp<0x143, 0xc>(0.f, x);
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), 63));
}

// ---------------------------------------------------------------------------
// element helpers
// ---------------------------------------------------------------------------

__device__ __forceinline__ float bf16_widen(uint32_t h) { return __builtin_bit_cast(float, h << 16); }

// Round-to-nearest-even of two binary32 values to the bf16 grid, widened back.  One
// v_cvt_pk_bf16_f32 (gfx950) converts both; the halves are then moved back to the top of a word.
typedef float f2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void bf16_round2(float a, float b, float& ra, float& rb)
{
    const f2 x = {a, b};
    const uint32_t w = __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf2));
    ra = __builtin_bit_cast(float, w << 16);
    rb = __builtin_bit_cast(float, w & 0xffff0000u);
}

// u = m / (sqrt(v) + eps_u) with the hardware's 1-ulp square root and reciprocal
__device__ __forceinline__ float direction(float m, float v, float eps_u)
{
    return m * __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf(v) + eps_u);
}

// Preconditioner of Eq. 6, p = 1 / (sqrt(v) + eps), with one transcendental instead of two where eps is small
// against sqrt(v): with r = 1/sqrt(v), p = r / (1 + eps r) = r (1 - eps r) up to (eps r)^2 < 1e-6.  Elsewhere
// (v tiny, zero, sub-normal or NaN) the plain form.
__device__ __forceinline__ float preconditioner_series(float v, float eps)
{
    const float r = __builtin_amdgcn_rsqf(v);
    return __builtin_fmaf(-(eps * r), r, r);
}

__device__ __forceinline__ float preconditioner(float v, float eps)
{
    const float r = __builtin_amdgcn_rsqf(v);
    const float er = eps * r;
    float p = __builtin_fmaf(-er, r, r);
    if (!(er < 1e-3f)) p = __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf(v) + eps);
    return p;
}

// Every array is touched exactly once per pass: the states are loaded with the nontemporal hint so the
// stream does not displace anything in L2 / MALL on its way through.
template <typename T> __host__ __device__ __forceinline__ T ld_stream(const void* p)
{
    return __builtin_nontemporal_load(reinterpret_cast<const T*>(p));
}

// How a step's stores and gradient loads pass the caches (states are always loaded with the hint):
//   kThrough  stores carry the hint and go through to memory, so that no line stays in the L2 to be written back between the
//             reads of others; the gradient is loaded without the hint.  Large layouts.  (On one workspace, hint on all accesses ->
//             stores through -> the gradient without the hint: 3.5 G coordinates bf16 12.79 -> 12.60 -> 12.22 ms, 1.3 G fp32 5.76 ->
//             5.67 -> 5.67, bf16 4.83 -> 4.73 -> 4.56, 60 M bf16 at odd offsets 216 -> 212 -> 202 us.)
//   kKept     stores go through to memory without the hint and stay in the memory-side cache.  Layouts whose states fill half of it
//             at most.
//   kHinted   the hint on all accesses, stores wait in the L2.  fp32 layouts between kSmallLayout and kHintedLayout.
// us a step, kThrough and kKept: fp32 2 M coordinates 14.1 and 13.0, 8 M 39.6 and 38.4, 17 M 77 and 76, 25 M 108 and 124; bf16 2 M 12.8
// and 11.5, 8 M 33.3 and 30.9, 17 M 62 and 59, 25 M 88 and 94.  (In a training step other kernels pass between two of these, so the line
// lies below the 170 to 200 MB where kKept begins to lose here.)  kThrough and kHinted, each with its best workgroups, fp32: 34 M 147 to
// 159 and 152 to 161, 42 M 189 to 198 and 185 to 192, 48 M 214 to 236 and 211 to 234, 55 M 245 to 253 and 245 to 255, 62 M 277 to 286
// and 279 to 291.
enum Memory : int { kThrough, kKept, kHinted };
constexpr uint64_t kKeptBytes = 128ull << 20;             // of states
template <int MEM> constexpr int kStoreBits = MEM == kThrough ? 2 | 16 : MEM == kKept ? 16 : 2;   // nt = 2, sc1 = 16

// A chunk's part of one state array, as a buffer: no builtin sets these bits on a 16-byte global store.
typedef __amdgpu_buffer_rsrc_t StateArray;
template <typename E> __device__ __forceinline__ StateArray state_array(E* first, uint32_t n)
{
    return __builtin_amdgcn_make_buffer_rsrc(first, 0, n * sizeof(E), 0x00020000);
}
template <int MEM> __device__ __forceinline__ void st_state(StateArray a, uint32_t byte, f4 x)
{
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, x), a, byte, 0, kStoreBits<MEM>);
}
template <int MEM> __device__ __forceinline__ void st_state(StateArray a, uint32_t byte, u2 x)
{
    __builtin_amdgcn_raw_buffer_store_b64(x, a, byte, 0, kStoreBits<MEM>);
}

template <int GT> struct GradIO;

// Loads of the caller's buffers (gradients, parameters) assume the alignment of one element only: gfx950 takes global
// loads at any address, and a 16- or 8-byte load that crosses a cache line is still one request where four
// element loads are four (step on bf16 blocks packed at odd offsets, 60 M coordinates: 271 -> 224 us a launch).
template <> struct GradIO<BAOC_GRAD_F32> {
    typedef float elem;
    typedef f4 vec4;                                      // four elements as loaded
    typedef f4 vec4_any __attribute__((aligned(4)));
    __host__ __device__ static __forceinline__ vec4 loadv(const elem* p) { return ld_stream<f4>(p); }
    __host__ __device__ static __forceinline__ vec4 loadv_any(const elem* p) { return ld_stream<vec4_any>(p); }
    __host__ __device__ static __forceinline__ vec4 loadv_shared(const elem* p) { return *reinterpret_cast<const vec4_any*>(p); }
    __device__ static __forceinline__ void unpack(vec4 t, float g[4]) { g[0] = t.x; g[1] = t.y; g[2] = t.z; g[3] = t.w; }
    __device__ static __forceinline__ float load1(const elem* p) { return *p; }
    template <int MEM> __device__ static __forceinline__ void store4(StateArray a, uint32_t e, const float g[4])
    {
        st_state<MEM>(a, e * 4, f4{g[0], g[1], g[2], g[3]});
    }
};

template <> struct GradIO<BAOC_GRAD_BF16> {
    typedef uint16_t elem;
    typedef u2 vec4;
    typedef u2 vec4_any __attribute__((aligned(2)));
    __host__ __device__ static __forceinline__ vec4 loadv(const elem* p) { return ld_stream<u2>(p); }
    __host__ __device__ static __forceinline__ vec4 loadv_any(const elem* p) { return ld_stream<vec4_any>(p); }
    __host__ __device__ static __forceinline__ vec4 loadv_shared(const elem* p) { return *reinterpret_cast<const vec4_any*>(p); }
    __device__ static __forceinline__ void unpack(vec4 t, float g[4])
    {
        g[0] = __builtin_bit_cast(float, t.x << 16); g[1] = __builtin_bit_cast(float, t.x & 0xffff0000u);
        g[2] = __builtin_bit_cast(float, t.y << 16); g[3] = __builtin_bit_cast(float, t.y & 0xffff0000u);
    }
    __device__ static __forceinline__ float load1(const elem* p) { return bf16_widen(*p); }
    // g holds exact bf16 values: the upper half of each word is the stored pattern
    template <int MEM> __device__ static __forceinline__ void store4(StateArray a, uint32_t e, const float g[4])
    {
        u2 t;
        t.x = (__builtin_bit_cast(uint32_t, g[0]) >> 16) | (__builtin_bit_cast(uint32_t, g[1]) & 0xffff0000u);
        t.y = (__builtin_bit_cast(uint32_t, g[2]) >> 16) | (__builtin_bit_cast(uint32_t, g[3]) & 0xffff0000u);
        st_state<MEM>(a, e * 2, t);
    }
};

// ---------------------------------------------------------------------------
// what crosses workgroups inside a launch
// ---------------------------------------------------------------------------

// Written by device-scope atomics and stores that go through to memory, and read the same way, so no cache is written back
// or invalidated; vmcnt(0) before the arrival counter is all the order they need.
template <typename T> __device__ __forceinline__ void st_device(T* p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T> __device__ __forceinline__ T ld_device(const T* p) { return __hip_atomic_load(const_cast<T*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

constexpr uint32_t kArriveStride = 32;    // words from one block's arrival counter to the next: atomics on one cache line queue up

// Called by a whole workgroup: true in the last of the n that share the counter, which is then back at zero.
__device__ __forceinline__ bool arrive_last(uint32_t* counter, uint32_t n)
{
    __shared__ uint32_t last;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");          // this wavefront's stores and atomics have been performed
    __syncthreads();
    if (threadIdx.x == 0) {
        last = n == 1 || __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n - 1;
        if (last && n > 1) st_device(counter, 0u);
    }
    __syncthreads();
    return last;
}

// ---------------------------------------------------------------------------
// a step's sums into the block's record
// ---------------------------------------------------------------------------

// What fold_step needs of the record, asked for by every thread before the sums: five loads one after another at the end of a launch
// are what a small step then waits for.
__device__ __forceinline__ double fold_state(const double* rec) { return rec[R_SPP + (threadIdx.x & 7u)]; }
static_assert(R_RHO == R_SPP + 1 && R_NCOS == R_SPP + 3 && R_STEPS == R_SPP + 4 && R_SPP + 8 <= kRecDoubles, "lanes of fold_state");

// Thread s < 16 of the workgroup holds sum s of the block; `state` is fold_state's.
__device__ __forceinline__ void fold_step(double total, double state, double* rec, double beta_rho, double eps)
{
    const uint32_t tid = threadIdx.x;
    if (tid < kNumSums) rec[tid] = total;
    // Fold the step into the running direction stability (Eq. 5, left):
    //   cos_t = <g_t,g_{t-1}> / (|g_t| |g_{t-1}| + eps), NaN -> 0 (App. A.1);
    //   the first cosine initialises rho_bar, later ones enter with weight 1 - beta_rho.
    static_assert(S_GG == 0 && S_GP == 1, "lane 0 holds |g|^2 and takes <g, g'> from lane 1");
    if (tid < 64) {
        const double S_gp = __shfl_down(total, 1);
        const double spp = __shfl(state, 0), rho = __shfl(state, 1), cosines = __shfl(state, 3), steps = __shfl(state, 4);
        if (tid == 0) {
            // The step index lives in the block's record, not in a launch argument: a captured launch of a
            // steady-state step can be replayed for later steps.
            const uint32_t step = (uint32_t)steps + 1u;
            if (step >= 2) {
                double c = S_gp / (sqrt(total) * sqrt(spp) + eps);
                if (c != c) c = 0.0;
                rec[R_RHO] = (cosines == 0.0) ? c : beta_rho * rho + (1.0 - beta_rho) * c;
                rec[R_COS] = c;
                rec[R_NCOS] = cosines + 1.0;
            }
            rec[R_SPP] = total;
            rec[R_STEPS] = (double)step;
        }
    }
}

// ---------------------------------------------------------------------------
// the fused per-step pass
// ---------------------------------------------------------------------------

// FIRST: the states are known to be zero (first step after begin), so they are not read.
// A workgroup of NW wavefronts takes one slice of a chunk (`slice_groups` quantisation groups, `slices`
// slices per chunk) and writes one partial row.  G: groups a wavefront takes per round, next to each
// other (G * 1 KB of m and of v per wavefront and round); the workgroup covers NW * G groups per round.
// The loads of a round are issued together, one round ahead of their use.  With the default shapes a
// slice is a single round, so no wavefront ever waits on its own stores.
// FOLD (small layouts): the workgroup of a block that arrives last adds the block's partial rows and folds the step into
// its record; otherwise k_reduce does.
template <int GT, bool FIRST, int G, int NW, bool FOLD, int MEM>
__global__ __launch_bounds__(64 * NW) void k_step(
    const typename GradIO<GT>::elem* __restrict__ grad,
    float* __restrict__ m_all, float* __restrict__ v_all,
    typename GradIO<GT>::elem* __restrict__ gp_all,
    const Chunk* __restrict__ chunks, float* __restrict__ partials, StepConsts k,
    uint32_t slices, uint32_t slice_groups, FoldArgs fold)
{
    typedef GradIO<GT> IO;
    const uint32_t chunk = blockIdx.x / slices, slice = blockIdx.x - chunk * slices;
    const Chunk ck = chunks[chunk];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    uint32_t fold_rows = 0, fold_first = 0;
    double* fold_rec = nullptr;
    double fold_before = 0.0;
    if (FOLD) {
        fold_rows = fold.rows[ck.block].n_prows; fold_first = fold.rows[ck.block].first_prow;
        fold_rec = fold.rec_all + (uint64_t)ck.block * kRecDoubles;
        fold_before = fold_state(fold_rec);
    }
    // this workgroup's groups of the chunk: [g_begin, ngroups)
    const uint32_t g_begin = slice * slice_groups;
    const uint32_t ngroups = min((ck.count + (kQB - 1)) / kQB, g_begin + slice_groups);
    const typename IO::elem* gsrc = grad + ck.grad_start;
    const uint32_t padded = (ck.count + (kQB - 1)) / kQB * kQB;
    const StateArray m_dst = state_array(m_all + ck.state_start, padded), v_dst = state_array(v_all + ck.state_start, padded);
    const StateArray gp_dst = state_array(gp_all + ck.state_start, padded);

    float acc[kNumSums];
#pragma unroll
    for (int i = 0; i < (int)kNumSums; ++i) acc[i] = 0.f;

    typedef typename IO::vec4 GV;
    f4 nm[G], nv[G];
    GV np[G], ng[G];
#pragma unroll
    for (int i = 0; i < G; ++i) { nm[i] = f4{0.f, 0.f, 0.f, 0.f}; nv[i] = nm[i]; np[i] = GV{}; ng[i] = GV{}; }
    auto issue = [&](uint32_t first) {                    // first: the wavefront's first group of a round
#pragma unroll
        for (int i = 0; i < G; ++i) {
            const uint32_t grp = first + i;
            if (grp < ngroups) {
                const uint32_t e = grp * kQB + lane * 4;
                const uint64_t si = ck.state_start + e;   // states are padded to whole groups
                if (!FIRST) { nm[i] = ld_stream<f4>(m_all + si); nv[i] = ld_stream<f4>(v_all + si); np[i] = IO::loadv(gp_all + si); }
                if (e + 4 <= ck.count) ng[i] = MEM == kHinted ? IO::loadv_any(gsrc + e) : IO::loadv_shared(gsrc + e);
            }
        }
    };
    if (g_begin + wave * G < ngroups) issue(g_begin + wave * G);

    for (uint32_t first = g_begin + wave * G; first < ngroups; first += NW * G) {
        f4 cm[G], cv[G];
        GV cp[G], cg[G];
#pragma unroll
        for (int i = 0; i < G; ++i) { cm[i] = nm[i]; cv[i] = nv[i]; cp[i] = np[i]; cg[i] = ng[i]; }
        if (first + NW * G < ngroups) issue(first + NW * G);
#pragma unroll
        for (int i = 0; i < G; ++i) {
            const uint32_t grp = first + i;
            if (grp >= ngroups) break;
            const uint32_t e = grp * kQB + lane * 4;          // first of this lane's 4 coordinates
            float g[4], p[4], m[4], v[4];
            if (FIRST) {
#pragma unroll
                for (int j = 0; j < 4; ++j) m[j] = v[j] = p[j] = 0.f;
            } else {
                m[0] = cm[i].x; m[1] = cm[i].y; m[2] = cm[i].z; m[3] = cm[i].w;
                v[0] = cv[i].x; v[1] = cv[i].y; v[2] = cv[i].z; v[3] = cv[i].w;
                IO::unpack(cp[i], p);
            }
            if (e + 4 <= ck.count) {
                IO::unpack(cg[i], g);
            } else {                                          // ragged tail
#pragma unroll
                for (int j = 0; j < 4; ++j) g[j] = (e + j < ck.count) ? IO::load1(gsrc + e + j) : 0.f;
            }

            // Eq. 3 in fp32: the new term is rounded, then one fused multiply-add
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float tm = k.om_m * g[j];
                const float tv = (k.om_v * g[j]) * g[j];
                m[j] = __builtin_fmaf(k.beta_m, m[j], tm);
                v[j] = __builtin_fmaf(k.beta_v, v[j], tv);
            }
            {
                st_state<MEM>(m_dst, e * 4, f4{m[0], m[1], m[2], m[3]});
                st_state<MEM>(v_dst, e * 4, f4{v[0], v[1], v[2], v[3]});
            }
            IO::template store4<MEM>(gp_dst, e, g);

            // group absmax of the 256 coordinates this wavefront holds
            const float a_m = wave_max_nonneg(fmaxf(fmaxf(fabsf(m[0]), fabsf(m[1])), fmaxf(fabsf(m[2]), fabsf(m[3]))));
            const float a_v = wave_max_nonneg(fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])));
            // 8-bit code = rint(x * (L / a)) decided in fp32 with a correctly rounded quotient;
            // an infinite scale (a == 0 or tiny) means all codes are 0
            float s_m = 127.0f / a_m, s_v = 255.0f / a_v;
            s_m = s_m < INFINITY ? s_m : 0.f;
            s_v = s_v < INFINITY ? s_v : 0.f;
            const float d_m = a_m * (1.0f / 127.0f), d_v = a_v * (1.0f / 255.0f);

#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float mj = m[j], vj = v[j];
                acc[S_GG] = __builtin_fmaf(g[j], g[j], acc[S_GG]);
                acc[S_GP] = __builtin_fmaf(g[j], p[j], acc[S_GP]);
                acc[S_MM] = __builtin_fmaf(mj, mj, acc[S_MM]);
                acc[S_V1] += vj;
                acc[S_VV] = __builtin_fmaf(vj, vj, acc[S_VV]);
                const float u32 = direction(mj, vj, k.eps_u);
                acc[U0] = __builtin_fmaf(u32, u32, acc[U0]);
                {   // bf16 round trip
                    float mb, vb;
                    bf16_round2(mj, vj, mb, vb);
                    const float ub = direction(mb, vb, k.eps_u);
                    const float du = ub - u32, dm = mb - mj, dv = vb - vj;
                    acc[U1_16] = __builtin_fmaf(u32, ub, acc[U1_16]);
                    acc[D_16] = __builtin_fmaf(du, du, acc[D_16]);
                    acc[U2_16] = __builtin_fmaf(ub, ub, acc[U2_16]);
                    acc[EM_16] = __builtin_fmaf(dm, dm, acc[EM_16]);
                    acc[EV_16] = __builtin_fmaf(dv, dv, acc[EV_16]);
                }
                {   // block-wise absmax 8-bit round trip
                    const float mb = __builtin_rintf(mj * s_m) * d_m;
                    const float vb = __builtin_rintf(vj * s_v) * d_v;
                    const float ub = direction(mb, vb, k.eps_u);
                    const float du = ub - u32, dm = mb - mj, dv = vb - vj;
                    acc[U1_8] = __builtin_fmaf(u32, ub, acc[U1_8]);
                    acc[D_8] = __builtin_fmaf(du, du, acc[D_8]);
                    acc[U2_8] = __builtin_fmaf(ub, ub, acc[U2_8]);
                    acc[EM_8] = __builtin_fmaf(dm, dm, acc[EM_8]);
                    acc[EV_8] = __builtin_fmaf(dv, dv, acc[EV_8]);
                }
            }
        }
    }

    // Sixteen sums held by sixteen lanes: a halving exchange inside each row of 16 lanes (after the
    // level that pairs lanes differing in bit b, a lane keeps only the sums whose index has its own
    // bit b) leaves lane l of a row with that row's total of sum l & 15, in 8+4+2+1 DPP additions.
    // Then LDS (4 wavefronts x 4 rows) -> one partial row per workgroup, in a fixed order.
    static_assert(kNumSums == 16, "the exchange below is written for 16 sums");
    {
        const bool b3 = lane & 8u, b2 = lane & 4u, b1 = lane & 2u, b0 = lane & 1u;
#pragma unroll
        for (int i = 0; i < 8; ++i) {                     // partner lane ^ 8 (row_ror:8)
            const float keep = b3 ? acc[i + 8] : acc[i], send = b3 ? acc[i] : acc[i + 8];
            acc[i] = keep + dpp<0x128, 0xf>(0.f, send);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {                     // partner 7 - (lane & 7) in the same half (row_half_mirror)
            const float keep = b2 ? acc[i + 4] : acc[i], send = b2 ? acc[i] : acc[i + 4];
            acc[i] = keep + dpp<0x141, 0xf>(0.f, send);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {                     // partner lane ^ 2
            const float keep = b1 ? acc[i + 2] : acc[i], send = b1 ? acc[i] : acc[i + 2];
            acc[i] = keep + dpp<0x4E, 0xf>(0.f, send);
        }
        const float keep = b0 ? acc[1] : acc[0], send = b0 ? acc[0] : acc[1];
        acc[0] = keep + dpp<0xB1, 0xf>(0.f, send);       // partner lane ^ 1
    }
    __shared__ float red[NW * 4 * kNumSums];              // [wavefront * 4 + row][sum]
    red[threadIdx.x] = acc[0];
    __syncthreads();
    float s = 0.f;
    if (threadIdx.x < kNumSums) {
#pragma unroll
        for (int q = 0; q < NW * 4; ++q) s += red[q * kNumSums + threadIdx.x];
        float* out = partials + (uint64_t)blockIdx.x * kNumSums + threadIdx.x;
        if (!FOLD) *out = s;
        else if (fold_rows > 1) st_device(out, s);
    }
    if (FOLD) {
        double total = (double)s;
        if (fold_rows > 1) {
            if (!arrive_last(fold.arrived + ck.block * kArriveStride, fold_rows)) return;
            __shared__ double sh[NW * 4][kNumSums];
            const float* base = partials + (uint64_t)fold_first * kNumSums;
            double t = 0.0;
#pragma unroll 8
            for (uint32_t r = threadIdx.x / kNumSums; r < fold_rows; r += NW * 4) t += (double)ld_device(base + (uint64_t)r * kNumSums + threadIdx.x % kNumSums);
            sh[threadIdx.x / kNumSums][threadIdx.x % kNumSums] = t;
            __syncthreads();
            total = 0.0;
            if (threadIdx.x < kNumSums) {
#pragma unroll
                for (int q = 0; q < NW * 4; ++q) total += sh[q][threadIdx.x];
            }
        }
        fold_step(total, fold_before, fold_rec, fold.beta_rho, fold.eps);
    }
}

// Per-block sums of the partial rows, in fp64.  A block of more than kDirectRows rows is summed in parts first (k_reduce_parts,
// one workgroup each); k_reduce adds a block's rows, or the sums of its parts, and folds the step into the block's record. Bound
// by latency: a chain of descriptor load, row loads and reduction, and for the largest layouts by the rows themselves (64 B for
// every 256 coordinates of a large fp32 layout).  A lane reads 16 bytes of a row, a wavefront 1 KB at a time, a workgroup 32 KB
// per round; the 64 row slots of a sum meet in two exchange levels and one trip through LDS.  Measured (16 LDS trees of eight
// barriers and parts of 4,096 rows before): 32,768 coordinates 14.3 -> 3.0 us.  Both launches: 124 M fp32, 486,000 rows, 17 us;
// 860 M 50 us; 1.3 G 68 us, where the rows, 329 MB, are more than the memory-side cache holds (half as many rows took 30).  One
// launch in which the last part of a block to arrive folds it was slower where there are many parts (1.3 G with half the rows:
// 106 us): its release writes back the whole L2 of an XCD for every part. kDirectRows: the second launch costs 4.7 us, about what
// six rounds take.  (With 6,144 rows and parts of 2,048 k_reduce of 860 M in 686 blocks takes 12.6 us instead of 7.5, a step of
// 74 M coordinates 340 instead of 333.)
constexpr uint32_t kPartRows = 1024, kDirectRows = 3072;

struct alignas(8) Part { uint32_t block, part; };

// Sum of n partial rows; thread s < 16 returns sum s.  Called by a whole workgroup of 256.
__device__ __forceinline__ double sum_rows(const float* __restrict__ partials, uint32_t n, double (*sh)[kNumSums])
{
    const uint32_t tid = threadIdx.x, quad = tid & 3u, slot = tid >> 2;
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    for (uint32_t c = slot; c < n; c += 512) {
        f4 x[8];
#pragma unroll
        for (int q = 0; q < 8; ++q)
            x[q] = c + 64 * q < n ? *reinterpret_cast<const f4*>(partials + (uint64_t)(c + 64 * q) * kNumSums + 4 * quad) : f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < 8; ++q) { a[0] += (double)x[q].x; a[1] += (double)x[q].y; a[2] += (double)x[q].z; a[3] += (double)x[q].w; }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {                              // the four slots of a row of 16 lanes
        a[i] += __shfl_xor(a[i], 4);
        a[i] += __shfl_xor(a[i], 8);
    }
    if ((tid & 12u) == 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) sh[tid >> 4][4 * quad + i] = a[i];
    }
    __syncthreads();
    double total = 0.0;
    if (tid < kNumSums) {
#pragma unroll
        for (int q = 0; q < 16; ++q) total += sh[q][tid];
    }
    return total;
}

// A block's rows are cut into n_prows / kPartRows parts, the last one with the remainder (so no part has fewer than
// two rows).  The part's sums take the place of its first two rows, which nobody else reads.
__global__ __launch_bounds__(256) void k_reduce_parts(float* partials, const BlockRow* __restrict__ rows, const Part* __restrict__ parts)
{
    __shared__ double sh[16][kNumSums];
    const Part p = parts[blockIdx.x];
    const uint32_t first = p.part * kPartRows, left = rows[p.block].n_prows - first;
    const uint32_t n = left < 2 * kPartRows ? left : kPartRows;
    float* mine = partials + (uint64_t)(rows[p.block].first_prow + first) * kNumSums;
    const double total = sum_rows(mine, n, sh);
    if (threadIdx.x < kNumSums) reinterpret_cast<double*>(mine)[threadIdx.x] = total;
}

__global__ __launch_bounds__(256) void k_reduce(const float* __restrict__ partials, const BlockRow* __restrict__ rows,
                                                double* __restrict__ rec_all, double beta_rho, double eps)
{
    __shared__ double sh[16][kNumSums];
    const uint32_t tid = threadIdx.x, n_prows = rows[blockIdx.x].n_prows;
    const float* base = partials + (uint64_t)rows[blockIdx.x].first_prow * kNumSums;
    double* rec = rec_all + (uint64_t)blockIdx.x * kRecDoubles;
    const double before = fold_state(rec);
    double total = 0.0;
    if (n_prows <= kDirectRows) {
        total = sum_rows(base, n_prows, sh);
    } else {
        const uint32_t s = tid & 15u, g = tid >> 4, n_parts = n_prows / kPartRows;
        double t = 0.0;
#pragma unroll 4
        for (uint32_t q = g; q < n_parts; q += 16)
            t += reinterpret_cast<const double*>(base + (uint64_t)q * kPartRows * kNumSums)[s];
        sh[g][s] = t;
        __syncthreads();
        if (tid < kNumSums) {
#pragma unroll
            for (int q = 0; q < 16; ++q) total += sh[q][tid];
        }
    }
    fold_step(total, before, rec, beta_rho, eps);
}

// ---------------------------------------------------------------------------
// Finalize: three passes over the blocks' workgroups, and two small launches between them
// (large layouts read v once instead, see baoc_once.h, and come here with the blocks that this leaves)
//   k_final1: first radix digit (Eq. 4); sum of p = 1/(sqrt(v)+eps) (Eq. 6); matrix blocks: mu, row and
//             column partial sums (Eq. 7)
//   k_fold1:  first digit of the ranks, sums, r and c, where a block has several workgroups
//   k_final2: second digit; ((p/p-bar - 1) theta)^2 and theta^2 (Eq. 6); |S - r c^T / mu|^2 (Eq. 7; |S|^2 is the
//             step's own sum of v^2)
//   k_fold2:  second digit of the ranks, sums, where a block has several workgroups
//   k_final3: last digit
// The quantiles are exact order statistics, found by a three-digit radix selection on the bit patterns (v >= 0, so
// the pattern order is the value order).  Digits: bits 30..19, 18..9, 8..0.  Four ranks per block share every pass.
// A block of one workgroup is folded by it, from LDS.  A block of several is folded between the passes: with a counter per block and
// the last workgroup to arrive doing it, every workgroup holds its place until its atomics and the counter have answered, and the last
// one's chain of loads ends the pass (passes of 25.6 M coordinates 36 + 49 us, now 27 + 43 and 5 + 5 for the launches between them; 124 M
// 106 + 146, now 94 + 141 and 6 + 5; 32,768 coordinates, one workgroup a block, 29 us of kernels, now 18).  Pass 3 is short, and its
// last workgroup does fold.
// ---------------------------------------------------------------------------

// How finalize walks a block: tiles of a matrix (rows, cols > 0) or runs of coordinates (rows = cols = 0), a
// workgroup (task) each.
struct alignas(8) TileRow {
    uint64_t state_start;                 // first coordinate of the block in v
    uint64_t grad_start;                  // the block's offset in the caller's flat buffers (theta)
    uint64_t numel;
    uint64_t off_r, off_c;                // into the r / c vectors (floats)
    uint64_t off_rowpart, off_colpart;    // into the partial-sum arrays (floats): [tile][row] and [seg][column]
    uint64_t cand_base;                   // the block's first candidate list (words into the candidate buffer)
    uint32_t rows, cols;
    uint32_t n_tiles, n_segs;             // tiles side by side and below each other
    uint32_t strips, n_across;            // neighbouring tiles that a task takes one after another; tasks side by side
    uint32_t seg_len;                     // rows of a tile, or coordinates of a run
    uint32_t wc_log;                      // a tile is seg_len x (64 << wc_log)
    uint32_t first_task;
    uint32_t cand_cap;                    // words per candidate list (one list per wavefront)
    uint32_t first_fin;                   // first of the block's workgroups that fold row and column sums in k_fold1
    uint32_t n_tasks;                     // workgroups of a pass over the block
    uint32_t rank[4];                     // order statistics wanted from v: lo(0.1), lo+1, lo(0.9), lo+1
};

constexpr uint32_t kHistWords = 4096;     // histogram words a block owns
constexpr uint32_t kBits2 = 10, kBits3 = 9;                       // 12 + 10 + 9 bits of the 31-bit key
constexpr uint32_t kShift1 = kBits2 + kBits3, kShift2 = kBits3;   // key >> kShift1: first digit; key >> kShift2: first two
constexpr uint32_t kBins1 = 1u << (31 - kShift1), kBins2 = 1u << kBits2, kBins3 = 1u << kBits3;
static_assert(kBins1 <= kHistWords && 4 * kBins2 <= kHistWords && 4 * kBins3 <= kHistWords, "one first-digit histogram, four of the others");

// A block's share of the pass that reads v once (baoc_once.h).  Offsets count 64-byte units from the vectors r and c on.
struct alignas(16) OnceRow {
    uint32_t first_task, first_wide;          // of the tasks of 8 and of those of 16 wavefronts
    uint32_t n_tasks;                         // 0: the block goes through the passes here
    uint32_t first_unit;                      // of k_once_select
    uint32_t geom;                            // lanes_log | strips << 4 | across << 8 | down << 16 | 16 wavefronts << 24
    uint32_t off_list, list_cap;              // a list per task, its words; then one of half their size for what these have no room for
    uint32_t off_cols;                        // [task][column] float2, then the collected keys of both intervals
};

// Words of a block's arrival line.
enum Line : uint32_t { L_COUNT, L_SCAN3, L_REDO, L_ARRIVED, L_KEYS, L_SPILL = L_KEYS + 2, L_BRACKET = 8, L_INV_P0 = 12 };

// Whether the one pass has done with a block; `scan3` points at L_SCAN3 of the first block.
__device__ __forceinline__ bool settled(const OnceRow* once, const uint32_t* scan3, uint32_t block)
{
    return once && once[block].n_tasks && !scan3[block * kArriveStride + (L_REDO - L_SCAN3)];
}

// Tables that begin() leaves on the device, and the clearing of what must start at zero: chunks from the block rows
// (the owning block by bisection on first_chunk; a block's groups are split evenly over its chunks, whole groups
// each) and the owning block of every workgroup of the finalize passes and of k_fold1.
__global__ __launch_bounds__(256) void k_build(const BlockRow* __restrict__ rows, const TileRow* __restrict__ tiles, uint32_t n_blocks,
                                               Chunk* __restrict__ chunks, uint32_t n_chunks, uint32_t* __restrict__ task_block, uint32_t n_tasks,
                                               uint32_t* __restrict__ fin_block, uint32_t n_fin, uint4* __restrict__ clear, uint64_t n_clear)
{
    const uint64_t id0 = (uint64_t)blockIdx.x * 256 + threadIdx.x, stride = (uint64_t)gridDim.x * 256;
    auto owner = [&](uint32_t id, auto first_of) {
        uint32_t lo = 0, hi = n_blocks - 1;
        while (lo < hi) {
            const uint32_t mid = (lo + hi + 1) >> 1;
            if (first_of(mid) <= id) lo = mid; else hi = mid - 1;
        }
        return lo;
    };
    for (uint64_t c = id0; c < n_chunks; c += stride) {
        const uint32_t b = owner((uint32_t)c, [&](uint32_t i) { return rows[i].first_chunk; });
        const BlockRow r = rows[b];
        const uint64_t g0 = (c - r.first_chunk) * r.groups_per_chunk;
        const uint64_t groups = (r.numel + kQB - 1) / kQB;
        const uint64_t g1 = min(groups, g0 + r.groups_per_chunk);
        Chunk ck;
        ck.grad_start = r.grad_start + g0 * kQB;
        ck.state_start = r.state_start + g0 * kQB;
        ck.count = (uint32_t)(min(r.numel, g1 * kQB) - g0 * kQB);
        ck.block = b;
        chunks[c] = ck;
    }
    for (uint64_t t = id0; t < n_tasks; t += stride) task_block[t] = owner((uint32_t)t, [&](uint32_t i) { return tiles[i].first_task; });
    for (uint64_t f = id0; f < n_fin; f += stride) fin_block[f] = owner((uint32_t)f, [&](uint32_t i) { return tiles[i].first_fin; });
    for (uint64_t i = id0; i < n_clear; i += stride) clear[i] = uint4{0u, 0u, 0u, 0u};
}

// Per block: histogram words; four key prefixes and four ranks within them, which stand in the record where the order statistics come (not next to
// the arrival counter, whose line goes back and forth between the last pass's workgroups).
struct Selection { uint32_t *hist, *prefix, *rank; };
constexpr uint32_t kSelStride = 2 * kRecDoubles;

// The four ranks of a block usually share their key prefix pairwise (lo and lo+1 of a quantile fall
// into one bin).  Elements are matched against the distinct prefixes only; slot_of[t] names the
// histogram that serves rank t.
struct Prefixes { uint32_t pre[4]; uint32_t slot_of[4]; uint32_t n; };
constexpr uint32_t kNoPrefix = 0xffffffffu;             // never equals a key prefix (at most 22 bits)
__device__ __forceinline__ Prefixes distinct_prefixes(const uint32_t* __restrict__ sel_prefix, uint32_t block)
{
    // fully unrolled with static indices so that everything stays in (scalar) registers
    Prefixes d;
    d.n = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) d.pre[j] = kNoPrefix;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const uint32_t p = sel_prefix[block * kSelStride + t];
        uint32_t slot = 4;
#pragma unroll
        for (int j = 3; j >= 0; --j)
            if (d.pre[j] == p) slot = j;
        const bool fresh = slot == 4;
        if (fresh) slot = d.n;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (fresh && (uint32_t)j == d.n) d.pre[j] = p;
        if (fresh) d.n += 1;
        d.slot_of[t] = slot;
    }
    return d;
}

// h[u * nb + bin] += 1 for the slot u whose prefix equals hi (the prefixes are distinct, so at most
// one does): the slot is selected first and a single LDS atomic follows.  Slots 2 and 3 are rarely in use.
__device__ __forceinline__ void count_match(uint32_t* h, const Prefixes& d, uint32_t nb, uint32_t hi, uint32_t bin)
{
    bool hit = hi == d.pre[0];
    uint32_t at = bin;
    if (hi == d.pre[1]) { at = nb + bin; hit = true; }
    if (d.n > 2) {
        if (hi == d.pre[2]) { at = 2 * nb + bin; hit = true; }
        if (hi == d.pre[3]) { at = 3 * nb + bin; hit = true; }
    }
    if (hit) atomicAdd(&h[at], 1u);
}

// Inclusive sum over the lanes of a wavefront.
__device__ __forceinline__ uint32_t wave_scan(uint32_t x)
{
    x += dpp_u32<0x111, 0xf>(0u, x);                          // row_shr:1, 2, 4, 8, then the rows' totals upwards
    x += dpp_u32<0x112, 0xf>(0u, x);
    x += dpp_u32<0x114, 0xf>(0u, x);
    x += dpp_u32<0x118, 0xf>(0u, x);
    x += dpp_u32<0x142, 0xa>(0u, x);
    x += dpp_u32<0x143, 0xc>(0u, x);
    return x;
}

struct Digit { uint32_t bin, rank, count; };              // the bin that holds a rank, the rank inside it, the bin's keys

constexpr uint32_t kBinsPerLane = kBins2 / 64;            // consecutive bins of a lane: 256 lanes cover the first digit, 64 one of the others
static_assert(kBins1 == 256 * kBinsPerLane && kBins3 == 64 * kBinsPerLane / 2, "shares of the lanes");

// The bin among the lane's N consecutive ones, the first of which starts at key number `at`, that holds `rank`.
template <uint32_t N>
__device__ __forceinline__ Digit bin_of(const uint32_t (&c)[N], uint32_t first_bin, uint32_t at, uint32_t rank)
{
    Digit d{first_bin, rank - at, c[0]};
    uint32_t below = 0;
#pragma unroll
    for (uint32_t i = 1; i < N; ++i) {
        below += c[i - 1];
        if (rank - at >= below) d = Digit{first_bin + i, rank - at - below, c[i]};
    }
    return d;
}

// N consecutive words; `hist` is LDS or, in another launch than the one that counted, global memory.
template <uint32_t N>
__device__ __forceinline__ void load_bins(uint32_t (&c)[N], const uint32_t* hist)
{
#pragma unroll
    for (uint32_t i = 0; i < N / 4; ++i) {
        const uint4 x = reinterpret_cast<const uint4*>(hist)[i];
        c[4 * i] = x.x; c[4 * i + 1] = x.y; c[4 * i + 2] = x.z; c[4 * i + 3] = x.w;
    }
}

// First digit of a block's four ranks from its histogram, which the threads leave cleared; the block's sums of v (`total`) and p
// (`psum`), known to thread 0; the flag of blocks that go without candidate lists.  Called by a whole workgroup.  Counts fit 32
// bits (numel < 2^32).
__device__ __forceinline__ void fold_first(const Selection& sel, const TileRow& m, uint32_t block, uint32_t* hist, double total, double psum,
                                           uint32_t lane, uint32_t wave, double* rec, uint32_t* __restrict__ scan3)
{
    __shared__ uint32_t sums[4];
    __shared__ Digit found[4];
    uint32_t c[kBinsPerLane], mine = 0;
    hist += threadIdx.x * kBinsPerLane;
    load_bins(c, hist);
#pragma unroll
    for (uint32_t i = 0; i < kBinsPerLane; ++i) mine += c[i];
    const uint32_t incl = wave_scan(mine);
    if (lane == 63) sums[wave] = incl;
    __syncthreads();
    uint32_t at = incl - mine;
    for (uint32_t w = 0; w < wave; ++w) at += sums[w];
#pragma unroll
    for (uint32_t t = 0; t < 4; ++t)
        if (m.rank[t] >= at && m.rank[t] - at < mine) found[t] = bin_of(c, threadIdx.x * kBinsPerLane, at, m.rank[t]);
    for (uint32_t i = 0; i < kBinsPerLane / 4; ++i) reinterpret_cast<uint4*>(hist)[i] = uint4{0u, 0u, 0u, 0u};
    __syncthreads();
    if (threadIdx.x < 4) { sel.prefix[block * kSelStride + threadIdx.x] = found[threadIdx.x].bin; sel.rank[block * kSelStride + threadIdx.x] = found[threadIdx.x].rank; }
    if (threadIdx.x == 0) {
        // mu is the mean of the row means to the last bit of what they are made of: the tiles' row sums, added in fp64
        if (m.rows) rec[R_MU] = total / ((double)m.rows * (double)m.cols);
        rec[R_PSUM] = psum;
        // Where the keys that carry a selected first digit would fill three quarters of the lists of a whole task, the block goes
        // without lists: its keys are counted as they come, and the last digit takes another walk over v, which is cheaper from
        // about there on.  k_final2 raises the flag where a single list overflows.  (39 blocks of 2,405 x 3,443, 20 % of them
        // zero: finalize 2.18 ms with lists that overflow and a second walk over their tiles, 1.55 with the keys past their end
        // counted at once, 1.32 now; 4,096 x 4,096 1.70, 1.20, 1.02.)
        uint64_t keys = 0;
        for (uint32_t t = 0; t < 4; ++t) {
            bool fresh = true;
            for (uint32_t u = 0; u < t; ++u) fresh = fresh && found[u].bin != found[t].bin;
            if (fresh) keys += found[t].count;
        }
        const uint64_t part = (uint64_t)min(m.rows, m.seg_len) * min(m.cols, m.strips * (64u << m.wc_log));   // coordinates of a whole task
        scan3[block * kArriveStride] = m.rows == 0 || keys * part > 3ull * m.cand_cap * m.numel;
    }
}

// The PASS-th digit (2 or 3) of a block's four ranks, a wavefront each; `hist` has a histogram for every distinct prefix and is left
// cleared.  `load` reads consecutive bins; the last digit completes the order statistics.  Called by a whole workgroup.
template <int PASS, typename L>
__device__ __forceinline__ void pick_digit(const Selection& sel, uint32_t block, uint32_t* hist, uint32_t lane, uint32_t wave, double* order, L load)
{
    constexpr uint32_t NB = PASS == 2 ? kBins2 : kBins3, N = NB / 64;
    const uint32_t id = block * kSelStride + wave;
    const Prefixes d = distinct_prefixes(sel.prefix, block);
    const uint32_t slot = wave == 0 ? d.slot_of[0] : (wave == 1 ? d.slot_of[1] : (wave == 2 ? d.slot_of[2] : d.slot_of[3]));
    const uint32_t rank = sel.rank[id], prefix = sel.prefix[id];
    uint32_t c[N], mine = 0;
    load(c, hist + slot * NB + lane * N);
#pragma unroll
    for (uint32_t i = 0; i < N; ++i) mine += c[i];
    const uint32_t at = wave_scan(mine) - mine;
    __syncthreads();                                          // all four have read the prefixes and the histogram
    if (rank >= at && rank - at < mine) {
        const Digit f = bin_of(c, lane * N, at, rank);
        const uint32_t key = (prefix << (PASS == 2 ? kBits2 : kBits3)) | f.bin;
        if (PASS == 2) { sel.prefix[id] = key; sel.rank[id] = f.rank; }
        else order[wave] = (double)__builtin_bit_cast(float, key);
    }
    for (uint32_t i = threadIdx.x; i < NB; i += 256) reinterpret_cast<uint4*>(hist)[i] = uint4{0u, 0u, 0u, 0u};
}

// Adds a workgroup's LDS histogram to the block's.
__device__ __forceinline__ void flush_hist(uint32_t* hist, const uint32_t* h, uint32_t n)
{
    for (uint32_t i = threadIdx.x; i < n; i += 256)
        if (h[i]) atomicAdd(&hist[i], h[i]);
}

// Sum over the workgroup in a fixed order; every thread calls it, thread 0 has the result.
__device__ __forceinline__ double group_sum(double x, uint32_t lane, uint32_t wave, double* sh)
{
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) x += __shfl_xor(x, d);
    __syncthreads();
    if (lane == 0) sh[wave] = x;
    __syncthreads();
    return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// ---------------------------------------------------------------------------
// Matrix blocks (v viewed as rows x cols), tiled.
// A workgroup takes 64 * wc columns and up to seg_len rows; its four wavefronts stand wc across the columns
// and 4 / wc down the rows.  A wavefront reads 4 rows x 64 columns (256 bytes a row) with one load, a lane 4
// consecutive columns of a row, at any alignment: a row sum then takes four exchange levels for four rows at
// once, and narrow or odd-sized matrices keep their lanes busy.  Loads are issued one round of kQuads * 4 rows
// ahead of their use; only rounds with a missing row load for themselves.  A wavefront that lacks columns keeps the others of its workgroup
// waiting at every row-sum exchange, and it did load for itself: 500 M coordinates of odd shapes 434 + 487 -> 411 + 461 us.
// The rows of a workgroup are not next to each other: of the n_segs workgroups of a tile column each takes every n_segs-th round.
// What is read at one time then lies close together, whatever the row length, where workgroups a power of two apart meet
// in the same memory channels (a plain read of 4,096 x 4,096 matrices in this pattern: runs of 256 or 1,024 rows 6.0 - 6.3 TB/s, every
// n_segs-th 16 rows 6.7 - 6.9; 4,096 x 11,008 6.8 - 7.0 either way.  Finalize passes of 3.5 G coordinates: 2323 -> 2270 and
// 3580 -> 3516 us, 124 M unchanged).
// In the second pass the keys that carry a selected first digit (a few per cent) gather in LDS, a thousand at a time
// are counted by their second digit and appended to a candidate list per wavefront; k_final3 counts the last digit on the lists.  Where
// a list has no room the last digit takes a walk over v.
// Large layouts are bound by HBM with the vector ALUs close behind, small ones by the number of wavefronts in flight.
// Measured (first / second pass, us; before: one wavefront per 256 x 256 tile, scalar loads where a row is not a
// multiple of 4, keys stored as they were found): 25.6 M coordinates of
// convolutions 189 / 416 -> 27 / 43, 124 M 136 / 323 -> 94 / 141, 60 M of odd shapes, a third of them vectors,
// 254 / 535 -> 60 / 119, 3.5 G 2492 / 3887 -> 2250 / 3505 (6.2 and 6.0 TB/s).
// ---------------------------------------------------------------------------

constexpr uint32_t kQuads = 4;                        // loads of 4 rows a wavefront has in flight
constexpr uint32_t kRoundRows = 4 * kQuads;
constexpr uint32_t kSubRounds = 256 / kRoundRows;     // rounds between two row-sum exchanges (256 rows per wavefront)

__device__ __forceinline__ uint32_t scalar_u32(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }
__device__ __forceinline__ uint32_t scalar_wave_index() { return scalar_u32(threadIdx.x >> 6); }

// Where a wavefront reads (task_of, tile_part, load_full, load_edge and what they call) is host code as well, for the tests: a
// read past the parameters shows there against a page without access and would not on the GPU.

// A wavefront's part of its workgroup's tile.  `wave` must be uniform over the wavefront (callers pass it through
// readfirstlane), so that the task and every address derived from it live in scalar registers.
struct TilePart {
    uint32_t tile, seg;
    uint32_t rows;                        // of the block
    uint32_t first, stride;               // first row of the wavefront's first round; rows from one round to the next
    uint32_t wcol, wrow, wr;              // place of the wavefront in the workgroup; wavefronts down the rows
    uint32_t col;                         // first of the lane's 4 columns
    uint32_t lrow;                        // the lane's row in a quad
    uint32_t n_ok;                        // how many of the lane's columns exist (0..4)
    uint32_t rounds, full;                // rounds of the workgroup; rounds of the wavefront without a missing row
    bool any, all;                        // some, all of the wavefront's columns exist
    uint32_t offset;                      // the lane's first element of a full round, from the round's first row
    uint32_t base;                        // the lane's first column (clamped to an existing one)
};

// The tiles of a workgroup: [tile, last) of the segment.
struct Task { uint32_t seg, tile, last; };
template <bool STRIPS>
__host__ __device__ __forceinline__ Task task_of(const TileRow& m, uint32_t wg)
{
    const uint32_t local = wg - m.first_task, seg = local / m.n_across, across = local - seg * m.n_across;
    if (!STRIPS) return Task{seg, across, across + 1};
    const uint32_t tile = across * m.strips;
    return Task{seg, tile, (uint32_t)min(m.n_tiles, tile + m.strips)};
}

// `left`: elements from the block's first one that may be read.
__host__ __device__ __forceinline__ TilePart tile_part(const TileRow& m, uint32_t seg, uint32_t tile, uint32_t lane, uint32_t wave, uint64_t left)
{
    TilePart t;
    t.seg = seg; t.tile = tile;
    t.wr = 4u >> m.wc_log;
    t.wcol = wave & ((1u << m.wc_log) - 1u); t.wrow = wave >> m.wc_log;
    t.rows = m.rows;
    const uint32_t mine = t.seg * t.wr + t.wrow, step = m.n_segs * t.wr;      // in rounds
    t.first = mine * kRoundRows; t.stride = step * kRoundRows;
    const uint32_t col0 = ((t.tile << m.wc_log) + t.wcol) * 64;
    t.col = col0 + 4 * (lane & 15u); t.lrow = lane >> 4;
    t.n_ok = t.col < m.cols ? min(4u, m.cols - t.col) : 0u;
    t.any = col0 < m.cols; t.all = col0 + 64 <= m.cols;
    const uint32_t log_wr = 2 - m.wc_log, stripes = (m.rows + (kRoundRows << log_wr) - 1) / (kRoundRows << log_wr);
    t.rounds = (stripes - t.seg + m.n_segs - 1) / m.n_segs;
    // Offsets of a full round are 32-bit byte offsets.  Where columns are missing its loads reach up to 3 elements past their row.
    uint32_t whole = m.rows / kRoundRows;
    if (!t.all && (uint64_t)whole * kRoundRows * m.cols + 3 > left) --whole;
    t.full = t.any && m.cols < (1u << 28) && whole > mine ? (whole - mine - 1) / step + 1 : 0;
    t.base = min(t.col, m.cols - 1);
    t.offset = t.lrow * m.cols + t.base;
    return t;
}

// First row (of the block) of a wavefront's round.
__host__ __device__ __forceinline__ uint32_t round_row(const TilePart& t, uint32_t i) { return t.first + i * t.stride; }

// Whether rows start on cache lines.  Where they do not, wavefronts side by side share a line at every row's joint, and a line that
// is loaded with the nontemporal hint is gone when the second one asks for it (303 M coordinates in rows of 1,500 and 4,031, bf16
// parameters: passes 262 + 480 us with the hint, 248 + 412 without; in rows of 1,536 and 4,096 223 + 340 with it, 249 + 387 without).
template <typename E> __host__ __device__ __forceinline__ bool whole_lines(const E* src, uint32_t cols)
{
    return ((reinterpret_cast<uintptr_t>(src) | (uintptr_t)cols * sizeof(E)) & 127u) == 0;
}

// Keeps the compiler from making one load of two that differ in the hint alone.
__host__ __device__ __forceinline__ void apart() { asm volatile(""); }

// Four elements per lane and quad of a full round (of lanes without a column, some).  The address is a scalar base and a 32-bit
// lane offset.
template <int TT>
__host__ __device__ __forceinline__ void load_full(typename GradIO<TT>::vec4 (&x)[kQuads], const typename GradIO<TT>::elem* __restrict__ src, bool lines,
                                          const TilePart& t, uint32_t cols, uint32_t i)
{
    typedef typename GradIO<TT>::elem E;
    const char* p = reinterpret_cast<const char*>(src) + (uint64_t)round_row(t, i) * cols * sizeof(E);
    const uint32_t lane = (uint32_t)(t.offset * sizeof(E));
    const uint64_t step = (uint64_t)cols * (4 * sizeof(E));
    if (lines) {
#pragma unroll
        for (uint32_t q = 0; q < kQuads; ++q) x[q] = GradIO<TT>::loadv_any(reinterpret_cast<const E*>(p + q * step + lane));
    } else {
        apart();
#pragma unroll
        for (uint32_t q = 0; q < kQuads; ++q) x[q] = GradIO<TT>::loadv_shared(reinterpret_cast<const E*>(p + q * step + lane));
        apart();
    }
}

// The same at the edge of a matrix.  Rows and columns past the matrix are replaced by its last ones; a lane then reads up to 3
// elements past its row.  `left`: elements from src that may be read.
template <int TT>
__host__ __device__ __forceinline__ void load_edge(typename GradIO<TT>::vec4 (&x)[kQuads], const typename GradIO<TT>::elem* __restrict__ src,
                                          uint64_t left, const TilePart& t, uint32_t cols, uint32_t i)
{
    typedef GradIO<TT> IO;
    const uint32_t first = round_row(t, i);
    const bool wide = (uint64_t)min(first + kRoundRows, t.rows) * cols + 3 <= left;     // the same for the whole wavefront
#pragma unroll
    for (uint32_t q = 0; q < kQuads; ++q) {
        const typename IO::elem* p = src + ((uint64_t)min(first + 4 * q + t.lrow, t.rows - 1) * cols + t.base);
        if (wide) {
            x[q] = IO::loadv_shared(p);
        } else {
            typename IO::elem e[4];
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k) e[k] = k < t.n_ok ? p[k] : typename IO::elem(0);
            x[q] = __builtin_bit_cast(typename IO::vec4, e);
        }
    }
}

constexpr uint64_t kAnywhere = ~0ull;                 // v may be read past its end: g_prev follows it in the workspace

// First pass over a tile.  Returns the lane's sum of p and adds the thread's part of the sum of v to `total`; counts
// into h, which the `first` tile of the workgroup clears.
__device__ __forceinline__ double tile_pass1(const float* __restrict__ v_all, const TileRow& m, const TilePart& t, bool first, uint32_t lane, uint32_t wave,
                                             float* __restrict__ rowpart, float* __restrict__ colpart, float* __restrict__ rvec, float* __restrict__ cvec,
                                             uint32_t* h, float* rowsum, double* colsum,
                                             float eps, float eps_low, bool want_p, double& total)
{
    const float* src = v_all + m.state_start;
    const uint32_t cols = scalar_u32(m.cols);
    const bool lines = whole_lines(src, cols);
    f4 nx[kQuads];
#pragma unroll
    for (uint32_t q = 0; q < kQuads; ++q) nx[q] = f4{0.f, 0.f, 0.f, 0.f};
    if (t.full) load_full<BAOC_GRAD_F32>(nx, src, lines, t, cols, 0);
    if (first)
        for (uint32_t i = threadIdx.x; i < kBins1; i += 256) h[i] = 0;
    // Column sums and the sum of p run over many rows per lane: kept in fp64 so that a constant
    // v (rank one, p constant) comes out as such to ~1e-7 instead of the ~1e-5 of a long fp32 chain.
    double cs[4] = {0.0, 0.0, 0.0, 0.0}, psum = 0.0;
    __syncthreads();
    for (uint32_t i = 0; i < t.rounds; ++i) {
        if (t.any) {
            float x[kQuads][4];
            const bool full = i < t.full;
            if (!full) load_edge<BAOC_GRAD_F32>(nx, src, kAnywhere, t, cols, i);
#pragma unroll
            for (uint32_t q = 0; q < kQuads; ++q) { x[q][0] = nx[q].x; x[q][1] = nx[q].y; x[q][2] = nx[q].z; x[q][3] = nx[q].w; }
            if (i + 1 < t.full) load_full<BAOC_GRAD_F32>(nx, src, lines, t, cols, i + 1);
            if (full && t.all) {
#pragma unroll
                for (uint32_t q = 0; q < kQuads; ++q)
#pragma unroll
                    for (int k = 0; k < 4; ++k) atomicAdd(&h[(__builtin_bit_cast(uint32_t, x[q][k]) >> kShift1) & (kBins1 - 1)], 1u);
                if (want_p) {
                    float low = x[0][0];
#pragma unroll
                    for (uint32_t q = 0; q < kQuads; ++q) low = fminf(fminf(fminf(low, x[q][0]), fminf(x[q][1], x[q][2])), x[q][3]);
                    auto add_p = [&](auto p_of) {
#pragma unroll
                        for (uint32_t q = 0; q < kQuads; ++q)
                            psum += (double)((p_of(x[q][0]) + p_of(x[q][1])) + (p_of(x[q][2]) + p_of(x[q][3])));
                    };
                    if (__builtin_amdgcn_ballot_w64(!(low > eps_low)) == 0) add_p([&](float v) { return preconditioner_series(v, eps); });
                    else add_p([&](float v) { return preconditioner(v, eps); });
                }
            } else {
                const uint32_t row = round_row(t, i);
#pragma unroll
                for (uint32_t q = 0; q < kQuads; ++q) {
                    const bool in_row = row + 4 * q + t.lrow < t.rows;
                    float prow = 0.f;
#pragma unroll
                    for (uint32_t k = 0; k < 4; ++k) {
                        if (in_row && k < t.n_ok) {
                            atomicAdd(&h[(__builtin_bit_cast(uint32_t, x[q][k]) >> kShift1) & (kBins1 - 1)], 1u);
                            if (want_p) prow += preconditioner(x[q][k], eps);
                        } else {
                            x[q][k] = 0.f;
                        }
                    }
                    psum += (double)prow;
                }
            }
            float s[kQuads];
#pragma unroll
            for (uint32_t q = 0; q < kQuads; ++q) {
#pragma unroll
                for (int k = 0; k < 4; ++k) cs[k] += (double)x[q][k];
                s[q] = (x[q][0] + x[q][1]) + (x[q][2] + x[q][3]);
            }
            // Row sums: a halving exchange over the 16 lanes of a row leaves quad 2 b3 + b2 with the lanes whose
            // index has these bits.
            static_assert(kQuads == 4, "the exchange is written for four quads");
            {
                const bool b3 = lane & 8u, b2 = lane & 4u;
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const float keep = b3 ? s[q + 2] : s[q], send = b3 ? s[q] : s[q + 2];
                    s[q] = keep + dpp<0x128, 0xf>(0.f, send);
                }
                const float keep = b2 ? s[1] : s[0], send = b2 ? s[0] : s[1];
                float a = keep + dpp<0x141, 0xf>(0.f, send);
                a += dpp<0x4E, 0xf>(0.f, a);
                a += dpp<0xB1, 0xf>(0.f, a);
                if ((lane & 3u) == 0) rowsum[wave * 256 + (i % kSubRounds) * kRoundRows + (b3 ? 8u : 0u) + (b2 ? 4u : 0u) + t.lrow] = a;
            }
        }
        if ((i + 1) % kSubRounds == 0 || i + 1 == t.rounds) {
            // row sums of the last rounds: rowpart is tile-major ([tile][row]); a round of the workgroup is a run of 16, 32 or 64 rows
            __syncthreads();
            const uint32_t i0 = i / kSubRounds * kSubRounds, n = (i + 1 - i0) * t.wr * kRoundRows;
            const uint32_t first_row = t.seg * t.wr * kRoundRows + i0 * t.stride;
            const uint32_t n_wc = min(1u << m.wc_log, (m.cols - ((t.tile << m.wc_log) * 64) + 63) / 64);   // wavefronts that have columns
            for (uint32_t rs = threadIdx.x; rs < n; rs += 256) {
                const uint32_t step = rs / kRoundRows, wrow = step & (t.wr - 1), ii = step >> (2 - m.wc_log);
                const uint32_t row = first_row + ii * t.stride + rs % (t.wr * kRoundRows);
                if (row >= t.rows) break;
                const float* in = rowsum + (wrow << m.wc_log) * 256 + ii * kRoundRows + rs % kRoundRows;
                float sum = in[0];
                for (uint32_t w = 1; w < n_wc; ++w) sum += in[w * 256];
                if (m.n_tiles == 1) rvec[m.off_r + row] = (float)((double)sum / (double)m.cols);
                else rowpart[m.off_rowpart + (uint64_t)t.tile * m.rows + row] = sum;
                total += (double)sum;
            }
            __syncthreads();
        }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        cs[k] += __shfl_xor(cs[k], 16);
        cs[k] += __shfl_xor(cs[k], 32);
        if (lane < 16) colsum[wave * 64 + 4 * lane + k] = cs[k];
    }
    __syncthreads();
    const uint32_t tile_cols = 64u << m.wc_log, col = t.tile * tile_cols + threadIdx.x;
    if (threadIdx.x < tile_cols && col < m.cols) {
        double a = 0.0;
        for (uint32_t w = 0; w < t.wr; ++w) a += colsum[w * tile_cols + threadIdx.x];
        if (m.n_segs == 1) cvec[m.off_c + col] = (float)((double)(float)a / (double)m.rows);
        else colpart[m.off_colpart + (uint64_t)t.seg * m.cols + col] = (float)a;
    }
    return psum;
}

// A run of a block without a matrix shape: 16 coordinates per thread and round.  Calls f(v, theta, how many of
// the 4 exist); the loads of a round are issued together.  Runs start on a multiple of 4 coordinates, so a quad of v is
// aligned and inside the padded state; theta is read at any alignment and not past the block's last coordinate.  (Loads a round ahead of
// their use, with theta's hint by alignment: bf16 theta on runs that start on lines 777 -> 832 us, finalize of 28 vectors of 300 M
// coordinates in all, 3 of 1.2 G 2777 -> 3041; 60 M of odd shapes, a third vectors, 214 -> 216.)
template <int TT, bool THETA, typename Fn>
__device__ __forceinline__ void walk_run(const float* __restrict__ v_all, const typename GradIO<TT>::elem* __restrict__ theta, const TileRow& m, uint32_t len, Fn f)
{
    typedef GradIO<TT> IO;
    const uint64_t e0 = (uint64_t)(blockIdx.x - m.first_task) * len;
    const uint32_t n = e0 < m.numel ? (uint32_t)min((uint64_t)len, m.numel - e0) : 0u;
    const float* src = v_all + m.state_start + e0;
    const typename IO::elem* tsrc = theta + (m.grad_start + e0);
    for (uint32_t at = threadIdx.x * 4; at < n; at += 4096) {
        f4 x[4];
        typename IO::vec4 th[4];
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) { x[q] = f4{0.f, 0.f, 0.f, 0.f}; th[q] = typename IO::vec4{}; }
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q)
            if (at + q * 1024 < n) x[q] = ld_stream<f4>(src + at + q * 1024);
        if (THETA) {
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q) {
                const uint32_t e = at + q * 1024;
                if (e + 4 <= n) th[q] = IO::loadv_any(tsrc + e);
                else if (e < n) {
                    typename IO::elem part[4];
#pragma unroll
                    for (uint32_t k = 0; k < 4; ++k) part[k] = e + k < n ? tsrc[e + k] : typename IO::elem(0);
                    th[q] = __builtin_bit_cast(typename IO::vec4, part);
                }
            }
        }
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) {
            const uint32_t e = at + q * 1024;
            if (e >= n) break;
            const float xv[4] = {x[q].x, x[q].y, x[q].z, x[q].w};
            float tv[4];
            IO::unpack(th[q], tv);
            f(xv, tv, min(4u, n - e));
        }
    }
}

// STRIPS: the layout has blocks whose tasks take several tiles.  Layouts without such blocks have kernels without the loop over tiles
// (with it finalize of 1.5 G coordinates takes 3.72 instead of 3.70 ms).
template <bool STRIPS>
__global__ __launch_bounds__(256, STRIPS ? 4 : 5) void k_final1(
    const float* __restrict__ v_all, const TileRow* __restrict__ tiles, const uint32_t* __restrict__ task_block,
    float* __restrict__ rowpart, float* __restrict__ colpart, float* __restrict__ rvec, float* __restrict__ cvec, double2* __restrict__ taskpart,
    Selection sel, uint32_t* __restrict__ scan3, double* __restrict__ rec_all, float eps, float eps_low, bool want_p, const OnceRow* __restrict__ once)
{
    __shared__ alignas(16) uint32_t h[kBins1];
    __shared__ float rowsum[4 * 256];                     // [wavefront][its rows of a sub-segment]
    __shared__ double colsum[4 * 64], sums[8];
    const uint32_t lane = threadIdx.x & 63u, wave = scalar_wave_index(), block = task_block[blockIdx.x];
    if (settled(once, scan3, block)) return;
    const TileRow& m = tiles[block];
    double psum = 0.0, total = 0.0;
    if (m.rows) {
        const Task k = task_of<STRIPS>(m, blockIdx.x);
        for (uint32_t tile = k.tile; tile < k.last; ++tile)
            psum += tile_pass1(v_all, m, tile_part(m, k.seg, tile, lane, wave, kAnywhere), tile == k.tile, lane, wave, rowpart, colpart, rvec, cvec, h, rowsum, colsum,
                               eps, eps_low, want_p, total);
    } else {
        for (uint32_t i = threadIdx.x; i < kBins1; i += 256) h[i] = 0;
        __syncthreads();
        walk_run<BAOC_GRAD_F32, false>(v_all, nullptr, m, m.seg_len, [&](const float x[4], const float*, uint32_t n) {
            float prow = 0.f;
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k)
                if (k < n) {
                    atomicAdd(&h[(__builtin_bit_cast(uint32_t, x[k]) >> kShift1) & (kBins1 - 1)], 1u);
                    if (want_p) prow += preconditioner(x[k], eps);
                }
            psum += (double)prow;
        });
    }
    total = group_sum(total, lane, wave, sums);
    psum = group_sum(psum, lane, wave, sums + 4);             // ends with every wavefront's counts in h
    if (m.n_tasks == 1) {
        fold_first(sel, m, block, h, total, psum, lane, wave, rec_all + (uint64_t)block * kRecDoubles, scan3);
        return;
    }
    if (threadIdx.x == 0) taskpart[blockIdx.x] = double2{total, psum};
    flush_hist(sel.hist + (uint64_t)block * kHistWords, h, kBins1);
}

// Between the first two passes, for blocks of several tasks: the first n_multi workgroups fold what a block's tasks left (digit of the
// ranks, sums), the others r_i and c_j (fp32 for the second pass) from the partial sums of the first, 64 rows or 64 columns each, summed
// over the tiles or segments by 4 wavefronts in parallel: a 50257 x 768 block has hundreds of segments, whose loads would
// otherwise wait for each other (62 -> 6 us on that layout).
__global__ __launch_bounds__(256) void k_fold1(const TileRow* __restrict__ tiles, const uint32_t* __restrict__ multi, uint32_t n_multi,
                                               const uint32_t* __restrict__ fin_block, const float* __restrict__ rowpart, const float* __restrict__ colpart,
                                               float* __restrict__ rvec, float* __restrict__ cvec, const double2* __restrict__ taskpart,
                                               Selection sel, uint32_t* __restrict__ scan3, double* __restrict__ rec_all, const OnceRow* __restrict__ once)
{
    __shared__ double sh[4][64];
    const uint32_t lane = threadIdx.x & 63u, wave = scalar_wave_index();
    if (blockIdx.x < n_multi) {
        const uint32_t block = multi[blockIdx.x];
        if (settled(once, scan3, block)) return;
        const TileRow& m = tiles[block];
        double total = 0.0, psum = 0.0;
        for (uint32_t i = threadIdx.x; i < m.n_tasks; i += 256) {
            const double2 x = taskpart[m.first_task + i];
            total += x.x; psum += x.y;
        }
        total = group_sum(total, lane, wave, sh[0]);
        psum = group_sum(psum, lane, wave, sh[1]);
        fold_first(sel, m, block, sel.hist + (uint64_t)block * kHistWords, total, psum, lane, wave, rec_all + (uint64_t)block * kRecDoubles, scan3);
        return;
    }
    const uint32_t unit = blockIdx.x - n_multi;
    if (settled(once, scan3, fin_block[unit])) return;
    const TileRow& m = tiles[fin_block[unit]];
    const uint32_t local = unit - m.first_fin, row_wgs = m.n_tiles > 1 ? (m.rows + 63) / 64 : 0;
    const bool is_row = local < row_wgs;
    const uint32_t at = (is_row ? local : local - row_wgs) * 64 + lane, len = is_row ? m.rows : m.cols;
    const uint32_t count = is_row ? m.n_tiles : m.n_segs;
    const float* src = (is_row ? rowpart + m.off_rowpart : colpart + m.off_colpart) + at;
    double s = 0.0;
    if (at < len) {
#pragma unroll 8
        for (uint32_t k = wave; k < count; k += 4) s += (double)src[(uint64_t)k * len];
    }
    sh[wave][lane] = s;
    __syncthreads();
    if (wave != 0 || at >= len) return;
    s = (sh[0][lane] + sh[1][lane]) + (sh[2][lane] + sh[3][lane]);
    if (is_row) rvec[m.off_r + at] = (float)(s / (double)m.cols);
    else cvec[m.off_c + at] = (float)(s / (double)m.rows);
}

// Words per wavefront in which matching keys gather: with the histogram 37 KB of LDS, four workgroups per CU.  Where theta is read the
// registers allow no more (104 to 128).  Without theta (61 to 81 registers) five would fit with 960 words and six with 480, which
// pays where v has many equal values and costs elsewhere (finalize without theta, us with 1,280, 960 and 480 words: 39 matrices of 2,405 x
// 3,443 with 20 % zeros 874, 859, 854, without 569, 572, 576; 124 M 251, 250, 250; 500 M of odd shapes 1015, 1019, 1026; 1.3 G 1811,
// 1830, 1844).
constexpr uint32_t kStage = 1280;

// The same value, unknown to the compiler: what is cheap to form from it again keeps no register over a loop.
__device__ __forceinline__ uint32_t again(uint32_t x) { asm("" : "+v"(x)); return x; }

// F, C: Eq. 7 and Eq. 6 are wanted.
template <int TT, bool F, bool C, bool STRIPS>
__global__ __launch_bounds__(256, 4) void k_final2(
    const float* __restrict__ v_all, const typename GradIO<TT>::elem* __restrict__ theta, uint64_t theta_numel,
    const TileRow* __restrict__ tiles, const uint32_t* __restrict__ task_block, const float* __restrict__ rvec, const float* __restrict__ cvec,
    float4* __restrict__ residpart, Selection sel, uint32_t* cand, uint32_t* __restrict__ cand_count,
    uint32_t* __restrict__ scan3, double* __restrict__ rec_all, float eps, float eps_low, const OnceRow* __restrict__ once)
{
    typedef GradIO<TT> IO;
    typedef typename IO::vec4 TV;
    __shared__ alignas(16) uint32_t h[4 * kBins2];        // a histogram per distinct prefix
    __shared__ uint32_t staged[4 * kStage];
    __shared__ float red[4][4];
    const uint32_t lane = threadIdx.x & 63u, wave = scalar_wave_index(), block = task_block[blockIdx.x];
    if (settled(once, scan3, block)) return;
    const TileRow& m = tiles[block];
    const Prefixes d = distinct_prefixes(sel.prefix, block);
    const double* rec_in = rec_all + (uint64_t)block * kRecDoubles;
    float inv_pbar = 0.f;
    if (C) inv_pbar = (float)((double)m.numel / rec_in[R_PSUM]);
    auto count2 = [&](uint32_t bits) { count_match(h, d, kBins2, (bits >> kShift1) & (kBins1 - 1), (bits >> kShift2) & (kBins2 - 1)); };
    // A lane adds at most 256 terms in fp32 before they go to fp64 (16 at the edges, where narrow matrices stay all the way): the sums
    // of a constant theta drift with the length of the chain (300,000 x 4 in a large layout: C off by 3e-5 with a chain over the
    // tile, by 6e-8 now).
    float res = 0.f, cn = 0.f, cd = 0.f;
    double rsum = 0.0, nsum = 0.0, dsum = 0.0;
    auto settle = [&]() {
        if (F) { rsum += (double)res; res = 0.f; }
        if (C) { nsum += (double)cn; dsum += (double)cd; cn = 0.f; cd = 0.f; }
    };
    for (uint32_t i = threadIdx.x; i < 4 * kBins2; i += 256) h[i] = 0;
    __syncthreads();
    if (m.rows) {
        const Task k = task_of<STRIPS>(m, blockIdx.x);
        const float* src = v_all + m.state_start;
        const typename IO::elem* tsrc = theta + m.grad_start;
        const uint64_t tleft = C ? theta_numel - m.grad_start : kAnywhere;
        TilePart t = tile_part(m, k.seg, k.tile, lane, wave, tleft);
        const float* rr = rvec + m.off_r;
        // no room where the first pass has found the block to go without lists (or a list of this pass overflowed meanwhile, which comes
        // to the same: the last digit is then not taken from the lists)
        const uint32_t cols = scalar_u32(m.cols), cap = scalar_u32(scan3[block * kArriveStride] ? 0u : m.cand_cap);
        const bool lines = whole_lines(src, cols), tlines = C && whole_lines(tsrc, cols);
        f4 nx[kQuads]; TV nt[kQuads]; float nr[kQuads];
#pragma unroll
        for (uint32_t q = 0; q < kQuads; ++q) { nx[q] = f4{0.f, 0.f, 0.f, 0.f}; nt[q] = TV{}; nr[q] = 0.f; }
        auto issue = [&](uint32_t i) {
            load_full<BAOC_GRAD_F32>(nx, src, lines, t, cols, i);
            if (C) load_full<TT>(nt, tsrc, tlines, t, cols, i);
            if (F) {
                // a scalar base and a 32-bit lane offset that is not kept: as a 64-bit address per lane it makes the registers
                // spill with fp32 theta (finalize of 1.3 G coordinates 2651 -> 2640 us)
                const char* p = reinterpret_cast<const char*>(rr + round_row(t, i));
                const uint32_t at = again(lane) >> 4 << 2;
#pragma unroll
                for (uint32_t q = 0; q < kQuads; ++q) nr[q] = *reinterpret_cast<const float*>(p + 16 * q + at);
            }
        };
        // tiles side by side have one round each, which the loop over the edges takes
        const bool one = !STRIPS || m.strips == 1;
        const uint32_t full = one ? t.full : 0, rounds = one ? t.rounds : k.last - k.tile;
        if (full) issue(0);
        const double mu = F ? rec_in[R_MU] : 0.0;
        // c_j / mu is formed in fp64 (mu may lie below the fp32 normal range); S~ = 0 when mu = 0
        float cm[4];
        auto load_means = [&]() {
#pragma unroll
            for (uint32_t e = 0; e < 4; ++e)
                cm[e] = (F && e < t.n_ok && mu != 0.0) ? (float)((double)cvec[m.off_c + t.col + e] / mu) : 0.f;
        };
        load_means();
        uint32_t* list = cand + m.cand_base + ((uint64_t)(blockIdx.x - m.first_task) * 4 + wave) * cap;
        uint32_t n_cand = 0;                                      // uniform over the wavefront; may grow past the list
        // Matching keys gather in LDS and leave many at a time: stores of a few keys each would be waited for together with
        // the next round's loads.
        uint32_t* stage = staged + wave * kStage;
        uint32_t n_stage = 0;
        auto append = [&](bool hit, uint64_t hits, uint32_t bits) {
            const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(hits >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)hits, 0u));
            if (hit) stage[n_stage + at] = bits;
            n_stage += (uint32_t)__builtin_popcountll(hits);
        };
        // Whole sets of 64 are counted and go to the list as far as it has room; what is left moves to the front.  The list is written
        // through to memory: left in the L2 the lines go out one by one later, between the reads (3.5 G coordinates, 0.25 GB of keys:
        // the pass takes 3470 us with plain stores, 3405 with nontemporal ones, 3355 so, 3210 with no stores at all).
        auto flush = [&](bool all) {
            const uint32_t n = all ? n_stage : n_stage & ~63u;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");    // lanes read what other lanes staged
            for (uint32_t i = lane; i < n; i += 256) {
                uint32_t key[4];
#pragma unroll
                for (uint32_t q = 0; q < 4; ++q) key[q] = stage[min(i + 64 * q, kStage - 1)];
#pragma unroll
                for (uint32_t q = 0; q < 4; ++q)
                    if (i + 64 * q < n) {
                        if (n_cand + i + 64 * q < cap) st_device(&list[n_cand + i + 64 * q], key[q]);
                        count2(key[q]);
                    }
            }
            n_cand += n; n_stage -= n;
            const uint32_t rest = lane < n_stage ? stage[n + lane] : 0u;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (lane < n_stage) stage[lane] = rest;
        };
        static_assert(kStage >= 63 + 64 * 4, "a quad of keys and what the last flush left");
        const uint32_t p0 = d.pre[0], p1 = d.pre[1];
        // a round that lacks rows or columns
        auto masked = [&](const f4 (&vx)[kQuads], const TV (&vt)[kQuads], const float (&vr)[kQuads], uint32_t first) {
#pragma unroll
            for (uint32_t q = 0; q < kQuads; ++q) {
                const bool in_row = first + 4 * q + t.lrow < t.rows;
                const float x[4] = {vx[q].x, vx[q].y, vx[q].z, vx[q].w};
                float th[4] = {0.f, 0.f, 0.f, 0.f};
                if (C) IO::unpack(vt[q], th);
#pragma unroll
                for (uint32_t k = 0; k < 4; ++k) {
                    const bool in = in_row && k < t.n_ok;
                    const uint32_t bits = __builtin_bit_cast(uint32_t, x[k]), hi = (bits >> kShift1) & (kBins1 - 1);
                    const bool hit = in && (hi == p0 || hi == p1 || hi == d.pre[2] || hi == d.pre[3]);
                    append(hit, __builtin_amdgcn_ballot_w64(hit), bits);
                    if (F) {
                        const float dd = in ? __builtin_fmaf(-vr[q], cm[k], x[k]) : 0.f;
                        res = __builtin_fmaf(dd, dd, res);
                    }
                    if (C) {
                        const float tk = in ? th[k] : 0.f;
                        const float y = in ? __builtin_fmaf(preconditioner(x[k], eps), inv_pbar, -1.0f) * tk : 0.f;
                        cn = __builtin_fmaf(y, y, cn);
                        cd = __builtin_fmaf(tk, tk, cd);
                    }
                }
                if (n_stage >= kStage - 256) flush(false);
            }
            settle();
        };
        for (uint32_t i = 0, n = t.all ? full : 0; i < n; ++i) {
            float x[kQuads][4], th[kQuads][4], ri[kQuads];
#pragma unroll
            for (uint32_t q = 0; q < kQuads; ++q) {
                x[q][0] = nx[q].x; x[q][1] = nx[q].y; x[q][2] = nx[q].z; x[q][3] = nx[q].w;
                IO::unpack(nt[q], th[q]);
                ri[q] = nr[q];
            }
            if (i + 1 < full) issue(i + 1);
            if (d.n <= 2) {
#pragma unroll
                for (uint32_t q = 0; q < kQuads; ++q) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const uint32_t bits = __builtin_bit_cast(uint32_t, x[q][k]), hi = (bits >> kShift1) & (kBins1 - 1);
                        append(hi == p0 || hi == p1, __builtin_amdgcn_ballot_w64(hi == p0) | __builtin_amdgcn_ballot_w64(hi == p1), bits);
                    }
                    if (n_stage >= kStage - 256) flush(false);
                }
            } else {
#pragma unroll
                for (uint32_t q = 0; q < kQuads; ++q) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const uint32_t bits = __builtin_bit_cast(uint32_t, x[q][k]), hi = (bits >> kShift1) & (kBins1 - 1);
                        const bool hit = hi == p0 || hi == p1 || hi == d.pre[2] || hi == d.pre[3];
                        append(hit, __builtin_amdgcn_ballot_w64(hit), bits);
                    }
                    if (n_stage >= kStage - 256) flush(false);
                }
            }
            if (F) {
#pragma unroll
                for (uint32_t q = 0; q < kQuads; ++q)
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const float dd = __builtin_fmaf(-ri[q], cm[k], x[q][k]);
                        res = __builtin_fmaf(dd, dd, res);
                    }
            }
            if (C) {
                float low = x[0][0];
#pragma unroll
                for (uint32_t q = 0; q < kQuads; ++q) low = fminf(fminf(fminf(low, x[q][0]), fminf(x[q][1], x[q][2])), x[q][3]);
                auto distort = [&](auto p_of) {
#pragma unroll
                    for (uint32_t q = 0; q < kQuads; ++q)
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            const float y = __builtin_fmaf(p_of(x[q][k]), inv_pbar, -1.0f) * th[q][k];
                            cn = __builtin_fmaf(y, y, cn);
                            cd = __builtin_fmaf(th[q][k], th[q][k], cd);
                        }
                };
                if (__builtin_amdgcn_ballot_w64(!(low > eps_low)) == 0) distort([&](float v) { return preconditioner_series(v, eps); });
                else distort([&](float v) { return preconditioner(v, eps); });
            }
            if ((i + 1) % kSubRounds == 0) settle();
        }
        if (!t.all) {
            for (uint32_t i = 0; i < full; ++i) {
                f4 ex[kQuads]; TV et[kQuads]; float er[kQuads];
#pragma unroll
                for (uint32_t q = 0; q < kQuads; ++q) { ex[q] = nx[q]; et[q] = nt[q]; er[q] = nr[q]; }
                if (i + 1 < full) issue(i + 1);
                masked(ex, et, er, round_row(t, i));
            }
        }
        for (uint32_t i = full; i < rounds; ++i) {
            if (!one && i > 0) { t = tile_part(m, k.seg, k.tile + i, lane, wave, tleft); load_means(); }
            if (!t.any) break;
            const uint32_t round = one ? i : 0, first = round_row(t, round);
            f4 ex[kQuads]; TV et[kQuads]; float er[kQuads];
            load_edge<BAOC_GRAD_F32>(ex, src, kAnywhere, t, cols, round);
#pragma unroll
            for (uint32_t q = 0; q < kQuads; ++q) { et[q] = TV{}; er[q] = F ? rr[min(first + 4 * q + t.lrow, t.rows - 1)] : 0.f; }
            if (C) load_edge<TT>(et, tsrc, tleft, t, cols, round);
            masked(ex, et, er, first);
        }
        settle();
        flush(true);
        if (lane == 0) {
            cand_count[blockIdx.x * 4 + wave] = n_cand;
            // list too short: the last digit of the block takes another walk over v
            if (n_cand > cap) scan3[block * kArriveStride] = 1u;
        }
    } else {
        walk_run<TT, C>(v_all, theta, m, m.seg_len, [&](const float x[4], const float th[4], uint32_t n) {
            float yn = 0.f, yd = 0.f;
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k)
                if (k < n) {
                    count2(__builtin_bit_cast(uint32_t, x[k]));
                    if (C) {
                        const float y = __builtin_fmaf(preconditioner(x[k], eps), inv_pbar, -1.0f) * th[k];
                        yn = __builtin_fmaf(y, y, yn);
                        yd = __builtin_fmaf(th[k], th[k], yd);
                    }
                }
            nsum += (double)yn; dsum += (double)yd;
        });
    }
    res = wave_sum((float)rsum); cn = wave_sum((float)nsum); cd = wave_sum((float)dsum);
    if (lane == 0) { red[wave][0] = res; red[wave][1] = cn; red[wave][2] = cd; }
    __syncthreads();
    auto task_sum = [&](uint32_t q) { return (float)(((double)red[0][q] + (double)red[1][q]) + ((double)red[2][q] + (double)red[3][q])); };
    double* rec = rec_all + (uint64_t)block * kRecDoubles;
    if (m.n_tasks == 1) {
        if (threadIdx.x == 0) { rec[R_FRES] = (double)task_sum(0); rec[R_CNUM] = (double)task_sum(1); rec[R_CDEN] = (double)task_sum(2); }
        pick_digit<2>(sel, block, h, lane, wave, nullptr, [](auto& c, const uint32_t* at) { load_bins(c, at); });
        return;
    }
    if (threadIdx.x == 0) residpart[blockIdx.x] = float4{task_sum(0), task_sum(1), task_sum(2), 0.f};
    flush_hist(sel.hist + (uint64_t)block * kHistWords, h, d.n * kBins2);
}

// Between the last two passes, for blocks of several tasks: second digit of the ranks, sums of Eq. 7 and Eq. 6.
__global__ __launch_bounds__(256) void k_fold2(const TileRow* __restrict__ tiles, const uint32_t* __restrict__ multi, const float4* __restrict__ residpart,
                                               Selection sel, const uint32_t* __restrict__ scan3, double* __restrict__ rec_all, const OnceRow* __restrict__ once)
{
    __shared__ double sh[3][4];
    const uint32_t lane = threadIdx.x & 63u, wave = scalar_wave_index(), block = multi[blockIdx.x];
    if (settled(once, scan3, block)) return;
    const TileRow& m = tiles[block];
    double* rec = rec_all + (uint64_t)block * kRecDoubles;
    double res = 0.0, cn = 0.0, cd = 0.0;
    for (uint32_t i = threadIdx.x; i < m.n_tasks; i += 256) {
        const float4 x = residpart[m.first_task + i];
        res += (double)x.x; cn += (double)x.y; cd += (double)x.z;
    }
    res = group_sum(res, lane, wave, sh[0]);
    cn = group_sum(cn, lane, wave, sh[1]);
    cd = group_sum(cd, lane, wave, sh[2]);
    if (threadIdx.x == 0) { rec[R_FRES] = res; rec[R_CNUM] = cn; rec[R_CDEN] = cd; }
    pick_digit<2>(sel, block, sel.hist + (uint64_t)block * kHistWords, lane, wave, nullptr, [](auto& c, const uint32_t* at) { load_bins(c, at); });
}

// Last digit: on the candidate lists that the second pass wrote, or on v where a block has none or one of them
// overflowed.  Leaves the records in `out_all`, host memory or the records themselves.
__global__ __launch_bounds__(256) void k_final3(
    const float* __restrict__ v_all, const TileRow* __restrict__ tiles, const uint32_t* __restrict__ task_block, const uint32_t* __restrict__ cand,
    const uint32_t* __restrict__ cand_count, Selection sel, uint32_t* __restrict__ arrived, const uint32_t* __restrict__ scan3, const double* __restrict__ rec_all, double* __restrict__ out_all,
    const OnceRow* __restrict__ once)
{
    __shared__ alignas(16) uint32_t h[4 * kBins3];
    const uint32_t lane = threadIdx.x & 63u, wave = scalar_wave_index(), block = task_block[blockIdx.x];
    if (settled(once, scan3, block)) return;
    const TileRow& m = tiles[block];
    for (uint32_t i = threadIdx.x; i < 4 * kBins3; i += 256) h[i] = 0;
    const Prefixes d = distinct_prefixes(sel.prefix, block);
    auto count3 = [&](uint32_t bits) { count_match(h, d, kBins3, (bits & 0x7fffffffu) >> kShift2, bits & (kBins3 - 1)); };
    __syncthreads();
    if (m.rows && !scan3[block * kArriveStride]) {
        const uint32_t n = min(cand_count[blockIdx.x * 4 + wave], m.cand_cap);
        const uint32_t* list = cand + m.cand_base + ((uint64_t)(blockIdx.x - m.first_task) * 4 + wave) * m.cand_cap;
        for (uint32_t at = lane; at < n; at += 512) {          // eight loads in flight
            uint32_t key[8];
#pragma unroll
            for (uint32_t q = 0; q < 8; ++q) key[q] = list[min(at + 64 * q, n - 1)];
#pragma unroll
            for (uint32_t q = 0; q < 8; ++q)
                if (at + 64 * q < n) count3(key[q]);
        }
    } else {
        // a matrix is no more than its coordinates here, shared evenly over its tasks
        const uint32_t len = m.rows ? (uint32_t)((m.numel + m.n_tasks - 1) / m.n_tasks + 3) & ~3u : m.seg_len;
        walk_run<BAOC_GRAD_F32, false>(v_all, nullptr, m, len, [&](const float x[4], const float*, uint32_t n) {
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k)
                if (k < n) count3(__builtin_bit_cast(uint32_t, x[k]));
        });
    }
    __syncthreads();
    // the block's record as it leaves the device; the order statistics are new
    auto finish = [&](uint32_t* hist, auto load) {
        const double* rec = rec_all + (uint64_t)block * kRecDoubles;
        double* out = out_all + (uint64_t)block * kRecDoubles;
        if (out != rec && threadIdx.x < kRecDoubles && threadIdx.x - R_ORDER >= 4) out[threadIdx.x] = rec[threadIdx.x];
        pick_digit<3>(sel, block, hist, lane, wave, out + R_ORDER, load);
    };
    uint32_t* hist = sel.hist + (uint64_t)block * kHistWords;
    if (m.n_tasks == 1) {
        finish(h, [](auto& c, const uint32_t* at) { load_bins(c, at); });
        return;
    }
    flush_hist(hist, h, d.n * kBins3);
    if (!arrive_last(arrived + block * kArriveStride, m.n_tasks)) return;
    finish(hist, [](auto& c, const uint32_t* at) {
#pragma unroll
        for (uint32_t i = 0; i < kBins3 / 64; ++i) c[i] = ld_device(at + i);
    });
}

}  // namespace baoc

#include "baoc_once.h"

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

using namespace baoc;

// Workspace of baoc_profile_begin_static: one array per GPU, resident from the moment the code object is
// loaded until the process ends.  In host code the name below is only a handle for hipGetSymbolAddress;
// the device address is looked up once per device and kept in g_scratch_ptr.
static __device__ __align__(256) unsigned char scratch[BAOC_STATIC_WORKSPACE_BYTES];

constexpr int kMaxDevices = 64;
static void* g_scratch_ptr[kMaxDevices] = {};      // device address of `scratch` on each GPU
static bool g_scratch_busy[kMaxDevices] = {};      // a handle begun with baoc_profile_begin_static is alive

struct Plan {
    uint64_t n_chunks = 0;
    uint32_t gpw = 1, nw = 4, slices = 1, slice_groups = 4, resident = 8;   // launch shape of the step kernel
    uint64_t n_prows = 0;         // partial rows of the step kernel = n_chunks * slices
    bool fold_in_step = false;    // the step kernel folds its own partial rows
    Memory memory = kThrough;
    std::vector<BlockRow> rows;
    std::vector<TileRow> tiles;   // how finalize walks each block
    bool any_matrix = false, any_strips = false;
    uint64_t n_tasks = 0, n_fin = 0;   // workgroups of the finalize passes; those of k_fold1 that fold row and column sums
    std::vector<Part> parts;      // of blocks of more than kDirectRows partial rows
    std::vector<uint32_t> multi;  // blocks of several tasks
    std::vector<OnceRow> once;    // every block's share of the one pass
    uint32_t once_tasks = 0, once_narrow = 0;   // its workgroups, and those of 8 wavefronts among them; 0: the layout goes through the passes
    uint32_t once_units = 0, once_multi = 0;    // workgroups of k_once_select; blocks of several tasks
    bool once_all = false;        // every block takes it
    bool once_worth[2] = {};      // it is faster than the passes without theta, with theta
    bool once_lines = true;       // rows are whole cache lines
    uint64_t off_once_sums = 0, off_once_units = 0;
    uint64_t padded = 0;          // coordinates in m / v / g_prev
    uint64_t off_m = 0, off_v = 0, off_gp = 0, off_partials = 0, off_step_rows = 0, off_chunks = 0;   // the step's rows stand at off_step_rows
    uint64_t off_rows = 0, off_tiles = 0, off_parts = 0, off_multi = 0, off_once = 0, off_task_block = 0, off_fin_block = 0;   // the first five are uploaded in one piece
    uint64_t off_rec = 0, off_hist = 0, off_arrived = 0, off_cleared = 0;                         // cleared up to off_cleared
    uint64_t off_rvec = 0, off_cvec = 0, off_residpart = 0, off_candcount = 0,
             off_cand = 0, off_rowpart = 0, off_colpart = 0, total = 0;
};

struct baoc_profiler {
    baoc_profile_params params;
    Plan plan;
    std::vector<baoc_block> blocks;
    char* ws = nullptr;
    int static_device = -1;       // >= 0: the workspace is that device's `scratch` array
    uint32_t steps = 0;
    uint64_t max_end = 0;         // largest offset + numel over the blocks
    int sticky = BAOC_OK;
    double* host_rec = nullptr;   // where finalize leaves the records: memory of the pool below, or h_rec
    uint64_t host_bytes = 0;      // its size in the pool
    bool host_lost = false;       // waiting for a finalize failed: a kernel may still write to host_rec
    std::vector<double> h_rec;
};

// Pinned host memory that the last kernel of finalize writes the records to.  A copy to pageable memory is staged by the runtime
// after the kernels have ended (finalize of 25.6 M coordinates, 41 KB: 135 us with the copy, 125 so; of 32,768 49.6 and 40.5).
// Pinning takes longer than that, so buffers are kept for the next handle: at most kPoolBytes in all are ever pinned, in powers
// of two up to kPoolBuffer; a handle that finds none, and a static one, which allocates nothing, has the copy.
constexpr uint64_t kPoolBytes = 4ull << 20, kPoolBuffer = 1ull << 20, kPoolSmallest = 4096;
// Objects without destructors: a handle may be ended while the program's own are running.
struct Pinned { double* p; uint64_t bytes; };
static std::mutex g_pool_mutex;
static_assert(std::is_trivially_destructible<std::mutex>::value, "lives until the process ends");
static Pinned g_pool_free[kPoolBytes / kPoolSmallest];
static uint32_t g_pool_n = 0;                 // buffers in g_pool_free
static uint64_t g_pool_pinned = 0;

static double* pool_take(uint64_t bytes, uint64_t* got)
{
    uint64_t size = kPoolSmallest;
    while (size < bytes) size *= 2;
    if (size > kPoolBuffer) return nullptr;
    std::lock_guard<std::mutex> lock(g_pool_mutex);
    for (uint32_t i = 0; i < g_pool_n; ++i)
        if (g_pool_free[i].bytes >= size) {
            const Pinned found = g_pool_free[i];
            g_pool_free[i] = g_pool_free[--g_pool_n];
            *got = found.bytes;
            return found.p;
        }
    if (g_pool_pinned + size > kPoolBytes) return nullptr;
    void* p = nullptr;
    if (hipHostMalloc(&p, size, hipHostMallocPortable | hipHostMallocMapped) != hipSuccess || !p) { (void)hipGetLastError(); return nullptr; }
    g_pool_pinned += size;
    *got = size;
    return static_cast<double*>(p);
}

static void pool_give(double* p, uint64_t bytes)
{
    std::lock_guard<std::mutex> lock(g_pool_mutex);
    g_pool_free[g_pool_n++] = Pinned{p, bytes};
}

static uint64_t align_up(uint64_t x, uint64_t a) { return (x + a - 1) / a * a; }

// Layouts whose step kernel folds its own partial rows: up to this many rows in all and in one block.  It saves a launch
// (32,768 coordinates: 9.3 -> 6.5 us a step, 1 M in 64 blocks 9.3 -> 8.0) and costs every workgroup the wait for its
// stores and an arrival, about 25 ns each where they share a counter: 256 rows of one block take 11.4 us instead of 9.4,
// 2,000 rows of 100 blocks 14.2 instead of 13.4, 2,048 rows of 16 blocks 15.5 instead of 13.5.
constexpr uint64_t kFoldRows = 1024, kFoldBlockRows = 64;

// Coordinates of a tile (one workgroup of the tile passes): the layout's by kTileTarget, between the smallest and the cap.  Partial tiles
// come on top, and beyond 537 M coordinates the cap leaves more.  The chip holds 1,024 workgroups of k_final2 and 1,280 of k_final1
// at a time.  In powers of two a layout just past one had little more than 1,024 of them, and a second round of a few (303 M coordinates,
// rows of 1,500 and 4,031: passes 282 + 540 us, now 262 + 478).  A smaller tile pays for its histograms more often (kernels of a finalize
// of 124 M coordinates with 3,000 tiles 273 us, with 4,000 285, now 262; 25.6 M 93, 107 and 90; layouts of odd shapes gain up to 5 %), and
// so does a cap below 262,144 on large layouts (3.5 G coordinates: 5.92 ms with 131,072, 5.68 now).
constexpr uint64_t kTileCoordsMin = 8192, kTileCoordsMax = 262144, kTileTarget = 2048;
// Rows of a tile: those of a 64-column tile of the largest size.  A matrix of fewer columns still occupies 64 columns of lanes, so
// without this line its workgroups walk up to 131,072 rows one round after another (40 matrices of 50,000 x 4 and 32 of 4,096 x
// 4,096: finalize 4.13 -> 1.26 ms, one of 300,000 x 4 next to 566 M coordinates 5.30 -> 1.59 ms; with 2,048 rows 1.37 and 1.61 ms,
// with 1,024 1.41 and 1.62 ms).
constexpr uint64_t kTileRowsMax = kTileCoordsMax / 64;
// Coordinates of a run of a block without a matrix shape, in layouts whose tiles are larger.  Blocks of very different sizes leave the last
// workgroups few and long, most of all where many coordinates share a key and the histogram's bins are what everything waits for
// (finalize of 3,000 vectors, 300 M coordinates, 70 % of them zero: 2.64 ms with one chunk at a time, 3.66 with runs of
// 262,144, 3.03 with 131,072, 2.62 with 65,536, 2.47 with 32,768; dense 1.20, 0.99, 0.91, 0.92 and 0.95).  All runs of a block meet in
// one histogram and one counter, so a large block has longer ones (3 blocks of 579 M coordinates in all 1.68 ms with 262,144 and up
// to 512 runs a block, 1.75 with up to 2,048; 28 of 430 M 1.16, 1.21 and 1.26).
constexpr uint64_t kRunCoords = 32768, kBlockRuns = 512;

static int check_params(const baoc_profile_params* p)
{
    if (!p) return BAOC_ERR_INVALID;
    if (!(p->beta_m > 0.f && p->beta_m < 1.f) || !(p->beta_v > 0.f && p->beta_v < 1.f)) return BAOC_ERR_INVALID;
    if (!(p->beta_rho >= 0.0 && p->beta_rho < 1.0)) return BAOC_ERR_INVALID;
    if (!(p->eps >= 0.0) || !(p->eps_update > 0.f)) return BAOC_ERR_INVALID;   // u = m / (sqrt(v) + eps_update) must exist where v = 0
    if (p->grad_dtype != BAOC_GRAD_F32 && p->grad_dtype != BAOC_GRAD_BF16) return BAOC_ERR_INVALID;
    if (p->quant_block != kQB) return BAOC_ERR_UNSUPPORTED;
    if (p->chunk_groups > 4096 || p->groups_per_wave > 2 || p->chunk_slices > 64) return BAOC_ERR_INVALID;
    if (p->waves_per_workgroup != 0 && p->waves_per_workgroup != 1 && p->waves_per_workgroup != 2 && p->waves_per_workgroup != 4)
        return BAOC_ERR_INVALID;
    if (p->resident_workgroups != 0 && (p->resident_workgroups < 3 || p->resident_workgroups > 32)) return BAOC_ERR_INVALID;
    return BAOC_OK;
}

// Groups per chunk where a block's groups are spread evenly over as few chunks of up to `most` groups as hold them.
static uint64_t even_groups(uint64_t groups, uint32_t most)
{
    const uint64_t chunks = (groups + most - 1) / most;
    return (groups + chunks - 1) / chunks;
}

// The blocks' shares of the one pass, in the memory that the passes have for r, c and the candidate lists.  A block takes part where a
// workgroup's wavefronts hold a whole row of it: up to 6,144 columns with 8 wavefronts, 12,288 with 16; and up to 2^28 coordinates, where a bin
// still has fewer keys than can be ordered.  A layout takes part where these blocks have kOnceSmallest coordinates and no others are there, or
// kOnceSmallestPart next to others, which go through the passes: a sample, a workgroup's start and end (25 us) and the selection cost
// more than a second read where there is little to read.  Whole finalize, us, passes and one pass: 25.6 M 127 and 172, 124 M (148 blocks) 305 and 330,
// 134 M (8 blocks) 292 and 254, 178 M 410 and 375, 252 M (15 blocks) 496 and 379, (240 blocks) 530 and 444, 503 M 904 and 658, 1.3 G 2670 and
// 2110, 3.5 G 5700 and 4450.  Next to others: 26 M of 150 M 325 and 398, 229 M of 252 M 715 and 766, 319 M of 430 M 1061 and 1081, 371 M of 436 M 1196
// and 1125, 430 M of 851 M 1498 and 1206.
// Layouts of many small blocks keep the passes as well: 2,100 of 65,536 coordinates 472 and 602, 1,000 of 160,000 536 and 658, 300 of 490,000 414
// and 358, 240 of 1 M 530 and 440.
// And those whose matrices leave lanes or wavefronts of the one pass idle (see OnceCost).
constexpr uint64_t kOnceSmallest = 1ull << 27, kOnceSmallestPart = 3ull << 27, kOnceMeanBlock = 3ull << 17;

// Fewer tasks than this, those of 16 wavefronts counted twice, leave too much of the chip idle for the one pass (tasks grow until lists and column sums have
// room): 150 of 1.3 M coordinates 486 us by the passes and 2,741 by the one pass, 447 of 0.36 M 416 and 770, 640 of 0.3 M 491 and 608; from 820 on as
// OnceCost has it.
constexpr uint64_t kOnceTasks = 768;

// Whole finalize, us, of the blocks that take part, with theta [1] and without [0]: what each adds by either way, and what comes with it once.
// `full` is the share of a task's lanes and rows that have work: where it is small, arithmetic costs more than the second read.  Rows that are no
// whole cache lines cost the passes more, and so do vectors, whose v they read a third time.  Fitted to 230 layouts of 134 M to 3.5 G coordinates; the
// residuals' deviation is 5 to 6 %, and the line leaves 2 % to the passes with theta.  Of 420 M, bf16 theta, us, passes and one pass: 100 of 4,096
// columns 790 and 611, 3,328 (full = 0.81) 767 and 679, 4,864 (0.79) 759 and 717, 4,352 (0.71) 774 and 776; with 16 wavefronts 8,192 798 and 652,
// 10,240 (0.83) 786 and 735, 6,400 (0.78) 747 and 776, 9,216 (0.75) 758 and 857; 400 of 1,024 x 1,024 804 and 682, 712 of 768 x 768 852 and 759, 316 of
// 1,152 x 1,152 (0.75) 825 and 855, 1,025 of 640 x 640 (0.83) 885 and 977, 606 of 832 x 832 (0.81) 843 and 1088.
struct OnceCost {
    double passes[2] = {63.0, 67.0}, once[2] = {112.0, 85.0};
    void add(const TileRow& m, bool wide, double full)
    {
        const double n = 1e-6 * (double)m.numel;
        const bool broken = m.rows && m.cols % 64, vector = m.rows == 0;
        passes[0] += 0.23 + n * (1.32 + (broken ? 0.25 : vector ? 0.54 : 0.0));
        passes[1] += 0.14 + n * (1.67 + (broken ? 0.48 : vector ? 0.48 : 0.0));
        once[0] += 0.42 + n * (0.04 + (0.75 + (wide ? 0.15 : 0.0) + (broken ? 0.05 : 0.0)) / full);
        once[1] += 0.29 + n * (0.41 + (0.81 + (wide ? 0.12 : 0.0) + (broken ? 0.10 : 0.0)) / full);
    }
    // Next to blocks that go through the passes more is left to these, whose workgroups are launched for all blocks (a UNet of 860 M coordinates in
    // 686 blocks, 7 of which do not take part, 1,853 and 2,023 us; this says 1.06).
    bool worth(bool with_theta, bool others) const { return (others ? 1.08 : with_theta ? 1.02 : 1.0) * once[with_theta] < passes[with_theta]; }
};
constexpr uint64_t kOnceBlock = 1ull << 28;
constexpr uint64_t kOnceSingle = 65536;                   // coordinates that one workgroup reads again for its quantiles, from the L2
constexpr uint32_t kOnceColumns = 768;                    // per wavefront
static void plan_once(Plan& P, uint64_t total)
{
    const uint32_t n = (uint32_t)P.tiles.size();
    P.once.assign(n, OnceRow{});
    P.once_tasks = 0;
    if (total < kOnceSmallest) return;
    const uint64_t room = (P.total - P.off_rvec) / 64;                         // 64-byte units
    auto units64 = [](uint64_t bytes) { return (bytes + 63) / 64; };
    for (uint64_t share = std::min<uint64_t>(1u << 19, std::max<uint64_t>(1u << 14, total / 1024)); share <= 4 << 20; share *= 2) {
        double listed = 0.0;
        uint64_t narrow = 0, wide = 0, columns = 0, at = 0, multi = 0, part = 0, taking = 0, broken = 0, aligned = 0;
        OnceCost cost;
        for (uint32_t i = 0; i < n; ++i) {
            const TileRow& m = P.tiles[i];
            OnceRow& o = P.once[i];
            o = OnceRow{};
            o.first_task = (uint32_t)narrow; o.first_wide = (uint32_t)wide;
            if (m.numel > kOnceBlock || m.numel < 4 || (m.rows && (m.cols < 4 || m.cols > 16 * kOnceColumns))) continue;
            ++part; taking += m.numel;
            const uint32_t waves = m.rows && m.cols > 8 * kOnceColumns ? 16 : 8;
            uint64_t most = (m.numel + waves * 1024 - 1) / (waves * 1024);      // batches or rounds
            double full = 1.0;
            if (m.rows) {
                ((m.state_start | m.cols | m.grad_start) & 63u ? broken : aligned) += m.numel;
                // lanes of a row in a load, strips of a wavefront, wavefronts side by side: as few lanes without columns, wavefronts
                // without rows and batches without work as possible
                double best = 0.0;
                for (uint32_t lanes_log = m.rows >= 4 ? 4 : m.rows >= 2 ? 5 : 6; lanes_log <= 6; ++lanes_log)
                    for (uint32_t strips = 1; strips <= 3; ++strips) {
                        const uint32_t width = 4u << lanes_log, across = (uint32_t)((m.cols + (uint64_t)width * strips - 1) / (width * strips));
                        if (across > waves) continue;
                        const uint32_t down = waves / across, loads = strips == 1 ? 4 : strips == 2 ? 2 : 1, batch = down * (loads << (6 - lanes_log));
                        const double busy = (double)m.cols / ((double)across * strips * width) * (across * down) / waves * m.rows / (double)align_up(m.rows, batch);
                        const double use = busy * (across == 1 ? 1.1 : 1.0) * (strips == 1 ? 1.02 : 1.0) * (lanes_log == 6 ? 1.03 : 1.0);
                        if (use <= best) continue;
                        best = use; full = busy;
                        o.geom = lanes_log | strips << 4 | across << 8 | down << 16 | (waves == 16 ? 1u << 24 : 0u);
                        most = (m.rows + batch - 1) / batch;
                    }
            }
            cost.add(m, waves == 16, full);
            o.n_tasks = m.numel <= kOnceSingle && waves == 8 ? 1 : (uint32_t)std::max<uint64_t>(2, std::min(most, (m.numel + share / 2) / share));
            (waves == 16 ? wide : narrow) += o.n_tasks;
            if (o.n_tasks == 1) continue;
            ++multi;
            columns += once_col_units(m.rows, m.cols);
            listed += listed_share(m.numel) * (double)m.numel;
            o.off_cols = (uint32_t)at;
            at += once_cols_units(o.n_tasks, m.rows ? m.cols : 0) + units64(once_keys_cap(m.numel) * 8);
        }
        // The lists have room for 1.2 to 2.4 times what independent coordinates bring: neighbours that are alike bring up to twice as much.  A third of
        // it is common to a block's tasks.
        const uint64_t tasks = narrow + wide, units_at = at + units64(tasks * sizeof(OnceSums)), most_units = columns + tasks + (uint64_t)(listed / 2048.0) + multi;
        const uint64_t lists_at = units_at + units64(most_units * sizeof(OnceUnit));
        if (taking < (part == n ? kOnceSmallest : kOnceSmallestPart) || taking < n * kOnceMeanBlock || narrow + 2 * wide < kOnceTasks || tasks > 0x7fffffffull || most_units > 0x7fffffffull) return;
        for (int i = 0; i < 2; ++i) P.once_worth[i] = cost.worth(i, part != n);
        if (!P.once_worth[0] && !P.once_worth[1]) return;
        if (lists_at + tasks > room || (double)(room - lists_at - tasks) * 16.0 < kListSlack * listed) continue;
        const double words = multi ? std::min(2.0 * kListSlack, (double)(room - lists_at - tasks) * 16.0 / listed) : 0.0;
        P.off_once_sums = P.off_rvec + at * 64; P.off_once_units = P.off_rvec + units_at * 64;
        at = lists_at;
        for (uint32_t i = 0; i < n; ++i) {
            OnceRow& o = P.once[i];
            if (o.n_tasks < 2) continue;
            const TileRow& m = P.tiles[i];
            o.off_list = (uint32_t)at;
            o.list_cap = (uint32_t)(words * listed_share(m.numel) * (double)m.numel * (2.0 / 3.0) / o.n_tasks) / 16 * 16;
            at += ((uint64_t)o.n_tasks * o.list_cap + once_spill(o)) / 16;
        }
        uint64_t units = 0;
        for (uint32_t i = 0; i < n; ++i) {
            OnceRow& o = P.once[i];
            o.first_unit = (uint32_t)units;
            if (o.n_tasks > 1) units += once_list_units(o) + once_col_units(P.tiles[i].rows, P.tiles[i].cols);
        }
        if (at > room || units > most_units) return;
        P.once_narrow = (uint32_t)narrow; P.once_units = (uint32_t)units; P.once_multi = (uint32_t)multi; P.once_all = part == n;
        P.once_tasks = (uint32_t)tasks; P.once_lines = broken <= aligned;
        return;
    }
}

static int make_plan(const baoc_block* blocks, uint32_t n, const baoc_profile_params* prm, Plan* out, uint64_t* max_end)
{
    if (!blocks || n == 0) return BAOC_ERR_INVALID;
    int rc = check_params(prm);
    if (rc) return rc;
    // no overlap: sort a copy by offset
    std::vector<std::pair<uint64_t, uint64_t>> iv(n);
    uint64_t end_max = 0;
    for (uint32_t i = 0; i < n; ++i) {
        const baoc_block& b = blocks[i];
        if (b.numel == 0) return BAOC_ERR_INVALID;
        if (b.numel > 0xffffffffull) return BAOC_ERR_UNSUPPORTED;      // 32-bit histogram counters
        if (b.offset + b.numel < b.offset) return BAOC_ERR_INVALID;
        if ((b.rows || b.cols) && (uint64_t)b.rows * b.cols != b.numel) return BAOC_ERR_INVALID;
        iv[i] = {b.offset, b.numel};
        end_max = std::max(end_max, b.offset + b.numel);
    }
    std::sort(iv.begin(), iv.end());
    for (uint32_t i = 1; i < n; ++i)
        if (iv[i - 1].first + iv[i - 1].second > iv[i].first) return BAOC_ERR_INVALID;
    if (max_end) *max_end = end_max;

    Plan& P = *out;
    uint64_t total = 0;
    for (uint32_t i = 0; i < n; ++i) total += blocks[i].numel;
    // a caller's own groups or wavefronts do not stand next to the medium shape's: its other half would mean more workgroups
    const bool f32 = prm->grad_dtype == BAOC_GRAD_F32, medium = total >= kHintedLayout && !prm->groups_per_wave && !prm->waves_per_workgroup;
    const LaunchShape& ds = total >= kMediumLayout ? kDefaultShape[prm->grad_dtype]
                            : f32 && medium        ? kMediumF32Shape
                            : f32 && total >= kSmallLayout ? kHintedF32Shape : kSmallShape[prm->grad_dtype];
    P.gpw = prm->groups_per_wave ? prm->groups_per_wave : ds.groups_per_wave;
    P.nw = prm->waves_per_workgroup ? prm->waves_per_workgroup : ds.waves_per_workgroup;
    P.resident = prm->resident_workgroups ? prm->resident_workgroups : ds.resident_workgroups;
    const uint32_t round = P.gpw * P.nw;                            // groups a workgroup takes per round
    const uint32_t cg = prm->chunk_groups ? prm->chunk_groups : std::max(ds.chunk_groups, round);
    P.slices = prm->chunk_slices ? std::min(prm->chunk_slices, cg) : std::max(1u, cg / round);   // default: one round per slice
    P.slice_groups = (cg + P.slices - 1) / P.slices;
    // Cuts the blocks into chunks of up to `groups` groups, `slices` workgroups each.
    auto cut = [&](uint32_t groups_max, uint32_t slices) {
        P.n_chunks = 0; P.rows.resize(n); P.parts.clear();
        uint64_t state = 0;
        for (uint32_t i = 0; i < n; ++i) {
            const baoc_block& b = blocks[i];
            const uint64_t groups = (b.numel + kQB - 1) / kQB, per = even_groups(groups, groups_max);
            BlockRow& r = P.rows[i];
            r.grad_start = b.offset; r.state_start = state; r.numel = b.numel;
            r.first_chunk = (uint32_t)P.n_chunks;
            r.n_chunks = (uint32_t)((groups + per - 1) / per);
            r.groups_per_chunk = (uint32_t)per; r.pad_ = 0;
            const uint64_t prows = (uint64_t)r.n_chunks * slices, first_prow = P.n_chunks * slices;
            if (first_prow + prows > 0x7fffffffull) return false;
            r.first_prow = (uint32_t)first_prow; r.n_prows = (uint32_t)prows;
            for (uint32_t q = 0; prows > kDirectRows && q < prows / kPartRows; ++q) P.parts.push_back(Part{i, q});
            P.n_chunks += r.n_chunks;
            state += groups * kQB;
            if (P.n_chunks > 0x7fffffffull) return false;
        }
        P.padded = state;
        P.n_prows = P.n_chunks * slices;
        P.slices = slices;
        return true;
    };
    if (!cut(cg, P.slices)) return BAOC_ERR_UNSUPPORTED;
    P.memory = P.padded * (f32 ? 12 : 10) <= kKeptBytes ? kKept : f32 && total >= kSmallLayout && total < kHintedLayout ? kHinted : kThrough;
    P.multi.clear();
    uint32_t most_prows = 0;
    for (const BlockRow& r : P.rows) most_prows = std::max(most_prows, r.n_prows);
    P.fold_in_step = P.n_prows <= kFoldRows && most_prows <= kFoldBlockRows;
    // Finalize walks blocks with a real matrix shape tile-wise and the rest in runs.  A shape with a
    // single row or column is rank one by construction (F = 0 exactly) and counts as a run.
    P.tiles.resize(n); P.any_matrix = P.any_strips = false; P.n_tasks = 0; P.n_fin = 0;
    uint64_t n_r = 0, n_c = 0, n_rowpart = 0, n_colpart = 0, n_cand = 0;
    const uint64_t tile_coords = std::min(kTileCoordsMax, std::max(kTileCoordsMin, align_up(total / kTileTarget, 1024)));
    uint64_t run_max = kTileCoordsMin;                               // the longest run: a power of two
    while (run_max < tile_coords) run_max *= 2;
    uint64_t matrix_tasks = 0, run_budget = 0;
    for (uint32_t i = 0; i < n; ++i) {
        const baoc_block& b = blocks[i];
        TileRow& m = P.tiles[i];
        m = TileRow{};
        if (b.rows < 2 || b.cols < 2) { run_budget += 15360 + 4ull * P.rows[i].n_chunks; continue; }
        m.rows = b.rows; m.cols = b.cols;
        // columns of a tile: 256, 128 or 64, the widest that leaves at most an eighth of the lanes without a column, or the
        // narrowest that has rows for wavefronts below each other
        m.wc_log = 2;
        while (m.wc_log > 0 && b.rows > (4u >> m.wc_log) * kRoundRows && align_up(b.cols, 64u << m.wc_log) * 8 > (uint64_t)b.cols * 9) --m.wc_log;
        const uint64_t round_rows = (4u >> m.wc_log) * kRoundRows, tile_cols = 64u << m.wc_log;
        m.seg_len = (uint32_t)align_up(std::min<uint64_t>(kTileRowsMax, tile_coords / std::min<uint64_t>(b.cols, tile_cols)), round_rows);
        m.n_tiles = (uint32_t)((b.cols + tile_cols - 1) / tile_cols); m.n_segs = (uint32_t)(((uint64_t)b.rows + m.seg_len - 1) / m.seg_len);
        // even shares of the rows (39 blocks of 2,405 x 3,443 without theta: 750 -> 676 us, with 70 % zeros 3.03 -> 2.72 ms)
        m.seg_len = (uint32_t)align_up(((uint64_t)b.rows + m.n_segs - 1) / m.n_segs, round_rows);
        // A matrix of so few rows that its tiles, 256 columns wide, have a single round: a task takes as many of them side by side as
        // make up the smallest tile (16 of 2 x 262,144: finalize 432 -> 241 us, 400 of 8 x 4,096 264 -> 188 us, 4,000 of 2 x 300 852 -> 438
        // us).  With more rows a tile is worth its workgroup (a model of 64 channels, 1.5 M coordinates: 92 us, with two tiles
        // of 64 x 64 to a task 98 us).
        m.strips = b.rows > kRoundRows ? 1 : (uint32_t)std::min<uint64_t>(m.n_tiles, std::max<uint64_t>(1, kTileCoordsMin / (b.rows * tile_cols)));
        m.n_across = (m.n_tiles + m.strips - 1) / m.strips;
        P.any_strips |= m.strips > 1;
        matrix_tasks += (uint64_t)m.n_across * m.n_segs;
    }
    // The tasks' sums (16 bytes each) and the lengths of their candidate lists (16 bytes, only where there are matrices) go where
    // the step's partial rows are, as far as these have room.
    auto task_bytes = [](uint64_t tasks) { return align_up(tasks * 16, 256); };
    const uint64_t partial_bytes = P.n_prows * kNumSums * 4;
    auto sums_fit = [&](uint64_t tasks) { return task_bytes(tasks) <= partial_bytes; };
    auto counts_fit = [&](uint64_t tasks) { return 2 * task_bytes(tasks) <= partial_bytes; };
    // Coordinates of a run: kRunCoords, or as many as leave a block kBlockRuns of them; and at least `least`.  A run takes 4 bytes in
    // task_block and up to 32 for what does not fit the partial rows (with large chunks these are few).  Runs are lengthened
    // until that is within run_budget, 15 KB per block and 4 bytes per chunk, which keeps the workspace of a layout from growing
    // with the number of runs whatever the launch shape.
    uint64_t least = kTileCoordsMin;
    auto run_coords = [&](uint64_t numel) {
        uint64_t r = std::min(run_max, kRunCoords);
        while (r < run_max && r * kBlockRuns < numel) r *= 2;
        return std::max(r, least);
    };
    for (; least < (1u << 30); least = align_up(least * 5 / 4, 1024)) {
        uint64_t runs = 0;
        for (uint32_t i = 0; i < n; ++i)
            if (P.tiles[i].rows == 0) { const uint64_t r = run_coords(blocks[i].numel); runs += (blocks[i].numel + r - 1) / r; }
        const uint64_t tasks = matrix_tasks + runs;
        if (runs * (4 + (sums_fit(tasks) ? 0 : 16) + (matrix_tasks == 0 || counts_fit(tasks) ? 0 : 16)) <= run_budget) break;
    }
    for (uint32_t i = 0; i < n; ++i) {
        const baoc_block& b = blocks[i];
        TileRow& m = P.tiles[i];
        m.state_start = P.rows[i].state_start; m.grad_start = b.offset; m.numel = b.numel;
        m.first_task = (uint32_t)P.n_tasks; m.first_fin = (uint32_t)P.n_fin;
        for (int q = 0; q < 2; ++q) {                                // ranks bracketing position q (d-1)
            const uint64_t lo = (uint64_t)std::floor((q == 0 ? 0.1 : 0.9) * (double)(b.numel - 1));
            m.rank[2 * q] = (uint32_t)lo;
            m.rank[2 * q + 1] = (uint32_t)std::min<uint64_t>(lo + 1, b.numel - 1);
        }
        uint64_t tasks;
        if (m.rows == 0) {
            m.seg_len = (uint32_t)run_coords(b.numel); m.n_tiles = m.strips = m.n_across = 1;
            tasks = (b.numel + m.seg_len - 1) / m.seg_len;
            m.n_segs = (uint32_t)tasks;
        } else {
            P.any_matrix = true;
            m.off_r = n_r; m.off_c = n_c; m.off_rowpart = n_rowpart; m.off_colpart = n_colpart;
            n_r += b.rows; n_c += b.cols;
            if (m.n_tiles > 1) { n_rowpart += (uint64_t)b.rows * m.n_tiles; P.n_fin += ((uint64_t)b.rows + 63) / 64; }
            if (m.n_segs > 1) { n_colpart += (uint64_t)m.n_segs * b.cols; P.n_fin += ((uint64_t)b.cols + 63) / 64; }
            tasks = (uint64_t)m.n_across * m.n_segs;
            // One candidate list per wavefront; a block's lists have room for an eighth of its coordinates, less the 48 bytes that a task
            // takes elsewhere.  The keys that share a selected first digit are a few per cent of a block unless many coordinates have
            // the same v.
            m.cand_cap = (uint32_t)((std::max<uint64_t>(b.numel / (32 * tasks), 3) - 3) / 4 * 4);
            m.cand_base = n_cand;
            n_cand += tasks * 4 * m.cand_cap;
        }
        m.n_tasks = (uint32_t)tasks;
        if (tasks > 1) P.multi.push_back(i);
        P.n_tasks += tasks;
        if (P.n_tasks > 0x7fffffffull || P.n_fin > 0x7fffffffull) return BAOC_ERR_UNSUPPORTED;
    }
    // the row and column partial sums of the first pass are folded before the second writes the candidate lists in their place
    const uint64_t list_bytes = std::max(align_up(n_cand * 4, 256), align_up(n_rowpart * 4, 256) + align_up(n_colpart * 4, 256));
    // Large fp32 layouts: single-wavefront workgroups of one group, 16 resident.  They write twice the partial rows, which stand where
    // finalize has its lists if these leave room (the matrix blocks' lists take half a byte a coordinate, the rows a quarter), so that
    // the workspace stays as it is.  Every workgroup reads its chunk's table entry, so chunks have eight groups: with four the step
    // moves 1.022 of its algorithmic bytes, with eight 1.016.  Blocks of a few groups leave workgroups of such a chunk without
    // one; where that would be more than a sixteenth of all, chunks have four groups.
    // (In one process, us a step: two groups and 10 resident against this: 74 M coordinates of odd shapes 340 and 333, 100 M 457 and
    // 436, 124 M 544 and 540, 860 M 3720 and 3646, 1.3 G 5632 and 5579.)
    const bool own_shape = prm->chunk_groups || prm->chunk_slices || prm->groups_per_wave || prm->waves_per_workgroup || prm->resident_workgroups;
    uint32_t fine = 0;                                               // groups, and workgroups, of a chunk
    for (uint32_t g = 8; g >= 4 && !fine && !own_shape && &ds == &kDefaultShape[BAOC_GRAD_F32]; g -= 4) {
        uint64_t rows = 0, groups = 0;
        for (const BlockRow& r : P.rows) {
            const uint64_t all = (r.numel + kQB - 1) / kQB, per = even_groups(all, g);
            groups += all; rows += (all + per - 1) / per * g;
        }
        // a launch has fewer than 2^32 threads (reached at 17.2 G coordinates)
        if (rows * 64 <= 0xffffffffull && rows * kNumSums * 4 <= list_bytes && (g == 4 || rows <= groups + groups / 16)) fine = g;
    }
    if (fine) { cut(fine, fine); P.gpw = P.nw = P.slice_groups = 1; P.resident = 16; }
    const uint64_t gsz = prm->grad_dtype == BAOC_GRAD_F32 ? 4 : 2;
    uint64_t o = 0;
    auto place = [&](uint64_t& off, uint64_t bytes) { off = o; o = align_up(o + bytes, 256); };
    place(P.off_m, P.padded * 4);
    place(P.off_v, P.padded * 4);
    place(P.off_gp, P.padded * gsz);
    place(P.off_partials, partial_bytes);
    place(P.off_chunks, P.n_chunks * sizeof(Chunk));
    place(P.off_rows, (uint64_t)n * sizeof(BlockRow));
    place(P.off_tiles, (uint64_t)n * sizeof(TileRow));
    place(P.off_parts, P.parts.size() * sizeof(Part));
    place(P.off_multi, P.multi.size() * 4);
    place(P.off_once, (uint64_t)n * sizeof(OnceRow));
    place(P.off_task_block, P.n_tasks * 4);
    place(P.off_fin_block, P.n_fin * 4);
    place(P.off_rec, (uint64_t)n * kRecDoubles * 8);
    place(P.off_hist, (uint64_t)n * kHistWords * 4);
    place(P.off_arrived, (uint64_t)n * kArriveStride * 4);
    P.off_cleared = o;
    place(P.off_rvec, n_r * 4);
    place(P.off_cvec, n_c * 4);
    // The partial rows of the step are free in finalize.  The first pass's sums per task are folded before the second
    // leaves its own in their place.
    const uint64_t per_task = task_bytes(P.n_tasks);
    if (sums_fit(P.n_tasks)) P.off_residpart = P.off_partials; else place(P.off_residpart, per_task);
    if (counts_fit(P.n_tasks)) P.off_candcount = P.off_partials + per_task; else if (P.any_matrix) place(P.off_candcount, per_task);
    P.off_cand = o; P.off_rowpart = o; P.off_colpart = align_up(o + n_rowpart * 4, 256);
    P.total = o + list_bytes;
    P.off_step_rows = fine ? P.off_cand : P.off_partials;
    plan_once(P, total);
    return BAOC_OK;
}

template <int GT, int G, int NW, int MEM, typename... Args>
static void launch_step_as(bool first, bool fold, uint32_t grid, uint32_t lds, hipStream_t st, Args... a)
{
    const dim3 g(grid), b(64 * NW);
    if (first && fold) hipLaunchKernelGGL((k_step<GT, true, G, NW, true, MEM>), g, b, lds, st, a...);
    else if (first) hipLaunchKernelGGL((k_step<GT, true, G, NW, false, MEM>), g, b, lds, st, a...);
    else if (fold) hipLaunchKernelGGL((k_step<GT, false, G, NW, true, MEM>), g, b, lds, st, a...);
    else hipLaunchKernelGGL((k_step<GT, false, G, NW, false, MEM>), g, b, lds, st, a...);
}

// The instantiation for groups per wavefront and wavefronts per workgroup; the values were validated at begin.  What small layouts do with
// the caches is built for the shapes that they have by default.
template <int GT, typename... Args>
static void launch_step(uint32_t gpw, uint32_t nw, Memory memory, Args... a)
{
    constexpr uint32_t G = kSmallShape[GT].groups_per_wave, N = kSmallShape[GT].waves_per_workgroup;
    if (gpw == G && nw == N && memory == kKept) { launch_step_as<GT, G, N, kKept>(a...); return; }
    if constexpr (GT == BAOC_GRAD_F32)
        if (gpw == G && nw == N && memory == kHinted) { launch_step_as<GT, G, N, kHinted>(a...); return; }
#define BAOC_STEP_CASE(GG, NN) if (gpw == GG && nw == NN) { launch_step_as<GT, GG, NN, kThrough>(a...); return; }
    BAOC_STEP_CASE(1, 1) BAOC_STEP_CASE(2, 1) BAOC_STEP_CASE(1, 2) BAOC_STEP_CASE(2, 2) BAOC_STEP_CASE(1, 4) BAOC_STEP_CASE(2, 4)
#undef BAOC_STEP_CASE
}

extern "C" void baoc_profile_params_default(baoc_profile_params* p)
{
    if (!p) return;
    p->beta_m = 0.9f; p->beta_v = 0.999f; p->beta_rho = 0.9; p->eps = 1e-12; p->eps_update = 1e-8f;
    p->quant_block = kQB; p->grad_dtype = BAOC_GRAD_F32;
    p->chunk_groups = 0; p->chunk_slices = 0; p->groups_per_wave = 0; p->waves_per_workgroup = 0; p->resident_workgroups = 0;
}

extern "C" int baoc_profile_workspace_bytes(const baoc_block* blocks, uint32_t n_blocks,
                                            const baoc_profile_params* params, uint64_t* out_bytes)
{
    if (!out_bytes) return BAOC_ERR_INVALID;
    Plan P;
    int rc = make_plan(blocks, n_blocks, params, &P, nullptr);
    if (rc) return rc;
    *out_bytes = P.total;
    return BAOC_OK;
}

// Shared by the two begin calls: plan, carve `d_workspace`, clear what must start at zero, upload the tables.
static int begin_on(const baoc_block* blocks, uint32_t n_blocks, const baoc_profile_params* params,
                    void* d_workspace, uint64_t workspace_bytes, bool pinned, baoc_profiler** out)
{
    baoc_profiler* h = new (std::nothrow) baoc_profiler();
    if (!h) return BAOC_ERR_INVALID;
    int rc = make_plan(blocks, n_blocks, params, &h->plan, &h->max_end);
    if (rc) { delete h; return rc; }
    if (workspace_bytes < h->plan.total || (reinterpret_cast<uintptr_t>(d_workspace) & 255)) { delete h; return BAOC_ERR_WORKSPACE; }
    h->params = *params;
    h->blocks.assign(blocks, blocks + n_blocks);
    h->ws = static_cast<char*>(d_workspace);
    const Plan& P = h->plan;
    // The tables go up in one piece.  The first step treats m, v and g_prev as zero without reading them and writes
    // all of them (padding included), so only the records, histograms and counters are cleared.
    std::vector<char> tables(P.off_task_block - P.off_rows);
    std::memcpy(tables.data(), P.rows.data(), P.rows.size() * sizeof(BlockRow));
    std::memcpy(tables.data() + (P.off_tiles - P.off_rows), P.tiles.data(), P.tiles.size() * sizeof(TileRow));
    if (!P.parts.empty()) std::memcpy(tables.data() + (P.off_parts - P.off_rows), P.parts.data(), P.parts.size() * sizeof(Part));
    if (!P.multi.empty()) std::memcpy(tables.data() + (P.off_multi - P.off_rows), P.multi.data(), P.multi.size() * 4);
    std::memcpy(tables.data() + (P.off_once - P.off_rows), P.once.data(), P.once.size() * sizeof(OnceRow));
    hipError_t e = hipMemcpy(h->ws + P.off_rows, tables.data(), tables.size(), hipMemcpyHostToDevice);
    if (e == hipSuccess) {
        const uint64_t n_clear = (P.off_cleared - P.off_rec) / 16, work = std::max({P.n_chunks, P.n_tasks, P.n_fin, n_clear});
        hipLaunchKernelGGL(k_build, dim3((uint32_t)std::min<uint64_t>((work + 255) / 256, 8192)), dim3(256), 0, nullptr,
                           reinterpret_cast<const BlockRow*>(h->ws + P.off_rows), reinterpret_cast<const TileRow*>(h->ws + P.off_tiles), n_blocks,
                           reinterpret_cast<Chunk*>(h->ws + P.off_chunks), (uint32_t)P.n_chunks,
                           reinterpret_cast<uint32_t*>(h->ws + P.off_task_block), (uint32_t)P.n_tasks,
                           reinterpret_cast<uint32_t*>(h->ws + P.off_fin_block), (uint32_t)P.n_fin,
                           reinterpret_cast<uint4*>(h->ws + P.off_rec), n_clear);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e != hipSuccess) { (void)hipGetLastError(); delete h; return BAOC_ERR_HIP; }
    const uint64_t rec_bytes = (uint64_t)n_blocks * kRecDoubles * sizeof(double);
    if (pinned) h->host_rec = pool_take(rec_bytes, &h->host_bytes);
    if (!h->host_rec) h->h_rec.resize((size_t)n_blocks * kRecDoubles);
    *out = h;
    return BAOC_OK;
}

extern "C" int baoc_profile_begin(const baoc_block* blocks, uint32_t n_blocks,
                                  const baoc_profile_params* params,
                                  void* d_workspace, uint64_t workspace_bytes, baoc_profiler** out)
{
    if (!out || !d_workspace) return BAOC_ERR_INVALID;
    return begin_on(blocks, n_blocks, params, d_workspace, workspace_bytes, true, out);
}

extern "C" int baoc_profile_begin_static(const baoc_block* blocks, uint32_t n_blocks,
                                         const baoc_profile_params* params, baoc_profiler** out)
{
    if (!out) return BAOC_ERR_INVALID;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) { (void)hipGetLastError(); return BAOC_ERR_HIP; }
    if (dev < 0 || dev >= kMaxDevices) return BAOC_ERR_UNSUPPORTED;
    if (g_scratch_busy[dev]) return BAOC_ERR_STATE;            // one handle at a time shares the array
    if (!g_scratch_ptr[dev]) {                                 // first use on this device: where its copy of the array lives
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) { (void)hipGetLastError(); return BAOC_ERR_HIP; }
        g_scratch_ptr[dev] = ptr;
    }
    const int rc = begin_on(blocks, n_blocks, params, g_scratch_ptr[dev], BAOC_STATIC_WORKSPACE_BYTES, false, out);
    if (rc == BAOC_OK) { (*out)->static_device = dev; g_scratch_busy[dev] = true; }
    return rc;
}

extern "C" int baoc_profile_step(baoc_profiler* h, const void* d_grad_flat, uint64_t grad_numel, void* hip_stream)
{
    if (!h || !d_grad_flat) return BAOC_ERR_INVALID;
    if (h->sticky) return h->sticky;
    if (grad_numel < h->max_end) return BAOC_ERR_INVALID;
    const Plan& P = h->plan;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const baoc_profile_params& q = h->params;
    StepConsts k{q.beta_m, q.beta_v, 1.0f - q.beta_m, 1.0f - q.beta_v, q.eps_update};
    float* m = reinterpret_cast<float*>(h->ws + P.off_m);
    float* v = reinterpret_cast<float*>(h->ws + P.off_v);
    const Chunk* ch = reinterpret_cast<const Chunk*>(h->ws + P.off_chunks);
    float* part = reinterpret_cast<float*>(h->ws + P.off_step_rows);
    const bool first = h->steps == 0;
    // The first launch is bound by its arithmetic and runs at full residency.  Later launches are bound
    // by DRAM and run with fewer resident workgroups: each is given so much unused LDS that only about
    // `resident` of them fit a compute unit (allocations are counted in multiples of 2 KB here).
    const uint32_t static_lds = P.nw * 4 * kNumSums * (P.fold_in_step ? 4 + 8 : 4) + (P.fold_in_step ? 8 : 0);
    uint32_t lds = 0;
    if (!first && P.resident * P.nw < 32) lds = kLdsBytesPerCU / P.resident / 2048 * 2048 - static_lds;
    const uint32_t grid = (uint32_t)P.n_prows;
    const BlockRow* rows = reinterpret_cast<const BlockRow*>(h->ws + P.off_rows);
    double* rec = reinterpret_cast<double*>(h->ws + P.off_rec);
    const FoldArgs fold{rows, reinterpret_cast<uint32_t*>(h->ws + P.off_arrived), rec, q.beta_rho, q.eps};
    if (q.grad_dtype == BAOC_GRAD_F32)
        launch_step<BAOC_GRAD_F32>(P.gpw, P.nw, P.memory, first, P.fold_in_step, grid, lds, st, static_cast<const float*>(d_grad_flat), m, v,
                                   reinterpret_cast<float*>(h->ws + P.off_gp), ch, part, k, P.slices, P.slice_groups, fold);
    else
        launch_step<BAOC_GRAD_BF16>(P.gpw, P.nw, P.memory, first, P.fold_in_step, grid, lds, st, static_cast<const uint16_t*>(d_grad_flat), m, v,
                                    reinterpret_cast<uint16_t*>(h->ws + P.off_gp), ch, part, k, P.slices, P.slice_groups, fold);
    h->steps += 1;
    if (!P.fold_in_step) {
        if (!P.parts.empty())
            hipLaunchKernelGGL(k_reduce_parts, dim3((uint32_t)P.parts.size()), dim3(256), 0, st,
                               part, rows, reinterpret_cast<const Part*>(h->ws + P.off_parts));
        hipLaunchKernelGGL(k_reduce, dim3((uint32_t)P.rows.size()), dim3(256), 0, st, part, rows, rec, q.beta_rho, q.eps);
    }
    if (hipGetLastError() != hipSuccess) { h->sticky = BAOC_ERR_HIP; return BAOC_ERR_HIP; }
    return BAOC_OK;
}

extern "C" int baoc_profile_finalize(baoc_profiler* h, const baoc_config* configs, uint32_t n_configs,
                                     const baoc_risk_params* risk_params,
                                     baoc_block_stats* out_stats, double* out_risk, void* hip_stream)
{
    if (!h) return BAOC_ERR_INVALID;
    if (h->sticky) return h->sticky;
    if (h->steps == 0) return BAOC_ERR_STATE;
    if (out_risk && (!configs || n_configs == 0)) return BAOC_ERR_INVALID;
    for (uint32_t c = 0; out_risk && c < n_configs; ++c) {
        const baoc_config& k = configs[c];
        if ((k.bits != 32 && k.bits != 16 && k.bits != 8) || k.y_a > 1 || k.y_m > 1 || k.y_d > 1 || k.y_f > 1) return BAOC_ERR_INVALID;
    }
    baoc_risk_params rp;
    if (risk_params) rp = *risk_params; else baoc_risk_params_default(&rp);
    if (!(rp.A_high != rp.A_low) || !(rp.rho_high != rp.rho_low) || !(rp.eta_high != rp.eta_low)) return BAOC_ERR_INVALID;

    const bool want_F = !rp.F_raw && rp.compute_F && h->plan.any_matrix;
    const bool want_C = !rp.C_raw && rp.d_theta_flat;
    if (want_C && (rp.theta_numel < h->max_end || (rp.theta_dtype != BAOC_GRAD_F32 && rp.theta_dtype != BAOC_GRAD_BF16)))
        return BAOC_ERR_INVALID;

    const Plan& P = h->plan;
    const uint32_t N = (uint32_t)P.rows.size(), n_tasks = (uint32_t)P.n_tasks;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    auto f32_at = [&](uint64_t off) { return reinterpret_cast<float*>(h->ws + off); };
    auto u32_at = [&](uint64_t off) { return reinterpret_cast<uint32_t*>(h->ws + off); };
    const float* v = f32_at(P.off_v);
    const TileRow* tiles = reinterpret_cast<const TileRow*>(h->ws + P.off_tiles);
    const uint32_t* task_block = u32_at(P.off_task_block);
    uint32_t *arrived = u32_at(P.off_arrived), *scan3 = arrived + L_SCAN3;   // a block's flag stands next to its counter
    uint32_t *cand = u32_at(P.off_cand), *cand_count = u32_at(P.off_candcount);
    const uint32_t* multi = u32_at(P.off_multi);
    const uint32_t n_multi = (uint32_t)P.multi.size(), n_fold1 = n_multi + (want_F ? (uint32_t)P.n_fin : 0);
    float *rvec = f32_at(P.off_rvec), *cvec = f32_at(P.off_cvec), *rowpart = f32_at(P.off_rowpart), *colpart = f32_at(P.off_colpart);
    double2* taskpart = reinterpret_cast<double2*>(h->ws + P.off_residpart);
    float4* residpart = reinterpret_cast<float4*>(h->ws + P.off_residpart);
    double* rec = reinterpret_cast<double*>(h->ws + P.off_rec);
    const Selection sel{u32_at(P.off_hist), u32_at(P.off_rec) + 2 * R_ORDER, u32_at(P.off_rec) + 2 * R_ORDER + 4};
    const float epsf = (float)h->params.eps;
    // v above which eps stays below a thousandth of sqrt(v) (and v is a normal number)
    const float eps_low = std::max(std::numeric_limits<float>::min(), (float)(1e6 * h->params.eps * h->params.eps));

    const std::true_type yes; const std::false_type no;
    const std::integral_constant<int, BAOC_GRAD_F32> t32; const std::integral_constant<int, BAOC_GRAD_BF16> t16;
    auto with_kinds = [&](auto f) {                            // calls f(type of theta, F wanted, C wanted)
        if (!want_C) { if (want_F) f(t32, yes, no); else f(t32, no, no); }
        else if (rp.theta_dtype == BAOC_GRAD_F32) { if (want_F) f(t32, yes, yes); else f(t32, no, yes); }
        else if (want_F) f(t16, yes, yes);
        else f(t16, no, yes);
    };
    double* const out = h->host_rec ? h->host_rec : rec;
    const OnceRow* once = P.once_tasks && P.once_worth[want_C] ? reinterpret_cast<const OnceRow*>(h->ws + P.off_once) : nullptr;
    auto one_pass = [&]() {
        const OnceMem mem{h->ws + P.off_rvec, reinterpret_cast<OnceSums*>(h->ws + P.off_once_sums), reinterpret_cast<OnceUnit*>(h->ws + P.off_once_units),
                          once, N, P.once_narrow, arrived, sel.hist, rec, out};
        if (P.once_multi) hipLaunchKernelGGL(k_bracket, dim3(N), dim3(1024), 0, st, v, tiles, mem, epsf);
        with_kinds([&](auto tt, auto f, auto c) {
            constexpr int TT = decltype(tt)::value;
            constexpr bool F = decltype(f)::value, C = decltype(c)::value;
            auto pass = [&](auto waves, uint32_t tasks) {
                constexpr uint32_t NW = decltype(waves)::value;
                if (tasks)
                    hipLaunchKernelGGL((P.once_lines ? k_once<NW, TT, F, C, true> : k_once<NW, TT, F, C, false>), dim3(tasks), dim3(64 * NW), 0, st,
                                       v, static_cast<const typename GradIO<TT>::elem*>(rp.d_theta_flat), tiles, mem, epsf, eps_low);
            };
            pass(std::integral_constant<uint32_t, 16>(), P.once_tasks - P.once_narrow);
            pass(std::integral_constant<uint32_t, 8>(), P.once_narrow);
            if (P.once_units) hipLaunchKernelGGL((k_once_select<F, C>), dim3(P.once_units), dim3(256), 0, st, tiles, mem);
        });
    };
    auto passes = [&]() {
        hipLaunchKernelGGL(P.any_strips ? k_final1<true> : k_final1<false>, dim3(n_tasks), dim3(256), 0, st, v, tiles, task_block, rowpart, colpart,
                           rvec, cvec, taskpart, sel, scan3, rec, epsf, eps_low, want_C, once);
        if (n_fold1)
            hipLaunchKernelGGL(k_fold1, dim3(n_fold1), dim3(256), 0, st, tiles, multi, n_multi, u32_at(P.off_fin_block), rowpart, colpart, rvec, cvec,
                               taskpart, sel, scan3, rec, once);
        with_kinds([&](auto tt, auto f, auto c) {
            constexpr int TT = decltype(tt)::value;
            constexpr bool F = decltype(f)::value, C = decltype(c)::value;
            hipLaunchKernelGGL((P.any_strips ? k_final2<TT, F, C, true> : k_final2<TT, F, C, false>), dim3(n_tasks), dim3(256), 0, st,
                               v, static_cast<const typename GradIO<TT>::elem*>(rp.d_theta_flat), rp.theta_numel, tiles, task_block, rvec, cvec,
                               residpart, sel, cand, cand_count, scan3, rec, epsf, eps_low, once);
        });
        if (n_multi) hipLaunchKernelGGL(k_fold2, dim3(n_multi), dim3(256), 0, st, tiles, multi, residpart, sel, scan3, rec, once);
        hipLaunchKernelGGL(k_final3, dim3(n_tasks), dim3(256), 0, st, v, tiles, task_block, cand, cand_count, sel, arrived, scan3, rec, out, once);
    };
    // Waits for the records.  After an error too: the kernels are in flight, and the last one writes to host memory.
    auto wait = [&]() {
        hipError_t e = hipGetLastError();
        if (e == hipSuccess && !h->host_rec) e = hipMemcpyAsync(h->h_rec.data(), rec, h->h_rec.size() * 8, hipMemcpyDeviceToHost, st);
        const hipError_t waited = hipStreamSynchronize(st);
        if (waited != hipSuccess) h->host_lost = true;
        if (e == hipSuccess && waited == hipSuccess) return true;
        (void)hipGetLastError(); h->sticky = BAOC_ERR_HIP;
        return false;
    };
    const double* host = h->host_rec ? h->host_rec : h->h_rec.data();
    if (once) one_pass();
    if (!once || !P.once_all) passes();                       // and what the one pass left
    if (!wait()) return BAOC_ERR_HIP;
    if (once && P.once_all) {
        bool redo = false;
        for (uint32_t i = 0; i < N; ++i) redo |= host[(size_t)i * kRecDoubles + R_REDO] != 0.0;
        if (redo) {
            passes();
            if (!wait()) return BAOC_ERR_HIP;
        }
    }

    std::vector<baoc_block_stats> stats(N);
    for (uint32_t i = 0; i < N; ++i) {
        RawBlock r;
        const double* rec = host + (size_t)i * kRecDoubles;
        r.numel = P.rows[i].numel;
        for (int s = 0; s < (int)kNumSums; ++s) r.sums[s] = rec[s];
        r.rho_bar = rec[R_RHO]; r.cos_last = rec[R_COS];
        r.n_cos = (uint32_t)rec[R_NCOS]; r.steps = (uint32_t)rec[R_STEPS];
        for (int t = 0; t < 4; ++t) r.order_stat[t] = (float)rec[R_ORDER + t];
        const double p10 = 0.1 * (double)(r.numel - 1), p90 = 0.9 * (double)(r.numel - 1);
        r.frac10 = p10 - std::floor(p10); r.frac90 = p90 - std::floor(p90);
        const double eps = h->params.eps;
        double C_raw = rp.C_raw ? rp.C_raw[i] : 0.0, F_raw = rp.F_raw ? rp.F_raw[i] : 0.0;
        if (want_C) C_raw = std::sqrt(rec[R_CNUM]) / (std::sqrt(rec[R_CDEN]) + eps);                  // Eq. 6
        if (want_F && P.tiles[i].rows) F_raw = std::sqrt(rec[R_FRES]) / (std::sqrt(rec[S_VV]) + eps);   // Eq. 7
        block_metrics(r, eps, rp, C_raw, F_raw, &stats[i]);
    }
    if (out_stats) std::memcpy(out_stats, stats.data(), sizeof(baoc_block_stats) * N);
    if (out_risk)
        for (uint32_t i = 0; i < N; ++i)
            for (uint32_t c = 0; c < n_configs; ++c)
                out_risk[(size_t)i * n_configs + c] =
                    config_phi(stats[i], configs[c], rp.pref_mask && rp.pref_mask[c], rp);
    return BAOC_OK;
}

extern "C" int baoc_profile_state(const baoc_profiler* h, uint32_t block,
                                  const float** d_m, const float** d_v, const void** d_g_prev)
{
    if (!h || block >= h->plan.rows.size()) return BAOC_ERR_INVALID;
    const Plan& P = h->plan;
    const uint64_t s = P.rows[block].state_start;
    const uint64_t gsz = h->params.grad_dtype == BAOC_GRAD_F32 ? 4 : 2;
    if (d_m) *d_m = reinterpret_cast<const float*>(h->ws + P.off_m) + s;
    if (d_v) *d_v = reinterpret_cast<const float*>(h->ws + P.off_v) + s;
    if (d_g_prev) *d_g_prev = h->ws + P.off_gp + s * gsz;
    return BAOC_OK;
}

extern "C" int baoc_profile_end(baoc_profiler* h)
{
    if (!h) return BAOC_ERR_INVALID;
    if (h->static_device >= 0) g_scratch_busy[h->static_device] = false;
    if (h->host_rec && !h->host_lost) pool_give(h->host_rec, h->host_bytes);   // a lost buffer stays counted as pinned
    delete h;
    return BAOC_OK;
}

extern "C" const char* baoc_status_string(int s)
{
    switch (s) {
    case BAOC_OK: return "ok";
    case BAOC_ERR_INVALID: return "invalid argument";
    case BAOC_ERR_WORKSPACE: return "workspace too small or misaligned";
    case BAOC_ERR_UNSUPPORTED: return "unsupported parameter";
    case BAOC_ERR_HIP: return "HIP runtime error";
    case BAOC_ERR_INFEASIBLE: return "no assignment satisfies the budgets";
    case BAOC_ERR_LIMIT: return "solver node limit reached";
    case BAOC_ERR_STATE: return "call out of order";
    default: return "unknown status";
    }
}
