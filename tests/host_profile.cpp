// The host side of the profiler without a GPU: the library's own source, compiled for the host alone, on a HIP runtime that
// only keeps a record of the calls made to it.  argv[1] names the check; a failed one prints what is wrong and returns 1.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>

// Constructed before the library's own objects and so destroyed after them, as an object of a program that loads the library later.
static struct AtExit { void (*last)() = nullptr; ~AtExit() { if (last) last(); } } g_at_exit;

#include "baoc_profile.hip"

#include <string>
#include <sys/mman.h>
#include <sys/wait.h>
#include <unistd.h>

// Freed memory is kept, filled with a pattern, once g_keep_freed is set.
static bool g_keep_freed = false;
static struct { unsigned char* p; size_t n; } g_freed[4096];
static size_t g_n_freed = 0;
void* operator new(size_t n)
{
    auto* p = static_cast<size_t*>(std::malloc(n + 16));
    if (!p) throw std::bad_alloc();
    *p = n;
    return reinterpret_cast<char*>(p) + 16;
}
void operator delete(void* p) noexcept
{
    if (!p) return;
    size_t* whole = reinterpret_cast<size_t*>(static_cast<char*>(p) - 16);
    if (!g_keep_freed || g_n_freed == 4096) { std::free(whole); return; }
    std::memset(p, 0xdd, *whole);
    g_freed[g_n_freed].p = static_cast<unsigned char*>(p); g_freed[g_n_freed++].n = *whole;
}
void operator delete(void* p, size_t) noexcept { operator delete(p); }

#define CHECK(cond, ...) \
    do { if (!(cond)) { std::printf("line %d: %s ", __LINE__, #cond); std::printf(__VA_ARGS__); std::printf("\n"); return 1; } } while (0)

// ---------------------------------------------------------------------------
// the runtime
// ---------------------------------------------------------------------------

static std::string g_calls;                               // L launch, S wait for a stream, P pinned allocation
static hipError_t g_last_error = hipSuccess, g_wait = hipSuccess;   // what the next hipGetLastError and every wait return
static void* g_pinned = nullptr;                          // the last pinned allocation

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* handle = nullptr; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t*, hipStream_t*) { return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { g_calls += 'L'; return hipSuccess; }
hipError_t hipGetLastError() { const hipError_t e = g_last_error; g_last_error = hipSuccess; return e; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { g_calls += 'S'; return g_wait; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { *p = scratch; return hipSuccess; }
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned)
{
    g_calls += 'P';
    *p = g_pinned = std::calloc(1, n);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
}

// ---------------------------------------------------------------------------
// layouts
// ---------------------------------------------------------------------------

static void add(std::vector<baoc_block>& l, uint64_t rows, uint64_t cols, uint32_t times = 1)
{
    for (; times; --times) {
        const uint64_t at = l.empty() ? 0 : l.back().offset + l.back().numel;
        l.push_back(cols ? baoc_block{at, rows * cols, (uint32_t)rows, (uint32_t)cols} : baoc_block{at, rows, 0, 0});
    }
}

static baoc_profile_params params_of(uint32_t dtype)
{
    baoc_profile_params p;
    baoc_profile_params_default(&p);
    p.grad_dtype = dtype;
    return p;
}

// ---------------------------------------------------------------------------
// the plan of a step
// ---------------------------------------------------------------------------

// Workgroups of the step and of the reduction cover every group and every row once, and the rows stand inside the workspace.
static int check_step(const Plan& P, const char* name)
{
    uint64_t chunks = 0, rows = 0, part = 0;
    for (const BlockRow& r : P.rows) {
        const uint64_t groups = (r.numel + kQB - 1) / kQB;
        CHECK(r.first_chunk == chunks && r.first_prow == rows && r.n_prows == (uint64_t)r.n_chunks * P.slices, "%s", name);
        CHECK((uint64_t)r.n_chunks * r.groups_per_chunk >= groups && (uint64_t)(r.n_chunks - 1) * r.groups_per_chunk < groups, "%s", name);
        CHECK((uint64_t)P.slices * P.slice_groups >= r.groups_per_chunk, "%s", name);
        // what six rounds of a workgroup take is summed in one launch, more in parts of at most 2,047 rows
        const uint32_t n_parts = r.n_prows > kDirectRows ? r.n_prows / kPartRows : 0;
        for (uint32_t q = 0; q < n_parts; ++q, ++part)
            CHECK(part < P.parts.size() && P.parts[part].block == (uint32_t)(&r - P.rows.data()) && P.parts[part].part == q, "%s: %u rows", name,
                  r.n_prows);
        chunks += r.n_chunks; rows += r.n_prows;
    }
    CHECK(chunks == P.n_chunks && rows == P.n_prows && part == P.parts.size(), "%s", name);
    CHECK(P.off_step_rows == P.off_partials ? P.off_step_rows + rows * kNumSums * 4 <= P.off_chunks : P.off_step_rows == P.off_cand, "%s", name);
    CHECK(P.n_prows * 64 * P.nw <= 0xffffffffull, "%s: a launch has fewer than 2^32 threads", name);
    CHECK(P.off_step_rows + rows * kNumSums * 4 <= P.total && P.off_chunks + chunks * sizeof(Chunk) <= P.off_rows, "%s", name);
    return 0;
}

// Large fp32 layouts: workgroups of one wavefront and one group, chunks of eight groups unless these would leave many workgroups
// without one, rows in the region of the lists; elsewhere, and next to a caller's own values, the other shapes.
static int check_plans()
{
    struct Want { const char* name; uint32_t dtype, gpw, nw, slices, resident; bool in_lists; };
    auto run = [&](const std::vector<baoc_block>& l, baoc_profile_params p, Want w) {
        Plan P;
        CHECK(make_plan(l.data(), (uint32_t)l.size(), &p, &P, nullptr) == BAOC_OK, "%s", w.name);
        CHECK(P.gpw == w.gpw && P.nw == w.nw && P.slices == w.slices && P.resident == w.resident, "%s: %u %u %u %u", w.name, P.gpw, P.nw,
              P.slices, P.resident);
        CHECK((P.off_step_rows == P.off_cand) == w.in_lists, "%s", w.name);
        return check_step(P, w.name);
    };
    std::vector<baoc_block> matrices, vectors, tiny, below, edges, huge;
    add(matrices, 4096, 2048, 9); add(matrices, 2049, 4099); add(matrices, 5, 0, 7);
    add(vectors, (1u << 26) + 5, 0);
    add(tiny, 30, 40, 60000);
    add(below, 4096, 2048, 7);
    for (uint64_t g : {1u, 7u, 8u, 9u, 3064u, 3071u, 3072u, 3073u, 3080u, 4095u, 4097u, 5119u, 6144u, 6145u}) { add(edges, g, 256); add(edges, 1, 0); }
    add(edges, 4096, 8192, 2);
    add(huge, 65535, 65535, 4); add(huge, 4096, 4096);                      // 17.2 G coordinates, 67.2 M groups
    const baoc_profile_params f32 = params_of(BAOC_GRAD_F32), bf16 = params_of(BAOC_GRAD_BF16);
    baoc_profile_params own = f32;
    own.resident_workgroups = 12;
    return run(matrices, f32, {"matrices", 0, 1, 1, 8, 16, true}) || run(edges, f32, {"edges", 0, 1, 1, 8, 16, true}) ||
           run(huge, f32, {"huge", 0, 2, 1, 2, 10, false}) || run(vectors, f32, {"vectors", 0, 2, 1, 2, 10, false}) || run(tiny, f32, {"tiny", 0, 1, 1, 4, 16, true}) ||
           run(below, f32, {"below", 0, 2, 2, 1, 5, false}) || run(matrices, own, {"own", 0, 2, 1, 2, 12, false}) ||
           run(matrices, bf16, {"bf16", 1, 2, 4, 1, 3, false});
}

// ---------------------------------------------------------------------------
// pinned memory
// ---------------------------------------------------------------------------

static baoc_profiler* stepped(const std::vector<baoc_block>& l, void* workspace, uint64_t bytes)
{
    const baoc_profile_params p = params_of(BAOC_GRAD_F32);
    baoc_profiler* h = nullptr;
    if (baoc_profile_begin(l.data(), (uint32_t)l.size(), &p, workspace, bytes, &h) != BAOC_OK) return nullptr;
    return baoc_profile_step(h, workspace, l.back().offset + l.back().numel, nullptr) == BAOC_OK ? h : nullptr;
}

// The last kernel of finalize writes the records to pinned memory.  After an error it may still be in flight: the call waits
// before it returns, and where waiting fails the buffer goes to no other handle.
static int check_finalize_error()
{
    std::vector<baoc_block> l;
    add(l, 64, 64, 8);
    const baoc_profile_params p = params_of(BAOC_GRAD_F32);
    uint64_t bytes = 0;
    CHECK(baoc_profile_workspace_bytes(l.data(), (uint32_t)l.size(), &p, &bytes) == BAOC_OK, " ");
    void* workspace = std::aligned_alloc(256, (bytes + 255) / 256 * 256);
    std::vector<baoc_block_stats> stats(l.size());
    auto finalize = [&](baoc_profiler* h) { return baoc_profile_finalize(h, nullptr, 0, nullptr, stats.data(), nullptr, nullptr); };

    baoc_profiler* h = stepped(l, workspace, bytes);
    CHECK(h && finalize(h) == BAOC_OK, " ");
    const void* first = g_pinned;
    CHECK(first && baoc_profile_end(h) == BAOC_OK, " ");

    h = stepped(l, workspace, bytes);                         // takes the buffer that was given back
    CHECK(h && g_pinned == first, " ");
    g_calls.clear();
    g_last_error = hipErrorInvalidValue;                      // of a launch, or the caller's own
    CHECK(finalize(h) == BAOC_ERR_HIP, " ");
    CHECK(g_calls.rfind('S') != std::string::npos && g_calls.rfind('S') > g_calls.rfind('L'), "%s", g_calls.c_str());
    CHECK(finalize(h) == BAOC_ERR_HIP && baoc_profile_end(h) == BAOC_OK, " ");

    h = stepped(l, workspace, bytes);                         // waited for: the buffer is free
    CHECK(h && g_pinned == first, " ");
    g_wait = hipErrorLaunchFailure;
    CHECK(finalize(h) == BAOC_ERR_HIP && baoc_profile_end(h) == BAOC_OK, " ");
    g_wait = hipSuccess;
    h = stepped(l, workspace, bytes);
    CHECK(h && g_pinned != first && finalize(h) == BAOC_OK && baoc_profile_end(h) == BAOC_OK, " ");
    return 0;
}

// A handle that is ended by the last destructor of the program, after the library's own objects: nothing of theirs is touched.
static baoc_profiler* g_last_handle = nullptr;
static int check_end_at_exit()
{
    static std::vector<baoc_block> l;
    add(l, 64, 64, 8);
    static std::vector<char> workspace(64 << 20);
    baoc_profiler* a = stepped(l, reinterpret_cast<void*>((reinterpret_cast<uintptr_t>(workspace.data()) + 255) / 256 * 256), 32 << 20);
    baoc_profiler* b = stepped(l, reinterpret_cast<void*>((reinterpret_cast<uintptr_t>(workspace.data()) + (32 << 20) + 255) / 256 * 256), 31 << 20);
    CHECK(a && b && baoc_profile_end(a) == BAOC_OK, " ");
    g_last_handle = b;
    g_keep_freed = true;
    g_at_exit.last = [] {
        int bad = baoc_profile_end(g_last_handle) != BAOC_OK;
        for (size_t i = 0; i < g_n_freed; ++i)
            for (size_t k = 0; k < g_freed[i].n; ++k) bad |= g_freed[i].p[k] != 0xdd;
        if (bad) { std::printf("memory that was given back is written\n"); std::fflush(stdout); std::_Exit(1); }
    };
    return 0;
}

// ---------------------------------------------------------------------------
// reads of the second finalize pass
// ---------------------------------------------------------------------------

// Memory that ends with a page without access: room for `n` elements right before it.
template <typename E> static E* before_wall(uint64_t n)
{
    const uint64_t page = 4096, bytes = (n * sizeof(E) + page - 1) / page * page;
    char* p = static_cast<char*>(mmap(nullptr, bytes + page, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0));
    if (p == MAP_FAILED || mprotect(p + bytes, page, PROT_NONE) != 0) std::abort();
    return reinterpret_cast<E*>(p + bytes) - n;
}

// Every load of every lane of a pass over the last block of a layout, in the order of k_final2, by the kernel's own
// functions.  `behind` elements past the block may be read; the pass is told that `claimed` may.  Counts how often an element
// is given to a lane that uses it.
template <int TT>
static int read_block(const Plan& P, uint64_t behind, uint64_t claimed)
{
    typedef typename GradIO<TT>::elem E;
    const TileRow& m = P.tiles.back();
    const uint64_t n = m.numel;
    E* const src = before_wall<E>(n + behind);
    for (uint64_t i = 0; i < n; ++i) src[i] = TT == BAOC_GRAD_F32 ? (E)(i % 8191) : (E)(i % 65521);
    std::vector<uint8_t> used(n, 0);
    const uint64_t left = claimed == kAnywhere ? kAnywhere : n + claimed;
    const bool lines = whole_lines(src, m.cols);
    typename GradIO<TT>::vec4 x[kQuads];
    auto take = [&](const TilePart& t, uint32_t i) {
        for (uint32_t q = 0; q < kQuads; ++q) {
            E e[4];
            std::memcpy(e, &x[q], sizeof e);
            const uint64_t row = round_row(t, i) + 4 * q + t.lrow;
            for (uint32_t k = 0; k < t.n_ok && row < t.rows; ++k) {
                const uint64_t at = row * m.cols + t.col + k;
                if (e[k] != src[at]) return false;
                ++used[at];
            }
        }
        return true;
    };
    for (uint32_t wg = m.first_task; wg < m.first_task + m.n_tasks; ++wg) {
        const Task task = task_of<true>(m, wg);
        for (uint32_t thread = 0; thread < 256; ++thread)
            for (uint32_t tile = task.tile; tile < task.last; ++tile) {
                const TilePart t = tile_part(m, task.seg, tile, thread & 63u, thread >> 6, left);
                const uint32_t full = tile == task.tile ? t.full : 0;            // of tiles side by side only the first has its loads issued ahead
                CHECK(t.full <= t.rounds && (m.strips == 1 || t.rounds == 1), "%u x %u", m.rows, m.cols);
                for (uint32_t i = 0; i < t.rounds && t.any; ++i) {
                    if (i < full) load_full<TT>(x, src, lines, t, m.cols, i);
                    else load_edge<TT>(x, src, left, t, m.cols, i);
                    CHECK(take(t, i), "%u x %u: round %u of thread %u", m.rows, m.cols, i, thread);
                }
            }
    }
    for (uint64_t i = 0; i < n; ++i) CHECK(used[i] == 1, "%u x %u: element %llu is used %u times", m.rows, m.cols, (unsigned long long)i, used[i]);
    return 0;
}

// Whether reading ends at the wall.
template <int TT> static bool hits_wall(const Plan& P, uint64_t behind, uint64_t claimed)
{
    std::fflush(stdout);
    const pid_t child = fork();
    if (child == 0) std::_Exit(read_block<TT>(P, behind, claimed) ? 3 : 0);
    int status = 0;
    waitpid(child, &status, 0);
    return WIFSIGNALED(status) && WTERMSIG(status) == SIGSEGV;
}

// The parameters' last block, at any alignment: nothing behind it is read, every element is used once.  v may be read up to
// three elements past the block.  A pass that is told of three elements more than there are runs into the wall where its last
// round has all rows and lacks columns.
static int check_reads()
{
    static const uint32_t shapes[][2] = {{2, 2}, {2, 3}, {3, 5}, {15, 63}, {16, 2}, {17, 2}, {16, 64}, {16, 65}, {32, 63}, {48, 67}, {64, 127},
                                         {64, 128}, {65, 127}, {160, 129}, {16, 1027}, {16, 2049}, {5, 2049}, {256, 257}, {512, 61}, {513, 66},
                                         {1025, 62}, {129, 4}, {4097, 5}, {130, 256}, {48, 100}};
    for (const auto& shape : shapes)
        for (uint32_t vector : {0u, 1u << 29}) {                             // next to a large block tiles are the largest
            std::vector<baoc_block> l;
            if (vector) add(l, vector, 0);
            add(l, shape[0], shape[1]);
            const baoc_profile_params p = params_of(BAOC_GRAD_BF16);
            Plan P;
            CHECK(make_plan(l.data(), (uint32_t)l.size(), &p, &P, nullptr) == BAOC_OK, "%u x %u", shape[0], shape[1]);
            if (read_block<BAOC_GRAD_F32>(P, 0, 0) || read_block<BAOC_GRAD_BF16>(P, 0, 0) || read_block<BAOC_GRAD_F32>(P, 3, kAnywhere)) return 1;
            // a lane without a column reads from the last one on, the last lane with one from its own
            const uint32_t rest = shape[1] % 64, past = rest <= 60 ? 3 : 64 - rest;
            if (shape[0] % kRoundRows == 0 && rest != 0)
                CHECK(hits_wall<BAOC_GRAD_F32>(P, 0, 3) && hits_wall<BAOC_GRAD_BF16>(P, 0, 3) && hits_wall<BAOC_GRAD_F32>(P, past - 1, kAnywhere),
                      "%u x %u", shape[0], shape[1]);
        }
    return 0;
}

// States that fill half of the memory-side cache at most stay there, larger ones go past it; fp32 layouts of 35 to 58 M coordinates
// carry the hint on all accesses, with the workgroups that go with it.
static int check_memory()
{
    for (uint32_t dtype : {BAOC_GRAD_F32, BAOC_GRAD_BF16}) {
        const uint64_t most = (128ull << 20) / (dtype == BAOC_GRAD_F32 ? 12 : 10) / kQB * kQB;
        const Memory middle = dtype == BAOC_GRAD_F32 ? kHinted : kThrough;
        for (const auto& [n, want] : {std::pair<uint64_t, Memory>{1, kKept}, {most, kKept}, {most + 1, kThrough},
                                      {kSmallLayout - 1, kThrough}, {kSmallLayout, middle}, {kHintedLayout - 1, middle}, {kHintedLayout, kThrough}, {1u << 28, kThrough}}) {
            std::vector<baoc_block> l;
            add(l, n, 0);
            const baoc_profile_params p = params_of(dtype);
            Plan P;
            CHECK(make_plan(l.data(), 1, &p, &P, nullptr) == BAOC_OK && P.memory == want, "%llu", (unsigned long long)n);
            CHECK(want != kHinted || (P.gpw == 1 && P.nw == 4 && P.resident == 4), "%llu", (unsigned long long)n);
        }
    }
    return 0;
}

// ---------------------------------------------------------------------------
// finalize with one read of v
// ---------------------------------------------------------------------------

// Every element of a block is given to one lane that counts it, and no load leaves its row.
static int check_once_loads(const OnceRow& o, const TileRow& m)
{
    const uint32_t waves = o.geom >> 24 ? 16 : 8, lanes_log = o.geom & 15u, strips = (o.geom >> 4) & 15u, across = (o.geom >> 8) & 255u, down = (o.geom >> 16) & 255u;
    const uint32_t rpl = 6 - lanes_log, loads = strips == 1 ? 4 : strips == 2 ? 2 : 1, my_rows = loads << rpl, batch = down * my_rows;
    uint32_t wide = 1;
    while (wide < across) wide *= 2;
    CHECK(across * down <= waves && down >= 1 && lanes_log >= 4 && lanes_log <= 6 && strips >= 1 && strips <= 3, "%u x %u", m.rows, m.cols);
    CHECK((uint64_t)across * strips * (4u << lanes_log) >= m.cols && (1u << rpl) <= m.rows, "%u x %u", m.rows, m.cols);
    CHECK(across == 1 || down * wide * 16 <= waves * 32, "%u x %u: sums of a batch's rows", m.rows, m.cols);
    std::vector<uint8_t> used(m.numel, 0);
    for (uint32_t task = 0; task < o.n_tasks; ++task)
        for (uint32_t first = task * batch; first < m.rows; first += batch * o.n_tasks)
            for (uint32_t wave = 0; wave < across * down; ++wave)
                for (uint32_t q = 0; q < loads; ++q)
                    for (uint32_t k = 0; k < strips; ++k)
                        for (uint32_t lane = 0; lane < 64; ++lane) {
                            const uint32_t row = first + wave / across * my_rows + (q << rpl), lrow = lane >> lanes_log;
                            const uint32_t col = ((wave % across * strips + k) << (lanes_log + 2)) + 4 * (lane & ((1u << lanes_log) - 1u));
                            const uint32_t r = once_first_row(row, rpl, m.rows) + lrow, c = once_first_col(col, m.cols);
                            CHECK(r < m.rows && c + 4 <= m.cols, "%u x %u: row %u, column %u", m.rows, m.cols, r, c);
                            for (uint32_t e = once_skip(row, lrow, rpl, m.rows, col, m.cols); e < 4; ++e) ++used[(uint64_t)r * m.cols + c + e];
                        }
    for (uint64_t i = 0; i < m.numel; ++i) CHECK(used[i] == 1, "%u x %u: element %llu is counted %u times", m.rows, m.cols, (unsigned long long)i, used[i]);
    return 0;
}

// Keys of an interval have bins, and those of a crowded range cells, inside their words; intervals are in order and apart.
static int check_once_intervals()
{
    for (uint32_t numel : {12290u, 65537u, (1u << 20) - 1, 1u << 21, 1u << 28}) {
        const uint32_t bins_log = once_bins_log(numel), slots = 1u << once_slots_log(bins_log), cap = once_keys_cap(numel), cells = 1u << once_cells_log(cap);
        CHECK(2 * slots <= kHistWords && 3 * cells <= cap && cells <= 1024 && cap <= kOnceKeys, "%u", numel);
        for (uint32_t bits = 0; bits < 31; ++bits)
            for (uint32_t width : {(1u << bits) - 1, 1u << bits, (1u << bits) + 1}) {
                if (width == 0) continue;
                CHECK((width - 1) >> once_shift(width, bins_log) < slots && (width - 1) >> width_shift(width, once_cells_log(cap)) < cells, "%u of %u", width, numel);
            }
    }
    const uint32_t n = 1u << 22, top = 0x7f800000u >> kBits3;
    const struct { uint32_t prefix[4]; bool ok, one; } cases[] = {
        {{100, 200, 300, 400}, true, false}, {{0, 0, 300, 400}, true, false}, {{0, 0, 0, 400}, true, true}, {{0, 0, 0, 0}, true, true},
        {{7, 7, 7, 7}, true, true}, {{100, 200, 200, 300}, false, true}, {{100, 200, 201, 300}, true, false}, {{100, 200, 300, top}, false, false},
        {{top, n - 1, n - 1, n - 1}, false, false}};
    for (const auto& c : cases) {
        uint32_t end[4];
        CHECK(once_intervals(c.prefix, end) == c.ok, "%u %u %u %u", c.prefix[0], c.prefix[1], c.prefix[2], c.prefix[3]);
        if (!c.ok) continue;
        CHECK(end[0] >= 1 && end[0] < end[1] && end[1] <= end[2] && (end[2] == end[3]) == c.one && end[2] <= end[3], "%u %u %u %u", end[0], end[1], end[2], end[3]);
        CHECK(end[3] == (c.prefix[3] + 1) << kBits3, "%u", end[3]);
    }
    return 0;
}

// Which layouts and blocks take the one pass, and that its memory is what the passes have for r, c and the lists, each part of it apart.
static int check_once()
{
    std::vector<baoc_block> edges, few, small, vectors, many, tiny, idle, idle_wide, vectors_most, whole, whole_wide;
    for (uint32_t c : {2u, 3u, 4u, 5u, 63u, 64u, 65u, 127u, 128u, 129u, 191u, 192u, 193u, 255u, 256u, 257u, 511u, 513u, 767u, 768u, 769u, 1023u, 1025u, 2305u, 4095u,
                       4097u, 4608u, 6143u, 6144u, 6145u, 11008u, 12287u, 12288u, 12289u, 30000u})
        for (uint32_t r : {2u, 3u, 5u, 17u, 33u}) add(edges, r, c);
    add(edges, 1030, 67); add(edges, 300, 2304); add(edges, 41, 11008); add(edges, 700, 100); add(edges, 3, 0); add(edges, 4, 0); add(edges, 65536, 0); add(edges, 65537, 0);
    few = edges;
    add(edges, 16384, 8192, 3); add(edges, 16385, 16384);                    // the latter has more than 2^28 coordinates
    add(few, 16384, 8192, 2);                                                // blocks that do not take part next to fewer than 3 * 2^27
    add(small, 16384, 8191);                                                 // below 2^27 in all
    add(vectors, 1u << 28, 0);                                               // no matrix: no room for lists
    add(tiny, 600, 500, 1000);                                               // blocks of 300,000 coordinates
    add(idle, 1152, 1152, 316); add(idle_wide, 455, 9216, 100);              // a quarter of the lanes has no work; without theta the first are worth it
    add(vectors_most, 20000000, 0, 7); add(vectors_most, 5802, 3484); add(vectors_most, 893, 11114); add(vectors_most, 979, 8138);   // room for long lists only
    add(whole, 1024, 1024, 400); add(whole_wide, 512, 8192, 100);
    add(many, 1024, 1024, 600); add(many, 4096, 11008, 3); add(many, 50000, 0, 100);
    for (uint32_t dtype : {BAOC_GRAD_F32, BAOC_GRAD_BF16})
        for (const auto* l : {&edges, &few, &small, &vectors, &many, &tiny, &idle, &idle_wide, &vectors_most, &whole, &whole_wide}) {
            const baoc_profile_params p = params_of(dtype);
            Plan P;
            CHECK(make_plan(l->data(), (uint32_t)l->size(), &p, &P, nullptr) == BAOC_OK, " ");
            CHECK((P.once_tasks != 0 && P.once_worth[1]) == (l == &edges || l == &many || l == &whole || l == &whole_wide), "%u tasks", P.once_tasks);
            CHECK((P.once_tasks != 0 && P.once_worth[0]) == (l == &edges || l == &many || l == &whole || l == &whole_wide || l == &idle), "%u tasks", P.once_tasks);
            if (!P.once_tasks) continue;
            uint64_t narrow = 0, wide = 0, units = 0, part = 0, fixed = 0, lists = 0, first_list = ~0ull;
            for (size_t i = 0; i < l->size(); ++i) {
                const OnceRow& o = P.once[i];
                const TileRow& m = P.tiles[i];
                const bool takes = m.numel >= 4 && m.numel <= 1ull << 28 && (!m.rows || (m.cols >= 4 && m.cols <= 12288));
                CHECK((o.n_tasks != 0) == takes && o.first_task == narrow && o.first_wide == wide && o.first_unit == units, "%u x %u", m.rows, m.cols);
                if (!takes) continue;
                ++part;
                CHECK((o.geom >> 24 != 0) == (m.rows && m.cols > 6144) && (m.numel > 65536 ? o.n_tasks > 1 : o.n_tasks == 1 || o.geom >> 24), "%u x %u", m.rows, m.cols);
                if (m.rows && m.numel < 1u << 21 && check_once_loads(o, m)) return 1;
                (o.geom >> 24 ? wide : narrow) += o.n_tasks;
                if (o.n_tasks == 1) continue;
                units += once_list_units(o) + once_col_units(m.rows, m.cols);
                CHECK(o.off_cols == fixed && o.list_cap % 16 == 0 && o.list_cap > 0, "%u x %u", m.rows, m.cols);
                fixed += once_cols_units(o.n_tasks, m.rows ? m.cols : 0) + ((uint64_t)once_keys_cap(m.numel) * 8 + 63) / 64;
                first_list = std::min<uint64_t>(first_list, o.off_list);
                CHECK(lists == 0 || o.off_list == lists, "%u x %u", m.rows, m.cols);
                lists = o.off_list + ((uint64_t)o.n_tasks * o.list_cap + once_spill(o)) / 16;
            }
            CHECK(narrow == P.once_narrow && narrow + wide == P.once_tasks && units == P.once_units && P.once_all == (part == l->size()), " ");
            CHECK(P.off_rvec + fixed * 64 <= P.off_once_sums && P.off_once_sums + P.once_tasks * sizeof(OnceSums) <= P.off_once_units, " ");
            CHECK(P.off_once_units + units * sizeof(OnceUnit) <= P.off_rvec + first_list * 64 && P.off_rvec + lists * 64 <= P.total, " ");
        }
    return 0;
}

int main(int argc, char** argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "plans") return check_plans();
    if (what == "finalize_error") return check_finalize_error();
    if (what == "memory") return check_memory();
    if (what == "reads") return check_reads();
    if (what == "end_at_exit") return check_end_at_exit();
    if (what == "once") return check_once();
    if (what == "once_intervals") return check_once_intervals();
    std::printf("no check named '%s'\n", what.c_str());
    return 2;
}
