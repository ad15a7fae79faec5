// Heap use of baoc_allocate on instances whose budgets do not bind: every block keeps its cheapest configuration and
// no list of the search ever holds two states.  Prints calls of operator new and bytes per block and instance.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <new>
#include <random>
#include <vector>
#include "baoc.h"

static uint64_t g_calls = 0, g_bytes = 0;
void* operator new(size_t n)
{
    ++g_calls; g_bytes += n;
    if (void* p = std::malloc(n)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

int main()
{
    std::mt19937_64 rng(7);
    for (uint32_t N : {64u, 1000u, 5000u})
        for (uint32_t K : {4u, 21u}) {
            std::vector<double> risk((size_t)N * K), tc((size_t)N * K);
            std::vector<int64_t> mem((size_t)N * K);
            for (size_t i = 0; i < risk.size(); ++i) {
                risk[i] = (double)(rng() >> 11) * (1.0 / 9007199254740992.0); tc[i] = (double)(rng() % 1000) / 1000; mem[i] = (int64_t)(rng() % 1000000);
            }
            std::vector<uint32_t> choice(N);
            double obj, ot; int64_t om;
            g_calls = g_bytes = 0;
            const int rc = baoc_allocate(risk.data(), mem.data(), tc.data(), N, K, (int64_t)N * 1000000, 1.0 * N, nullptr, choice.data(), &obj, &om, &ot);
            std::printf("%u %u %d %.2f %.1f\n", N, K, rc, (double)g_calls / N, (double)g_bytes / N);
        }
    return 0;
}
