// The pool of pinned host blocks on the CPU: what it keeps is bounded, large blocks
// go back at once, kept ones are handed out again, from several threads.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <atomic>
#include <thread>
#include <vector>

#include "pinned_pool.h"

static std::atomic<long> g_blocks{0};
static bool g_full = false;
static void* sys_alloc(size_t n) {
    if (g_full) return nullptr;
    ++g_blocks;
    return std::malloc(n);
}
static void sys_free(void* p) {
    --g_blocks;
    std::free(p);
}

#define CHECK(c)                                                     \
    do {                                                             \
        if (!(c)) {                                                  \
            std::printf("failed: %s (line %d)\n", #c, __LINE__);     \
            return 1;                                                \
        }                                                            \
    } while (0)

int main() {
    using namespace pair;
    PinnedPool pool(sys_alloc, sys_free);
    // a freed block serves the next request of its size
    void* a = pool.get(8);
    std::memset(a, 1, 4096);
    pool.put(a);
    CHECK(pool.kept() == 4096 && g_blocks == 1);
    CHECK(pool.get(4096) == a && pool.kept() == 0);
    pool.put(a);
    pool.put(a);                       // not live: ignored
    CHECK(pool.kept() == 4096);
    // blocks of growing sizes, as a hierarchy's levels ask for: none above the limit stays
    for (size_t n = kPinnedBlock; n <= (size_t(1) << 26); n += n / 3) {
        void* p = pool.get(n);
        std::memset(p, 2, n);
        pool.put(p);
        CHECK(pool.kept() <= 4096 + kPinnedBlock);
    }
    // many at once
    std::vector<void*> many;
    for (int i = 0; i < 1000; ++i) many.push_back(pool.get(kPinnedBlock));
    for (void* p : many) pool.put(p);
    CHECK(pool.kept() <= kPinnedKept);
    pool.release();
    CHECK(pool.kept() == 0 && g_blocks == 0);
    g_full = true;
    CHECK(pool.get(1) == nullptr);
    g_full = false;
    // threads
    std::vector<std::thread> th;
    std::atomic<int> bad{0};
    for (int t = 0; t < 8; ++t)
        th.emplace_back([&, t] {
            for (int i = 0; i < 2000; ++i) {
                const size_t n = size_t(1) << (8 + (i + t) % 12);
                unsigned char* p = static_cast<unsigned char*>(pool.get(n));
                std::memset(p, t, n);
                for (size_t k = 0; k < n; k += 97)
                    if (p[k] != t) ++bad;
                pool.put(p);
            }
        });
    for (auto& x : th) x.join();
    CHECK(bad == 0 && pool.kept() <= kPinnedKept);
    pool.release();
    CHECK(g_blocks == 0);
    std::printf("ok\n");
    return 0;
}
