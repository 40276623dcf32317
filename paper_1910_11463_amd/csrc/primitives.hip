// Device primitives: caching allocator, exclusive scan, member-id fill.
#include <algorithm>
#include <map>
#include <mutex>
#include <unordered_map>

#include "amg.h"
#include "kernels_common.h"
#include "pinned_pool.h"

namespace pair {

// ---------------------------------------------------------------- allocator
namespace {
struct Block {
    size_t size;
    hipStream_t stream;
};
void* pinned_malloc(size_t bytes) {
    void* p = nullptr;
    if (hipHostMalloc(&p, bytes, hipHostMallocCoherent | hipHostMallocPortable) == hipSuccess) return p;
    (void)hipGetLastError();
    return nullptr;
}
struct Pool {
    std::mutex mu;
    std::multimap<std::pair<hipStream_t, size_t>, void*> free_blocks;   // (stream, size) -> ptr
    std::unordered_map<void*, Block> live;
    size_t in_use = 0;
    PinnedPool pinned{pinned_malloc, [](void* p) { (void)hipHostFree(p); }};
};
Pool& pool() {
    static Pool* p = new Pool();   // intentionally leaked: outlives static destructors
    return *p;
}
thread_local hipStream_t t_pool_stream = nullptr;
// blocks of retired streams, usable by all
hipStream_t const kShared = reinterpret_cast<hipStream_t>(~uintptr_t(0));
size_t round_size(size_t b) {
    size_t r = 256;
    while (r < b) r <<= 1;
    return r;
}
}  // namespace

PoolStream::PoolStream(hipStream_t s) : prev(t_pool_stream) { t_pool_stream = s; }
PoolStream::~PoolStream() { t_pool_stream = prev; }

void* pool_alloc(size_t bytes) {
    Pool& P = pool();
    const size_t sz = round_size(bytes);
    const hipStream_t st = t_pool_stream;
    {
        std::lock_guard<std::mutex> g(P.mu);
        for (hipStream_t key : {st, kShared}) {
            auto it = P.free_blocks.find({key, sz});
            if (it != P.free_blocks.end()) {
                void* p = it->second;
                P.free_blocks.erase(it);
                P.live[p] = Block{sz, st};
                P.in_use += sz;
                return p;
            }
        }
    }
    void* p = nullptr;
    hipError_t e = hipMalloc(&p, sz);
    if (e != hipSuccess) {
        // release cached blocks and retry once
        pool_release_all();
        (void)hipGetLastError();
        e = hipMalloc(&p, sz);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            throw Error(E_OOM, "device allocation of " + std::to_string(sz) + " bytes failed");
        }
    }
    std::lock_guard<std::mutex> g(P.mu);
    P.live[p] = Block{sz, st};
    P.in_use += sz;
    return p;
}

void pool_free(void* p) {
    if (!p) return;
    Pool& P = pool();
    std::lock_guard<std::mutex> g(P.mu);
    auto it = P.live.find(p);
    if (it == P.live.end()) return;
    P.free_blocks.emplace(std::make_pair(it->second.stream, it->second.size), p);
    P.in_use -= it->second.size;
    P.live.erase(it);
}

void pool_retire_stream(hipStream_t s) {
    Pool& P = pool();
    std::lock_guard<std::mutex> g(P.mu);
    for (auto it = P.free_blocks.begin(); it != P.free_blocks.end();) {
        if (it->first.first == s) {
            P.free_blocks.emplace(std::make_pair(kShared, it->first.second), it->second);
            it = P.free_blocks.erase(it);
        } else {
            ++it;
        }
    }
    for (auto& kv : P.live)
        if (kv.second.stream == s) kv.second.stream = kShared;
}

void pool_release_all() {
    Pool& P = pool();
    std::lock_guard<std::mutex> g(P.mu);
    for (auto& kv : P.free_blocks) (void)hipFree(kv.second);
    P.free_blocks.clear();
    P.pinned.release();
}

void* pinned_alloc(size_t bytes) {
    void* p = pool().pinned.get(bytes);
    if (!p) throw Error(E_OOM, "pinned host allocation of " + std::to_string(bytes) + " bytes failed");
    return p;
}

void pinned_free(void* p) { pool().pinned.put(p); }

size_t pool_bytes_in_use() { return pool().in_use; }

// ---------------------------------------------------------------- scan
namespace {
constexpr int kScanBlock = 256;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanBlock * kScanItems;

// One pass: a tile's values through LDS, its prefix by look-back.  status:
// ntiles words and the ticket, zero on entry.  The last tile writes the total to
// out[n] and to the host page.  Bound by its loads and stores (16 B per value);
// a pass for the tiles' sums, one for their offsets and a wait per level before:
// 14 M values 3 launches and 2 waits, now one each.
// A single tile needs no status.  Value(in[i]) is what is summed.
struct ScanValue {
    __device__ int64_t operator()(int64_t v) const { return v; }
};
struct ScanEqual {
    int8_t to;
    __device__ int64_t operator()(int8_t v) const { return v == to ? 1 : 0; }
};

template <class T, class Value>
__global__ void __launch_bounds__(kScanBlock)
k_scan(const T* __restrict__ in, Value value, int64_t* __restrict__ out, int64_t n, int64_t ntiles,
       unsigned long long* __restrict__ status, int64_t* __restrict__ host_total) {
    __shared__ int64_t sh[kScanTile];
    __shared__ int64_t wsum[kScanBlock / 64];
    __shared__ int64_t s_before;
    __shared__ unsigned s_tile;
    const int64_t tile = ntiles > 1 ? tile_ticket(reinterpret_cast<unsigned*>(status + ntiles), &s_tile) : 0;
    const int64_t base = tile * kScanTile;
    for (int i = threadIdx.x; i < kScanTile; i += kScanBlock) {
        const int64_t g = base + i;
        sh[i] = g < n ? value(in[g]) : 0;
    }
    __syncthreads();
    int64_t v[kScanItems];
    int64_t run = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        v[k] = run;
        run += sh[threadIdx.x * kScanItems + k];
    }
    // exclusive scan of the per-thread totals across the block
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int64_t incl = wave_inclusive_scan(run);
    if (lane == 63) wsum[wid] = incl;
    __syncthreads();
    int64_t woff = 0, total = 0;
    for (int w = 0; w < kScanBlock / 64; ++w) {
        if (w < wid) woff += wsum[w];
        total += wsum[w];
    }
    if (wid == 0) {
        const int64_t before = ntiles > 1 ? tile_prefix(status, tile, total) : 0;
        if (lane == 0) {
            s_before = before;
            if (tile == ntiles - 1) {
                out[n] = before + total;
                *host_total = before + total;
            }
        }
    }
    __syncthreads();
    const int64_t excl = s_before + woff + incl - run;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) sh[threadIdx.x * kScanItems + k] = v[k] + excl;
    __syncthreads();
    for (int i = threadIdx.x; i < kScanTile; i += kScanBlock) {
        const int64_t g = base + i;
        if (g < n) out[g] = sh[i];
    }
}

template <class T, class Value>
int64_t scan(const T* in, Value value, int64_t* out, int64_t n, hipStream_t s) {
    if (n <= 0) {
        int64_t z = 0;
        PAIR_HIP(hipMemcpyAsync(out, &z, sizeof(int64_t), hipMemcpyHostToDevice, s));
        PAIR_HIP(hipStreamSynchronize(s));
        return 0;
    }
    const int64_t ntiles = (n + kScanTile - 1) / kScanTile;
    DBuf<unsigned long long> status(ntiles > 1 ? ntiles + 1 : 0);
    HBuf<int64_t> total(1);
    if (ntiles > 1) PAIR_HIP(hipMemsetAsync(status.p, 0, status.bytes(), s));
    hipLaunchKernelGGL((k_scan<T, Value>), dim3(static_cast<unsigned>(ntiles)), dim3(kScanBlock), 0, s, in, value,
                       out, n, ntiles, status.p, total.p);
    PAIR_LAUNCH_CHECK();
    PAIR_HIP(hipStreamSynchronize(s));
    return *total.p;
}
}  // namespace

int64_t exclusive_scan(const int64_t* in, int64_t* out, int64_t n, hipStream_t s) {
    return scan(in, ScanValue{}, out, n, s);
}

int64_t exclusive_count(const int8_t* in, int8_t value, int64_t* out, int64_t n, hipStream_t s) {
    return scan(in, ScanEqual{value}, out, n, s);
}

// ---------------------------------------------------------------- segments
namespace {
// Member of every row, all members in one launch (blockIdx.y: the member).
__global__ void __launch_bounds__(256)
k_fill_seg(uint16_t* __restrict__ seg, const int64_t* __restrict__ off, const int64_t* __restrict__ cnt) {
    const int b = blockIdx.y;
    const int64_t o = off[b], n = cnt[b];
    if (o < 0) return;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * 256)
        seg[o + i] = static_cast<uint16_t>(b);
}
}  // namespace

void fill_segments(uint16_t* seg, int members, int64_t most, const int64_t* off_d, const int64_t* cnt_d,
                   hipStream_t s) {
    const unsigned gx = static_cast<unsigned>(std::min<int64_t>((most + 2047) / 2048, 4096));
    hipLaunchKernelGGL(k_fill_seg, dim3(std::max(1u, gx), static_cast<unsigned>(members)), dim3(256), 0, s, seg,
                       off_d, cnt_d);
    PAIR_LAUNCH_CHECK();
}

int choose_lpr(double avg) {
    int l = 1;
    while (l < 64 && l * 1.5 < avg) l <<= 1;
    return l;
}

}  // namespace pair
