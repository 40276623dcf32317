// Device-side helpers shared by the HIP kernels (wave64 reductions and scans,
// the SplitMix64 generator).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace pair {

__device__ __forceinline__ int64_t wave_inclusive_scan(int64_t v) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        int64_t u = __shfl_up(v, d, 64);
        if (lane >= d) v += u;
    }
    return v;
}

__device__ __forceinline__ int wave_inclusive_scan_int(int v) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        int u = __shfl_up(v, d, 64);
        if (lane >= d) v += u;
    }
    return v;
}

// Sum over groups of G consecutive lanes (G a power of two <= 64); every lane of
// the group receives the group total.  The reduction tree is fixed, so the
// result is bitwise reproducible.
template <int G>
__device__ __forceinline__ double group_sum(double v) {
#pragma unroll
    for (int d = G / 2; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}

template <int G>
__device__ __forceinline__ int group_sum_int(int v) {
#pragma unroll
    for (int d = G / 2; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}

template <int G>
__device__ __forceinline__ double group_max(double v) {
#pragma unroll
    for (int d = G / 2; d >= 1; d >>= 1) v = fmax(v, __shfl_xor(v, d, 64));
    return v;
}

// Exclusive prefix of one tile's total over the tiles before it, in one pass over
// the data (decoupled look-back; Merrill and Garland 2016): every tile publishes
// its total and then its inclusive prefix in `status` (zero before the launch),
// value << 2 | state (0 nothing, 1 total, 2 inclusive prefix).  Tiles are numbered
// by tile_ticket, in the order in which their blocks start, so the tiles a block
// waits for are running or done, and each publishes its total before it waits:
// every wait ends.  Call with one whole wave; every lane gets the prefix.
// Values below 2^61.
__device__ __forceinline__ int64_t tile_prefix(unsigned long long* status, int64_t tile, int64_t total) {
    const int lane = threadIdx.x & 63;
    auto put = [&](unsigned long long w) {
        if (lane == 0) __hip_atomic_store(&status[tile], w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    int64_t before = 0;
    if (tile > 0) {
        put(static_cast<unsigned long long>(total) << 2 | 1ull);
        for (int64_t last = tile - 1;; last -= 64) {
            const int64_t i = last - lane;
            unsigned long long w = 2ull;         // before the first tile: prefix 0
            if (i >= 0)
                do {
                    w = __hip_atomic_load(&status[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                } while ((w & 3ull) == 0);
            const uint64_t full = __ballot((w & 3ull) == 2ull);
            const int stop = full ? __ffsll(static_cast<unsigned long long>(full)) - 1 : 63;
            int64_t v = lane <= stop ? static_cast<int64_t>(w >> 2) : 0;
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
            before += v;
            if (full) break;
        }
    }
    put(static_cast<unsigned long long>(before + total) << 2 | 2ull);
    return before;
}

// The calling block's tile number (all threads; shared storage of the caller).
__device__ __forceinline__ int64_t tile_ticket(unsigned* counter, unsigned* shared) {
    if (threadIdx.x == 0) *shared = atomicAdd(counter, 1u);
    __syncthreads();
    return *shared;
}

// Appends to a global list with one atomicAdd on `counter` per block: R rows per
// thread that lie NT apart (so that the block's accesses to them are contiguous),
// bit r of `bits` keeps row r * NT + threadIdx.x of the tile, slot[r] is its place,
// in row order.  Every thread of the NT-thread block must call it.  The order of
// entries across blocks is not fixed.
template <int NT, int R>
__device__ __forceinline__ void block_reserve_rows(unsigned bits, int* counter, int (&slot)[R]) {
    constexpr int W = NT / 64;
    static_assert(R * W <= 64, "one wave scans the counts");
    __shared__ int s_c[R * W];
    const int wid = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint64_t m = __ballot((bits >> r) & 1u);
        slot[r] = __popcll(m & below);
        if (lane == 0) s_c[r * W + wid] = __popcll(m);
    }
    __syncthreads();
    if (wid == 0) {
        const int c = lane < R * W ? s_c[lane] : 0;
        int x = c;
#pragma unroll
        for (int d = 1; d < R * W; d <<= 1) {
            const int y = __shfl_up(x, d, 64);
            if (lane >= d) x += y;
        }
        const int tot = __shfl(x, R * W - 1, 64);
        int base = 0;
        if (lane == 0 && tot > 0) base = atomicAdd(counter, tot);
        base = __shfl(base, 0, 64);
        if (lane < R * W) s_c[lane] = base + x - c;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) slot[r] += s_c[r * W + wid];
    __syncthreads();   // the next call may overwrite s_c
}

// SplitMix64 (Steele, Lea & Flood 2014): add the golden-ratio increment, then
// the variant-13 finaliser.
__device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
    uint64_t z = x + 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// 53-bit random integer of local row i on a level (PMIS measure tie-breaker).
__device__ __forceinline__ uint64_t pmis_rand(uint64_t seed, int level, int64_t i) {
    uint64_t key = (seed << 40) + (static_cast<uint64_t>(level) << 32) + static_cast<uint64_t>(i);
    return splitmix64(key) >> 11;
}

}  // namespace pair
