// The small levels of a V-cycle in one launch: one workgroup takes a member
// (direction) from the first level on which it has at most kTailRows rows, there and
// further down at most kTailEntries entries, down to its coarsest level and up again.
//
// What bounds it: a small level's half-sweep, residual, restriction or
// interpolation costs 3-4 us as a launch of its own whatever its size, about six
// of them per level and cycle.  Members do not couple, so block barriers can take
// the launches' place.  Inside the workgroup the instructions per entry count
// (the level kernels' layout, lanes along a row with clamped places and a
// reduction, took 40 us for two levels of 346 and 53 rows, as long as the fifteen
// launches it replaced), so the setup lays these levels out for it: F rows before
// C rows, each sorted by length, in slices of 64 rows, a slice's entries column by
// column (value and 16-bit column, padded to the slice's longest row).  A lane
// takes a row, every load of a wave is contiguous, and vectors, 1/a_ii and the
// interpolation stay in LDS.
// LDS gathers bound it then (27000 entries: 11000 cycles for a pass).  8^3 S2, 8
// directions of 1357, 346 and 53 rows: 37 us for what 20 launches took (a V-cycle
// 100 -> 85 us); from 400 rows on, 22 us.
//
// A row is summed in the order of its entries, which differs from the level
// kernels' order; whether a member's level is in the tail depends on that
// member's rows and entries alone, so a member rounds the same alone and in a batch.
#include <algorithm>
#include <type_traits>
#include <vector>

#include "amg.h"
#include "kernels_common.h"

namespace pair {
namespace {

// Threads of a member's workgroup (its results do not depend on them).  As long as
// the members have a CU or half of one each, 1024; with more of them the chip holds
// as many at once as their waves and LDS allow, so a member's workgroup has a wave
// per slice or two of its first level.  us per cycle without tail / 1024 for all / so:
// 1000 members of 150 rows 139 / 134 / 99; 16000 1427 / 1493 / 716; 1000 of 600
// 377 / 262 / 216; solve of 64000 of 40 rows 23.9 / 34.4 / 13.0 ms.
constexpr int kTailThreads = 1024;
constexpr int kTailFew = 512;
int tail_threads(size_t members, int64_t rows) {
    return members <= kTailFew || rows > 256 ? kTailThreads : rows > 64 ? 256 : 64;
}
constexpr int kPlanThreads = 256;
constexpr int kTailPad = 4;               // slice widths are multiples of this
constexpr uint16_t kNoRow = 0xffff;

// positions and slices of a matrix of n rows, at most (two classes, each padded
// to whole slices)
int64_t max_positions(int64_t n) { return (n + 63) / 64 * 64 + 64; }

}  // namespace

// One matrix (rows of A or of R of one member and level) to lay out.
struct TailTask {
    const int64_t* rowptr;        // of the member's first row
    const int32_t* col;
    const double* val;
    const float* valf;            // FP32 copies where the coarse levels use them
    const int8_t* cf;             // classes of the rows (null: one class)
    const double* dinv;           // A only: 1/a_ii, its FP32 copy, interpolation
    const float* dinvf;
    const int32_t* p;
    int n, col0, p0;              // rows, first column of the member, first row of the next level
    int perm, slice, rows;        // places in the packed arrays
};

// One level of a member in the tail.
struct TailLevel {
    int n, nc;                    // rows, rows of the next level (0: the coarsest)
    int perm_a, slice_a, posf, pos_a;   // A: places, positions of the F rows, of all rows
    int perm_r, slice_r, pos_r;
    int rows;                     // place of 1/a_ii and the interpolation
    const double* inv;            // the coarsest level's inverse
    const double* b;              // right-hand side and solution (first level only)
    double* x;
};

namespace {

// Pointers read from memory have no known address space; they are global.
template <class T>
using Global = const __attribute__((address_space(1))) T*;

// Order of a task's rows and widths of its slices; count[task] = {positions of
// the F rows, positions, slots (64 entries each)}.
__global__ void __launch_bounds__(kPlanThreads)
k_tail_plan(const TailTask* __restrict__ tasks, uint16_t* __restrict__ perm, int2* __restrict__ slices,
            int* __restrict__ count) {
    __shared__ int s_hist[2][256];
    __shared__ int s_width[kTailRows / 64 + 2];
    const TailTask T = tasks[blockIdx.x];
    const auto rp = (Global<int64_t>)T.rowptr;
    const auto cf = (Global<int8_t>)T.cf;
    const int t = threadIdx.x;
    for (int i = t; i < 512; i += kPlanThreads) s_hist[i >> 8][i & 255] = 0;
    for (int i = t; i < kTailRows / 64 + 2; i += kPlanThreads) s_width[i] = 0;
    __syncthreads();
    auto key = [&](int i, int& cls) {
        cls = T.cf && cf[i] > 0 ? 1 : 0;
        const int64_t len = rp[i + 1] - rp[i];
        return static_cast<int>(255 - (len < 255 ? len : 255));      // longest first
    };
    for (int i = t; i < T.n; i += kPlanThreads) {
        int c;
        const int k = key(i, c);
        atomicAdd(&s_hist[c][k], 1);
    }
    __syncthreads();
    int h[2];
    for (int c = 0; c < 2; ++c) h[c] = s_hist[c][t];
    for (int d = 1; d < 256; d *= 2) {        // running sums of both classes
        int v[2];
        for (int c = 0; c < 2; ++c) v[c] = t >= d ? s_hist[c][t - d] : 0;
        __syncthreads();
        for (int c = 0; c < 2; ++c) s_hist[c][t] += v[c];
        __syncthreads();
    }
    const int nf = s_hist[0][255], first_c = (nf + 63) & ~63;
    const int npos = (first_c + s_hist[1][255] + 63) & ~63;
    __syncthreads();
    s_hist[0][t] -= h[0];
    s_hist[1][t] += first_c - h[1];
    __syncthreads();
    for (int i = t; i < npos; i += kPlanThreads) perm[T.perm + i] = kNoRow;
    __syncthreads();
    for (int i = t; i < T.n; i += kPlanThreads) {
        int c;
        const int k = key(i, c);
        const int pos = atomicAdd(&s_hist[c][k], 1);
        perm[T.perm + pos] = static_cast<uint16_t>(i);
        atomicMax(&s_width[pos >> 6], static_cast<int>(rp[i + 1] - rp[i]));
    }
    __syncthreads();
    if (t == 0) {
        int o = 0;
        for (int s = 0; s < npos / 64; ++s) {
            const int w = (s_width[s] + kTailPad - 1) / kTailPad * kTailPad;
            slices[T.slice + s] = make_int2(o, w);
            o += w;
        }
        count[3 * blockIdx.x] = first_c;
        count[3 * blockIdx.x + 1] = npos;
        count[3 * blockIdx.x + 2] = o;
    }
}

// The entries in their places, a block per slice (blockIdx.y), a lane per row and
// every fourth column to a wave; a slice's padding adds 0 times the row's own first
// column.  Slices become absolute.
__global__ void __launch_bounds__(kPlanThreads)
k_tail_fill(const TailTask* __restrict__ tasks, const int* __restrict__ count, const int* __restrict__ entry,
            const uint16_t* __restrict__ perm, int2* __restrict__ slices, double* __restrict__ val,
            uint16_t* __restrict__ col, double* __restrict__ dinv, int16_t* __restrict__ interp) {
    if (entry[blockIdx.x] < 0) return;      // its level stays with the level kernels
    const TailTask T = tasks[blockIdx.x];
    const auto rp = (Global<int64_t>)T.rowptr;
    const auto tc = (Global<int32_t>)T.col;
    const auto tv = (Global<double>)T.val;
    const auto tf = (Global<float>)T.valf;
    const int npos = count[3 * blockIdx.x + 1];
    if (static_cast<int>(blockIdx.y) < npos / 64) {
        const int pos = static_cast<int>(blockIdx.y) * 64 + (threadIdx.x & 63);
        int2 sl = slices[T.slice + blockIdx.y];
        __syncthreads();
        sl.x += entry[blockIdx.x];
        if (threadIdx.x == 0) slices[T.slice + blockIdx.y].x = sl.x;
        const int row = perm[T.perm + pos];
        int64_t e = 0;
        int len = 0;
        if (row != kNoRow) {
            e = rp[row];
            len = static_cast<int>(rp[row + 1] - e);
        }
        const int64_t base = static_cast<int64_t>(sl.x) * 64 + (pos & 63);
        const uint16_t first = len > 0 ? static_cast<uint16_t>(tc[e] - T.col0) : 0;
#pragma unroll 4
        for (int u = threadIdx.x >> 6; u < sl.y; u += kPlanThreads / 64) {
            double v = 0.0;
            uint16_t c = first;
            if (u < len) {
                v = T.valf ? static_cast<double>(tf[e + u]) : tv[e + u];
                c = static_cast<uint16_t>(tc[e + u] - T.col0);
            }
            val[base + static_cast<int64_t>(u) * 64] = v;
            col[base + static_cast<int64_t>(u) * 64] = c;
        }
    }
    if (T.dinv)
        for (int i = static_cast<int>(blockIdx.y) * kPlanThreads + threadIdx.x; i < T.n;
             i += static_cast<int>(gridDim.y) * kPlanThreads) {
            dinv[T.rows + i] = T.dinvf ? static_cast<double>(((Global<float>)T.dinvf)[i]) : ((Global<double>)T.dinv)[i];
            const int32_t p = ((Global<int32_t>)T.p)[i];
            interp[T.rows + i] = p >= 0 ? static_cast<int16_t>(p - T.p0) : int16_t(-1);
        }
}

// f(row, sum of the row times x) for the rows at positions [from, to) (multiples
// of 64), a lane per row.
template <int NT, class F>
__device__ __forceinline__ void tail_rows(int from, int to, const uint16_t* perm, const int2* slices,
                                          const double* __restrict__ val, const uint16_t* __restrict__ col,
                                          const double* x, F&& f) {
    const int lane = threadIdx.x & 63;
    for (int s = from / 64 + static_cast<int>(threadIdx.x >> 6); s < to / 64; s += NT / 64) {
        const int2 sl = slices[s];
        const int w = __builtin_amdgcn_readfirstlane(sl.y);
        const int64_t base = static_cast<int64_t>(__builtin_amdgcn_readfirstlane(sl.x)) * 64;
        const double* v = val + base + lane;
        const uint16_t* c = col + base + lane;
        double sum = 0.0;
        auto add = [&](auto count, int u) {       // `count` entries, their loads together
            constexpr int U = decltype(count)::value;
            double a[U];
            int k[U];
#pragma unroll
            for (int j = 0; j < U; ++j) {
                a[j] = v[(u + j) * 64];
                k[j] = c[(u + j) * 64];
            }
#pragma unroll
            for (int j = 0; j < U; ++j) sum += a[j] * x[k[j]];
        };
        int u = 0;
        for (; u + 16 <= w; u += 16) add(std::integral_constant<int, 16>(), u);
        if (u + 8 <= w) {
            add(std::integral_constant<int, 8>(), u);
            u += 8;
        }
        if (u < w) add(std::integral_constant<int, kTailPad>(), u);
        const int row = perm[s * 64 + lane];
        if (row != kNoRow) f(row, sum);
    }
}

template <int NT>
__global__ void __launch_bounds__(NT)
k_tail(const int4* __restrict__ members, const TailLevel* __restrict__ levels, const uint8_t* __restrict__ active,
       const uint16_t* __restrict__ perm, const int2* __restrict__ slices, const double* __restrict__ val,
       const uint16_t* __restrict__ col, const double* __restrict__ dinv, const int16_t* __restrict__ interp,
       double omega, uint32_t pre, int npre, uint32_t post, int npost) {
    extern __shared__ double lds[];
    __shared__ TailLevel lev[kTailLevels];
    __shared__ int s_row[kTailLevels], s_perm[kTailLevels], s_slice[kTailLevels];   // places in LDS
    __shared__ int s_tot[3];
    const int tid = threadIdx.x;
    const int4 mb = members[blockIdx.x];    // first level's entry, levels, member
    if (!active[mb.z]) return;
    if (tid < mb.y) lev[tid] = levels[mb.x + tid];
    __syncthreads();
    if (tid == 0) {
        int r = 0, p = 0, s = 0;
        for (int l = 0; l < mb.y; ++l) {
            s_row[l] = r;
            s_perm[l] = p;
            s_slice[l] = s;
            r += lev[l].n;
            if (lev[l].nc > 0) {
                p += lev[l].pos_a + lev[l].pos_r;
                s += (lev[l].pos_a + lev[l].pos_r) / 64;
            }
        }
        s_tot[0] = r;
        s_tot[1] = s;
        s_tot[2] = p;
    }
    __syncthreads();
    const int rows = s_tot[0], last = mb.y - 1;
    // LDS: x, b, 1/a_ii of every level, two work vectors; slices; row orders; interpolation
    double* const xs = lds;
    double* const bs = xs + rows;
    double* const ds = bs + rows;
    double* const work = ds + rows;
    int2* const sl = reinterpret_cast<int2*>(work + 2 * lev[0].n);
    uint16_t* const pm = reinterpret_cast<uint16_t*>(sl + s_tot[1]);
    int16_t* const ip = reinterpret_cast<int16_t*>(pm + s_tot[2]);
    for (int l = 0; l < last; ++l) {
        const int n = lev[l].n, pa = lev[l].pos_a, pr = lev[l].pos_r;
        for (int i = tid; i < n; i += NT) {
            ds[s_row[l] + i] = dinv[lev[l].rows + i];
            ip[s_row[l] + i] = interp[lev[l].rows + i];
        }
        for (int i = tid; i < pa; i += NT) pm[s_perm[l] + i] = perm[lev[l].perm_a + i];
        for (int i = tid; i < pr; i += NT) pm[s_perm[l] + pa + i] = perm[lev[l].perm_r + i];
        for (int i = tid; i < pa / 64; i += NT) sl[s_slice[l] + i] = slices[lev[l].slice_a + i];
        for (int i = tid; i < pr / 64; i += NT) sl[s_slice[l] + pa / 64 + i] = slices[lev[l].slice_r + i];
    }
    {
        const auto b = (Global<double>)lev[0].b;
        for (int i = tid; i < lev[0].n; i += NT) bs[i] = b[i];
    }
    __syncthreads();
    // a half-sweep of level l from cur into oth: the class's rows, the others kept
    auto half_sweep = [&](int l, bool c, const double* cur, double* oth) {
        const double* b = bs + s_row[l];
        const double* d = ds + s_row[l];
        const int pf = lev[l].posf, pa = lev[l].pos_a;
        const uint16_t* q = pm + s_perm[l];
        for (int i = (c ? 0 : pf) + tid; i < (c ? pf : pa); i += NT)
            if (q[i] != kNoRow) oth[q[i]] = cur[q[i]];
        tail_rows<NT>(c ? pf : 0, c ? pa : pf, q, sl + s_slice[l], val, col, cur,
                  [&](int i, double s) { oth[i] = cur[i] + omega * (b[i] - s) * d[i]; });
    };
    // down
    for (int l = 0; l < last; ++l) {
        const int n = lev[l].n, pf = lev[l].posf, pa = lev[l].pos_a;
        const uint16_t* q = pm + s_perm[l];
        double* const x = xs + s_row[l];
        double* const b = bs + s_row[l];
        double* const r = work + lev[0].n;
        // an even number of exchanges ends in x, an odd one starts from work
        double *cur = (npre & 1) ? work : x, *oth = (npre & 1) ? x : work;
        if (npre == 0) {
            for (int i = tid; i < n; i += NT) x[i] = 0.0;
            __syncthreads();
        }
        for (int k = 0; k < npre; ++k) {
            const bool c = (pre >> k & 1u) != 0;
            if (k == 0) {                   // from x = 0
                const double* d = ds + s_row[l];
                for (int i = tid; i < pa; i += NT)
                    if (q[i] != kNoRow) oth[q[i]] = (i >= pf) == c ? omega * b[q[i]] * d[q[i]] : 0.0;
            } else {
                half_sweep(l, c, cur, oth);
            }
            double* sw = cur;
            cur = oth;
            oth = sw;
            __syncthreads();
        }
        tail_rows<NT>(0, pa, q, sl + s_slice[l], val, col, x, [&](int i, double s) { r[i] = b[i] - s; });
        __syncthreads();
        double* const bc = b + n;
        tail_rows<NT>(0, lev[l].pos_r, q + pa, sl + s_slice[l] + pa / 64, val, col, r,
                  [&](int i, double s) { bc[i] = s; });
        __syncthreads();
    }
    // the coarsest level: x = A^{-1} b (inverse stored column-major)
    {
        const int n = lev[last].n, o = s_row[last];
        const auto Inv = (Global<double>)lev[last].inv;
        const double* b = bs + o;
        for (int r = tid; r < n; r += NT) {
            double s = 0.0;
            int c = 0;
            for (; c + 16 <= n; c += 16) {
                double a[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) a[u] = Inv[static_cast<int64_t>(c + u) * n + r];
#pragma unroll
                for (int u = 0; u < 16; ++u) s += a[u] * b[c + u];
            }
            for (; c < n; ++c) s += Inv[static_cast<int64_t>(c) * n + r] * b[c];
            xs[o + r] = s;
        }
        __syncthreads();
    }
    // up
    for (int l = last - 1; l >= 0; --l) {
        const int n = lev[l].n;
        double* const x = xs + s_row[l];
        const int16_t* p = ip + s_row[l];
        for (int i = tid; i < n; i += NT) {
            const int c = p[i];
            if (c >= 0) x[i] += x[n + c];
        }
        __syncthreads();
        double *cur = x, *oth = work;
        for (int k = 0; k < npost; ++k) {
            half_sweep(l, (post >> k & 1u) != 0, cur, oth);
            double* sw = cur;
            cur = oth;
            oth = sw;
            __syncthreads();
        }
        if (cur != x) {
            for (int i = tid; i < n; i += NT) x[i] = cur[i];
            __syncthreads();
        }
    }
    auto out = (__attribute__((address_space(1))) double*)lev[0].x;
    for (int i = tid; i < lev[0].n; i += NT) out[i] = xs[i];
}

// LDS of a member with these rows per tail level, at most.
size_t tail_lds(const std::vector<int64_t>& n) {
    size_t rows = 0, pos = 0;
    for (size_t l = 0; l < n.size(); ++l) {
        rows += static_cast<size_t>(n[l]);
        if (l + 1 < n.size()) pos += static_cast<size_t>(max_positions(n[l]) + (n[l + 1] + 63) / 64 * 64);
    }
    return (3 * rows + 2 * static_cast<size_t>(n[0])) * sizeof(double) + pos / 64 * sizeof(int2) +
           (pos + rows + 4) * sizeof(uint16_t);
}

}  // namespace

void Hierarchy::build_tail() {
    tail_on_ = false;
    tail_launches_.clear();
    const int nl = static_cast<int>(levels_.size());
    std::vector<int> first(B_, -1);
    size_t lds = 0;
    for (int b = 0; b < B_; ++b) {
        const int last = nlev_[b] - 1;
        for (int l = last; l >= 1; --l) {
            std::vector<int64_t> n;
            for (int k = l; k <= last; ++k) n.push_back(levels_[k].cnt[b]);
            const size_t need = tail_lds(n);
            if (n[0] > kTailRows || need > kTailLds) break;
            first[b] = l;
            lds = std::max(lds, need);
        }
    }
    level_on_.assign(nl, 1);
    for (int l = 0; l < nl; ++l) levels_[l].coarse_launch = static_cast<int>(levels_[l].coarse_members.size());
    if (lds == 0) return;

    // place of every member's inverse on its coarsest level
    std::vector<int64_t> inv_off(B_, 0);
    for (const Level& L : levels_) {
        int64_t o = 0;
        for (int b : L.coarse_members) {
            inv_off[b] = o;
            o += L.cnt[b] * L.cnt[b];
        }
    }
    std::vector<TailTask> tasks;
    std::vector<TailLevel> lev;
    std::vector<int4> members(B_, make_int4(0, 0, 0, 0));
    int64_t nperm = 0, nslice = 0, nrows = 0;
    auto place = [&](TailTask& T, int64_t n, bool classes) {
        const int64_t pos = classes ? max_positions(n) : (n + 63) / 64 * 64;
        T.n = static_cast<int>(n);
        T.perm = static_cast<int>(nperm);
        T.slice = static_cast<int>(nslice);
        nperm += pos;
        nslice += pos / 64;
    };
    for (int b = 0; b < B_; ++b) {
        if (first[b] < 0) continue;
        members[b] = make_int4(static_cast<int>(lev.size()), nlev_[b] - first[b], b, 0);
        for (int l = first[b]; l < nlev_[b]; ++l) {
            Level& L = levels_[l];
            TailLevel q{};
            q.n = static_cast<int>(L.cnt[b]);
            q.b = L.b.p + L.off[b];
            q.x = L.x.p + L.off[b];
            if (l + 1 < nlev_[b]) {
                const Level& C = levels_[l + 1];
                const bool f32 = prm_.coarse_fp32;
                q.nc = static_cast<int>(C.cnt[b]);
                q.rows = static_cast<int>(nrows);
                TailTask A{};
                A.rowptr = L.A.rowptr.p + L.off[b];
                A.col = L.A.col.p;
                A.val = L.A.val.p;
                A.valf = f32 ? L.valf.p : nullptr;
                A.cf = L.cf.p + L.off[b];
                A.dinv = L.dinv.p + L.off[b];
                A.dinvf = f32 ? L.dinvf.p + L.off[b] : nullptr;
                A.p = L.p.p + L.off[b];
                A.col0 = static_cast<int>(L.off[b]);
                A.p0 = static_cast<int>(C.off[b]);
                A.rows = q.rows;
                place(A, q.n, true);
                q.perm_a = A.perm;
                q.slice_a = A.slice;
                tasks.push_back(A);
                TailTask Rt{};
                Rt.rowptr = L.R.rowptr.p + C.off[b];
                Rt.col = L.R.col.p;
                Rt.val = L.R.val.p;
                Rt.valf = f32 ? L.rvalf.p : nullptr;
                Rt.col0 = static_cast<int>(L.off[b]);
                place(Rt, q.nc, false);
                q.perm_r = Rt.perm;
                q.slice_r = Rt.slice;
                tasks.push_back(Rt);
                nrows += q.n;
            } else {
                q.inv = L.coarse_inv.p + inv_off[b];
            }
            lev.push_back(q);
        }
    }
    const int nt = static_cast<int>(tasks.size());
    if (nperm >= (int64_t(1) << 31)) return;       // place numbers are 32-bit
    std::vector<int> cnt(3 * static_cast<size_t>(nt), 0), entry(nt, -1);
    tail_perm_.alloc(std::max<int64_t>(nperm, 1));
    tail_slice_.alloc(std::max<int64_t>(nslice, 1));
    tail_dinv_.alloc(std::max<int64_t>(nrows, 1));
    tail_p_.alloc(std::max<int64_t>(nrows, 1));
    DBuf<TailTask> tasks_d(std::max(nt, 1));
    DBuf<int> cnt_d(4 * std::max(nt, 1));
    int64_t slots = 0;
    if (nt > 0) {
        h2d(tasks_d.p, tasks.data(), nt, s_);
        hipLaunchKernelGGL(k_tail_plan, dim3(nt), dim3(kPlanThreads), 0, s_, tasks_d.p, tail_perm_.p, tail_slice_.p,
                           cnt_d.p);
        PAIR_LAUNCH_CHECK();
        read_back(cnt.data(), cnt_d.p, cnt.size(), s_);
    }
    // a member's levels from its coarsest up to the first whose A or R has too many
    // entries; tasks are A and R of its levels in order
    std::vector<size_t> need(B_, 0);
    int task = 0;
    for (int b = 0; b < B_; ++b) {
        if (first[b] < 0) continue;
        const int last = nlev_[b] - 1, skip_to = task + 2 * (last - first[b]);
        int l = last, k = skip_to;
        while (l > first[b] && std::max(cnt[3 * (k - 2) + 2], cnt[3 * (k - 1) + 2]) <= kTailEntries / 64) {
            --l;
            k -= 2;
        }
        members[b].x += l - first[b];
        members[b].y = last - l + 1;
        first[b] = l;
        for (; k < skip_to; ++k) {
            entry[k] = static_cast<int>(slots);
            slots += cnt[3 * k + 2];
            if (slots >= (int64_t(1) << 31)) return;
        }
        task = skip_to;
        std::vector<int64_t> n;
        for (; l <= last; ++l) n.push_back(levels_[l].cnt[b]);
        need[b] = tail_lds(n);
    }
    // the level kernels' members: those whose tail starts further down
    level_on_.assign(nl, 0);
    for (int b = 0; b < B_; ++b)
        for (int l = 0; l + 1 < nlev_[b]; ++l)
            if (first[b] < 0 || l < first[b]) level_on_[l] = 1;
    tail_val_.alloc(std::max<int64_t>(64 * slots, 1));
    tail_col_.alloc(std::max<int64_t>(64 * slots, 1));
    if (nt > 0) {
        h2d(cnt_d.p + 3 * nt, entry.data(), nt, s_);
        hipLaunchKernelGGL(k_tail_fill, dim3(nt, static_cast<unsigned>(max_positions(kTailRows) / 64)),
                           dim3(kPlanThreads), 0, s_, tasks_d.p, cnt_d.p, cnt_d.p + 3 * nt, tail_perm_.p,
                           tail_slice_.p, tail_val_.p, tail_col_.p, tail_dinv_.p, tail_p_.p);
        PAIR_LAUNCH_CHECK();
    }
    int t = 0;
    for (TailLevel& q : lev)
        if (q.nc > 0) {
            q.posf = cnt[3 * t];
            q.pos_a = cnt[3 * t + 1];
            q.pos_r = cnt[3 * (t + 1) + 1];
            t += 2;
        }
    tail_lev_.alloc(lev.size());
    h2d(tail_lev_.p, lev.data(), lev.size(), s_);
    // the launches: members by the size of their workgroups
    std::vector<int4> order;
    const size_t in_tail = B_ - std::count(first.begin(), first.end(), -1);
    for (int nt : {kTailThreads, 256, 64}) {
        TailLaunch g{static_cast<int>(order.size()), 0, nt, 0};
        for (int b = 0; b < B_; ++b)
            if (first[b] >= 0 && tail_threads(in_tail, levels_[first[b]].cnt[b]) == nt) {
                order.push_back(members[b]);
                g.lds = std::max(g.lds, need[b]);
                ++g.count;
            }
        if (g.count > 0) tail_launches_.push_back(g);
    }
    tail_mem_.alloc(order.size());
    h2d(tail_mem_.p, order.data(), order.size(), s_);
    // the level kernels and coarse solves leave the tail's members out
    std::vector<std::vector<int>> mem(nl);
    std::vector<std::vector<int64_t>> moff(nl), mn(nl), ioff(nl);
    for (int l = 0; l < nl; ++l) {
        Level& L = levels_[l];
        for (int b : L.coarse_members)
            if (first[b] < 0) {
                mem[l].push_back(b);
                moff[l].push_back(L.off[b]);
                mn[l].push_back(L.cnt[b]);
                ioff[l].push_back(inv_off[b]);
            }
        L.coarse_launch = static_cast<int>(mem[l].size());
        bool relax = false;
        for (int b = 0; b < B_; ++b)
            if (first[b] >= 0 && l >= first[b] && L.relax_h[b]) {
                L.relax_h[b] = 0;
                relax = true;
            }
        if (relax) h2d(L.relax.p, L.relax_h.data(), B_, s_);
        if (!mem[l].empty() && mem[l].size() != L.coarse_members.size()) {
            h2d(L.coarse_member_d.p, mem[l].data(), mem[l].size(), s_);
            h2d(L.coarse_off_d.p, moff[l].data(), mem[l].size(), s_);
            h2d(L.coarse_n_d.p, mn[l].data(), mem[l].size(), s_);
            h2d(L.coarse_inv_off_d.p, ioff[l].data(), mem[l].size(), s_);
        }
    }
    for (const void* k : {reinterpret_cast<const void*>(&k_tail<64>), reinterpret_cast<const void*>(&k_tail<256>),
                          reinterpret_cast<const void*>(&k_tail<kTailThreads>)})
        PAIR_HIP(hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(kTailLds)));
    PAIR_HIP(hipStreamSynchronize(s_));         // the host arrays go
    tail_on_ = true;
}

void Hierarchy::launch_tail() {
    auto bits = [](const std::string& s) {
        uint32_t w = 0;
        for (size_t k = 0; k < s.size(); ++k)
            if (s[k] == 'C') w |= 1u << k;
        return w;
    };
    const std::string& pre = prm_.relax_pre_coarse;
    const std::string& post = prm_.relax_post_coarse;
    for (const TailLaunch& g : tail_launches_) {
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(g.count)), dim3(g.threads), g.lds, s_,
                               tail_mem_.p + g.at, tail_lev_.p, sv_.active, tail_perm_.p, tail_slice_.p, tail_val_.p,
                               tail_col_.p, tail_dinv_.p, tail_p_.p, prm_.omega, bits(pre),
                               static_cast<int>(pre.size()), bits(post), static_cast<int>(post.size()));
        };
        if (g.threads == 64) launch(k_tail<64>);
        else if (g.threads == 256) launch(k_tail<256>);
        else launch(k_tail<kTailThreads>);
    }
    PAIR_LAUNCH_CHECK();
}

}  // namespace pair
