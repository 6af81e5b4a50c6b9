// binned.hpp -- sparse products whose gathers all come from LDS, for vectors
// too long for an XCD's L2 (shared by the UV-decomposition solver and the
// standard-ADMM baseline).
//
// out[g] = sum over the entries k of segment g of val[k] * vec[idx[k]], in
// two launches.  The vector is cut into parts of kPart values (one part fits
// a compute unit's LDS) and the segments into groups of at most kCap entries
// (a group's products fit the LDS too):
//   k_bin_mult  the entries are stored part by part, within a part group by
//               group; a workgroup stages its part and streams the part's
//               entries (8- or 4-byte value, 16-bit place in the part),
//               multiplies and writes the products group by group, so the
//               run of one (part, group) pair is contiguous on both sides
//   k_bin_sum   a workgroup reads its group's products, puts each at its
//               entry's place in LDS (16 bits), and a thread per segment (a
//               wavefront for a long one) adds them in a fixed order and goes
//               on with the update
// What bounds it: streaming, 28 bytes an entry in FP64 (8 + 2 read, 8
// written, 8 + 2 read) and 16 in FP32, against 12 (8) bytes and one random
// 64-byte L2 request an entry of the slab product.  On the 1e6 x 2e6 LP (2e7
// entries, FP64; a copy of 1 GiB runs at 5.15 TB/s here): k_bin_mult 73 us =
// 360 MB and 48 MB of staged parts at 5.6 TB/s, k_bin_sum with the update
// fused 54 us (columns) and 44 us (rows); column pass 182 -> 127 us, row
// pass 170 -> 119 us.  Flat optimum: parts of 8192 values, groups of 6656 to
// 20000 products, batches of 256 or 1024 entries, runs aligned to 32 or 64
// bytes and a second workgroup a CU are all 0-8 % slower; non-temporal
// stores of the products 14-20 % slower (they then leave the Infinity Cache
// before k_bin_sum reads them).
// The order in which a run stores its entries is not fixed, but each product
// is added at its entry's place, so results are bitwise reproducible.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "common.hpp"
#include "setup.hpp"

namespace {

constexpr int kPart = 16384;       // vector values a part (128 KiB in FP64)
constexpr int kCap = 10240;        // products a group may hold (80 KiB in FP64: two workgroups a CU)
constexpr int kBinU = 8;           // 64-entry steps of a wavefront's batch
constexpr int kBatch = 64 * kBinU;
constexpr int kMultThreads = 1024;
constexpr int kSumThreads = 512;
constexpr int kMaxParts = 1024;    // LDS counters of the set-up kernels
constexpr int kGroupSegs = 5120;   // segments a group may hold
constexpr int kLong = 64;          // entries from which a wavefront adds a segment
constexpr unsigned kFirst = 0x8000u;  // flag of a run's first entry

// A batch of k_bin_mult: the part, the run of its first entry (an index of
// `shift`) and its entries.
struct BinBatch {
    int part, run, count, pad;
};

// One direction's plan (device pointers; ptr is the matrix's own).
struct BinPlan {
    int nseg = 0, len = 0, nnz = 0, groups = 0, parts = 0, batches = 0, grid = 0;
    const int *ptr = nullptr;
    int *gseg = nullptr;              // first segment of each group (groups + 1)
    int *pend = nullptr;              // first batch after each part
    BinBatch *batch = nullptr;
    int *shift = nullptr;             // run -> place of its products less place of its entries
    unsigned short *place = nullptr;  // entry's place in its part, with kFirst
    unsigned short *pos = nullptr;    // product's entry within its group
    double *val64 = nullptr;
    void *val = nullptr;              // sweep values (val64 in FP64)
    bool on() const { return batches > 0; }
};

// ---- set-up ----

__global__ void __launch_bounds__(kWG) k_bin_longest(int nseg, const int *__restrict__ ptr, int *__restrict__ out)
{
    const int g = blockIdx.x * kWG + threadIdx.x;
    int len = g < nseg ? ptr[g + 1] - ptr[g] : 0;
    for (int off = 32; off > 0; off >>= 1) len = max(len, __shfl_xor(len, off));
    if ((threadIdx.x & 63) == 0) atomicMax(out, len);
}

// First segment of each group: the first whose entries start at or after
// g * step (so a group holds fewer than step + the longest segment).
__global__ void __launch_bounds__(kWG)
k_bin_groups(int nseg, const int *__restrict__ ptr, int groups, int step, int *__restrict__ gseg)
{
    const int g = blockIdx.x * kWG + threadIdx.x;
    if (g > groups) return;
    if (g == 0 || g == groups) {
        gseg[g] = g == 0 ? 0 : nseg;
        return;
    }
    const int64_t want = (int64_t)g * step;
    int lo = 0, hi = nseg;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (ptr[mid] >= want) hi = mid;
        else lo = mid + 1;
    }
    gseg[g] = lo;
}

// cnt[part * groups + g] = entries of group g in each part.
__global__ void __launch_bounds__(kWG)
k_bin_count(const int *__restrict__ ptr, const int *__restrict__ idx, int groups, int parts,
            const int *__restrict__ gseg, int *__restrict__ cnt)
{
    __shared__ int c[kMaxParts];
    const int g = blockIdx.x;
    for (int p = threadIdx.x; p < parts; p += kWG) c[p] = 0;
    __syncthreads();
    for (int k = ptr[gseg[g]] + threadIdx.x; k < ptr[gseg[g + 1]]; k += kWG) atomicAdd(&c[idx[k] / kPart], 1);
    __syncthreads();
    for (int p = threadIdx.x; p < parts; p += kWG) cnt[(size_t)p * groups + g] = c[p];
}

// Entries before each part (off: exclusive sums of cnt, part by part).
__global__ void __launch_bounds__(kWG)
k_bin_part_starts(int parts, int groups, const int *__restrict__ off, int *__restrict__ start)
{
    const int p = blockIdx.x * kWG + threadIdx.x;
    if (p <= parts) start[p] = off[(size_t)p * groups];
}

// Places the entries of a group: entry k of part p goes to place
// off[p * groups + g] + adj[p] + rank of the entry stream, its product to
// the group's range from ptr[gseg[g]] on, part by part.
__global__ void __launch_bounds__(kWG)
k_bin_fill(const int *__restrict__ ptr, const int *__restrict__ idx, const double *__restrict__ val, int groups,
           int parts, const int *__restrict__ gseg, const int *__restrict__ cnt, const int *__restrict__ off,
           const int *__restrict__ adj, unsigned short *__restrict__ place, double *__restrict__ val1,
           unsigned short *__restrict__ pos, int *__restrict__ dest)
{
    __shared__ int src[kMaxParts], to[kMaxParts], used[kMaxParts];
    const int g = blockIdx.x, k0 = ptr[gseg[g]], k1 = ptr[gseg[g + 1]];
    for (int p = threadIdx.x; p < parts; p += kWG) {
        src[p] = off[(size_t)p * groups + g] + adj[p];
        to[p] = cnt[(size_t)p * groups + g];
        used[p] = 0;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = k0;
        for (int p = 0; p < parts; ++p) {
            const int c = to[p];
            to[p] = t;
            t += c;
        }
    }
    __syncthreads();
    for (int p = threadIdx.x; p < parts; p += kWG) dest[(size_t)p * groups + g] = to[p];
    for (int k = k0 + threadIdx.x; k < k1; k += kWG) {
        const int j = idx[k], p = j / kPart, r = atomicAdd(&used[p], 1);
        place[src[p] + r] = (unsigned short)((j - p * kPart) | (r == 0 ? kFirst : 0u));
        val1[src[p] + r] = val[k];
        pos[to[p] + r] = (unsigned short)(k - k0);
    }
}

// Numbers a part's non-empty runs, stores each run's shift and the run and
// length of the batches that start in it.  One workgroup a part.
__global__ void __launch_bounds__(kWG)
k_bin_runs(int groups, const int *__restrict__ cnt, const int *__restrict__ off, const int *__restrict__ adj,
           const int *__restrict__ dest, const int *__restrict__ start, int *__restrict__ shift,
           BinBatch *__restrict__ batch)
{
    __shared__ int s[kWG];
    __shared__ int carry;
    const int p = blockIdx.x;
    const size_t row = (size_t)p * groups;
    const int end = start[p + 1] + adj[p];  // past the part's last entry
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int base = 0; base < groups; base += kWG) {
        const int g = base + threadIdx.x;
        const int c = g < groups ? cnt[row + g] : 0;
        s[threadIdx.x] = c > 0;
        __syncthreads();
        for (int o = 1; o < kWG; o <<= 1) {
            const int a = threadIdx.x >= o ? s[threadIdx.x - o] : 0;
            __syncthreads();
            s[threadIdx.x] += a;
            __syncthreads();
        }
        if (c > 0) {
            const int r = carry + s[threadIdx.x] - 1, a = off[row + g] + adj[p];
            shift[row + r] = dest[row + g] - a;
            for (int b = (a + kBatch - 1) / kBatch; b * kBatch < a + c; ++b)
                batch[b] = BinBatch{p, (int)(row + r), min(kBatch, end - b * kBatch), 0};
        }
        __syncthreads();
        if (threadIdx.x == kWG - 1) carry += s[kWG - 1];
        __syncthreads();
    }
}

// ---- the product ----

// Products of a range of batches (see the header comment).  Dynamic LDS:
// kPart values of the vector.  A workgroup's range is contiguous, so it
// stages a new part only where its range passes from one to the next.
template <typename T, typename TV, typename G>
__global__ void __launch_bounds__(kMultThreads)
k_bin_mult(int batches, int len, const BinBatch *__restrict__ batch, const int *__restrict__ pend,
           const unsigned short *__restrict__ place, const TV *__restrict__ val, const G *__restrict__ vec,
           const int *__restrict__ shift, T *__restrict__ Q, const int *skip)
{
    if (skip && *skip) return;
    extern __shared__ __align__(16) unsigned char bin_lds[];
    G *xs = (G *)bin_lds;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    int b = (int)((int64_t)batches * blockIdx.x / gridDim.x);
    const int b1 = (int)((int64_t)batches * (blockIdx.x + 1) / gridDim.x);
    while (b < b1) {
        const int p = batch[b].part, be = min(b1, pend[p]);
        const G *src = vec + (size_t)p * kPart;
        const int cnt = min(kPart, len - p * kPart);
        __syncthreads();  // the last part is no longer read
        uv::stage_lds<kMultThreads>(xs, src, cnt);
        __syncthreads();
        for (int q0 = b + w; q0 < be; q0 += kMultThreads / 64) {
            const int q = __builtin_amdgcn_readfirstlane(q0);
            const BinBatch B = batch[q];
            const int P = q * kBatch;
            unsigned j[kBinU];
            TV v[kBinU];
#pragma unroll
            for (int u = 0; u < kBinU; ++u) {
                const int k = u * 64 + lane, kk = P + (k < B.count ? k : B.count - 1);
                j[u] = __builtin_nontemporal_load(place + kk);
                v[u] = __builtin_nontemporal_load(val + kk);
            }
            int run = B.run, to[kBinU];
#pragma unroll
            for (int u = 0; u < kBinU; ++u) {
                const int k = u * 64 + lane;
                const bool first = k > 0 && k < B.count && (j[u] & kFirst);
                const unsigned long long mask = __ballot(first);
                const int before = __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32),
                                                             __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0));
                to[u] = P + k + shift[run + before + (first ? 1 : 0)];
                run += __popcll(mask);
            }
#pragma unroll
            for (int u = 0; u < kBinU; ++u)
                if (u * 64 + lane < B.count) Q[to[u]] = (T)v[u] * (T)xs[j[u] & (kPart - 1)];
        }
        b = be;
    }
}

// Segment sums of a group's products, handed to the epilogue: E has
// load(segment) (operands that do not depend on the sum, read while the
// products arrive) and put(segment, entries, sum).  Dynamic LDS: kCap
// products.
template <typename T, typename E>
__global__ void __launch_bounds__(kSumThreads)
k_bin_sum(const int *__restrict__ ptr, const int *__restrict__ gseg, const unsigned short *__restrict__ pos,
          const T *__restrict__ Q, E epi, const int *skip)
{
    if (skip && *skip) return;
    extern __shared__ __align__(16) unsigned char bin_lds[];
    T *ps = (T *)bin_lds;
    const int s0 = gseg[blockIdx.x], s1 = gseg[blockIdx.x + 1];
    const int k0 = ptr[s0], cnt = ptr[s1] - k0;
    constexpr int U = kCap / kSumThreads;  // all of a thread's products in flight
    for (int i = threadIdx.x; i < cnt; i += U * kSumThreads) {
        T q[U];
        unsigned o[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = i + u * kSumThreads, kk = k0 + (k < cnt ? k : cnt - 1);
            q[u] = Q[kk];
            o[u] = __builtin_nontemporal_load(pos + kk);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i + u * kSumThreads < cnt) ps[o[u]] = q[u];
    }
    const int lane = threadIdx.x & 63;
    int s = s0 + threadIdx.x, a = 0, z = 0;
    auto next = [&]() {
        a = z = 0;
        if (s < s1) {
            a = ptr[s] - k0;
            z = ptr[s + 1] - k0;
            epi.load(s);
        }
    };
    next();
    __syncthreads();
    // A thread adds entry k in sum k mod 4 of its segment, four LDS reads in
    // flight; the wavefront adds each long segment among its 64 (a thread took
    // 150 us for 5000 entries while the group waited, and the rounding error of
    // its one running sum grew with them).
    for (int sb = s0 + (int)(threadIdx.x & ~63u); sb < s1; sb += kSumThreads) {
        const bool chain = z - a <= kLong;
        T p[4] = {0, 0, 0, 0};
        if (chain)
            for (int k = a; k < z; k += 4) {
                T v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = ps[min(k + u, z - 1)];
#pragma unroll
                for (int u = 0; u < 4; ++u) p[u] = k + u < z ? p[u] + v[u] : p[u];
            }
        T acc = (p[0] + p[1]) + (p[2] + p[3]);
        for (unsigned long long left = __ballot(!chain); left; left &= left - 1) {
            const int j = __ffsll(left) - 1;
            const int aj = __builtin_amdgcn_readlane(a, j), zj = __builtin_amdgcn_readlane(z, j);
            T t = 0;
            for (int k = aj + lane; k < zj; k += 64) t += ps[k];
            t = uv::group_sum<64>(t);
            if (lane == j) acc = t;
        }
        if (s < s1) epi.put(s, z - a, acc);
        s += kSumThreads;
        next();
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) epi.once();
}

// Epilogue: the plain product.
template <typename T>
struct BinStore {
    T *__restrict__ out;
    __device__ void load(int) {}
    __device__ void put(int s, int, T sum) { out[s] = sum; }
    __device__ void once() {}
};

template <typename T, typename TV, typename G>
void bin_mult(const BinPlan &p, const TV *val, const G *vec, T *Q, const int *skip, hipStream_t st)
{
    k_bin_mult<T, TV, G><<<p.grid, kMultThreads, kPart * sizeof(G), st>>>(p.batches, p.len, p.batch, p.pend, p.place,
                                                                          val, vec, p.shift, Q, skip);
}

template <typename T, typename E>
void bin_sum(const BinPlan &p, const T *Q, E epi, const int *skip, hipStream_t st)
{
    k_bin_sum<T, E><<<p.groups, kSumThreads, kCap * sizeof(T), st>>>(p.ptr, p.gseg, p.pos, Q, epi, skip);
}

// LDS above the default 64 KiB a workgroup has to be asked for.
template <typename T, typename TV, typename G>
bool bin_mult_ready()
{
    return hipFuncSetAttribute((const void *)k_bin_mult<T, TV, G>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               kPart * sizeof(G)) == hipSuccess;
}

template <typename T, typename E>
bool bin_sum_ready()
{
    return hipFuncSetAttribute((const void *)k_bin_sum<T, E>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               kCap * sizeof(T)) == hipSuccess;
}

// Whether the binned product is the faster one for a matrix whose slab
// product would take S > 1 slabs.  Its two launches cost about 25 us before
// the first byte (staging the parts), the slab product a random L2 request
// an entry and S partials a segment.  Measured pass times, binned / slab, by
// nnz + 2 S nseg: 2.2e6 30.0 / 23.4 us, 4.5e6 36.6 / 34.2, 5.3e6 40.0 / 38.3,
// 5.9e6 41.2 / 43.6, 6.6e6 37.9 / 54.2, 9.6e6 50.9 / 70.6, 2.8e7 127 / 182
// (FP64); 2.2e6 25.9 / 20.4, 4.3e6 30.9 / 30.0, 5.6e6 29.0 / 36.9, 9.6e6
// 38.9 / 56.6 (mixed); at 6e7 entries and vectors of 15e6, whose runs are
// only 11 entries long, still 724 / 1261 and 412 / 854.
// (Not at the end of the 32-bit range, where the set-up's strides would pass it.)
inline bool bins_pay(int S, int nseg, int nnz)
{
    return (int64_t)nnz + (int64_t)2 * S * nseg >= 5600000 && nnz <= INT32_MAX - (1 << 20);
}

// A block of device scratch of a plan's set-up, given back at its end.
struct BinScratch {
    unsigned char *p = nullptr;
    size_t at = 0;
    bool reserve(size_t bytes) { return uv::dev_malloc(&p, bytes) == hipSuccess; }
    template <typename T>
    T *take(size_t count)
    {
        T *q = (T *)(p + at);
        at += (count * sizeof(T) + 255) / 256 * 256;
        return q;
    }
    ~BinScratch()
    {
        if (p) (void)hipFree(p);
    }
};

enum BinBuilt { BIN_OK = 0, BIN_NO = 1, BIN_NOMEM = 2, BIN_HIP = 3 };  // BIN_NO: the matrix does not suit the plan

// Builds the plan of a compressed matrix (nseg segments, ptr, idx, FP64
// val; vector length len).  alloc(bytes) gives device memory that lives as
// long as the plan; scratch comes from it too.  BIN_NO where a segment is
// longer than half a group or the vector has more than kMaxParts parts.
template <typename A>
BinBuilt build_bins(int nseg, int len, int nnz, const int *ptr, const int *idx, const double *val, bool fp32, A alloc,
                    hipStream_t st, BinPlan *out)
{
    BinPlan p;
    p.nseg = nseg;
    p.len = len;
    p.nnz = nnz;
    p.ptr = ptr;
    p.parts = (len + kPart - 1) / kPart;
    if (nnz < 1 || p.parts > kMaxParts) return BIN_NO;
#define UV_BIN(expr) \
    if ((expr) != hipSuccess) return BIN_HIP
    BinScratch one, two;  // what the groups need, and the cells
    const size_t most = (size_t)(nnz / (kCap / 2) + 2);  // groups before they are cut, at most
    if (!one.reserve(4 * most + 1024)) return BIN_NOMEM;
    int longest = 0, *dl = one.take<int>(1);
    UV_BIN(hipMemsetAsync(dl, 0, 4, st));
    k_bin_longest<<<blocks_for(nseg, kWG), kWG, 0, st>>>(nseg, ptr, dl);
    UV_BIN(hipMemcpyAsync(&longest, dl, 4, hipMemcpyDeviceToHost, st));
    UV_BIN(hipStreamSynchronize(st));
    if (longest > kCap / 2) return BIN_NO;
    const int step = kCap - longest + 1;
    // Groups of equal entries, cut further where that leaves many segments
    // (empty ones above all) to one workgroup: 6e5 x 1e6 with 1e7 entries, row
    // pass 69 us, and 1165 us with 9e5 empty rows after them (slabs 102); cut,
    // 77 us.
    const int rough = (int)(((int64_t)nnz + step - 1) / step);
    int *droug = one.take<int>((size_t)rough + 1);
    k_bin_groups<<<blocks_for(rough + 1, kWG), kWG, 0, st>>>(nseg, ptr, rough, step, droug);
    std::vector<int> hg((size_t)rough + 1), gs(1, 0);
    UV_BIN(hipMemcpyAsync(hg.data(), droug, 4 * hg.size(), hipMemcpyDeviceToHost, st));
    UV_BIN(hipStreamSynchronize(st));
    for (int g = 0; g < rough; ++g) {
        const int s0 = hg[g], s1 = hg[g + 1], cuts = (s1 - s0 + kGroupSegs - 1) / kGroupSegs;
        for (int q = 1; q <= cuts; ++q) gs.push_back(s0 + (int)((int64_t)(s1 - s0) * q / cuts));
    }
    p.groups = (int)gs.size() - 1;
    const int64_t cells = (int64_t)p.groups * p.parts;
    if (cells >= (1 << 28)) return BIN_NO;
    p.gseg = (int *)alloc(4 * ((size_t)p.groups + 1));
    if (!two.reserve(13 * (size_t)cells + 8 * ((size_t)p.parts + 1) + 8192)) return BIN_NOMEM;
    int *cnt = two.take<int>(cells), *off = two.take<int>(cells + 1), *dest = two.take<int>(cells);
    int *bsum = two.take<int>((size_t)blocks_for(cells, 4 * kWG));
    int *start = two.take<int>((size_t)p.parts + 1), *adj = two.take<int>((size_t)p.parts);
    p.pend = (int *)alloc(4 * (size_t)p.parts);
    p.shift = (int *)alloc(4 * cells);
    if (!p.gseg || !p.pend || !p.shift) return BIN_NOMEM;
    UV_BIN(hipMemcpyAsync(p.gseg, gs.data(), 4 * gs.size(), hipMemcpyHostToDevice, st));
    k_bin_count<<<p.groups, kWG, 0, st>>>(ptr, idx, p.groups, p.parts, p.gseg, cnt);
    if (!scan_exclusive((int)cells, cnt, off, bsum, st)) return BIN_HIP;
    k_bin_part_starts<<<blocks_for(p.parts + 1, kWG), kWG, 0, st>>>(p.parts, p.groups, off, start);
    std::vector<int> hs((size_t)p.parts + 1), ha(p.parts), he(p.parts);
    UV_BIN(hipMemcpyAsync(hs.data(), start, 4 * hs.size(), hipMemcpyDeviceToHost, st));
    UV_BIN(hipStreamSynchronize(st));
    int64_t nb = 0;  // a part starts on a batch of its own
    for (int q = 0; q < p.parts; ++q) {
        const int64_t a = nb * kBatch - hs[q];
        if (a > INT32_MAX - (int64_t)nnz) return BIN_NO;
        ha[q] = (int)a;
        nb += (hs[q + 1] - hs[q] + kBatch - 1) / kBatch;
        he[q] = (int)nb;
    }
    const size_t slots = (size_t)nb * kBatch;
    if (slots >= (size_t)INT32_MAX) return BIN_NO;
    p.batches = (int)nb;
    p.batch = (BinBatch *)alloc(sizeof(BinBatch) * (size_t)nb);
    p.place = (unsigned short *)alloc(2 * slots);
    p.pos = (unsigned short *)alloc(2 * (size_t)nnz);
    p.val64 = (double *)alloc(8 * slots);
    p.val = fp32 ? alloc(4 * slots) : (void *)p.val64;
    if (!p.batch || !p.place || !p.pos || !p.val64 || !p.val) return BIN_NOMEM;
    UV_BIN(hipMemcpyAsync(adj, ha.data(), 4 * ha.size(), hipMemcpyHostToDevice, st));
    UV_BIN(hipMemcpyAsync(p.pend, he.data(), 4 * he.size(), hipMemcpyHostToDevice, st));
    k_bin_fill<<<p.groups, kWG, 0, st>>>(ptr, idx, val, p.groups, p.parts, p.gseg, cnt, off, adj, p.place, p.val64,
                                         p.pos, dest);
    k_bin_runs<<<p.parts, kWG, 0, st>>>(p.groups, cnt, off, adj, dest, start, p.shift, p.batch);
    if (fp32) k_narrow<float><<<blocks_for((int64_t)slots, kWG), kWG, 0, st>>>((int64_t)slots, p.val64, (float *)p.val);
    UV_BIN(hipGetLastError());
    UV_BIN(hipStreamSynchronize(st));  // the host copies end here
    int dev = 0, cus = 0;
    UV_BIN(hipGetDevice(&dev));
    UV_BIN(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    p.grid = std::max(1, std::min(cus * (fp32 ? 2 : 1), p.batches));
#undef UV_BIN
    *out = p;
    return BIN_OK;
}

}  // namespace
