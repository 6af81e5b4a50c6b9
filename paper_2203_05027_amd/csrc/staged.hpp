// staged.hpp -- sparse products with long segments over a vector that a few
// compute units' LDS can hold (up to 8 parts), for matrices large enough to
// pay for staging it on every compute unit.
//
// The entries are the slab-major copy of the slab product, slab s holding
// the entries whose index falls in part s, with a 16-bit place in the part
// for each entry.  A workgroup (one a compute unit) stages its part and
// walks a contiguous range of the part's segments, L lanes a segment; with
// one part the row or column update follows in the same launch, otherwise
// each part leaves one partial a segment.
// What bounds it: the entry stream (10 bytes an entry in FP64, 6 in FP32) and
// the staging, with one workgroup's loads in flight a compute unit; the
// lane-group kernels it replaces gather from L1 and L2 and are bound by those
// requests.  2e4 x 1e5 at 1e7 entries, FP64 (mixed): column pass, one part,
// 82.9 -> 26.7 us (63.9 -> 20.3), row pass, eight parts, 72.2 -> 33.8 us
// (64.5 -> 25.3); with cones of size 4 the column pass was 323 us (a lane a
// column).  Four entries in flight a lane instead of eight are 4-25 %
// slower, and so is one chunk at a time; non-temporal entry loads 15-60 %
// slower (neighbouring segments share their first and last lines).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <utility>
#include <vector>

#include "common.hpp"
#include "setup.hpp"

namespace {

constexpr int kStagedThreads = 1024;
constexpr int kStagedBytes = 160000;  // LDS for the staged part
constexpr int kStagedParts = 8;
constexpr int kStagedE = 8;           // entries in flight per lane

// A workgroup's share: segments s0..s1-1 of a part.
struct StagedShare {
    int part, s0, s1, pad;
};

// One direction's plan (device pointers).
struct StagedPlan {
    int nseg = 0, len = 0, S = 0, width = 0, L = 4, grid = 0;
    const int *off = nullptr;        // S * nseg + 1 offsets (the matrix's own with one part)
    StagedShare *share = nullptr;    // a workgroup's share (grid of them)
    unsigned short *place = nullptr;
    const double *val64 = nullptr;
    const void *val = nullptr;
    bool on() const { return S > 0; }
};

// Shares of equal work: a segment's entries and `each` more for the segment
// itself (a lane group takes a whole chunk of L * kStagedE entries for the
// shortest one).  In: part, s0 = share i of s1 of the part's; out: its segments.
// Shares of the entries alone gave a run of short segments to one workgroup:
// 1e4 x 3e4 with 3e6 entries, column pass 14 us, and 333 us with 1e4 slack
// columns after them, 1075 us with 1.3e5 empty ones (lane groups 30 us); now 17
// and 21 us.
__global__ void __launch_bounds__(kWG)
k_staged_split(int grid, int nseg, int each, const int *__restrict__ off, StagedShare *__restrict__ share)
{
    const int t = blockIdx.x * kWG + threadIdx.x;
    if (t >= grid) return;
    StagedShare &w = share[t];
    const int *o = off + (size_t)w.part * nseg;
    const int i = w.s0, per = w.s1;
    const int64_t all = (int64_t)o[nseg] - o[0] + (int64_t)nseg * each;
    auto first = [&](int q) {
        int lo = 0, hi = nseg;
        if (q == 0) hi = 0;
        else if (q == per) lo = nseg;
        const int64_t want = o[0] + all * q / per;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (o[mid] + (int64_t)mid * each >= want) hi = mid;
            else lo = mid + 1;
        }
        return lo;
    };
    w.s0 = first(i);
    w.s1 = first(i + 1);
}

// The workgroups of the parts, as many for each as it has of the work (at
// least one), the parts' taken in turn; `entries` of each part.  The entries
// may lie in few of the parts: 7e4 x 3e4 with 3e6 entries in the first seventh
// of the rows, column pass 34 us with as many workgroups for each of the four
// parts (lane groups 28 us), 21 us so.
inline std::vector<StagedShare> staged_shares(int cus, int S, int nseg, int each, const std::vector<int64_t> &entries)
{
    std::vector<int> per(S, 1);
    std::vector<double> work(S);
    for (int p = 0; p < S; ++p) work[p] = (double)entries[p] + (double)nseg * each;
    for (int left = cus - S; left > 0; --left) {  // the next one where the shares are largest
        int at = 0;
        for (int p = 1; p < S; ++p)
            if (work[p] / per[p] > work[at] / per[at]) at = p;
        per[at] += 1;
    }
    std::vector<std::pair<double, StagedShare>> w;
    for (int p = 0; p < S; ++p)
        for (int i = 0; i < per[p]; ++i) w.push_back({(i + 0.5) / per[p], StagedShare{p, i, per[p], 0}});
    std::stable_sort(w.begin(), w.end(), [](const auto &a, const auto &b) { return a.first < b.first; });
    std::vector<StagedShare> out;
    for (const auto &e : w) out.push_back(e.second);
    return out;
}

// Place of each entry in its part (k_slab_count's parts).
__global__ void __launch_bounds__(kWG)
k_staged_place(int nnz, const int *__restrict__ idx, int S, int w, unsigned short *__restrict__ place)
{
    const int k = blockIdx.x * kWG + threadIdx.x;
    if (k < nnz) place[k] = (unsigned short)(idx[k] - min(idx[k] / w, S - 1) * w);
}

// The product (see the header comment): the epilogue's put(segment, entries,
// sum) is called for part 0 of a one-part plan, else out takes the partials.
template <typename T, typename TV, typename G, int L, typename E>
__global__ void __launch_bounds__(kStagedThreads)
k_staged(int nseg, int len, int width, const int *__restrict__ off, const StagedShare *__restrict__ share,
         const unsigned short *__restrict__ place, const TV *__restrict__ val, const G *__restrict__ vec, E epi,
         const int *skip)
{
    if (skip && *skip) return;
    extern __shared__ __align__(16) unsigned char staged_lds[];
    G *xs = (G *)staged_lds;
    const StagedShare own = share[blockIdx.x];
    const int p = own.part, s1 = own.s1;
    const int *o = off + (size_t)p * nseg;
    const int lane = threadIdx.x & (L - 1);
    int s = own.s0 + threadIdx.x / L;
    const int cnt = min(width, len - p * width);
    constexpr int EL = L * kStagedE, step = kStagedThreads / L;
    // A lane group's chunks in order: the next chunk's entries (of this
    // segment or the first of the group's next one) are read while this
    // one's are multiplied, and a segment's bounds one segment ahead.
    unsigned j[kStagedE], jn[kStagedE];
    TV v[kStagedE], vn[kStagedE];
    auto fetch = [&](int b, int e, unsigned (&jj)[kStagedE], TV (&vv)[kStagedE]) {
#pragma unroll
        for (int q = 0; q < kStagedE; ++q) {
            const int k = b + lane + q * L, kk = max(k < e ? k : e - 1, 0);
            jj[q] = place[kk];
            vv[q] = val[kk];
        }
    };
    int base = 0, end = 0, nb = 0, ne = 0, total = 0;
    if (s < s1) {
        base = o[s];
        end = o[s + 1];
        total = end - base;
        fetch(base, end, j, v);
        if (s + step < s1) {
            nb = o[s + step];
            ne = o[s + step + 1];
        }
    }
    uv::stage_lds<kStagedThreads>(xs, vec + (size_t)p * width, cnt);
    __syncthreads();
    T acc = 0;
    while (s < s1) {
        const bool last = base + EL >= end;
        if (!last) fetch(base + EL, end, jn, vn);
        else if (s + step < s1) fetch(nb, ne, jn, vn);
        if (last && lane == 0) epi.load(s);
#pragma unroll
        for (int q = 0; q < kStagedE; ++q)
            if (base + lane + q * L < end) acc += (T)v[q] * (T)xs[j[q]];
        if (last) {
            acc = uv::group_sum<L>(acc);
            if (lane == 0) epi.put(p * nseg + s, total, acc);
            acc = 0;
            s += step;
            base = nb;
            end = ne;
            total = end - base;
            if (s + step < s1) {
                nb = o[s + step];
                ne = o[s + step + 1];
            }
        } else {
            base += EL;
        }
#pragma unroll
        for (int q = 0; q < kStagedE; ++q) {
            j[q] = jn[q];
            v[q] = vn[q];
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) epi.once();
}

template <typename T, typename TV, typename G, typename E>
void staged(const StagedPlan &p, const TV *val, const G *vec, E epi, const int *skip, hipStream_t st)
{
    const unsigned grid = (unsigned)p.grid;
    const size_t lds = (size_t)p.width * sizeof(G);
#define UV_STAGED_ARGS p.nseg, p.len, p.width, p.off, p.share, p.place, val, vec, epi, skip
    switch (p.L) {
    case 4: k_staged<T, TV, G, 4, E><<<grid, kStagedThreads, lds, st>>>(UV_STAGED_ARGS); break;
    case 8: k_staged<T, TV, G, 8, E><<<grid, kStagedThreads, lds, st>>>(UV_STAGED_ARGS); break;
    case 16: k_staged<T, TV, G, 16, E><<<grid, kStagedThreads, lds, st>>>(UV_STAGED_ARGS); break;
    case 32: k_staged<T, TV, G, 32, E><<<grid, kStagedThreads, lds, st>>>(UV_STAGED_ARGS); break;
    default: k_staged<T, TV, G, 64, E><<<grid, kStagedThreads, lds, st>>>(UV_STAGED_ARGS); break;
    }
#undef UV_STAGED_ARGS
}

template <typename T, typename TV, typename G, typename E>
bool staged_ready()
{
    const auto a = hipFuncAttributeMaxDynamicSharedMemorySize;
    return hipFuncSetAttribute((const void *)k_staged<T, TV, G, 4, E>, a, kStagedBytes) == hipSuccess &&
           hipFuncSetAttribute((const void *)k_staged<T, TV, G, 8, E>, a, kStagedBytes) == hipSuccess &&
           hipFuncSetAttribute((const void *)k_staged<T, TV, G, 16, E>, a, kStagedBytes) == hipSuccess &&
           hipFuncSetAttribute((const void *)k_staged<T, TV, G, 32, E>, a, kStagedBytes) == hipSuccess &&
           hipFuncSetAttribute((const void *)k_staged<T, TV, G, 64, E>, a, kStagedBytes) == hipSuccess;
}

// Parts the staged product would take (a power of two), 0 where it does not
// apply: `elem` is the gathered type's size (the largest of the sweep's and
// the check's).
inline int staged_parts(int len, int elem)
{
    for (int S = 1; S <= kStagedParts; S *= 2)
        if ((int64_t)(((int64_t)len + S - 1) / S + 3) / 4 * 4 * elem <= kStagedBytes) return S;
    return 0;
}

// Part width: 16-byte multiples, so that every part starts aligned.
inline int staged_width(int len, int S) { return ((len + S - 1) / S + 3) / 4 * 4; }

// Whether the staged product is the faster one where the slab rule takes one
// slab.  Below about 9e5 entries staging costs more than the gathers it
// saves (1.8e5: 8.0 / 8.5 us for the column / row pass against 6.7 / 6.4 us;
// 4e5: 13.1 / 14.8 against 8.1 / 7.8; 1.0e6: 9.9 / 9.7 against 12.2 / 11.8),
// and below about ten entries a segment and part the lane groups idle
// (1.0e6, five a segment: 13.3 against 11.5; 2.0e6, twelve: 14.8 against
// 20.2).
inline bool staged_pays(int S, int nseg, int nnz)
{
    return S > 0 && nnz >= 900000 && nnz <= INT32_MAX - (1 << 20) && (int64_t)nnz >= (int64_t)10 * S * nseg;
}

}  // namespace
