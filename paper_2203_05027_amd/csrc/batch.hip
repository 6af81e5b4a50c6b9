// batch.hip -- many independent problems (orthant cone) solved together by
// one persistent launch.
//
// The instances are packed as one block-diagonal matrix with global row and
// column numbers, so the setup (CSC copy, F_U) is the single-problem setup
// run once.  A workgroup takes the next instance from a queue (instances
// ordered by decreasing nonzero count, so the long ones start first), stages
// its x and u in LDS (the two gathered vectors of the sweep), and runs the
// reduced-form iteration of Algorithm 1 on it -- column pass (A'u, x-step,
// projection, delta update), barrier, row pass (A x, lambda update),
// barrier -- for up to `budget` iterations, checking the FP64 residuals every
// check_every iterations.  A finished instance (converged, max_iter or
// numeric failure) is masked out of later launches.
//
// Within an instance rows and columns are renumbered by falling entry count
// (row r of the device is row rmap[r] of the caller), so that the 64 segments
// of a slice are about equally long; b, c and starts are permuted on the way
// in, solutions on the way out.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <functional>
#include <memory>
#include <new>
#include <numeric>
#include <queue>
#include <thread>
#include <vector>

#include "../../include/uvadmm.h"
#include "common.hpp"
#include "setup.hpp"

namespace {

constexpr int kMaxThreads = 1024;
constexpr int kLdsMax = 160 * 1024 - 1024;  // LDS of one gfx950 CU less the kernel's static LDS
constexpr int kLdsFree = 160 * 1024 - 1040; // what a launch is really left with

struct BInst {
    int m, n;
    int row_off, col_off;  // first global row / column of the instance
    int Lr, Lc;            // lanes per row / per column, 0: its sliced copy
    int status;
    int ch_off;            // first 64-column slice of the instance (-1: it has none)
    int rh_off;            // first 64-row slice (likewise)
    long long iter, check_iter;
    double r_prim, r_dual, r_gap, kkt, pobj, dobj, res_ax_b;
    double bnorm2, cnorm2;
};

template <typename T>
__device__ __forceinline__ T group_sum_rt(T v, int L)
{
    return uv::lane_sum<T>(v, L);
}

// Sum over the workgroup (blockDim.x a multiple of 64), deterministic;
// result in thread 0.
template <int K>
__device__ __forceinline__ void block_sum_rt(double (&v)[K])
{
    __shared__ double s[K][kMaxThreads / 64];
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = uv::group_sum<64>(v[k]);
    const int w = threadIdx.x / 64, lane = threadIdx.x % 64, nw = blockDim.x / 64;
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < K; ++k) s[k][w] = v[k];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            double t = 0.0;
            for (int i = 0; i < nw; ++i) t += s[k][i];
            v[k] = t;
        }
    }
}

// Instance-local row and column numbers fit 16 bits: x and u of an
// instance must fit in LDS, so m + n < 40,704 in either precision.
typedef unsigned short lidx_t;

// sum over the entries k = beg + lane, beg + lane + L, ... < end of
// val[k] * vs[idx[k]] (idx instance-local): U entries per lane have their
// index and value loads in flight together (the entries are added in the
// same order as one at a time, so the result does not depend on U).
template <int U, typename T, typename TV, typename TS>
__device__ __forceinline__ T seg_sum(int beg, int end, int lane, int L, const lidx_t *__restrict__ idx,
                                     const TV *__restrict__ val, const TS *vs)
{
    T acc = 0;
    for (int k0 = beg + lane; k0 < end; k0 += L * U) {
        int j[U];
        TV v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = k0 + u * L;
            j[u] = 0;
            v[u] = (TV)0;
            if (k < end) {
                j[u] = idx[k];
                v[u] = val[k];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (k0 + u * L < end) acc += (T)v[u] * (T)vs[j[u]];
    }
    return acc;
}

// The same over two vectors at once (the residual check's A z and A x): one
// stream of the entries for both sums.
template <int U, typename TS1, typename TS2>
__device__ __forceinline__ void seg_sum2(int beg, int end, int lane, int L, const lidx_t *__restrict__ idx,
                                         const double *__restrict__ val, const TS1 *vs1, const TS2 *vs2,
                                         double &s1, double &s2)
{
    double a1 = 0.0, a2 = 0.0;
    for (int k0 = beg + lane; k0 < end; k0 += L * U) {
        int j[U];
        double v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = k0 + u * L;
            j[u] = 0;
            v[u] = 0.0;
            if (k < end) {
                j[u] = idx[k];
                v[u] = val[k];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (k0 + u * L < end) {
                a1 += v[u] * (double)vs1[j[u]];
                a2 += v[u] * (double)vs2[j[u]];
            }
    }
    s1 = a1;
    s2 = a2;
}

// Sliced copies (0 lanes): the segments of
// an instance are cut into slices of 64, a lane each; entry t of the slice's
// lane l is stored at s0 + 128 (t / 2) + 2 l + t % 2 (s0 the slice's first
// slot), so a wavefront reads two entries a lane with one 4-byte load of their
// 16-bit numbers and one 8- or 16-byte load of their values.  A slice is as
// wide as its longest segment (rounded up to two); the slots past a segment's
// end hold the value 0 and the number `pad` (the gathered vector's length:
// the sweep's vectors in LDS have a zero there).  A lane adds its column's
// entries in order, and its row's even and odd ones apart: the sums of one lane
// walking the column and of two lanes walking the row.
struct Slices {
    const int *ptr;               // first slot of every slice, all instances
    const unsigned *idx;          // pairs of numbers
    const void *val;              // pairs of sweep values
    const double *val64;          // pairs of FP64 values
};

constexpr int kPairs = 4;  // pairs in flight per lane

template <typename T>
struct Two {
    typedef T type __attribute__((ext_vector_type(2)));
};

// One pass over an instance's slices by wavefronts, the next four pairs (of
// this slice or the wavefront's next one) and the next slice's operands in
// flight while four are multiplied.  Op: load(segment) reads what the update
// needs besides the sum, put(segment, sum) makes it.
// What bounds it: instructions (a wavefront's takes four cycles of its SIMD):
// lanes walking their segments spent dozens an entry on bounds, clamps and
// 64-bit addresses, here an entry costs half of two loads, two to unpack and
// scale its number, an LDS read and a multiply-add.  An iteration of a 5000 x
// 10000 LP with 6e4 entries alone, mixed (FP64), checks included: 44 (52) ->
// 21 (28) us; streaming the entries 64 wide through LDS instead measured 46
// (56) us.
// PAIR: the even and the odd entries are added apart.
template <bool PAIR, typename T, typename Op>
__device__ __forceinline__ void sell_pass(int wv, int nwv, int lane, int nseg, const int *__restrict__ sp,
                                          const unsigned *__restrict__ idx,
                                          const typename Two<T>::type *__restrict__ val, const T *vs, Op op)
{
    const int nch = (nseg + 63) >> 6;
    int h = wv;
    if (h >= nch) return;
    unsigned j[kPairs], jn[kPairs];
    typename Two<T>::type v[kPairs], vn[kPairs];
    int base = sp[h] >> 1, np = (sp[h + 1] >> 1) - base;  // in pairs, 64 lanes each
    np >>= 6;
    op.load(min(h * 64 + lane, nseg - 1));
#pragma unroll
    for (int q = 0; q < kPairs; ++q) {
        const int o = base + (q << 6) + lane;
        j[q] = idx[o];
        v[q] = val[o];
    }
    for (;;) {
        const int hn = h + nwv, hh = min(hn, nch - 1);
        const int nbase = sp[hh] >> 1, nnp = ((sp[hh + 1] >> 1) - nbase) >> 6;
        Op nop = op;
        nop.load(min(hh * 64 + lane, nseg - 1));
        T acc = 0, odd = 0;
        for (int p = 0;; p += kPairs) {
            const bool more = p + kPairs < np;
            const int from = more ? base + ((p + kPairs) << 6) : nbase;
#pragma unroll
            for (int q = 0; q < kPairs; ++q) {
                const int o = from + (q << 6) + lane;
                jn[q] = idx[o];
                vn[q] = val[o];
            }
#pragma unroll
            for (int q = 0; q < kPairs; ++q)
                if (p + q < np) {
                    acc += v[q].x * vs[j[q] & 0xffffu];
                    T &a = PAIR ? odd : acc;
                    a += v[q].y * vs[j[q] >> 16];
                }
#pragma unroll
            for (int q = 0; q < kPairs; ++q) {
                j[q] = jn[q];
                v[q] = vn[q];
            }
            if (!more) break;
        }
        if (h * 64 + lane < nseg) op.put(h * 64 + lane, PAIR ? acc + odd : acc);
        if (hn >= nch) return;
        h = hn;
        op = nop;
        base = nbase;
        np = nnp;
    }
}

// FP64 sums of one slice's segments over one or two vectors (a check's
// products of columns, V = 1, and rows, V = 2), lane l reading only its cnt
// entries, in the order of sell_pass.
template <int V, typename S>
__device__ __forceinline__ void sell_check(int s0, int cnt, int w, int lane, const unsigned *__restrict__ idx,
                                           const double *__restrict__ val64, const S *v1, const S *v2, double &q1,
                                           double &q2)
{
    double a1 = 0.0, a2 = 0.0, b1 = 0.0, b2 = 0.0;
#pragma unroll 4
    for (int t = 0; t < w; t += 2) {
        const int o = ((s0 + 64 * t) >> 1) + lane;
        const unsigned j = idx[o];
        const typename Two<double>::type v = ((const typename Two<double>::type *)val64)[o];
        if (t < cnt) {
            a1 += v.x * (double)v1[j & 0xffffu];
            if (V == 2) a2 += v.x * (double)v2[j & 0xffffu];
        }
        if (t + 1 < cnt) {
            if (V == 2) {
                b1 += v.y * (double)v1[j >> 16];
                b2 += v.y * (double)v2[j >> 16];
            } else {
                a1 += v.y * (double)v1[j >> 16];
            }
        }
    }
    q1 = a1 + b1;
    q2 = a2 + b2;
}

// The updates of a sliced sweep pass; pointers are the instance's own.
template <typename T>
struct SellCol {
    T *xs, *zi;
    const T *ci;
    double *__restrict__ delta;
    const lidx_t *__restrict__ cnt;
    double mu, inv_mu;
    double d;
    T zj, cj;
    int k;
    __device__ __forceinline__ void load(int j)
    {
        d = delta[j];
        zj = zi[j];
        cj = ci[j];
        k = cnt[j];
    }
    __device__ __forceinline__ void put(int j, T atu)
    {
        const T dm = (T)(d * inv_mu);
        const T p = (T)k * xs[j] + atu;
        const T xn = (p + zj + dm - cj * (T)inv_mu) / (T)(1 + k);
        const T v = xn - dm;
        const T zn = v > (T)0 ? v : (T)0;
        xs[j] = xn;
        zi[j] = zn;
        delta[j] = d + mu * ((double)zn - (double)xn);
    }
};

template <typename T>
struct SellRow {
    T *us;
    const T *__restrict__ fu, *__restrict__ b;
    double *__restrict__ lam;
    double mu, inv_mu;
    double l0;
    T fi, bi;
    __device__ __forceinline__ void load(int i)
    {
        fi = fu[i];
        bi = b[i];
        l0 = lam[i];
    }
    __device__ __forceinline__ void put(int i, T q)
    {
        const T e = fi * (bi - q);
        const double li = l0 - mu * (double)e;
        lam[i] = li;
        us[i] = (T)((double)e - li * inv_mu);
    }
};

// Fills a sliced copy from the compressed segments (rows or columns), one
// workgroup per instance.
__global__ void __launch_bounds__(256)
k_sell_fill(const BInst *__restrict__ inst, int rows, const int *__restrict__ ptr, const int *__restrict__ idx,
            const double *__restrict__ val, const int *__restrict__ sptr, lidx_t *__restrict__ sidx,
            double *__restrict__ sval)
{
    const BInst &I = inst[blockIdx.x];
    const int nseg = rows ? I.m : I.n, off = rows ? I.row_off : I.col_off, sub = rows ? I.col_off : I.row_off;
    const int pad = rows ? I.n : I.m, h0 = rows ? I.rh_off : I.ch_off;
    if (h0 < 0) return;
    const int nch = (nseg + 63) >> 6;
    for (int p = threadIdx.x; p < nch * 64; p += 256) {
        const int h = p >> 6, l = p & 63;
        const int s0 = sptr[h0 + h], w = (sptr[h0 + h + 1] - s0) >> 6;
        const int beg = p < nseg ? ptr[off + p] : 0, len = p < nseg ? ptr[off + p + 1] - beg : 0;
        for (int t = 0; t < w; ++t) {
            const int k = s0 + 128 * (t >> 1) + 2 * l + (t & 1);
            sidx[k] = t < len ? (lidx_t)(idx[beg + t] - sub) : (lidx_t)pad;
            sval[k] = t < len ? val[beg + t] : 0.0;
        }
    }
}

// Entries of each column.
__global__ void __launch_bounds__(256) k_col_entries(int n, const int *__restrict__ cp, lidx_t *__restrict__ cnt)
{
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j < n) cnt[j] = (lidx_t)(cp[j + 1] - cp[j]);
}

// One instance's vectors in the caller's numbering as FP64, straight into
// (pinned host) memory: x, z, delta (n each), lambda (m).
template <typename T>
__global__ void __launch_bounds__(256)
k_batch_out(int c0, int n, int r0, int m, const T *__restrict__ x, const T *__restrict__ z,
            const double *__restrict__ delta, const double *__restrict__ lam, const int *__restrict__ cmap,
            const int *__restrict__ rmap, double *__restrict__ out)
{
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t < n) {
        const int j = cmap[c0 + t];
        out[j] = (double)x[c0 + t];
        out[n + j] = (double)z[c0 + t];
        out[2 * n + j] = delta[c0 + t];
    } else if (t < n + m) {
        out[3 * n + rmap[r0 + t - n]] = lam[r0 + t - n];
    }
}

// Instance-local copies of the global row (CSC) and column (CSR) numbers,
// one workgroup per instance: its entries are contiguous in both forms.
__global__ void __launch_bounds__(256)
k_local_idx(const BInst *__restrict__ inst, const int *__restrict__ rp, const int *__restrict__ ci,
            const int *__restrict__ cp, const int *__restrict__ ri, lidx_t *__restrict__ cl, lidx_t *__restrict__ rl)
{
    const BInst &I = inst[blockIdx.x];
    for (int k = rp[I.row_off] + threadIdx.x; k < rp[I.row_off + I.m]; k += 256) cl[k] = (lidx_t)(ci[k] - I.col_off);
    for (int k = cp[I.col_off] + threadIdx.x; k < cp[I.col_off + I.n]; k += 256) rl[k] = (lidx_t)(ri[k] - I.row_off);
}

// ||b_i||^2, ||c_i||^2 per instance (one workgroup each).
__global__ void __launch_bounds__(256)
k_batch_norms(BInst *inst, const double *__restrict__ b64, const double *__restrict__ c64)
{
    BInst *I = inst + blockIdx.x;
    double v[2] = {0.0, 0.0};
    for (int i = threadIdx.x; i < I->m; i += 256) v[0] += b64[I->row_off + i] * b64[I->row_off + i];
    for (int j = threadIdx.x; j < I->n; j += 256) v[1] += c64[I->col_off + j] * c64[I->col_off + j];
    block_sum_rt<2>(v);
    if (threadIdx.x == 0) {
        I->bnorm2 = v[0];
        I->cnorm2 = v[1];
    }
}

__global__ void k_batch_reset(int *queue) { *queue = 0; }

// One instance's start from (pinned host) memory in the device's numbering, laid
// out as k_batch_out's vectors: x, z, delta, lambda where `have` has bit 0, 1, 2, 3
// and zeros elsewhere, and u = -lambda/mu (the start mapping).
template <typename T>
__global__ void __launch_bounds__(256)
k_batch_in(int c0, int n, int r0, int m, int have, const double *__restrict__ in, T *__restrict__ x, T *__restrict__ z,
           double *__restrict__ delta, double *__restrict__ lam, T *__restrict__ u, double inv_mu)
{
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t < n) {
        x[c0 + t] = have & 1 ? (T)in[t] : (T)0;
        z[c0 + t] = have & 2 ? (T)in[n + t] : (T)0;
        delta[c0 + t] = have & 4 ? in[2 * n + t] : 0.0;
    } else if (t < n + m) {
        const double l = have & 8 ? in[2 * n + t] : 0.0;  // 3 n + (t - n)
        lam[r0 + t - n] = l;
        u[r0 + t - n] = (T)(-l * inv_mu);
    }
}

template <typename T, bool ZC>
__global__ void __launch_bounds__(kMaxThreads)
k_batch(BInst *__restrict__ inst, const int *__restrict__ order, int nq, int *__restrict__ queue,
        const int *__restrict__ budget_p, const int *__restrict__ rp, const lidx_t *__restrict__ cl,
        const T *__restrict__ va, const double *__restrict__ va64, const int *__restrict__ cp,
        const lidx_t *__restrict__ rl, const T *__restrict__ vc, const double *__restrict__ vc64,
        const T *__restrict__ b, const double *__restrict__ b64, const T *__restrict__ fu,
        const T *__restrict__ c, const double *__restrict__ c64, T *__restrict__ x, T *__restrict__ z,
        T *__restrict__ u, double *__restrict__ lam, double *__restrict__ delta, double mu, double inv_mu,
        double eps, int check_every, long long max_iter, Slices srow, Slices scol,
        const lidx_t *__restrict__ ccnt, int sliced, int gated)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    T *xs = reinterpret_cast<T *>(lds_raw);
    __shared__ int s_q, s_stop, s_skip;
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int budget = *budget_p;
    for (;;) {
        if (tid == 0) s_q = atomicAdd(queue, 1);
        __syncthreads();
        const int q = s_q;
        __syncthreads();  // every thread has read s_q before it is reused
        if (q >= nq) return;
        BInst *I = inst + order[q];
        if (I->status != UV_STATUS_RUNNING) continue;
        const int m = I->m, n = I->n, r0 = I->row_off, c0 = I->col_off;
        const int Lr = I->Lr, Lc = I->Lc;
        long long it = I->iter;
        T *us = xs + n + sliced;  // the sliced copies' padding reads a zero after each vector
        // ZC: z and c of the instance in LDS as well (after u), so the column
        // pass streams only delta and the entries
        T *zi = ZC ? us + m + sliced : z + c0;
        const T *ci_ = ZC ? zi + n : c + c0;
        for (int j = tid; j < n; j += nthr) xs[j] = x[c0 + j];
        for (int i = tid; i < m; i += nthr) us[i] = u[r0 + i];
        if (ZC)
            for (int j = tid; j < n; j += nthr) {
                zi[j] = z[c0 + j];
                zi[n + j] = c[c0 + j];
            }
        if (sliced && tid == 0) {
            xs[n] = (T)0;
            us[m] = (T)0;
        }
        __syncthreads();
        // lane groups per segment, or the sliced copies (a wavefront per 64)
        const bool sc = Lc == 0, sr = Lr == 0;
        const int Lc1 = max(Lc, 1), Lr1 = max(Lr, 1);  // lane groups step by them: never zero
        const int gc = tid / Lc1, lc = tid % Lc1, Gc = nthr / Lc1;
        const int wv = tid >> 6, lane64 = tid & 63, nwv = nthr >> 6, nch = (n + 63) >> 6;
        const int *sp_c = scol.ptr + I->ch_off, *sp_r = srow.ptr + I->rh_off;
        const int gr = tid / Lr1, lr = tid % Lr1, Gr = nthr / Lr1;
        int stop = 0;
        for (int k = 0; k < budget && !stop; ++k) {
            // column pass: p = N x + A'u, x-step, projection onto R_+, delta
            auto col_update = [&](int j, int cnt, T atu, double d, T zj, T cj) {
                const T dm = (T)(d * inv_mu);
                const T p = (T)cnt * xs[j] + atu;
                const T xn = (p + zj + dm - cj * (T)inv_mu) / (T)(1 + cnt);
                const T v = xn - dm;
                const T zn = v > (T)0 ? v : (T)0;
                xs[j] = xn;
                zi[j] = zn;
                delta[c0 + j] = d + mu * ((double)zn - (double)xn);
            };
            if (sc) {
                sell_pass<false, T>(wv, nwv, lane64, n, sp_c, scol.idx, (const typename Two<T>::type *)scol.val, us,
                             SellCol<T>{xs, zi, ci_, delta + c0, ccnt + c0, mu, inv_mu, 0.0, 0, 0, 0});
            } else
            for (int jb = 0; jb < n; jb += Gc) {
                const int j = jb + gc;
                T atu = 0, zj = 0, cj = 0;
                double d = 0.0;
                int beg = 0, end = 0;
                if (j < n) {
                    beg = cp[c0 + j];
                    end = cp[c0 + j + 1];
                    if (lc == 0) {  // the update's own loads, in flight with the sum's
                        d = delta[c0 + j];
                        zj = zi[j];
                        cj = ci_[j];
                    }
                    atu = seg_sum<4, T>(beg, end, lc, Lc1, rl, vc, us);
                }
                atu = group_sum_rt(atu, Lc1);
                if (j < n && lc == 0) col_update(j, end - beg, atu, d, zj, cj);
            }
            __syncthreads();
            // row pass: q = A x, lambda update, u.  At a check iteration the
            // row pass forms A x and A z in FP64 with the FP64 values of A
            // (the check's row sums) and the iteration takes its q from that
            // A x, so the check adds no second row product.
            const bool chk = (it + 1) % check_every == 0 || (max_iter > 0 && it + 1 >= max_iter);
            double a[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
            auto row_check = [&](int i, double qz, double qx, double li) {
                const double bd = b64[r0 + i];
                a[0] += (qz - bd) * (qz - bd);
                a[1] += bd * li;
                a[2] += (qx - bd) * (qx - bd);
            };
            if (sr && !chk) {
                sell_pass<true, T>(wv, nwv, lane64, m, sp_r, srow.idx, (const typename Two<T>::type *)srow.val, xs,
                             SellRow<T>{us, fu + r0, b + r0, lam + r0, mu, inv_mu, 0.0, 0, 0});
            } else if (sr) {
                for (int h = wv; h < (m + 63) >> 6; h += nwv) {
                    const int i = (h << 6) + lane64, s0 = sp_r[h], w = (sp_r[h + 1] - s0) >> 6;
                    const int cnt = i < m ? rp[r0 + i + 1] - rp[r0 + i] : 0;
                    double qz, qx;
                    sell_check<2>(s0, cnt, w, lane64, srow.idx, srow.val64, (const T *)zi, (const T *)xs, qz, qx);
                    if (i < m) {
                        const T e = fu[r0 + i] * (b[r0 + i] - (T)qx);
                        const double li = lam[r0 + i] - mu * (double)e;
                        lam[r0 + i] = li;
                        us[i] = (T)((double)e - li * inv_mu);
                        row_check(i, qz, qx, li);
                    }
                }
            } else
            for (int ib = 0; ib < m; ib += Gr) {
                const int i = ib + gr;
                T q = 0, fi = 0, bi = 0;
                double l0 = 0.0, qz = 0.0, qx = 0.0;
                if (i < m) {
                    const int beg = rp[r0 + i], end = rp[r0 + i + 1];
                    if (lr == 0) {
                        fi = fu[r0 + i];
                        bi = b[r0 + i];
                        l0 = lam[r0 + i];
                    }
                    if (chk) seg_sum2<4>(beg, end, lr, Lr1, cl, va64, zi, xs, qz, qx);
                    else q = seg_sum<4, T>(beg, end, lr, Lr1, cl, va, xs);
                }
                if (chk) {
                    qz = group_sum_rt(qz, Lr1);
                    qx = group_sum_rt(qx, Lr1);
                    q = (T)qx;
                } else {
                    q = group_sum_rt(q, Lr1);
                }
                if (i < m && lr == 0) {
                    const T e = fi * (bi - q);
                    const double li = l0 - mu * (double)e;
                    lam[r0 + i] = li;
                    us[i] = (T)((double)e - li * inv_mu);
                    if (chk) row_check(i, qz, qx, li);
                }
            }
            __syncthreads();
            ++it;
            if (chk && gated && !(max_iter > 0 && it >= max_iter)) {
                // primal half first: when r_prim > eps (with finite row sums)
                // this check cannot stop the instance, and its column half is
                // skipped (the row sums are reduced as below, bit for bit)
                double g[3] = {a[0], a[1], a[2]};
                block_sum_rt<3>(g);
                if (tid == 0)
                    s_skip = !(sqrt(g[0]) / (1.0 + sqrt(I->bnorm2)) <= eps) && isfinite(g[0]) && isfinite(g[1]) &&
                             isfinite(g[2]);
                __syncthreads();
                if (s_skip) continue;
            }
            if (chk) {
                // FP64 residuals at (z, lambda, delta) with the FP64 values of A:
                // the row sums came with the row pass, the column sums here
                auto col_res = [&](int j, double atl) {
                    const double r = atl + c64[c0 + j] - delta[c0 + j];
                    a[3] += r * r;
                    a[4] += c64[c0 + j] * (double)zi[j];
                };
                if (sc) {
                    for (int h = wv; h < nch; h += nwv) {
                        const int j = (h << 6) + lane64, s0 = sp_c[h], w = (sp_c[h + 1] - s0) >> 6;
                        const int cnt = j < n ? ccnt[c0 + j] : 0;
                        double atl, none;
                        sell_check<1>(s0, cnt, w, lane64, scol.idx, scol.val64, (const double *)lam + r0,
                                      (const double *)lam + r0, atl, none);
                        if (j < n) col_res(j, atl);
                    }
                } else
                for (int jb = 0; jb < n; jb += Gc) {
                    const int j = jb + gc;
                    double atl = 0.0;
                    if (j < n) atl = seg_sum<4, double>(cp[c0 + j], cp[c0 + j + 1], lc, Lc1, rl, vc64, lam + r0);
                    atl = group_sum_rt(atl, Lc1);
                    if (j < n && lc == 0) col_res(j, atl);
                }
                block_sum_rt<5>(a);
                if (tid == 0) {
                    const double rpr = sqrt(a[0]) / (1.0 + sqrt(I->bnorm2));
                    const double rdu = sqrt(a[3]) / (1.0 + sqrt(I->cnorm2));
                    const double cz = a[4], bl = a[1];
                    const double rg = fabs(cz + bl) / (1.0 + fabs(cz) + fabs(bl));
                    const double kkt = uv::kkt_of(rpr, rdu, rg);
                    I->r_prim = rpr;
                    I->r_dual = rdu;
                    I->r_gap = rg;
                    I->kkt = kkt;
                    I->pobj = cz;
                    I->dobj = -bl;
                    I->res_ax_b = sqrt(a[2]);
                    I->check_iter = it;
                    int st = UV_STATUS_RUNNING;
                    if (!isfinite(kkt)) st = UV_STATUS_NUMERIC;
                    else if (kkt <= eps) st = UV_STATUS_CONVERGED;
                    else if (max_iter > 0 && it >= max_iter) st = UV_STATUS_MAX_ITER;
                    I->status = st;
                    s_stop = st != UV_STATUS_RUNNING;
                }
                __syncthreads();
                stop = s_stop;
            }
        }
        for (int j = tid; j < n; j += nthr) x[c0 + j] = xs[j];
        if (ZC)
            for (int j = tid; j < n; j += nthr) z[c0 + j] = zi[j];
        for (int i = tid; i < m; i += nthr) u[r0 + i] = us[i];
        if (tid == 0) I->iter = it;
        __syncthreads();  // LDS is reused by the next instance
    }
}

inline int bucket_of(int m) { return m < 128 ? 0 : m < 512 ? 1 : m < 2048 ? 2 : 3; }

}  // namespace

struct uv_batch {
    int count = 0;
    int M = 0, N = 0;  // total rows / columns
    int nnz = 0;
    uv_opts o{};
    hipStream_t stream = nullptr, cap = nullptr;
    bool own_stream = false;
    std::vector<void *> allocs;
    int *rp = nullptr, *ci = nullptr, *cp = nullptr, *ri = nullptr;
    lidx_t *cl = nullptr, *rl = nullptr;  // instance-local column (CSR) and row (CSC) numbers
    Slices srow{}, scol{};       // sliced copies of the rows and columns, made when tiles first ask for them
    lidx_t *ccnt = nullptr;      // entries of each column
    bool sliced = false;         // their padding's zeros fit LDS with x and u
    std::vector<int> rmap, cmap; // instance-local numbers of the caller for the device's rows and columns
    int *rmap_d = nullptr, *cmap_d = nullptr;
    double *out = nullptr;       // pinned: one instance's solution or start
    double *va64 = nullptr, *vc64 = nullptr, *b64 = nullptr, *c64 = nullptr;
    void *va = nullptr, *vc = nullptr, *b = nullptr, *c = nullptr, *fu = nullptr;
    void *x = nullptr, *z = nullptr, *u = nullptr;
    double *lam = nullptr, *delta = nullptr;
    BInst *inst = nullptr;
    BInst *inst_host = nullptr;  // pinned mirror
    int *order = nullptr, *queue = nullptr, *budget = nullptr;
    int *budget_host = nullptr;  // pinned
    std::vector<int> order_host;
    int threads = 0;
    int xu_bytes = 0;   // x and u of the largest instance with the sliced copies' zeros (16-byte aligned)
    int zc_bytes = 0;   // x, u, z and c likewise
    bool zc = false;    // z and c staged in LDS too
    int lds_bytes = 0;  // dynamic LDS per workgroup of the launch
    int grid = 0;
    int tiles[2 * 4] = {};  // (Lr, Lc) per size bucket
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
};

namespace {

template <typename T>
T *balloc(uv_batch *h, size_t count)
{
    void *p = nullptr;
    if (uv::dev_malloc(&p, std::max<size_t>(count, 1) * sizeof(T)) != hipSuccess) return nullptr;
    h->allocs.push_back(p);
    return (T *)p;
}

#define UV_BTRY(expr)                              \
    do {                                           \
        if ((expr) != hipSuccess) return UV_EHIP;  \
    } while (0)

int batch_launch(uv_batch *h, hipStream_t st, const int *order, int nq)
{
    k_batch_reset<<<1, 1, 0, st>>>(h->queue);
    const uv_opts &o = h->o;
    const double mu = o.mu, im = 1.0 / o.mu;
#define UV_BATCH_ARGS(T)                                                                                     \
    h->inst, order, nq, h->queue, h->budget, h->rp, h->cl, (const T *)h->va, h->va64, h->cp, h->rl,          \
        (const T *)h->vc, h->vc64, (const T *)h->b, h->b64, (const T *)h->fu, (const T *)h->c, h->c64,      \
        (T *)h->x, (T *)h->z, (T *)h->u, h->lam, h->delta, mu, im, o.eps_kkt, o.check_every, (long long)o.max_iter, \
        h->srow, h->scol, h->ccnt, h->sliced ? 1 : 0, o.full_checks == 0 ? 1 : 0
    const int grid = std::max(1, std::min(h->grid, nq));
    if (o.precision == UV_MIXED)
        h->zc ? k_batch<float, true><<<grid, h->threads, h->lds_bytes, st>>>(UV_BATCH_ARGS(float))
              : k_batch<float, false><<<grid, h->threads, h->lds_bytes, st>>>(UV_BATCH_ARGS(float));
    else
        h->zc ? k_batch<double, true><<<grid, h->threads, h->lds_bytes, st>>>(UV_BATCH_ARGS(double))
              : k_batch<double, false><<<grid, h->threads, h->lds_bytes, st>>>(UV_BATCH_ARGS(double));
#undef UV_BATCH_ARGS
    return hipGetLastError() == hipSuccess ? UV_OK : UV_EHIP;
}

// Slots a sliced copy of an instance with `entries` entries may take.  A slice
// is 64 times its longest segment, so one dense row of 20,000 entries would
// take 1.3e6 slots (18 MB in mixed precision); padded that far, the slices also
// lose the time they save.  Instances past it keep their lane groups, whose
// sums are the same.
inline int64_t slots_allowed(int64_t entries) { return 4 * entries + 8192; }

// A sliced copy of the rows or columns of every instance it suits: slices of
// 64 segments, each as wide as its longest, filled on the device from the
// compressed form.  Sets every instance's rh_off or ch_off on the host.
int build_slices(uv_batch *h, bool rows)
{
    const bool mixed = h->o.precision == UV_MIXED;
    hipStream_t st = h->stream;
    std::vector<int> ptr((size_t)(rows ? h->M : h->N) + 1), sptr(1, 0);
    UV_BTRY(hipMemcpy(ptr.data(), rows ? h->rp : h->cp, sizeof(int) * ptr.size(), hipMemcpyDeviceToHost));
    int64_t slots = 0;
    for (int i = 0; i < h->count; ++i) {
        BInst &I = h->inst_host[i];
        const int off = rows ? I.row_off : I.col_off, nseg = rows ? I.m : I.n;
        int &first = rows ? I.rh_off : I.ch_off;
        const size_t at = sptr.size();
        const int64_t before = slots;
        first = (int)at - 1;
        for (int j0 = 0; j0 < nseg; j0 += 64) {
            int w = 0;
            for (int j = j0; j < std::min(j0 + 64, nseg); ++j) w = std::max(w, ptr[(size_t)off + j + 1] - ptr[(size_t)off + j]);
            slots += 64 * (int64_t)((w + 1) / 2 * 2);
            if (slots + 1024 >= ((int64_t)1 << 31)) break;
            sptr.push_back((int)slots);
        }
        if (slots - before > slots_allowed(ptr[(size_t)off + nseg] - ptr[off]) || slots + 1024 >= ((int64_t)1 << 31)) {
            first = -1;
            slots = before;
            sptr.resize(at);
        }
    }
    const size_t room = (size_t)slots + 128 * kPairs;  // a pass reads whole groups of pairs
    int *dptr = balloc<int>(h, sptr.size());
    unsigned *idx = balloc<unsigned>(h, room / 2);
    double *val64 = balloc<double>(h, room);
    float *val = mixed ? balloc<float>(h, room) : nullptr;
    if (!dptr || !idx || !val64 || (mixed && !val)) return UV_ENOMEM;
    UV_BTRY(hipMemcpy(dptr, sptr.data(), sizeof(int) * sptr.size(), hipMemcpyHostToDevice));
    UV_BTRY(hipMemcpy(h->inst, h->inst_host, sizeof(BInst) * h->count, hipMemcpyHostToDevice));
    k_sell_fill<<<h->count, 256, 0, st>>>(h->inst, rows ? 1 : 0, rows ? h->rp : h->cp, rows ? h->ci : h->ri,
                                          rows ? h->va64 : h->vc64, dptr, (lidx_t *)idx, val64);
    if (mixed && slots > 0) k_narrow<float><<<blocks_for(slots, kWG), kWG, 0, st>>>(slots, val64, val);
    UV_BTRY(hipGetLastError());
    UV_BTRY(hipStreamSynchronize(st));
    (rows ? h->srow : h->scol) = Slices{dptr, idx, mixed ? (const void *)val : (const void *)val64, val64};
    return UV_OK;
}

// The instances' lanes from the tile table, by size bucket: one lane per row
// asks for the sliced rows (two lanes a row, the same sums, where an instance
// has none), none per column for the sliced columns (one lane likewise).
int apply_tiles(uv_batch *h)
{
    for (int d = 0; d < 2; ++d) {  // a copy is made when an instance first asks for it
        bool asked = false;
        for (int i = 0; i < h->count; ++i) asked = asked || h->tiles[2 * bucket_of(h->inst_host[i].m) + d] == (d == 0 ? 1 : 0);
        if (!asked || !h->sliced || (d == 0 ? h->srow : h->scol).ptr) continue;
        const int rc = build_slices(h, d == 0);
        if (rc != UV_OK) return rc;
    }
    for (int i = 0; i < h->count; ++i) {
        BInst &I = h->inst_host[i];
        const int *t = h->tiles + 2 * bucket_of(I.m);
        I.Lr = t[0] > 1 ? t[0] : h->srow.ptr && I.rh_off >= 0 ? 0 : 2;
        I.Lc = t[1] > 0 ? t[1] : h->scol.ptr && I.ch_off >= 0 ? 0 : 1;
    }
    UV_BTRY(hipMemcpyAsync(h->inst, h->inst_host, sizeof(BInst) * h->count, hipMemcpyHostToDevice, h->stream));
    UV_BTRY(hipStreamSynchronize(h->stream));
    return UV_OK;
}

template <typename T, bool ZC>
int occupancy_of(uv_batch *h, int *per_cu)
{
    // LDS above the default 64 KiB per workgroup has to be asked for
    if (h->lds_bytes > 64 * 1024 &&
        hipFuncSetAttribute((const void *)k_batch<T, ZC>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            h->lds_bytes) != hipSuccess) {
        (void)hipGetLastError();  // the refusal is reported here, not by the next launch's check
        return UV_ETOOBIG;
    }
    UV_BTRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, k_batch<T, ZC>, h->threads, h->lds_bytes));
    return UV_OK;
}

// LDS per workgroup (x and u of the largest instance, and z and c too when
// every instance's fit: ZC) and the persistent grid the occupancy allows.
int occupancy_grid(uv_batch *h)
{
    h->zc = h->zc_bytes <= kLdsFree;
    h->lds_bytes = h->zc ? h->zc_bytes : h->xu_bytes;
    int dev = 0, cus = 0;
    UV_BTRY(hipGetDevice(&dev));
    UV_BTRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    int per_cu = 0, rc;
    if (h->o.precision == UV_MIXED)
        rc = h->zc ? occupancy_of<float, true>(h, &per_cu) : occupancy_of<float, false>(h, &per_cu);
    else
        rc = h->zc ? occupancy_of<double, true>(h, &per_cu) : occupancy_of<double, false>(h, &per_cu);
    if (rc != UV_OK) return rc;
    h->grid = std::max(1, per_cu) * cus;
    return UV_OK;
}

// The default tiles.  A workgroup's time for an iteration of an instance with
// w = rows + columns + entries on T threads is about 2.5 + 0.2 w / T us (0.27 on
// 1024; in FP64 a fifth more), and a compute unit cannot do it in less than 0.2 +
// 0.0005 w + 0.0008 T us (0.28 + 0.0007 w + 0.0011 T in FP64) however many
// workgroups share it; a sweep takes about the root of the squares of what the
// workgroups need that fetch the instances one by one and of what the compute
// units do.  Large or few instances want the widest workgroup, many small ones
// as many narrow workgroups as a compute unit holds.  Measured (us a sweep, mixed, T = 64 / 128 / 256 / 512 /
// 1024): 4096 of 20 x 40 5.3 / 6.4 / 9.1 / 19 / 37, of 50 x 100 9.7 / 10.6 / 11.3 /
// 23 / 42, of 200 x 400 30 / 30 / 29 / 37 / 50, 1024 of 1200 x 2400 69 / 43 / 36 /
// 35 / 38, of 5000 x 10000 - / - / 318 / 192 / 146; 64 of 200 x 400 8.5 / 5.5 / 3.9
// / 3.5 / 3.2.
// Rows: the sliced copy, but four lanes while an instance has fewer rows than
// the workgroup about a quarter of its threads (200 rows on 1024: 3.2 against
// 3.7 us; on 256: 5.6 against 3.9), two on narrow workgroups (4096 of 100 x 200 on
// 64: 16.4 against 18.9 us sliced and 17.2 with four; in FP64 up to 512 rows, of
// 200 x 400 on 128: 38.9 against 44.6 and 39.1).
int default_tiles(uv_batch *h, const std::vector<double> &weight)  // the instances', longest first
{
    const bool fp64 = h->o.precision == UV_FP64;
    int dev = 0, cus = 0, best_t = 1024;
    UV_BTRY(hipGetDevice(&dev));
    UV_BTRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    double best = 0.0;
    for (int t = 1024, rc; t >= 64; t /= 2) {
        h->threads = t;
        if ((rc = occupancy_grid(h)) != UV_OK) return rc;
        std::priority_queue<double, std::vector<double>, std::greater<double>> free_at;
        double last = 0.0, cu = 0.0;
        for (double w : weight) {
            double at = (fp64 ? 1.2 : 1.0) * (2.5 + (t == 1024 ? 0.27 : 0.2) * w / t);
            if ((int)free_at.size() == h->grid) {
                at += free_at.top();
                free_at.pop();
            }
            free_at.push(at);
            last = std::max(last, at);
            cu += fp64 ? 0.28 + 0.0007 * w + 0.0011 * t : 0.2 + 0.0005 * w + 0.0008 * t;
        }
        const double us = std::hypot(last, cu / cus);
        if (t == 1024 || us < 0.9 * best) {  // a wider one unless a narrower is clearly faster
            best = us;
            best_t = t;
        }
    }
    h->threads = best_t;
    const int narrow = best_t <= 128;
    const int tiles[2 * 4] = {narrow ? 2 : 4, 0, best_t == 1024 ? 4 : narrow && fp64 ? 2 : 1, 0, 1, 0, 1, 0};
    std::memcpy(h->tiles, tiles, sizeof(tiles));
    return UV_OK;
}

int rebuild_graph(uv_batch *h)
{
    if (h->exec) (void)hipGraphExecDestroy(h->exec);
    if (h->graph) (void)hipGraphDestroy(h->graph);
    h->exec = nullptr;
    h->graph = nullptr;
    if (!h->o.use_graph) return UV_OK;
    if (hipStreamBeginCapture(h->cap, hipStreamCaptureModeRelaxed) != hipSuccess) return UV_EHIP;
    int rc = batch_launch(h, h->cap, h->order, h->count);
    if (hipStreamEndCapture(h->cap, &h->graph) != hipSuccess || rc != UV_OK) return UV_EHIP;
    if (hipGraphInstantiate(&h->exec, h->graph, nullptr, nullptr, 0) != hipSuccess) return UV_EHIP;
    return UV_OK;
}

}  // namespace

extern "C" {

void batch_destroy(uv_batch *h)
{
    if (!h) return;
    if (h->stream) (void)hipStreamSynchronize(h->stream);
    if (h->exec) (void)hipGraphExecDestroy(h->exec);
    if (h->graph) (void)hipGraphDestroy(h->graph);
    for (void *p : h->allocs) (void)hipFree(p);
    if (h->inst_host) (void)hipHostFree(h->inst_host);
    if (h->out) (void)hipHostFree(h->out);
    if (h->budget_host) (void)hipHostFree(h->budget_host);
    if (h->cap) (void)hipStreamDestroy(h->cap);
    if (h->own_stream && h->stream) (void)hipStreamDestroy(h->stream);
    delete h;
}

int batch_create(int32_t count, const uv_csr *A, const double *const *b, const double *const *c,
                 const uv_opts *opts, uv_batch **out)
{
    if (!out) return UV_EINVAL;
    *out = nullptr;
    if (count < 1 || !A || !b || !c) return UV_EINVAL;
    uv_opts o;
    uv_default_opts(&o);
    if (opts) o = *opts;
    if (!(o.mu > 0.0) || !std::isfinite(o.mu) || o.check_every < 1 || !(o.eps_kkt >= 0.0) || o.max_iter < 0 ||
        (o.precision != UV_FP64 && o.precision != UV_MIXED) || o.full_checks < 0 || o.full_checks > 1)
        return UV_EINVAL;
    const size_t ts = o.precision == UV_MIXED ? 4 : 8;
    int64_t M = 0, N = 0, NNZ = 0;
    size_t lds = 0, lds_zc = 0, largest = 0;
    for (int i = 0; i < count; ++i) {
        const uv_csr &a = A[i];
        if (!b[i] || !c[i] || !a.row_ptr || a.m < 1 || a.n < 1 || a.nnz < 0) return UV_EINVAL;
        if (a.nnz > 0 && (!a.col_idx || !a.val)) return UV_EINVAL;
        if (a.row_ptr[0] != 0 || a.row_ptr[a.m] != a.nnz) return UV_EBADCSR;
        for (int32_t r = 0; r < a.m; ++r) {
            const int64_t b0 = a.row_ptr[r], b1 = a.row_ptr[r + 1];
            if (b1 < b0 || b1 > a.nnz) return UV_EBADCSR;
            for (int64_t k = b0; k < b1; ++k) {
                if (a.col_idx[k] < 0 || a.col_idx[k] >= a.n) return UV_EBADCSR;
                if (k > b0 && a.col_idx[k] <= a.col_idx[k - 1]) return UV_EBADCSR;
            }
        }
        M += a.m;
        N += a.n;
        NNZ += a.nnz;
        lds = std::max(lds, (size_t)(a.m + a.n) * ts);
        lds_zc = std::max(lds_zc, (size_t)(a.m + 3 * (size_t)a.n) * ts);
        largest = std::max(largest, 3 * (size_t)a.n + a.m);
    }
    if (NNZ >= ((int64_t)1 << 31) || M >= ((int64_t)1 << 31) || N >= ((int64_t)1 << 31)) return UV_ETOOBIG;
    if (lds > (size_t)kLdsMax) return UV_ETOOBIG;  // x and u of every instance must fit in LDS

    uv_batch *h = new (std::nothrow) uv_batch();
    if (!h) return UV_ENOMEM;
    h->count = count;
    h->M = (int)M;
    h->N = (int)N;
    h->nnz = (int)NNZ;
    h->o = o;
    h->sliced = (lds + 2 * ts + 15) / 16 * 16 <= (size_t)kLdsFree;
    if (h->sliced) {
        lds += 2 * ts;
        lds_zc += 2 * ts;
    }
    h->xu_bytes = (int)((lds + 15) / 16 * 16);
    h->zc_bytes = (int)std::min<size_t>((lds_zc + 15) / 16 * 16, (size_t)1 << 30);
    h->lds_bytes = h->xu_bytes;
    int rc = UV_OK;
    auto fail = [&](int code) {
        batch_destroy(h);
        return code;
    };
    if (o.hip_stream) h->stream = (hipStream_t)o.hip_stream;
    else {
        if (hipStreamCreateWithFlags(&h->stream, hipStreamNonBlocking) != hipSuccess) return fail(UV_EHIP);
        h->own_stream = true;
    }
    if (hipStreamCreateWithFlags(&h->cap, hipStreamNonBlocking) != hipSuccess) return fail(UV_EHIP);
    hipStream_t st = h->stream;
    const bool mixed = o.precision == UV_MIXED;

    h->rp = balloc<int>(h, M + 1);
    h->ci = balloc<int>(h, NNZ);
    h->va64 = balloc<double>(h, NNZ);
    h->cp = balloc<int>(h, N + 1);
    h->ri = balloc<int>(h, NNZ);
    h->vc64 = balloc<double>(h, NNZ);
    h->cl = balloc<lidx_t>(h, NNZ);
    h->rl = balloc<lidx_t>(h, NNZ);
    h->b64 = balloc<double>(h, M);
    h->c64 = balloc<double>(h, N);
    h->lam = balloc<double>(h, M);
    h->delta = balloc<double>(h, N);
    h->x = balloc<char>(h, ts * N);
    h->z = balloc<char>(h, ts * N);
    h->u = balloc<char>(h, ts * M);
    h->fu = balloc<char>(h, ts * M);
    if (mixed) {
        h->va = balloc<float>(h, NNZ);
        h->vc = balloc<float>(h, NNZ);
        h->b = balloc<float>(h, M);
        h->c = balloc<float>(h, N);
    } else {
        h->va = h->va64;
        h->vc = h->vc64;
        h->b = h->b64;
        h->c = h->c64;
    }
    h->inst = balloc<BInst>(h, count);
    h->order = balloc<int>(h, count);
    h->queue = balloc<int>(h, 1);
    h->rmap_d = balloc<int>(h, M);
    h->cmap_d = balloc<int>(h, N);
    h->ccnt = balloc<lidx_t>(h, N);
    h->budget = balloc<int>(h, 1);
    int *cnt = balloc<int>(h, N);
    int *bsum = balloc<int>(h, blocks_for(N, 4 * kWG));
    for (void *p : {(void *)h->rp, (void *)h->ci, (void *)h->va64, (void *)h->cp, (void *)h->ri, (void *)h->vc64, (void *)h->cl, (void *)h->rl,
                    (void *)h->b64, (void *)h->c64, (void *)h->lam, (void *)h->delta, h->x,
                    h->z, h->u, h->fu, h->va, h->vc, h->b, h->c, (void *)h->inst, (void *)h->order,
                    (void *)h->queue, (void *)h->budget, (void *)h->rmap_d, (void *)h->cmap_d, (void *)h->ccnt,
                    (void *)cnt, (void *)bsum})
        if (!p) return fail(UV_ENOMEM);
    if (uv::host_malloc(&h->out, sizeof(double) * largest, hipHostMallocDefault) != hipSuccess) {
        h->out = nullptr;
        return fail(UV_ENOMEM);
    }
    if (uv::host_malloc(&h->inst_host, sizeof(BInst) * count, hipHostMallocDefault) != hipSuccess) {
        h->inst_host = nullptr;
        return fail(UV_ENOMEM);
    }
    if (uv::host_malloc(&h->budget_host, sizeof(int), hipHostMallocDefault) != hipSuccess) {
        h->budget_host = nullptr;
        return fail(UV_ENOMEM);
    }

    // Pack the block-diagonal matrix with global indices, rows and columns
    // of an instance in falling order of their entries (stable).  The instances
    // are packed by a few threads (5.5 ns an entry: 1024 LPs of 50 to 5000 rows
    // took 68 ms of a create of 102 on one, 52 in all on eight).
    h->rmap.resize(M);
    h->cmap.resize(N);
    {
        std::vector<int64_t> first(count);  // an instance's first entry
        int64_t ro = 0, co = 0, ko = 0;
        for (int i = 0; i < count; ++i) {
            BInst &I = h->inst_host[i];
            std::memset(&I, 0, sizeof(I));
            I.m = A[i].m;
            I.n = A[i].n;
            I.row_off = (int)ro;
            I.col_off = (int)co;
            I.status = UV_STATUS_RUNNING;
            I.check_iter = -1;
            first[i] = ko;
            ro += A[i].m;
            co += A[i].n;
            ko += A[i].nnz;
        }
        std::vector<int> rp32(M + 1);
        std::vector<double> bb(M), cc(N);
        const std::unique_ptr<int[]> ci32(new (std::nothrow) int[std::max<int64_t>(NNZ, 1)]);
        const std::unique_ptr<double[]> va(new (std::nothrow) double[std::max<int64_t>(NNZ, 1)]);
        if (!ci32 || !va) return fail(UV_ENOMEM);
        std::atomic<int> next{0};
        std::atomic<bool> failed{false};
        auto pack = [&]() {
            std::vector<int> inv, cc0, slot;
            // map[slot] = original number, by falling count: a counting sort
            auto by_count = [&](int len, auto count, int *map) {
                int top = 0;
                for (int q = 0; q < len; ++q) top = std::max(top, count(q));
                slot.assign((size_t)top + 2, 0);
                for (int q = 0; q < len; ++q) slot[(size_t)(top - count(q)) + 1] += 1;
                for (int q = 0; q <= top; ++q) slot[(size_t)q + 1] += slot[q];
                for (int q = 0; q < len; ++q) map[slot[(size_t)(top - count(q))]++] = q;
            };
            for (int i; (i = next++) < count;) {
                const uv_csr &a = A[i];
                const int64_t ro = h->inst_host[i].row_off, co = h->inst_host[i].col_off;
                int *rm = h->rmap.data() + ro, *cm = h->cmap.data() + co;
                by_count(a.m, [&](int r) { return (int)(a.row_ptr[r + 1] - a.row_ptr[r]); }, rm);
                cc0.assign(a.n, 0);
                for (int64_t k = 0; k < a.nnz; ++k) cc0[a.col_idx[k]] += 1;
                by_count(a.n, [&](int j) { return cc0[j]; }, cm);
                inv.resize(a.n);
                for (int j = 0; j < a.n; ++j) inv[cm[j]] = j;
                for (int j = 0; j < a.n; ++j) cc[co + j] = c[i][cm[j]];
                int64_t w = first[i];
                for (int r = 0; r < a.m; ++r) {
                    rp32[ro + r] = (int)w;
                    bb[ro + r] = b[i][rm[r]];
                    for (int64_t k = a.row_ptr[rm[r]]; k < a.row_ptr[rm[r] + 1]; ++k, ++w) {
                        ci32[w] = (int)(co + inv[a.col_idx[k]]);
                        va[w] = a.val[k];
                    }
                }
            }
        };
        auto guarded = [&]() {
            try {
                pack();
            } catch (...) {
                failed = true;
            }
        };
        std::vector<std::thread> pool;
        const int64_t threads = std::min<int64_t>({8, (int64_t)std::thread::hardware_concurrency(), count, 1 + NNZ / 400000});
        try {
            for (int64_t q = 1; q < threads; ++q) pool.emplace_back(guarded);
        } catch (...) {  // as many as there are
        }
        guarded();
        for (std::thread &t : pool) t.join();
        if (failed) return fail(UV_ENOMEM);
        rp32[M] = (int)NNZ;
        if (hipMemcpy(h->rp, rp32.data(), sizeof(int) * (M + 1), hipMemcpyHostToDevice) != hipSuccess) return fail(UV_EHIP);
        if (NNZ > 0) {
            if (hipMemcpy(h->ci, ci32.get(), sizeof(int) * NNZ, hipMemcpyHostToDevice) != hipSuccess) return fail(UV_EHIP);
            if (hipMemcpy(h->va64, va.get(), sizeof(double) * NNZ, hipMemcpyHostToDevice) != hipSuccess) return fail(UV_EHIP);
        }
        if (hipMemcpy(h->b64, bb.data(), sizeof(double) * M, hipMemcpyHostToDevice) != hipSuccess) return fail(UV_EHIP);
        if (hipMemcpy(h->c64, cc.data(), sizeof(double) * N, hipMemcpyHostToDevice) != hipSuccess) return fail(UV_EHIP);
        if (hipMemcpy(h->rmap_d, h->rmap.data(), sizeof(int) * M, hipMemcpyHostToDevice) != hipSuccess ||
            hipMemcpy(h->cmap_d, h->cmap.data(), sizeof(int) * N, hipMemcpyHostToDevice) != hipSuccess)
            return fail(UV_EHIP);
    }
    // Longest instances first.
    h->order_host.resize(count);
    std::iota(h->order_host.begin(), h->order_host.end(), 0);
    std::stable_sort(h->order_host.begin(), h->order_host.end(), [&](int p, int q) {
        return A[p].nnz + A[p].m + A[p].n > A[q].nnz + A[q].m + A[q].n;
    });
    if (hipMemcpy(h->order, h->order_host.data(), sizeof(int) * count, hipMemcpyHostToDevice) != hipSuccess) return fail(UV_EHIP);

    if (!build_csc((int)M, (int)N, (int)NNZ, h->rp, h->ci, h->va64, h->cp, h->ri, h->vc64, cnt, bsum, st))
        return fail(UV_EHIP);
    if (mixed) {
        k_row_factor<float><<<blocks_for(M, kWG), kWG, 0, st>>>((int)M, h->rp, h->va64, (float *)h->fu);
        if (NNZ > 0) {
            k_narrow<float><<<blocks_for(NNZ, kWG), kWG, 0, st>>>(NNZ, h->va64, (float *)h->va);
            k_narrow<float><<<blocks_for(NNZ, kWG), kWG, 0, st>>>(NNZ, h->vc64, (float *)h->vc);
        }
        k_narrow<float><<<blocks_for(M, kWG), kWG, 0, st>>>(M, h->b64, (float *)h->b);
        k_narrow<float><<<blocks_for(N, kWG), kWG, 0, st>>>(N, h->c64, (float *)h->c);
    } else {
        k_row_factor<double><<<blocks_for(M, kWG), kWG, 0, st>>>((int)M, h->rp, h->va64, (double *)h->fu);
    }
    // zero start
    if (hipMemsetAsync(h->x, 0, ts * N, st) != hipSuccess || hipMemsetAsync(h->z, 0, ts * N, st) != hipSuccess ||
        hipMemsetAsync(h->u, 0, ts * M, st) != hipSuccess || hipMemsetAsync(h->lam, 0, 8 * M, st) != hipSuccess ||
        hipMemsetAsync(h->delta, 0, 8 * N, st) != hipSuccess)
        return fail(UV_EHIP);
    if (hipMemcpyAsync(h->inst, h->inst_host, sizeof(BInst) * count, hipMemcpyHostToDevice, st) != hipSuccess)
        return fail(UV_EHIP);
    k_batch_norms<<<count, 256, 0, st>>>(h->inst, h->b64, h->c64);
    k_local_idx<<<count, 256, 0, st>>>(h->inst, h->rp, h->ci, h->cp, h->ri, h->cl, h->rl);
    if (hipGetLastError() != hipSuccess) return fail(UV_EHIP);
    if (hipMemcpyAsync(h->inst_host, h->inst, sizeof(BInst) * count, hipMemcpyDeviceToHost, st) != hipSuccess ||
        hipStreamSynchronize(st) != hipSuccess)
        return fail(UV_EHIP);
    k_col_entries<<<blocks_for(N, 256), 256, 0, st>>>((int)N, h->cp, h->ccnt);
    std::vector<double> weight(count);
    for (int q = 0; q < count; ++q) {
        const uv_csr &a = A[h->order_host[q]];
        weight[q] = (double)a.nnz + a.m + a.n;
    }
    if ((rc = default_tiles(h, weight)) != UV_OK) return fail(rc);
    if ((rc = apply_tiles(h)) != UV_OK) return fail(rc);
    if ((rc = occupancy_grid(h)) != UV_OK) return fail(rc);
    if ((rc = rebuild_graph(h)) != UV_OK) return fail(rc);
    *out = h;
    return UV_OK;
}

int batch_set_tiles(uv_batch *h, int32_t threads, const int32_t *lanes)
{
    if (!h || !lanes) return UV_EINVAL;
    if (threads != 64 && threads != 128 && threads != 256 && threads != 512 && threads != 1024) return UV_EINVAL;
    for (int k = 0; k < 8; ++k) {
        const int lo = k % 2 ? 0 : 1;  // lanes per row >= 1; lanes per column >= 0 (0: sliced copy)
        if (lanes[k] < lo || lanes[k] > 64 || (lanes[k] & (lanes[k] - 1)) || lanes[k] > threads) return UV_EINVAL;
    }
    UV_BTRY(hipStreamSynchronize(h->stream));
    UV_BTRY(hipMemcpy(h->inst_host, h->inst, sizeof(BInst) * h->count, hipMemcpyDeviceToHost));
    h->threads = threads;
    std::memcpy(h->tiles, lanes, sizeof(h->tiles));
    int rc;
    if ((rc = apply_tiles(h)) != UV_OK) return rc;
    if ((rc = occupancy_grid(h)) != UV_OK) return rc;
    return rebuild_graph(h);
}

int batch_get_tiles(const uv_batch *h, int32_t *threads, int32_t *lanes)
{
    if (!h) return UV_EINVAL;
    if (threads) *threads = h->threads;
    if (lanes) std::memcpy(lanes, h->tiles, sizeof(h->tiles));
    return UV_OK;
}

int batch_iterate(uv_batch *h, int64_t k, int32_t *n_active)
{
    if (!h || k < 0) return UV_EINVAL;
    int64_t left = k;
    while (left > 0) {
        const int step = (int)std::min<int64_t>(left, 1 << 30);
        *h->budget_host = step;
        UV_BTRY(hipMemcpyAsync(h->budget, h->budget_host, sizeof(int), hipMemcpyHostToDevice, h->stream));
        if (h->exec) UV_BTRY(hipGraphLaunch(h->exec, h->stream));
        else {
            int rc = batch_launch(h, h->stream, h->order, h->count);
            if (rc != UV_OK) return rc;
        }
        left -= step;
    }
    UV_BTRY(hipMemcpyAsync(h->inst_host, h->inst, sizeof(BInst) * h->count, hipMemcpyDeviceToHost, h->stream));
    UV_BTRY(hipStreamSynchronize(h->stream));
    if (n_active) {
        int a = 0;
        for (int i = 0; i < h->count; ++i) a += h->inst_host[i].status == UV_STATUS_RUNNING;
        *n_active = a;
    }
    return UV_OK;
}

int batch_residuals(uv_batch *h, int32_t i, uv_residuals *r)
{
    if (!h || !r || i < 0 || i >= h->count) return UV_EINVAL;
    const BInst &I = h->inst_host[i];
    r->r_prim = I.r_prim;
    r->r_dual = I.r_dual;
    r->r_gap = I.r_gap;
    r->kkt = I.kkt;
    r->pobj = I.pobj;
    r->dobj = I.dobj;
    r->res_ax_b = I.res_ax_b;
    r->prim_inf = r->dual_inf = r->scale_p = r->scale_d = 0.0;
    r->pobj_x = r->gap_x = 0.0;
    r->iter = I.iter;
    r->status = I.status;
    return I.status == UV_STATUS_NUMERIC ? UV_ENUMERIC : UV_OK;
}

int batch_solution(uv_batch *h, int32_t i, double *x, double *z, double *lambda, double *delta)
{
    if (!h || i < 0 || i >= h->count) return UV_EINVAL;
    const BInst &I = h->inst_host[i];
    hipStream_t st = h->stream;
    // one launch writes the four vectors to pinned memory, one wait
    const unsigned g = blocks_for((int64_t)I.n + I.m, 256);
#define UV_OUT_ARGS(T)                                                                                     \
    I.col_off, I.n, I.row_off, I.m, (const T *)h->x, (const T *)h->z, h->delta, h->lam, h->cmap_d, h->rmap_d, h->out
    if (h->o.precision == UV_MIXED) k_batch_out<float><<<g, 256, 0, st>>>(UV_OUT_ARGS(float));
    else k_batch_out<double><<<g, 256, 0, st>>>(UV_OUT_ARGS(double));
#undef UV_OUT_ARGS
    UV_BTRY(hipGetLastError());
    UV_BTRY(hipStreamSynchronize(st));
    const size_t n = (size_t)I.n;
    if (x) std::memcpy(x, h->out, 8 * n);
    if (z) std::memcpy(z, h->out + n, 8 * n);
    if (delta) std::memcpy(delta, h->out + 2 * n, 8 * n);
    if (lambda) std::memcpy(lambda, h->out + 3 * n, 8 * (size_t)I.m);
    return UV_OK;
}

int batch_set_start(uv_batch *h, int32_t i, const double *x, const double *z, const double *delta,
                    const double *lambda)
{
    if (!h || i < 0 || i >= h->count) return UV_EINVAL;
    BInst &I = h->inst_host[i];
    hipStream_t st = h->stream;
    // into the device's numbering on the way to the pinned buffer, then one launch and one wait
    const double *src[4] = {x, z, delta, lambda};
    int have = 0;
    double *to = h->out;
    for (int q = 0; q < 4; ++q) {
        const int len = q < 3 ? I.n : I.m, *map = q < 3 ? h->cmap.data() + I.col_off : h->rmap.data() + I.row_off;
        if (src[q]) {
            have |= 1 << q;
            for (int k = 0; k < len; ++k) to[k] = src[q][map[k]];
        }
        to += len;
    }
    const unsigned g = blocks_for((int64_t)I.n + I.m, 256);
#define UV_IN_ARGS(T)                                                                                            \
    I.col_off, I.n, I.row_off, I.m, have, h->out, (T *)h->x, (T *)h->z, h->delta, h->lam, (T *)h->u, 1.0 / h->o.mu
    if (h->o.precision == UV_MIXED) k_batch_in<float><<<g, 256, 0, st>>>(UV_IN_ARGS(float));
    else k_batch_in<double><<<g, 256, 0, st>>>(UV_IN_ARGS(double));
#undef UV_IN_ARGS
    UV_BTRY(hipGetLastError());
    I.iter = 0;
    I.check_iter = -1;
    I.status = UV_STATUS_RUNNING;
    UV_BTRY(hipMemcpyAsync(h->inst + i, &I, sizeof(BInst), hipMemcpyHostToDevice, st));
    UV_BTRY(hipStreamSynchronize(st));
    return UV_OK;
}

// Times `iters` iterations of the instances in size bucket `bucket` (-1 =
// all) with the current tiles, from a copy of the current state that is put
// back afterwards.  *ms is the launch's duration.
int batch_time(uv_batch *h, int32_t bucket, int32_t iters, double *ms)
{
    if (!h || !ms || iters < 1 || bucket < -1 || bucket > 3) return UV_EINVAL;
    hipStream_t st = h->stream;
    const size_t ts = h->o.precision == UV_MIXED ? 4 : 8;
    std::vector<int> sel;
    UV_BTRY(hipStreamSynchronize(st));
    UV_BTRY(hipMemcpy(h->inst_host, h->inst, sizeof(BInst) * h->count, hipMemcpyDeviceToHost));
    for (int q = 0; q < h->count; ++q) {
        const int i = h->order_host[q];
        if (bucket < 0 || bucket_of(h->inst_host[i].m) == bucket) sel.push_back(i);
    }
    *ms = 0.0;
    if (sel.empty()) return UV_OK;
    // save state
    std::vector<BInst> inst_save(h->inst_host, h->inst_host + h->count);
    char *save = nullptr;
    const size_t bytes_xz = ts * h->N, bytes_u = ts * h->M;
    const size_t total = 2 * bytes_xz + bytes_u + 8 * (size_t)h->M + 8 * (size_t)h->N;
    if (uv::dev_malloc(&save, total) != hipSuccess) return UV_ENOMEM;
    char *p = save;
    int rc = UV_OK;
    auto cp_ = [&](void *dst, const void *src, size_t n) {
        if (rc == UV_OK && hipMemcpyAsync(dst, src, n, hipMemcpyDeviceToDevice, st) != hipSuccess) rc = UV_EHIP;
    };
    cp_(p, h->x, bytes_xz);
    cp_(p + bytes_xz, h->z, bytes_xz);
    cp_(p + 2 * bytes_xz, h->u, bytes_u);
    cp_(p + 2 * bytes_xz + bytes_u, h->lam, 8 * (size_t)h->M);
    cp_(p + 2 * bytes_xz + bytes_u + 8 * (size_t)h->M, h->delta, 8 * (size_t)h->N);
    const bool saved = rc == UV_OK;  // restore below only from a complete copy
    int *dsel = nullptr;
    if (rc == UV_OK && uv::dev_malloc(&dsel, sizeof(int) * sel.size()) != hipSuccess) rc = UV_ENOMEM;
    if (rc == UV_OK && hipMemcpyAsync(dsel, sel.data(), sizeof(int) * sel.size(), hipMemcpyHostToDevice, st) != hipSuccess)
        rc = UV_EHIP;
    // run the timed launch with every selected instance marked running
    std::vector<BInst> tmp = inst_save;
    for (int i : sel) tmp[i].status = UV_STATUS_RUNNING;
    if (rc == UV_OK && hipMemcpyAsync(h->inst, tmp.data(), sizeof(BInst) * h->count, hipMemcpyHostToDevice, st) != hipSuccess)
        rc = UV_EHIP;
    // no early stop while timing: eps = 0 and no iteration cap
    const uv_opts keep = h->o;
    h->o.eps_kkt = 0.0;
    h->o.max_iter = 0;
    *h->budget_host = iters;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (rc == UV_OK && (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess)) rc = UV_EHIP;
    if (rc == UV_OK && hipMemcpyAsync(h->budget, h->budget_host, sizeof(int), hipMemcpyHostToDevice, st) != hipSuccess)
        rc = UV_EHIP;
    if (rc == UV_OK) {
        (void)hipEventRecord(e0, st);
        rc = batch_launch(h, st, dsel, (int)sel.size());
        (void)hipEventRecord(e1, st);
    }
    if (rc == UV_OK && hipStreamSynchronize(st) != hipSuccess) rc = UV_EHIP;
    float t = 0.f;
    if (rc == UV_OK) {
        (void)hipEventElapsedTime(&t, e0, e1);
        *ms = t;
    }
    h->o = keep;
    // restore, whatever happened in between (an error keeps its code)
    auto back = [&](void *dst, const void *src, size_t n) {
        if (hipMemcpyAsync(dst, src, n, hipMemcpyDeviceToDevice, st) != hipSuccess) rc = UV_EHIP;
    };
    if (saved) {
        back(h->x, p, bytes_xz);
        back(h->z, p + bytes_xz, bytes_xz);
        back(h->u, p + 2 * bytes_xz, bytes_u);
        back(h->lam, p + 2 * bytes_xz + bytes_u, 8 * (size_t)h->M);
        back(h->delta, p + 2 * bytes_xz + bytes_u + 8 * (size_t)h->M, 8 * (size_t)h->N);
    }
    if (hipMemcpyAsync(h->inst, inst_save.data(), sizeof(BInst) * h->count, hipMemcpyHostToDevice, st) != hipSuccess)
        rc = UV_EHIP;
    if (hipStreamSynchronize(st) != hipSuccess) rc = UV_EHIP;
    std::memcpy(h->inst_host, inst_save.data(), sizeof(BInst) * h->count);
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    if (dsel) (void)hipFree(dsel);
    (void)hipFree(save);
    return rc;
}

int batch_info(const uv_batch *h, int64_t *info)
{
    if (!h || !info) return UV_EINVAL;
    info[0] = h->count;
    info[1] = h->M;
    info[2] = h->N;
    info[3] = h->nnz;
    info[4] = h->grid;
    info[5] = h->lds_bytes;
    return UV_OK;
}

}  // extern "C"
