// dense.hip -- dense linear algebra for the learned warm start: an FP32
// GEMM, a randomized principal-component fit built on it, and the small
// (l x l, l <= 1024) host-side factorizations the fit needs.
//
// PCA of the solution matrix Y (N samples x D features, D large):
//   mean, center Y in place, Z = Y Omega (Omega Gaussian, D x l),
//   q rounds of Z <- orth(Y (orth(Y' Z))),  Q = orth(Z),  B = Q' Y (l x D),
//   B B' = U S^2 U' (Jacobi),  basis = top-k rows of S^{-1} U' B, orthonormalized,
// i.e. the randomized range finder with power iterations of Halko,
// Martinsson and Tropp; orth() is Cholesky QR of FP64 Gram matrices, applied
// until the columns are orthonormal, with a random column for a dependent one.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <vector>

#include "../../include/uvadmm.h"
#include "common.hpp"

namespace {

typedef float v4u __attribute__((ext_vector_type(4), aligned(4)));  // four floats at any float address
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));

// How an operand is read: four elements at a time along k (KC) or along its
// other dimension (MC), or element by element (EL) when neither stride is 1.
enum Load { LD_KC = 0, LD_MC = 1, LD_EL = 2 };

constexpr int kTile = 64;         // rows and columns of C a workgroup owns
constexpr int kTK = 32;           // k per staged step
constexpr int kPK = kTK + 4;      // LDS pitch of [row][k] tiles (KC, EL)
constexpr int kPM = kTile + 4;    // LDS pitch of [k][row] tiles (MC)
constexpr int kLds = kTile * kPK; // floats of either form (32 * 68 < 64 * 36)
static_assert(kTK * kPM <= kLds, "both forms fit");

// One operand's 64 x 32 tile (rows of its m or n dimension), element (r, k)
// at P[r * rs + k * ks], held in registers between the global loads and the
// LDS stores.  Rows past R repeat the last one or are zero (their results
// are not written); k past K is zero.
template <int MODE>
struct Tile {
    v4f v[2];

    __device__ __forceinline__ void load(int t, const float *__restrict__ P, int64_t rs, int64_t ks, int r0, int R,
                                         int k0, int K)
    {
        const bool inside = k0 + kTK <= K && (MODE == LD_KC || r0 + kTile <= R);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int c = t + q * 256;
            if (MODE == LD_KC) {
                const int r = min(r0 + (c >> 3), R - 1), k = k0 + (c & 7) * 4;
                const float *p = P + (int64_t)r * rs + k;
                if (inside) v[q] = *(const v4u *)p;
                else
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[q][e] = k + e < K ? p[e] : 0.f;
            } else if (MODE == LD_MC) {
                const int r = r0 + (c & 15) * 4, k = k0 + (c >> 4);
                const float *p = P + (int64_t)k * ks + r;
                if (inside) v[q] = *(const v4u *)p;
                else
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[q][e] = k < K && r + e < R ? p[e] : 0.f;
            } else {
                const int r = min(r0 + (c >> 3), R - 1), k = k0 + (c & 7) * 4;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    v[q][e] = k + e < K ? P[(int64_t)r * rs + (int64_t)(k + e) * ks] : 0.f;
            }
        }
    }

    __device__ __forceinline__ void store(int t, float *__restrict__ T) const
    {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int c = t + q * 256;
            if (MODE == LD_MC) *(v4f *)(T + (c >> 4) * kPM + (c & 15) * 4) = v[q];
            else *(v4f *)(T + (c >> 3) * kPK + (c & 7) * 4) = v[q];
        }
    }

    // The operand's values for row `row` and k = 8 c + 4 h + 0..3.
    static __device__ __forceinline__ v4f frag(const float *__restrict__ T, int row, int c, int h)
    {
        const int k = c * 8 + h * 4;
        if (MODE != LD_MC) return *(const v4f *)(T + row * kPK + k);
        v4f r;
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = T[(k + e) * kPM + row];
        return r;
    }
};

// C = alpha A B + beta C, A(i,k) = A[i*a_rs + k*a_cs], B(k,j) = B[k*b_rs +
// j*b_cs], C row-major with leading dimension ldc; any M, N, K.  A workgroup
// owns a 64 x 64 block of C for a share of k (blockIdx.z of `splits`); KS
// groups of four wavefronts (2 x 2, 32 x 32 each: v_mfma_f32_32x32x2_f32, FP32
// products and sums) take its 32-deep steps in turn, each with tiles of its
// own in LDS, the next step's loads in flight, and are added in order at the
// end.  A lane holds four consecutive k of its row, so an MFMA adds k = 8 c +
// s and 8 c + 4 + s.  With splits > 1 the blocks' sums go to W[split][M][N]
// and k_gemm_sum adds them.
// What bounds it: the FP32 matrix cores (154 TFLOP/s for a large product on
// this card) where C has enough blocks; with a long k and few blocks of C,
// reading A from HBM, which the split shares among the compute units.
// Against the vector units' 16-deep slices and no split: 4096^3 2.36 -> 1.35
// ms (102 TFLOP/s), 2000 x 30000 x 96 253 -> 187 us, 2000 x 96 x 30000 4.86
// -> 0.58 ms without a workspace and under 0.25 ms with one; the products of a PCA
// fit of 2000 x 30000 samples (l = 128) 51 -> 2.5 ms.
template <int AM, int BM, int KS>
__global__ void __launch_bounds__(256 * KS)
k_gemm_f32(int M, int N, int K, const float *__restrict__ A, int64_t a_rs, int64_t a_cs,
           const float *__restrict__ B, int64_t b_rs, int64_t b_cs, float *__restrict__ C, int64_t ldc,
           float alpha, float beta, int splits, float *__restrict__ W)
{
    __shared__ __align__(16) float lds[KS][2][kLds];
    const int grp = threadIdx.x >> 8, t = threadIdx.x & 255;
    const int wave = t >> 6, lane = t & 63, wm = (wave >> 1) * 32, wn = (wave & 1) * 32, r = lane & 31, h = lane >> 5;
    const int m0 = blockIdx.y * kTile, n0 = blockIdx.x * kTile;
    const int steps = (K + kTK - 1) / kTK, z = blockIdx.z;
    const int s0 = (int)((int64_t)steps * z / splits), s1 = (int)((int64_t)steps * (z + 1) / splits);
    float *As = lds[grp][0], *Bs = lds[grp][1];
    v16f acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    Tile<AM> ta;
    Tile<BM> tb;
    // a group past its last step multiplies zeros (k past K), so that every
    // group takes the same number of barriers
    auto fetch = [&](int s) {
        const int k0 = s < s1 ? s * kTK : K;
        ta.load(t, A, a_rs, a_cs, m0, M, k0, K);
        tb.load(t, B, b_cs, b_rs, n0, N, k0, K);
    };
    fetch(s0 + grp);
    for (int s = s0; s < s1; s += KS) {
        ta.store(t, As);
        tb.store(t, Bs);
        __syncthreads();
        if (s + KS < s1) fetch(s + KS + grp);
#pragma unroll
        for (int c = 0; c < kTK / 8; ++c) {
            const v4f a = Tile<AM>::frag(As, wm + r, c, h), b = Tile<BM>::frag(Bs, wn + r, c, h);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[e], acc, 0, 0, 0);
        }
        __syncthreads();
    }
    if (KS > 1) {  // the groups' blocks meet in LDS, group by group
        float *sum = &lds[0][0][0];
        static_assert(KS == 1 || KS * 2 * kLds >= kTile * kTile, "a block of C fits");
        for (int g = 0; g < KS; ++g) {
            if (grp == g)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int o = (wm + 8 * (e >> 2) + 4 * h + (e & 3)) * kTile + wn + r;
                    if (g == 0) sum[o] = acc[e];
                    else acc[e] = sum[o] += acc[e];
                }
            __syncthreads();
        }
        if (grp != KS - 1) return;
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const int i = m0 + wm + 8 * (e >> 2) + 4 * h + (e & 3), j = n0 + wn + r;
        if (i >= M || j >= N) continue;
        if (splits > 1) {
            W[((int64_t)z * M + i) * N + j] = acc[e];
        } else {
            float *p = C + (int64_t)i * ldc + j;
            *p = alpha * acc[e] + (beta != 0.f ? beta * *p : 0.f);
        }
    }
}

// C = alpha (W[0] + W[1] + ...) + beta C
__global__ void __launch_bounds__(256)
k_gemm_sum(int M, int N, int splits, const float *__restrict__ W, float *__restrict__ C, int64_t ldc, float alpha,
           float beta)
{
    const int64_t o = (int64_t)blockIdx.x * 256 + threadIdx.x, len = (int64_t)M * N;
    if (o >= len) return;
    float s = 0.f;
#pragma unroll 8
    for (int z = 0; z < splits; ++z) s += W[z * len + o];
    float *p = C + o / N * ldc + o % N;
    *p = alpha * s + (beta != 0.f ? beta * *p : 0.f);
}

// Gram matrix of l vectors of length K in FP64 (FP32 elements, whose products
// are exact): element k of vector i at P[i * rs + k * ks].  A workgroup owns a
// 64 x 64 block for a share of k (blockIdx.z of `splits`), 4 x 4 entries a
// thread, and leaves its sums in W[split][l][l]; k_gram_sum adds them in order.
// FP64 because the factor of a Gram matrix resolves singular values only down
// to the root of its rounding: 5e-4 of the largest in FP32, which is where a
// smooth family's spectrum goes on, 1e-7 in FP64, where the FP32 samples end.
template <int MODE>
__global__ void __launch_bounds__(256)
k_gram(int l, int K, const float *__restrict__ P, int64_t rs, int64_t ks, int splits, double *__restrict__ W)
{
    __shared__ __align__(16) float As[kLds], Bs[kLds];
    const int t = threadIdx.x, ty = t >> 4, tx = t & 15, i0 = blockIdx.y * kTile, j0 = blockIdx.x * kTile;
    const int steps = (K + kTK - 1) / kTK, z = blockIdx.z;
    const int s0 = (int)((int64_t)steps * z / splits), s1 = (int)((int64_t)steps * (z + 1) / splits);
    double acc[4][4] = {};
    Tile<MODE> ta, tb;
    for (int s = s0; s < s1; ++s) {
        ta.load(t, P, rs, ks, i0, l, s * kTK, K);
        tb.load(t, P, rs, ks, j0, l, s * kTK, K);
        __syncthreads();  // the last step's tiles are no longer read
        ta.store(t, As);
        tb.store(t, Bs);
        __syncthreads();
#pragma unroll 4
        for (int k = 0; k < kTK; ++k) {
            double a[4], b[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                a[e] = MODE == LD_MC ? As[k * kPM + ty * 4 + e] : As[(ty * 4 + e) * kPK + k];
                b[e] = MODE == LD_MC ? Bs[k * kPM + tx * 4 + e] : Bs[(tx * 4 + e) * kPK + k];
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int f = 0; f < 4; ++f) acc[e][f] += a[e] * b[f];
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            const int i = i0 + ty * 4 + e, j = j0 + tx * 4 + f;
            if (i < l && j < l) W[((int64_t)z * l + i) * l + j] = acc[e][f];
        }
}

__global__ void __launch_bounds__(256)
k_gram_sum(int ll, int splits, const double *__restrict__ W, double *__restrict__ G)
{
    const int o = blockIdx.x * 256 + threadIdx.x;
    if (o >= ll) return;
    double s = 0.0;
#pragma unroll 8
    for (int z = 0; z < splits; ++z) s += W[(int64_t)z * ll + o];
    G[o] = s;
}

// Column means of Y (N x D, leading dimension ld) and Y -= mean: FP64 sums
// of `per` rows each (part[chunk * D + j]), added in order.
__global__ void __launch_bounds__(256)
k_center_part(int64_t N, int64_t D, int per, const float *__restrict__ Y, int64_t ld, double *__restrict__ part)
{
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x, i0 = (int64_t)blockIdx.y * per;
    if (j >= D) return;
    const int rows = (int)min((int64_t)per, N - i0);
    double s = 0.0;
#pragma unroll 16
    for (int i = 0; i < rows; ++i) s += Y[(i0 + i) * ld + j];
    part[blockIdx.y * D + j] = s;
}

__global__ void __launch_bounds__(256)
k_center_mean(int64_t N, int64_t D, int chunks, const double *__restrict__ part, float *__restrict__ mean)
{
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= D) return;
    double s = 0.0;
#pragma unroll 8
    for (int c = 0; c < chunks; ++c) s += part[c * D + j];
    mean[j] = (float)(s / (double)N);
}

__global__ void __launch_bounds__(256)
k_center(int64_t N, int64_t D, int per, float *__restrict__ Y, int64_t ld, const float *__restrict__ mean)
{
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x, i0 = (int64_t)blockIdx.y * per;
    if (j >= D) return;
    const float mu = mean[j];
    const int rows = (int)min((int64_t)per, N - i0);
#pragma unroll 16
    for (int i = 0; i < rows; ++i) Y[(i0 + i) * ld + j] -= mu;
}

// Gaussian matrix from a counter-based generator: splitmix64 of
// (seed, index) gives two uniforms, Box-Muller turns them into N(0,1).
__device__ __forceinline__ uint64_t splitmix64(uint64_t x)
{
    x += 0x9E3779B97F4A7C15ull;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}

__device__ __forceinline__ double gauss(uint64_t seed, int64_t t)
{
    const uint64_t r = splitmix64(seed ^ splitmix64((uint64_t)t));
    const double u1 = ((r >> 11) + 1.0) * (1.0 / 9007199254740993.0);  // (0, 1]
    const double u2 = (double)(splitmix64(r) >> 11) * (1.0 / 9007199254740992.0);
    return sqrt(-2.0 * log(u1)) * cos(6.283185307179586 * u2);
}

__global__ void __launch_bounds__(256) k_gauss(int64_t len, uint64_t seed, float *__restrict__ out)
{
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t < len) out[t] = (float)gauss(seed, t);
}

// A random vector of about unit length: out[t * stride] for t < len.
__global__ void __launch_bounds__(256)
k_gauss_unit(int64_t len, int64_t stride, uint64_t seed, float *__restrict__ out)
{
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t < len) out[t * stride] = (float)(gauss(seed, t) / sqrt((double)len));
}

// y_i += v (row-broadcast add): Y (N x D, ld).
__global__ void __launch_bounds__(256)
k_add_row(int64_t N, int64_t D, float *__restrict__ Y, int64_t ld, const float *__restrict__ v)
{
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= N * D) return;
    const int64_t i = t / D, j = t % D;
    Y[i * ld + j] += v[j];
}

__global__ void __launch_bounds__(256)
k_mul_row(int64_t N, int64_t D, float *__restrict__ Y, int64_t ld, const float *__restrict__ v)
{
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= N * D) return;
    const int64_t i = t / D, j = t % D;
    Y[i * ld + j] *= v[j];
}

// Eigen-decomposition of a symmetric l x l matrix by Jacobi rotations, a
// launch per round of l / 2 disjoint rotations (a round-robin of the index
// pairs: l - 1 rounds are a sweep).  A thread owns the 2 x 2 block of two
// pairs, (p_i, q_i) x (p_j, q_j), or the entries of one row of V in a pair's
// columns; S is read from one buffer and written to the other, so every
// thread can form the rotations it needs from the diagonal blocks.
// What bounds it: the rounds' launches, about 4 us each (l = 128: eight
// sweeps of 127), against the host's rotations one by one (l = 128 about 17
// ms, l = 288 over 200 ms).
struct Rot {
    int p, q;
    double c, s;
};

// Pair i of a round among L (even) indices: index L - 1 meets `round`, the
// others pair up around it.  An index past l - 1 (l odd) rests.
__device__ __forceinline__ Rot jacobi_rot(int l, int L, int round, int i, const double *__restrict__ S)
{
    const int w = L - 1;
    Rot r;
    int a = i == 0 ? w : (round + i) % w, b = i == 0 ? round : (round - i + w) % w;
    r.p = min(a, b);
    r.q = max(a, b);
    r.c = 1.0;
    r.s = 0.0;
    if (r.q >= l) return r;
    const double apq = S[(size_t)r.p * l + r.q];
    if (fabs(apq) < 1e-300) return r;
    const double theta = (S[(size_t)r.q * l + r.q] - S[(size_t)r.p * l + r.p]) / (2.0 * apq);
    const double t = (theta >= 0.0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
    r.c = 1.0 / sqrt(t * t + 1.0);
    r.s = t * r.c;
    return r;
}

__global__ void __launch_bounds__(256)
k_jacobi(int l, int L, int round, const double *__restrict__ S, double *__restrict__ T, double *__restrict__ V)
{
    const int h = L / 2, n = blockIdx.x * 256 + threadIdx.x;
    if (n < h * h) {
        const int i = n / h, j = n % h;
        const Rot a = jacobi_rot(l, L, round, i, S), b = jacobi_rot(l, L, round, j, S);
        const bool qi = a.q < l, qj = b.q < l;  // p is always an index
        const double *P = S + (size_t)a.p * l, *Q = S + (size_t)a.q * l;
        const double pp = P[b.p], pq = qj ? P[b.q] : 0.0, qp = qi ? Q[b.p] : 0.0, qq = qi && qj ? Q[b.q] : 0.0;
        const double up = a.c * pp - a.s * qp, uq = a.c * pq - a.s * qq;   // rows
        const double dp = a.s * pp + a.c * qp, dq = a.s * pq + a.c * qq;
        T[(size_t)a.p * l + b.p] = b.c * up - b.s * uq;                    // columns
        if (qj) T[(size_t)a.p * l + b.q] = b.s * up + b.c * uq;
        if (qi) T[(size_t)a.q * l + b.p] = b.c * dp - b.s * dq;
        if (qi && qj) T[(size_t)a.q * l + b.q] = b.s * dp + b.c * dq;
        return;
    }
    const int m = n - h * h, k = m / h, j = m % h;
    if (k >= l) return;
    const Rot b = jacobi_rot(l, L, round, j, S);
    if (b.q >= l) return;
    double *R = V + (size_t)k * l;
    const double x = R[b.p], y = R[b.q];
    R[b.p] = b.c * x - b.s * y;
    R[b.q] = b.s * x + b.c * y;
}

__global__ void __launch_bounds__(256)
k_jacobi_init(int l, const double *__restrict__ G, double *__restrict__ S, double *__restrict__ V)
{
    const int n = blockIdx.x * 256 + threadIdx.x;
    if (n >= l * l) return;
    S[n] = G[n];
    V[n] = n / l == n % l ? 1.0 : 0.0;
}

// out[0] = sum of the off-diagonal squares, out[1] = of all (one workgroup).
__global__ void __launch_bounds__(uv::kWG) k_jacobi_off(int l, const double *__restrict__ S, double *__restrict__ out)
{
    double v[2] = {0.0, 0.0};
    for (int n = threadIdx.x; n < l * l; n += uv::kWG) {
        const double q = S[n] * S[n];
        v[1] += q;
        if (n / l != n % l) v[0] += q;
    }
    uv::block_sum<2>(v, out, 1);
}

inline unsigned nblk(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

// Workspace of a product: `floats` values for the blocks' sums of a split k
// (none: k is split within the workgroups only).
struct GemmWork {
    float *p;
    size_t floats;
};

Load load_mode(int64_t rs, int64_t ks) { return ks == 1 ? LD_KC : rs == 1 ? LD_MC : LD_EL; }

template <int AM, int BM>
void gemm_launch(bool wide, dim3 g, hipStream_t st, int M, int N, int K, const float *A, int64_t a_rs, int64_t a_cs,
                 const float *B, int64_t b_rs, int64_t b_cs, float *C, int64_t ldc, float alpha, float beta,
                 int splits, float *W)
{
#define UV_GEMM_ARGS M, N, K, A, a_rs, a_cs, B, b_rs, b_cs, C, ldc, alpha, beta, splits, W
    if (wide) k_gemm_f32<AM, BM, 4><<<g, 1024, 0, st>>>(UV_GEMM_ARGS);
    else k_gemm_f32<AM, BM, 1><<<g, 256, 0, st>>>(UV_GEMM_ARGS);
}

template <int AM>
void gemm_b(Load bm, bool wide, dim3 g, hipStream_t st, int M, int N, int K, const float *A, int64_t a_rs, int64_t a_cs,
            const float *B, int64_t b_rs, int64_t b_cs, float *C, int64_t ldc, float alpha, float beta, int splits,
            float *W)
{
    if (bm == LD_KC) gemm_launch<AM, LD_KC>(wide, g, st, UV_GEMM_ARGS);
    else if (bm == LD_MC) gemm_launch<AM, LD_MC>(wide, g, st, UV_GEMM_ARGS);
    else gemm_launch<AM, LD_EL>(wide, g, st, UV_GEMM_ARGS);
}

int gemm(hipStream_t st, int M, int N, int K, const float *A, int64_t a_rs, int64_t a_cs, const float *B,
         int64_t b_rs, int64_t b_cs, float *C, int64_t ldc, float alpha, float beta, GemmWork work = {nullptr, 0})
{
    if (M <= 0 || N <= 0) return UV_OK;
    dim3 g(nblk(N, kTile), nblk(M, kTile));
    const int64_t tiles = (int64_t)g.x * g.y;
    // Too few blocks of C for the chip's 256 compute units: split k, with
    // at least eight steps a share (over the grid where there is a
    // workspace, and within a workgroup where that leaves few of them).
    const int steps = (K + kTK - 1) / kTK;
    int64_t splits = std::min<int64_t>({(1024 + tiles - 1) / tiles, steps / 8, (int64_t)(work.floats / ((size_t)M * N)), 256});
    splits = work.p ? std::max<int64_t>(splits, 1) : 1;
    const bool wide = tiles * splits < 512 && steps / splits >= 16;
    g.z = (unsigned)splits;
    const Load am = load_mode(a_rs, a_cs), bm = load_mode(b_cs, b_rs);
    float *W = splits > 1 ? work.p : nullptr;
    {
        const int sp = (int)splits;
#define UV_G M, N, K, A, a_rs, a_cs, B, b_rs, b_cs, C, ldc, alpha, beta, sp, W
        if (am == LD_KC) gemm_b<LD_KC>(bm, wide, g, st, UV_G);
        else if (am == LD_MC) gemm_b<LD_MC>(bm, wide, g, st, UV_G);
        else gemm_b<LD_EL>(bm, wide, g, st, UV_G);
#undef UV_G
        if (sp > 1) k_gemm_sum<<<nblk((int64_t)M * N, 256), 256, 0, st>>>(M, N, sp, W, C, ldc, alpha, beta);
    }
#undef UV_GEMM_ARGS
    return hipGetLastError() == hipSuccess ? UV_OK : UV_EHIP;
}

// ---- host-side small dense factorizations (l x l, row-major) ----

// Lower Cholesky G = L L' of an FP64 Gram matrix, over G.  A column whose
// pivot is at the rounding level of the products (1e-14 of the largest
// diagonal entry: a singular value under 1e-7 of the largest) has no
// direction of its own left: it goes to `lost` and its row and column of L
// are the identity's.  Returns the smallest other pivot over the largest
// diagonal entry.
double chol_lower(std::vector<double> &G, int l, std::vector<int> &lost)
{
    double scale = 0.0, least = 1.0;
    for (int i = 0; i < l; ++i) scale = std::max(scale, G[(size_t)i * l + i]);
    lost.clear();
    for (int j = 0; j < l; ++j) {
        double d = G[(size_t)j * l + j];
        for (int k = 0; k < j; ++k) d -= G[(size_t)j * l + k] * G[(size_t)j * l + k];
        const bool gone = !(d > 1e-14 * scale);
        if (gone) {
            lost.push_back(j);
            for (int k = 0; k < j; ++k) G[(size_t)j * l + k] = 0.0;
            d = 1.0;
        } else {
            least = std::min(least, d / scale);
        }
        d = std::sqrt(d);
        G[(size_t)j * l + j] = d;
        for (int i = j + 1; i < l; ++i) {
            double s = G[(size_t)i * l + j];
            for (int k = 0; k < j; ++k) s -= G[(size_t)i * l + k] * G[(size_t)j * l + k];
            G[(size_t)i * l + j] = gone ? 0.0 : s / d;
        }
        for (int k = j + 1; k < l; ++k) G[(size_t)j * l + k] = 0.0;
    }
    return least;
}

// Inverse of a lower-triangular matrix (forward substitution, a row of the
// inverse at a time).
std::vector<double> inv_lower(const std::vector<double> &L, int l)
{
    std::vector<double> X((size_t)l * l, 0.0);
    for (int i = 0; i < l; ++i) {
        double *x = X.data() + (size_t)i * l;
        x[i] = 1.0;
        for (int k = 0; k < i; ++k) {
            const double f = L[(size_t)i * l + k], *y = X.data() + (size_t)k * l;
            for (int c = 0; c <= k; ++c) x[c] -= f * y[c];
        }
        for (int c = 0; c <= i; ++c) x[c] /= L[(size_t)i * l + i];
    }
    return X;
}

// Largest l whose eigenproblem is left to the host: its time grows as l^3, the
// device's as l with about 4 us a round.  A fit of 300 x 3000 samples, device /
// host, us: l = 16 1277 / 869, 32 1786 / 1150, 48 2398 / 1605, 64 3087 / 2774 (2552
// / 2572 with a falling spectrum), 72 3722 / 3577 (3071 / 2980), 80 3885 / 4732, 128
// 6747 / 20329.
constexpr int kHostEig = 64;

// Eigenvalues (descending) and eigenvectors (columns of the row-major V) of
// the symmetric l x l matrix G, by k_jacobi; dev: 3 l^2 + 2 doubles of
// device scratch.
int sym_eig_device(int l, const double *G, double *dev, std::vector<double> &w, std::vector<double> &V, hipStream_t st)
{
    const size_t ll = (size_t)l * l;
    double *S = dev, *T = dev + ll, *Vd = dev + 2 * ll, *off = dev + 3 * ll;
    k_jacobi_init<<<nblk(ll, 256), 256, 0, st>>>(l, G, S, Vd);
    const int L = (l + 1) / 2 * 2, h = L / 2;
    const unsigned g = nblk((int64_t)h * h + (int64_t)h * l, 256);
    for (int sweep = 0; sweep < 100 && l > 1; ++sweep) {
        if (sweep == 0 || sweep >= 5) {  // as the host routine: stop at off <= 1e-30 of the whole
            double o[2];
            k_jacobi_off<<<1, uv::kWG, 0, st>>>(l, S, off);
            if (hipMemcpyAsync(o, off, sizeof(o), hipMemcpyDeviceToHost, st) != hipSuccess ||
                hipStreamSynchronize(st) != hipSuccess)
                return UV_EHIP;
            if (!(o[0] > 1e-30 * std::max(o[1], 1e-300))) break;
        }
        for (int round = 0; round < L - 1; ++round) {
            k_jacobi<<<g, 256, 0, st>>>(l, L, round, S, T, Vd);
            std::swap(S, T);
        }
    }
    std::vector<double> Sh(ll), Vh(ll);
    if (hipGetLastError() != hipSuccess ||
        hipMemcpyAsync(Sh.data(), S, 8 * ll, hipMemcpyDeviceToHost, st) != hipSuccess ||
        hipMemcpyAsync(Vh.data(), Vd, 8 * ll, hipMemcpyDeviceToHost, st) != hipSuccess ||
        hipStreamSynchronize(st) != hipSuccess)
        return UV_EHIP;
    std::vector<int> idx(l);
    for (int i = 0; i < l; ++i) idx[i] = i;
    std::sort(idx.begin(), idx.end(), [&](int a, int b) { return Sh[(size_t)a * l + a] > Sh[(size_t)b * l + b]; });
    for (int c = 0; c < l; ++c) {
        w[c] = Sh[(size_t)idx[c] * l + idx[c]];
        for (int r = 0; r < l; ++r) V[(size_t)r * l + c] = Vh[(size_t)r * l + idx[c]];
    }
    return UV_OK;
}

}  // namespace

extern "C" {

// Symmetric eigen-decomposition by cyclic Jacobi rotations: S (l x l,
// row-major, destroyed) -> eigenvalues w (descending) and eigenvectors as
// the columns of V (row-major l x l).
int uvla_sym_eig(int32_t l, double *S, double *w, double *V)
{
    if (l < 1 || !S || !w || !V) return UV_EINVAL;
    for (int i = 0; i < l; ++i)
        for (int j = 0; j < l; ++j) V[(size_t)i * l + j] = (i == j) ? 1.0 : 0.0;
    for (int sweep = 0; sweep < 100; ++sweep) {
        double off = 0.0, tot = 0.0;
        for (int i = 0; i < l; ++i)
            for (int j = 0; j < l; ++j) {
                const double v = S[(size_t)i * l + j] * S[(size_t)i * l + j];
                tot += v;
                if (i != j) off += v;
            }
        if (off <= 1e-30 * std::max(tot, 1e-300)) break;
        for (int p = 0; p < l - 1; ++p) {
            for (int q = p + 1; q < l; ++q) {
                const double apq = S[(size_t)p * l + q];
                if (std::fabs(apq) < 1e-300) continue;
                const double app = S[(size_t)p * l + p], aqq = S[(size_t)q * l + q];
                const double theta = (aqq - app) / (2.0 * apq);
                const double t = (theta >= 0 ? 1.0 : -1.0) / (std::fabs(theta) + std::sqrt(theta * theta + 1.0));
                const double cs = 1.0 / std::sqrt(t * t + 1.0), sn = t * cs;
                for (int k = 0; k < l; ++k) {  // rows p, q
                    const double a = S[(size_t)p * l + k], b = S[(size_t)q * l + k];
                    S[(size_t)p * l + k] = cs * a - sn * b;
                    S[(size_t)q * l + k] = sn * a + cs * b;
                }
                for (int k = 0; k < l; ++k) {  // columns p, q
                    const double a = S[(size_t)k * l + p], b = S[(size_t)k * l + q];
                    S[(size_t)k * l + p] = cs * a - sn * b;
                    S[(size_t)k * l + q] = sn * a + cs * b;
                }
                for (int k = 0; k < l; ++k) {
                    const double a = V[(size_t)k * l + p], b = V[(size_t)k * l + q];
                    V[(size_t)k * l + p] = cs * a - sn * b;
                    V[(size_t)k * l + q] = sn * a + cs * b;
                }
            }
        }
    }
    // sort descending
    std::vector<int> idx(l);
    for (int i = 0; i < l; ++i) idx[i] = i;
    std::sort(idx.begin(), idx.end(), [&](int a, int b) { return S[(size_t)a * l + a] > S[(size_t)b * l + b]; });
    std::vector<double> Vs((size_t)l * l);
    for (int c = 0; c < l; ++c) {
        w[c] = S[(size_t)idx[c] * l + idx[c]];
        for (int r = 0; r < l; ++r) Vs[(size_t)r * l + c] = V[(size_t)r * l + idx[c]];
    }
    std::memcpy(V, Vs.data(), sizeof(double) * l * l);
    return UV_OK;
}

int gemm_f32(int32_t M, int32_t N, int32_t K, const float *A, int64_t a_rs, int64_t a_cs, const float *B,
             int64_t b_rs, int64_t b_cs, float *C, int64_t ldc, float alpha, float beta, void *stream)
{
    if (M < 0 || N < 0 || K < 0 || !A || !B || !C) return UV_EINVAL;
    int rc = gemm((hipStream_t)stream, M, N, K, A, a_rs, a_cs, B, b_rs, b_cs, C, ldc, alpha, beta);
    if (rc != UV_OK) return rc;
    return hipStreamSynchronize((hipStream_t)stream) == hipSuccess ? UV_OK : UV_EHIP;
}

int add_row_vector(int64_t N, int64_t D, float *Y, int64_t ld, const float *v, void *stream)
{
    if (!Y || !v || N < 0 || D < 0) return UV_EINVAL;
    if (N * D == 0) return UV_OK;
    k_add_row<<<nblk(N * D, 256), 256, 0, (hipStream_t)stream>>>(N, D, Y, ld, v);
    if (hipGetLastError() != hipSuccess) return UV_EHIP;
    return hipStreamSynchronize((hipStream_t)stream) == hipSuccess ? UV_OK : UV_EHIP;
}

int mul_row_vector(int64_t N, int64_t D, float *Y, int64_t ld, const float *v, void *stream)
{
    if (!Y || !v || N < 0 || D < 0 || (N > 0 && ld < D)) return UV_EINVAL;
    if (N * D == 0) return UV_OK;
    k_mul_row<<<nblk(N * D, 256), 256, 0, (hipStream_t)stream>>>(N, D, Y, ld, v);
    if (hipGetLastError() != hipSuccess) return UV_EHIP;
    return hipStreamSynchronize((hipStream_t)stream) == hipSuccess ? UV_OK : UV_EHIP;
}

int pca_fit(float *Y, int64_t N, int64_t D, int64_t ld, int32_t k, int32_t oversample, int32_t power_iters,
            uint64_t seed, float *mean, float *basis, float *sv, void *stream)
{
    if (!Y || !mean || !basis || !sv || N < 1 || D < 1 || ld < D || k < 1 || oversample < 0 || power_iters < 0)
        return UV_EINVAL;
    const int l = (int)std::min<int64_t>(std::min<int64_t>(k + oversample, N), D);
    if (k > l || l > 1024 || N >= ((int64_t)1 << 31) || D >= ((int64_t)1 << 31)) return UV_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    // one allocation: Om and W (D x l), Z (N x l), G (l x l, FP64) and R (l x
    // l), Bm (l x D), Tm (max(N, D) x l), the centring's partial sums, the
    // eigen-decomposition's matrices and the products' workspace (a product is
    // split while it has fewer than 1024 blocks of C)
    const int per = (int)std::max<int64_t>(64, (N + 1023) / 1024), chunks = (int)((N + per - 1) / per);
    const size_t nl = (size_t)N * l, dl = (size_t)D * l, ll = (size_t)l * l;
    const size_t wlen = (size_t)2048 * kTile * kTile;
    float *base = nullptr;
    size_t len = 0;
    auto room = [&](size_t floats) {
        const size_t at = len;
        len += (floats + 63) / 64 * 64;
        return at;
    };
    const size_t oOm = room(dl), oZ = room(nl), oW = room(dl), oG = room(2 * ll), oR = room(ll), oB = room(dl),
                 oT = room(std::max(nl, dl)), oP = room(2 * (size_t)chunks * D), oE = room(6 * ll + 4), oS = room(wlen);
    if (uv::dev_malloc(&base, sizeof(float) * len) != hipSuccess) return UV_ENOMEM;
    float *Om = base + oOm, *Z = base + oZ, *W = base + oW, *R = base + oR, *Bm = base + oB, *Tm = base + oT;
    double *G = (double *)(base + oG), *part = (double *)(base + oP), *eig = (double *)(base + oE);
    const GemmWork work{base + oS, wlen};
    auto cleanup = [&]() { (void)hipFree(base); };
    int rc = UV_OK;
    std::vector<float> rh(ll);
    std::vector<double> gd(ll);
    std::vector<int> lost;
    uint64_t drawn = 0;  // random columns so far
    // FP64 Gram matrix of c vectors (vector i, element e at X[i * rs + e * es])
    // into G and gd; whether it is finite
    auto gram = [&](const float *X, int c, int64_t rs, int64_t es, int64_t rows, bool &finite) -> int {
        const unsigned g = nblk(c, kTile);
        const int steps = (int)((rows + kTK - 1) / kTK);
        const int64_t most = (int64_t)(wlen / 2) / ((int64_t)c * c);  // at least four for c = 1024
        const int splits = (int)std::max<int64_t>(1, std::min<int64_t>({(512 + g * g - 1) / (g * g), steps / 4, most}));
        double *sums = (double *)(base + oS);
        if (rs == 1) k_gram<LD_MC><<<dim3(g, g, splits), 256, 0, st>>>(c, (int)rows, X, rs, es, splits, sums);
        else k_gram<LD_KC><<<dim3(g, g, splits), 256, 0, st>>>(c, (int)rows, X, rs, es, splits, sums);
        k_gram_sum<<<nblk((int64_t)c * c, 256), 256, 0, st>>>(c * c, splits, sums, G);
        const size_t cc = (size_t)c * c;
        if (hipGetLastError() != hipSuccess ||
            hipMemcpyAsync(gd.data(), G, sizeof(double) * cc, hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess)
            return UV_EHIP;
        finite = true;
        for (size_t t = 0; t < cc; ++t) finite = finite && std::isfinite(gd[t]);
        return UV_OK;
    };
    // Orthonormalizes c vectors of length rows, the columns of a row-major
    // rows x c matrix or (`byrow`) the rows of a c x rows one: X <- X L^{-T}
    // with X'X = L L' (Cholesky QR), twice at least, until the Gram matrix was
    // that of well-conditioned vectors.  A vector without a direction of its
    // own is replaced by a random one, which the next pass makes orthogonal to
    // the others.  Samples with NaN or Inf leave NaN.
    auto orth = [&](float *X, int c, int64_t rows, bool byrow) -> int {
        for (int pass = 0; pass < 8; ++pass) {
            bool finite = false;
            int r = byrow ? gram(X, c, rows, 1, rows, finite) : gram(X, c, 1, c, rows, finite);
            if (r != UV_OK) return r;
            if (byrow && pass == 0 && finite) {  // the rows of the basis mostly are orthonormal as they come
                double off = 0.0;
                for (int i = 0; i < c; ++i)
                    for (int j = 0; j < c; ++j) off = std::max(off, std::fabs(gd[(size_t)i * c + j] - (i == j ? 1.0 : 0.0)));
                if (off <= 4e-6) return UV_OK;
            }
            const double least = finite ? chol_lower(gd, c, lost) : 1.0;
            const std::vector<double> Li = finite ? inv_lower(gd, c) : std::vector<double>((size_t)c * c, std::nan(""));
            for (int i = 0; i < c; ++i)  // R^{-1} = (L^{-1})' for columns, L^{-1} for rows
                for (int j = 0; j < c; ++j) rh[(size_t)i * c + j] = (float)(byrow ? Li[(size_t)i * c + j] : Li[(size_t)j * c + i]);
            if (hipMemcpyAsync(R, rh.data(), sizeof(float) * c * c, hipMemcpyHostToDevice, st) != hipSuccess)
                return UV_EHIP;
            // through the scratch Tm (max(N, D) x l)
            r = byrow ? gemm(st, c, (int)rows, c, R, c, 1, X, rows, 1, Tm, rows, 1.f, 0.f, work)
                      : gemm(st, (int)rows, c, c, X, c, 1, R, c, 1, Tm, c, 1.f, 0.f, work);
            if (r != UV_OK) return r;
            if (hipMemcpyAsync(X, Tm, sizeof(float) * rows * c, hipMemcpyDeviceToDevice, st) != hipSuccess)
                return UV_EHIP;
            if (!finite) return UV_OK;
            for (int j : lost)
                k_gauss_unit<<<nblk(rows, 256), 256, 0, st>>>(rows, byrow ? 1 : c, seed + 0x632be59bd9b4e019ull * ++drawn,
                                                              X + (byrow ? j * rows : j));
            if (pass > 0 && lost.empty() && least >= 0.01) break;
        }
        return UV_OK;
    };
    do {
        const dim3 gc(nblk(D, 256), (unsigned)chunks);
        k_center_part<<<gc, 256, 0, st>>>(N, D, per, Y, ld, part);
        k_center_mean<<<gc.x, 256, 0, st>>>(N, D, chunks, part, mean);
        k_center<<<gc, 256, 0, st>>>(N, D, per, Y, ld, mean);
        k_gauss<<<nblk(D * l, 256), 256, 0, st>>>(D * l, seed, Om);
        if (hipGetLastError() != hipSuccess) { rc = UV_EHIP; break; }
        if ((rc = gemm(st, (int)N, l, (int)D, Y, ld, 1, Om, l, 1, Z, l, 1.f, 0.f, work)) != UV_OK) break;   // Z = Y Om
        for (int q = 0; q < power_iters && rc == UV_OK; ++q) {
            if ((rc = orth(Z, l, N, false)) != UV_OK) break;
            if ((rc = gemm(st, (int)D, l, (int)N, Y, 1, ld, Z, l, 1, W, l, 1.f, 0.f, work)) != UV_OK) break;  // W = Y'Z
            if ((rc = orth(W, l, D, false)) != UV_OK) break;
            rc = gemm(st, (int)N, l, (int)D, Y, ld, 1, W, l, 1, Z, l, 1.f, 0.f, work);                          // Z = Y W
        }
        if (rc != UV_OK) break;
        if ((rc = orth(Z, l, N, false)) != UV_OK) break;
        if ((rc = gemm(st, l, (int)D, (int)N, Z, 1, l, Y, ld, 1, Bm, D, 1.f, 0.f, work)) != UV_OK) break;   // Bm = Z'Y
        bool finite = false;
        if ((rc = gram(Bm, l, D, 1, D, finite)) != UV_OK) break;                                             // G = Bm Bm'
        std::vector<double> w(l, std::nan("")), V(ll, std::nan(""));
        if (finite && l <= kHostEig) uvla_sym_eig(l, gd.data(), w.data(), V.data());
        else if (finite && (rc = sym_eig_device(l, G, eig, w, V, st)) != UV_OK) break;
        // basis row c = (V[:, c]' Bm) / sigma_c for the top k
        std::vector<float> P((size_t)k * l);
        for (int c = 0; c < k; ++c) {
            const double sg = std::sqrt(std::max(w[c], 0.0));
            sv[c] = (float)sg;
            const double inv = sg > 0 ? 1.0 / sg : 0.0;
            for (int r = 0; r < l; ++r) P[(size_t)c * l + r] = (float)(V[(size_t)r * l + c] * inv);
        }
        if (hipMemcpyAsync(R, P.data(), sizeof(float) * k * l, hipMemcpyHostToDevice, st) != hipSuccess) { rc = UV_EHIP; break; }
        rc = gemm(st, k, (int)D, l, R, l, 1, Bm, D, 1, basis, D, 1.f, 0.f, work);
        if (rc == UV_OK) rc = orth(basis, k, D, true);  // small singular values leave their rows rough, zeros none at all
        if (rc == UV_OK && hipStreamSynchronize(st) != hipSuccess) rc = UV_EHIP;
    } while (false);
    if (hipStreamSynchronize(st) != hipSuccess && rc == UV_OK) rc = UV_EHIP;
    cleanup();
    return rc;
}

}  // extern "C"
