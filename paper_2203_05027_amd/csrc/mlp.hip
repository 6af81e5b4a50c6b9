// mlp.hip -- the learned warm start's network: a multilayer perceptron
// (ReLU hidden layers, linear output) whose GEMMs run on gfx950's BF16
// matrix cores (v_mfma_f32_16x16x32_bf16, FP32 accumulation) from
// LDS-staged tiles, trained on a mean squared error with Adam.  Master
// weights, biases, gradients and the Adam moments are FP32; each GEMM reads
// BF16 copies of its operands.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <new>
#include <vector>

#include "../../include/uvadmm.h"
#include "common.hpp"

namespace {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

// FP32 -> BF16, round to nearest even (NaN stays NaN).
__device__ __forceinline__ uint16_t f2bf(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x007fffffu)) return (uint16_t)((u >> 16) | 0x40);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

enum Epi {
    EPI_F32 = 0,        // C (FP32)
    EPI_BIAS_RELU = 1,  // relu(C + bias) -> BF16 activation
    EPI_BIAS_F32 = 2,   // C + bias -> FP32 output
    EPI_MASK = 3,       // C * [act > 0] -> BF16 (gradient through a ReLU), and its column sums
    EPI_MSE = 4,        // 2 (C + bias - target) / len -> BF16, its column sums and the squared error's
    EPI_ADAM = 5,       // C is a weight gradient: the Adam step of the weights and their BF16 copy
};

// Adam's constants of one step (bias corrections c1, c2).
struct AdamStep {
    float lr, b1, b2, eps, c1, c2;
};

__device__ __forceinline__ float adam(float p, float g, float &m1, float &m2, const AdamStep &s)
{
    const float a = s.b1 * m1 + (1.f - s.b1) * g;
    const float v = s.b2 * m2 + (1.f - s.b2) * g * g;
    m1 = a;
    m2 = v;
    const float upd = s.lr * (a / s.c1) / (sqrtf(v / s.c2) + s.eps);
    return p - upd;
}

// What an epilogue reads and writes (see Epi).
struct EpiArgs {
    float *Cf;
    uint16_t *Cb;
    int64_t ldc;
    const float *bias;
    const uint16_t *act;
    const float *target;
    float scale;        // 2 / len
    float *colsum;      // [2 * block row + wave row][N]: column sums of the FP32 gradient
    double *sqerr;      // one per workgroup
    float *m1, *m2;
    AdamStep step;
};

// How a GEMM operand tile is read from global memory: 16-byte loads of
// eight elements consecutive along k (KC) or along the tile's other
// dimension (MC: m for A, n for B), or one element at a time (EL) when
// neither stride is 1 or the addresses are not 16-byte aligned.
enum LoadMode { LD_KC = 0, LD_MC = 1, LD_EL = 2 };

constexpr int kBK = 64;           // k per staged step of the 64 x 64 and larger blocks
constexpr int kDeep = 256;        // k per staged step of the 32 x 32 blocks
// LDS row pitch in elements of a BK-deep tile (16-byte aligned rows)
constexpr int pitch(int BK) { return BK + 8; }

// The loads of one operand tile (ROWS rows of the tile's m or n dimension,
// k0..k0+BK-1) of a thread: ROWS * BK / 8 / 256 chunks of eight elements, held in
// registers between the global loads and the LDS stores so that the next
// tile's loads are in flight while the current tile is multiplied.
// Element (r, k) of the operand is P[r * rs + k * ks]; rows >= R and k >= K
// are zero.  KC: chunks along k (row c / 8, k (c % 8) * 8); MC: chunks along
// the rows (k c % 64, rows (c / 64) * 8), so that the 64 lanes of a
// wavefront store their transposed elements to 64 consecutive k of one row
// (no LDS bank conflicts; lanes eight rows apart would all meet in one or
// two banks, whatever the 16-byte-aligned pitch).
template <int MODE, int ROWS, int BK>
struct TileLoad {
    static constexpr int kChunks = ROWS * BK / 8 / 256, kKC = BK / 8, kLK = pitch(BK);
    static_assert(kChunks >= 1 && ROWS * BK / 8 % 256 == 0, "whole chunks per thread");
    uint4 v[kChunks];

    __device__ __forceinline__ void load(const uint16_t *__restrict__ P, int64_t rs, int64_t ks, int r0, int R,
                                         int k0, int K)
    {
#pragma unroll
        for (int q = 0; q < kChunks; ++q) {
            const int c = threadIdx.x + q * 256;
            v[q] = uint4{0u, 0u, 0u, 0u};
            if (MODE == LD_KC) {
                const int gr = r0 + c / kKC, gk = k0 + c % kKC * 8;
                if (gr < R && gk < K) v[q] = *(const uint4 *)(P + (int64_t)gr * rs + gk);
            } else {
                const int gk = k0 + c % BK, gr = r0 + (c / BK) * 8;
                if (gr < R && gk < K) v[q] = *(const uint4 *)(P + (int64_t)gk * ks + gr);
            }
        }
    }

    // into LDS as T[row][k] (k contiguous, pitch kLK)
    __device__ __forceinline__ void store(uint16_t *__restrict__ T) const
    {
#pragma unroll
        for (int q = 0; q < kChunks; ++q) {
            const int c = threadIdx.x + q * 256;
            if (MODE == LD_KC) {
                *(uint4 *)(T + c / kKC * kLK + c % kKC * 8) = v[q];
            } else {
                const int kk = c % BK, r8 = (c / BK) * 8;
                const uint16_t *e = (const uint16_t *)&v[q];
#pragma unroll
                for (int t = 0; t < 8; ++t) T[(r8 + t) * kLK + kk] = e[t];
            }
        }
    }
};

// The element-wise form (no unit stride or unaligned operands): straight
// into LDS.
template <int ROWS, int BK>
__device__ __forceinline__ void stage_el(const uint16_t *__restrict__ P, int64_t rs, int64_t ks, int r0, int R,
                                         int k0, int K, uint16_t *__restrict__ T)
{
    for (int c = threadIdx.x; c < ROWS * BK; c += 256) {
        const int r = c / BK, kk = c % BK, gr = r0 + r, gk = k0 + kk;
        T[r * pitch(BK) + kk] = (gr < R && gk < K) ? P[(int64_t)gr * rs + (int64_t)gk * ks] : (uint16_t)0;
    }
}

// C (M x N) = A (M x K) B (K x N) on BF16 operands with FP32 accumulation;
// A(i,k) = A[i*a_rs + k*a_cs], B(k,j) = B[k*b_rs + j*b_cs]; M, N, K
// multiples of 16.  A workgroup (four wavefronts, 2 x 2) owns a block of
// (32 TM) x (32 TN) entries of C, a wavefront (16 TM) x (16 TN): TM x TN
// accumulators of the 16x16x32 MFMA.  Each BK-deep k step stages the
// block's A rows and B columns in LDS, k contiguous, from coalesced 16-byte
// loads issued during the previous step's products; lane l reads its
// operands as one 16-byte LDS load each: A[l % 16][8 (l / 16) .. +7] and
// B[8 (l / 16) .. +7][l % 16] of a 32-wide half step (zero past K), and holds
// C[4 (l / 16) .. +3][l % 16] of each tile.  Every block shape adds an entry's
// products in the same order, 32 at a time, so results do not depend on it.
template <int EPI, int TM, int TN, int BK, int AM, int BMODE>
__global__ void __launch_bounds__(256)
k_mfma_gemm(int M, int N, int K, const uint16_t *__restrict__ A, int64_t a_rs, int64_t a_cs,
            const uint16_t *__restrict__ B, int64_t b_rs, int64_t b_cs, EpiArgs x)
{
    constexpr int BM = 32 * TM, BN = 32 * TN, kLK = pitch(BK);
    constexpr bool PREFETCH = AM != LD_EL && BMODE != LD_EL;
    __shared__ __align__(16) uint16_t As[BM * kLK];
    __shared__ __align__(16) uint16_t Bs[BN * kLK];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int wm = wave >> 1, wn = wave & 1;
    const int tiles_n = (N + BN - 1) / BN;
    const int m0 = (blockIdx.x / tiles_n) * BM, n0 = (blockIdx.x % tiles_n) * BN;
    const int r = lane & 15, kq = lane >> 4;
    v4f acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
    // A tile: rows m (A(m, k) = A[m a_rs + k a_cs]); B tile: rows n (B(k, n) = B[n b_cs + k b_rs])
    TileLoad<AM == LD_EL ? LD_KC : AM, BM, BK> la;
    TileLoad<BMODE == LD_EL ? LD_KC : BMODE, BN, BK> lb;
    if (PREFETCH) {
        la.load(A, a_rs, a_cs, m0, M, 0, K);
        lb.load(B, b_cs, b_rs, n0, N, 0, K);
    }
    for (int k0 = 0; k0 < K; k0 += BK) {
        if (PREFETCH) {
            la.store(As);
            lb.store(Bs);
        } else {
            stage_el<BM, BK>(A, a_rs, a_cs, m0, M, k0, K, As);
            stage_el<BN, BK>(B, b_cs, b_rs, n0, N, k0, K, Bs);
        }
        __syncthreads();
        if (PREFETCH && k0 + BK < K) {
            la.load(A, a_rs, a_cs, m0, M, k0 + BK, K);
            lb.load(B, b_cs, b_rs, n0, N, k0 + BK, K);
        }
#pragma unroll
        for (int h = 0; h < BK / 32; ++h) {
            v8bf af[TM], bf[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i)
                af[i] = *(const v8bf *)(As + (wm * 16 * TM + i * 16 + r) * kLK + h * 32 + kq * 8);
#pragma unroll
            for (int j = 0; j < TN; ++j)
                bf[j] = *(const v8bf *)(Bs + (wn * 16 * TN + j * 16 + r) * kLK + h * 32 + kq * 8);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bf[j], acc[i][j], 0, 0, 0);
        }
        __syncthreads();
    }
    // Row by row: a wavefront's stores to one row of C follow each other (column
    // by column a 65536 x 1024 x 256 product took 130 us, so 105).
    double sq = 0.0;
    float cs[TN];  // this lane's part of the columns' sums
#pragma unroll
    for (int j = 0; j < TN; ++j) cs[j] = 0.f;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int col = n0 + wn * 16 * TN + j * 16 + r;
            if (col >= N) continue;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = m0 + wm * 16 * TM + i * 16 + kq * 4 + e;
                if (row >= M) continue;
                const int64_t o = (int64_t)row * x.ldc + col;
                float v = acc[i][j][e];
                if (EPI == EPI_F32) {
                    x.Cf[o] = v;
                } else if (EPI == EPI_BIAS_RELU) {
                    v += x.bias[col];
                    x.Cb[o] = f2bf(v > 0.f ? v : 0.f);
                } else if (EPI == EPI_BIAS_F32) {
                    x.Cf[o] = v + x.bias[col];
                } else if (EPI == EPI_MASK) {
                    v = bf2f(x.act[o]) > 0.f ? v : 0.f;
                    x.Cb[o] = f2bf(v);
                    cs[j] += v;
                } else if (EPI == EPI_MSE) {
                    const float d = v + x.bias[col] - x.target[o];
                    sq += (double)d * d;
                    const float g = x.scale * d;
                    x.Cb[o] = f2bf(g);
                    cs[j] += g;
                } else {
                    float a = x.m1[o], b = x.m2[o];
                    const float p = adam(x.Cf[o], v, a, b, x.step);
                    x.m1[o] = a;
                    x.m2[o] = b;
                    x.Cf[o] = p;
                    x.Cb[o] = f2bf(p);
                }
            }
        }
    if (EPI == EPI_MASK || EPI == EPI_MSE) {  // each column's rows of this wavefront, in a fixed order
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int col = n0 + wn * 16 * TN + j * 16 + r;
            float t = cs[j];
            t += __shfl_xor(t, 16);
            t += __shfl_xor(t, 32);
            if (kq == 0 && col < N) x.colsum[(int64_t)(m0 / BM * 2 + wm) * N + col] = t;
        }
    }
    if (EPI == EPI_MSE) uv::block_sum<1>(reinterpret_cast<double(&)[1]>(sq), x.sqerr + blockIdx.x, 1);
}

__global__ void __launch_bounds__(256) k_to_bf16(int64_t len, const float *__restrict__ x, uint16_t *__restrict__ y)
{
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t < len) y[t] = f2bf(x[t]);
}

__device__ __forceinline__ uint64_t mix64(uint64_t x)
{
    x += 0x9E3779B97F4A7C15ull;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}

// He-uniform initialisation, U(-sqrt(6/fan_in), sqrt(6/fan_in)).
__global__ void __launch_bounds__(256)
k_init(int64_t len, int fan_in, uint64_t seed, float *__restrict__ w, uint16_t *__restrict__ wb)
{
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= len) return;
    const double u = (double)(mix64(seed ^ mix64((uint64_t)t)) >> 11) * (1.0 / 9007199254740992.0);
    const float v = (float)((2.0 * u - 1.0) * sqrt(6.0 / fan_in));
    w[t] = v;
    wb[t] = f2bf(v);
}

constexpr int kMaxLayers = 16;

// The biases' part of a step, all layers in one launch: db from the
// gradient's column sums (`rows` of them per layer, added in order), then
// stored (gb) or, with `train`, Adam's step.  Workgroup 0 also adds the
// workgroups' squared errors to the loss, on the device and (if given) in
// host memory.
struct BiasArgs {
    int layers, train;
    int width[kMaxLayers], rows[kMaxLayers];
    const float *colsum[kMaxLayers];
    float *gb[kMaxLayers], *b[kMaxLayers], *mb[kMaxLayers], *vb[kMaxLayers];
    const double *sqerr;
    int nsq;
    double len;
    float *loss, *loss_host;
    AdamStep step;
};

__global__ void __launch_bounds__(256) k_bias(BiasArgs a)
{
    int j = blockIdx.x * 256 + threadIdx.x, l = 0;
    while (l < a.layers && j >= a.width[l]) j -= a.width[l++];
    if (l < a.layers) {
        float g = 0.f;
#pragma unroll 8
        for (int q = 0; q < a.rows[l]; ++q) g += a.colsum[l][(int64_t)q * a.width[l] + j];
        if (a.train) a.b[l][j] = adam(a.b[l][j], g, a.mb[l][j], a.vb[l][j], a.step);
        else a.gb[l][j] = g;
    }
    if (blockIdx.x > 0) return;
    double s[1] = {0.0};
    for (int q = threadIdx.x; q < a.nsq; q += 256) s[0] += a.sqerr[q];
    __shared__ double sum;
    uv::block_sum<1>(s, &sum, 1);
    if (threadIdx.x == 0) {
        const float loss = (float)(sum / a.len);
        *a.loss = loss;
        if (a.loss_host) *a.loss_host = loss;
    }
}

inline unsigned nb256(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

struct uv_mlp {
    int L = 0;                       // layers
    std::vector<int> d;              // widths d[0..L]
    int max_batch = 0;
    hipStream_t stream = nullptr;
    std::vector<void *> allocs;
    std::vector<float *> W, b, gW, gb, mW, vW, mb, vb;
    std::vector<uint16_t *> Wb;      // BF16 weight copies
    std::vector<uint16_t *> act;     // BF16 activations a_0 (input) .. a_{L-1}
    std::vector<uint16_t *> dzb;     // BF16 gradient w.r.t. pre-activations
    std::vector<float *> colsum;     // column sums of its FP32 values (2 per block row)
    std::vector<int> rows;           // how many the last backward pass left
    double *sqerr = nullptr;         // squared errors of the last layer's workgroups
    int nsq = 0;
    float *loss = nullptr;
    float *loss_host = nullptr;      // pinned
    int64_t step = 0;
};

namespace {

template <typename T>
T *malloc_d(uv_mlp *h, size_t count)
{
    void *p = nullptr;
    if (uv::dev_malloc(&p, std::max<size_t>(count, 1) * sizeof(T)) != hipSuccess) return nullptr;
    h->allocs.push_back(p);
    return (T *)p;
}

// Load mode of an operand whose element (r, k) is P[r * rs + k * ks]:
// 16-byte loads need a unit stride along them, the other stride a multiple
// of eight elements and a 16-byte-aligned base.
int load_mode(const uint16_t *P, int64_t rs, int64_t ks)
{
    const bool aligned = ((uintptr_t)P & 15) == 0;
    if (aligned && ks == 1 && rs % 8 == 0) return LD_KC;
    if (aligned && rs == 1 && ks % 8 == 0) return LD_MC;
    return LD_EL;
}

template <int EPI, int TM, int TN, int BK, int AM>
void gemm_launch_b(int bmode, unsigned grid, hipStream_t st, int M, int N, int K, const uint16_t *A, int64_t a_rs,
                   int64_t a_cs, const uint16_t *B, int64_t b_rs, int64_t b_cs, const EpiArgs &x)
{
#define UV_GEMM_ARGS M, N, K, A, a_rs, a_cs, B, b_rs, b_cs, x
    if (bmode == LD_KC) k_mfma_gemm<EPI, TM, TN, BK, AM, LD_KC><<<grid, 256, 0, st>>>(UV_GEMM_ARGS);
    else if (bmode == LD_MC) k_mfma_gemm<EPI, TM, TN, BK, AM, LD_MC><<<grid, 256, 0, st>>>(UV_GEMM_ARGS);
    else k_mfma_gemm<EPI, TM, TN, BK, AM, LD_EL><<<grid, 256, 0, st>>>(UV_GEMM_ARGS);
}

template <int EPI, int TM, int TN, int BK>
void gemm_launch(hipStream_t st, int M, int N, int K, const uint16_t *A, int64_t a_rs, int64_t a_cs,
                 const uint16_t *B, int64_t b_rs, int64_t b_cs, const EpiArgs &x)
{
    const unsigned grid = (unsigned)(((M + 32 * TM - 1) / (32 * TM)) * ((N + 32 * TN - 1) / (32 * TN)));
    const int am = load_mode(A, a_rs, a_cs), bm = load_mode(B, b_cs, b_rs);
    if (am == LD_KC) gemm_launch_b<EPI, TM, TN, BK, LD_KC>(bm, grid, st, UV_GEMM_ARGS);
    else if (am == LD_MC) gemm_launch_b<EPI, TM, TN, BK, LD_MC>(bm, grid, st, UV_GEMM_ARGS);
    else gemm_launch_b<EPI, TM, TN, BK, LD_EL>(bm, grid, st, UV_GEMM_ARGS);
}

// Rows (columns) of C a workgroup's block has, over 32: 128 x 128 blocks when
// they still give every CU a block, 64 x 64 blocks likewise, else 32 x 32
// with 256-deep steps: the network's own products (256 x 512 x 512) have 32
// blocks of 64 x 64 and eight steps, each a trip to memory (8.6-12 us), and
// 128 blocks of 32 x 32 with two steps (5.3 us).
int gemm_block(int M, int N)
{
    if ((int64_t)((M + 127) / 128) * ((N + 127) / 128) >= 256) return 4;
    return (int64_t)((M + 63) / 64) * ((N + 63) / 64) >= 256 ? 2 : 1;
}

template <int EPI>
int gemm_any(hipStream_t st, int M, int N, int K, const uint16_t *A, int64_t a_rs, int64_t a_cs,
             const uint16_t *B, int64_t b_rs, int64_t b_cs, const EpiArgs &x)
{
    const int b = gemm_block(M, N);
    if (b == 4) gemm_launch<EPI, 4, 4, kBK>(st, UV_GEMM_ARGS);
    else if (b == 2) gemm_launch<EPI, 2, 2, kBK>(st, UV_GEMM_ARGS);
    else gemm_launch<EPI, 1, 1, kDeep>(st, UV_GEMM_ARGS);
#undef UV_GEMM_ARGS
    return hipGetLastError() == hipSuccess ? UV_OK : UV_EHIP;
}

// The forward pass: the output into y, or (target given) straight into the
// loss's gradient.
int forward(uv_mlp *h, int batch, const float *x, float *y, const float *target)
{
    k_to_bf16<<<nb256((int64_t)batch * h->d[0]), 256, 0, h->stream>>>((int64_t)batch * h->d[0], x, h->act[0]);
    int rc = UV_OK;
    for (int l = 0; l < h->L && rc == UV_OK; ++l) {
        const int K = h->d[l], N = h->d[l + 1];
        EpiArgs e{};
        e.ldc = N;
        e.bias = h->b[l];
#define UV_MM_FWD h->stream, batch, N, K, h->act[l], K, 1, h->Wb[l], N, 1, e
        if (l < h->L - 1) {
            e.Cb = h->act[l + 1];
            rc = gemm_any<EPI_BIAS_RELU>(UV_MM_FWD);
        } else if (!target) {
            e.Cf = y;
            rc = gemm_any<EPI_BIAS_F32>(UV_MM_FWD);
        } else {
            const int b = 32 * gemm_block(batch, N);
            e.Cb = h->dzb[l];
            e.target = target;
            e.scale = 2.0f / (float)((int64_t)batch * N);
            e.colsum = h->colsum[l];
            e.sqerr = h->sqerr;
            h->rows[l] = 2 * ((batch + b - 1) / b);
            h->nsq = ((batch + b - 1) / b) * ((N + b - 1) / b);
            rc = gemm_any<EPI_MSE>(UV_MM_FWD);
        }
#undef UV_MM_FWD
    }
    return rc;
}

// The backward pass from the gradient that forward() left.  step null:
// the gradients into gW and gb; else Adam's step of every parameter.  A
// layer's weights are updated only after the gradient has passed them.
int backward(uv_mlp *h, int batch, const AdamStep *step, float *loss_host)
{
    const int L = h->L;
    int rc = UV_OK;
    for (int l = L - 1; l >= 0 && rc == UV_OK; --l) {
        const int K = h->d[l], N = h->d[l + 1];
        EpiArgs e{};
        if (l > 0) {  // dz_{l-1} = (dz_l W_l') * [a_l > 0]
            const int b = 32 * gemm_block(batch, K);
            e.ldc = K;
            e.Cb = h->dzb[l - 1];
            e.act = h->act[l];
            e.colsum = h->colsum[l - 1];
            h->rows[l - 1] = 2 * ((batch + b - 1) / b);
            rc = gemm_any<EPI_MASK>(h->stream, batch, K, N, h->dzb[l], N, 1, h->Wb[l], 1, N, e);
        }
        // dW_l = a_l' dz_l  (K x N)
        e = EpiArgs{};
        e.ldc = N;
        if (step) {
            e.Cf = h->W[l];
            e.Cb = h->Wb[l];
            e.m1 = h->mW[l];
            e.m2 = h->vW[l];
            e.step = *step;
            if (rc == UV_OK)
                rc = gemm_any<EPI_ADAM>(h->stream, K, N, batch, h->act[l], 1, K, h->dzb[l], N, 1, e);
        } else {
            e.Cf = h->gW[l];
            if (rc == UV_OK)
                rc = gemm_any<EPI_F32>(h->stream, K, N, batch, h->act[l], 1, K, h->dzb[l], N, 1, e);
        }
    }
    if (rc != UV_OK) return rc;
    BiasArgs a{};
    a.layers = L;
    a.train = step ? 1 : 0;
    int64_t total = 0;
    for (int l = 0; l < L; ++l) {
        a.width[l] = h->d[l + 1];
        a.rows[l] = h->rows[l];
        a.colsum[l] = h->colsum[l];
        a.gb[l] = h->gb[l];
        a.b[l] = h->b[l];
        a.mb[l] = h->mb[l];
        a.vb[l] = h->vb[l];
        total += h->d[l + 1];
    }
    a.sqerr = h->sqerr;
    a.nsq = h->nsq;
    a.len = (double)((int64_t)batch * h->d[L]);
    a.loss = h->loss;
    a.loss_host = loss_host;
    if (step) a.step = *step;
    k_bias<<<nb256(total), 256, 0, h->stream>>>(a);
    return hipGetLastError() == hipSuccess ? UV_OK : UV_EHIP;
}

bool dims_ok(int batch, const uv_mlp *h) { return batch >= 16 && batch % 16 == 0 && batch <= h->max_batch; }

}  // namespace

extern "C" {

void mlp_destroy(uv_mlp *h)
{
    if (!h) return;
    if (h->stream) (void)hipStreamSynchronize(h->stream);
    for (void *p : h->allocs) (void)hipFree(p);
    if (h->loss_host) (void)hipHostFree(h->loss_host);
    delete h;
}

int mlp_create(int32_t nlayers, const int32_t *dims, int32_t max_batch, uint64_t seed, void *stream, uv_mlp **out)
{
    if (!out) return UV_EINVAL;
    *out = nullptr;
    if (nlayers < 1 || nlayers > 16 || !dims || max_batch < 16 || max_batch % 16) return UV_EINVAL;
    for (int l = 0; l <= nlayers; ++l)
        if (dims[l] < 16 || dims[l] % 16 || dims[l] > 65536) return UV_EINVAL;
    uv_mlp *h = new (std::nothrow) uv_mlp();
    if (!h) return UV_ENOMEM;
    h->L = nlayers;
    h->d.assign(dims, dims + nlayers + 1);
    h->max_batch = max_batch;
    h->stream = (hipStream_t)stream;
    const int L = nlayers;
    h->W.resize(L); h->b.resize(L); h->gW.resize(L); h->gb.resize(L); h->mW.resize(L); h->vW.resize(L);
    h->mb.resize(L); h->vb.resize(L); h->Wb.resize(L); h->act.resize(L); h->dzb.resize(L);
    h->colsum.resize(L); h->rows.resize(L);
    bool ok = true;
    for (int l = 0; l < L; ++l) {
        const size_t nw = (size_t)h->d[l] * h->d[l + 1], nbias = h->d[l + 1];
        ok &= (h->W[l] = malloc_d<float>(h, nw)) != nullptr;
        ok &= (h->gW[l] = malloc_d<float>(h, nw)) != nullptr;
        ok &= (h->mW[l] = malloc_d<float>(h, nw)) != nullptr;
        ok &= (h->vW[l] = malloc_d<float>(h, nw)) != nullptr;
        ok &= (h->Wb[l] = malloc_d<uint16_t>(h, nw)) != nullptr;
        ok &= (h->b[l] = malloc_d<float>(h, nbias)) != nullptr;
        ok &= (h->gb[l] = malloc_d<float>(h, nbias)) != nullptr;
        ok &= (h->mb[l] = malloc_d<float>(h, nbias)) != nullptr;
        ok &= (h->vb[l] = malloc_d<float>(h, nbias)) != nullptr;
        ok &= (h->act[l] = malloc_d<uint16_t>(h, (size_t)max_batch * h->d[l])) != nullptr;
        ok &= (h->colsum[l] = malloc_d<float>(h, (size_t)2 * ((max_batch + 31) / 32) * h->d[l + 1])) != nullptr;
        ok &= (h->dzb[l] = malloc_d<uint16_t>(h, (size_t)max_batch * h->d[l + 1])) != nullptr;
    }
    ok &= (h->sqerr = malloc_d<double>(h, (size_t)((max_batch + 31) / 32) * ((h->d[L] + 31) / 32))) != nullptr;
    ok &= (h->loss = malloc_d<float>(h, 1)) != nullptr;
    if (ok && uv::host_malloc(&h->loss_host, sizeof(float), hipHostMallocDefault) != hipSuccess) {
        h->loss_host = nullptr;
        ok = false;
    }
    if (!ok) {
        mlp_destroy(h);
        return UV_ENOMEM;
    }
    for (int l = 0; l < L && ok; ++l) {
        const int64_t nw = (int64_t)h->d[l] * h->d[l + 1];
        k_init<<<nb256(nw), 256, 0, h->stream>>>(nw, h->d[l], seed + 0x1000003ull * (l + 1), h->W[l], h->Wb[l]);
        ok &= hipMemsetAsync(h->b[l], 0, 4 * (size_t)h->d[l + 1], h->stream) == hipSuccess;
        ok &= hipMemsetAsync(h->mW[l], 0, 4 * nw, h->stream) == hipSuccess;
        ok &= hipMemsetAsync(h->vW[l], 0, 4 * nw, h->stream) == hipSuccess;
        ok &= hipMemsetAsync(h->mb[l], 0, 4 * (size_t)h->d[l + 1], h->stream) == hipSuccess;
        ok &= hipMemsetAsync(h->vb[l], 0, 4 * (size_t)h->d[l + 1], h->stream) == hipSuccess;
    }
    ok &= hipGetLastError() == hipSuccess && hipStreamSynchronize(h->stream) == hipSuccess;
    if (!ok) {
        mlp_destroy(h);
        return UV_EHIP;
    }
    *out = h;
    return UV_OK;
}

int mlp_get_params(uv_mlp *h, float *w, float *b)
{
    if (!h) return UV_EINVAL;
    size_t ow = 0, ob = 0;
    for (int l = 0; l < h->L; ++l) {
        const size_t nw = (size_t)h->d[l] * h->d[l + 1], nbias = h->d[l + 1];
        if (w && hipMemcpy(w + ow, h->W[l], 4 * nw, hipMemcpyDeviceToHost) != hipSuccess) return UV_EHIP;
        if (b && hipMemcpy(b + ob, h->b[l], 4 * nbias, hipMemcpyDeviceToHost) != hipSuccess) return UV_EHIP;
        ow += nw;
        ob += nbias;
    }
    return UV_OK;
}

int mlp_set_params(uv_mlp *h, const float *w, const float *b)
{
    if (!h) return UV_EINVAL;
    size_t ow = 0, ob = 0;
    for (int l = 0; l < h->L; ++l) {
        const size_t nw = (size_t)h->d[l] * h->d[l + 1], nbias = h->d[l + 1];
        if (w) {
            if (hipMemcpy(h->W[l], w + ow, 4 * nw, hipMemcpyHostToDevice) != hipSuccess) return UV_EHIP;
            k_to_bf16<<<nb256(nw), 256, 0, h->stream>>>((int64_t)nw, h->W[l], h->Wb[l]);
        }
        if (b && hipMemcpy(h->b[l], b + ob, 4 * nbias, hipMemcpyHostToDevice) != hipSuccess) return UV_EHIP;
        ow += nw;
        ob += nbias;
    }
    return hipStreamSynchronize(h->stream) == hipSuccess ? UV_OK : UV_EHIP;
}

int mlp_forward(uv_mlp *h, int32_t batch, const float *x_dev, float *y_dev)
{
    if (!h || !x_dev || !y_dev || !dims_ok(batch, h)) return UV_EINVAL;
    int rc = forward(h, batch, x_dev, y_dev, nullptr);
    if (rc != UV_OK) return rc;
    return hipStreamSynchronize(h->stream) == hipSuccess ? UV_OK : UV_EHIP;
}

int mlp_gradients(uv_mlp *h, int32_t batch, const float *x_dev, const float *t_dev, float *gw, float *gb,
                  float *loss)
{
    if (!h || !x_dev || !t_dev || !dims_ok(batch, h)) return UV_EINVAL;
    int rc = forward(h, batch, x_dev, nullptr, t_dev);
    if (rc == UV_OK) rc = backward(h, batch, nullptr, nullptr);
    if (rc != UV_OK) return rc;
    if (hipStreamSynchronize(h->stream) != hipSuccess) return UV_EHIP;
    size_t ow = 0, ob = 0;
    for (int l = 0; l < h->L; ++l) {
        const size_t nw = (size_t)h->d[l] * h->d[l + 1], nbias = h->d[l + 1];
        if (gw && hipMemcpy(gw + ow, h->gW[l], 4 * nw, hipMemcpyDeviceToHost) != hipSuccess) return UV_EHIP;
        if (gb && hipMemcpy(gb + ob, h->gb[l], 4 * nbias, hipMemcpyDeviceToHost) != hipSuccess) return UV_EHIP;
        ow += nw;
        ob += nbias;
    }
    if (loss && hipMemcpy(loss, h->loss, 4, hipMemcpyDeviceToHost) != hipSuccess) return UV_EHIP;
    return UV_OK;
}

int mlp_train_step(uv_mlp *h, int32_t batch, const float *x_dev, const float *t_dev, float lr, float *loss)
{
    if (!h || !x_dev || !t_dev || !dims_ok(batch, h) || !(lr > 0.f)) return UV_EINVAL;
    const double step = (double)(h->step + 1);
    const AdamStep a{lr, 0.9f, 0.999f, 1e-8f, 1.f - (float)std::pow((double)0.9f, step),
                     1.f - (float)std::pow((double)0.999f, step)};
    int rc = forward(h, batch, x_dev, nullptr, t_dev);
    if (rc == UV_OK) rc = backward(h, batch, &a, loss ? h->loss_host : nullptr);
    if (rc != UV_OK) return rc;
    h->step += 1;
    if (loss) {
        if (hipStreamSynchronize(h->stream) != hipSuccess) return UV_EHIP;
        *loss = *h->loss_host;
    }
    return UV_OK;
}

int mlp_gemm_bf16(int32_t M, int32_t N, int32_t K, const uint16_t *A, int64_t a_rs, int64_t a_cs, const uint16_t *B,
                  int64_t b_rs, int64_t b_cs, float *C, int64_t ldc, void *stream)
{
    if (M < 16 || N < 16 || K < 16 || M % 16 || N % 16 || K % 16 || !A || !B || !C) return UV_EINVAL;
    EpiArgs e{};
    e.Cf = C;
    e.ldc = ldc;
    if (gemm_any<EPI_F32>((hipStream_t)stream, M, N, K, A, a_rs, a_cs, B, b_rs, b_cs, e) != UV_OK)
        return UV_EHIP;
    return hipStreamSynchronize((hipStream_t)stream) == hipSuccess ? UV_OK : UV_EHIP;
}

}  // extern "C"
