// Learned surrogate for the per-cell dt-advance: BF16-MFMA MLP training and
// inference, element conservation and acceptance gate.
//
// Network: features x = (ln T, ln p, Y_1..Y_N, ln dt), normalised and padded
// to 64, four hidden layers of 256 with GELU (erf form), output 64 of which
// the first N+1 are the normalised increments in an inverse hyperbolic-sine
// scale: t = o sd_o + mu_o, dY_k = S_Y sinh(t_k), dT = S_T sinh(t_N).
// Weights and activations are bfloat16, products accumulate in FP32 on the
// matrix cores (v_mfma_f32_16x16x32_bf16), biases and GELU in FP32.
// Training: mean-squared error on the normalised outputs, Adam on FP32 master
// weights.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <cmath>
#include <numeric>
#include <random>
#include <vector>

#include "mech_dev.hpp"
#include "surrogate.hpp"

namespace chem {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));   // in a caller's array

__device__ __forceinline__ uint16_t f2bf(float x) {
    uint32_t u = __float_as_uint(x);
    if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x7fffffu)) return (uint16_t)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
__device__ __forceinline__ float gelu_f(float z) {
    return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f));
}
__device__ __forceinline__ float gelu_df(float z) {
    return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) +
           z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pk_bf16(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

// Workgroup barrier for what is in LDS.  __syncthreads also waits for every
// global access of the wavefront: the weights on their way for the next layer,
// and stores that nothing in the kernel reads.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// GELU of four values as bfloat16, the bits of f2bf(gelu_f(z)).  The network
// spends more vector time here than matrix time (about 46 instructions a value
// with the library's erf, which takes both of its branches in most
// wavefronts), so a value is first formed as max(z, 0) - t Q(t), t = min(|z|,
// 5.5), Q(t) = erfc(t / sqrt 2) / 2 = 2^P(t) with P a polynomial of degree 7
// fitted on [0, 5.5] (Q within 7e-8; past 5.5 |z| Q(|z|) is below 1.1e-7).  That
// and gelu_f are within 3e-7 |z| of each other (2.2e-7 over all floats, with
// exp2 off by two units in its last place); where both ends of that interval
// round to the same bfloat16 the result is known, and only where they do not
// (some 0.1 % of the values, z < -4, and infinities) is it computed the long way.
__device__ __forceinline__ uint2 gelu_bf16x4(f32x4 z) {
    uint32_t w[4], bad = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float a = fabsf(z[r]), t = fminf(a, 5.5f);
        float P = fmaf(t, 8.47015417e-06f, -5.39036701e-05f);
        P = fmaf(t, P, -0.000421235978f);
        P = fmaf(t, P, 0.0073892721f);
        P = fmaf(t, P, -0.0526911095f);
        P = fmaf(t, P, -0.459153146f);
        P = fmaf(t, P, -1.15111089f);
        P = fmaf(t, P, -0.999999881f);
        const float g = fmaf(-t, __builtin_amdgcn_exp2f(P), fmaxf(z[r], 0.0f));
        const float d = fmaf(3e-7f, a, 1e-37f);   // and subnormal results
        w[r] = pk_bf16(g - d, g + d);
        bad |= w[r] ^ (w[r] >> 16);
    }
    if (__builtin_amdgcn_ballot_w64((bad & 0xffffu) != 0)) {
        // one copy of the long way for the four: it is rarely taken, and four
        // copies at every call made the kernels larger than the instruction cache
#pragma unroll 1
        for (int r = 0; r < 4; ++r) {
            const float zr = r == 0 ? z[0] : r == 1 ? z[1] : r == 2 ? z[2] : z[3];
            const uint32_t v = f2bf(gelu_f(zr));
            w[0] = r == 0 ? v : w[0];
            w[1] = r == 1 ? v : w[1];
            w[2] = r == 2 ? v : w[2];
            w[3] = r == 3 ? v : w[3];
        }
    }
    return {(w[0] & 0xffffu) | (w[1] << 16), (w[2] & 0xffffu) | (w[3] << 16)};
}

// Place of element (r, k) of a matrix with K columns in operand order: blocks of
// 16 rows and 32 columns, each lane's eight values in a row, lane after lane, so
// that an operand is one contiguous kilobyte.  All bf16 operands in memory
// (weights, their transposes, and what the weight gradients contract) lie so.
// Row by row, 16 lanes of a load touched 16 cache lines for 16 bytes each, and
// the address unit bound the tile kernels (forward of 100,003 rows 197 us).
__host__ __device__ __forceinline__ int64_t op_place(int64_t r, int64_t k, int64_t K) {
    return (((r >> 4) * (K >> 5) + (k >> 5)) << 9) + ((((k >> 3) & 3) << 4) + (r & 15)) * 8 + (k & 7);
}

// ------------------------------------------------------------ tile layers ----
// One layer for a tile of 16 RB rows in one workgroup of four wavefronts: a
// wavefront takes NBK blocks of 16 output columns from n0, with 16x16x32 MFMA
// blocks accumulating over k in order.  Operands (gfx950, checked on hardware):
// lane l holds A row l%16, k = 8(l/16)..+7; B column l%16, same k; D rows
// 4(l/16)+i, column l%16.  The weights are the A operand, so a lane's four
// results are four neighbouring columns of one batch row and leave in one
// store.  The weights of a layer (K x 16 NBK per wavefront) are loaded in one
// go, ahead of the previous layer's activation function, which covers their
// way from L2.
template <int K, int NBK>
struct WTile {
    bf16x8 w[K / 32][NBK];
    __device__ __forceinline__ void load(const uint16_t *__restrict__ W, int n0) {
        const uint16_t *q = W + n0 * K + (threadIdx.x & 63) * 8;   // n0 is a multiple of 16
#pragma unroll
        for (int ks = 0; ks < K / 32; ++ks)
#pragma unroll
            for (int j = 0; j < NBK; ++j) w[ks][j] = *(const bf16x8 *)(q + (j * (K / 32) + ks) * 512);
    }
    template <int RB>
    __device__ __forceinline__ void apply(const uint16_t *In, int ldi, f32x4 (&acc)[RB][NBK]) const {
        const int lane = threadIdx.x & 63;
        const uint16_t *q = In + (lane & 15) * ldi + (lane >> 4) * 8;
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int j = 0; j < NBK; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < K / 32; ++ks) {
            bf16x8 b[RB];
#pragma unroll
            for (int i = 0; i < RB; ++i) b[i] = *(const bf16x8 *)(q + 16 * i * ldi + 32 * ks);
#pragma unroll
            for (int i = 0; i < RB; ++i)
#pragma unroll
                for (int j = 0; j < NBK; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[ks][j], b[i], acc[i][j], 0, 0, 0);
        }
    }
};

// ------------------------------------------------------------- features ----
__device__ __forceinline__ double raw_feature(const FeatSrc &f, int64_t i, int c) {
    if (c == 0) return log(f.T[i]);
    if (c == 1) return log(f.p[i]);
    if (c < f.N + 2) return f.Y[(int64_t)(c - 2) * f.n + i];
    if (c == f.N + 2) return log(f.dt_scalar > 0.0 ? f.dt_scalar : f.dt[i]);
    return 0.0;
}

// targets: the increments dY_k = Y1_k - Y0_k (k < N) and dT = T1 - T0
// Increments in the network's output scale: asinh(dY_k / S_Y), asinh(dT / S_T).
constexpr double S_Y = 1e-12, S_T = 1e-6;
__device__ __forceinline__ double raw_target(const TgtSrc &t, int64_t i, int c) {
    if (c < t.N) return asinh((t.Y1[(int64_t)c * t.n + i] - t.Y0[(int64_t)c * t.n + i]) / S_Y);
    return asinh((t.T1[i] - t.T0[i]) / S_T);
}

// Per column sum and sum of squares (FP64), for the nfeat features also min and
// max, one block per column: column c < nfeat is a feature (4 results from
// out + 4 c), the others targets (2 each from out + 4 nfeat).  The values take
// longest (asinh, log: some 200 vector instructions), so 1024 threads form them,
// and 256 add them up in LDS in the order i = t, t + 256, ... .
// 65,536 samples, 110 columns: 135 us, beside the host's draw of the initial
// weights; 341 us with 256 threads and a launch each for features and targets.
constexpr int MOM_T = 1024;
__global__ __launch_bounds__(MOM_T) void k_moments(FeatSrc f, TgtSrc t, int nfeat, double *out) {
    const int c = blockIdx.x, tid = threadIdx.x;
    __shared__ double val[2][MOM_T];
    __shared__ double sh[4][256];
    double s = 0.0, s2 = 0.0, mn = INFINITY, mx = -INFINITY;
    int buf = 0;
    for (int64_t base = 0; base < f.n; base += MOM_T, buf ^= 1) {
        const int64_t i = base + tid;
        if (i < f.n) val[buf][tid] = c < nfeat ? raw_feature(f, i, c) : raw_target(t, i, c - nfeat);
        __syncthreads();
        if (tid < 256) {
#pragma unroll
            for (int q = 0; q < MOM_T / 256; ++q) {
                if (base + 256 * q + tid >= f.n) break;
                const double v = val[buf][256 * q + tid];
                s += v;
                s2 += v * v;
                mn = fmin(mn, v);
                mx = fmax(mx, v);
            }
        }
    }
    if (tid < 256) { sh[0][tid] = s; sh[1][tid] = s2; sh[2][tid] = mn; sh[3][tid] = mx; }
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if (tid < st) {
            sh[0][tid] += sh[0][tid + st];
            sh[1][tid] += sh[1][tid + st];
            sh[2][tid] = fmin(sh[2][tid], sh[2][tid + st]);
            sh[3][tid] = fmax(sh[3][tid], sh[3][tid + st]);
        }
        __syncthreads();
    }
    if (tid == 0) {
        double *o = c < nfeat ? out + 4 * c : out + 4 * nfeat + 2 * (c - nfeat);
        o[0] = sh[0][0];
        o[1] = sh[1][0];
        if (c < nfeat) { o[2] = sh[2][0]; o[3] = sh[3][0]; }
    }
}

// Rows r < B from samples idx[r] (nullable: r): X[r][c] bf16 normalised
// features and Tg[r][c] normalised targets.  A block takes 64 rows, lane = row,
// so that neighbouring samples of a feature are one read, and turns them in LDS.
__global__ __launch_bounds__(256) void k_build_rows(FeatSrc f, TgtSrc t, const int *idx, int64_t B,
                                                    const float *norm, uint16_t *X, float *Tg) {
    __shared__ uint16_t xs[64][S_IN + 2];
    __shared__ float ts[64][S_OUT + 1];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t r0 = (int64_t)blockIdx.x * 64;
    const int rows = B - r0 < 64 ? (int)(B - r0) : 64;
    const int nfeat = f.N + 3;
    const int64_t r = r0 + (lane < rows ? lane : 0);
    const int64_t i = idx ? (int64_t)idx[r] : r;
    for (int c = w; c < S_IN; c += 4) {
        uint16_t v = 0;
        if (c < nfeat) v = f2bf((float)((raw_feature(f, i, c) - norm[c]) / norm[64 + c]));
        xs[lane][c] = v;
        float tv = 0.0f;
        if (c < t.N + 1) tv = (float)((raw_target(t, i, c) - norm[128 + c]) / norm[192 + c]);
        ts[lane][c] = tv;
    }
    __syncthreads();
    for (int q = w; q < rows; q += 4) {
        X[(r0 + q) * S_IN + lane] = xs[q][lane];
        Tg[(r0 + q) * S_OUT + lane] = ts[q][lane];
    }
}

// ------------------------------------------------------------- backward ----
// loss[0] = sum of the n per-block running sums (one block, fixed order)
__global__ __launch_bounds__(256) void k_sum_loss(const double *part, int n, double *loss) {
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) s += part[i];
    __shared__ double sh[256];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (threadIdx.x < h) sh[threadIdx.x] += sh[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) loss[0] = sh[0];
}

constexpr int CS_CHUNKS = 64;
// slices of a split-K weight gradient: at most 256 workgroups of 64 x 64
// outputs, so S M N <= 256 * 4096
constexpr int64_t kSplitFloats = (int64_t)256 * 4096;

// Column sums of the FP32 output gradients (bias gradients), first of two
// fixed-order passes, all layers in one launch (z; 4 is the output layer, 64
// columns): block (x, y) sums rows y, y + CS_CHUNKS, ... of 64 columns into
// part[z][y][c] (four row phases per block, combined in order); k_gradients
// adds the CS_CHUNKS partial sums in order.
struct ColSrc {
    const float *G[5];
};
__global__ __launch_bounds__(256) void k_colsum_part(ColSrc src, int B, float *part) {
    const int z = blockIdx.z, ncol = z == 4 ? S_OUT : S_HID;
    const int c = blockIdx.x * 64 + (threadIdx.x & 63), ph = threadIdx.x >> 6;
    if (blockIdx.x * 64 >= ncol) return;   // whole workgroup
    const float *g = src.G[0];
#pragma unroll
    for (int q = 1; q < 5; ++q)
        if (z == q) g = src.G[q];
    float s = 0.0f;
#pragma unroll 8
    for (int r = blockIdx.y + CS_CHUNKS * ph; r < B; r += 4 * CS_CHUNKS) s += g[(size_t)r * ncol + c];
    __shared__ float sh[4][64];
    sh[ph][threadIdx.x & 63] = s;
    __syncthreads();
    if (ph == 0)
        part[((size_t)z * CS_CHUNKS + blockIdx.y) * S_HID + c] = (sh[0][threadIdx.x] + sh[1][threadIdx.x]) +
                                                                 (sh[2][threadIdx.x] + sh[3][threadIdx.x]);
}

// Weight gradients dW_l = dZ_l^T H_{l-1} of all layers in one launch: M x N is
// a few 64 x 64 tiles and K (the batch) is long, so a layer's K range is cut
// into S slices that fill the chip; slice z writes its partial product to slab
// z of its part (M x N), and k_gradients adds the slabs in order.  Both operands
// are k-contiguous (the transposes written by k_mlp_train) and go straight from
// memory to the MFMA layout; one workgroup a tile and slice, four wavefronts of
// 32 x 32.
struct WgradJob {
    const uint16_t *A, *B;
    float *C;
    int M, N, S, first;   // first: the job's first workgroup
};
struct WgradJobs {
    WgradJob j[5];
    int ld;               // batch: row length of the operands
};
__global__ __launch_bounds__(256) void k_wgrad(WgradJobs jobs) {
    WgradJob jb = jobs.j[0];
#pragma unroll
    for (int q = 1; q < 5; ++q)
        if ((int)blockIdx.x >= jobs.j[q].first) jb = jobs.j[q];
    const int t = blockIdx.x - jb.first, tm = jb.M / 64, tn = jb.N / 64;
    const int tiles = tm * tn, z = t / tiles, xy = t - z * tiles;
    const int x = xy / tn, y = xy - x * tn;
    const int ld = jobs.ld, K = ld / jb.S;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int m0 = x * 64 + (w >> 1) * 32, n0 = y * 64 + (w & 1) * 32;
    const uint16_t *A = jb.A + op_place(m0, (int64_t)z * K, ld) + lane * 8;
    const uint16_t *B = jb.B + op_place(n0, (int64_t)z * K, ld) + lane * 8;
    const size_t next16 = (size_t)16 * ld;   // to the next 16 rows
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // four k steps at a time, the next four on their way (K is a multiple of 32)
    bf16x8 a[2][4][2], b[2][4][2];
    auto load = [&](bf16x8 (&la)[4][2], bf16x8 (&lb)[4][2], int k0) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (k0 + 32 * u < K) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    la[u][i] = *(const bf16x8 *)(A + i * next16 + (k0 + 32 * u) * 16);
                    lb[u][i] = *(const bf16x8 *)(B + i * next16 + (k0 + 32 * u) * 16);
                }
            }
    };
    auto mul = [&](const bf16x8 (&la)[4][2], const bf16x8 (&lb)[4][2], int k0) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (k0 + 32 * u < K) {
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(la[u][i], lb[u][j], acc[i][j], 0, 0, 0);
            }
    };
    load(a[0], b[0], 0);
    for (int k0 = 0; k0 < K; k0 += 256) {
        load(a[1], b[1], k0 + 128);
        mul(a[0], b[0], k0);
        load(a[0], b[0], k0 + 256);
        mul(a[1], b[1], k0 + 128);
    }
    float *C = jb.C + (size_t)z * jb.M * jb.N;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                C[(size_t)(m0 + 16 * i + 4 * (lane >> 4) + r) * jb.N + n0 + 16 * j + (lane & 15)] = acc[i][j][r];
}

// where each layer's weights sit in the FP32 blob and their bf16 copies
struct WeightCopies {
    int64_t off[5];
    int no[5], ni[5];
    uint16_t *Wb[5], *WbT[5];
};

// The gradient of parameter i: the slabs of its weight gradient, or the partial
// column sums of its bias gradient, added in order.
struct GradParts {
    const float *W[5];    // slabs of dW_l
    int S[5];
    const float *col;     // [5][CS_CHUNKS][S_HID]
};
// ADAM: the step on the FP32 masters, a weight (not a bias) also written to its
// layer's bf16 copies Wb [no x ni] and WbT [ni x no]; otherwise the gradient
// itself to G.
template <bool ADAM>
__global__ __launch_bounds__(256) void k_gradients(GradParts gp, WeightCopies wc, int64_t n, float *G, float *P,
                                                   float *m, float *v, float lr, float b1, float b2,
                                                   float eps, float c1, float c2) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    int l = 0;
    int64_t off = wc.off[0];
    int no = wc.no[0], ni = wc.ni[0], S = gp.S[0];
    const float *part = gp.W[0];
    uint16_t *wb = wc.Wb[0], *wbt = wc.WbT[0];
#pragma unroll
    for (int q = 1; q < 5; ++q)
        if (i >= wc.off[q]) {
            l = q; off = wc.off[q]; no = wc.no[q]; ni = wc.ni[q]; S = gp.S[q]; part = gp.W[q];
            wb = wc.Wb[q]; wbt = wc.WbT[q];
        }
    const int t = (int)(i - off), mn = no * ni;
    float g = 0.0f;
    if (t < mn) {
#pragma unroll 8
        for (int z = 0; z < S; ++z) g += part[(size_t)z * mn + t];
    } else {
        const float *col = gp.col + (size_t)l * CS_CHUNKS * S_HID + (t - mn);
#pragma unroll 8
        for (int y = 0; y < CS_CHUNKS; ++y) g += col[(size_t)y * S_HID];
    }
    if (!ADAM) {
        G[i] = g;
        return;
    }
    const float mi = b1 * m[i] + (1.0f - b1) * g;
    const float vi = b2 * v[i] + (1.0f - b2) * g * g;
    m[i] = mi;
    v[i] = vi;
    const float p = P[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    P[i] = p;
    if (t < mn) {
        const int o = t / ni, k = t - o * ni;
        const uint16_t b = f2bf(p);
        wb[op_place(o, k, ni)] = b;
        wbt[op_place(k, o, no)] = b;
    }
}

// bf16 copies of a layer's weights in operand order: Wb [no x ni] and WbT [ni x no]
__global__ __launch_bounds__(256) void k_refresh(const float *W, int no, int ni, uint16_t *Wb,
                                                 uint16_t *WbT) {
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= no * ni) return;
    const int o = t / ni, i = t % ni;
    const uint16_t b = f2bf(W[t]);
    Wb[op_place(o, i, ni)] = b;
    WbT[op_place(i, o, no)] = b;
}

// ------------------------------------------------- conservation + gate ----
struct PostParams {
    int N, nel;
    const double *E;       // [nel][N] a_ek / W_k
    const double *nasa_t;  // species thermo [14][N] (a1..a7, a2/2, a3/3, a4/4, a5/5, ...)
    const double *invW;
    const float *norm;     // mu_x, sd_x, mu_o, sd_o, xmin, xmax
    double tau_T, y_min, margin, max_dT, T_max;
};

__device__ __forceinline__ double pred_y(const PostParams &q, const float *outT, int m, int r, int k,
                                         double yk) {
    const double t = (double)outT[(size_t)k * m + r] * q.norm[192 + k] + q.norm[128 + k];
    const double v = yk + S_Y * sinh(t);
    return v > 0.0 ? v : 0.0;
}

// One cell per thread.  outT [64][m] normalised network outputs of chunk
// rows; row r is cell base + r.  The clipped prediction Y1 = max(Y + dY, 0)
// is corrected by Y1_k (E^T lam)_k with (E W E^T) lam = E (Y1 - Y), W =
// diag(Y1); T' solves h(T', Y') = h(T, Y).  Accepted cells are updated and
// flagged 3; rejected cells are left untouched.
template <int NEL>
__global__ __launch_bounds__(256) void k_surrogate_post(FeatSrc f, int64_t base, int m,
                                                        const float *outT, PostParams q, double *T,
                                                        double *Y, uint8_t *flags,
                                                        unsigned long long *stats) {
    const int r = blockIdx.x * 256 + threadIdx.x;
    bool accept = false, tried = false;
    if (r < m) {
        const int64_t i = base + r;
        const int N = q.N;
        if (!flags || flags[i] == 0) {
            tried = true;
            bool ok = T[i] <= q.T_max;
            // out-of-distribution box on the raw features
            for (int c = 0; c < N + 3 && ok; ++c) {
                const double v = raw_feature(f, i, c);
                const double lo = q.norm[256 + c], hi = q.norm[320 + c];
                const double span = hi - lo;
                ok = v >= lo - q.margin * span && v <= hi + q.margin * span;
            }
            double lam[NEL];
            double Tn = 0.0, dT = 0.0;
            if (ok) {
                double G[NEL][NEL], rr[NEL];
#pragma unroll
                for (int a = 0; a < NEL; ++a) {
                    rr[a] = 0.0;
#pragma unroll
                    for (int b = 0; b < NEL; ++b) G[a][b] = 0.0;
                }
                for (int k = 0; k < N; ++k) {
                    const double y0 = Y[(int64_t)k * f.n + i];
                    const double y1 = pred_y(q, outT, m, r, k, y0);
                    double ek[NEL];
#pragma unroll
                    for (int a = 0; a < NEL; ++a) ek[a] = q.E[a * N + k];
#pragma unroll
                    for (int a = 0; a < NEL; ++a) {
                        rr[a] += ek[a] * (y1 - y0);
#pragma unroll
                        for (int b = 0; b < NEL; ++b) G[a][b] += ek[a] * y1 * ek[b];
                    }
                }
                // Gaussian elimination with partial pivoting
#pragma unroll
                for (int c = 0; c < NEL; ++c) {
                    int pr = c;
#pragma unroll
                    for (int a = c + 1; a < NEL; ++a)
                        if (fabs(G[a][c]) > fabs(G[pr][c])) pr = a;
#pragma unroll
                    for (int a = c + 1; a < NEL; ++a) {
                        if (a == pr) {
#pragma unroll
                            for (int b = 0; b < NEL; ++b) {
                                const double t0 = G[c][b];
                                G[c][b] = G[a][b];
                                G[a][b] = t0;
                            }
                            const double t1 = rr[c];
                            rr[c] = rr[a];
                            rr[a] = t1;
                        }
                    }
                    ok = ok && G[c][c] != 0.0;
                    const double dinv = 1.0 / G[c][c];
#pragma unroll
                    for (int a = c + 1; a < NEL; ++a) {
                        const double l = G[a][c] * dinv;
#pragma unroll
                        for (int b = c; b < NEL; ++b) G[a][b] -= l * G[c][b];
                        rr[a] -= l * rr[c];
                    }
                }
#pragma unroll
                for (int c = NEL - 1; c >= 0; --c) {
                    double s = rr[c];
#pragma unroll
                    for (int b = c + 1; b < NEL; ++b) s -= G[c][b] * lam[b];
                    lam[c] = s / G[c][c];
                }
#pragma unroll
                for (int a = 0; a < NEL; ++a) ok = ok && isfinite(lam[a]);
                dT = S_T * sinh((double)outT[(size_t)N * m + r] * q.norm[192 + N] + q.norm[128 + N]);
                ok = ok && fabs(dT) <= q.max_dT;
                // corrected state: positivity gate and the enthalpy polynomial
                double Bo[6] = {0, 0, 0, 0, 0, 0}, Bn[6] = {0, 0, 0, 0, 0, 0};
                for (int k = 0; k < N && ok; ++k) {
                    const double y0 = Y[(int64_t)k * f.n + i];
                    const double y1 = pred_y(q, outT, m, r, k, y0);
                    double s = 0.0;
#pragma unroll
                    for (int a = 0; a < NEL; ++a) s += q.E[a * N + k] * lam[a];
                    const double yn = y1 - y1 * s;
                    ok = yn >= q.y_min;
                    const double iw = q.invW[k];
                    const double c6[6] = {q.nasa_t[k], q.nasa_t[7 * N + k], q.nasa_t[8 * N + k],
                                          q.nasa_t[9 * N + k], q.nasa_t[10 * N + k], q.nasa_t[5 * N + k]};
#pragma unroll
                    for (int t = 0; t < 6; ++t) {
                        Bo[t] += y0 * iw * c6[t];
                        Bn[t] += yn * iw * c6[t];
                    }
                }
                if (ok) {
                    const double T0 = T[i];
                    const double h0 = Bo[5] + T0 * (Bo[0] + T0 * (Bo[1] + T0 * (Bo[2] + T0 * (Bo[3] + T0 * Bo[4]))));
                    Tn = T0 + dT;
                    for (int it = 0; it < 50; ++it) {
                        const double F = Bn[5] + Tn * (Bn[0] + Tn * (Bn[1] + Tn * (Bn[2] + Tn * (Bn[3] + Tn * Bn[4])))) - h0;
                        const double dF = Bn[0] + Tn * (2.0 * Bn[1] + Tn * (3.0 * Bn[2] + Tn * (4.0 * Bn[3] + Tn * 5.0 * Bn[4])));
                        const double step = F / dF;
                        Tn -= step;
                        if (fabs(step) < 1e-10) break;
                    }
                    ok = fabs(T0 + dT - Tn) <= q.tau_T && Tn > 0.0;
                }
            }
            if (ok) {
                for (int k = 0; k < N; ++k) {
                    double *yp = Y + (int64_t)k * f.n + i;
                    const double y1 = pred_y(q, outT, m, r, k, *yp);
                    double s = 0.0;
#pragma unroll
                    for (int a = 0; a < NEL; ++a) s += q.E[a * N + k] * lam[a];
                    *yp = y1 - y1 * s;
                }
                T[i] = Tn;
                if (flags) flags[i] = 3;
                accept = true;
            }
        }
    }
    const unsigned long long na = __ballot(accept), nt = __ballot(tried);
    if ((threadIdx.x & 63) == 0) {
        if (na) atomicAdd(&stats[6], (unsigned long long)__popcll(na));
        if (nt & ~na) atomicAdd(&stats[7], (unsigned long long)__popcll(nt & ~na));
    }
}

// ------------------------------------------------------ fused inference ----
// Rows offered to the surrogate (no flag, T <= T_max): their chunk positions,
// in any order, and their count (zeroed by k_zero_int first).
__global__ void k_zero_int(int *p) { if (threadIdx.x == 0 && blockIdx.x == 0) *p = 0; }

__global__ __launch_bounds__(256) void k_sur_select(const uint8_t *flags, const double *T, int64_t base,
                                                    int m, double T_max, int *idx, int *cnt) {
    const int r = blockIdx.x * 256 + threadIdx.x;
    bool sel = false;
    if (r < m) {
        const int64_t i = base + r;
        sel = (!flags || flags[i] == 0) && T[i] <= T_max;
    }
    const unsigned long long b = __ballot(sel);
    const int lane = threadIdx.x & 63;
    int off = 0;
    if (lane == 0 && b) off = atomicAdd(cnt, __popcll(b));
    off = __shfl(off, 0);
    if (sel) idx[off + __popcll(b & ((1ull << lane) - 1ull))] = r;
}

// The whole network for a tile of 16 RB rows in one workgroup: the input tile and
// the hidden activations stay in LDS (bf16), weights stream from L2.
// Wavefront w computes output columns [64w, 64w + 64) of the hidden layers, 16
// of the 64 outputs of the last.  SELECTED: rows idx[0 .. *cnt) of the chunk,
// row r's outputs to outT[c][r] as the acceptance kernel reads them; otherwise
// all m rows from base, outputs row-major (of the caller's array no more than a
// float's alignment is asked).
// 100,003 rows: 150 us a call (167 in a kernel trace, at lower clocks), bound by
// the GELU's vector instructions and three and a bit rounds of two workgroups per
// CU; layer by layer through memory 505 us.
// A call of at most 16 rows per CU (narrow_tiles) takes tiles of 16 rows: each
// lane then has a quarter of the GELUs behind one another, which is most of a
// tile's time (one row 11 us against 28, 4096 rows 16 against 37).
constexpr int FT = 64;             // rows per tile of a large call, and of selected rows
static bool narrow_tiles(int64_t rows) { return rows <= 16 * 256; }
constexpr int XLD = S_IN + 8;      // LDS row strides (bf16), padded against bank conflicts
constexpr int HLD = S_HID + 8;
struct MlpW {
    const uint16_t *W[5];
    const float *b[5];
};

// bf16(GELU(acc + bias)) of the wavefront's 64 columns into the tile Out
template <int RB>
__device__ __forceinline__ void gelu_tile(const f32x4 (&acc)[RB][4], const float *__restrict__ bias, int n0,
                                          uint16_t *Out) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int col = n0 + 16 * j + 4 * (lane >> 4);
        const f32x4 bc = *(const f32x4 *)(bias + col);
#pragma unroll
        for (int i = 0; i < RB; ++i)
            *(uint2 *)(Out + (16 * i + (lane & 15)) * HLD + col) = gelu_bf16x4(acc[i][j] + bc);
    }
}

template <bool SELECTED, int RB>
__global__ __launch_bounds__(256, 2) void k_mlp_infer(FeatSrc f, int64_t base, int m, const int *idx,
                                                      const int *cnt, const float *norm, MlpW wt,
                                                      float *out) {
    constexpr int R = 16 * RB;
    extern __shared__ __align__(16) uint16_t sm16[];
    uint16_t *Xs = sm16, *Ha = Xs + R * XLD, *Hb = Ha + R * HLD;
    const int n_sel = SELECTED ? *cnt : m;
    const int t0 = blockIdx.x * R;
    if (t0 >= n_sel) return;                       // whole workgroup
    const int rows = n_sel - t0 < R ? n_sel - t0 : R;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int n0 = 64 * w;
    WTile<S_IN, 4> w0;
    w0.load(wt.W[0], n0);
    {
        // neighbouring lanes on neighbouring rows, so that each feature of a tile
        // is one coalesced read
        const int nfeat = f.N + 3, q = tid % R;
        const int64_t i = base + (SELECTED ? idx[t0 + (q < rows ? q : 0)] : t0 + (q < rows ? q : 0));
#pragma unroll 4
        for (int c = tid / R; c < S_IN; c += 256 / R) {
            uint16_t v = 0;
            if (q < rows && c < nfeat) v = f2bf((float)((raw_feature(f, i, c) - norm[c]) / norm[64 + c]));
            Xs[q * XLD + c] = v;
        }
    }
    lds_barrier();
    f32x4 acc[RB][4];
    w0.template apply<RB>(Xs, XLD, acc);
    WTile<S_HID, 4> wh;
    WTile<S_HID, 1> wo;
    wh.load(wt.W[1], n0);
    gelu_tile<RB>(acc, wt.b[0], n0, Ha);
    lds_barrier();
#pragma unroll
    for (int l = 1; l < 4; ++l) {   // the last leaves its result in Hb
        uint16_t *In = (l & 1) ? Ha : Hb, *Out = (l & 1) ? Hb : Ha;
        wh.template apply<RB>(In, HLD, acc);
        if (l < 3) wh.load(wt.W[l + 1], n0);
        else wo.load(wt.W[4], 16 * w);
        gelu_tile<RB>(acc, wt.b[l], n0, Out);
        lds_barrier();
    }
    f32x4 o[RB][1];
    wo.template apply<RB>(Hb, HLD, o);
    const int col = 16 * w + 4 * (lane >> 4);
    const f32x4 bc = *(const f32x4 *)(wt.b[4] + col);
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        const int row = 16 * i + (lane & 15);
        if (row >= rows) continue;
        const f32x4 v = o[i][0] + bc;
        if (SELECTED) {
            const int r = idx[t0 + row];
#pragma unroll
            for (int q = 0; q < 4; ++q) out[(size_t)(col + q) * m + r] = v[q];
        } else {
            *(f32x4_any *)(out + (size_t)(t0 + row) * S_OUT + col) = v;
        }
    }
}
static constexpr size_t infer_lds(int rows) { return sizeof(uint16_t) * (size_t)rows * (XLD + 2 * HLD); }
static constexpr size_t kInferLds = infer_lds(FT);

// ------------------------------------------------------- training: a tile ----
// Forward and backward of 16 RB rows of the batch in one workgroup.  The tile's
// activations and output gradients stay in LDS; what leaves are the transposes
// that the weight gradients contract over the batch (X, H_l, dZ_l) and the FP32
// output gradients whose column sums are the bias gradients.  The
// pre-activations go through a scratch array laid out by thread (each thread
// reads back what it wrote).  Layer by layer through memory, with a launch per
// product and 2-byte transposed stores, this was 21 of an Adam step's 36
// launches.  A batch of 4096: 44 us of the step's 70 (300 before).
struct TrainBufs {
    float *Z;                              // [tile][layer][block][thread] f32x4
    uint16_t *XT, *HT[4], *dZT[4], *dZ5T;  // [column][B], operand order
    float *G[4], *dOf;                     // [row][column]
    double *lpart;                         // squared error per workgroup, running
};

// The columns of a tile of 16 RB rows into dst [column][B], in operand order
template <int RB, int NC>
__device__ __forceinline__ void store_transposed(const uint16_t *tile, int ld, uint16_t *__restrict__ dst, int B,
                                                 int r0) {
#pragma unroll
    for (int u0 = 0; u0 < NC * 2 * RB; u0 += 256) {
        const int u = u0 + threadIdx.x;
        if (NC * 2 * RB < 256 && u >= NC * 2 * RB) break;
        const int c = u % NC, part = u / NC;
        uint32_t v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            v[q] = tile[(8 * part + 2 * q) * ld + c] | ((uint32_t)tile[(8 * part + 2 * q + 1) * ld + c] << 16);
        *(uint4 *)(dst + op_place(c, r0 + 8 * part, B)) = uint4{v[0], v[1], v[2], v[3]};
    }
}

// z = acc + bias kept in the scratch, bf16(GELU(z)) into the tile Out
template <int RB>
__device__ __forceinline__ void train_hidden(const f32x4 (&acc)[RB][4], const float *__restrict__ bias, int n0,
                                             f32x4 *__restrict__ Z, uint16_t *Out) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int col = n0 + 16 * j + 4 * (lane >> 4);
        const f32x4 bc = *(const f32x4 *)(bias + col);
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            const f32x4 z = acc[i][j] + bc;
            Z[(size_t)(4 * i + j) * 256 + threadIdx.x] = z;
            *(uint2 *)(Out + (16 * i + (lane & 15)) * HLD + col) = gelu_bf16x4(z);
        }
    }
}

// dZ = dH GELU'(Z): FP32 to G, bf16 into the tile Out
template <int RB>
__device__ __forceinline__ void train_back(const f32x4 (&acc)[RB][4], int n0, const f32x4 *__restrict__ Z, int r0,
                                           float *__restrict__ G, uint16_t *Out) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int col = n0 + 16 * j + 4 * (lane >> 4);
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            const int row = 16 * i + (lane & 15);
            const f32x4 z = Z[(size_t)(4 * i + j) * 256 + threadIdx.x];
            f32x4 g;
#pragma unroll
            for (int r = 0; r < 4; ++r) g[r] = acc[i][j][r] * gelu_df(z[r]);
            *(f32x4 *)(G + (size_t)(r0 + row) * S_HID + col) = g;
            *(uint2 *)(Out + row * HLD + col) = uint2{pk_bf16(g[0], g[1]), pk_bf16(g[2], g[3])};
        }
    }
}

struct TrainW {
    const uint16_t *W[5], *WT[5];
    const float *b[5];
};

template <int RB>
__global__ __launch_bounds__(256, 2) void k_mlp_train(const uint16_t *__restrict__ X, const float *__restrict__ Tg,
                                                      const int *__restrict__ idx, int B, int nout, TrainW wt,
                                                      TrainBufs t) {
    constexpr int R = 16 * RB;
    extern __shared__ __align__(16) uint16_t sm16[];
    uint16_t *Xs = sm16, *Ha = Xs + R * XLD, *Hb = Ha + R * HLD;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, n0 = 64 * w;
    const int r0 = blockIdx.x * R;
    f32x4 *Z = reinterpret_cast<f32x4 *>(t.Z) + (size_t)blockIdx.x * (16 * RB) * 256;
    constexpr size_t ZL = (size_t)4 * RB * 256;   // a layer's part
    WTile<S_IN, 4> w0;
    w0.load(wt.W[0], n0);
    for (int q = tid; q < R * 8; q += 256) {
        const int row = q >> 3, c8 = q & 7;
        const int64_t src = idx ? idx[r0 + row] : r0 + row;
        *(uint4 *)(Xs + row * XLD + 8 * c8) = *(const uint4 *)(X + src * S_IN + 8 * c8);
    }
    lds_barrier();
    f32x4 acc[RB][4];
    WTile<S_HID, 4> wh;
    w0.template apply<RB>(Xs, XLD, acc);
    store_transposed<RB, S_IN>(Xs, XLD, t.XT, B, r0);
    wh.load(wt.W[1], n0);
    train_hidden<RB>(acc, wt.b[0], n0, Z, Ha);
    lds_barrier();
    WTile<S_HID, 1> wo;
#pragma unroll
    for (int l = 1; l < 4; ++l) {   // the last leaves its result in Hb
        uint16_t *In = (l & 1) ? Ha : Hb, *Out = (l & 1) ? Hb : Ha;
        wh.template apply<RB>(In, HLD, acc);
        store_transposed<RB, S_HID>(In, HLD, t.HT[l - 1], B, r0);
        if (l < 3) wh.load(wt.W[l + 1], n0);
        else wo.load(wt.W[4], 16 * w);
        train_hidden<RB>(acc, wt.b[l], n0, Z + l * ZL, Out);
        lds_barrier();
    }
    f32x4 o[RB][1];
    wo.template apply<RB>(Hb, HLD, o);
    store_transposed<RB, S_HID>(Hb, HLD, t.HT[3], B, r0);
    WTile<S_OUT, 4> w5;
    w5.load(wt.WT[4], n0);
    // dO = 2 (out - target) / (B nout) for the first nout columns, 0 elsewhere
    double l2 = 0.0;
    {
        const int col = 16 * w + 4 * (lane >> 4);
        const f32x4 bc = *(const f32x4 *)(wt.b[4] + col);
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            const int row = 16 * i + (lane & 15);
            const int64_t src = idx ? idx[r0 + row] : r0 + row;
            const f32x4 v = o[i][0] + bc;
            const f32x4 tg = *(const f32x4 *)(Tg + src * S_OUT + col);
            f32x4 g;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float e = v[r] - tg[r];
                const bool live = col + r < nout;
                g[r] = live ? 2.0f * e / ((float)B * (float)nout) : 0.0f;
                l2 += live ? (double)e * e : 0.0;
            }
            *(f32x4 *)(t.dOf + (size_t)(r0 + row) * S_OUT + col) = g;
            *(uint2 *)(Xs + row * XLD + col) = uint2{pk_bf16(g[0], g[1]), pk_bf16(g[2], g[3])};
        }
    }
    for (int m = 32; m > 0; m >>= 1) l2 += __shfl_xor(l2, m);
    __shared__ double sh[4];
    if (lane == 0) sh[w] = l2;
    lds_barrier();
    if (tid == 0) t.lpart[blockIdx.x] += (sh[0] + sh[1]) + (sh[2] + sh[3]);
    // backward: dH = dZ W layer by layer
    w5.template apply<RB>(Xs, XLD, acc);
    store_transposed<RB, S_OUT>(Xs, XLD, t.dZ5T, B, r0);
#pragma unroll
    for (int l = 3; l >= 0; --l) {
        uint16_t *Out = (l & 1) ? Ha : Hb;
        if (l > 0) wh.load(wt.WT[l], n0);
        train_back<RB>(acc, n0, Z + l * ZL, r0, t.G[l], Out);
        lds_barrier();
        if (l > 0) wh.template apply<RB>(Out, HLD, acc);
        store_transposed<RB, S_HID>(Out, HLD, t.dZT[l], B, r0);
    }
}
static constexpr size_t train_lds(int RB) { return sizeof(uint16_t) * (size_t)16 * RB * (XLD + 2 * HLD); }

// Every row of a chunk selected, in order (the fused kernel's check entry).
__global__ __launch_bounds__(256) void k_select_all(int m, int *idx, int *cnt) {
    const int r = blockIdx.x * 256 + threadIdx.x;
    if (r < m) idx[r] = r;
    if (r == 0) *cnt = m;
}

// out[r][c] = outT[c][r] for a chunk of m rows and 64 outputs
__global__ __launch_bounds__(256) void k_untranspose(const float *outT, int m, float *out) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (int64_t)m * S_OUT) return;
    const int r = (int)(i / S_OUT), c = (int)(i % S_OUT);
    out[i] = outT[(size_t)c * m + r];
}

static void launch_post(int nel, dim3 g, hipStream_t s, const FeatSrc &f, int64_t base, int m,
                        const float *outT, const PostParams &q, double *T, double *Y, uint8_t *flags,
                        unsigned long long *stats) {
    switch (nel) {
#define POST(E_)                                                                                   \
    case E_:                                                                                       \
        hipLaunchKernelGGL(k_surrogate_post<E_>, g, dim3(256), 0, s, f, base, m, outT, q, T, Y,   \
                           flags, stats);                                                          \
        break;
        POST(1) POST(2) POST(3) POST(4) POST(5) POST(6) POST(7) POST(8)
#undef POST
    }
}

// ================================================================ host ======
static int layer_in(int l) { return l == 0 ? S_IN : S_HID; }
static int layer_out(int l) { return l == 4 ? S_OUT : S_HID; }

int64_t surrogate_param_count() {
    int64_t n = 0;
    for (int l = 0; l < 5; ++l) n += (int64_t)layer_out(l) * layer_in(l) + layer_out(l);
    return n + 6 * S_IN;
}
static int64_t weights_count() { return surrogate_param_count() - 6 * S_IN; }
static int64_t layer_offset(int l) {
    int64_t o = 0;
    for (int q = 0; q < l; ++q) o += (int64_t)layer_out(q) * layer_in(q) + layer_out(q);
    return o;
}

#define SCHK(x)                                                         \
    do {                                                                \
        hipError_t e_ = (x);                                            \
        if (e_ != hipSuccess) {                                         \
            snprintf(err, 256, "%s: %s", #x, hipGetErrorString(e_));    \
            return -3;                                                  \
        }                                                               \
    } while (0)

template <class T>
static hipError_t dalloc(T **p, size_t count) {
    return hipMalloc((void **)p, std::max<size_t>(1, count) * sizeof(T));
}

Surrogate::~Surrogate() {
    for (void *p : bufs) (void)hipFree(p);
    for (void *p : ws) (void)hipFree(p);
}

int Surrogate::init(int N_, int nel_, const std::vector<double> &E_host, char *err) {
    N = N_;
    nel = nel_;
    SCHK(hipFuncSetAttribute((const void *)k_mlp_infer<true, 4>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)kInferLds));
    SCHK(hipFuncSetAttribute((const void *)k_mlp_infer<false, 4>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)kInferLds));
    SCHK(hipFuncSetAttribute((const void *)k_mlp_train<2>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)train_lds(2)));
    const int64_t np = surrogate_param_count();
    float *fp = nullptr;
    SCHK(dalloc(&fp, np)); bufs.push_back(fp); P = fp;
    SCHK(dalloc(&fp, np)); bufs.push_back(fp); G = fp;
    SCHK(dalloc(&fp, np)); bufs.push_back(fp); mA = fp;
    SCHK(dalloc(&fp, np)); bufs.push_back(fp); vA = fp;
    for (int l = 0; l < 5; ++l) {
        uint16_t *b = nullptr;
        SCHK(dalloc(&b, (size_t)layer_out(l) * layer_in(l))); bufs.push_back(b); Wb[l] = b;
        SCHK(dalloc(&b, (size_t)layer_out(l) * layer_in(l))); bufs.push_back(b); WbT[l] = b;
    }
    double *dp = nullptr;
    SCHK(dalloc(&dp, E_host.size())); bufs.push_back(dp); E = dp;
    SCHK(hipMemcpy(E, E_host.data(), sizeof(double) * E_host.size(), hipMemcpyHostToDevice));
    SCHK(dalloc(&dp, 1)); bufs.push_back(dp); d_loss = dp;
    return 0;
}

int Surrogate::refresh(hipStream_t s, char *err) {
    for (int l = 0; l < 5; ++l) {
        const int no = layer_out(l), ni = layer_in(l);
        hipLaunchKernelGGL(k_refresh, dim3((no * ni + 255) / 256), dim3(256), 0, s,
                           P + layer_offset(l), no, ni, Wb[l], WbT[l]);
    }
    SCHK(hipGetLastError());
    return 0;
}

int Surrogate::set_params(const float *host, hipStream_t s, char *err) {
    SCHK(hipMemcpyAsync(P, host, sizeof(float) * surrogate_param_count(), hipMemcpyHostToDevice, s));
    SCHK(hipStreamSynchronize(s));
    int rc = refresh(s, err);
    if (rc) return rc;
    trained = true;
    return 0;
}

int Surrogate::get_params(float *host, hipStream_t s, char *err) {
    SCHK(hipMemcpyAsync(host, P, sizeof(float) * surrogate_param_count(), hipMemcpyDeviceToHost, s));
    SCHK(hipStreamSynchronize(s));
    return 0;
}

// Workspace for up to B rows.  Inference: the selected rows and their outputs.
// Training: the tile kernel's arrays, and the slabs of the weight gradients.
int Surrogate::reserve_ws(int B, bool training, char *err) {
    if (B <= ws_rows && (!training || ws_training)) return 0;
    for (void *p : ws) (void)hipFree(p);
    ws.clear();
    ws_rows = 0;
    auto get16 = [&](uint16_t **p, size_t n) { hipError_t e = dalloc(p, n); ws.push_back(*p); return e; };
    auto get32 = [&](float **p, size_t n) { hipError_t e = dalloc(p, n); ws.push_back(*p); return e; };
    SCHK(get32(&out, (size_t)B * S_OUT));
    if (training) {
        SCHK(get16(&X, (size_t)B * S_IN));
        SCHK(get32(&Tg, (size_t)B * S_OUT));
        SCHK(get16(&XT, (size_t)B * S_IN));
        for (int l = 0; l < 4; ++l) {
            SCHK(get16(&HT[l], (size_t)B * S_HID));
            SCHK(get16(&dZT[l], (size_t)B * S_HID));
            SCHK(get32(&dZ[l], (size_t)B * S_HID));
        }
        SCHK(get32(&Z, (size_t)4 * B * S_HID));
        SCHK(get32(&dOf, (size_t)B * S_OUT));
        SCHK(get16(&dZ5T, (size_t)B * S_OUT));
        SCHK(get32(&csum, (size_t)5 * CS_CHUNKS * S_HID));
        SCHK(get32(&kpart, (size_t)5 * kSplitFloats));
        double *dp = nullptr;
        SCHK(dalloc(&dp, (size_t)(B + 15) / 16)); ws.push_back(dp); lpart = dp;
    }
    int *ip = nullptr;
    SCHK(dalloc(&ip, (size_t)B)); ws.push_back(ip); idx = ip;
    SCHK(dalloc(&ip, (size_t)1)); ws.push_back(ip); sel_cnt = ip;
    ws_rows = B;
    ws_training = training;
    return 0;
}

// Rows of a training tile: 32 where that leaves a tile for every CU (a tile
// streams the weights of both passes, 0.9 MB, so fewer tiles read less), else 16
// (a batch of 4096 is then 256 tiles).  64 rows spill 119 registers.
static bool wide_tiles(int B) { return B >= 32 * 256; }

// Forward and backward of B rows from X / Tg (rows idx[r], or r), then the
// partial sums of every gradient, which k_gradients adds up.  False (nothing
// enqueued) if a launch would not fit the workspace.
bool Surrogate::gradients(int B, const uint16_t *Xr, const float *Tr, const int *rows, hipStream_t s,
                          GradParts &gp) {
    if (B > ws_rows || !ws_training || B % 64 != 0) return false;
    WgradJobs jobs{};
    jobs.ld = B;
    int first = 0;
    for (int l = 0; l < 5; ++l) {
        const int M = layer_out(l), Nl = layer_in(l), tiles = (M / 64) * (Nl / 64);
        int S = 1;
        while (tiles * 2 * S <= 256 && B % (64 * S) == 0 && B / (2 * S) >= 128 &&
               (int64_t)2 * S * M * Nl <= kSplitFloats)
            S *= 2;
        // launch invariants, checked on the host before anything is enqueued:
        // every slice is a whole number of 32-wide k steps of the batch, and
        // the S slabs of M x N partial sums fit the layer's part of the buffer
        if (B % S != 0 || (B / S) % 32 != 0 || (int64_t)S * M * Nl > kSplitFloats) return false;
        WgradJob &j = jobs.j[l];
        j.A = l == 4 ? dZ5T : dZT[l];
        j.B = l == 0 ? XT : HT[l - 1];
        j.C = kpart + (size_t)l * kSplitFloats;
        j.M = M; j.N = Nl; j.S = S; j.first = first;
        first += tiles * S;
        gp.W[l] = j.C;
        gp.S[l] = S;
    }
    gp.col = csum;
    TrainW wt{};
    TrainBufs t{};
    ColSrc cs{};
    for (int l = 0; l < 5; ++l) {
        wt.W[l] = Wb[l];
        wt.WT[l] = WbT[l];
        wt.b[l] = P + layer_offset(l) + (int64_t)layer_out(l) * layer_in(l);
    }
    for (int l = 0; l < 4; ++l) {
        t.HT[l] = HT[l];
        t.dZT[l] = dZT[l];
        t.G[l] = dZ[l];
        cs.G[l] = dZ[l];
    }
    cs.G[4] = dOf;
    t.Z = Z; t.XT = XT; t.dZ5T = dZ5T; t.dOf = dOf; t.lpart = lpart;
    if (wide_tiles(B))
        hipLaunchKernelGGL(k_mlp_train<2>, dim3(B / 32), dim3(256), train_lds(2), s, Xr, Tr, rows, B, N + 1, wt, t);
    else
        hipLaunchKernelGGL(k_mlp_train<1>, dim3(B / 16), dim3(256), train_lds(1), s, Xr, Tr, rows, B, N + 1, wt, t);
    hipLaunchKernelGGL(k_colsum_part, dim3(S_HID / 64, CS_CHUNKS, 5), dim3(256), 0, s, cs, B, csum);
    hipLaunchKernelGGL(k_wgrad, dim3(first), dim3(256), 0, s, jobs);
    return true;
}
static int loss_blocks(int B) { return wide_tiles(B) ? B / 32 : B / 16; }

WeightCopies Surrogate::weight_copies() const {
    WeightCopies wc{};
    for (int l = 0; l < 5; ++l) {
        wc.off[l] = layer_offset(l);
        wc.no[l] = layer_out(l);
        wc.ni[l] = layer_in(l);
        wc.Wb[l] = Wb[l];
        wc.WbT[l] = WbT[l];
    }
    return wc;
}

// Standard normal floats by Marsaglia's polar method over a 64-bit Mersenne
// Twister, the sequence of std::normal_distribution<float>: two uniforms x, y in
// [-1, 1) until 0 < x^2 + y^2 <= 1, then y f is returned and x f kept for the next
// call, f = sqrt(-2 ln r2 / r2).  The library's uniform takes a long-double
// logarithm per draw as built here: 230 K draws cost 15.7 ms against 4.1.
class PolarNormal {
    std::mt19937_64 rng;
    float kept = 0.0f;
    bool has = false;
    float unit() {
        // rounds as the 64-bit number does: the bit shifted out stays as a
        // sticky one (an unsigned conversion branches on the top bit, a coin toss)
        const uint64_t x = rng();
        if (x < (1ull << 26)) return (float)x * 0x1p-64f;
        const float u = (float)(int64_t)((x >> 1) | (x & 1)) * 0x1p-63f;
        return u < 1.0f ? u : 0x1.fffffep-1f;
    }

public:
    explicit PolarNormal(uint64_t seed) : rng(seed) {}
    float operator()() {
        if (has) {
            has = false;
            return kept;
        }
        float x, y, r2;
        do {
            x = 2.0f * unit() - 1.0f;
            y = 2.0f * unit() - 1.0f;
            r2 = x * x + y * y;
        } while (r2 > 1.0f || r2 == 0.0f);
        const float f = std::sqrt(-2.0f * std::log(r2) / r2);
        kept = x * f;
        has = true;
        return y * f;
    }
};

// Normalisation and training box from the device's moments dm into the parameters.
int Surrogate::compute_norm(const FeatSrc &f, const double *dm, hipStream_t s, char *err) {
    const int nfeat = N + 3, nout = N + 1;
    std::vector<double> hm(4 * nfeat + 2 * nout);
    SCHK(hipMemcpyAsync(hm.data(), dm, sizeof(double) * hm.size(), hipMemcpyDeviceToHost, s));
    SCHK(hipStreamSynchronize(s));
    std::vector<float> nb(6 * S_IN, 0.0f);
    const double n = (double)f.n;
    for (int c = 0; c < S_IN; ++c) { nb[64 + c] = 1.0f; nb[192 + c] = 1.0f; }
    for (int c = 0; c < nfeat; ++c) {
        const double mu = hm[4 * c] / n;
        const double var = std::max(0.0, hm[4 * c + 1] / n - mu * mu);
        const double sd = sqrt(var);
        nb[c] = (float)mu;
        nb[64 + c] = sd > 1e-30 ? (float)sd : 1.0f;
        // the stored box must contain every training feature after rounding
        float lo = (float)hm[4 * c + 2], hi = (float)hm[4 * c + 3];
        if ((double)lo > hm[4 * c + 2]) lo = nextafterf(lo, -INFINITY);
        if ((double)hi < hm[4 * c + 3]) hi = nextafterf(hi, INFINITY);
        nb[256 + c] = lo;
        nb[320 + c] = hi;
    }
    for (int c = 0; c < nout; ++c) {
        const double mu = hm[4 * nfeat + 2 * c] / n;
        const double var = std::max(0.0, hm[4 * nfeat + 2 * c + 1] / n - mu * mu);
        const double sd = sqrt(var);
        nb[128 + c] = (float)mu;
        nb[192 + c] = sd > 1e-30 ? (float)sd : 1.0f;
    }
    SCHK(hipMemcpyAsync(P + weights_count(), nb.data(), sizeof(float) * nb.size(),
                        hipMemcpyHostToDevice, s));
    SCHK(hipStreamSynchronize(s));   // nb is released on return
    return 0;
}

int Surrogate::train(const FeatSrc &f, const TgtSrc &t, int epochs, int B, double lr0, double lr1,
                     uint64_t seed, float *loss_hist, int verbose, hipStream_t s, char *err) {
    if (B % 64 != 0 || B < 64) { snprintf(err, 256, "batch must be a positive multiple of 64"); return -1; }
    const int64_t n = f.n;
    if (n < B) { snprintf(err, 256, "fewer samples than one batch"); return -1; }
    int rc = reserve_ws(B, true, err);
    if (rc) return rc;
    // Host arrays that copies read, then per-call buffers, released on every
    // return: the buffers go first, and freeing them waits for the device, so no
    // copy outlives its source when a later allocation or launch fails.
    std::vector<float> h(weights_count(), 0.0f);
    std::vector<int> perm;
    struct Bufs {
        std::vector<void *> v;
        ~Bufs() { for (void *p : v) (void)hipFree(p); }
    } own;
    const int nfeat = N + 3, nout = N + 1;
    double *dm = nullptr;
    SCHK(dalloc(&dm, (size_t)4 * nfeat + 2 * nout)); own.v.push_back(dm);
    hipLaunchKernelGGL(k_moments, dim3(nfeat + nout), dim3(MOM_T), 0, s, f, t, nfeat, dm);
    SCHK(hipGetLastError());
    // He-style initialisation (seeded), zero biases, small output layer, drawn
    // while the device forms the moments
    {
        PolarNormal nd(seed);
        for (int l = 0; l < 5; ++l) {
            const int no = layer_out(l), ni = layer_in(l);
            const float sc = (l == 4 ? 0.1f : 1.0f) * sqrtf(2.0f / (float)ni);
            float *W = h.data() + layer_offset(l);
            for (int o = 0; o < no; ++o)
                for (int i = 0; i < ni; ++i) {
                    const bool live_in = l > 0 || i < N + 3;
                    const bool live_out = l < 4 || o < N + 1;
                    W[o * ni + i] = (live_in && live_out) ? sc * nd() : 0.0f;
                }
        }
    }
    rc = compute_norm(f, dm, s, err);
    if (rc) return rc;
    SCHK(hipMemcpyAsync(P, h.data(), sizeof(float) * h.size(), hipMemcpyHostToDevice, s));
    SCHK(hipMemsetAsync(mA, 0, sizeof(float) * weights_count(), s));
    SCHK(hipMemsetAsync(vA, 0, sizeof(float) * weights_count(), s));
    rc = refresh(s, err);
    if (rc) return rc;
    const int64_t nb = n / B;
    const int64_t total = nb * epochs;
    int *d_perm = nullptr;
    SCHK(dalloc(&d_perm, (size_t)n)); own.v.push_back(d_perm);
    // The normalised rows of every sample are built once (384 bytes each) and
    // gathered by each step; where they do not fit, each batch builds its own.
    uint16_t *Xall = nullptr;
    float *Tall = nullptr;
    if (dalloc(&Xall, (size_t)n * S_IN) == hipSuccess) {
        own.v.push_back(Xall);
        if (dalloc(&Tall, (size_t)n * S_OUT) == hipSuccess) own.v.push_back(Tall);
        else Tall = nullptr;
    }
    (void)hipGetLastError();   // a failed allocation is not the launches' error
    const bool all_rows = Tall != nullptr;
    if (all_rows)
        hipLaunchKernelGGL(k_build_rows, dim3((unsigned)((n + 63) / 64)), dim3(256), 0, s, f, t, (const int *)nullptr,
                           n, P + weights_count(), Xall, Tall);
    perm.resize(n);
    std::mt19937_64 rng(seed ^ 0x9e3779b97f4a7c15ull);
    auto shuffle = [&] {
        std::iota(perm.begin(), perm.end(), 0);
        std::shuffle(perm.begin(), perm.end(), rng);
    };
    if (epochs > 0) shuffle();
    SCHK(hipStreamSynchronize(s));   // h has been read
    int64_t step = 0;
    const int64_t nw = weights_count();
    const WeightCopies wc = weight_copies();
    for (int ep = 0; ep < epochs; ++ep) {
        SCHK(hipMemcpyAsync(d_perm, perm.data(), sizeof(int) * n, hipMemcpyHostToDevice, s));
        SCHK(hipMemsetAsync(lpart, 0, sizeof(double) * loss_blocks(B), s));
        SCHK(hipStreamSynchronize(s));   // perm has been read
        for (int64_t bi = 0; bi < nb; ++bi, ++step) {
            const int *rows = d_perm + bi * B;
            if (!all_rows) {
                hipLaunchKernelGGL(k_build_rows, dim3(B / 64), dim3(256), 0, s, f, t, rows, (int64_t)B,
                                   P + weights_count(), X, Tg);
                rows = nullptr;
            }
            GradParts gp{};
            if (!gradients(B, all_rows ? Xall : X, all_rows ? Tall : Tg, rows, s, gp)) {
                snprintf(err, 256, "backward: launch does not fit the workspace (batch %d)", B);
                return -1;
            }
            const double frac = total > 1 ? (double)step / (double)(total - 1) : 1.0;
            const float lr = (float)(lr1 + 0.5 * (lr0 - lr1) * (1.0 + cos(M_PI * frac)));
            const float b1 = 0.9f, b2 = 0.999f;
            const float c1 = 1.0f - powf(b1, (float)(step + 1)), c2 = 1.0f - powf(b2, (float)(step + 1));
            hipLaunchKernelGGL(k_gradients<true>, dim3((unsigned)((nw + 255) / 256)), dim3(256), 0, s, gp, wc, nw,
                               (float *)nullptr, P, mA, vA, lr, b1, b2, 1e-8f, c1, c2);
        }
        hipLaunchKernelGGL(k_sum_loss, dim3(1), dim3(256), 0, s, lpart, loss_blocks(B), d_loss);
        if (ep + 1 < epochs) shuffle();   // the next epoch's order while this one runs
        double l = 0.0;
        SCHK(hipMemcpyAsync(&l, d_loss, sizeof(double), hipMemcpyDeviceToHost, s));
        SCHK(hipStreamSynchronize(s));
        const double mean = l / ((double)nb * B * (N + 1));
        if (loss_hist) loss_hist[ep] = (float)mean;
        if (verbose) fprintf(stderr, "[libchem] surrogate epoch %d/%d: loss %.4e\n", ep + 1, epochs, mean);
    }
    SCHK(hipStreamSynchronize(s));
    SCHK(hipGetLastError());
    trained = true;
    return 0;
}

int Surrogate::loss_grad(const FeatSrc &f, const TgtSrc &t, float *grad_host, double *loss,
                         hipStream_t s, char *err) {
    const int B = (int)f.n;
    if (B % 64 != 0 || B < 64 || B > 65536) { snprintf(err, 256, "n must be a multiple of 64, <= 65536"); return -1; }
    int rc = reserve_ws(B, true, err);
    if (rc) return rc;
    SCHK(hipMemsetAsync(lpart, 0, sizeof(double) * loss_blocks(B), s));
    hipLaunchKernelGGL(k_build_rows, dim3(B / 64), dim3(256), 0, s, f, t, (const int *)nullptr, (int64_t)B,
                       P + weights_count(), X, Tg);
    GradParts gp{};
    if (!gradients(B, X, Tg, nullptr, s, gp)) {
        snprintf(err, 256, "backward: launch does not fit the workspace (%d rows)", B);
        return -1;
    }
    const int64_t nw = weights_count();
    hipLaunchKernelGGL(k_gradients<false>, dim3((unsigned)((nw + 255) / 256)), dim3(256), 0, s, gp, weight_copies(),
                       nw, G, (float *)nullptr, (float *)nullptr, (float *)nullptr, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f);
    hipLaunchKernelGGL(k_sum_loss, dim3(1), dim3(256), 0, s, lpart, loss_blocks(B), d_loss);
    SCHK(hipMemcpyAsync(grad_host, G, sizeof(float) * nw, hipMemcpyDeviceToHost, s));
    double l = 0.0;
    SCHK(hipMemcpyAsync(&l, d_loss, sizeof(double), hipMemcpyDeviceToHost, s));
    SCHK(hipStreamSynchronize(s));
    *loss = l / ((double)B * (N + 1));
    return 0;
}

MlpW Surrogate::infer_weights() const {
    MlpW wts{};
    for (int l = 0; l < 5; ++l) {
        wts.W[l] = Wb[l];
        wts.b[l] = P + layer_offset(l) + (int64_t)layer_out(l) * layer_in(l);
    }
    return wts;
}

// Raw outputs of every row, straight to the caller's array.
int Surrogate::forward_rows(const FeatSrc &f, float *out_dev, hipStream_t s, char *err) {
    const int64_t n = f.n;
    const int chunk = 1 << 24;
    for (int64_t base = 0; base < n; base += chunk) {
        const int m = (int)std::min<int64_t>(chunk, n - base);
        const int rows = narrow_tiles(n) ? 16 : FT;
        hipLaunchKernelGGL((rows == 16 ? k_mlp_infer<false, 1> : k_mlp_infer<false, 4>), dim3((m + rows - 1) / rows),
                           dim3(256), infer_lds(rows), s, f, base, m, (const int *)nullptr, (const int *)nullptr,
                           P + weights_count(), infer_weights(), out_dev + base * S_OUT);
    }
    SCHK(hipGetLastError());
    return 0;
}

// Raw outputs of the fused inference kernel (the one apply() runs), every row
// selected, in the row-major layout of forward_rows.
int Surrogate::forward_fused_rows(const FeatSrc &f, float *out_dev, hipStream_t s, char *err) {
    const int64_t n = f.n;
    const int chunk = 262144;
    int rc = reserve_ws((int)std::min<int64_t>(n, chunk), false, err);
    if (rc) return rc;
    const MlpW wts = infer_weights();
    for (int64_t base = 0; base < n; base += chunk) {
        const int m = (int)std::min<int64_t>(chunk, n - base);
        hipLaunchKernelGGL(k_select_all, dim3((m + 255) / 256), dim3(256), 0, s, m, idx, sel_cnt);
        hipLaunchKernelGGL((k_mlp_infer<true, 4>), dim3((m + FT - 1) / FT), dim3(256), kInferLds, s, f, base, m,
                           idx, sel_cnt, P + weights_count(), wts, out);
        hipLaunchKernelGGL(k_untranspose, dim3((unsigned)(((int64_t)m * S_OUT + 255) / 256)), dim3(256),
                           0, s, out, m, out_dev + base * S_OUT);
    }
    SCHK(hipGetLastError());
    return 0;
}

int Surrogate::apply(const FeatSrc &f, double *T, double *Y, uint8_t *flags, const PostIn &pin,
                     unsigned long long *stats, hipStream_t s, char *err) {
    const int64_t n = f.n;
    const int chunk = 262144;
    int rc = reserve_ws((int)std::min<int64_t>(n, chunk), false, err);
    if (rc) return rc;
    const MlpW wts = infer_weights();
    PostParams q{};
    q.N = N; q.nel = nel; q.E = E; q.nasa_t = pin.nasa_t; q.invW = pin.invW;
    q.norm = P + weights_count(); q.tau_T = pin.tau_T; q.y_min = pin.y_min; q.margin = pin.margin;
    q.max_dT = pin.max_dT;
    q.T_max = pin.T_max;
    for (int64_t base = 0; base < n; base += chunk) {
        const int m = (int)std::min<int64_t>(chunk, n - base);
        // only offered rows go through the network (fused, one kernel)
        hipLaunchKernelGGL(k_zero_int, dim3(1), dim3(64), 0, s, sel_cnt);
        hipLaunchKernelGGL(k_sur_select, dim3((m + 255) / 256), dim3(256), 0, s, flags, T, base, m,
                           pin.T_max, idx, sel_cnt);
        hipLaunchKernelGGL((k_mlp_infer<true, 4>), dim3((m + FT - 1) / FT), dim3(256), kInferLds, s, f, base, m,
                           idx, sel_cnt, P + weights_count(), wts, out);
        launch_post(nel, dim3((m + 255) / 256), s, f, base, m, out, q, T, Y, flags, stats);
    }
    SCHK(hipGetLastError());
    return 0;
}

}  // namespace chem
