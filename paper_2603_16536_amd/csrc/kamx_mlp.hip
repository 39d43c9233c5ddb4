// Learned warm start: a three-layer perceptron (two GELU hidden layers)
// that maps a world's state features to the dual impulses of the coming
// step.  Not part of the paper, whose only warm start is the previous
// step's impulses (Sec. 4.1): the network only moves the starting point of
// the ADMM iteration, whose exit test is unchanged.
//
// Every contraction runs on the matrix cores: v_mfma_f32_16x16x32_bf16 with
// BF16 operands (round to nearest even from FP32) and FP32 accumulation.
// Master weights, biases, Adam moments and gradients stay FP32.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <string>
#include <type_traits>
#include <vector>

#include "kamx_internal.h"

namespace kamx {

namespace {

constexpr int kTileM = 64, kTileN = 64, kTileK = 32;
constexpr int kLdsRow = kTileK + 8;  // bf16 per LDS tile row (16-byte pad)
constexpr int kGemmThreads = 256;
constexpr int kColBlocks = 32;  // row blocks of the bias-gradient column sums

// Weight gradients are sums over the batch (K): split K so that the
// launch has about 512 workgroups, each slice at least 128 rows long.
inline int grad_splits(int M, int N, int K) {
    const int tiles = (M / kTileM) * (N / kTileN);
    int s = 1;
    while (tiles * s < 512 && K % (2 * s * kTileK) == 0 && K / (2 * s) >= 128) s *= 2;
    return s;
}


// element (i, k) of an operand at p[i * si + k * sk]; one of the strides is 1
struct Operand {
    const __bf16 *p;
    long si, sk;
};

enum Epilogue { kEpiHidden = 0, kEpiOut = 1, kEpiBackward = 2, kEpiStore = 3 };

struct EpiArgs {
    const float *bias;  // [N] (hidden, out)
    float *f32;         // hidden: z; out: normalised output; backward: dz; store: C
    __bf16 *b16;        // hidden: gelu(z); backward: dz
    long ld;            // row stride of f32 / b16 / z
    const float *z;     // backward: pre-activation
    float *y;           // out: de-standardised output [batch, n_out] (may be null)
    long ldy;
    int batch, n_out;
    const float *mu, *sigma;
    long split;         // store: stride between the K slices' partial results
};


// Stage a 64 x 32 tile of an operand (rows i0.., columns k0..) into LDS as
// [row][k] so that every matrix-core operand is one 16-byte LDS read.
__device__ inline void stage(const Operand &o, long i0, long k0, __bf16 *tile) {
    const int t = threadIdx.x;
    if (o.sk == 1) {
        const int r = t >> 2, kc = (t & 3) * 8;
        bf16x8 v = *reinterpret_cast<const bf16x8 *>(o.p + (i0 + r) * o.si + k0 + kc);
        *reinterpret_cast<bf16x8 *>(tile + r * kLdsRow + kc) = v;
    } else {
        const int k = t >> 3, ic = (t & 7) * 8;
        bf16x8 v = *reinterpret_cast<const bf16x8 *>(o.p + (k0 + k) * o.sk + i0 + ic);
#pragma unroll
        for (int j = 0; j < 8; ++j) tile[(ic + j) * kLdsRow + k] = v[j];
    }
}

// The same from a weight matrix of K columns in the order of weight_at.
__device__ inline void stage_blocked(const __bf16 *W, int K, long n0, long k0, __bf16 *tile) {
    const int t = threadIdx.x, r = t >> 2, kc = (t & 3) * 8;
    const bf16x8 v = *reinterpret_cast<const bf16x8 *>(W + weight_at((int)n0 + r, kc, K) + k0 * 16);
    *reinterpret_cast<bf16x8 *>(tile + r * kLdsRow + kc) = v;
}

// C[M, N] = sum_k A(m, k) B(n, k), M, N multiples of 64 and K of 32 (the
// host pads every dimension).  Four waves, each a 32 x 32 quarter of the
// tile as 2 x 2 matrix-core blocks of 16 x 16.  BLOCKED: B in the order of weight_at.
template <int EPI, bool BLOCKED = false>
__global__ __launch_bounds__(kGemmThreads) void gemm_kernel(Operand A, Operand B, int M, int N, int K, EpiArgs e) {
    __shared__ __attribute__((aligned(16))) __bf16 As[kTileM * kLdsRow];
    __shared__ __attribute__((aligned(16))) __bf16 Bs[kTileN * kLdsRow];
    const long m0 = (long)blockIdx.y * kTileM, n0 = (long)blockIdx.x * kTileN;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = (wave & 1) * 32, wn = (wave >> 1) * 32;
    const int fr = lane & 15, fk = (lane >> 4) * 8;
    floatx4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    // split K: slice blockIdx.z of gridDim.z takes K / gridDim.z of the sum
    const int kspan = K / (int)gridDim.z, kb = (int)blockIdx.z * kspan;
    for (int k0 = kb; k0 < kb + kspan; k0 += kTileK) {
        __syncthreads();
        stage(A, m0, k0, As);
        if (BLOCKED) stage_blocked(B.p, K, n0, k0, Bs);
        else stage(B, n0, k0, Bs);
        __syncthreads();
        bf16x8 a[2], b[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) a[i] = *reinterpret_cast<const bf16x8 *>(As + (wm + 16 * i + fr) * kLdsRow + fk);
#pragma unroll
        for (int j = 0; j < 2; ++j) b[j] = *reinterpret_cast<const bf16x8 *>(Bs + (wn + 16 * j + fr) * kLdsRow + fk);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    // lane holds rows 4 (lane / 16) + c of column lane % 16 of each block
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const long m = m0 + wm + 16 * i + (lane >> 4) * 4 + c;
                const long n = n0 + wn + 16 * j + (lane & 15);
                const float v = acc[i][j][c];
                if (EPI == kEpiHidden) {
                    float z = v + e.bias[n];
                    if (e.f32) e.f32[m * e.ld + n] = z;
                    e.b16[m * e.ld + n] = to_bf16(gelu(z));
                } else if (EPI == kEpiOut) {
                    float yn = v + e.bias[n];
                    if (e.f32) e.f32[m * e.ld + n] = yn;
                    if (e.y && m < e.batch && n < e.n_out) e.y[m * e.ldy + n] = __builtin_fmaf(e.sigma[n], yn, e.mu[n]);
                } else if (EPI == kEpiBackward) {
                    float dz = v * gelu_grad(e.z[m * e.ld + n]);
                    e.f32[m * e.ld + n] = dz;
                    e.b16[m * e.ld + n] = to_bf16(dz);
                } else {
                    e.f32[(long)blockIdx.z * e.split + m * e.ld + n] = v;
                }
            }
}

// x^ = (x - mu) * s in BF16, zero in padded rows and columns.
__global__ void normalise_kernel(const float *x, long ldx, int batch, int n_in, const float *mu, const float *s,
                                 __bf16 *xh, int rows, int fp) {
    long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (long)rows * fp) return;
    int b = (int)(idx / fp), i = (int)(idx - (long)b * fp);
    float v = 0.f;
    if (b < batch && i < n_in) v = (x[(long)b * ldx + i] - mu[i]) * s[i];
    xh[idx] = to_bf16(v);
}

// Output gradient of the mean squared error on standardised targets, and
// per-block partial sums of the squared error (fixed order).
__global__ void loss_grad_kernel(const float *yn, const float *t, int batch, int n_out, int op, const float *mu,
                                 const float *sigma, float *dy, __bf16 *dyb, int rows, float *partial) {
    __shared__ float red[256];
    long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    float sq = 0.f;
    if (idx < (long)rows * op) {
        int b = (int)(idx / op), o = (int)(idx - (long)b * op);
        float g = 0.f;
        if (b < batch && o < n_out) {
            float tn = (t[(long)b * n_out + o] - mu[o]) / sigma[o];
            float err = yn[idx] - tn;
            sq = err * err;
            g = 2.f * err / ((float)batch * (float)n_out);
        }
        dy[idx] = g;
        dyb[idx] = to_bf16(g);
    }
    red[threadIdx.x] = sq;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

__global__ void loss_final_kernel(const float *partial, int n, float scale, float *loss) {
    __shared__ float red[256];
    float s = 0.f;
    for (int i = threadIdx.x; i < n; i += 256) s += partial[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if (threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) loss[0] = red[0] * scale;
}

// Column sums of a [rows, n] FP32 matrix (bias gradients) in two passes
// with a fixed order: block (x, y) sums rows y*rows/ny .. of 64 columns in
// 4 row groups into partial[y][col]; then every column adds its ny partials.
__global__ __launch_bounds__(256) void colsum_partial_kernel(const float *a, int rows, int n, float *partial) {
    __shared__ float red[4][64];
    const int c = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int col = blockIdx.x * 64 + c;
    const int span = rows / (int)gridDim.y, r0 = (int)blockIdx.y * span;
    float s = 0.f;
    if (col < n)
        for (int r = r0 + g; r < r0 + span; r += 4) s += a[(long)r * n + col];
    red[g][c] = s;
    __syncthreads();
    if (g == 0 && col < n) partial[(long)blockIdx.y * n + col] = (red[0][c] + red[1][c]) + (red[2][c] + red[3][c]);
}

// out[i] = sum over s of part[s * stride + i], s in order (the partial
// results of a split sum)
__global__ void sum_slices_kernel(const float *part, long stride, int ns, long n, float *out) {
    long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float t = 0.f;
    for (int k = 0; k < ns; ++k) t += part[(long)k * stride + i];
    out[i] = t;
}

// A network of the row kernel keeps its BF16 weights in the order of weight_at, those of
// the second and third layer transposed as well; one of a product per layer keeps
// them row-major, whose 128-byte lines serve a tile of 32 columns and the next (in the
// other order a thousand rows of 667-576-224 took 64 us instead of 53).
struct Layout {
    long oW1, ob1, oW2, ob2, oW3, ob3, total;  // packed FP32 parameters
    long bW1, bW2, bW3, btotal;                // BF16 weight copies
    long bT2, bT3;                             // transposed ones, [H][H] and [H][op] (0: none)
    int fp, H, op;
};

// The BF16 copies of element (r, c) of layer p's weights in a network of the row kernel.
__device__ inline void store_weight(const Layout &L, int p, int r, int c, float wi, __bf16 *wb) {
    const __bf16 v = to_bf16(wi);
    if (p == 0) {
        wb[L.bW1 + weight_at(r, c, L.fp)] = v;
    } else if (p == 1) {
        wb[L.bW2 + weight_at(r, c, L.H)] = v;
        wb[L.bT2 + weight_at(c, r, L.H)] = v;
    } else {
        wb[L.bW3 + weight_at(r, c, L.H)] = v;
        wb[L.bT3 + weight_at(c, r, L.op)] = v;
    }
}

// Where the BF16 copy of parameter i lies in a network of a product per layer (-1: a bias).
__device__ inline long row_major_at(const Layout &L, long i) {
    if (i >= L.oW1 && i < L.ob1) return L.bW1 + (i - L.oW1);
    if (i >= L.oW2 && i < L.ob2) return L.bW2 + (i - L.oW2);
    if (i >= L.oW3 && i < L.ob3) return L.bW3 + (i - L.oW3);
    return -1;
}

// One bias-corrected Adam update of parameter i by its gradient.
__device__ inline float adam_update(float *w, float *m, float *v, long i, float gi, float lr, float c1, float c2) {
    const float mi = 0.9f * m[i] + 0.1f * gi;
    const float vi = 0.999f * v[i] + 0.001f * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float wi = w[i] - lr * (mi / c1) / (sqrtf(vi / c2) + 1e-8f);
    w[i] = wi;
    return wi;
}

// Bias-corrected Adam on the packed FP32 parameters; weights also refresh
// their BF16 copies (networks of a product per layer).
__global__ void adam_kernel(float *w, const float *g, float *m, float *v, long n, float lr, float c1, float c2,
                            Layout L, __bf16 *wb) {
    long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float wi = adam_update(w, m, v, i, g[i], lr, c1, c2);
    const long bi = row_major_at(L, i);
    if (bi >= 0) wb[bi] = to_bf16(wi);
}

__global__ void refresh_bf16_kernel(const float *w, Layout L, __bf16 *wb) {
    long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= L.total) return;
    const long bi = row_major_at(L, i);
    if (bi < 0) return;
    if (!L.bT2) {
        wb[bi] = to_bf16(w[i]);
        return;
    }
    const int p = i >= L.oW3 ? 2 : (i >= L.oW2 ? 1 : 0), cols = p ? L.H : L.fp;
    const long k = i - (p == 2 ? L.oW3 : (p == 1 ? L.oW2 : L.oW1));
    const int r = (int)(k / cols);
    store_weight(L, p, r, (int)(k - (long)r * cols), w[i], wb);
}

// s = 1 / sigma (0 for constant features); sigma_out floored at 1e-12 -> 1.
__global__ void set_norm_kernel(const float *mu_in, const float *sd_in, int n_in, const float *mu_out,
                                const float *sd_out, int n_out, float *mu_i, float *s_i, float *mu_o, float *sd_o) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n_in) {
        float sd = sd_in[i];
        mu_i[i] = mu_in[i];
        s_i[i] = sd > 1e-12f ? 1.f / sd : 0.f;
    }
    if (i < n_out) {
        float sd = sd_out[i];
        mu_o[i] = mu_out[i];
        sd_o[i] = sd > 1e-12f ? sd : 1.f;
    }
}

// ---- rows of the batch through the whole network ---------------------------
//
// A layer of this network is small (the biped's: 704 x 256, 256 x 256, 256 x 256)
// and a product of its own per layer is launch and load latency: 41 us for a
// batch of 1000 in four launches of 64-row tiles that waited for memory twice per
// 32 of K.  Instead a workgroup takes 16 or 32 rows through every layer, and in
// training back again: activations stay in LDS as BF16 operands, the
// activations' derivatives (FP32) in the registers of the lanes that computed them,
// and weights come from L2 straight into operand registers, four steps of K ahead
// (eight ahead, or every line touched at the start, gained nothing).  Every sum over
// K runs in the order of gemm_kernel, so outputs have its bits.  15.5 us for the
// batch of 1000 (3 standardising, 4 in the first layer's 360 KB of weights, 2 in each
// hidden layer's error functions, 3 of launch) on weights and inputs that are in the caches
// (42 us on inputs not seen before, 67 us in four launches); a training batch of 4096
// takes 31 us.

constexpr int kRowThreads = 512, kRowWaves = kRowThreads / 64;
constexpr int kRowTiles = 4;  // hidden column tiles a wave keeps, at most
constexpr int kAhead = 4;     // steps of K loaded ahead
constexpr int kRowLine = 256;  // workgroups of 16 rows, at most

struct RowArgs {
    const float *x;
    long ldx;
    int batch, n_in, fp, H, n_out, op, R;
    const float *mu_in, *s_in, *mu_out, *sd_out;
    const __bf16 *w1, *w2, *w3, *w2t, *w3t;
    const float *b1, *b2, *b3;
    float *y;  // prediction
    long ldy;
    // training: targets, activations and their gradients as operands of the weight
    // gradients ([R / 32][columns][32 rows]), the gradients' FP32 values [R][columns]
    // for the bias gradients, and the squared error per workgroup
    const float *t;
    const __bf16 *xh;  // prediction: the standardised input [R][fp] in x's place, or null
    __bf16 *xk, *h1k, *h2k, *dyk, *dz2k, *dz1k;
    float *dy, *dz2, *dz1, *loss_part;
};

__host__ __device__ inline int row_lda(int fp, int H) { return (fp > H ? fp : H) + 8; }
__host__ __device__ inline int row_ldb(int H, int op, bool train) { return (train && op > H ? op : H) + 8; }

inline size_t row_lds_bytes(int fp, int H, int op, int mb, bool train) {
    return sizeof(__bf16) * 16 * mb * (size_t)(row_lda(fp, H) + row_ldb(H, op, train));
}

// Networks whose rows fit 64 KB of LDS and whose hidden columns fit the registers;
// wider ones go through one product per layer.  Training keeps the derivatives of both
// hidden layers: 385 to 512 columns spill 115 registers a lane, 257 to 384 nine, and
// are still the faster path at every batch from 1 to 65536.  Microseconds of a
// training step, row kernel and one product per layer: 667-384-224 50 and 123 for 64
// rows, 74 and 235 for 4096, 1101 and 2214 for 65536; 667-512-224 77 and 130, 107 and
// 248, 1691 and 2559; 64-512-64 53 and 111, 76 and 193, 1109 and 1588.
inline bool rows_kernel_takes(int fp, int H, int op) {
    return H <= 16 * kRowTiles * kRowWaves && row_lds_bytes(fp, H, op, 1, true) <= kPlainLds;
}

// Weights of up to TN column tiles on their way from L2: kAhead steps of K.  The first
// steps of a layer are asked for before the layer in front of it has ended.
template <int TN>
struct Weights {
    const __bf16 *w[TN];
    int K;
    bf16x8 b[kAhead][TN];
    // W [n][K] in the order of weight_at, K a multiple of 64
    __device__ inline void begin(const __bf16 *W, int K_, const int (&tile)[TN]) {
        const int lane = threadIdx.x & 63;
        K = K_;
#pragma unroll
        for (int j = 0; j < TN; ++j) w[j] = W + (long)tile[j] * (K >> 5) * 512 + (lane & 15) * 32 + (lane >> 4) * 8;
        load(0);
    }
    __device__ inline void load(int k0) {
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
            const int k = (min(k0 + kTileK * q, K - kTileK) >> 5) * 512;  // (past the end: not used)
#pragma unroll
            for (int j = 0; j < TN; ++j) b[q][j] = *reinterpret_cast<const bf16x8 *>(w[j] + k);
        }
    }
};

// acc[i][j] = sum over k of act(16 i + row, k) W(16 tile[j] + column, k); act in LDS
// (row stride ld).
template <int MB, int TN>
__device__ inline void rows_times(const __bf16 *act, int ld, Weights<TN> &W, floatx4 (&acc)[MB][TN]) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    const __bf16 *a0 = act + (lane & 15) * ld + (lane >> 4) * 8;
    for (int k0 = 0; k0 < W.K; k0 += kTileK * kAhead) {
        bf16x8 c[kAhead][TN];
#pragma unroll
        for (int q = 0; q < kAhead; ++q)
#pragma unroll
            for (int j = 0; j < TN; ++j) c[q][j] = W.b[q][j];
        if (k0 + kTileK * kAhead < W.K) W.load(k0 + kTileK * kAhead);
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
            if (k0 + kTileK * q >= W.K) break;
            bf16x8 av[MB];
#pragma unroll
            for (int i = 0; i < MB; ++i) av[i] = *reinterpret_cast<const bf16x8 *>(a0 + 16 * i * ld + k0 + kTileK * q);
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[i], c[q][j], acc[i][j], 0, 0, 0);
        }
    }
}

using bf16x4 = __bf16 __attribute__((ext_vector_type(4)));

// Four consecutive rows (from m, a multiple of 4) of column c, as an operand of a
// sum over the rows.
__device__ inline void store_k(__bf16 *o, int cols, long m, int c, bf16x4 v) {
    *reinterpret_cast<bf16x4 *>(o + ((m >> 5) * cols + c) * 32 + (m & 31)) = v;
}

template <int MB, int TN, bool TRAIN>
__global__ __launch_bounds__(kRowThreads) void rows_kernel(RowArgs a) {
    extern __shared__ float4 row_lds[];
    __shared__ float red[kRowWaves];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, rg = (lane >> 4) * 4, fr = lane & 15;
    constexpr int kRows = 16 * MB;
    const long m0 = (long)blockIdx.x * kRows;
    const int lda = row_lda(a.fp, a.H), ldb = row_ldb(a.H, a.op, TRAIN);
    __bf16 *P = reinterpret_cast<__bf16 *>(row_lds), *Q = P + kRows * lda;
    const int H = a.H, ht = H / 16, ot = a.op / 16;

    int tile[TN];
    bool mine[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        mine[j] = wave + kRowWaves * j < ht;
        tile[j] = min(wave + kRowWaves * j, ht - 1);
    }
    // (biases, and below the output layer's scales and targets, ahead of the weights
    // asked for with them: loads return in order, and an epilogue that loaded its own
    // waited for all of the next layer's)
    float b1[TN], b2[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        b1[j] = a.b1[16 * tile[j] + fr];
        b2[j] = a.b2[16 * tile[j] + fr];
    }
    Weights<TN> W;
    W.begin(a.w1, a.fp, tile);

    // x^ = (x - mu) s in BF16, zero in padded rows and columns: a wave's 2 MB rows
    // together, six loads of each in flight
    constexpr int kWaveRows = kRows / kRowWaves, kLoads = 6;
    const bool given = !TRAIN && a.xh;
    if (given)
        for (int i = threadIdx.x; i < kRows * (a.fp / 8); i += kRowThreads) {
            const int r = i / (a.fp / 8), c = 8 * (i - r * (a.fp / 8));
            *reinterpret_cast<bf16x8 *>(P + r * lda + c) = *reinterpret_cast<const bf16x8 *>(a.xh + (m0 + r) * a.fp + c);
        }
    for (int c0 = given ? a.fp : lane; c0 < a.fp; c0 += 64 * kLoads) {
        float v[kWaveRows][kLoads], mu[kLoads], sd[kLoads];
#pragma unroll
        for (int e = 0; e < kLoads; ++e) {
            const int c = min(c0 + 64 * e, a.n_in - 1);
            mu[e] = a.mu_in[c];
            sd[e] = a.s_in[c];
#pragma unroll
            for (int q = 0; q < kWaveRows; ++q)
                v[q][e] = a.x[min(m0 + wave + kRowWaves * q, (long)a.batch - 1) * a.ldx + c];
        }
#pragma unroll
        for (int e = 0; e < kLoads; ++e) {
            const int c = c0 + 64 * e;
            if (c >= a.fp) break;
#pragma unroll
            for (int q = 0; q < kWaveRows; ++q) {
                const int r = wave + kRowWaves * q;
                P[r * lda + c] = to_bf16(m0 + r < a.batch && c < a.n_in ? (v[q][e] - mu[e]) * sd[e] : 0.f);
            }
        }
    }
    __syncthreads();
    if (TRAIN)
        for (int i = threadIdx.x; i < a.fp * (kRows / 4); i += kRowThreads) {
            const int c = i / (kRows / 4), r = 4 * (i % (kRows / 4));
            const bf16x4 v = {P[r * lda + c], P[(r + 1) * lda + c], P[(r + 2) * lda + c], P[(r + 3) * lda + c]};
            store_k(a.xk, a.fp, m0 + r, c, v);
        }

    // z = act W^T + b; gelu(z) to LDS, and for the way back gelu'(z), which shares its
    // error function
    floatx4 acc[MB][TN], d1[MB][TN], d2[MB][TN];
    auto hidden = [&](const float (&bias)[TN], floatx4 (&dg)[MB][TN], __bf16 *h, int ld, __bf16 *hk) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int n = 16 * tile[j] + fr;
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                bf16x4 o;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const float zv = acc[i][j][c] + bias[j];
                    o[c] = to_bf16(gelu(zv));
                    if (TRAIN) dg[i][j][c] = gelu_grad(zv);
                }
                if (mine[j]) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) h[(16 * i + rg + c) * ld + n] = o[c];
                    if (TRAIN) store_k(hk, H, m0 + 16 * i + rg, n, o);
                }
            }
        }
    };
    rows_times<MB, TN>(P, lda, W, acc);
    W.begin(a.w2, H, tile);
    hidden(b1, d1, Q, ldb, a.h1k);
    __syncthreads();
    rows_times<MB, TN>(Q, ldb, W, acc);
    int otile[TN];
    float b3[TN], mu[TN], sd[TN], target[MB][TN][4];
    auto out_tiles = [&](int t0) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            otile[j] = min(t0 + kRowWaves * j, ot - 1);
            const int n = 16 * otile[j] + fr, nr = min(n, a.n_out - 1);
            b3[j] = a.b3[n];
            mu[j] = a.mu_out[nr];
            sd[j] = a.sd_out[nr];
            if (TRAIN) {
#pragma unroll
                for (int i = 0; i < MB; ++i)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        target[i][j][c] = a.t[min(m0 + 16 * i + rg + c, (long)a.batch - 1) * a.n_out + nr];
            }
        }
        W.begin(a.w3, H, otile);
    };
    out_tiles(wave);
    hidden(b2, d2, P, lda, a.h2k);
    __syncthreads();

    // outputs, in training their gradients of the mean squared error
    float sq = 0.f;
    for (int t0 = wave; t0 < ot; t0 += kRowWaves * TN) {
        if (t0 != wave) out_tiles(t0);
        rows_times<MB, TN>(P, lda, W, acc);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            if (t0 + kRowWaves * j >= ot) break;
            const int n = 16 * otile[j] + fr;
            const bool real = n < a.n_out;
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                bf16x4 o;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const long m = m0 + 16 * i + rg + c;
                    const float yn = acc[i][j][c] + b3[j];
                    if (TRAIN) {
                        float g = 0.f;
                        if (real && m < a.batch) {
                            const float tn = (target[i][j][c] - mu[j]) / sd[j];
                            const float err = yn - tn;
                            sq += err * err;
                            g = 2.f * err / ((float)a.batch * (float)a.n_out);
                        }
                        a.dy[m * a.op + n] = g;
                        o[c] = to_bf16(g);
                        Q[(16 * i + rg + c) * ldb + n] = o[c];
                    } else if (real && m < a.batch) {
                        a.y[m * a.ldy + n] = __builtin_fmaf(sd[j], yn, mu[j]);
                    }
                }
                if (TRAIN) store_k(a.dyk, a.op, m0 + 16 * i + rg, n, o);
            }
        }
    }
    if (!TRAIN) return;
    W.begin(a.w3t, a.op, tile);
    for (int o = 1; o < 64; o <<= 1) sq += __shfl_xor(sq, o);
    if (lane == 0) red[wave] = sq;
    __syncthreads();
    if (threadIdx.x == 0) {
        float s = 0.f;
        for (int k = 0; k < kRowWaves; ++k) s += red[k];
        a.loss_part[blockIdx.x] = s;
    }

    // dz = (d W) gelu'(z)
    auto back = [&](const floatx4 (&dg)[MB][TN], __bf16 *d, float *d32, __bf16 *dk) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            if (!mine[j]) break;
            const int n = 16 * tile[j] + fr;
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                bf16x4 o;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const float dz = acc[i][j][c] * dg[i][j][c];
                    d32[(m0 + 16 * i + rg + c) * H + n] = dz;
                    o[c] = to_bf16(dz);
                    if (d) d[(16 * i + rg + c) * lda + n] = o[c];
                }
                store_k(dk, H, m0 + 16 * i + rg, n, o);
            }
        }
    };
    rows_times<MB, TN>(Q, ldb, W, acc);
    W.begin(a.w2t, H, tile);
    back(d2, P, a.dz2, a.dz2k);
    __syncthreads();
    rows_times<MB, TN>(P, lda, W, acc);
    back(d1, nullptr, a.dz1, a.dz1k);
}

// The gradients of a training step and Adam's update in one launch: 24 us for a
// batch of 4096, where a product, a sum of its slices, two passes of column sums per
// layer and the update were thirteen launches and about 120 us.  A workgroup owns a
// 32 x 32 tile of a layer's weights: C[M, N] = sum over the rows of A(m, row) B(n, row),
// operands as rows_kernel writes them (1 KB of consecutive memory each).  Its 16 waves
// take a slice of the rows each, and the slices are added in order from LDS; through
// global memory their partial results were 28 MB written and read.  8 columns of
// the biases' sums are another workgroup's, in kColBlocks row ranges of four
// interleaved groups.
struct GradArgs {
    const __bf16 *A[3], *B[3];
    const float *d[3];
    int M[3], N[3], ns[3], first[3], col_first[3];  // first: a product's first workgroup
    int R, cols, loss_blocks;
    float *w, *g, *m, *v;
    float lr, c1, c2, loss_scale;
    const float *loss_part;
    float *loss;
    Layout L;
    __bf16 *wb;
};

constexpr int kGradWaves = 16;
static_assert(2 * kGradWaves == kColBlocks, "a thread per column, row group and row range");

__global__ __launch_bounds__(64 * kGradWaves) void grads_kernel(GradArgs g) {
    __shared__ float part[kGradWaves][1024];
    const Layout &L = g.L;
    const int bx = (int)blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (bx < g.loss_blocks) {
        float s = 0.f;
        for (int k = tid; k < g.R / 16; k += 64 * kGradWaves) s += g.loss_part[k];
        part[0][tid] = s;
        __syncthreads();
        for (int k = 32 * kGradWaves; k > 0; k >>= 1) {
            if (tid < k) part[0][tid] += part[0][tid + k];
            __syncthreads();
        }
        if (tid == 0) g.loss[0] = part[0][0] * g.loss_scale;
        return;
    }
    if (bx < g.first[0]) {
        // thread: column, row group, row range (neighbouring columns on one XCD: they share
        // cache lines)
        const int b = bx - g.loss_blocks, col = 8 * ((b & 7) * (g.cols / 64) + (b >> 3)) + (tid & 7);
        const int grp = (tid >> 3) & 3, y = tid >> 5;
        const int p = col >= g.col_first[2] ? 2 : (col >= g.col_first[1] ? 1 : 0);
        const int n = g.M[p], c = col - g.col_first[p], span = g.R / kColBlocks, rows = (span - grp + 3) / 4;
        const float *d = g.d[p] + (long)(y * span + grp) * n + c;
        float s = 0.f;
        for (int r = 0; r < rows; r += 16) {
            float v[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) v[q] = d[4l * min(r + q, rows - 1) * n];
            __builtin_amdgcn_sched_barrier(0);  // (all loads in flight)
#pragma unroll
            for (int q = 0; q < 16; ++q)
                if (r + q < rows) s += v[q];
        }
        part[0][tid] = s;
        __syncthreads();
        if (tid < 8) {
            float t = 0.f;
#pragma unroll
            for (int k = 0; k < kColBlocks; ++k) {
                const float *q = &part[0][32 * k + tid];
                t += (q[0] + q[8]) + (q[16] + q[24]);
            }
            const long i = (p == 2 ? L.ob3 : (p == 1 ? L.ob2 : L.ob1)) + c;
            g.g[i] = t;
            adam_update(g.w, g.m, g.v, i, t, g.lr, g.c1, g.c2);
        }
        return;
    }
    const int p = bx >= g.first[2] ? 2 : (bx >= g.first[1] ? 1 : 0);
    const int M = g.M[p], N = g.N[p], tn = N / 32, at = bx - g.first[p];
    // (workgroups go round the eight XCDs: a row of tiles on one, so that its L2 holds
    // the row's operand)
    const bool rows8 = (M / 32) % 8 == 0;
    const int tm = rows8 ? (at & 7) + 8 * ((at >> 3) / tn) : at / tn, tc = rows8 ? (at >> 3) % tn : at % tn;
    const int off = (lane & 15) * 32 + (lane >> 4) * 8, ns = g.ns[p], nk = g.R / kTileK / ns;
    const __bf16 *A = g.A[p] + (long)tm * 1024 + off, *B = g.B[p] + (long)tc * 1024 + off;
    // this thread's element of the tile
    const int em = tid >> 5, en = tid & 31;
    auto place = [](int m, int n) { return 32 * m + (n ^ ((m & 4) << 2)); };  // (rows 4 apart in other banks)
    float total = ns > 1 ? 0.f : -0.f;
    for (int s0 = 0; s0 < ns; s0 += kGradWaves) {
        const int slice = s0 + wave;
        if (slice < ns) {
            floatx4 acc[2][2];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
            const int k1 = (slice + 1) * nk;
            for (int k = slice * nk; k < k1; k += kAhead) {
                bf16x8 fa[kAhead][2], fb[kAhead][2];
#pragma unroll
                for (int q = 0; q < kAhead; ++q) {
                    const long kk = min(k + q, k1 - 1);  // (past the end: not used)
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        fa[q][i] = *reinterpret_cast<const bf16x8 *>(A + (kk * M + 16 * i) * 32);
                        fb[q][i] = *reinterpret_cast<const bf16x8 *>(B + (kk * N + 16 * i) * 32);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);  // (all loads in flight)
#pragma unroll
                for (int q = 0; q < kAhead; ++q) {
                    if (k + q >= k1) break;
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[q][i], fb[q][j], acc[i][j], 0, 0, 0);
                }
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        part[wave][place(16 * i + (lane >> 4) * 4 + c, 16 * j + (lane & 15))] = acc[i][j][c];
        }
        __syncthreads();
        float e[kGradWaves];
#pragma unroll
        for (int k = 0; k < kGradWaves; ++k) e[k] = part[k][place(em, en)];
#pragma unroll
        for (int k = 0; k < kGradWaves; ++k)
            if (s0 + k < ns) total += e[k];
        __syncthreads();
    }
    const int r = 32 * tm + em, c = 32 * tc + en;
    const long i = (p == 2 ? L.oW3 : (p == 1 ? L.oW2 : L.oW1)) + (long)r * N + c;
    g.g[i] = total;
    store_weight(L, p, r, c, adam_update(g.w, g.m, g.v, i, total, g.lr, g.c1, g.c2), g.wb);
}

inline int pad64(int n) { return (n + 63) / 64 * 64; }

}  // namespace
}  // namespace kamx

using namespace kamx;

struct kamx_mlp_s {
    int n_in = 0, fp = 0, H = 0, n_out = 0, op = 0, cap = 0;
    Layout L{};
    int t = 0;  // Adam steps taken
    float *w = nullptr, *g = nullptr, *am = nullptr, *av = nullptr;
    __bf16 *wb = nullptr;
    float *mu_in = nullptr, *s_in = nullptr, *mu_out = nullptr, *sd_out = nullptr;
    __bf16 *xh = nullptr, *h1 = nullptr, *h2 = nullptr, *dyb = nullptr, *dz2b = nullptr, *dz1b = nullptr;
    float *z1 = nullptr, *z2 = nullptr, *yn = nullptr, *dy = nullptr, *dz2 = nullptr, *dz1 = nullptr;
    float *partial = nullptr;
    float *ws = nullptr;  // partial sums of split weight gradients and bias gradients
    long ws_floats = 0;
    bool fused = false;  // the row kernel takes this network
    std::vector<void *> allocs;
};

namespace kamx {
// errors of this file go through the library's thread-local message
kamx_status mlp_fail(kamx_status st, const char *fmt, ...);
}  // namespace kamx

#define MLP_HIP(expr)                                                                                 \
    do {                                                                                              \
        hipError_t e_ = (expr);                                                                       \
        if (e_ != hipSuccess) return mlp_fail(KAMX_EDEVICE, "%s: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

template <typename T>
static kamx_status mlp_alloc(kamx_mlp n, T **p, size_t count) {
    void *ptr = nullptr;
    size_t bytes = std::max<size_t>(count, 1) * sizeof(T);
    hipError_t e = hipMalloc(&ptr, bytes);
    if (e != hipSuccess) return mlp_fail(KAMX_ENOMEM, "hipMalloc(%zu bytes): %s", bytes, hipGetErrorString(e));
    e = hipMemset(ptr, 0, bytes);
    if (e != hipSuccess) return mlp_fail(KAMX_EDEVICE, "hipMemset: %s", hipGetErrorString(e));
    n->allocs.push_back(ptr);
    *p = reinterpret_cast<T *>(ptr);
    return KAMX_OK;
}

static void mlp_free(kamx_mlp n) {
    for (void *p : n->allocs) (void)hipFree(p);
    delete n;
}

// splitmix64 (Steele, Lea and Flood 2014) for the initial weights
static uint64_t splitmix(uint64_t &s) {
    uint64_t z = (s += 0x9E3779B97F4A7C15ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

extern "C" kamx_status kamx_mlp_create(int32_t n_in, int32_t n_hidden, int32_t n_out, int32_t max_batch, uint64_t seed,
                                       kamx_mlp *out) {
    if (!out) return mlp_fail(KAMX_EINVAL, "out is NULL");
    *out = nullptr;
    if (n_in < 1 || n_in > 65536 || n_out < 1 || n_out > 65536 || n_hidden < 64 || n_hidden > 4096 ||
        n_hidden % 64 != 0 || max_batch < 1 || max_batch > (1 << 22))
        return mlp_fail(KAMX_EINVAL, "bad sizes (n_hidden must be a multiple of 64 in [64, 4096])");
    kamx_mlp n = new kamx_mlp_s;
    n->n_in = n_in;
    n->fp = pad64(n_in);
    n->H = n_hidden;
    n->n_out = n_out;
    n->op = pad64(n_out);
    n->cap = pad64(max_batch);
    Layout &L = n->L;
    const long H = n_hidden, fp = n->fp, op = n->op;
    L.oW1 = 0;
    L.ob1 = L.oW1 + H * fp;
    L.oW2 = L.ob1 + H;
    L.ob2 = L.oW2 + H * H;
    L.oW3 = L.ob2 + H;
    L.ob3 = L.oW3 + op * H;
    L.total = L.ob3 + op;
    L.bW1 = 0;
    L.bW2 = H * fp;
    L.bW3 = L.bW2 + H * H;
    L.btotal = L.bW3 + op * H;
    L.fp = n->fp;
    L.H = n->H;
    L.op = n->op;
    n->fused = rows_kernel_takes(n->fp, n->H, n->op);
    if (n->fused) {
        L.bT2 = L.btotal;
        L.bT3 = L.bT2 + H * H;
        L.btotal = L.bT3 + H * op;
    }
#define C_TRY(expr)                      \
    do {                                 \
        kamx_status s_ = (expr);         \
        if (s_ != KAMX_OK) {             \
            mlp_free(n);                 \
            return s_;                   \
        }                                \
    } while (0)
    C_TRY(mlp_alloc(n, &n->w, L.total));
    C_TRY(mlp_alloc(n, &n->g, L.total));
    C_TRY(mlp_alloc(n, &n->am, L.total));
    C_TRY(mlp_alloc(n, &n->av, L.total));
    C_TRY(mlp_alloc(n, &n->wb, L.btotal));
    C_TRY(mlp_alloc(n, &n->mu_in, fp));
    C_TRY(mlp_alloc(n, &n->s_in, fp));
    C_TRY(mlp_alloc(n, &n->mu_out, op));
    C_TRY(mlp_alloc(n, &n->sd_out, op));
    const long R = n->cap;
    C_TRY(mlp_alloc(n, &n->xh, R * fp));
    C_TRY(mlp_alloc(n, &n->h1, R * H));
    C_TRY(mlp_alloc(n, &n->h2, R * H));
    C_TRY(mlp_alloc(n, &n->dyb, R * op));
    C_TRY(mlp_alloc(n, &n->dz2b, R * H));
    C_TRY(mlp_alloc(n, &n->dz1b, R * H));
    if (!n->fused) {
        C_TRY(mlp_alloc(n, &n->z1, R * H));
        C_TRY(mlp_alloc(n, &n->z2, R * H));
        C_TRY(mlp_alloc(n, &n->yn, R * op));
        C_TRY(mlp_alloc(n, &n->partial, (R * std::max<long>(op, 1) + 255) / 256));
    }
    C_TRY(mlp_alloc(n, &n->dy, R * op));
    C_TRY(mlp_alloc(n, &n->dz2, R * H));
    C_TRY(mlp_alloc(n, &n->dz1, R * H));
    {
        // split-K weight gradients: each of M x N outputs gets up to
        // grad_splits(...) partials for the padded batch K of a training
        // call (any multiple of 64 up to the capacity: a smaller batch can
        // take more slices than the capacity itself); bias gradients up to
        // kColBlocks.  The fused step only leaves its row blocks' losses
        long most = (long)kColBlocks * std::max(H, op);
        for (long K = 64; K <= R && !n->fused; K += 64) {
            const long a = (long)grad_splits(op, H, (int)K) * op * H, b = (long)grad_splits(H, H, (int)K) * H * H,
                       c = (long)grad_splits(H, fp, (int)K) * H * fp;
            most = std::max(most, std::max(a, std::max(b, c)));
        }
        if (n->fused) most = R / 16;
        n->ws_floats = most;
        C_TRY(mlp_alloc(n, &n->ws, n->ws_floats));
    }
    // initial weights U(-1/sqrt(fan_in), 1/sqrt(fan_in)) on the active
    // entries, zero on padding; identity normalisation
    std::vector<float> w(L.total, 0.f), one_in(fp, 1.f), one_out(op, 1.f);
    uint64_t s = seed;
    auto uni = [&](float a) { return a * (2.f * (float)((splitmix(s) >> 40) * (1.0 / 16777216.0)) - 1.f); };
    const float a1 = 1.f / sqrtf((float)n_in), a2 = 1.f / sqrtf((float)H);
    for (long h = 0; h < H; ++h)
        for (long i = 0; i < n_in; ++i) w[L.oW1 + h * fp + i] = uni(a1);
    for (long h = 0; h < H; ++h) w[L.ob1 + h] = uni(a1);
    for (long h = 0; h < H * H; ++h) w[L.oW2 + h] = uni(a2);
    for (long h = 0; h < H; ++h) w[L.ob2 + h] = uni(a2);
    for (long o = 0; o < n_out; ++o)
        for (long h = 0; h < H; ++h) w[L.oW3 + o * H + h] = uni(a2);
    for (long o = 0; o < n_out; ++o) w[L.ob3 + o] = uni(a2);
    hipError_t e = hipMemcpy(n->w, w.data(), sizeof(float) * L.total, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(n->s_in, one_in.data(), sizeof(float) * fp, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(n->sd_out, one_out.data(), sizeof(float) * op, hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        mlp_free(n);
        return mlp_fail(KAMX_EDEVICE, "weight upload: %s", hipGetErrorString(e));
    }
    hipLaunchKernelGGL(refresh_bf16_kernel, dim3((unsigned)((L.total + 255) / 256)), dim3(256), 0, 0, n->w, L, n->wb);
    e = hipDeviceSynchronize();
    if (e != hipSuccess) {
        mlp_free(n);
        return mlp_fail(KAMX_EDEVICE, "weight conversion: %s", hipGetErrorString(e));
    }
#undef C_TRY
    *out = n;
    return KAMX_OK;
}

extern "C" kamx_status kamx_mlp_destroy(kamx_mlp n) {
    if (!n) return KAMX_OK;
    (void)hipDeviceSynchronize();
    mlp_free(n);
    return KAMX_OK;
}

extern "C" kamx_status kamx_mlp_info(kamx_mlp n, int32_t *n_in_pad, int32_t *n_out_pad, int64_t *n_params) {
    if (!n) return mlp_fail(KAMX_EINVAL, "network is NULL");
    if (n_in_pad) *n_in_pad = n->fp;
    if (n_out_pad) *n_out_pad = n->op;
    if (n_params) *n_params = n->L.total;
    return KAMX_OK;
}

extern "C" kamx_status kamx_mlp_set_normalization(kamx_mlp n, const float *mu_in, const float *sigma_in,
                                                  const float *mu_out, const float *sigma_out, kamx_stream stream) {
    if (!n || !mu_in || !sigma_in || !mu_out || !sigma_out) return mlp_fail(KAMX_EINVAL, "NULL argument");
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    int m = std::max(n->n_in, n->n_out);
    hipLaunchKernelGGL(set_norm_kernel, dim3((m + 255) / 256), dim3(256), 0, s, mu_in, sigma_in, n->n_in, mu_out,
                       sigma_out, n->n_out, n->mu_in, n->s_in, n->mu_out, n->sd_out);
    MLP_HIP(hipGetLastError());
    return KAMX_OK;
}

template <int EPI, bool BLOCKED = false>
static hipError_t gemm(const Operand &A, const Operand &B, int M, int N, int K, const EpiArgs &e, hipStream_t s) {
    if (M % kTileM || N % kTileN || K % kTileK || M <= 0 || N <= 0 || K <= 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL((gemm_kernel<EPI, BLOCKED>), dim3(N / kTileN, M / kTileM), dim3(kGemmThreads), 0, s, A, B, M, N, K, e);
    return hipGetLastError();
}

// C = A B^T summed over K into c (ldc = N), split over K with the partial
// results reduced in slice order
static hipError_t gemm_store(kamx_mlp n, const Operand &A, const Operand &B, int M, int N, int K, float *c,
                             hipStream_t s) {
    if (M % kTileM || N % kTileN || K % kTileK || M <= 0 || N <= 0 || K <= 0) return hipErrorInvalidValue;
    const int ns = grad_splits(M, N, K);
    if ((long)ns * M * N > n->ws_floats) return hipErrorInvalidValue;
    EpiArgs e{};
    e.f32 = ns > 1 ? n->ws : c;
    e.ld = N;
    e.split = (long)M * N;
    hipLaunchKernelGGL(gemm_kernel<kEpiStore>, dim3(N / kTileN, M / kTileM, ns), dim3(kGemmThreads), 0, s, A, B, M,
                       N, K, e);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess || ns == 1) return err;
    const long cnt = (long)M * N;
    hipLaunchKernelGGL(sum_slices_kernel, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, s, n->ws, cnt, ns, cnt,
                       c);
    return hipGetLastError();
}

// bias gradient: column sums of a [rows, cols] matrix
static hipError_t colsum(kamx_mlp n, const float *a, int rows, int cols, float *out, hipStream_t s) {
    int nb = kColBlocks;
    while (nb > 1 && rows % nb) nb >>= 1;
    hipLaunchKernelGGL(colsum_partial_kernel, dim3((cols + 63) / 64, nb), dim3(256), 0, s, a, rows, cols, n->ws);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(sum_slices_kernel, dim3((unsigned)((cols + 255) / 256)), dim3(256), 0, s, n->ws, (long)cols, nb,
                       (long)cols, out);
    return hipGetLastError();
}

static RowArgs row_args(kamx_mlp n, const float *x, long ldx, int batch) {
    const Layout &L = n->L;
    RowArgs r{};
    r.x = x;
    r.ldx = ldx;
    r.batch = batch;
    r.n_in = n->n_in;
    r.fp = n->fp;
    r.H = n->H;
    r.n_out = n->n_out;
    r.op = n->op;
    r.R = pad64(batch);
    r.mu_in = n->mu_in;
    r.s_in = n->s_in;
    r.mu_out = n->mu_out;
    r.sd_out = n->sd_out;
    r.w1 = n->wb + L.bW1;
    r.w2 = n->wb + L.bW2;
    r.w3 = n->wb + L.bW3;
    r.w2t = n->wb + L.bT2;
    r.w3t = n->wb + L.bT3;
    r.b1 = n->w + L.ob1;
    r.b2 = n->w + L.ob2;
    r.b3 = n->w + L.ob3;
    return r;
}

template <int MB, int TN, bool TRAIN>
static hipError_t launch_rows_tn(const RowArgs &r, hipStream_t s) {
    const size_t lds = row_lds_bytes(r.fp, r.H, r.op, MB, TRAIN);
    hipError_t e = allow_lds(reinterpret_cast<const void *>(&rows_kernel<MB, TN, TRAIN>), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((rows_kernel<MB, TN, TRAIN>), dim3((unsigned)(r.R / (16 * MB))), dim3(kRowThreads), lds, s, r);
    return hipGetLastError();
}

template <int MB, bool TRAIN>
static hipError_t launch_rows_mb(const RowArgs &r, hipStream_t s) {
    switch ((r.H + 16 * kRowWaves - 1) / (16 * kRowWaves)) {
    case 1: return launch_rows_tn<MB, 1, TRAIN>(r, s);
    case 2: return launch_rows_tn<MB, 2, TRAIN>(r, s);
    case 3: return launch_rows_tn<MB, 3, TRAIN>(r, s);
    case 4: return launch_rows_tn<MB, 4, TRAIN>(r, s);
    default: return hipErrorInvalidValue;
    }
}

// A prediction takes 16 rows a workgroup while that is not more than one workgroup per
// CU, then 32, which halves the weights' traffic.  Microseconds of 16 and 32 rows a
// workgroup: 667-256-224 15.4 and 16.8 for 4096 rows, 23.3 and 16.8 for 4160, 25.8 and
// 19.3 for 8192; 1300-256-100, whose 32 rows take 107 KB of LDS, 23.9 and 25.8, 36.4 and
// 26.0, 38.0 and 27.6; 667-512-224 32.7 and 36.3, 63.2 and 37.3, 66.8 and 39.0.  (Training
// keeps two layers' derivatives in registers and takes 16.)
static hipError_t predict_rows(const RowArgs &r, hipStream_t s) {
    return r.R > 16 * kRowLine ? launch_rows_mb<2, false>(r, s) : launch_rows_mb<1, false>(r, s);
}

// One training step: rows forward and back, weight gradients, update.
static hipError_t train_fused(kamx_mlp n, const float *x, const float *target, int batch, float lr, float *loss,
                              hipStream_t s) {
    const Layout &L = n->L;
    const int H = n->H, fp = n->fp, op = n->op, R = pad64(batch);
    RowArgs r = row_args(n, x, n->n_in, batch);
    r.t = target;
    r.xk = n->xh;
    r.h1k = n->h1;
    r.h2k = n->h2;
    r.dyk = n->dyb;
    r.dz2k = n->dz2b;
    r.dz1k = n->dz1b;
    r.dy = n->dy;
    r.dz2 = n->dz2;
    r.dz1 = n->dz1;
    r.loss_part = n->ws;
    hipError_t e = launch_rows_mb<1, true>(r, s);
    if (e != hipSuccess) return e;
    // (layer order of the parameters)
    const __bf16 *A[3] = {n->dz1b, n->dz2b, n->dyb}, *B[3] = {n->xh, n->h1, n->h2};
    const float *d[3] = {n->dz1, n->dz2, n->dy};
    GradArgs g{};
    g.loss_blocks = loss ? 1 : 0;
    g.cols = 2 * H + op;
    int wgs = g.loss_blocks + g.cols / 8, col = 0;
    for (int p = 0; p < 3; ++p) {
        const int M = p < 2 ? H : op, N = p ? H : fp;
        g.A[p] = A[p];
        g.B[p] = B[p];
        g.d[p] = d[p];
        g.M[p] = M;
        g.N[p] = N;
        g.ns[p] = grad_splits(M, N, R);
        g.first[p] = wgs;
        g.col_first[p] = col;
        wgs += (M / 32) * (N / 32);
        col += M;
    }
    g.R = R;
    g.w = n->w;
    g.g = n->g;
    g.m = n->am;
    g.v = n->av;
    g.lr = lr;
    g.c1 = (float)(1.0 - pow(0.9, n->t + 1));
    g.c2 = (float)(1.0 - pow(0.999, n->t + 1));
    g.loss_scale = 1.f / ((float)batch * (float)n->n_out);
    g.loss_part = n->ws;
    g.loss = loss;
    g.L = L;
    g.wb = n->wb;
    hipLaunchKernelGGL(grads_kernel, dim3(wgs), dim3(64 * kGradWaves), 0, s, g);
    return hipGetLastError();
}

// Where one product per layer predicts faster than the row kernel although the network
// fits it: its workgroup of a wide hidden layer (172 registers a lane from 257 columns
// on) has a CU to itself, with nothing beside its error functions.  That shows once
// each CU has more than four workgroups to run and these little else to do: inputs and
// outputs of at most 3/4 of the hidden columns together where the columns leave some of
// the waves a tile short, of 3/8 where every wave has four, and not where every wave
// has three.  Microseconds for 131072 rows, products and row kernel: 64-320-64 179 and
// 216, 64-448-128 301 and 375, 64-512-64 318 and 343; but 64-384-64 215 and 222 (at
// half the rows 110 and 101), 128-512-256 449 and 397, 192-320-256 313 and 270.
static bool products_faster(kamx_mlp n, int R) {
    const int each = 16 * kRowWaves;  // hidden columns at a tile to a wave
    const int eighths = n->H % each ? 6 : (n->H > 3 * each ? 3 : 0);
    return R > 4 * 32 * kRowLine && n->H > 2 * each && 8 * (n->fp + n->op) <= eighths * n->H;
}

// Activations of one forward pass: the normalised BF16 input, the two
// BF16 hidden activations and, for training, the FP32 pre-activations and
// normalised outputs (null when only the prediction is wanted).
struct Acts {
    __bf16 *xh, *h1, *h2;
    float *z1, *z2, *yn;
};

// forward over rows padded to a multiple of 64; y (optional) receives the
// de-standardised outputs of the first batch rows
static kamx_status mlp_forward_rows(kamx_mlp n, const Acts &a, const float *x, long ldx, int batch, float *y,
                                    long ldy, hipStream_t s) {
    const int R = pad64(batch), H = n->H, fp = n->fp, op = n->op;
    const Layout &L = n->L;
    const bool rows = n->fused && !a.z1 && !products_faster(n, R);
    // the row kernel writes a workgroup's outputs while others still read their inputs, so
    // outputs over their inputs (the arrays share memory) have the inputs standardised
    // by a launch of their own
    const uintptr_t x0 = (uintptr_t)x, x1 = (uintptr_t)(x + (batch - 1) * ldx + n->n_in);
    const uintptr_t y0 = (uintptr_t)y, y1 = (uintptr_t)(y + (batch - 1) * ldy + n->n_out);
    const bool overlap = y0 < x1 && x0 < y1;
    if (!rows || overlap) {
        const long cnt = (long)R * fp;
        hipLaunchKernelGGL(normalise_kernel, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, s, x, ldx, batch,
                           n->n_in, n->mu_in, n->s_in, a.xh, R, fp);
        MLP_HIP(hipGetLastError());
    }
    if (rows) {
        RowArgs r = row_args(n, x, ldx, batch);
        r.xh = overlap ? a.xh : nullptr;
        r.y = y;
        r.ldy = ldy;
        MLP_HIP(predict_rows(r, s));
        return KAMX_OK;
    }
    auto layers = [&](auto blocked) {
        constexpr bool kBlocked = decltype(blocked)::value;
        EpiArgs e{};
        e.bias = n->w + L.ob1;
        e.f32 = a.z1;
        e.b16 = a.h1;
        e.ld = H;
        MLP_HIP((gemm<kEpiHidden, kBlocked>(Operand{a.xh, fp, 1}, Operand{n->wb + L.bW1, fp, 1}, R, H, fp, e, s)));
        e.bias = n->w + L.ob2;
        e.f32 = a.z2;
        e.b16 = a.h2;
        MLP_HIP((gemm<kEpiHidden, kBlocked>(Operand{a.h1, H, 1}, Operand{n->wb + L.bW2, H, 1}, R, H, H, e, s)));
        EpiArgs o{};
        o.bias = n->w + L.ob3;
        o.f32 = a.yn;
        o.ld = op;
        o.y = y;
        o.ldy = ldy;
        o.batch = batch;
        o.n_out = n->n_out;
        o.mu = n->mu_out;
        o.sigma = n->sd_out;
        MLP_HIP((gemm<kEpiOut, kBlocked>(Operand{a.h2, H, 1}, Operand{n->wb + L.bW3, H, 1}, R, op, H, o, s)));
        return KAMX_OK;
    };
    return n->fused ? layers(std::true_type()) : layers(std::false_type());
}

static Acts own_acts(kamx_mlp n, bool keep) {
    Acts a{n->xh, n->h1, n->h2, nullptr, nullptr, nullptr};
    if (keep) {
        a.z1 = n->z1;
        a.z2 = n->z2;
        a.yn = n->yn;
    }
    return a;
}

namespace kamx {
// used by the model's learned warm start
kamx_status mlp_forward_internal(kamx_mlp n, const float *x, int batch, float *y, hipStream_t s) {
    if (batch > n->cap) return mlp_fail(KAMX_EINVAL, "batch %d above the network's capacity %d", batch, n->cap);
    return mlp_forward_rows(n, own_acts(n, false), x, n->n_in, batch, y, n->n_out, s);
}
int mlp_n_in(kamx_mlp n) { return n->n_in; }
MlpView mlp_view(kamx_mlp n) {
    MlpView v;
    v.w1 = n->wb + n->L.bW1;
    v.w2 = n->wb + n->L.bW2;
    v.w3 = n->wb + n->L.bW3;
    v.b1 = n->w + n->L.ob1;
    v.b2 = n->w + n->L.ob2;
    v.b3 = n->w + n->L.ob3;
    v.mu_in = n->mu_in;
    v.s_in = n->s_in;
    v.mu_out = n->mu_out;
    v.sd_out = n->sd_out;
    v.n_in = n->n_in;
    v.fp = n->fp;
    v.H = n->H;
    v.n_out = n->n_out;
    v.op = n->op;
    v.blocked = n->fused;
    return v;
}
int mlp_n_out(kamx_mlp n) { return n->n_out; }
int mlp_capacity(kamx_mlp n) { return n->cap; }
}  // namespace kamx

extern "C" kamx_status kamx_mlp_forward(kamx_mlp n, const float *x, int32_t batch, float *y, kamx_stream stream) {
    if (!n || !x || !y) return mlp_fail(KAMX_EINVAL, "NULL argument");
    if (batch < 1 || batch > n->cap) return mlp_fail(KAMX_EINVAL, "batch must be in [1, %d]", n->cap);
    return mlp_forward_rows(n, own_acts(n, false), x, n->n_in, batch, y, n->n_out,
                            reinterpret_cast<hipStream_t>(stream));
}

// ---- forward pass without allocation -------------------------------------
// The activations of kamx_mlp_forward_noalloc live in this fixed array: each
// GPU the library runs on holds its own copy until the process ends.  Host
// code never passes the array's name to a kernel (on the host it is only a
// stand-in for the symbol); it uses the device address that
// hipGetSymbolAddress returns for the current device.
constexpr size_t kNoallocScratchBytes = size_t(16) << 20;
static __device__ __align__(256) unsigned char scratch[kNoallocScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

// device address of this GPU's scratch array (looked up once per device)
kamx_status scratch_address(void **out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return mlp_fail(KAMX_EDEVICE, "hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return mlp_fail(KAMX_EUNSUPPORTED, "device %d beyond %d", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr)
            return mlp_fail(KAMX_EDEVICE, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return KAMX_OK;
}
}  // namespace

extern "C" kamx_status kamx_mlp_forward_noalloc(kamx_mlp n, const float *x, int32_t batch, float *y,
                                                kamx_stream stream) {
    if (!n || !x || !y) return mlp_fail(KAMX_EINVAL, "NULL argument");
    if (batch < 1 || batch > (1 << 24)) return mlp_fail(KAMX_EINVAL, "batch must be in [1, 2^24]");
    const size_t per_row = sizeof(__bf16) * ((size_t)n->fp + 2 * (size_t)n->H);
    const size_t rows_max = (kNoallocScratchBytes / per_row) / 64 * 64;
    if ((size_t)pad64(batch) > rows_max)
        return mlp_fail(KAMX_EINVAL, "batch %d above the %zu rows the fixed %zu-byte workspace holds for this network",
                        batch, rows_max, kNoallocScratchBytes);
    void *base = nullptr;
    kamx_status st = scratch_address(&base);
    if (st != KAMX_OK) return st;
    // every activation is written before it is read (padded rows included),
    // so nothing in the array has to start at zero
    const long R = pad64(batch);
    Acts a{};
    a.xh = reinterpret_cast<__bf16 *>(base);
    a.h1 = a.xh + R * n->fp;
    a.h2 = a.h1 + R * n->H;
    return mlp_forward_rows(n, a, x, n->n_in, batch, y, n->n_out, reinterpret_cast<hipStream_t>(stream));
}

extern "C" kamx_status kamx_mlp_train_step(kamx_mlp n, const float *x, const float *y_target, int32_t batch, float lr,
                                           float *loss_dev, kamx_stream stream) {
    if (!n || !x || !y_target) return mlp_fail(KAMX_EINVAL, "NULL argument");
    if (batch < 1 || batch > n->cap) return mlp_fail(KAMX_EINVAL, "batch must be in [1, %d]", n->cap);
    if (!(lr >= 0.f)) return mlp_fail(KAMX_EINVAL, "lr must be >= 0");
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const int R = pad64(batch), H = n->H, fp = n->fp, op = n->op;
    const Layout &L = n->L;
    if (n->fused) {
        MLP_HIP(train_fused(n, x, y_target, batch, lr, loss_dev, s));
        n->t += 1;
        return KAMX_OK;
    }
    kamx_status st = mlp_forward_rows(n, own_acts(n, true), x, n->n_in, batch, nullptr, 0, s);
    if (st != KAMX_OK) return st;
    const long cnt = (long)R * op;
    const int blocks = (int)((cnt + 255) / 256);
    hipLaunchKernelGGL(loss_grad_kernel, dim3(blocks), dim3(256), 0, s, n->yn, y_target, batch, n->n_out, op,
                       n->mu_out, n->sd_out, n->dy, n->dyb, R, n->partial);
    MLP_HIP(hipGetLastError());
    if (loss_dev) {
        hipLaunchKernelGGL(loss_final_kernel, dim3(1), dim3(256), 0, s, n->partial, blocks,
                           1.f / ((float)batch * (float)n->n_out), loss_dev);
        MLP_HIP(hipGetLastError());
    }
    EpiArgs e{};
    // layer 3: dW3 = dy^T h2, db3 = sum dy, dz2 = (dy W3) gelu'(z2)
    MLP_HIP(gemm_store(n, Operand{n->dyb, 1, op}, Operand{n->h2, 1, H}, op, H, R, n->g + L.oW3, s));
    MLP_HIP(colsum(n, n->dy, R, op, n->g + L.ob3, s));
    e = EpiArgs{};
    e.z = n->z2;
    e.f32 = n->dz2;
    e.b16 = n->dz2b;
    e.ld = H;
    MLP_HIP((gemm<kEpiBackward>(Operand{n->dyb, op, 1}, Operand{n->wb + L.bW3, 1, H}, R, H, op, e, s)));
    // layer 2
    MLP_HIP(gemm_store(n, Operand{n->dz2b, 1, H}, Operand{n->h1, 1, H}, H, H, R, n->g + L.oW2, s));
    MLP_HIP(colsum(n, n->dz2, R, H, n->g + L.ob2, s));
    e = EpiArgs{};
    e.z = n->z1;
    e.f32 = n->dz1;
    e.b16 = n->dz1b;
    e.ld = H;
    MLP_HIP((gemm<kEpiBackward>(Operand{n->dz2b, H, 1}, Operand{n->wb + L.bW2, 1, H}, R, H, H, e, s)));
    // layer 1
    MLP_HIP(gemm_store(n, Operand{n->dz1b, 1, H}, Operand{n->xh, 1, fp}, H, fp, R, n->g + L.oW1, s));
    MLP_HIP(colsum(n, n->dz1, R, H, n->g + L.ob1, s));
    // Adam
    const float c1 = (float)(1.0 - pow(0.9, n->t + 1)), c2 = (float)(1.0 - pow(0.999, n->t + 1));
    hipLaunchKernelGGL(adam_kernel, dim3((unsigned)((L.total + 255) / 256)), dim3(256), 0, s, n->w, n->g, n->am,
                       n->av, L.total, lr, c1, c2, L, n->wb);
    MLP_HIP(hipGetLastError());
    n->t += 1;
    return KAMX_OK;
}

extern "C" kamx_status kamx_mlp_weights(kamx_mlp n, float *buf, int32_t set, kamx_stream stream) {
    if (!n || !buf) return mlp_fail(KAMX_EINVAL, "NULL argument");
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const Layout &L = n->L;
    if (set) {
        MLP_HIP(hipMemcpyAsync(n->w, buf, sizeof(float) * L.total, hipMemcpyDeviceToDevice, s));
        hipLaunchKernelGGL(refresh_bf16_kernel, dim3((unsigned)((L.total + 255) / 256)), dim3(256), 0, s, n->w, L,
                           n->wb);
        MLP_HIP(hipGetLastError());
        MLP_HIP(hipMemsetAsync(n->am, 0, sizeof(float) * L.total, s));
        MLP_HIP(hipMemsetAsync(n->av, 0, sizeof(float) * L.total, s));
        n->t = 0;
    } else {
        MLP_HIP(hipMemcpyAsync(buf, n->w, sizeof(float) * L.total, hipMemcpyDeviceToDevice, s));
    }
    return KAMX_OK;
}

extern "C" kamx_status kamx_mlp_gradients(kamx_mlp n, float *buf, kamx_stream stream) {
    if (!n || !buf) return mlp_fail(KAMX_EINVAL, "NULL argument");
    MLP_HIP(hipMemcpyAsync(buf, n->g, sizeof(float) * n->L.total, hipMemcpyDeviceToDevice,
                           reinterpret_cast<hipStream_t>(stream)));
    return KAMX_OK;
}
