// Blocked Cholesky factorization and factor inverse of a packed lower triangle in
// LDS on the matrix cores, shared by the step kernel and forward kinematics.
#pragma once

#include "kamx_device.h"
#include "kamx_internal.h"

namespace kamx {

// ---- 16x16 tiles of the packed lower triangle on the matrix cores
// v_mfma_f32_16x16x4f32: lane l supplies A[l % 16][l / 16] and
// B[l / 16][l % 16] of a 16x4 by 4x16 product and holds rows
// 4 (l / 16) + c, column l % 16 of the 16x16 accumulator.
typedef float mfx4 __attribute__((ext_vector_type(4)));

__device__ inline mfx4 mfma4(float a, float b, mfx4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// element (r, c) of the packed lower triangle; 0 above the diagonal
__device__ inline float tri_at(const float *A, int r, int c) { return c <= r ? A[tri_row_offset(r) + c] : 0.f; }

// Orders a wave's own LDS writes before its later LDS reads (the hardware keeps
// them in order; this keeps the compiler from moving them).
__device__ inline void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Rank-one updates of a 16x16 tile held one row (a[0..15]) and one column of its
// inverse (x[0..15]) to a lane: for j > k, with l_jk = a[k] of lane j,
//   KAMX_UPDATE_AX   a_j -= l_jk a_k, x_j -= l_jk x_k
//   KAMX_UPDATE_X    x_j -= l_jk x_k
// The lane broadcast is an operand of the fused multiply-add (which the compiler
// does not form by itself), so an update is one instruction.  The s_nops are the
// two wait states between a vector write and a lane read of it: a_k before the
// block, and behind it what the block wrote.
#define KAMX_FMAC(d, j, k, m) \
    "v_fmac_f32_dpp %[" #d #j "], %[a" #k "], -%[" #m #k "] row_newbcast:" #j " row_mask:0xf bank_mask:0xf\n\t"
#define KAMX_UPDATE_AX(k, j) KAMX_FMAC(a, j, k, a) KAMX_FMAC(x, j, k, x)
#define KAMX_UPDATE_X(k, j) KAMX_FMAC(x, j, k, x)
#define KAMX_FROM2(M, k) M(k, 2) KAMX_FROM3(M, k)
#define KAMX_FROM3(M, k) M(k, 3) KAMX_FROM4(M, k)
#define KAMX_FROM4(M, k) M(k, 4) KAMX_FROM5(M, k)
#define KAMX_FROM5(M, k) M(k, 5) KAMX_FROM6(M, k)
#define KAMX_FROM6(M, k) M(k, 6) KAMX_FROM7(M, k)
#define KAMX_FROM7(M, k) M(k, 7) KAMX_FROM8(M, k)
#define KAMX_FROM8(M, k) M(k, 8) KAMX_FROM9(M, k)
#define KAMX_FROM9(M, k) M(k, 9) KAMX_FROM10(M, k)
#define KAMX_FROM10(M, k) M(k, 10) KAMX_FROM11(M, k)
#define KAMX_FROM11(M, k) M(k, 11) KAMX_FROM12(M, k)
#define KAMX_FROM12(M, k) M(k, 12) KAMX_FROM13(M, k)
#define KAMX_FROM13(M, k) M(k, 13) KAMX_FROM14(M, k)
#define KAMX_FROM14(M, k) M(k, 14) KAMX_FROM15(M, k)
#define KAMX_FROM15(M, k) M(k, 15)
#define KAMX_FROM16(M, k)
#define KAMX_TILE_STEPS(S)                                                                                            \
    S(0, 1, KAMX_FROM2) S(1, 2, KAMX_FROM3) S(2, 3, KAMX_FROM4) S(3, 4, KAMX_FROM5) S(4, 5, KAMX_FROM6)               \
    S(5, 6, KAMX_FROM7) S(6, 7, KAMX_FROM8) S(7, 8, KAMX_FROM9) S(8, 9, KAMX_FROM10) S(9, 10, KAMX_FROM11)            \
    S(10, 11, KAMX_FROM12) S(11, 12, KAMX_FROM13) S(12, 13, KAMX_FROM14) S(13, 14, KAMX_FROM15) S(14, 15, KAMX_FROM16)
#define KAMX_TILE_ASM(UPDATES)                                                                                      \
    asm("s_nop 1\n\t" UPDATES "s_nop 1"                                                                             \
        : [a0] "+v"(a[0]), [a1] "+v"(a[1]), [a2] "+v"(a[2]), [a3] "+v"(a[3]), [a4] "+v"(a[4]), [a5] "+v"(a[5]),     \
          [a6] "+v"(a[6]), [a7] "+v"(a[7]), [a8] "+v"(a[8]), [a9] "+v"(a[9]), [a10] "+v"(a[10]), [a11] "+v"(a[11]), \
          [a12] "+v"(a[12]), [a13] "+v"(a[13]), [a14] "+v"(a[14]), [a15] "+v"(a[15]), [x0] "+v"(x[0]),              \
          [x1] "+v"(x[1]), [x2] "+v"(x[2]), [x3] "+v"(x[3]), [x4] "+v"(x[4]), [x5] "+v"(x[5]), [x6] "+v"(x[6]),     \
          [x7] "+v"(x[7]), [x8] "+v"(x[8]), [x9] "+v"(x[9]), [x10] "+v"(x[10]), [x11] "+v"(x[11]),                  \
          [x12] "+v"(x[12]), [x13] "+v"(x[13]), [x14] "+v"(x[14]), [x15] "+v"(x[15]))

// Cholesky of a packed triangle, then the explicit inverse X of the factor in its
// place (Alg. 1 step 1), over 16x16 tiles.  Returns nonzero when a pivot is not
// positive.
//
// Right-looking: step K multiplies the panel below diagonal tile K by the tile's
// inverse (P phase) and gives the trailing tiles their rank-16 update (T phase),
// in which wave 0 updates and factors the next diagonal tile while the other
// waves take the rest.  The inverse follows one row behind in the same phases:
// row K of L is complete once its diagonal tile is, so P(K) inverts that tile
// (X_KK), T(K) forms M_Kk = X_KK L_Kk, P(K + 1) forms
// X_Kj = -sum_{k=j}^{K-1} M_Kk X_kj in registers and T(K + 1) writes it.  The
// trailing update shrinks with K as the inverse row grows, so the waves stay
// evenly loaded, and both together pass 2 (T + 2) barriers (4 where T is 1).  Wave 0's serial
// diagonal tile bounds a step: its broadcasts are operands of the fused
// multiply-adds (DPP), one instruction per entry and column.
// At 224 rows on eight waves: 65 us, against 106 us with the inverse after the
// factorization and the diagonal tile's broadcasts through scalar registers.
//
// A: the triangle in LDS, rows m .. the next multiple of 16 identity; Xs:
// kFactorScratch floats of LDS (the 16x16 inverse of the current diagonal factor
// tile, rows 17 apart for the LDS banks, and a spare place); flag: an int in LDS.
// 0 <= m <= MC rows, uniform; every thread of the workgroup calls.
constexpr int kFactorScratch = 288 + 64;

template <int MC, int NT>
__device__ __forceinline__ int factor_invert_tiles(float *A, float *Xs, int *flag, int m) {
    const int tid = threadIdx.x;
    const int T = (m + 15) >> 4;
    const int lane = tid & 63, wv = uniform(tid >> 6), fr = lane & 15, fk = lane >> 4;
    constexpr int NW = NT / 64;
    constexpr int NWP = NW > 1 ? NW - 1 : 1;  // waves of the P phase's tiles (the last inverts the diagonal tile)
    constexpr int NX = (MC / 16 - 1 + NWP - 1) / NWP;  // tiles of an inverse row per wave
    // one wave alone: at most two tile rows, so every trailing update is the
    // next diagonal tile
    static_assert(NW > 1 || MC <= 32, "a single-wave factorization covers two tile rows");
    // row fr of the diagonal tile at k0 (every row of 16 lanes holds the tile);
    // entries right of the diagonal are not used
    auto load_diag = [&](int k0, float (&a)[16]) {
        const float *R = A + tri_row_offset(k0 + fr) + k0;
#pragma unroll
        for (int c = 0; c < 16; c += 4) {
            const mfx4 v = *reinterpret_cast<const mfx4 *>(R + c);
#pragma unroll
            for (int e = 0; e < 4; ++e) a[c + e] = v[e];
        }
    };
    // factor diagonal tile K (wave 0 only) and write its inverse to Xs: column
    // k of the factor and row k of the inverse, then the rank-one updates of what
    // lies behind them
    auto factor_diag = [&](int K) {
        const int k0 = 16 * K;
        float a[16], x[16];  // row fr of the tile, column fr of the inverse
        load_diag(k0, a);
#pragma unroll
        for (int r = 0; r < 16; ++r) x[r] = fr == r ? 1.f : 0.f;
        float d = row_bcast<0>(a[0]);
        bool ok = __builtin_amdgcn_classf(d, 0x180);  // positive and finite
        float il = __builtin_amdgcn_rsqf(d);          // 1 / l_kk by the hardware (1 ulp); l_kk = d / sqrt(d)
        // the next pivot is ready after the first update: its root runs under the rest
#define KAMX_STEP(k, n, REST)                                \
    a[k] *= il;                                              \
    x[k] *= il;                                              \
    KAMX_TILE_ASM(KAMX_UPDATE_AX(k, n));                     \
    d = row_bcast<n>(a[n]);                                  \
    ok = ok && __builtin_amdgcn_classf(d, 0x180);            \
    il = __builtin_amdgcn_rsqf(d);                           \
    KAMX_TILE_ASM(REST(KAMX_UPDATE_AX, k));
        KAMX_TILE_STEPS(KAMX_STEP)
        a[15] *= il;
        x[15] *= il;
#undef KAMX_STEP
        // every row of 16 lanes holds the tile: row fk writes its quad of L (the
        // quad of the diagonal ends in the row's zero pads) and of X
        mfx4 lq, xq;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float l01 = fk & 1 ? a[4 + e] : a[e], l23 = fk & 1 ? a[12 + e] : a[8 + e];
            const float x01 = fk & 1 ? x[4 + e] : x[e], x23 = fk & 1 ? x[12 + e] : x[8 + e];
            lq[e] = 4 * fk + e <= fr ? (fk & 2 ? l23 : l01) : 0.f;
            xq[e] = fk & 2 ? x23 : x01;
        }
        if (4 * fk <= fr) *reinterpret_cast<mfx4 *>(A + tri_row_offset(k0 + fr) + k0 + 4 * fk) = lq;
#pragma unroll
        for (int e = 0; e < 4; ++e) Xs[17 * (4 * fk + e) + fr] = xq[e];  // zero above the diagonal
        if (!ok && lane == 0) *flag = 1;
    };
    // X_KK, the inverse of factor tile K, over it
    auto invert_diag = [&](int K) {
        const int k0 = 16 * K;
        float a[16], x[16];
        load_diag(k0, a);
#pragma unroll
        for (int r = 0; r < 16; ++r) x[r] = fr == r ? 1.f : 0.f;
        float il = __builtin_amdgcn_rcpf(row_bcast<0>(a[0]));  // hardware reciprocal (1 ulp)
#define KAMX_STEP(k, n, REST)                                     \
    x[k] *= il;                                                   \
    il = __builtin_amdgcn_rcpf(row_bcast<n>(a[n]));               \
    KAMX_TILE_ASM(KAMX_UPDATE_X(k, n) REST(KAMX_UPDATE_X, k));
        KAMX_TILE_STEPS(KAMX_STEP)
        x[15] *= il;
#undef KAMX_STEP
        // row fk of 16 lanes writes rows 4 fk .. 4 fk + 3; entries above the
        // diagonal go to a spare place behind Xs
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float x01 = fk & 1 ? x[4 + e] : x[e], x23 = fk & 1 ? x[12 + e] : x[8 + e];
            const int r = 4 * fk + e;
            *(r >= fr ? A + tri_row_offset(k0 + r) + k0 + fr : Xs + 288 + lane) = fk & 2 ? x23 : x01;
        }
    };
    // L and M tiles lie transposed in their places: an operand's lanes (row fr,
    // columns 4 ch + fk) then read runs of 16 floats instead of 16 rows that share
    // few LDS banks, and a result's four rows are one 16-byte write
    auto load_tile_t = [&](int row0, int col0, float (&v)[4]) {
#pragma unroll
        for (int ch = 0; ch < 4; ++ch) v[ch] = A[tri_row_offset(row0 + 4 * ch + fk) + col0 + fr];
    };
    auto store_tile_t = [&](int row0, int col0, const mfx4 &acc) {
        *reinterpret_cast<mfx4 *>(A + tri_row_offset(row0 + fr) + col0 + 4 * fk) = acc;
    };
    // A_IJ -= L_IK L_JK^T for N tiles of one tile column (matrix cores), their reads
    // and products in flight together.  D: the tiles' row 4 fk, column fr; their
    // rows are step floats apart.  DIAG: the first tile lies on the diagonal.
    auto update_tiles = [&](auto nc, auto diag, float *const *D, const int *step, const float (*li)[4],
                            const float (&lj)[4]) {
        constexpr int N = nc.value;
        float d[N][4];
        mfx4 acc[N];
#pragma unroll
        for (int n = 0; n < N; ++n) {
            acc[n] = mfx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < 4; ++c) d[n][c] = D[n][c * step[n]];
        }
#pragma unroll
        for (int ch = 0; ch < 4; ++ch)
#pragma unroll
            for (int n = 0; n < N; ++n) acc[n] = mfma4(li[n][ch], lj[ch], acc[n]);
#pragma unroll
        for (int n = 0; n < N; ++n)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                float *p = D[n] + c * step[n];
                if (diag.value && n == 0 && fr > 4 * fk + c) p = Xs + 288 + lane;  // above the diagonal: a spare place
                *p = d[n][c] - acc[n][c];
            }
    };
    if (tid == 0) *flag = 0;
    __syncthreads();
    if (T == 0) return 0;  // no rows: nothing has written the triangle
    if (wv == 0) factor_diag(0);
    __syncthreads();
    const int last = T > 1 ? T : 0;  // (one tile: P(0) puts its inverse in place)
    for (int K = 0; K <= last; ++K) {
        if (uniform(*flag)) return 1;
        const int k0 = 16 * K, nI = T - K - 1;
        // ---- P(K)
        if (K < T && wv == NW - 1) invert_diag(K);
        mfx4 xrow[NX];  // this wave's tiles of inverse row K - 1
        if (wv < NWP) {
            // panel: L_IK = A_IK Xkk^T for the tiles I below the diagonal, one
            // wave per tile (each wave reads its tile before overwriting it);
            // dealt from the last wave, the inverse row's longest sums being the
            // first waves'
            if (nI > 0) {
                float xk[4];
#pragma unroll
                for (int ch = 0; ch < 4; ++ch) xk[ch] = Xs[17 * fr + 4 * ch + fk];
                for (int Ii = NWP - 1 - wv; Ii < nI; Ii += NWP) {
                    const int I = K + 1 + Ii;
                    const float *R = A + tri_row_offset(16 * I + fr) + k0 + fk;
                    float av[4];
#pragma unroll
                    for (int ch = 0; ch < 4; ++ch) av[ch] = R[4 * ch];
                    mfx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ch = 0; ch < 4; ++ch) acc = mfma4(av[ch], xk[ch], acc);
                    store_tile_t(16 * I, k0, acc);
                }
            }
            // X_ij = -sum_k M_ik X_kj of row i = K - 1: the diagonal tile X_jj
            // (lower triangular) first, then the full tiles below it, alternating
            // between two accumulators so consecutive products do not wait on
            // each other; two tiles at a time, whose operands fit the registers (192
            // rows on six waves have three, and all at once spilled 12 us' worth)
            auto inverse_row = [&](auto first, auto count) {
                constexpr int Q0 = first.value, NQ = count.value;
                mfx4 xb[NQ];
#pragma unroll
                for (int q = 0; q < NQ; ++q) xrow[Q0 + q] = xb[q] = mfx4{0.f, 0.f, 0.f, 0.f};
                struct Terms {
                    float m[4], x[NQ][4];
                };
                const int T0 = wv + Q0 * NWP;  // the first of this wave's tiles
                auto read = [&](int Tk, Terms &h) {
                    load_tile_t(k0 - 16, 16 * Tk, h.m);
#pragma unroll
                    for (int ch = 0; ch < 4; ++ch) {
                        const float *R = A + tri_row_offset(16 * Tk + 4 * ch + fk) + fr;
#pragma unroll
                        for (int q = 0; q < NQ; ++q) h.x[q][ch] = R[16 * min(T0 + q * NWP, Tk)];
                    }
                };
                auto multiply = [&](int Tk, Terms &h) {
#pragma unroll
                    for (int q = 0; q < NQ; ++q) {
                        const int Tj = T0 + q * NWP;
                        mfx4 &x = xrow[Q0 + q];
                        if (Tj < Tk) {
#pragma unroll
                            for (int ch = 0; ch < 4; ch += 2) {
                                x = mfma4(h.m[ch], h.x[q][ch], x);
                                xb[q] = mfma4(h.m[ch + 1], h.x[q][ch + 1], xb[q]);
                            }
                        } else if (Tj == Tk) {
#pragma unroll
                            for (int ch = 0; ch < 4; ++ch)
                                x = mfma4(h.m[ch], fr <= 4 * ch + fk ? h.x[q][ch] : 0.f, x);
                        }
                    }
                };
                Terms ha, hb;
                int Tk = T0;
                if (Tk < K - 1) read(Tk, ha);
                for (; Tk + 1 < K - 1; Tk += 2) {
                    read(Tk + 1, hb);
                    multiply(Tk, ha);
                    if (Tk + 2 < K - 1) read(Tk + 2, ha);
                    multiply(Tk + 1, hb);
                }
                if (Tk < K - 1) multiply(Tk, ha);
#pragma unroll
                for (int q = 0; q < NQ; ++q) xrow[Q0 + q] += xb[q];
            };
            static_assert(NX <= 4, "tiles of an inverse row per wave");
            inverse_row(Const<0>{}, Const<(NX < 2 ? NX : 2)>{});
            if constexpr (NX > 2) inverse_row(Const<2>{}, Const<NX - 2>{});
        }
        __syncthreads();
        // ---- T(K)
        if (nI > 0 && wv == 0) {
            float lk[1][4];
            const int r4 = 4 * (K + 1) + fk, step = 4 * (r4 + 1);
            float *D = A + tri_row_offset(4 * r4) + k0 + 16 + fr;
            load_tile_t(k0 + 16, k0, lk[0]);
            update_tiles(Const<1>{}, Const<1>{}, &D, &step, lk, lk[0]);
            wave_lds_fence();
            factor_diag(K + 1);
        }
        if (wv > 0 || NW == 1) {
            // M_Kk = X_KK L_Kk in place
            if (K < T) {
                constexpr int W1 = NW > 1 ? 1 : 0;
                for (int Tk = NWP - 1 - (wv - W1); Tk < K; Tk += NWP) {
                    const float *R = A + tri_row_offset(k0 + fr) + 16 * Tk + fk;
                    float lv[4];
#pragma unroll
                    for (int ch = 0; ch < 4; ++ch) lv[ch] = R[4 * ch];
                    mfx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ch = 0; ch < 4; ++ch)
                        acc = mfma4(tri_at(A, k0 + fr, k0 + 4 * ch + fk), lv[ch], acc);
                    store_tile_t(k0, 16 * Tk, acc);
                }
            }
            // trailing update A_IJ -= L_IK L_JK^T, K < J <= I, without the next
            // diagonal tile: strips of two tile rows (2 S, 2 S + 1), a strip's 2 S + 2
            // columns a task each, and each wave a run of consecutive tasks, whose
            // strips' row operands stay in registers
            if (NW > 1 && nI > 1) {
                const int nstrip = (nI + 1) >> 1, ntask = nstrip * (nstrip + 1);
                const int per = (ntask + NWP - 1) / NWP;
                int p = (wv - 1) * per;
                const int pe = min(p + per, ntask);
                int S = (int)((sqrtf(4.f * (float)p + 1.f) - 1.f) * 0.5f);
                while ((S + 1) * (S + 2) <= p) ++S;
                while (S * (S + 1) > p) --S;
                S = uniform(S);
                int Jj = p - S * (S + 1);
                float li[2][4];
                float *row[2];  // the strip's rows of A
                int step[2];
                for (int have = -1; p < pe; ++p) {
                    const bool second = 2 * S + 1 < nI;  // the strip has its second row
                    float lj[4];
                    load_tile_t(16 * min(K + 1 + Jj, T - 1), k0, lj);  // (a strip without its second row: unused)
                    if (have != S) {
#pragma unroll
                        for (int n = 0; n < 2; ++n) {
                            const int I = min(K + 1 + 2 * S + n, T - 1), r4 = 4 * I + fk;
                            load_tile_t(16 * I, k0, li[n]);
                            row[n] = A + tri_row_offset(4 * r4) + fr;
                            step[n] = 4 * (r4 + 1);
                        }
                        have = S;
                    }
                    float *D[2] = {row[0] + 16 * (K + 1 + Jj), row[1] + 16 * (K + 1 + Jj)};
                    if (Jj < 2 * S) {
                        if (second) update_tiles(Const<2>{}, Const<0>{}, D, step, li, lj);
                        else update_tiles(Const<1>{}, Const<0>{}, D, step, li, lj);
                    } else if (Jj == 2 * S) {
                        if (p > 0) update_tiles(Const<1>{}, Const<1>{}, D, step, li, lj);
                        if (second) update_tiles(Const<1>{}, Const<0>{}, D + 1, step + 1, li + 1, lj);
                    } else if (second) {
                        update_tiles(Const<1>{}, Const<1>{}, D + 1, step + 1, li + 1, lj);
                    }
                    if (++Jj > 2 * S + 1) {
                        ++S;
                        Jj = 0;
                    }
                }
            }
        }
        if (wv < NWP) {
#pragma unroll
            for (int q = 0; q < NX; ++q) {
                const int Tj = wv + q * NWP;
                if (Tj >= K - 1) continue;
#pragma unroll
                for (int c = 0; c < 4; ++c) A[tri_row_offset(k0 - 16 + 4 * fk + c) + 16 * Tj + fr] = -xrow[q][c];
            }
        }
        __syncthreads();
    }
    return 0;
}

}  // namespace kamx
