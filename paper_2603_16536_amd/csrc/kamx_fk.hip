// Forward kinematics for resets (Sec. 6.3): the poses of every body of a
// world that satisfy all joint constraints -- the passive joints of
// kinematic loops included -- and put the targeted joints at given
// coordinates, found by Gauss-Newton.  One workgroup per world.
//
// Each iteration evaluates, in FP64, F = (the five constraint functions of
// every joint, c_j - target_j for every targeted joint) and its Jacobian J
// over the body twists, and takes the least-change step
//     Delta = -W J^T (J W J^T + mu)^-1 F,   W = M^-1 (the reset body's
//     block zero: it stays where it is),
// moving every body by the exponential map.  The normal matrix is scaled by
// its Jacobi diagonal, regularised by mu = 1e-5 on that unit diagonal (the
// redundant rows of planar loops make J W J^T singular), stored packed in
// LDS in FP32 and factored and inverted on the matrix cores by the step kernel's
// tile factorization, so that the solve is two triangular products; F and the
// poses stay FP64, so the iteration converges to FP64-level constraint residuals
// with FP32 linear solves.  Pivots are the hardware's reciprocals and reciprocal square
// roots (1 ulp), and a product with the explicit inverse rounds otherwise than a
// substitution: a step differs from one with exact pivots in its last bits, the
// poses it converges to by less than 3e-8.  A pivot that is not positive and finite
// fails the world.  Runs once per reset, not per step.
//
// An iteration is bound by the factorization's serial diagonal tiles and, like the
// step, by one world per compute unit (the triangle fills its LDS).  1024 bipeds
// with ten targets: 2.9 ms, against 34.9 ms with a column-by-column Cholesky and
// substitution, three barriers and a search for the entry's row to a column.
#include <math.h>

#include "kamx_factor.h"
#include "kamx_geom.h"
#include "kamx_internal.h"

namespace kamx {

namespace {

constexpr int kFkThreads = 512;
constexpr int kFkRows = kMaxRows;
constexpr float kFkMu = 1e-5f;

struct FkLds {
    double q[kMaxBodies][7];     // poses
    double F[kFkRows];           // residuals
    double dl[kMaxBodies][6];    // step per body
    float J[kFkRows][12];        // rows: side a, side b
    float W[kFkRows][12];        // M^-1 J^T of both sides
    float p[kFkRows];            // Jacobi scales
    alignas(16) float y[kFkRows];  // right-hand side, then the solution
    float t[2][kFkRows];         // X y, then the halves of X^T (X y)
    float Rm[kMaxBodies][9];     // body rotations
    float red[kFkThreads / 64];
    int ab[kFkRows];             // (a + 1) | (b + 1) << 16
    int trow[kMaxJoints];        // row of a targeted joint, -1
    int flag;
    float Xs[kFactorScratch];
};

// the triangle (tri_row_offset(kFkRows) floats) lies behind FkLds
constexpr size_t fk_lds_bytes() { return (sizeof(FkLds) + 15) & ~size_t(15); }

__device__ inline float block_max(float v, float *red) {
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    float r = red[0];
    for (int k = 1; k < kFkThreads / 64; ++k) r = fmaxf(r, red[k]);
    __syncthreads();
    return r;
}

__global__ __launch_bounds__(kFkThreads) void fk_kernel(const WorldInfo *worlds, const int32_t *jint, const float *jf,
                                                        const float *mass, const float *inertia, float *q, float *u,
                                                        const float *targets, int max_iters, float tol,
                                                        int32_t *iters_out, float *resid_out) {
    extern __shared__ float4 smem4[];
    FkLds &S = *reinterpret_cast<FkLds *>(smem4);
    float *A = reinterpret_cast<float *>(smem4 + fk_lds_bytes() / 16);
    const int tid = threadIdx.x;
    const int w = blockIdx.x;
    const WorldInfo Wd = worlds[w];
    const int nb = Wd.nb, nj = Wd.nj, base = Wd.reset_body;
    for (int t = tid; t < 7 * nb; t += kFkThreads) S.q[t / 7][t % 7] = q[7 * (long)Wd.b0 + t];
    if (tid == 0) {
        int r = 5 * nj;
        for (int j = 0; j < nj; ++j) {
            const float tj = targets[Wd.j0 + j];
            S.trow[j] = isnan(tj) ? -1 : r++;
        }
        S.flag = r;  // row count
    }
    __syncthreads();
    const int m = uniform(S.flag);
    if (m > kFkRows) {  // more targets than one world's rows: leave the world alone
        if (tid == 0) {
            if (iters_out) iters_out[w] = 0;
            if (resid_out) resid_out[w] = NAN;
        }
        return;
    }
    int it = 0;
    float fn = INFINITY;
    bool failed = false;
    for (;; ++it) {
        // ---- rows and residuals at the current poses (FP64 geometry)
        for (int j = tid; j < nj; j += kFkThreads) {
            const long gj = Wd.j0 + j;
            const int type = jint[4 * gj], la = jint[4 * gj + 1], lb = jint[4 * gj + 2];
            const float *f = jf + kJointFloats * gj;
            double qb[7];
            for (int k = 0; k < 7; ++k) qb[k] = lb >= 0 ? S.q[lb][k] : 0.0;
            JointGeo g;
            joint_geo_q(S.q[la], qb, lb >= 0, f, g);
            joint_constraints(type, g, [&](int e, const double Ja[6], const double Jb[6], double fv) {
                const int r = 5 * j + e;
                for (int k = 0; k < 6; ++k) {
                    S.J[r][k] = (float)Ja[k];
                    S.J[r][6 + k] = lb >= 0 ? (float)Jb[k] : 0.f;
                }
                S.F[r] = fv;
                S.ab[r] = (la + 1) | ((lb + 1) << 16);
            });
            const int rt = S.trow[j];
            if (rt >= 0) {
                float Ja[6], Jb[6];
                const double c = joint_coord(type, g, Ja, Jb);
                for (int k = 0; k < 6; ++k) {
                    S.J[rt][k] = Ja[k];
                    S.J[rt][6 + k] = lb >= 0 ? Jb[k] : 0.f;
                }
                S.F[rt] = c - (double)targets[gj];
                S.ab[rt] = (la + 1) | ((lb + 1) << 16);
            }
        }
        // body rotations for M^-1
        for (int b = tid; b < nb; b += kFkThreads) {
            double R[9], qq[4] = {S.q[b][3], S.q[b][4], S.q[b][5], S.q[b][6]};
            rot_of_quat(qq, R);
            for (int k = 0; k < 9; ++k) S.Rm[b][k] = (float)R[k];
        }
        __syncthreads();
        float lf = 0.f;
        for (int r = tid; r < m; r += kFkThreads) {
            const float a = (float)fabs(S.F[r]);
            lf = (a > lf || a != a) ? a : lf;
        }
        fn = block_max(lf, S.red);
        if (!(fn > tol) || it >= max_iters || failed) break;  // converged, budget spent, or non-finite
        // ---- W = M^-1 J^T per side (body frame: R diag(I^-1) R^T), reset body held
        for (int r = tid; r < m; r += kFkThreads) {
            float dsum = 0.f;
            for (int s = 0; s < 2; ++s) {
                const int b = (s ? S.ab[r] >> 16 : S.ab[r] & 0xffff) - 1;
                float out[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                if (b >= 0 && b != base) {
                    const long gb = Wd.b0 + b;
                    const float im = 1.f / mass[gb];
                    const float *in = S.J[r] + 6 * s;
                    const float *R = S.Rm[b];
                    float t[3], v[3];
                    mtv3(R, in + 3, t);
                    for (int k = 0; k < 3; ++k) t[k] /= inertia[3 * gb + k];
                    mv3(R, t, v);
                    for (int k = 0; k < 3; ++k) {
                        out[k] = in[k] * im;
                        out[3 + k] = v[k];
                    }
                }
                for (int k = 0; k < 6; ++k) {
                    S.W[r][6 * s + k] = out[k];
                    dsum += S.J[r][6 * s + k] * out[k];
                }
            }
            S.p[r] = dsum > 0.f ? 1.f / sqrtf(dsum) : 1.f;
        }
        __syncthreads();
        // ---- scaled normal matrix P J W J^T P + mu: a row to a wave, a column to
        //      a lane (rows sharing a body only; the rest, the pads and the rows up
        //      to a multiple of 16 zero, their diagonal one)
        const int wave = uniform(tid >> 6), lane = tid & 63;
        for (int i = wave; i < ((m + 15) & ~15); i += kFkThreads / 64) {
            float *R = A + tri_row_offset(i);
            const int abi = i < m ? S.ab[i] : 0;
            const int bi[2] = {(abi & 0xffff) - 1, (abi >> 16) - 1};
            for (int j = lane; j < ((i + 4) & ~3); j += 64) {
                float acc = 0.f;
                if (j <= i && i < m) {
                    const int abj = S.ab[j], bj[2] = {(abj & 0xffff) - 1, (abj >> 16) - 1};
                    for (int s = 0; s < 2; ++s)
                        for (int v = 0; v < 2; ++v)
                            if (bi[s] >= 0 && bi[s] == bj[v])
                                for (int k = 0; k < 6; ++k) acc += S.J[i][6 * s + k] * S.W[j][6 * v + k];
                    acc *= S.p[i] * S.p[j];
                    if (i == j) acc += kFkMu;
                } else if (j == i) {
                    acc = 1.f;
                }
                R[j] = acc;
            }
        }
        __syncthreads();
        if (factor_invert_tiles<kFkRows, kFkThreads>(A, S.Xs, &S.flag, m)) {
            failed = true;
            continue;  // reported as a non-finite residual below
        }
        // ---- solve (P A P) y~ = P F by y~ = X^T (X (P F)), then y = P y~
        for (int r = tid; r < kFkRows; r += kFkThreads) S.y[r] = r < m ? S.p[r] * (float)S.F[r] : 0.f;
        __syncthreads();
        // X: a row to 16 lanes
        for (int r = tid >> 4; r < m; r += kFkThreads / 16) {
            const float *R = A + tri_row_offset(r);
            float acc = 0.f;
            for (int c = 4 * (tid & 15); c <= r; c += 64) {
                const mfx4 x = *reinterpret_cast<const mfx4 *>(R + c), v = *reinterpret_cast<const mfx4 *>(S.y + c);
                for (int e = 0; e < 4; ++e) acc += x[e] * v[e];  // the pads hold 0
            }
            acc = lane_group_sum<16>(acc);
            if ((tid & 15) == 0) S.t[0][r] = acc;
        }
        __syncthreads();
        // X^T: a column to two threads, the even and the odd rows
        {
            const int c = tid >> 1, h = tid & 1;
            float acc = 0.f;
            if (c < m)
                for (int r = c + ((c ^ h) & 1); r < m; r += 2) acc += A[tri_row_offset(r) + c] * S.t[0][r];
            acc = lane_group_sum<2>(acc);
            if (c < m && h == 0) S.t[1][c] = acc;
        }
        __syncthreads();
        for (int r = tid; r < m; r += kFkThreads) S.y[r] = S.t[1][r] * S.p[r];
        __syncthreads();
        // ---- Delta = -W J^T y per body component (rows in order), FP64
        for (int t = tid; t < 6 * nb; t += kFkThreads) {
            const int b = t / 6, c = t - 6 * (t / 6);
            double acc = 0.0;
#pragma unroll 8
            for (int r = 0; r < m; ++r) {
                const int ab = S.ab[r];
                if ((ab & 0xffff) == b + 1) acc += (double)S.W[r][c] * (double)S.y[r];
                if (ab >> 16 == b + 1) acc += (double)S.W[r][6 + c] * (double)S.y[r];
            }
            S.dl[b][c] = -acc;
        }
        __syncthreads();
        // ---- move every body: r += Delta_v, R <- exp(Delta_w) R
        for (int b = tid; b < nb; b += kFkThreads) {
            const double *d = S.dl[b];
            for (int k = 0; k < 3; ++k) S.q[b][k] += d[k];
            const double wn = sqrt(d[3] * d[3] + d[4] * d[4] + d[5] * d[5]);
            if (wn > 0.0) {
                const double sh = sin(0.5 * wn) / wn;
                const double dq[4] = {d[3] * sh, d[4] * sh, d[5] * sh, cos(0.5 * wn)};
                double qo[4] = {S.q[b][3], S.q[b][4], S.q[b][5], S.q[b][6]}, qn[4];
                qprod(dq, qo, qn);
                const double nn = 1.0 / sqrt(qn[0] * qn[0] + qn[1] * qn[1] + qn[2] * qn[2] + qn[3] * qn[3]);
                for (int k = 0; k < 4; ++k) S.q[b][3 + k] = qn[k] * nn;
            }
        }
        __syncthreads();
    }
    // poses out (FP32), twists zero
    for (int t = tid; t < 7 * nb; t += kFkThreads) q[7 * (long)Wd.b0 + t] = (float)S.q[t / 7][t % 7];
    for (int t = tid; t < 6 * nb; t += kFkThreads) u[6 * (long)Wd.b0 + t] = 0.f;
    if (tid == 0) {
        if (iters_out) iters_out[w] = it;
        if (resid_out) resid_out[w] = failed ? NAN : fn;
    }
}

}  // namespace

size_t fk_smem_bytes() { return fk_lds_bytes() + sizeof(float) * (size_t)tri_row_offset(kFkRows); }

hipError_t launch_fk(const WorldInfo *worlds, int n_worlds, const int32_t *jint, const float *jf, const float *mass,
                     const float *inertia, float *q, float *u, const float *targets, int max_iters, float tol,
                     int32_t *iters, float *resid, hipStream_t stream) {
    if (n_worlds <= 0) return hipSuccess;
    const size_t bytes = fk_smem_bytes();
    hipError_t e = allow_lds((const void *)fk_kernel, bytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fk_kernel, dim3(n_worlds), dim3(kFkThreads), bytes, stream, worlds, jint, jf, mass, inertia, q,
                       u, targets, max_iters, tol, iters, resid);
    return hipGetLastError();
}

}  // namespace kamx
