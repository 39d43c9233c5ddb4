// Fused per-world time step on gfx950: one workgroup advances one world.
//
// Everything a world needs -- body state, joint frames, contact rows, the
// preconditioned Delassus matrix, its factor and the ADMM vectors -- lives in
// LDS for the whole step, so HBM sees only the per-world inputs and outputs.
// While the rows are built, thread i owns constraint row i (and the block that
// starts at row i: one row for joints and limits, three rows for a contact); the
// solve gives row i to the lane pair 2 i, 2 i + 1.
//
// Steps (Tsounis et al. 2026):
//   bodies: R(q), M^-1 applied in the body frame, Newton-Euler forces with
//           gyroscopic term and joint actuation (Sec. 3, Eq. 1);
//   rows:   joint / limit / contact Jacobians and Baumgarte bias (Sec. 3);
//   D~:     D = J M^-1 J^T (Eq. 4) scaled by the Jacobi preconditioner
//           (Sec. 4.1), shifted by eta + rho (Alg. 1 step 1);
//   factor: Cholesky once per step, then the explicit inverse of the factor,
//           so every iteration's solve is two parallel triangular mat-vecs
//           instead of two serial substitution sweeps;
//   PADMM:  Alg. 1 steps 4-10 with Nesterov restart (Sec. 4.1);
//   output: lambda = P y, u+ = u_f + M^-1 J^T lambda, SO(3) exponential map.
#include <math.h>

#include "kamx_boxbin.h"
#include "kamx_device.h"
#include "kamx_factor.h"
#include "kamx_geom.h"
#include "kamx_internal.h"

namespace kamx {

// ---------------------------------------------------------------------------
// LDS views
// ---------------------------------------------------------------------------

// body fields [field][kMaxBodies]
enum { BQ = 0, BU = 7, BUF = 13, BR = 19, BII = 28, BIM = 31 };
// joint fields [field][kMaxJoints]
enum { JTAU = 0, JC = 1, JA = 13, JB = 14, JTF = 15 };
// contact fields [field][kMaxContacts]
enum { CP = 0, CN = 3, CGAP = 6, CMU = 7, CA = 8, CB = 9, CKEY = 10 };
// row fields [field][MC]
enum { RJ = 0, RBIAS = 12, RMU = 13, RIA = 14, RIB = 15, RKIND = 16, RREG = 17 };
// vector fields [field][MC]
enum { VP = 0, VRHO, VVT, VX, VYH, VZH, VYP, VZP, VRHS, VXN, VWS, VAUX, VCOL, VDX };

struct Lds {
    float *b, *j, *c, *r, *v, *A, *red;
    double *wb;          // [6][kMaxBodies] FP64 body work vector
    double *qd;          // [7][kMaxBodies] FP64 poses the rows are built at
    int *inc_off;        // [kMaxBodies + 1] body -> row incidence offsets
    int *inc_list;       // [2 * MC] (row << 1) | side
    float *t;            // [t_floats(MC)] t = X r of the x update, 0 past the world's rows
    int *s_int;          // [12] values one thread hands to all
    int mc;
    __device__ float &bf(int f, int i) const { return b[f * kMaxBodies + i]; }
    __device__ float &jfld(int f, int i) const { return j[f * kMaxJoints + i]; }
    __device__ float &cf(int f, int i) const { return c[f * kMaxContacts + i]; }
    __device__ float &rf(int f, int i) const { return r[f * mc + i]; }
    __device__ int &ri(int f, int i) const { return reinterpret_cast<int *>(r)[f * mc + i]; }
    __device__ float *vec(int f) const { return v + f * mc; }
};

// The workgroup's views of its dynamic LDS.
template <int MC>
__device__ inline Lds lds_views() {
    extern __shared__ float4 smem4[];
    float *sm = reinterpret_cast<float *>(smem4);
    Lds L;
    L.mc = MC;
    L.b = sm;
    L.j = L.b + body_floats();
    L.c = L.j + joint_floats();
    L.r = L.c + contact_floats();
    L.v = L.r + row_floats(MC);
    L.A = L.v + vec_floats(MC);
    L.red = L.A + tri_row_offset(MC);
    L.wb = reinterpret_cast<double *>(L.red + 64);
    L.qd = L.wb + 6 * kMaxBodies;
    L.inc_off = reinterpret_cast<int *>(L.red + 64 + bodyw_floats() + posed_floats());
    L.inc_list = L.inc_off + kMaxBodies + 1;
    L.s_int = L.inc_list + 2 * MC;
    L.t = L.red + 64 + bodyw_floats() + posed_floats() + inc_floats(MC);
    return L;
}

// world-frame rotation of a body (from LDS)
__device__ inline void body_rot(const Lds &L, int b, float R[9]) {
    for (int k = 0; k < 9; ++k) R[k] = L.bf(BR + k, b);
}

// o = M_b^-1 [lin; ang], applied in the body frame: lin / m, R (I^-1 (R^T ang))
__device__ inline void apply_minv(const Lds &L, int b, const float in[6], float out[6]) {
    float im = L.bf(BIM, b);
    out[0] = in[0] * im;
    out[1] = in[1] * im;
    out[2] = in[2] * im;
    float R[9], t[3], s[3];
    body_rot(L, b, R);
    mtv3(R, in + 3, t);
    t[0] *= L.bf(BII + 0, b);
    t[1] *= L.bf(BII + 1, b);
    t[2] *= L.bf(BII + 2, b);
    mv3(R, t, s);
    out[3] = s[0];
    out[4] = s[1];
    out[5] = s[2];
}

// Joint geometry: anchors, lever arms and frame rotations of both sides.
// Evaluated in FP64: the Baumgarte bias multiplies the position-level
// constraint value by beta / dt, so FP32 rounding of near-cancelling anchor
// offsets and near-orthogonal axis products (about 1e-7 absolute) would
// become velocity errors of order 1e-5.  J and everything downstream stay
// FP32.
__device__ inline void joint_geo(const Lds &L, const float *jf, int la, int lb, JointGeo &g) {
    double qa[7], qb[7];
    for (int k = 0; k < 7; ++k) qa[k] = L.qd[k * kMaxBodies + la];
    for (int k = 0; k < 7; ++k) qb[k] = lb >= 0 ? L.qd[k * kMaxBodies + lb] : 0.0;
    joint_geo_q(qa, qb, lb >= 0, jf, g);
}

__device__ inline void put_row(const Lds &L, int r, const float Ja[6], int la, const float Jb[6], int lb, float f,
                               int kind, float mu, SolverArgs &P) {
    for (int k = 0; k < 6; ++k) {
        L.rf(RJ + k, r) = Ja[k];
        L.rf(RJ + 6 + k, r) = lb >= 0 ? Jb[k] : 0.f;
    }
    L.ri(RIA, r) = la;
    L.ri(RIB, r) = lb;
    L.ri(RKIND, r) = kind;
    L.rf(RMU, r) = mu;
    L.rf(RREG, r) = 0.f;
    // position-level terms act over the time from the rows' configuration to
    // the end of the step: dt, or dt / 2 from the Moreau-Jean half step
    float bias = 0.f;
    float inv_h = (P.integrator == KAMX_MOREAU_JEAN ? 2.f : 1.f) / P.dt;
    if (kind == kRowBilateral) bias = P.baumgarte * f * inv_h;
    else if (kind == kRowLimit || kind == kRowNormal) bias = (f >= 0.f ? f : P.baumgarte * f) * inv_h;
    L.rf(RBIAS, r) = bias;
}

// Rows of joint j (5 rows from r0), Sec. 3 bilateral constraints; geometry
// and constraint values in FP64, rows stored in FP32.
__device__ inline void put_row6(const Lds &L, int r, const double Ja[6], int la, const double Jb[6], int lb, double f,
                                int kind, SolverArgs &P) {
    float fa[6], fb[6];
    for (int k = 0; k < 6; ++k) {
        fa[k] = (float)Ja[k];
        fb[k] = (float)Jb[k];
    }
    put_row(L, r, fa, la, fb, lb, (float)f, kind, 0.f, P);
}

__device__ inline void joint_rows(const Lds &L, int type, const JointGeo &g, int la, int lb, int r0,
                                  SolverArgs &P) {
    joint_constraints(type, g, [&](int e, const double Ja[6], const double Jb[6], double f) {
        put_row6(L, r0 + e, Ja, la, Jb, lb, f, kRowBilateral, P);
    });
}

// ---------------------------------------------------------------------------
// block-wide reductions (fixed order: butterfly within a wave, then waves in
// index order), results uniform across the workgroup
// ---------------------------------------------------------------------------

template <int NT>
__device__ inline void reduce4(float &m0, float &m1, float &m2, float &s3, float *red) {
    // rows of 16 lanes by DPP, then the wave's four rows through readlane,
    // then the waves in order through LDS; every step combines two values
    // that the partner combines in the other order, so all lanes agree.
    // m0, m1, m2 are +0 or above, or NaN (maxima of absolute values)
    m0 = lane_group_max<16>(m0);
    m1 = lane_group_max<16>(m1);
    m2 = lane_group_max<16>(m2);
    s3 = lane_group_sum<16>(s3);
    m0 = max_nonneg(max_nonneg(rdlane(m0, 0), rdlane(m0, 16)), max_nonneg(rdlane(m0, 32), rdlane(m0, 48)));
    m1 = max_nonneg(max_nonneg(rdlane(m1, 0), rdlane(m1, 16)), max_nonneg(rdlane(m1, 32), rdlane(m1, 48)));
    m2 = max_nonneg(max_nonneg(rdlane(m2, 0), rdlane(m2, 16)), max_nonneg(rdlane(m2, 32), rdlane(m2, 48)));
    s3 = (rdlane(s3, 0) + rdlane(s3, 16)) + (rdlane(s3, 32) + rdlane(s3, 48));
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) {
        red[4 * wave + 0] = m0;
        red[4 * wave + 1] = m1;
        red[4 * wave + 2] = m2;
        red[4 * wave + 3] = s3;
    }
    __syncthreads();
    m0 = red[0];
    m1 = red[1];
    m2 = red[2];
    s3 = red[3];
    for (int k = 1; k < NT / 64; ++k) {
        m0 = max_nonneg(m0, red[4 * k]);
        m1 = max_nonneg(m1, red[4 * k + 1]);
        m2 = max_nonneg(m2, red[4 * k + 2]);
        s3 = s3 + red[4 * k + 3];
    }
}

// The largest m (values of +0 or above, or NaN) and the sum s over the
// workgroup, in reduce4's order: within rows of 16 lanes, the wave's four rows by
// row broadcasts (lane 63 ends with (row 3 + row 2) + (row 1 + row 0)), the waves
// in order through LDS.  Uniform results.
template <int NT>
__device__ inline void reduce_max_sum(float &m, float &s, float *red) {
    m = lane_group_max<16>(m);
    s = lane_group_sum<16>(s);
    m = max_nonneg(m, dpp_rows<kDppBcast15, 0xa>(m));
    s += dpp_rows<kDppBcast15, 0xa>(s);
    m = max_nonneg(m, dpp_rows<kDppBcast31, 0xc>(m));
    s += dpp_rows<kDppBcast31, 0xc>(s);
    constexpr int NW = NT / 64;
    if ((threadIdx.x & 63) == 63) {
        red[2 * (threadIdx.x >> 6)] = m;
        red[2 * (threadIdx.x >> 6) + 1] = s;
    }
    __syncthreads();
    float v[2 * NW];
#pragma unroll
    for (int k = 0; k < 2 * NW; ++k) v[k] = red[k];
    m = v[0];
    s = v[1];
#pragma unroll
    for (int k = 1; k < NW; ++k) {
        m = max_nonneg(m, v[2 * k]);
        s += v[2 * k + 1];
    }
    m = uniform(m);
    s = uniform(s);
}

// The default workgroup size of a bucket.  The gather's four-thread bodies
// are capped by it rather than by the launched size, so that every size of a
// bucket sums each body in the same order (a smaller size runs the gather's
// tasks in more than one pass).
constexpr int default_bucket_threads(int mc) {
    for (const BucketSizes &v : kBucketSizes)
        if (v.mc == mc) return v.nt[0];
    return 0;
}

// ---------------------------------------------------------------------------
// matrix-free preconditioned Delassus product out = P J M^-1 J^T P x (Eq. 4),
// accumulated in FP64 over the two 6-blocks of every row: bodies gather
// their incident rows (fixed row order), rows then read their two bodies.
// Costs O(rows) instead of O(rows^2); used for the refinement residual of
// every x-update and for the dual residual.
// ---------------------------------------------------------------------------

// Body gather of the matrix-free product: g_b = sum over the rows incident
// to body b of J_{r,b}^T p_r x_r, one thread per (body, component), FP64,
// rows in increasing order.  Ends with a barrier.
template <int NT>
__device__ inline void delassus_gather(const Lds &L, int nb, const float *vp, const float *x) {
    // two adjacent threads per (body, component) take alternate rows of the
    // incidence list; their partial sums meet by one shuffle
    const int tid = threadIdx.x;
    const int ntask = 12 * nb;
    for (int t0 = 0; t0 < ntask; t0 += NT) {
        const int t = t0 + tid;
        const int bc = t >> 1, h = t & 1;
        const int b = bc / 6, c = bc - 6 * (bc / 6);
        double g0 = 0.0, g1 = 0.0;
        if (t < ntask) {
            int k = L.inc_off[b] + h;
            const int k1 = L.inc_off[b + 1];
            for (; k + 2 < k1; k += 4) {
                int e0 = L.inc_list[k], e1 = L.inc_list[k + 2];
                int r0 = e0 >> 1, r1 = e1 >> 1;
                g0 += (double)L.rf(RJ + 6 * (e0 & 1) + c, r0) * ((double)vp[r0] * (double)x[r0]);
                g1 += (double)L.rf(RJ + 6 * (e1 & 1) + c, r1) * ((double)vp[r1] * (double)x[r1]);
            }
            if (k < k1) {
                int e0 = L.inc_list[k];
                int r0 = e0 >> 1;
                g0 += (double)L.rf(RJ + 6 * (e0 & 1) + c, r0) * ((double)vp[r0] * (double)x[r0]);
            }
        }
        // partner lane (t ^ 1) is the DPP neighbour in the same wave
        const double gs = lane_group_sum<2>(g0 + g1);
        if (t < ntask && h == 0) L.wb[c * kMaxBodies + b] = gs;
    }
    __syncthreads();
}

// The gather with the bodies balanced over the threads: bodies with long
// incidence lists take four threads per component, the others two, so every
// thread walks about the same number of rows. gorder[0] = nh, the count of
// four-thread bodies (passed as nh), and gorder[1..nb] the bodies in task
// order, those nh first. The 12 (nb + nh) tasks run in passes of NT (one
// pass when they fit); a pass starts at a multiple of NT, so the lanes of a
// body's component form an aligned group of 4 or 2 within one wave.
struct GatherTask {
    int b, c, h, S;  // body, component, this thread's place among its S threads
    int k, k1;       // its entries of the incidence list: k, k + S, ... below k1
    bool heavy;
};

__device__ inline GatherTask gather_task(const Lds &L, int t, int nheavy, int ntask, int nh,
                                         const unsigned char *gorder) {
    GatherTask g;
    g.heavy = t < nheavy;
    int j;
    if (g.heavy) {
        j = t / 24;
        const int r = t - 24 * j;
        g.c = r >> 2;
        g.h = r & 3;
        g.S = 4;
    } else {
        const int u = t - nheavy, q = u / 12, r = u - 12 * q;
        j = nh + q;
        g.c = r >> 1;
        g.h = r & 1;
        g.S = 2;
    }
    g.b = g.k = g.k1 = 0;
    if (t < ntask) {
        g.b = gorder[1 + j];
        g.k = L.inc_off[g.b] + g.h;
        g.k1 = L.inc_off[g.b + 1];
    }
    return g;
}

// The entries of a task from k on, alternately into g0 and g1 (k lies an even
// number of entries after the task's first); px holds p_r x_r in FP64 (exact:
// two 24-bit factors).
__device__ inline void gather_rest(const Lds &L, const GatherTask &t, int k, const double *px, double &g0, double &g1) {
    for (; k + t.S < t.k1; k += 2 * t.S) {
        int e0 = L.inc_list[k], e1 = L.inc_list[k + t.S];
        int r0 = e0 >> 1, r1 = e1 >> 1;
        g0 += (double)L.rf(RJ + 6 * (e0 & 1) + t.c, r0) * px[r0];
        g1 += (double)L.rf(RJ + 6 * (e1 & 1) + t.c, r1) * px[r1];
    }
    if (k < t.k1) {
        int e0 = L.inc_list[k];
        int r0 = e0 >> 1;
        g0 += (double)L.rf(RJ + 6 * (e0 & 1) + t.c, r0) * px[r0];
    }
}

// The sums of a task's threads meet by lane exchanges; the first writes.
__device__ inline void gather_store(const Lds &L, const GatherTask &t, bool on, double gs) {
    gs += dpp<kDppXor1>(gs);
    const double g4 = gs + dpp<kDppXor2>(gs);
    if (on && t.h == 0) L.wb[t.c * kMaxBodies + t.b] = t.heavy ? g4 : gs;
}

// Rows of a gather task held in registers through the iterations; longer
// lists read the rest from LDS.  The biped's longest list has 30 rows on four
// threads.
constexpr int kGatherRegs = 8;

// acc (rows 0 and 2) and acc2 (rows 1 and 3) of X^T t for four rows; explicit
// fused multiply-adds, so that every caller computes the same bits
__device__ inline void x_accumulate(const mfx4 (&x)[4], mfx4 tv, mfx4 &acc, mfx4 &acc2) {
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[c] = __builtin_fmaf(x[0][c], tv[0], acc[c]);
#pragma unroll
    for (int c = 0; c < 4; ++c) acc2[c] = __builtin_fmaf(x[1][c], tv[1], acc2[c]);
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[c] = __builtin_fmaf(x[2][c], tv[2], acc[c]);
#pragma unroll
    for (int c = 0; c < 4; ++c) acc2[c] = __builtin_fmaf(x[3][c], tv[3], acc2[c]);
}

// w = M_b^-1 g_b in FP64 (body frame: R diag(I^-1) R^T for the angular part)
// (the angular part from the body's symmetric R diag(I^-1) R^T, formed once
// per step in FP64 by body_angular_minv)
__device__ inline void body_minv64(const Lds &L, int b, double w[6]) {
    const double *mi = reinterpret_cast<const double *>(L.b);
    double g[6];
    for (int c = 0; c < 6; ++c) g[c] = L.wb[c * kMaxBodies + b];
    const double im = L.bf(BIM, b);
    const double m00 = mi[b], m11 = mi[kMaxBodies + b], m22 = mi[2 * kMaxBodies + b];
    const double m01 = mi[3 * kMaxBodies + b], m02 = mi[4 * kMaxBodies + b], m12 = mi[5 * kMaxBodies + b];
    for (int c = 0; c < 3; ++c) w[c] = g[c] * im;
    // explicit fused multiply-adds: every workgroup-size variant computes the same bits
    w[3] = __builtin_fma(m02, g[5], __builtin_fma(m01, g[4], m00 * g[3]));
    w[4] = __builtin_fma(m12, g[5], __builtin_fma(m11, g[4], m01 * g[3]));
    w[5] = __builtin_fma(m22, g[5], __builtin_fma(m12, g[4], m02 * g[3]));
}

// The angular inverse inertia R diag(I^-1) R^T of every body in FP64 (six
// entries: 00, 11, 22, 01, 02, 12), stored as doubles [6][kMaxBodies] over
// the bodies' pose and twist fields.  Called once the rows and contacts are
// built and a barrier has passed: nothing reads those fields afterwards, and
// the rotation and inertia fields read here lie above them.  Ends with a
// barrier.
template <int NT>
__device__ inline void body_angular_minv(const Lds &L, int nb) {
    double *mi = reinterpret_cast<double *>(L.b);
    static_assert(12 <= BUF && BR >= 12 && BII >= 12, "six doubles per body below the fields still in use");
    const int b = threadIdx.x;
    if (b < nb) {
        double m[6];
        double R[9], ii[3];
        for (int k = 0; k < 9; ++k) R[k] = L.bf(BR + k, b);
        for (int k = 0; k < 3; ++k) ii[k] = L.bf(BII + k, b);
        const int ij[6][2] = {{0, 0}, {1, 1}, {2, 2}, {0, 1}, {0, 2}, {1, 2}};
        for (int e = 0; e < 6; ++e) {
            const int i = ij[e][0], j = ij[e][1];
            double v = (R[3 * i] * ii[0]) * R[3 * j];
            v = __builtin_fma(R[3 * i + 1] * ii[1], R[3 * j + 1], v);
            m[e] = __builtin_fma(R[3 * i + 2] * ii[2], R[3 * j + 2], v);
        }
        for (int e = 0; e < 6; ++e) mi[e * kMaxBodies + b] = m[e];
    }
    __syncthreads();
}

// Row r of the product after a gather, given w_a, w_b = M^-1 g of its bodies.
// (drive rows add their regularisation: D = J M^-1 J^T + R, Eq. 4, so row r
// of D~ x gains p_r R_r p_r x_r)
__device__ inline float delassus_row_w(const Lds &L, const float *vp, int r, const double wa[6], const double wbv[6],
                                       bool has_b, float xr) {
    double a0 = 0.0, a1 = 0.0;
    for (int c = 0; c < 6; ++c) a0 += (double)L.rf(RJ + c, r) * wa[c];
    if (has_b)
        for (int c = 0; c < 6; ++c) a1 += (double)L.rf(RJ + 6 + c, r) * wbv[c];
    const double pr = (double)vp[r];
    return (float)((a0 + a1 + (double)L.rf(RREG, r) * pr * (double)xr) * pr);
}

__device__ inline float delassus_row(const Lds &L, const float *vp, int r, float xr) {
    int ia = L.ri(RIA, r), ib = L.ri(RIB, r);
    double wa[6], wbv[6];
    body_minv64(L, ia, wa);
    if (ib >= 0) body_minv64(L, ib, wbv);
    return delassus_row_w(L, vp, r, wa, wbv, ib >= 0, xr);
}

// Full product out = D~ x (gather, then every row).  Ends with a barrier.
template <int NT>
__device__ inline void delassus_apply(const Lds &L, int m, int nb, const float *vp, const float *x, float *out) {
    delassus_gather<NT>(L, nb, vp, x);
    for (int r = threadIdx.x; r < m; r += NT) out[r] = delassus_row(L, vp, r, x[r]);
    __syncthreads();
}

// ---------------------------------------------------------------------------
// the fused step kernel
// ---------------------------------------------------------------------------

// Cholesky of D~ + diag(eta + rho) and the explicit inverse of the factor (Alg. 1
// step 1) for m rows, in the triangle.  Out of line: used for the step's own
// factorization and after a change of the adaptive penalty.
template <int MC, int NT>
__device__ __attribute__((noinline)) int factor_invert(int m) {
    const Lds L = lds_views<MC>();
    // red and wb are free here
    return factor_invert_tiles<MC, NT>(L.A, L.red, L.s_int + 2, uniform(m));
}

// D~ + diag(eta + rho) rebuilt into A after the adaptive penalty changed
// rho: the pairs, products and order of the step's assembly, with the
// Jacobi scales of the step and W = M^-1 J^T formed per pair from the bodies
// (the vector region that held W now holds the iterates).  Uses the
// reduction area (free between iterations) for the pair-task offsets.
template <int MC, int NT>
__device__ __attribute__((noinline)) void reassemble(int m, int nb, float eta) {
    const int tid = threadIdx.x;
    const Lds L = lds_views<MC>();
    float *A = L.A;
    const float *vp = L.vec(VP), *vrho = L.vec(VRHO);
    m = uniform(m);
    nb = uniform(nb);
    const int Mp = (m + 15) & ~15;
    const int n4 = tri_row_offset(Mp) >> 2;
    for (int k = tid; k < n4; k += NT) reinterpret_cast<float4 *>(A)[k] = make_float4(0.f, 0.f, 0.f, 0.f);
    int *toff = reinterpret_cast<int *>(L.red);
    if (tid == 0) {
        toff[0] = 0;
        for (int b = 0; b < nb; ++b) {
            int kb = L.inc_off[b + 1] - L.inc_off[b];
            toff[b + 1] = toff[b] + kb * (kb + 1) / 2;
        }
    }
    __syncthreads();
    if (tid >= m && tid < Mp) A[tri_row_offset(tid) + tid] = 1.f;
    auto wside = [&](int r, int sd, float out[6]) {
        const int b = L.ri(sd ? RIB : RIA, r);
        float in[6];
        for (int k = 0; k < 6; ++k) in[k] = L.rf(RJ + 6 * sd + k, r);
        if (b >= 0) apply_minv(L, b, in, out);
        else
            for (int k = 0; k < 6; ++k) out[k] = 0.f;
    };
    const int ntask = toff[nb];
    for (int t = tid; t < ntask; t += NT) {
        int lo = 0, hi = nb - 1;
        while (lo < hi) {
            int mid = (lo + hi + 1) >> 1;
            if (toff[mid] <= t) lo = mid;
            else hi = mid - 1;
        }
        const int b = lo;
        const int loc = t - toff[b];
        int u = (int)((sqrtf(8.f * (float)loc + 1.f) - 1.f) * 0.5f);
        while ((u + 1) * (u + 2) / 2 <= loc) ++u;
        while (u * (u + 1) / 2 > loc) --u;
        const int v = loc - u * (u + 1) / 2;
        const int ri_ = L.inc_list[L.inc_off[b] + u] >> 1;
        const int rj_ = L.inc_list[L.inc_off[b] + v] >> 1;
        const int ia = L.ri(RIA, ri_), ib = L.ri(RIB, ri_), ja = L.ri(RIA, rj_), jb = L.ri(RIB, rj_);
        int first = 1 << 30;
        if (ia == ja || ia == jb) first = ia;
        if (ib >= 0 && (ib == ja || ib == jb) && ib < first) first = ib;
        if (first != b) continue;
        float acc = 0.f, wv[6];
        if (ia == ja) {
            wside(rj_, 0, wv);
            for (int k = 0; k < 6; ++k) acc += L.rf(RJ + k, ri_) * wv[k];
        }
        if (ia == jb) {
            wside(rj_, 1, wv);
            for (int k = 0; k < 6; ++k) acc += L.rf(RJ + k, ri_) * wv[k];
        }
        if (ib >= 0 && ib == ja) {
            wside(rj_, 0, wv);
            for (int k = 0; k < 6; ++k) acc += L.rf(RJ + 6 + k, ri_) * wv[k];
        }
        if (ib >= 0 && ib == jb) {
            wside(rj_, 1, wv);
            for (int k = 0; k < 6; ++k) acc += L.rf(RJ + 6 + k, ri_) * wv[k];
        }
        if (ri_ == rj_) acc += L.rf(RREG, ri_);
        acc *= vp[ri_] * vp[rj_];
        if (ri_ == rj_) acc += eta + vrho[ri_];
        A[tri_row_offset(ri_) + rj_] = acc;
    }
    __syncthreads();
}

constexpr int kSolveConverged = 1 << 8;  // beside the KAMX_WORLD bits in solve_pass's status

// One pass of the PADMM iteration (Alg. 1 steps 3-10) from iteration it on, with
// the factor inverse X in the triangle: until the solve exits (returns 0) or the
// adaptive penalty wants rho changed (returns the direction).  The x-update of
// step 5 is computed as x + X^T X (rhs - (D~ + eta + rho) x): one refinement step
// from the previous iterate with the FP32 factor inverse and an FP64 matrix-free
// residual, so the fixed point solves the linear system to the accuracy of the
// residual, not to cond(D~) times FP32 epsilon.
//
// Inlined into the kernel, whose other functions hold nothing in registers while it
// runs and which has no caller's registers to keep: as a function of its own it
// stored and loaded 85 to 101 registers a lane, which at a workgroup on every CU went
// past the L2 and took 6 to 7 us of a step.  Hands over, in s_int: [4] the next iteration, [5] status bits and kSolveConverged, [6..8] r_p,
// r_d, r_c; the iterates x, y, z (and y, z as the extrapolated ones) and D~ x in
// their fields.
//
// An iteration is a chain of short phases between barriers, each bound by the
// latency of the LDS reads it starts with, so whatever a thread reads in every
// iteration stays in its registers for the pass (its entries of X for the x
// update, its rows of the body gather, its row's Jacobian and M^-1, its block's
// iterates) and a phase is left with one round of LDS reads of what other threads
// wrote, all issued before the first is used.  On the biped (224 rows, one world
// of eight waves per compute unit) an iteration takes 3.0 us against 5.2 us with
// every operand read from LDS where it is used.  Sums of two products name the one that
// is fused: the compiler takes either, by the function around them.
template <int MC, int NT>
__device__ __forceinline__ int solve_pass(KernelArgs &a, int w, int m, int nb, int nc, int row_c0, int nlim, int it) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));  // addresses formed here, not held through the kernel's loops
    SolverArgs &P = a.p;
    const int n_uni = nlim + 3 * nc;  // limit and contact rows: what the adaptive penalty acts on
    const Lds L = lds_views<MC>();
    const float *A = L.A;
    float *vp = L.vec(VP), *vrho = L.vec(VRHO), *vvt = L.vec(VVT);
    float *vx = L.vec(VX), *vyh = L.vec(VYH), *vzh = L.vec(VZH), *vyp = L.vec(VYP), *vzp = L.vec(VZP);
    float *vrhs = L.vec(VRHS), *vt = L.t, *vxn = L.vec(VXN), *vrinv = L.vec(VCOL), *vdx = L.vec(VDX);
    // p x per row in FP64, over the warm-start and aux fields
    double *px = reinterpret_cast<double *>(L.vec(VWS));
    static_assert(VAUX == VWS + 1 && (VWS * MC) % 2 == 0, "MC doubles in two adjacent fields");
    const mfx4 kZero4 = {0.f, 0.f, 0.f, 0.f};
    const float eta = P.eta, eps = P.eps, restart_factor = P.restart_factor, adapt_ratio = P.adapt_ratio;
    const int fixed_iters = P.fixed_iters, max_iters = P.max_iters, accel = P.accel;
    const int N = fixed_iters > 0 ? fixed_iters : max_iters;
    // the next checkpoint of the adaptive penalty (adapt_first, then doubling; -1: none)
    int check = -1;
    if (adapt_ratio > 0.f && n_uni > 0 && P.adapt_first > 0)
        for (check = P.adapt_first; check < it; check = check < (1 << 29) ? 2 * check : 0x7fffffff) {}

    // ---- gather balance: bodies with more than half the longest incidence
    // list go first and take four threads per component, as far as
    // 12 (nb + nh) <= T allows for the bucket's default workgroup size T (the
    // same bodies, so the same sums, at every size: a four-thread body adds its
    // rows in another order than a two-thread one); the order is bytes in the
    // reduction area, behind the partial sums.  Wave 0 builds it, lane b for body
    // b: a wave max, then ranks from ballots.
    static_assert(kMaxBodies <= 64, "gather order: one lane per body");
    unsigned char *gorder = reinterpret_cast<unsigned char *>(L.red + 36);
    float *zero4 = L.red + 60;  // four zeros, read in place of entries a thread does not have
    if (tid < 64) {
        const int kb = tid < nb ? L.inc_off[tid + 1] - L.inc_off[tid] : 0;
        int kmax = kb;
        for (int o = 32; o > 0; o >>= 1) kmax = max(kmax, __shfl_xor(kmax, o));
        const unsigned long long below = (1ull << tid) - 1ull;
        const unsigned long long hv = __ballot(tid < nb && 2 * kb > kmax);
        constexpr int kGatherThreads = default_bucket_threads(MC);
        static_assert(kGatherThreads >= 64, "gather cap from the bucket's default size");
        const int cap = max(kGatherThreads / 12 - nb, 0);
        const bool heavy = ((hv >> tid) & 1ull) && __popcll(hv & below) < cap;
        const unsigned long long hm = __ballot(heavy);
        const int nh = __popcll(hm);
        if (tid < nb) gorder[1 + (heavy ? __popcll(hm & below) : nh + tid - __popcll(hm & below))] = (unsigned char)tid;
        if (tid == 0) gorder[0] = (unsigned char)nh;
        if (tid < 4) zero4[tid] = 0.f;
    }
    __syncthreads();
    const int gnh = uniform((int)gorder[0]);

    // ---- slots of X (4 rows of a column quad) for the x update: quads c and
    // Q-1-c form a pair (balanced: together they span m + 4 rows), 16 threads per
    // pair take every 16th group of 4 rows.  kX1 slots cover the pair's first
    // quad and kX2 its second, which starts at or below the middle.  A wave's
    // pairs g0 .. g0 + 3 take kX1 slots of the first only when g0 is small and
    // kX2 = 2 of the second only when g0 >= 16, so the last of both share one.
    constexpr int kX1 = (MC + 63) / 64, kX2 = (MC / 2 + 63) / 64;
    static_assert(kX2 == 1 || (kX2 == 2 && MC / 4 - 16 * (kX1 - 1) <= 16), "shared slot of the x update");
    constexpr int kOwn1 = kX2 == 2 ? kX1 - 1 : kX1;  // slots of the first quad alone
    constexpr int kXSlots = kOwn1 + 1 + (kX2 == 2 ? 1 : 0);
    const int Q = (m + 3) >> 2, g0 = tid >> 4, kq = tid & 15;
    const bool b3 = kq & 8, b2 = kq & 4, b1 = kq & 2;
    const int c1 = g0, c2 = Q - 1 - g0;
    const bool one = c1 <= c2, two = c1 < c2;  // the pair has a first, a second quad
    const bool share1 = kX2 == 1 || uniform(g0) < 16;
    mfx4 X[kXSlots][4];
    // t of the slots' rows: t is 0 from row m to the end of its field, past the
    // last slot's last row
    const float *xt1 = vt + 4 * (min(c1, MC / 8) + kq), *xt2 = vt + 4 * (min(max(c2, 0), MC / 4) + kq);
    {
        auto load = [&](mfx4 (&x)[4], bool on, int c, int q) {
            const int r = 4 * (c + kq) + 64 * q;
            on = on && r < m;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                x[e] = on ? *reinterpret_cast<const mfx4 *>(A + tri_row_offset(r + e) + 4 * c) : kZero4;
        };
#pragma unroll
        for (int q = 0; q < kOwn1; ++q) load(X[q], one, c1, q);
        load(X[kOwn1], two, c2, 0);
        if (kX2 == 2) {
            if (share1) load(X[kXSlots - 1], one, c1, kX1 - 1);
            else load(X[kXSlots - 1], two, c2, 1);
        }
    }
    // the row this lane's sum of a t or x pass belongs to (-1: none): the eight
    // sums of a pair are reduce-scattered over its 16 lanes
    int prow = 4 * (b3 ? c2 : c1) + (b2 ? 2 : 0) + (b1 ? 1 : 0);
    if ((kq & 1) || !one || (b3 && !two) || prow >= m) prow = -1;
    float xw = 0.f, xp = 0.f;  // x and p of that row
    if (prow >= 0) {
        xw = vx[prow];
        xp = vp[prow];
    }
    // sums over the 16 lanes of a pair: halve the eight at each exchange (row
    // mirror, half-row mirror, then pairs), so that lanes 2k and 2k+1 end with
    // sum 4 b3 + 2 b2 + b1 of the bits of k
    auto pair_sums = [&](const mfx4 &s1, const mfx4 &s2) {
        const float v8[8] = {s1[0], s1[1], s1[2], s1[3], s2[0], s2[1], s2[2], s2[3]};
        float u4[4], u2[2];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            u4[k] = (b3 ? v8[k + 4] : v8[k]) + dpp<kDppMirror16>(b3 ? v8[k] : v8[k + 4]);
#pragma unroll
        for (int k = 0; k < 2; ++k) u2[k] = (b2 ? u4[k + 2] : u4[k]) + dpp<kDppMirror8>(b2 ? u4[k] : u4[k + 2]);
        float z = (b1 ? u2[1] : u2[0]) + dpp<kDppXor2>(b1 ? u2[0] : u2[1]);
        z += dpp<kDppXor1>(z);
        return z;
    };

    // ---- gather: this thread's first task, its first kGatherRegs rows' J and
    // the places of their p x
    const int gnheavy = 24 * gnh, gntask = gnheavy + 12 * (nb - gnh);
    const GatherTask gt = gather_task(L, tid, gnheavy, gntask, gnh, gorder);
    float gJ[kGatherRegs];
    const double *gx[kGatherRegs];
#pragma unroll
    for (int q = 0; q < kGatherRegs; ++q) {
        const int k = gt.k + q * gt.S;
        gJ[q] = 0.f;
        gx[q] = reinterpret_cast<const double *>(zero4);
        if (k < gt.k1) {
            const int e = L.inc_list[k];
            gJ[q] = L.rf(RJ + 6 * (e & 1) + gt.c, e >> 1);
            gx[q] = px + (e >> 1);
        }
    }
    const int grest = gt.k + kGatherRegs * gt.S;

    // ---- row io = tid / 2 belongs to the lane pair (2 io, 2 io + 1): the pair
    // evaluates the row's matrix-free product (even lane body a's side, odd lane
    // body b's), and the even lane of a block's first row owns the block, so
    // owner work spreads over every wave
    const int io = tid >> 1, hh = tid & 1;
    const int kind_o = io < m ? L.ri(RKIND, io) : -1;
    const bool owner_o = io < m && kind_o != kRowTangent && hh == 0;
    const bool normal_o = owner_o && kind_o == kRowNormal;
    const int blk_o = kind_o == kRowNormal ? 3 : 1;
    const float mu_o = io < m ? L.rf(RMU, io) : 0.f;
    const float cone_o = hw_rcp(1.f + mu_o * mu_o);
    int sb = -1;
    float sJ[6], sim = 0.f, spr = 0.f, sreg = 0.f;
    double sM[6];
    for (int c = 0; c < 6; ++c) {
        sJ[c] = 0.f;
        sM[c] = 0.0;
    }
    if (io < m) {
        sb = hh == 0 ? L.ri(RIA, io) : L.ri(RIB, io);
        spr = vp[io];
        sreg = L.rf(RREG, io);
        for (int c = 0; c < 6; ++c) sJ[c] = L.rf(RJ + 6 * hh + c, io);
        if (sb >= 0) {
            const double *mi = reinterpret_cast<const double *>(L.b);
            for (int c = 0; c < 6; ++c) sM[c] = mi[c * kMaxBodies + sb];
            sim = L.bf(BIM, sb);
        }
    }
    const double *sg = L.wb + (sb >= 0 ? sb : 0);
    const float *sx = io < m ? vxn + io : zero4;
    // whether this wave has a contact's owner, and whether some contact's rows
    // lie in two waves (32 rows to a wave)
    const bool wave_contact = __ballot(normal_o) != 0;
    bool straddle = false;
    for (int c = 0; c < nc; ++c) straddle = straddle || ((row_c0 + 3 * c) & 31) > 29;

    // ---- block owners: iterates, free velocity and penalty (the same in all
    // rows of a block)
    float oyh[3], ozh[3], oyp[3], ozp[3], ovt[3], ox[3], odx[3];
    const float orho = owner_o ? vrho[io] : 1.f, ori = owner_o ? vrinv[io] : 1.f;
    _Pragma("unroll") for (int e = 0; e < 3; ++e) {
        const bool on = owner_o && e < blk_o;
        oyh[e] = on ? vyh[io + e] : 0.f;
        ozh[e] = on ? vzh[io + e] : 0.f;
        oyp[e] = on ? vyp[io + e] : 0.f;
        ozp[e] = on ? vzp[io + e] : 0.f;
        ovt[e] = on ? vvt[io + e] : 0.f;
        ox[e] = on ? vx[io + e] : 0.f;
        odx[e] = on ? vdx[io + e] : 0.f;
    }
    // steps 4-5: rhs = -v~_f - Gamma(z^) + eta x + rho y^ + z^, and its residual
    // against the current x
    auto put_rhs = [&]() {
        if (owner_o) {
            const float s_own = kind_o == kRowNormal ? mu_o * hw_sqrt(__builtin_fmaf(ozh[1], ozh[1], ozh[2] * ozh[2])) : 0.f;
            _Pragma("unroll") for (int e = 0; e < 3; ++e) if (e < blk_o) {
                float rhs = -ovt[e] - (e == 0 ? s_own : 0.f) + eta * ox[e] + orho * oyh[e] + ozh[e];
                vrhs[io + e] = rhs - (odx[e] + (eta + orho) * ox[e]);
            }
        }
    };
    put_rhs();

    float a_k = 1.f, c_prev = INFINITY;
    float rp = 0.f, rd = 0.f, rc = 0.f;
    if (it > 1) {  // a pass without an iteration leaves the previous one's residuals
        rp = __int_as_float(uniform(L.s_int[6]));
        rd = __int_as_float(uniform(L.s_int[7]));
        rc = __int_as_float(uniform(L.s_int[8]));
    }
    int adapt_pending = 0, status = 0;
    const int it0 = it;
    const bool timing = a.phase_clk != nullptr;
    uint64_t sub[6] = {0, 0, 0, 0, 0, 0}, tmark = 0;
#define KAMX_MARK(k)                                             \
    if (timing) {                                                \
        uint64_t now_ = wall_clock64();                          \
        if ((k) > 0) sub[(k) > 0 ? (k) - 1 : 0] += now_ - tmark; \
        tmark = now_;                                            \
    }
    for (; it <= N; ++it) {
        KAMX_MARK(0);
        __syncthreads();
        KAMX_MARK(1);
        // t = X r over groups of 4 rows: groups g and Q-1-g form a pair
        // (balanced: together they span Q+1 column quads); 16 threads per pair
        // take every 16th column quad, reading the quad of r once for the 4 rows
        // of a group.  The rows of a group lie back to back, 4(G+1) floats apart;
        // the pads of the diagonal quad hold 0 and r is 0 past row m, and rows
        // past m (up to the next multiple of 16) hold finite values whose sums are
        // not stored.  Two quads' reads are in flight at a time; a lane past its
        // group's last quad reads that quad against zeros, and threads past the
        // last pair read the last one's rows (96 rows on 512 threads have 32 thread
        // groups for 12 pairs) for sums that are not stored either.
        {
            int to = tid;
            asm volatile("" : "+v"(to));  // addresses formed here, not held through the loop
            const int gg = to >> 4, kk = to & 15;
            const int G1 = pair_first(gg, MC), G2 = max(Q - 1 - gg, 0);
            static_assert(4 * pair_first(NT / 16 - 1, MC) + 3 < MC, "the t pass stays in the triangle");
            const float *R1 = A + tri_row_offset(4 * G1), *R2 = A + tri_row_offset(4 * G2);
            mfx4 s1 = kZero4, s2 = kZero4;
            struct Chunk {
                mfx4 r, x[4];
            };
            auto read = [&](Chunk &h, const float *R, int G, int q) {
                const int c = kk + 16 * q, cc = min(c, G);
                h.r = *reinterpret_cast<const mfx4 *>(c <= G ? vrhs + 4 * c : zero4);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    h.x[e] = *reinterpret_cast<const mfx4 *>(R + 4 * e * (G + 1) + 4 * cc);
            };
            auto add = [&](const Chunk &h, mfx4 &s) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int k = 0; k < 4; ++k) s[k] = __builtin_fmaf(h.x[k][e], h.r[e], s[k]);
            };
            constexpr int kT1 = (MC / 8 + 15) / 16, kT2 = (MC / 4 + 15) / 16;
            static_assert(kT1 <= 2 && kT2 <= 4 && kT2 >= kT1, "chunks of a t-pass pair");
            // chunks a wave needs: its largest first and second group
            const int gw = uniform(gg);
            const int n1 = min((gw + 3) / 16 + 1, kT1), n2 = (max(Q - 1 - gw, 0)) / 16 + 1;
            if constexpr (kT2 <= 2) {
                // small worlds: every read in flight
                Chunk ha, hb;
                read(hb, R2, G2, 0);
                read(ha, R1, G1, 0);
                add(hb, s2);
                add(ha, s1);
                if (kT2 > 1 && n2 > 1) {
                    read(hb, R2, G2, 1);
                    add(hb, s2);
                }
                static_assert(kT2 > 2 || kT1 == 1, "first groups of small worlds fit one chunk");
            } else {
                // large ones have the waves to overlap and no registers to spare
                Chunk h;
#pragma clang loop unroll(disable)
                for (int q = 0; q < n2; ++q) {
                    read(h, R2, G2, q);
                    add(h, s2);
                }
#pragma clang loop unroll(disable)
                for (int q = 0; q < n1; ++q) {
                    read(h, R1, G1, q);
                    add(h, s1);
                }
            }
            const float z = pair_sums(s1, s2);
            if (prow >= 0) vt[prow] = z;
        }
        __syncthreads();
        KAMX_MARK(2);
        // x_new = x + X^T t: every slot's t against its X in registers (packed
        // rows are padded to 4 floats and the pads hold 0, so the quad that
        // contains the diagonal enters as-is, and t is 0 past row m, where the
        // rows up to the next multiple of 4 hold finite values)
        {
            mfx4 s1 = kZero4, s2 = kZero4, o1 = kZero4, o2 = kZero4;
            mfx4 tv[kXSlots];
#pragma unroll
            for (int q = 0; q < kOwn1; ++q) tv[q] = *reinterpret_cast<const mfx4 *>(xt1 + 64 * q);
            tv[kOwn1] = *reinterpret_cast<const mfx4 *>(xt2);
            if (kX2 == 2) tv[kXSlots - 1] = *reinterpret_cast<const mfx4 *>(share1 ? xt1 + 64 * (kX1 - 1) : xt2 + 64);
#pragma unroll
            for (int q = 0; q < kOwn1; ++q) x_accumulate(X[q], tv[q], s1, o1);
            x_accumulate(X[kOwn1], tv[kOwn1], s2, o2);
            if (kX2 == 2) {
                if (share1) x_accumulate(X[kXSlots - 1], tv[kXSlots - 1], s1, o1);
                else x_accumulate(X[kXSlots - 1], tv[kXSlots - 1], s2, o2);
            }
            s1 += o1;
            s2 += o2;
            const float z = pair_sums(s1, s2);
            if (prow >= 0) {
                xw = xw + z;
                vxn[prow] = xw;
                px[prow] = (double)xp * (double)xw;
            }
        }
        __syncthreads();
        KAMX_MARK(3);
        // v~ - v~_f = D~ x_new (matrix-free, FP64): bodies gather here, the rows
        // read their two bodies below
        {
            double s0 = 0.0, s1 = 0.0, xv[kGatherRegs];
#pragma unroll
            for (int q = 0; q < kGatherRegs; ++q) xv[q] = *gx[q];
#pragma unroll
            for (int q = 0; q < kGatherRegs; q += 2) {
                s0 += (double)gJ[q] * xv[q];
                s1 += (double)gJ[q + 1] * xv[q + 1];
            }
            gather_rest(L, gt, grest, px, s0, s1);
            gather_store(L, gt, tid < gntask, s0 + s1);
            // (only when the tasks outnumber the threads)
            for (int t0 = NT; t0 < gntask; t0 += NT) {
                const GatherTask g = gather_task(L, t0 + tid, gnheavy, gntask, gnh, gorder);
                s0 = s1 = 0.0;
                gather_rest(L, g, g.k, px, s0, s1);
                gather_store(L, g, t0 + tid < gntask, s0 + s1);
            }
        }
        __syncthreads();
        KAMX_MARK(4);
        // v~ - v~_f of row io in FP64: J_a M_a^-1 g_a on the even lane,
        // J_b M_b^-1 g_b on the odd lane, added by the pair sum (M^-1 as in
        // body_minv64)
        float yb[3], zb[3];
        float dxo;
        {
            double side = 0.0, g[6], wv[6];
            for (int c = 0; c < 6; ++c) g[c] = sg[c * kMaxBodies];
            ox[0] = *sx;
            if (wave_contact) {
                ox[1] = sx[1];
                ox[2] = sx[2];
            }
            for (int c = 0; c < 3; ++c) wv[c] = g[c] * (double)sim;
            wv[3] = __builtin_fma(sM[4], g[5], __builtin_fma(sM[3], g[4], sM[0] * g[3]));
            wv[4] = __builtin_fma(sM[5], g[5], __builtin_fma(sM[1], g[4], sM[3] * g[3]));
            wv[5] = __builtin_fma(sM[2], g[5], __builtin_fma(sM[5], g[4], sM[4] * g[3]));
            for (int c = 0; c < 6; ++c) side += (double)sJ[c] * wv[c];
            side = sb >= 0 ? side : 0.0;
            side = lane_group_sum<2>(side);
            const double pr = (double)spr;
            dxo = (float)((side + (double)sreg * pr * (double)ox[0]) * pr);
        }
        // a contact's tangent rows belong to the next two lane pairs, which hand
        // their rows to the owner: by lane exchange, or through LDS where some
        // contact lies in two waves
        odx[0] = dxo;
        if (straddle) {
            if (hh == 0 && io < m) vdx[io] = dxo;
            __syncthreads();
            if (normal_o) {
                odx[1] = vdx[io + 1];
                odx[2] = vdx[io + 2];
            }
        } else if (wave_contact) {
            odx[1] = __shfl_down(dxo, 2);
            odx[2] = __shfl_down(dxo, 4);
        }
        // steps 6-7 and the residuals of step 9 (block owners)
        float lrp = 0.f, lrd = 0.f, lrc = 0.f, lcc = 0.f;
        if (owner_o) {
            float vv[3];
            _Pragma("unroll") for (int e = 0; e < 3; ++e) if (e < blk_o) vv[e] = odx[e] + ovt[e];
            if (kind_o == kRowNormal) {
                // the cone's three cases as selections (proj_cone's values)
                const float w0 = ox[0] - ozh[0] * ori, w1 = ox[1] - ozh[1] * ori, w2 = ox[2] - ozh[2] * ori;
                const float tn = hw_sqrt(__builtin_fmaf(w1, w1, w2 * w2));
                const float mt = mu_o * tn, ln = add_rounded(mt, w0) * cone_o;
                const float sc = tn > 0.f ? mu_o * ln * hw_rcp(tn) : 0.f;
                const bool in = tn <= mu_o * w0, below = mt <= -w0;
                yb[0] = in ? w0 : (below ? 0.f : ln);
                yb[1] = in ? w1 : (below ? 0.f : sc * w1);
                yb[2] = in ? w2 : (below ? 0.f : sc * w2);
            } else if (kind_o == kRowLimit) {
                yb[0] = fmaxf(ox[0] - ozh[0] * ori, 0.f);
            } else {
                yb[0] = ox[0] - ozh[0] * ori;
            }
            _Pragma("unroll") for (int e = 0; e < 3; ++e) if (e < blk_o) {
                zb[e] = ozh[e] - orho * (ox[e] - yb[e]);
                lrp = fmaxf(lrp, fabsf(ox[e] - yb[e]));
                float dy = yb[e] - oyh[e], dz = zb[e] - ozh[e];
                lcc += __builtin_fmaf(orho * dy, dy, dz * dz * ori);
            }
            float g = kind_o == kRowNormal ? mu_o * hw_sqrt(__builtin_fmaf(vv[1], vv[1], vv[2] * vv[2])) : 0.f;
            _Pragma("unroll") for (int e = 0; e < 3; ++e) if (e < blk_o) {
                float d = vv[e] + (e == 0 ? g : 0.f) - zb[e];
                lrd = fmaxf(lrd, fabsf(d));
                if (d != d) lrd = fabsf(d);
            }
            if (kind_o == kRowNormal) lrc = fabsf(__builtin_fmaf(yb[2], vv[2], __builtin_fmaf(yb[0], vv[0] + g, yb[1] * vv[1])));
            else if (kind_o == kRowLimit) lrc = fabsf(yb[0] * vv[0]);
            if (lrp != lrp || lcc != lcc) lrp = NAN;
        }
        // step 8's next Nesterov weights, before the reduction that decides on them
        const float a_next = 0.5f * (1.f + hw_sqrt(1.f + 4.f * a_k * a_k));
        const float beta = (a_k - 1.f) * hw_rcp(a_next), c_most = restart_factor * c_prev;
        // every iteration needs the restart sum and whether all residuals are
        // finite and below eps: their largest.  Each for itself is reduced only
        // where it is read
        float rmax = max_nonneg(max_nonneg(lrp, lrd), lrc), csum = lcc;
        reduce_max_sum<NT>(rmax, csum, L.red);
        KAMX_MARK(5);
        // step 8: Nesterov with adaptive restart
        const bool restart = accel && !(csum < c_most);
        if (!accel || !restart) {
            if (accel) {
                a_k = a_next;
                c_prev = csum;
            }
            if (owner_o) {
                _Pragma("unroll") for (int e = 0; e < 3; ++e) if (e < blk_o) {
                    oyh[e] = accel ? yb[e] + beta * (yb[e] - oyp[e]) : yb[e];
                    ozh[e] = accel ? zb[e] + beta * (zb[e] - ozp[e]) : zb[e];
                }
            }
        } else {
            a_k = 1.f;
            c_prev = c_prev / restart_factor;
            _Pragma("unroll") for (int e = 0; e < 3; ++e) {
                oyh[e] = oyp[e];
                ozh[e] = ozp[e];
            }
        }
        if (owner_o) {
            _Pragma("unroll") for (int e = 0; e < 3; ++e) if (e < blk_o) {
                oyp[e] = yb[e];
                ozp[e] = zb[e];
            }
        }
        put_rhs();
        KAMX_MARK(6);
        // adaptive penalty (not in the paper: residual balancing) at the
        // checkpoints of a solve that does not exit here; every value here is
        // uniform
        const bool done = fixed_iters <= 0 && rmax < eps;
        int adapt_dir = 0;
        if (it == N || it == check || done || !isfinite(rmax)) {
            __syncthreads();  // every wave has read the partial results
            reduce4<NT>(lrp, lrd, lrc, lcc, L.red);
            rp = uniform(lrp);
            rd = uniform(lrd);
            rc = uniform(lrc);
            if (it == check) {
                check = check < (1 << 29) ? 2 * check : 0x7fffffff;
                if (!done) {
                    if (rd > adapt_ratio * rp) adapt_dir = 1;
                    else if (rp > adapt_ratio * rd) adapt_dir = 2;
                }
            }
        }
        if (tid == 0 && a.rlog && P.log_restarts && it <= max_iters)
            a.rlog[(size_t)w * max_iters + (it - 1)] = (uint8_t)((restart ? 1 : 0) | (adapt_dir << 1));
        if (!isfinite(rmax)) {
            status = KAMX_WORLD_NONFINITE;
            break;
        }
        if (done) {
            status = kSolveConverged;
            break;
        }
        if (adapt_dir) {
            adapt_pending = adapt_dir;
            ++it;
            break;
        }
    }
#undef KAMX_MARK
    // the owners' iterates back to LDS, for the outputs and the next pass
    if (owner_o) {
        _Pragma("unroll") for (int e = 0; e < 3; ++e) if (e < blk_o) {
            vx[io + e] = ox[e];
            vyp[io + e] = oyp[e];
            vzp[io + e] = ozp[e];
            vdx[io + e] = odx[e];
            vyh[io + e] = oyp[e];
            vzh[io + e] = ozp[e];
        }
    }
    if (tid == 0) {
        if (timing)
            for (int k = 0; k < 6; ++k)
                a.phase_clk[16 * w + 8 + k] = (it0 > 1 ? a.phase_clk[16 * w + 8 + k] : 0) + sub[k];
        L.s_int[4] = it;
        L.s_int[5] = status;
        L.s_int[6] = __float_as_int(rp);
        L.s_int[7] = __float_as_int(rd);
        L.s_int[8] = __float_as_int(rc);
    }
    __syncthreads();
    return adapt_pending;
}

// One step of world w in three parts (the workgroup owns the world): its rows and their
// factor, the solve, and the outputs.  step is the step index that keys the
// actuation noise; k the position of the step inside the launch.

// Rows of a world in the layout its contacts give it.
struct RowCounts {
    int nc, c0, m;  // contacts, first contact row, rows
    __device__ inline RowCounts(const WorldInfo &W, const Lds &L)
        : nc(uniform(L.s_int[1])), c0(5 * W.nj + W.nlim + W.ndrv), m(c0 + 3 * nc) {}
};

// What is left of a step once its rows are built.
enum StepLeft { kStepFeatures = -1 /* nothing: the launch wanted the features */, kStepSolve, kStepFailed, kStepNoRows };

// From the bodies to the factor inverse.
template <int MC, int NT>
__device__ __attribute__((noinline)) int step_begin(KernelArgs *args, int k) {
    const int tid = threadIdx.x;
    KernelArgs &a = *uniform_args(args);
    k = uniform(k);
    // read per step (not hoisted out of the caller's step loop)
    const int w = uniform(a.bucket_worlds[blockIdx.x]);
    const uint32_t step = (uint32_t)uniform((int)*a.step_ctr) + (uint32_t)k;
    const WorldInfo W = uniform_world(a.worlds + w);
    SolverArgs &P = a.p;

    const Lds L = lds_views<MC>();
    int *s_int = L.s_int;
    float *A = L.A;

    const int nb = W.nb, nj = W.nj;

    if (a.phase_clk && tid == 0) {
        a.phase_clk[16 * w + 0] = wall_clock64();
        a.phase_clk[16 * w + 14] = __smid();  // compute unit that runs this world
        a.phase_clk[16 * w + 15] = __builtin_amdgcn_s_getreg(GETREG_IMMED(31, 0, HW_ID));  // raw hardware id
    }
    // ---- reset: a world whose reset body fell below the threshold restarts
    if (tid == 0) {
        int rs = 0;
        if (W.reset_body >= 0) {
            float z = a.q[7 * (W.b0 + W.reset_body) + 2];
            rs = z < P.reset_height;
        }
        s_int[0] = rs;
        if (rs && a.stage == 0) a.reset_count[w] += 1;
    }
    __syncthreads();
    const int reset = uniform(s_int[0]);

    // ---- bodies: state, rotation, inverse mass properties
    for (int b = tid; b < nb; b += NT) {
        int gb = W.b0 + b;
        const float *qs = reset ? a.q0 : a.q;
        const float *us = reset ? a.u0 : a.u;
        float q[7], u6[6];
        for (int k = 0; k < 7; ++k) q[k] = qs[7 * gb + k];
        for (int k = 0; k < 6; ++k) u6[k] = us[6 * gb + k];
        // the configuration the rows are built at, in FP64: the pre-step pose,
        // or (Moreau-Jean) the half-step pose, whose joint geometry must not
        // carry FP32 rounding into the Baumgarte bias
        double qd[7];
        for (int k = 0; k < 7; ++k) qd[k] = q[k];
        if (P.integrator == KAMX_MOREAU_JEAN) {
            double u6d[6], qm[7];
            for (int k = 0; k < 6; ++k) u6d[k] = u6[k];
            advance_pose(qd, u6d, 0.5 * (double)P.dt, qm);
            for (int k = 0; k < 7; ++k) qd[k] = qm[k];
            for (int k = 0; k < 7; ++k) q[k] = (float)qm[k];
        }
        for (int k = 0; k < 7; ++k) L.qd[k * kMaxBodies + b] = qd[k];
        for (int k = 0; k < 7; ++k) L.bf(BQ + k, b) = q[k];
        for (int k = 0; k < 6; ++k) L.bf(BU + k, b) = u6[k];
        float R[9];
        rot_of_quat(q + 3, R);
        for (int k = 0; k < 9; ++k) L.bf(BR + k, b) = R[k];
        for (int k = 0; k < 3; ++k) L.bf(BII + k, b) = 1.f / a.inertia[3 * gb + k];
        L.bf(BIM, b) = 1.f / a.mass[gb];
    }
    __syncthreads();

    // ---- joints: coordinate, rate and actuation (generalized force along
    //      the coordinate: external + PD + noise)
    for (int j = tid; j < nj; j += NT) {
        int gj = W.j0 + j;
        int type = a.jint[4 * gj], la = a.jint[4 * gj + 1], lb = a.jint[4 * gj + 2], fl = a.jint[4 * gj + 3];
        const float *jf = a.jf + kJointFloats * gj;
        JointGeo g;
        joint_geo(L, jf, la, lb, g);
        float Ja[6], Jb[6];
        float c = (float)joint_coord(type, g, Ja, Jb);
        float rate = 0.f;
        for (int k = 0; k < 6; ++k) rate += Ja[k] * L.bf(BU + k, la);
        if (lb >= 0)
            for (int k = 0; k < 6; ++k) rate += Jb[k] * L.bf(BU + k, lb);
        float tau = a.ext_tau ? a.ext_tau[gj] : 0.f;
        float kp = jf[16], kd = jf[17], ref = jf[18];
        if (!(fl & kJointDriven) && (kp != 0.f || kd != 0.f)) tau += kp * (ref - c) - kd * rate;
        if ((fl & kJointActuated) && P.torque_sigma != 0.f)
            tau += P.torque_sigma * noise_normal(P.seed_lo, P.seed_hi, (uint32_t)w, step, (uint32_t)j);
        L.jfld(JTAU, j) = tau;
        for (int k = 0; k < 6; ++k) {
            L.jfld(JC + k, j) = Ja[k];
            L.jfld(JC + 6 + k, j) = Jb[k];
        }
        reinterpret_cast<int *>(L.j)[JA * kMaxJoints + j] = la;
        reinterpret_cast<int *>(L.j)[JB * kMaxJoints + j] = lb;
        reinterpret_cast<int *>(L.j)[JTF * kMaxJoints + j] = type | (fl << 4);
        a.tau_out[gj] = tau;
    }
    __syncthreads();

    // ---- feature pass of the learned warm start: the state the step starts
    //      from (positions relative to the reset body), the previous step's
    //      impulses by slot and the generalized forces of this step
    // feature t of this world (same layout as kamx_model_features)
    auto feature = [&](int t) -> float {
        const int rb = W.reset_body;
        const int rc0 = 5 * nj + W.nlim + W.ndrv;
        const int S = rc0 + 3 * a.n_contact_slots;
        if (t < 13 * nb) {
            const int b = t / 13, c = t - 13 * (t / 13);
            if (c < 3) return L.bf(BQ + c, b) - (rb >= 0 ? L.bf(BQ + c, rb) : 0.f);
            if (c < 7) return L.bf(BQ + c, b);
            return L.bf(BU + c - 7, b);
        }
        t -= 13 * nb;
        if (t < S) {
            float v = 0.f;
            if (!reset) {
                if (t < rc0) {
                    v = a.lambda[W.row_base + t];
                } else {
                    const int slot = (t - rc0) / 3, e = (t - rc0) - 3 * ((t - rc0) / 3);
                    const int nprev = a.ncontacts_out[w];
                    for (int q = 0; q < nprev && q < kMaxContacts; ++q)
                        if (a.keys[w * kMaxContacts + q] >= 0 && contact_slot(a.keys[w * kMaxContacts + q]) == slot) {
                            v = a.lambda[W.row_base + rc0 + 3 * q + e];
                            break;
                        }
                }
            }
            return v;
        }
        return L.jfld(JTAU, t - S);
    };
    if (a.stage == 1) {
        float *f = a.features + (long)w * a.n_feat;
        for (int t = tid; t < a.n_feat; t += NT) f[t] = feature(t);
        return kStepFeatures;
    }

    // ---- learned warm start: the network predicts this world's impulses by
    //      slot, on the matrix cores with the batched kernels' operand layout
    //      and accumulation order (so the prediction has the same bits); the
    //      features are row 0 of the 16-row operand, the other rows zero.
    //      The triangle region of LDS is free until the Delassus assembly.
    if (P.warmstart == KAMX_WARM_LEARNED && !reset) {
        const __attribute__((address_space(4))) MlpView &N = a.mlp;
        __bf16 *xh = reinterpret_cast<__bf16 *>(A);
        __bf16 *h1 = xh + N.fp;
        __bf16 *h2 = h1 + N.H;
        for (int t = tid; t < N.fp; t += NT) xh[t] = to_bf16(t < N.n_in ? (feature(t) - N.mu_in[t]) * N.s_in[t] : 0.f);
        __syncthreads();
        const int lane = tid & 63, wv = tid >> 6, fr = lane & 15, fk = (lane >> 4) * 8;
        constexpr int NW = NT / 64;
        const bf16x8 zero8 = {};
        auto layer = [&](const __bf16 *x, int K, const __bf16 *Wt, int nout_pad, auto &&epilogue) {
            for (int t = wv; t < nout_pad / 16; t += NW) {
                floatx4 acc = {0.f, 0.f, 0.f, 0.f};
                const __bf16 *wt = Wt + (long)t * 16 * K + fr * (N.blocked ? 32 : K) + fk;
                const int step32 = N.blocked ? 512 : 32;  // from 32 columns to the next
                constexpr int kAhead = 8;  // steps of K loaded together
                for (int k0 = 0; k0 < K; k0 += 32 * kAhead) {
                    bf16x8 bv[kAhead];
#pragma unroll
                    for (int q = 0; q < kAhead; ++q)
                        bv[q] = *reinterpret_cast<const bf16x8 *>(wt + (min(k0 + 32 * q, K - 32) >> 5) * step32);
#pragma unroll
                    for (int q = 0; q < kAhead; ++q) {
                        if (k0 + 32 * q >= K) break;
                        const bf16x8 av = fr == 0 ? *reinterpret_cast<const bf16x8 *>(x + k0 + 32 * q + fk) : zero8;
                        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv[q], acc, 0, 0, 0);
                    }
                }
                if (fk == 0) epilogue(16 * t + fr, acc[0]);  // row 0 of the block: lanes 0-15, component 0
            }
        };
        layer(xh, N.fp, N.w1, N.H, [&](int n, float v) { h1[n] = to_bf16(gelu(v + N.b1[n])); });
        __syncthreads();
        layer(h1, N.H, N.w2, N.H, [&](int n, float v) { h2[n] = to_bf16(gelu(v + N.b2[n])); });
        __syncthreads();
        float *ws = a.ws_slots + (long)w * N.n_out;
        layer(h2, N.H, N.w3, N.op, [&](int n, float v) {
            if (n < N.n_out) ws[n] = __builtin_fmaf(N.sd_out[n], v + N.b3[n], N.mu_out[n]);
        });
        __syncthreads();
    }

    // ---- free velocity of every body: u_f = u + dt M^-1 h
    for (int b = tid; b < nb; b += NT) {
        float m = 1.f / L.bf(BIM, b);
        float h[6];
        h[0] = m * P.gx;
        h[1] = m * P.gy;
        h[2] = m * P.gz;
        // gyroscopic -w x (I_w w), I_w w evaluated in the body frame
        float R[9], w3[3], t[3], Iw[3], gyro[3];
        body_rot(L, b, R);
        for (int k = 0; k < 3; ++k) w3[k] = L.bf(BU + 3 + k, b);
        mtv3(R, w3, t);
        for (int k = 0; k < 3; ++k) t[k] /= L.bf(BII + k, b);
        mv3(R, t, Iw);
        cross(w3, Iw, gyro);
        h[3] = -gyro[0];
        h[4] = -gyro[1];
        h[5] = -gyro[2];
        const int *ja = reinterpret_cast<const int *>(L.j) + JA * kMaxJoints;
        const int *jb = reinterpret_cast<const int *>(L.j) + JB * kMaxJoints;
        for (int j = 0; j < nj; ++j) {
            float tau = L.jfld(JTAU, j);
            if (tau == 0.f) continue;
            if (ja[j] == b)
                for (int k = 0; k < 6; ++k) h[k] += tau * L.jfld(JC + k, j);
            if (jb[j] == b)
                for (int k = 0; k < 6; ++k) h[k] += tau * L.jfld(JC + 6 + k, j);
        }
        float dv[6];
        apply_minv(L, b, h, dv);
        for (int k = 0; k < 6; ++k) L.bf(BUF + k, b) = L.bf(BU + k, b) + P.dt * dv[k];
    }

    // ---- contacts: explicit list, or probes below the margin (compacted in
    //      probe order by a wave ballot)
    int *cint = reinterpret_cast<int *>(L.c);
    constexpr bool kBoxFits = (long)sizeof(float) * (8L * (MC / 4) * (MC / 4 + 1)) >= (long)sizeof(BoxLds);
    if (kBoxFits && a.box_geom) {
        // boxes in a bin: contacts generated here from the poses the step
        // starts from, with the candidates in the LDS of the Delassus
        // triangle (free until the assembly)
        if constexpr (kBoxFits) {
            BoxLds &S = *reinterpret_cast<BoxLds *>(A);
            const int n = box_bin_generate<NT>(
                S, nb, a.box_geom + 4 * (long)W.b0, a.bin_wx, a.bin_wy, a.bin_margin, W.contact_cap,
                [&](int b, float c[3], float qt[4]) {
                    for (int e = 0; e < 3; ++e) c[e] = L.bf(BQ + e, b);
                    for (int e = 0; e < 4; ++e) qt[e] = L.bf(BQ + 3 + e, b);
                },
                [&](int c, int key, float gap, const float p[3], const float nn[3], float mu, int la, int lb) {
                    for (int e = 0; e < 3; ++e) {
                        L.cf(CP + e, c) = p[e];
                        L.cf(CN + e, c) = nn[e];
                    }
                    L.cf(CGAP, c) = gap;
                    L.cf(CMU, c) = mu;
                    cint[CA * kMaxContacts + c] = la;
                    cint[CB * kMaxContacts + c] = lb;
                    cint[CKEY * kMaxContacts + c] = key;
                });
            if (tid == 0) s_int[1] = n;
        }
    } else if (a.contacts) {
        int c0 = a.ccount ? w * kMaxContacts : a.coff[w];
        int n = a.ccount ? a.ccount[w] : a.coff[w + 1] - c0;
        if (n > W.contact_cap) n = W.contact_cap;
        if (n < 0) n = 0;
        if (tid == 0) s_int[1] = n;
        for (int c = tid; c < n; c += NT) {
            kamx_contact ct = a.contacts[c0 + c];
            int la = ct.body_a - W.b0;
            int lb = ct.body_b < 0 ? -1 : ct.body_b - W.b0;
            bool ok = la >= 0 && la < nb && lb < nb;
            for (int k = 0; k < 3; ++k) {
                L.cf(CP + k, c) = ct.point[k];
                L.cf(CN + k, c) = ct.normal[k];
            }
            L.cf(CGAP, c) = ct.gap;
            L.cf(CMU, c) = ct.mu;
            // an invalid body index turns the contact into an inert row pair
            cint[CA * kMaxContacts + c] = ok ? la : 0;
            cint[CB * kMaxContacts + c] = ok ? lb : -1;
            if (!ok) L.cf(CGAP, c) = 1e30f;
            cint[CKEY * kMaxContacts + c] = ct.key;
        }
    } else if (tid < 64) {
        int k = tid;
        bool act = false;
        float pw[3] = {0.f, 0.f, 0.f};
        int lbod = 0;
        float mu = 0.f;
        if (k < W.np) {
            int gp = W.p0 + k;
            lbod = a.pbody[gp];
            float pl[3] = {a.pf[4 * gp], a.pf[4 * gp + 1], a.pf[4 * gp + 2]};
            mu = a.pf[4 * gp + 3];
            // world point in FP64 (its height is the gap, which enters the
            // bias divided by dt), then rounded to FP32
            double qd[4], Rd[9], pld[3] = {pl[0], pl[1], pl[2]}, td[3];
            for (int e = 0; e < 4; ++e) qd[e] = L.qd[(3 + e) * kMaxBodies + lbod];
            rot_of_quat(qd, Rd);
            mv3(Rd, pld, td);
            for (int e = 0; e < 3; ++e) pw[e] = (float)(L.qd[e * kMaxBodies + lbod] + td[e]);
            act = pw[2] < P.contact_margin;
        }
        unsigned long long mask = __ballot(act);
        int slot = __popcll(mask & ((1ull << k) - 1ull));
        if (act && slot < W.contact_cap) {
            for (int e = 0; e < 3; ++e) L.cf(CP + e, slot) = pw[e];
            L.cf(CN + 0, slot) = 0.f;
            L.cf(CN + 1, slot) = 0.f;
            L.cf(CN + 2, slot) = 1.f;
            L.cf(CGAP, slot) = pw[2];
            L.cf(CMU, slot) = mu;
            cint[CA * kMaxContacts + slot] = lbod;
            cint[CB * kMaxContacts + slot] = -1;
            cint[CKEY * kMaxContacts + slot] = k;
        }
        if (k == 0) {
            int n = __popcll(mask);
            s_int[1] = n < W.contact_cap ? n : W.contact_cap;
        }
    }
    __syncthreads();
    const RowCounts rows(W, L);
    const int nc = rows.nc, row_c0 = rows.c0, m = rows.m;
    const int row_lim0 = 5 * nj;
    const int row_drv0 = 5 * nj + W.nlim;

    // ---- constraint rows
    for (int j = tid; j < nj; j += NT) {
        int gj = W.j0 + j;
        int type = a.jint[4 * gj], la = a.jint[4 * gj + 1], lb = a.jint[4 * gj + 2], fl = a.jint[4 * gj + 3];
        const float *jf = a.jf + kJointFloats * gj;
        JointGeo g;
        joint_geo(L, jf, la, lb, g);
        joint_rows(L, type, g, la, lb, 5 * j, P);
        if (fl & kJointLimited) {
            int rank = 0;
            const int *tf = reinterpret_cast<const int *>(L.j) + JTF * kMaxJoints;
            for (int k = 0; k < j; ++k) rank += (tf[k] >> 4) & kJointLimited ? 1 : 0;
            float Ja[6], Jb[6];
            double c = joint_coord(type, g, Ja, Jb);
            double lo = jf[14], hi = jf[15];
            bool use_lo;
            if (isnan(hi)) use_lo = true;
            else if (isnan(lo)) use_lo = false;
            else use_lo = (c - lo) <= (hi - c);
            float sg = use_lo ? 1.f : -1.f;
            float gval = (float)(use_lo ? c - lo : hi - c);
            for (int k = 0; k < 6; ++k) {
                Ja[k] *= sg;
                Jb[k] *= sg;
            }
            put_row(L, row_lim0 + rank, Ja, la, Jb, lb, gval, kRowLimit, 0.f, P);
        }
        if (fl & kJointDriven) {
            // drive row (Sec. 3 implicit PD, armature, damping; Eq. 2 R, v*):
            // along the coordinate c the impulse over the step is
            // dt [kp (ref - c - h c'+) - (kd + d) c'+ - I_a (c'+ - c'-) / dt],
            // i.e. J_c u+ + R lambda + v* = 0 with K = kp h + kd + d + I_a / dt,
            // R = 1 / (dt K), v* = -(kp (ref - c) + I_a c'- / dt) / K
            int rank = 0;
            const int *tf = reinterpret_cast<const int *>(L.j) + JTF * kMaxJoints;
            for (int k = 0; k < j; ++k) rank += (tf[k] >> 4) & kJointDriven ? 1 : 0;
            float Ja[6], Jb[6];
            const double c = joint_coord(type, g, Ja, Jb);
            float rate = 0.f;
            for (int k = 0; k < 6; ++k) rate += Ja[k] * L.bf(BU + k, la);
            if (lb >= 0)
                for (int k = 0; k < 6; ++k) rate += Jb[k] * L.bf(BU + k, lb);
            const float h = P.integrator == KAMX_MOREAU_JEAN ? 0.5f * P.dt : P.dt;
            const float kp = jf[16], kd = jf[17], ref = jf[18], damp = jf[19], arm = jf[20];
            const float K = kp * h + kd + damp + arm / P.dt;
            const int r = row_drv0 + rank;
            put_row(L, r, Ja, la, Jb, lb, 0.f, kRowBilateral, 0.f, P);
            L.rf(RBIAS, r) = -(float)((double)kp * ((double)ref - c) + (double)arm * (double)rate / (double)P.dt) / K;
            L.rf(RREG, r) = 1.f / (P.dt * K);
        }
    }
    for (int c = tid; c < nc; c += NT) {
        float p[3], n[3], t1[3], t2[3];
        for (int k = 0; k < 3; ++k) {
            p[k] = L.cf(CP + k, c);
            n[k] = L.cf(CN + k, c);
        }
        tangents(n, t1, t2);
        const float *dirs[3] = {n, t1, t2};
        int la = cint[CA * kMaxContacts + c], lb = cint[CB * kMaxContacts + c];
        float arm_a[3], arm_b[3] = {0.f, 0.f, 0.f};
        for (int k = 0; k < 3; ++k) {
            arm_a[k] = p[k] - L.bf(BQ + k, la);
            if (lb >= 0) arm_b[k] = p[k] - L.bf(BQ + k, lb);
        }
        for (int e = 0; e < 3; ++e) {
            float Ja[6], Jb[6], cc[3];
            cross(arm_a, dirs[e], cc);
            for (int k = 0; k < 3; ++k) {
                Ja[k] = dirs[e][k];
                Ja[3 + k] = cc[k];
            }
            cross(arm_b, dirs[e], cc);
            for (int k = 0; k < 3; ++k) {
                Jb[k] = -dirs[e][k];
                Jb[3 + k] = -cc[k];
            }
            put_row(L, row_c0 + 3 * c + e, Ja, la, Jb, lb, e == 0 ? L.cf(CGAP, c) : 0.f,
                    e == 0 ? kRowNormal : kRowTangent, L.cf(CMU, c), P);
        }
    }
    __syncthreads();

    // ---- body -> row incidence lists (CSR, rows in increasing order), one
    //      wave per body at a time, compacted with ballots
    {
        constexpr int NWAVE = NT / 64;
        const int lane = tid & 63, wave = tid >> 6;
        for (int b = wave; b < nb; b += NWAVE) {
            int cnt = 0;
            for (int r0 = 0; r0 < m; r0 += 64) {
                int r = r0 + lane;
                bool f = r < m && (L.ri(RIA, r) == b || L.ri(RIB, r) == b);
                cnt += __popcll(__ballot(f));
            }
            if (lane == 0) L.inc_off[b + 1] = cnt;
        }
        __syncthreads();
        if (tid == 0) {
            L.inc_off[0] = 0;
            for (int b = 0; b < nb; ++b) L.inc_off[b + 1] += L.inc_off[b];
        }
        __syncthreads();
        for (int b = wave; b < nb; b += NWAVE) {
            int base = L.inc_off[b];
            for (int r0 = 0; r0 < m; r0 += 64) {
                int r = r0 + lane;
                int side = -1;
                if (r < m) {
                    if (L.ri(RIA, r) == b) side = 0;
                    else if (L.ri(RIB, r) == b) side = 1;
                }
                unsigned long long msk = __ballot(side >= 0);
                if (side >= 0) L.inc_list[base + __popcll(msk & ((1ull << lane) - 1ull))] = (r << 1) | side;
                base += __popcll(msk);
            }
        }
        __syncthreads();
    }
    static_assert(kMaxBodies <= NT, "one thread per body");
    body_angular_minv<NT>(L, nb);

    // ---- W = M^-1 J^T for both sides of every row (in the vector region)
    float *Wv = L.v;  // [12][MC]
    for (int r = tid; r < m; r += NT) {
        for (int s = 0; s < 2; ++s) {
            int b = L.ri(s ? RIB : RIA, r);
            float in[6], out[6];
            for (int k = 0; k < 6; ++k) in[k] = L.rf(RJ + 6 * s + k, r);
            if (b >= 0) apply_minv(L, b, in, out);
            else
                for (int k = 0; k < 6; ++k) out[k] = 0.f;
            for (int k = 0; k < 6; ++k) Wv[(6 * s + k) * MC + r] = out[k];
        }
    }
    __syncthreads();

    if (a.phase_clk && tid == 0) a.phase_clk[16 * w + 1] = wall_clock64();
    // ---- Jacobi scales (Sec. 4.1) from the diagonal D_ii = J_i . W_i: per
    //      row for bilateral and limit rows, one scalar per contact block
    const int i = tid;
    float *vp = L.vec(VP), *vrho = L.vec(VRHO), *vvt = L.vec(VVT);
    float *tdiag = L.vec(VCOL), *tp = L.vec(VDX);  // free fields above W
    const int kind_row = i < m ? L.ri(RKIND, i) : -1;
    if (i < m) {
        float dsum = L.rf(RREG, i);  // D_ii = J_i M^-1 J_i^T + R_ii
        for (int k = 0; k < 12; ++k) dsum += L.rf(RJ + k, i) * Wv[k * MC + i];
        tdiag[i] = dsum;
    }
    __syncthreads();
    if (i < m) {
        if (kind_row == kRowNormal) {
            float t = (tdiag[i] + tdiag[i + 1] + tdiag[i + 2]) * (1.f / 3.f);
            float sc = (P.precond && t > 0.f) ? 1.f / sqrtf(t) : 1.f;
            tp[i] = tp[i + 1] = tp[i + 2] = sc;
        } else if (kind_row != kRowTangent) {
            float t = tdiag[i];
            tp[i] = (P.precond && t > 0.f) ? 1.f / sqrtf(t) : 1.f;
        }
    }
    __syncthreads();
    const float pi_reg = i < m ? tp[i] : 1.f;

    // ---- D~ = P J M^-1 J^T P + diag(eta + rho), packed lower triangle (rows
    //      padded to 4 floats).  Zero-fill, then every nonzero pair (i >= j)
    //      is formed once, by the first body the two rows share: the pairs of
    //      each body's incidence list are spread evenly over the threads.
    {
        const int Mp = (m + 15) & ~15;
        const int n4 = tri_row_offset(Mp) >> 2;
        for (int k = tid; k < n4; k += NT) reinterpret_cast<float4 *>(A)[k] = make_float4(0.f, 0.f, 0.f, 0.f);
        int *toff = reinterpret_cast<int *>(L.red);  // [nb + 1] pair-task offsets (red/wb free here)
        if (tid == 0) {
            toff[0] = 0;
            for (int b = 0; b < nb; ++b) {
                int kb = L.inc_off[b + 1] - L.inc_off[b];
                toff[b + 1] = toff[b] + kb * (kb + 1) / 2;
            }
        }
        __syncthreads();
        if (i >= m && i < Mp) A[tri_row_offset(i) + i] = 1.f;  // identity rows up to a multiple of 16
        const int ntask = toff[nb];
        for (int t = tid; t < ntask; t += NT) {
            int lo = 0, hi = nb - 1;  // body b with toff[b] <= t < toff[b+1]
            while (lo < hi) {
                int mid = (lo + hi + 1) >> 1;
                if (toff[mid] <= t) lo = mid;
                else hi = mid - 1;
            }
            const int b = lo;
            const int loc = t - toff[b];
            int u = (int)((sqrtf(8.f * (float)loc + 1.f) - 1.f) * 0.5f);
            while ((u + 1) * (u + 2) / 2 <= loc) ++u;
            while (u * (u + 1) / 2 > loc) --u;
            const int v = loc - u * (u + 1) / 2;
            const int ri_ = L.inc_list[L.inc_off[b] + u] >> 1;
            const int rj_ = L.inc_list[L.inc_off[b] + v] >> 1;
            const int ia = L.ri(RIA, ri_), ib = L.ri(RIB, ri_), ja = L.ri(RIA, rj_), jb = L.ri(RIB, rj_);
            int first = 1 << 30;
            if (ia == ja || ia == jb) first = ia;
            if (ib >= 0 && (ib == ja || ib == jb) && ib < first) first = ib;
            if (first != b) continue;
            float acc = 0.f;
            if (ia == ja)
                for (int k = 0; k < 6; ++k) acc += L.rf(RJ + k, ri_) * Wv[k * MC + rj_];
            if (ia == jb)
                for (int k = 0; k < 6; ++k) acc += L.rf(RJ + k, ri_) * Wv[(6 + k) * MC + rj_];
            if (ib >= 0 && ib == ja)
                for (int k = 0; k < 6; ++k) acc += L.rf(RJ + 6 + k, ri_) * Wv[k * MC + rj_];
            if (ib >= 0 && ib == jb)
                for (int k = 0; k < 6; ++k) acc += L.rf(RJ + 6 + k, ri_) * Wv[(6 + k) * MC + rj_];
            if (ri_ == rj_) acc += L.rf(RREG, ri_);  // drive rows: D = J M^-1 J^T + R
            acc *= tp[ri_] * tp[rj_];
            if (ri_ == rj_) {
                const int kd = L.ri(RKIND, ri_);
                acc += P.eta + (kd == kRowBilateral ? P.rho_bil : P.rho_c);
            }
            A[tri_row_offset(ri_) + rj_] = acc;
        }
        __syncthreads();
    }
    // the vector region held W and the scales until now: clear it (pads must
    // read as 0), then store P, rho and v~_f = P (J u_f + v*)
    for (int k = tid; k < vec_floats(MC); k += NT) L.v[k] = 0.f;
    for (int k = tid; k < t_floats(MC); k += NT) L.t[k] = 0.f;
    __syncthreads();
    if (i < m) {
        vp[i] = pi_reg;
        vrho[i] = kind_row == kRowBilateral ? P.rho_bil : P.rho_c;
        float v = L.rf(RBIAS, i);
        int ia = L.ri(RIA, i), ib = L.ri(RIB, i);
        for (int k = 0; k < 6; ++k) v += L.rf(RJ + k, i) * L.bf(BUF + k, ia);
        if (ib >= 0)
            for (int k = 0; k < 6; ++k) v += L.rf(RJ + 6 + k, i) * L.bf(BUF + k, ib);
        vvt[i] = pi_reg * v;
    }
    __syncthreads();

    if (a.phase_clk && tid == 0) a.phase_clk[16 * w + 2] = wall_clock64();
    // ---- warm start (Alg. 1 step 2; Sec. 4.1): y = x = Pi_K(lambda_ws / p),
    //      z = v~(y) + Gamma(v~(y)) on unilateral rows, 0 on bilateral rows
    float *vx = L.vec(VX), *vyh = L.vec(VYH), *vzh = L.vec(VZH), *vyp = L.vec(VYP), *vzp = L.vec(VZP);
    float *vws = L.vec(VWS), *vaux = L.vec(VAUX);
    float *vrinv = L.vec(VCOL), *vdx = L.vec(VDX);  // vrinv: 1/rho per row inside the iteration loop
    const int wmode = reset ? KAMX_WARM_COLD : P.warmstart;
    const int kind_i = i < m ? L.ri(RKIND, i) : -1;
    const bool owner = i < m && kind_i != kRowTangent;
    const int blk = kind_i == kRowNormal ? 3 : 1;
    if (wmode != KAMX_WARM_COLD) {
        if (i < m) {
            float lw = 0.f;
            if (wmode == KAMX_WARM_EXTERNAL) {
                lw = a.lambda_ext[W.row_base + i];
            } else if (wmode == KAMX_WARM_LEARNED) {
                // network output by slot: joint, limit and drive rows in
                // order, then three slots per contact slot (contact_slot)
                const float *ws = a.ws_slots + (long)w * a.mlp.n_out;
                if (i < row_c0) {
                    lw = ws[i];
                } else {
                    int c = (i - row_c0) / 3, e = (i - row_c0) % 3;
                    int key = cint[CKEY * kMaxContacts + c];
                    int sl = key >= 0 ? contact_slot(key) : -1;
                    lw = sl >= 0 && sl < a.n_contact_slots ? ws[row_c0 + 3 * sl + e] : 0.f;
                }
            } else if (i < row_c0) {
                lw = a.lambda[W.row_base + i];
            } else {
                // previous-step cache matched by contact key
                int c = (i - row_c0) / 3, e = (i - row_c0) % 3;
                int key = cint[CKEY * kMaxContacts + c];
                int nprev = a.ncontacts_out[w];
                for (int k = 0; k < nprev && k < kMaxContacts; ++k)
                    if (a.keys[w * kMaxContacts + k] == key) {
                        lw = a.lambda[W.row_base + row_c0 + 3 * k + e];
                        break;
                    }
            }
            vws[i] = isfinite(lw) ? lw / vp[i] : 0.f;
        }
        __syncthreads();
        if (owner) {
            if (kind_i == kRowNormal) {
                float o0, o1, o2;
                proj_cone(L.rf(RMU, i), vws[i], vws[i + 1], vws[i + 2], o0, o1, o2);
                vyp[i] = o0;
                vyp[i + 1] = o1;
                vyp[i + 2] = o2;
            } else if (kind_i == kRowLimit) {
                vyp[i] = fmaxf(vws[i], 0.f);
            } else {
                vyp[i] = vws[i];
            }
        }
        __syncthreads();
        delassus_apply<NT>(L, m, nb, vp, vyp, vdx);  // D~ y0 (x0 = y0)
        if (owner) {
            float v0 = vdx[i] + vvt[i];
            if (kind_i == kRowNormal) {
                float v1 = vdx[i + 1] + vvt[i + 1], v2 = vdx[i + 2] + vvt[i + 2];
                vzp[i] = v0 + L.rf(RMU, i) * sqrtf(v1 * v1 + v2 * v2);
                vzp[i + 1] = v1;
                vzp[i + 2] = v2;
            } else if (kind_i == kRowLimit) {
                vzp[i] = v0;
            } else {
                vzp[i] = 0.f;
            }
            _Pragma("unroll") for (int e = 0; e < 3; ++e) if (e < blk) {
                vx[i + e] = vyp[i + e];
                vyh[i + e] = vyp[i + e];
                vzh[i + e] = vzp[i + e];
            }
        }
        __syncthreads();
    }

    if (a.phase_clk && tid == 0) a.phase_clk[16 * w + 3] = wall_clock64();
    const int factor_fail = uniform(factor_invert<MC, NT>(m));
    // (the inverse comes with the factor: both stamps)
    if (a.phase_clk && tid == 0) a.phase_clk[16 * w + 4] = a.phase_clk[16 * w + 5] = wall_clock64();
    if (i < m) vrinv[i] = 1.f / vrho[i];  // rho is fixed for the solve: divide once
    if (factor_fail) {
        if (i < m) vyp[i] = 0.f;
    } else if (wmode == KAMX_WARM_COLD && i < m) {
        vx[i] = vyh[i] = vzh[i] = vyp[i] = vzp[i] = vdx[i] = 0.f;
    }
    if (m == 0) {
        bool converged;
        const int it = iterations_without_rows<NT>(a, w, converged);
        if (tid == 0) {
            s_int[4] = it;
            s_int[5] = converged ? kSolveConverged : 0;
            s_int[6] = s_int[7] = s_int[8] = 0;  // r_p, r_d, r_c
        }
    }
    __syncthreads();
    return m == 0 ? kStepNoRows : (factor_fail ? kStepFailed : kStepSolve);
}

// The solve (Alg. 1 steps 3-10), in passes: a pass ends when the solve exits or when the
// adaptive penalty changes rho, whose refactorization then runs outside the iteration
// loop.  Returns KAMX_WORLD_FACTOR_FAIL if that fails, else 0.
template <int MC, int NT>
__device__ __forceinline__ int step_solve(KernelArgs &a) {
    const int tid = threadIdx.x;
    const int w = uniform(a.bucket_worlds[blockIdx.x]);
    const WorldInfo W = uniform_world(a.worlds + w);
    const Lds L = lds_views<MC>();
    const RowCounts rows(W, L);
    int it = 1;
    for (;;) {
        const int adapt = solve_pass<MC, NT>(a, w, rows.m, W.nb, rows.nc, rows.c0, W.nlim, it);
        if (!adapt) return 0;
        it = uniform(L.s_int[4]);
        // the limit and contact rows' penalty changes by the factor; D~ +
        // diag(eta + rho) is rebuilt, refactored and inverted, and the
        // acceleration restarts at the current (y, z), which the owners have
        // written as the extrapolated iterates
        const float f = adapt == 1 ? 1.f / a.p.adapt_factor : a.p.adapt_factor;
        float *vrho = L.vec(VRHO), *vrinv = L.vec(VCOL);
        __syncthreads();
        for (int r = tid; r < rows.m; r += NT)
            if (L.ri(RKIND, r) != kRowBilateral) {
                vrho[r] *= f;
                vrinv[r] = 1.f / vrho[r];
            }
        __syncthreads();
        reassemble<MC, NT>(rows.m, W.nb, a.p.eta);
        if (uniform(factor_invert<MC, NT>(rows.m))) return KAMX_WORLD_FACTOR_FAIL;
    }
}

// Residual of the returned iterate, outputs, and the velocities and poses it leads to.
// left: what step_begin returned; status: of the solve.
template <int MC, int NT>
__device__ __attribute__((noinline)) void step_end(KernelArgs *args, int k, int left, int status) {
    const int tid = threadIdx.x, i = tid;
    KernelArgs &a = *uniform_args(args);
    k = uniform(k);
    const bool factor_fail = uniform(left) == kStepFailed;
    status = uniform(status);
    const int w = uniform(a.bucket_worlds[blockIdx.x]);
    const WorldInfo W = uniform_world(a.worlds + w);
    SolverArgs &P = a.p;
    const Lds L = lds_views<MC>();
    const int *s_int = L.s_int;
    const int nb = W.nb;
    const RowCounts rows(W, L);
    const int nc = rows.nc, m = rows.m;
    const int *cint = reinterpret_cast<const int *>(L.c);
    float *vp = L.vec(VP), *vvt = L.vec(VVT);
    float *vx = L.vec(VX), *vyp = L.vec(VYP), *vzp = L.vec(VZP), *vaux = L.vec(VAUX);
    const int kind_i = i < m ? L.ri(RKIND, i) : -1;
    const bool owner = i < m && kind_i != kRowTangent;
    const int blk = kind_i == kRowNormal ? 3 : 1;
    const float mu_i = i < m ? L.rf(RMU, i) : 0.f;
    const int N = P.fixed_iters > 0 ? P.fixed_iters : P.max_iters;
    int it = 0;
    float rp = 0.f, rd = 0.f, rc = 0.f, rncp = 0.f;
    if (factor_fail) {
        status = KAMX_WORLD_FACTOR_FAIL;
        rp = rd = rc = rncp = NAN;
    } else {
        it = uniform(s_int[4]);
        status |= uniform(s_int[5]) & ~kSolveConverged;
        const bool converged = uniform(s_int[5]) & kSolveConverged;
        rp = __int_as_float(uniform(s_int[6]));
        rd = __int_as_float(uniform(s_int[7]));
        rc = __int_as_float(uniform(s_int[8]));
        if (it > N) it = N;
        if (P.fixed_iters <= 0 && !converged && status == 0) status = KAMX_WORLD_MAXITER;
        __syncthreads();
        // natural-map residual of the NCP at the returned y (Eq. 3)
        delassus_apply<NT>(L, m, nb, vp, vyp, vaux);
        float lncp = 0.f;
        if (owner) {
            float v[3], o[3], y[3], nm[3];
            _Pragma("unroll") for (int e = 0; e < 3; ++e) if (e < blk) {
                v[e] = vaux[i + e] + vvt[i + e];
                y[e] = vyp[i + e];
            }
            float g = kind_i == kRowNormal ? mu_i * sqrtf(v[1] * v[1] + v[2] * v[2]) : 0.f;
            _Pragma("unroll") for (int e = 0; e < 3; ++e) if (e < blk) nm[e] = y[e] - (v[e] + (e == 0 ? g : 0.f));
            if (kind_i == kRowNormal) proj_cone(mu_i, nm[0], nm[1], nm[2], o[0], o[1], o[2]);
            else if (kind_i == kRowLimit) o[0] = fmaxf(nm[0], 0.f);
            else o[0] = nm[0];
            _Pragma("unroll") for (int e = 0; e < 3; ++e) if (e < blk) lncp = fmaxf(lncp, fabsf(y[e] - o[e]));
        }
        float l1 = 0.f, l2 = 0.f, l3 = 0.f;
        reduce4<NT>(lncp, l1, l2, l3, L.red);
        rncp = lncp;
    }
    __syncthreads();

    if (a.phase_clk && tid == 0) a.phase_clk[16 * w + 6] = wall_clock64();
    // ---- outputs: lambda = P y (Alg. 1 step 11), stats, caches
    if (i < W.row_cap) {
        float lam = 0.f;
        if (i < m) lam = vp[i] * vyp[i];
        a.lambda[W.row_base + i] = lam;
        if (i < m) vaux[i] = lam;
        if (a.iterate_out) {
            // the returned iterate in preconditioned units and the scales
            const bool act = i < m;
            *reinterpret_cast<float4 *>(a.iterate_out + 4 * ((long)W.row_base + i)) =
                make_float4(act ? vx[i] : 0.f, act ? vyp[i] : 0.f, act ? vzp[i] : 0.f, act ? vp[i] : 0.f);
        }
    }
    if (tid == 0) {
        a.iters[w] = it;
        a.status[w] = status;
        if (a.iter_log && k < a.iter_log_rows) {
            a.iter_log[(long)k * a.n_worlds + w] = it;
            if (a.row_log) a.row_log[(long)k * a.n_worlds + w] = m;
            if (a.status_log) a.status_log[(long)k * a.n_worlds + w] = status;
        }
        a.rows[w] = m;
        a.resid[4 * w + 0] = rp;
        a.resid[4 * w + 1] = rd;
        a.resid[4 * w + 2] = rc;
        a.resid[4 * w + 3] = rncp;
        a.ncontacts_out[w] = nc;
    }
    for (int c = tid; c < nc; c += NT) {
        kamx_contact ct;
        ct.body_a = cint[CA * kMaxContacts + c] + W.b0;
        int lb = cint[CB * kMaxContacts + c];
        ct.body_b = lb >= 0 ? lb + W.b0 : -1;
        for (int k = 0; k < 3; ++k) {
            ct.point[k] = L.cf(CP + k, c);
            ct.normal[k] = L.cf(CN + k, c);
        }
        ct.gap = L.cf(CGAP, c);
        ct.mu = L.cf(CMU, c);
        ct.key = cint[CKEY * kMaxContacts + c];
        a.contacts_out[w * kMaxContacts + c] = ct;
        a.keys[w * kMaxContacts + c] = ct.key;
    }
    __syncthreads();

    // ---- u+ = u_f + M^-1 J^T lambda (FP64 accumulation over the incident
    //      rows: light links carry large, nearly cancelling impulses), then
    //      poses by the exponential map
    for (int b = tid; b < nb; b += NT) {
        double imp[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        for (int k = L.inc_off[b]; k < L.inc_off[b + 1]; ++k) {
            int e = L.inc_list[k];
            int r = e >> 1, side = e & 1;
            double lam = (double)vp[r] * (double)vyp[r];
            if (factor_fail) lam = 0.0;
            for (int c = 0; c < 6; ++c) imp[c] += (double)L.rf(RJ + 6 * side + c, r) * lam;
        }
        double R[9], t[3], sv[3];
        for (int c = 0; c < 9; ++c) R[c] = L.bf(BR + c, b);
        mtv3(R, imp + 3, t);
        for (int c = 0; c < 3; ++c) t[c] *= (double)L.bf(BII + c, b);
        mv3(R, t, sv);
        double im = L.bf(BIM, b);
        float un[6];
        for (int c = 0; c < 3; ++c) {
            un[c] = (float)((double)L.bf(BUF + c, b) + imp[c] * im);
            un[3 + c] = (float)((double)L.bf(BUF + 3 + c, b) + sv[c]);
        }
        int gb = W.b0 + b;
        for (int k = 0; k < 6; ++k) a.u[6 * gb + k] = un[k];
        // poses over the rest of the step from the rows' configuration: dt
        // (Euler) or dt / 2 from the half-step poses (Moreau-Jean)
        double q[7], ud[6], qn[7];
        for (int k = 0; k < 7; ++k) q[k] = L.qd[k * kMaxBodies + b];
        for (int k = 0; k < 6; ++k) ud[k] = un[k];
        advance_pose(q, ud, (P.integrator == KAMX_MOREAU_JEAN ? 0.5 : 1.0) * (double)P.dt, qn);
        for (int k = 0; k < 7; ++k) a.q[7 * gb + k] = (float)qn[k];
    }
    __syncthreads();
    if (a.phase_clk && tid == 0) a.phase_clk[16 * w + 7] = wall_clock64();
}

// A launch advances every world of the bucket by a.nsteps steps, the
// workgroup keeping its world for all of them: worlds are independent, so a
// slow solve delays only its own world and the hardware's dispatch balances
// whole chains of steps rather than single steps.
// At most 256 VGPRs (two waves per SIMD), which the solve and the factorization use to
// the last ten; a workgroup smaller than 512 threads then leaves room on its
// compute unit for another world's workgroup.
template <int MC, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2))) void step_kernel(StepArgs a) {
    KernelArgs *args = (KernelArgs *)__builtin_amdgcn_kernarg_segment_ptr();
#pragma clang loop unroll(disable)
    for (int k = 0; k < a.nsteps; ++k) {
        const int left = uniform(step_begin<MC, NT>(args, k));
        if (left >= kStepSolve) step_end<MC, NT>(args, k, left, left > kStepSolve ? 0 : step_solve<MC, NT>(*args));
        __syncthreads();
    }
}

// Impulses of the last step in slot layout (joint, limit and drive rows, then three
// slots per contact key; slots of absent contacts are zero), one thread per
// world and slot.
__global__ void impulse_slots_kernel(const WorldInfo *worlds, int n_worlds, int n_contact_slots, const float *lambda,
                                     const int32_t *keys, const int32_t *ncontacts, float *out) {
    const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const WorldInfo W0 = worlds[0];
    const int S = 5 * W0.nj + W0.nlim + W0.ndrv + 3 * n_contact_slots;
    if (idx >= (long)n_worlds * S) return;
    const int w = (int)(idx / S), t = (int)(idx - (long)w * S);
    const WorldInfo W = worlds[w];
    const int rc0 = 5 * W.nj + W.nlim + W.ndrv;
    float v = 0.f;
    if (t < rc0) {
        v = lambda[W.row_base + t];
    } else {
        const int slot = (t - rc0) / 3, e = (t - rc0) % 3;
        const int n = ncontacts[w];
        for (int k = 0; k < n && k < kMaxContacts; ++k)
            if (keys[w * kMaxContacts + k] >= 0 && contact_slot(keys[w * kMaxContacts + k]) == slot) {
                v = lambda[W.row_base + rc0 + 3 * k + e];
                break;
            }
    }
    out[idx] = v;
}

hipError_t launch_impulse_slots(const WorldInfo *worlds, int n_worlds, int n_contact_slots, int n_slots,
                                const float *lambda, const int32_t *keys, const int32_t *ncontacts, float *out,
                                hipStream_t stream) {
    const long total = (long)n_worlds * n_slots;
    if (total <= 0) return hipSuccess;
    hipLaunchKernelGGL(impulse_slots_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream, worlds,
                       n_worlds, n_contact_slots, lambda, keys, ncontacts, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// launch table
// ---------------------------------------------------------------------------

template <int MC, int NT>
static hipError_t launch_mc(const StepArgs &args, int n, hipStream_t stream) {
    static_assert(NT % 64 == 0 && NT >= 64 && NT >= 2 * MC && NT <= 512, "unsupported workgroup size");
    size_t bytes = sizeof(float) * (size_t)smem_floats(MC);
    hipError_t e = allow_lds((const void *)step_kernel<MC, NT>, bytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((step_kernel<MC, NT>), dim3(n), dim3(NT), bytes, stream, args);
    return hipGetLastError();
}

int bucket_capacity(int rows) {
    static const int caps[] = {32, 64, 96, 128, 160, 192, 224};
    for (int c : caps)
        if (rows <= c) return c;
    return -1;
}

// Workgroup sizes each row bucket is built for.  Every iteration pass gives
// each pair of rows (and each pair of column quads) its own threads, so a
// workgroup has at least two threads per row; the larger size runs the
// passes with more threads, the smaller one lets more worlds share a compute
// unit where LDS allows.  The 32-row bucket also runs one wavefront per
// world (its 16x16 tile factorization needs no second wave: the trailing
// update of two tiles is the next diagonal tile, which wave 0 takes).  The first entry is the
// default.  Results do not depend on the choice: every row, tile and
// reduction is evaluated in the same order at every size.
int step_threads_variants(int mc, int out[4]) {
    if (mc == 256 || mc == 512 || mc == 1024) {  // matrix-free: one thread per row
        out[0] = mc;
        return 1;
    }
    for (const BucketSizes &v : kBucketSizes)  // 32 rows: 64 is one wavefront per world
        if (v.mc == mc) {
            for (int k = 0; k < v.n; ++k) out[k] = v.nt[k];
            return v.n;
        }
    return 0;
}

hipError_t launch_sparse_step(const StepArgs &args, int nt, int n, hipStream_t stream);
size_t sparse_smem_bytes(int nt);

hipError_t launch_step(const StepArgs &args, int mc, int nt, int n, hipStream_t stream) {
    if (mc > kMaxRows) return launch_sparse_step(args, nt, n, stream);  // matrix-free row classes
    switch (mc * 1024 + nt) {
    case 32 * 1024 + 64: return launch_mc<32, 64>(args, n, stream);
    case 32 * 1024 + 128: return launch_mc<32, 128>(args, n, stream);
    case 32 * 1024 + 256: return launch_mc<32, 256>(args, n, stream);
    case 64 * 1024 + 128: return launch_mc<64, 128>(args, n, stream);
    case 64 * 1024 + 256: return launch_mc<64, 256>(args, n, stream);
    case 96 * 1024 + 256: return launch_mc<96, 256>(args, n, stream);
    case 96 * 1024 + 512: return launch_mc<96, 512>(args, n, stream);
    case 128 * 1024 + 256: return launch_mc<128, 256>(args, n, stream);
    case 128 * 1024 + 512: return launch_mc<128, 512>(args, n, stream);
    case 160 * 1024 + 384: return launch_mc<160, 384>(args, n, stream);
    case 160 * 1024 + 512: return launch_mc<160, 512>(args, n, stream);
    case 192 * 1024 + 384: return launch_mc<192, 384>(args, n, stream);
    case 192 * 1024 + 512: return launch_mc<192, 512>(args, n, stream);
    case 224 * 1024 + 512: return launch_mc<224, 512>(args, n, stream);
    default: return hipErrorInvalidValue;
    }
}

size_t step_smem_bytes(int mc) { return mc > kMaxRows ? sparse_smem_bytes(mc) : sizeof(float) * (size_t)smem_floats(mc); }

// whether the step kernel of a row bucket can generate box-bin contacts
// itself (the candidates must fit in the LDS of its Delassus triangle)
bool step_generates_box_contacts(int mc) {
    return mc <= kMaxRows && sizeof(float) * (size_t)tri_row_offset(mc) >= sizeof(BoxLds);
}

}  // namespace kamx
