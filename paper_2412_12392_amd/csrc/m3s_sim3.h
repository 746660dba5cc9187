// Device helpers shared by the pose solves (MASt3R-SLAM, Sec. 3.3 and 3.5):
// Sim(3) algebra in fp64 and the per-match accumulation of the ray and
// distance normal equations in fp32.
//
// Pose layout: row-major 3x4 [sR | t].  Tangent order tau = (v, omega, sigma),
// matching the point Jacobian [I, -[x]_x, x] of Supp. A; updates are left plus,
// T <- Exp(tau) o T (Eq. 1).
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace m3s {

// Loads of neighbouring pixels: whole vectors at any alignment (gfx950 takes
// 16-byte loads at a float's alignment and 4-byte loads at a byte's).
typedef float f4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef int32_t i4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32_any __attribute__((aligned(1)));

// Number of normal-equation values of a match set: the upper triangle of the 7x7
// J^T W J (28, rows of 7, 6, ..., 1), J^T W r (7), robust cost, match count.
constexpr int kPoseVals = 28 + 7 + 2;
// What the matches are summed into: the 28 of those values that are neither zero
// nor the negative of another (accumulate_match), kept in rows of 32 floats.
constexpr int kMoments = 28;
constexpr int kMomentStride = 32;

__device__ __forceinline__ constexpr int upper_index(int a, int b) { return a * 7 - a * (a - 1) / 2 + (b - a); }

// Weights of the two residual blocks: 1 / sigma^2 (0 drops the residual), and
// the Huber width.
struct RobustWeights {
    float w_ray, w_dist, huber;
};

inline RobustWeights robust_weights(float sigma_ray, float sigma_dist, float huber) {
    RobustWeights w;
    w.w_ray = isinf(sigma_ray) ? 0.f : 1.f / (sigma_ray * sigma_ray);
    w.w_dist = isinf(sigma_dist) ? 0.f : 1.f / (sigma_dist * sigma_dist);
    w.huber = huber;
    return w;
}

// Confidence gate of a match (Sec. 3.3): q = sqrt(Qa Qb) > q_min, decided
// exactly as in fp64 (the product of two fp32 values is exact there).  Outside
// the band [lo, hi] the fp32 product gives the fp64 answer; inside, the fp64 root
// decides, which costs a match about as much as all the rest of it.
//   q_min well inside the normal range: the fp32 product is within 2^-24 of the
//   exact one, and the band is q_min^2 (1 -+ 1e-5).
//   q_min <= 1e-18, also an open gate (zero or negative): a product above 1e-30
//   passes, a negative one has no root; what is left is zero or next to it, and
//   there the fp32 product may have lost its sign or its value.
//   Larger: the product may overflow, and fp64 decides all.
// (With no band for an open gate, 65 edges at 512 x 384 took 995 us, with it 914.)
struct ConfGate {
    double q_min;
    float lo, hi;
};

inline ConfGate conf_gate(float q_min) {
    ConfGate g;
    g.q_min = (double)q_min;
    if (q_min <= 1e-18f) {
        g.lo = 0.f;
        g.hi = 1e-30f;
    } else if (q_min < 1e18f) {
        g.lo = (float)(g.q_min * g.q_min * (1.0 - 1e-5));
        g.hi = (float)(g.q_min * g.q_min * (1.0 + 1e-5));
    } else {
        g.lo = -INFINITY;
        g.hi = INFINITY;
    }
    return g;
}

// Writes the fp32 confidence to q, as good as a rounded root: it scales a match's
// whole share, and the hardware's root alone, whose errors lean to one side, left
// H with a largest error of 6.6e-8 of its diagonal over 196,608 matches, this
// 5.5e-8 (1.5 % of a 512 x 384 solve).
__device__ __forceinline__ bool confidence_gate(float Qa, float Qb, const ConfGate& g, float& q) {
    const float p = Qa * Qb;
    // The reciprocal root and one Newton step (p = +inf has no residual; p = 0 and
    // subnormal products take the fp64 root below).
    const float r = __builtin_amdgcn_rsqf(p), s = p * r;
    q = p < INFINITY ? fmaf(0.5f * r, fmaf(-s, s, p), s) : p;
    if (p > g.hi) return true;
    if (p < g.lo) return false;
    const double e = sqrt((double)Qa * (double)Qb);
    q = (float)e;
    return e > g.q_min;
}

// 1 / |x| and |x| from n2 = |x|^2 (positive, finite, not subnormal): the
// hardware reciprocal root, and one Newton step on n2 / |x| that makes |x| as
// good as a rounded root.
__device__ __forceinline__ void norm_of(float n2, float& id, float& d) {
    id = __builtin_amdgcn_rsqf(n2);
    d = n2 * id;
    d = fmaf(0.5f * id, fmaf(-d, d, n2), d);
}

// One match: x = T X (X the point that moves with the pose), Y the measured
// point, q its confidence.  Ray residual e = psi(x) - psi(Y) and distance
// residual rd = |x| - |Y| (Sec. 3.3); their Jacobians w.r.t. a left
// perturbation of T (Supp. A) are J_ray = [P/d, -[x]_x/d, 0] and
// J_dist = [u^T, 0, d] with d = |x|, u = x/d and the projector P = I - u u^T;
// weights wr = q/sigma_ray^2 and wd = q/sigma_dist^2, each times the Huber
// weight of its whitened block norm |r| sqrt(q)/sigma.  Since P^T P = P,
// P [x]_x = [x]_x and [x]_x^T [x]_x = d^2 P, the weighted normal equations
// have the closed form (ar = wr/d^2)
//   H_vv = ar I + (wd - ar) u u^T   H_vw = -ar [x]_x   H_vs = wd d u
//   H_ww = wr P                     H_ws = 0           H_ss = wd d^2
//   g_v  = wr P e / d + wd rd u     g_w = wr u x e     g_s  = wd rd d
// Each of its entries but the mirrored ones of H_vw is a sum of its own over the
// matches, the diagonals of P from the other two squares (P_00 = u1^2 + u2^2):
//   0-5 H_vv (upper)   6-8 ar x   9-11 H_vs   12-17 H_ww (upper)   18 H_ss
//   19-25 g   26 robust cost   27 count
// (H_ww as the difference of two totals, wr I - wr u u^T, would need two sums
// fewer, but in a view of a few degrees, where u u^T is nearly I for one axis,
// that leaves the roll's entry with 1e-5 of it in error, from 3e-8.)
// A pose solve is bound by vector issue here (its operands come from L2): all 37
// values with correctly rounded roots took about 240 instructions a match and
// 89 us for 65 edges at 512 x 384, this about 150 and 62 us.
// Adds nothing for a point at the origin or non-finite.  A pass sums either the
// system (COST = false: moments 0 .. 25) or the cost and the count (moments 26
// and 27), never both: the solves read the latter at the final pose only.
template <bool COST>
__device__ __forceinline__ void accumulate_match(const float* T, float X0, float X1, float X2, float Y0, float Y1,
                                                 float Y2, float q, const RobustWeights& rw, float* m) {
    const float x0 = fmaf(T[0], X0, fmaf(T[1], X1, fmaf(T[2], X2, T[3])));
    const float x1 = fmaf(T[4], X0, fmaf(T[5], X1, fmaf(T[6], X2, T[7])));
    const float x2 = fmaf(T[8], X0, fmaf(T[9], X1, fmaf(T[10], X2, T[11])));
    const float n2 = fmaf(x0, x0, fmaf(x1, x1, x2 * x2)), ny2 = fmaf(Y0, Y0, fmaf(Y1, Y1, Y2 * Y2));
    if (!(n2 > 0.f && n2 < INFINITY && ny2 > 0.f && ny2 < INFINITY)) return;
    float id, d, idy, dy;
    norm_of(n2, id, d);
    norm_of(ny2, idy, dy);
    id = fmaf(fmaf(-d, id, 1.f), id, id);  // 1 / d to a rounding: it enters H squared
    // The hardware flushes a subnormal square (a norm below 1.1e-19).
    if (__builtin_expect(fminf(n2, ny2) < 1.17549435e-38f, 0)) {
        d = sqrtf(n2);
        dy = sqrtf(ny2);
        id = 1.0f / d;
        idy = 1.0f / dy;
    }
    const float u0 = x0 * id, u1 = x1 * id, u2 = x2 * id;
    const float e0 = fmaf(-Y0, idy, u0), e1 = fmaf(-Y1, idy, u1), e2 = fmaf(-Y2, idy, u2), rd = d - dy;
    // Whitened norms a, Huber weights min(1, width / a), and Huber costs.
    const float qr = q * rw.w_ray, qd = q * rw.w_dist;
    const float a_ray = __builtin_amdgcn_sqrtf(fmaf(e0, e0, fmaf(e1, e1, e2 * e2)) * qr);
    const float a_dist = fabsf(rd) * __builtin_amdgcn_sqrtf(qd);
    if constexpr (COST) {
        // (Branches, since an infinite norm costs +inf at any width, also an infinite one.)
        auto cost = [&](float a) { return a <= rw.huber ? 0.5f * a * a : rw.huber * fmaf(-0.5f, rw.huber, a); };
        m[26] += cost(a_ray) + cost(a_dist);
        m[27] += 1.f;
        return;
    }
    const float wr = qr * fminf(1.f, rw.huber * __builtin_amdgcn_rcpf(a_ray));
    const float wd = qd * fminf(1.f, rw.huber * __builtin_amdgcn_rcpf(a_dist));
    const float wri = wr * id, ar = wri * id, cv = wd - ar, wdd = wd * d, wdr = wd * rd;
    const float s0 = u0 * u0, s1 = u1 * u1, s2 = u2 * u2;
    const float p0 = s1 + s2, p1 = s0 + s2, p2 = s0 + s1;  // diagonal of P
    const float cu0 = cv * u0, cu1 = cv * u1;
    m[0] = fmaf(ar, p0, fmaf(wd, s0, m[0]));
    m[1] = fmaf(cu0, u1, m[1]);
    m[2] = fmaf(cu0, u2, m[2]);
    m[3] = fmaf(ar, p1, fmaf(wd, s1, m[3]));
    m[4] = fmaf(cu1, u2, m[4]);
    m[5] = fmaf(ar, p2, fmaf(wd, s2, m[5]));
    m[6] = fmaf(ar, x0, m[6]);
    m[7] = fmaf(ar, x1, m[7]);
    m[8] = fmaf(ar, x2, m[8]);
    m[9] = fmaf(wdd, u0, m[9]);
    m[10] = fmaf(wdd, u1, m[10]);
    m[11] = fmaf(wdd, u2, m[11]);
    const float wu0 = wr * u0, wu1 = wr * u1, wu2 = wr * u2;
    m[12] = fmaf(wr, p0, m[12]);
    m[13] = fmaf(-wu0, u1, m[13]);
    m[14] = fmaf(-wu0, u2, m[14]);
    m[15] = fmaf(wr, p1, m[15]);
    m[16] = fmaf(-wu1, u2, m[16]);
    m[17] = fmaf(wr, p2, m[17]);
    m[18] = fmaf(wdd, d, m[18]);
    const float ue = fmaf(u0, e0, fmaf(u1, e1, u2 * e2));
    m[19] = fmaf(wri, fmaf(-u0, ue, e0), fmaf(wdr, u0, m[19]));
    m[20] = fmaf(wri, fmaf(-u1, ue, e1), fmaf(wdr, u1, m[20]));
    m[21] = fmaf(wri, fmaf(-u2, ue, e2), fmaf(wdr, u2, m[21]));
    m[22] = fmaf(wu1, e2, fmaf(-wu2, e1, m[22]));
    m[23] = fmaf(wu2, e0, fmaf(-wu0, e2, m[23]));
    m[24] = fmaf(wu0, e1, fmaf(-wu1, e0, m[24]));
    m[25] = fmaf(wdr, d, m[25]);
}

// Value v of the normal equations (kPoseVals) from the summed moments.
__device__ __forceinline__ double pose_value(const double* m, int v) {
    // Per value its moment (or -1 for a zero), and whether it enters negated (H_vw = -ar [x]_x).
    constexpr int8_t kOf[kPoseVals] = {0, 1, 2, -1, 8, 7, 9,  3, 4, 8, -1, 6, 10,  5, 7, 6, -1, 11,
                                       12, 13, 14, -1,  15, 16, -1,  17, -1,  18,
                                       19, 20, 21, 22, 23, 24, 25, 26, 27};
    const bool minus = v == upper_index(0, 5) || v == upper_index(1, 3) || v == upper_index(2, 4);
    const double a = kOf[v] >= 0 ? m[kOf[v]] : 0.0;
    return minus ? -a : a;
}

// Fixed-order fp64 sum of nparts fp32 rows of kMoments values (kMomentStride
// floats each) by a workgroup of NT threads, and the normal equations they
// give: G = NT / 32 groups of 32 threads, thread (g, v) adding value v of the
// rows g, g + G, g + 2G, ... in that order (a group reads whole rows, and
// every group's reads are in flight together); then thread v adds the G group
// sums in group order.  The kPoseVals values land in out (LDS), visible to the
// whole workgroup on return.
template <int NT>
struct SumLds {
    double part[NT];
    double mom[kMomentStride];
};

template <int NT>
__device__ void sum_partials(const float* __restrict__ parts, int nparts, SumLds<NT>& S, double* out) {
    constexpr int G = NT / kMomentStride;
    const int t = threadIdx.x, g = t / kMomentStride, v = t % kMomentStride;
    if (t < NT) {  // threads beyond NT only join the barriers
        double acc = 0.0;
#pragma unroll 8
        for (int b = g; b < nparts; b += G) acc += (double)parts[(size_t)b * kMomentStride + v];
        S.part[t] = acc;
    }
    __syncthreads();
    if (t < kMomentStride) {
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < G; ++k) s += S.part[k * kMomentStride + t];
        S.mom[t] = s;
    }
    __syncthreads();
    if (t < kPoseVals) out[t] = pose_value(S.mom, t);
    __syncthreads();
}

template <int CTRL>
__device__ __forceinline__ float dpp_add(float x) {
    return x + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}

// Sums of a workgroup's moments (m, every lane active) to row[0 .. 32), in a
// fixed order.  Two swaps across the wave's halves and rows leave each of the
// four 16-lane rows with a quarter of the moments, so the sums within a row
// are formed for four moments at once (80 instructions a wave; 37 full
// wave sums took about 400).  red: LDS of NT / 64 rows.
template <int NT>
__device__ __forceinline__ void block_moments(const float* m, float (*red)[kMomentStride], float* __restrict__ row) {
    float h[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const uint32_t a = __builtin_bit_cast(uint32_t, m[i]);
        const uint32_t b = i + 16 < kMoments ? __builtin_bit_cast(uint32_t, m[i + 16]) : 0u;
        const auto s = __builtin_amdgcn_permlane32_swap(a, b, false, false);
        h[i] = __builtin_bit_cast(float, (uint32_t)s[0]) + __builtin_bit_cast(float, (uint32_t)s[1]);
    }
    // h[i]: moment i in the lower half wave, i + 16 in the upper one.
    float r[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const auto s = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, h[i]),
                                                        __builtin_bit_cast(uint32_t, h[i + 8]), false, false);
        r[i] = __builtin_bit_cast(float, (uint32_t)s[0]) + __builtin_bit_cast(float, (uint32_t)s[1]);
    }
    // r[i]: moment i + 8 j in row j of the wave.
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        r[i] = dpp_add<0xB1>(r[i]);   // quad_perm [1,0,3,2]
        r[i] = dpp_add<0x4E>(r[i]);   // quad_perm [2,3,0,1]
        r[i] = dpp_add<0x141>(r[i]);  // row_half_mirror
        r[i] = dpp_add<0x140>(r[i]);  // row_mirror
        if ((lane & 15) == 0) red[wave][i + 8 * (lane >> 4)] = r[i];
    }
    __syncthreads();
    if (threadIdx.x < kMomentStride) {
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < NT / 64; ++w) v += red[w][threadIdx.x];
        row[threadIdx.x] = v;
    }
}

// Scale of a similarity [sR | t]: the cube root of det(sR).
__device__ inline double sim3_scale(const double* T) {
    const double det = T[0] * (T[5] * T[10] - T[6] * T[9]) - T[1] * (T[4] * T[10] - T[6] * T[8]) +
                       T[2] * (T[4] * T[9] - T[5] * T[8]);
    return cbrt(det);
}

// out = T^-1 = [R^T / s | -R^T t / s].
__device__ inline void sim3_inverse(const double* T, double* out) {
    const double s = sim3_scale(T), s2 = s * s;
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) out[4 * i + j] = T[4 * j + i] / s2;
    for (int i = 0; i < 3; ++i)
        out[4 * i + 3] = -(out[4 * i] * T[3] + out[4 * i + 1] * T[7] + out[4 * i + 2] * T[11]);
}

// out = A B (out must not alias A or B).
__device__ inline void sim3_mul(const double* A, const double* B, double* out) {
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 4; ++j)
            out[4 * i + j] = A[4 * i] * B[j] + A[4 * i + 1] * B[4 + j] + A[4 * i + 2] * B[8 + j] +
                             (j == 3 ? A[4 * i + 3] : 0.0);
}

// Ad(T) on (v, omega, sigma): [[sR, [t]_x R, -t], [0, R, 0], [0, 0, 1]], row-major 7x7.
__device__ inline void sim3_adjoint(const double* T, double* A) {
    const double s = sim3_scale(T);
    double R[3][3];
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) R[i][j] = T[4 * i + j] / s;
    const double t[3] = {T[3], T[7], T[11]};
    const double S[3][3] = {{0.0, -t[2], t[1]}, {t[2], 0.0, -t[0]}, {-t[1], t[0], 0.0}};
    for (int k = 0; k < 49; ++k) A[k] = 0.0;
    for (int i = 0; i < 3; ++i) {
        for (int j = 0; j < 3; ++j) {
            A[7 * i + j] = s * R[i][j];
            A[7 * i + 3 + j] = S[i][0] * R[0][j] + S[i][1] * R[1][j] + S[i][2] * R[2][j];
            A[7 * (3 + i) + 3 + j] = R[i][j];
        }
        A[7 * i + 6] = -t[i];
    }
    A[48] = 1.0;
}

// Coefficients of sim3_exp for a small tangent (theta^2 < 2.5e-3, |sigma| <
// 0.05: every Gauss-Newton step but the first ones of a poor start), to fp64
// rounding, without library calls or divisions.  With J_m = int s^m e^{sigma s}
// over [0, 1]: a0 = J_0, a1 = sum (-theta^2)^n J_{2n+1} / (2n+1)! and
// a2 = sum (-theta^2)^n J_{2n+2} / (2n+2)!; J_8 by its series and the others
// downwards by J_{m-1} = (e^sigma - sigma J_m) / m (integration by parts),
// which damps the error.
__device__ inline void sim3_exp_small(double sg, double th2, double& ka, double& kb, double& es, double& a0, double& a1,
                                      double& a2) {
    es = 1.0 / 362880.0;
    es = fma(es, sg, 1.0 / 40320.0);
    es = fma(es, sg, 1.0 / 5040.0);
    es = fma(es, sg, 1.0 / 720.0);
    es = fma(es, sg, 1.0 / 120.0);
    es = fma(es, sg, 1.0 / 24.0);
    es = fma(es, sg, 1.0 / 6.0);
    es = fma(es, sg, 0.5);
    es = fma(es, sg, 1.0);
    es = fma(es, sg, 1.0);
    double J[9];
    // sum sigma^k / (k! (k + 9))
    J[8] = 1.0 / (40320.0 * 17.0);
    J[8] = fma(J[8], sg, 1.0 / (5040.0 * 16.0));
    J[8] = fma(J[8], sg, 1.0 / (720.0 * 15.0));
    J[8] = fma(J[8], sg, 1.0 / (120.0 * 14.0));
    J[8] = fma(J[8], sg, 1.0 / (24.0 * 13.0));
    J[8] = fma(J[8], sg, 1.0 / (6.0 * 12.0));
    J[8] = fma(J[8], sg, 1.0 / (2.0 * 11.0));
    J[8] = fma(J[8], sg, 1.0 / 10.0);
    J[8] = fma(J[8], sg, 1.0 / 9.0);
#pragma unroll
    for (int m = 8; m > 0; --m) J[m - 1] = fma(-sg, J[m], es) * (1.0 / m);
    const double z = -th2;
    ka = fma(z, fma(z, fma(z, fma(z, 1.0 / 362880.0, 1.0 / 5040.0), 1.0 / 120.0), 1.0 / 6.0), 1.0);
    kb = fma(z, fma(z, fma(z, fma(z, 1.0 / 3628800.0, 1.0 / 40320.0), 1.0 / 720.0), 1.0 / 24.0), 0.5);
    a0 = J[0];
    a1 = fma(z, fma(z, fma(z, J[7] * (1.0 / 5040.0), J[5] * (1.0 / 120.0)), J[3] * (1.0 / 6.0)), J[1]);
    a2 = fma(z, fma(z, fma(z, J[8] * (1.0 / 40320.0), J[6] * (1.0 / 720.0)), J[4] * (1.0 / 24.0)), J[2] * 0.5);
}

// Exp of sim(3): tau = (v, omega, sigma) -> [e^sigma R | V v], R by Rodrigues
// and V = a0 I + a1 [omega]_x + a2 [omega]_x^2 with a0 = int e^{sigma s},
// a1 = int e^{sigma s} sin(theta s) / theta and
// a2 = int e^{sigma s} (1 - cos(theta s)) / theta^2 over s in [0, 1]; their
// series near theta = 0 and sigma = 0.
__device__ inline void sim3_exp(const double* tau, double* E) {
    const double sg = tau[6];
    const double w0 = tau[3], w1 = tau[4], w2 = tau[5];
    const double th2 = w0 * w0 + w1 * w1 + w2 * w2;
    const double S[3][3] = {{0.0, -w2, w1}, {w2, 0.0, -w0}, {-w1, w0, 0.0}};
    double S2[3][3];
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) S2[i][j] = S[i][0] * S[0][j] + S[i][1] * S[1][j] + S[i][2] * S[2][j];
    double ka, kb, es, a0, a1, a2;
    if (th2 < 2.5e-3 && fabs(sg) < 0.05) {
        sim3_exp_small(sg, th2, ka, kb, es, a0, a1, a2);
    } else {
        const double th = sqrt(th2);
        double sn, cs;
        sincos(th, &sn, &cs);
        const bool small = th < 1e-4;
        ka = small ? 1.0 - th2 / 6.0 : sn / th;
        kb = small ? 0.5 - th2 / 24.0 : (1.0 - cs) / th2;
        es = exp(sg);
        a0 = sg == 0.0 ? 1.0 : expm1(sg) / sg;
        if (small) {
            // |sigma| is at least 0.05 here.
            const double s2 = sg * sg;
            a1 = (es * (sg - 1.0) + 1.0) / s2;
            a2 = (es * (s2 - 2.0 * sg + 2.0) - 2.0) / (2.0 * s2 * sg);
        } else {
            const double den = sg * sg + th2;
            const double is = (es * (sg * sn - th * cs) + th) / den;
            const double ic = (es * (sg * cs + th * sn) - sg) / den;
            a1 = is / th;
            a2 = (a0 - ic) / th2;
        }
    }
    for (int i = 0; i < 3; ++i) {
        double tv = 0.0;
        for (int j = 0; j < 3; ++j) {
            const double I = i == j ? 1.0 : 0.0;
            E[4 * i + j] = es * (I + ka * S[i][j] + kb * S2[i][j]);
            tv += (I * a0 + a1 * S[i][j] + a2 * S2[i][j]) * tau[j];
        }
        E[4 * i + 3] = tv;
    }
}

}  // namespace m3s
