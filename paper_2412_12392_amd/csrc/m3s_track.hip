// gfx950 kernels of the tracking pose solve and of the canonical pointmap
// fusion that follows it (MASt3R-SLAM, Sec. 3.3).
//
// Robustly weighted Gauss-Newton, the weights recomputed every iteration
// (Eq. gauss_newton), for the Sim(3) pose T_kf that maps frame points X^f_f into the
// keyframe, over the matches of the keyframe's pixels found by the matcher.
// One launch per iteration:
//
//   step    every workgroup first sums the previous iteration's partials in
//           fp64 in a fixed order, solves the 7x7 system by Cholesky and
//           applies T <- Exp(tau) o T (Eq. 1, left plus on Sim(3)) in fp64:
//           the same arithmetic in every workgroup, so every workgroup holds
//           the same new pose, and workgroup 0 records it.  Then one lane per
//           match n: x = T Xf[m] with m = idx[n]; ray residual psi(x) -
//           psi(Xk[n]) (Eq. track_ray) and distance residual |x| - |Xk[n]|
//           (the small-weight distance term); Jacobians w.r.t. a left
//           perturbation (Supp. A); weights q / sigma^2 (match confidence q =
//           sqrt(Qf[m] Qk[n]) gated at q_min, Sec. 3.3) times the Huber weight
//           of the whitened block norm; one fp32 row of the moments that give
//           J^T W J, J^T W r, robust cost and count per workgroup.
//   final   one workgroup: the last partials summed (cost and count at the
//           final pose), the fp32 pose and the statistics written.
//
// The partials and the fp64 pose are double-buffered by iteration parity, so
// a launch reads what the previous launch wrote and no workgroup overwrites
// what another still reads; kernel boundaries order every hand-off (no
// device-scope fence: on this part a device-scope release writes back the
// XCD's L2).  Launches are stream-ordered with no host synchronisation, so
// the whole solve can be captured into a graph.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "m3s_internal.h"
#include "m3s_sim3.h"

namespace m3s {

namespace {

constexpr int kThreads = 256;
constexpr int kVals = kPoseVals;
constexpr int kMaxBlocks = 2048;

// Workspace layout (bytes): poses and statistics, then the partials.
constexpr size_t kOffT = 0;         // double[2][12]: pose by iteration parity
constexpr size_t kOffStat = 192;    // double[2][2]: solved iterations and last step norm by iteration parity
constexpr size_t kOffPart = 256;    // float[2][nblocks * kMomentStride]: partials by iteration parity

struct TrackArgs {
    int N;
    const float* Xk;
    const float* Xf;
    const int32_t* idx;
    const uint8_t* valid;
    const float* Qf;
    const float* Qk;
    ConfGate gate;
    RobustWeights rw;
    double* T64;            // [2][12]
    double* stat;           // [2][2]
    float* partials;        // [2][nb * kMomentStride]
    int nb;
    float* T;               // in: the initial pose (read by iteration 0), out: the final one
    float* info;
};

// Solve H tau = -g (7x7 SPD) and apply T <- Exp(tau) o T.  Returns false
// (pose unchanged) when H is not positive definite.
__device__ bool solve_and_update(const double* sum, double* T, double* step_norm) {
    // Cholesky by rows; each pivot's reciprocal root serves its column and both
    // substitutions.
    double L[7][7], inv[7];
    for (int r = 0; r < 7; ++r)
        for (int c = 0; c < 7; ++c) L[r][c] = 0.0;
    for (int r = 0; r < 7; ++r) {
        for (int c = 0; c <= r; ++c) {
            double s = sum[upper_index(c, r)];
            for (int q = 0; q < c; ++q) s -= L[r][q] * L[c][q];
            if (r == c) {
                if (!(s > 0.0) || !isfinite(s)) return false;
                // 1/sqrt(s): hardware estimate and two Newton steps (no fp64
                // division or square root in the chain).
                double is = __builtin_amdgcn_rsq(s);
                is = is * fma(-0.5 * s * is, is, 1.5);
                is = is * fma(-0.5 * s * is, is, 1.5);
                L[r][r] = s * is;
                inv[r] = is;
            } else {
                L[r][c] = s * inv[c];
            }
        }
    }
    double y[7], tau[7];
    for (int r = 0; r < 7; ++r) {
        double s = -sum[28 + r];
        for (int q = 0; q < r; ++q) s -= L[r][q] * y[q];
        y[r] = s * inv[r];
    }
    for (int r = 6; r >= 0; --r) {
        double s = y[r];
        for (int q = r + 1; q < 7; ++q) s -= L[q][r] * tau[q];
        tau[r] = s * inv[r];
    }
    double E[12], Tn[12];
    sim3_exp(tau, E);
    for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 4; ++c)
            Tn[4 * r + c] = E[4 * r] * T[c] + E[4 * r + 1] * T[4 + c] + E[4 * r + 2] * T[8 + c] +
                            (c == 3 ? E[4 * r + 3] : 0.0);
    for (int j = 0; j < 12; ++j) T[j] = Tn[j];
    double tn = 0.0;
    for (int j = 0; j < 7; ++j) tn += tau[j] * tau[j];
    *step_norm = sqrt(tn);
    return true;
}

// The neighbouring matches of a lane (pixels n0 .. n0 + PER - 1), as loaded.
template <int PER>
struct MatchGroup {
    bool ok[PER];
    float qf[PER], qk[PER], xf[PER][3], xk[PER][3];
};

template <int PER>
__device__ __forceinline__ void load_group(const TrackArgs& A, int n0, MatchGroup<PER>& M) {
    static_assert(PER == 1 || PER == 4, "single loads, or vector loads of 4 pixels");
    int mm[PER];
    bool whole = false;
    if constexpr (PER == 4) whole = n0 + PER <= A.N;
    if (whole) {
        const float* x = A.Xk + 3 * (long)n0;
        float xs[12];
        const uint32_t v = *reinterpret_cast<const u32_any*>(A.valid + n0);
        const i4_any i = *reinterpret_cast<const i4_any*>(A.idx + n0);
        const f4_any q = *reinterpret_cast<const f4_any*>(A.Qk + n0);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const f4_any t = reinterpret_cast<const f4_any*>(x)[k];
#pragma unroll
            for (int j = 0; j < 4; ++j) xs[4 * k + j] = t[j];
        }
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            mm[u] = i[u];
            M.qk[u] = q[u];
            M.ok[u] = ((v >> (8 * u)) & 0xffu) != 0u;
#pragma unroll
            for (int j = 0; j < 3; ++j) M.xk[u][j] = xs[3 * u + j];
        }
    } else {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const bool in = n0 + u < A.N;
            const long n = in ? n0 + u : 0;
            mm[u] = A.idx[n];
            M.ok[u] = in && A.valid[n] != 0;
            M.qk[u] = A.Qk[n];
#pragma unroll
            for (int j = 0; j < 3; ++j) M.xk[u][j] = A.Xk[3 * n + j];
        }
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        M.ok[u] = M.ok[u] && (uint32_t)mm[u] < (uint32_t)A.N;
        const long m = M.ok[u] ? mm[u] : 0;
        M.qf[u] = A.Qf[m];
#pragma unroll
        for (int j = 0; j < 3; ++j) M.xf[u][j] = A.Xf[3 * m + j];
    }
}

// Normal equations of the matches of this workgroup at the current pose: one
// fp32 row of moments per workgroup.  A step is bound by latency: the sum and
// the solve of the previous system are a serial chain (1.7 and 1.8 us by clock
// stamps), the matches' reads another (flag and index, then the points they
// name), and the arithmetic of a lane's matches a third.  The reads do not
// depend on the solve, so each lane's first matches (all of them up to 2048
// workgroups) are read before it; the solve has no fp64 division, root or
// library call in its usual case.  A step of 320 x 240: 9.3 us before, 7.0 now.
template <int NT, int PER, bool COST>
__global__ void __launch_bounds__(NT) track_step_kernel(TrackArgs A, int it) {
    __shared__ float red[NT / 64][kMomentStride];
    __shared__ double sum[kVals];
    __shared__ SumLds<NT> part;
    __shared__ double Tn[12];
    constexpr int kStep = NT * PER;
    int n0 = blockIdx.x * kStep + PER * threadIdx.x;
    MatchGroup<PER> M;
    load_group(A, n0, M);
    // Workgroup 0 records the iteration's pose and statistics, after its
    // partials are on their way.
    double Tl[12], solved = 0.0, step = 0.0;
    if (it > 0) {
        // Iteration it - 1's system: the same fixed-order sum and solve in
        // every workgroup, from the pose of the previous parity buffer.
        const int prev = (it + 1) & 1;
        sum_partials<NT>(A.partials + (size_t)prev * A.nb * kMomentStride, A.nb, part, sum);
        if (threadIdx.x == 0) {
            for (int j = 0; j < 12; ++j) Tl[j] = A.T64[12 * prev + j];
            solved = A.stat[2 * prev];
            step = A.stat[2 * prev + 1];
            if (solve_and_update(sum, Tl, &step)) solved += 1.0;
        }
    } else if (threadIdx.x == 0) {
        for (int j = 0; j < 12; ++j) Tl[j] = (double)A.T[j];
    }
    if (threadIdx.x == 0)
        for (int j = 0; j < 12; ++j) Tn[j] = Tl[j];
    __syncthreads();
    float T[12];
#pragma unroll
    for (int i = 0; i < 12; ++i) T[i] = (float)Tn[i];
    float acc[kMoments];
#pragma unroll
    for (int i = 0; i < kMoments; ++i) acc[i] = 0.f;
    for (;;) {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            float q;
            if (M.ok[u] && confidence_gate(M.qf[u], M.qk[u], A.gate, q))
                accumulate_match<COST>(T, M.xf[u][0], M.xf[u][1], M.xf[u][2], M.xk[u][0], M.xk[u][1], M.xk[u][2], q, A.rw, acc);
        }
        n0 += gridDim.x * kStep;
        if (n0 >= A.N) break;
        load_group(A, n0, M);
    }
    block_moments<NT>(acc, red, A.partials + ((size_t)(it & 1) * A.nb + blockIdx.x) * kMomentStride);
    if (blockIdx.x == 0 && threadIdx.x < 12) A.T64[12 * (it & 1) + threadIdx.x] = Tn[threadIdx.x];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        A.stat[2 * (it & 1)] = solved;
        A.stat[2 * (it & 1) + 1] = step;
    }
}

// One workgroup: the last iteration's partials summed (cost and count at the
// final pose), the fp32 pose and the statistics written.
__global__ void __launch_bounds__(kThreads) track_final_kernel(TrackArgs A, int it) {
    __shared__ double sum[kVals];
    __shared__ SumLds<kThreads> part;
    sum_partials<kThreads>(A.partials + (size_t)(it & 1) * A.nb * kMomentStride, A.nb, part, sum);
    if (threadIdx.x != 0) return;
    const double* T = A.T64 + 12 * (it & 1);
    for (int j = 0; j < 12; ++j) A.T[j] = (float)T[j];
    if (A.info) {
        A.info[0] = (float)sum[35];
        A.info[1] = (float)sum[36];
        A.info[2] = (float)A.stat[2 * (it & 1)];
        A.info[3] = (float)A.stat[2 * (it & 1) + 1];
    }
}

// Canonical pointmap update (Sec. 3.3, Eq. 8), per keyframe pixel n:
//   Xc[n] <- (Cc[n] Xc[n] + C[n] (T X[n])) / (Cc[n] + C[n]),  Cc[n] <- Cc[n] + C[n];
// a pixel whose summed confidence is not positive keeps its point.  VEC
// pixels per lane: with VEC = 4 every array is read and written as float4
// (3 per point quad, 1 per confidence quad); VEC = 1 handles any alignment
// and the tail.
__device__ __forceinline__ void fuse_one(const float* T, float& x0, float& x1, float& x2, float& cc, float X0, float X1,
                                         float X2, float c) {
    const float t0 = T[0] * X0 + T[1] * X1 + T[2] * X2 + T[3];
    const float t1 = T[4] * X0 + T[5] * X1 + T[6] * X2 + T[7];
    const float t2 = T[8] * X0 + T[9] * X1 + T[10] * X2 + T[11];
    const float cs = cc + c;
    if (cs > 0.f) {
        const float inv = 1.f / cs;
        x0 = (cc * x0 + c * t0) * inv;
        x1 = (cc * x1 + c * t1) * inv;
        x2 = (cc * x2 + c * t2) * inv;
    }
    cc = cs;
}

template <int VEC>
__global__ void __launch_bounds__(256) fuse_kernel(int N, int first, const float* __restrict__ Tg, float* __restrict__ Xc,
                                                   float* __restrict__ Cc, const float* __restrict__ X,
                                                   const float* __restrict__ C) {
    float T[12];
#pragma unroll
    for (int i = 0; i < 12; ++i) T[i] = Tg[i];
    const long g = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (VEC == 4) {
        const long n0 = first + 4 * g;
        if (n0 + 4 > N) return;
        float4* xc4 = reinterpret_cast<float4*>(Xc + 3 * n0);
        const float4* x4 = reinterpret_cast<const float4*>(X + 3 * n0);
        float4 a = xc4[0], b = xc4[1], d = xc4[2];
        const float4 p = x4[0], q = x4[1], r = x4[2];
        float4 cc = *reinterpret_cast<const float4*>(Cc + n0);
        const float4 c = *reinterpret_cast<const float4*>(C + n0);
        fuse_one(T, a.x, a.y, a.z, cc.x, p.x, p.y, p.z, c.x);
        fuse_one(T, a.w, b.x, b.y, cc.y, p.w, q.x, q.y, c.y);
        fuse_one(T, b.z, b.w, d.x, cc.z, q.z, q.w, r.x, c.z);
        fuse_one(T, d.y, d.z, d.w, cc.w, r.y, r.z, r.w, c.w);
        xc4[0] = a; xc4[1] = b; xc4[2] = d;
        *reinterpret_cast<float4*>(Cc + n0) = cc;
    } else {
        const long n = first + g;
        if (n >= N) return;
        float x0 = Xc[3 * n], x1 = Xc[3 * n + 1], x2 = Xc[3 * n + 2], cc = Cc[n];
        fuse_one(T, x0, x1, x2, cc, X[3 * n], X[3 * n + 1], X[3 * n + 2], C[n]);
        Xc[3 * n] = x0; Xc[3 * n + 1] = x1; Xc[3 * n + 2] = x2;
        Cc[n] = cc;
    }
}

}  // namespace

// Threads and matches per lane of a workgroup: 512 x 1 while that needs at most
// one workgroup per CU (an MI355X has 256), else 256 x 4, since every workgroup
// sums all rows.  10-iteration solve at 320 x 240: 78.6 us with 512 x 1, 86 with
// 256 x 2, 84.8 with 1024 x 1; tracked frame at 512 x 384: 183 us with 256 x 4 or
// 512 x 2, 196 with 512 x 4, 189 with 1024 x 1.
constexpr int kSmallMatches = 256 * 512;

// Calls f with the threads of a workgroup and the matches of a lane.
template <class F>
static auto with_track_shape(int N, F f) {
    return N <= kSmallMatches ? f(std::integral_constant<int, 512>{}, std::integral_constant<int, 1>{})
                              : f(std::integral_constant<int, 256>{}, std::integral_constant<int, 4>{});
}

int track_blocks(int N) {
    const int per = with_track_shape(N, [](auto threads, auto per) { return threads * per; });
    const int nb = N / per + (N % per != 0);
    return nb < 1 ? 1 : (nb > kMaxBlocks ? kMaxBlocks : nb);
}

// Enough for every smaller frame as well (which may have more workgroups), so that
// a workspace kept for a program's largest frame serves them all.
size_t track_workspace_bytes(int N) {
    int nb = track_blocks(N);
    if (N > kSmallMatches && nb < track_blocks(kSmallMatches)) nb = track_blocks(kSmallMatches);
    return kOffPart + 2 * (size_t)nb * kMomentStride * sizeof(float);
}

hipError_t launch_track(int N, const float* Xk, const float* Xf, const int32_t* idx, const uint8_t* valid,
                        const float* Qf, const float* Qk, float q_min, float sigma_ray, float sigma_dist, float huber,
                        int iters, float* T, float* info, void* ws, hipStream_t s) {
    char* w = reinterpret_cast<char*>(ws);
    TrackArgs A;
    A.N = N;
    A.Xk = Xk; A.Xf = Xf; A.idx = idx; A.valid = valid; A.Qf = Qf; A.Qk = Qk;
    A.gate = conf_gate(q_min);
    // An infinite sigma drops its residual from the system and the cost.
    A.rw = robust_weights(sigma_ray, sigma_dist, huber);
    A.T64 = reinterpret_cast<double*>(w + kOffT);
    A.stat = reinterpret_cast<double*>(w + kOffStat);
    A.partials = reinterpret_cast<float*>(w + kOffPart);
    A.T = T;
    A.info = info;
    const int nb = track_blocks(N);
    A.nb = nb;
    for (int it = 0; it <= iters; ++it) {
        timer_begin("track_step", s);
        auto step = [&](auto cost) {
            with_track_shape(N, [&](auto threads, auto per) {
                track_step_kernel<decltype(threads)::value, decltype(per)::value, decltype(cost)::value>
                    <<<nb, decltype(threads)::value, 0, s>>>(A, it);
            });
        };
        // The last launch sums the cost and the count at the final pose.
        if (it == iters) step(std::true_type{});
        else step(std::false_type{});
        timer_end(s);
    }
    timer_begin("track_final", s);
    track_final_kernel<<<1, kThreads, 0, s>>>(A, iters);
    timer_end(s);
    return hipGetLastError();
}

hipError_t launch_fuse(int N, const float* T, float* Xc, float* Cc, const float* X, const float* C, hipStream_t s) {
    auto al16 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
    const bool vec = al16(Xc) && al16(Cc) && al16(X) && al16(C);
    const int quads = vec ? N / 4 : 0;
    const int tail = N - 4 * quads;
    if (quads > 0) {
        timer_begin("fuse", s);
        fuse_kernel<4><<<(quads + 255) / 256, 256, 0, s>>>(N, 0, T, Xc, Cc, X, C);
        timer_end(s);
    }
    if (tail > 0) fuse_kernel<1><<<(tail + 255) / 256, 256, 0, s>>>(N, 4 * quads, T, Xc, Cc, X, C);
    return hipGetLastError();
}

}  // namespace m3s
