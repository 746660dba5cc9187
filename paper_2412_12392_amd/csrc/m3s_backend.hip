// gfx950 kernels of the backend optimisation (MASt3R-SLAM, Sec. 3.5).
//
// Gauss-Newton over the world poses T_WC of N keyframes on the global ray
// objective (Eq. backend_ray) plus the small-weight distance term, summed over
// every edge (i, j) and every valid match (n of keyframe j, m = idx[n] of
// keyframe i) with confidence q = sqrt(Q_i[m] Q_j[n]) > q_min.  The residuals
// of an edge depend on the relative pose T_ij = T_WC[i]^-1 T_WC[j] only, and
// the world-pose Jacobians are -J Ad(T_WC[i]^-1) and J Ad(T_WC[i]^-1) (Supp. A,
// relative to global pose), so with A = Ad(T_WC[i]^-1) an edge contributes
//   H_ii += A^T H_e A,  H_jj += A^T H_e A,  H_ij = H_ji^T -= A^T H_e A,
//   g_i  -= A^T g_e,    g_j  += A^T g_e
// where (H_e, g_e) are the edge's 7x7 normal equations w.r.t. a left
// perturbation of T_ij.  Per iteration:
//
//   accum   grid (blocks, edges): every lane sums the relative normal
//           equations of its matches in fp32 (the tracking residuals with
//           x = T_ij X_j[n] transformed and X_i[m] measured); one partial per
//           workgroup.
//   edge    one workgroup per edge: the edge's partials summed in fp64 in a
//           fixed order; A^T H_e A and A^T g_e.
//   solve   one launch.  Usually one workgroup works: the block-sparse Cholesky
//           of the reduced 7(N-1) system (keyframe 0 holds the gauge) in a
//           fill-reducing order, level by level, in LDS (in the workspace when
//           the factor exceeds LDS), with the edges' blocks gathered straight
//           from the edge kernel's output.  For a graph so dense that its
//           factor has no sparsity to use, one workgroup per block row
//           assembles the dense system and the last one to finish factors it:
//           blocked right-looking Cholesky in fp64 with 32 x 32 tiles (the
//           diagonal tile factored one column group per barrier, the panel
//           kept in LDS, the backward substitution blocked).
//           T_WC[k] <- Exp(tau_k) o T_WC[k] (Eq. 1).  A system that is not
//           positive definite, or a step norm below step_tol, ends the loop:
//           later launches of the call return at once.
//
// Kernel boundaries order every hand-off but the dense assembly's, so no other
// workgroup needs a device-scope fence.  A final accumulation at the last poses gives the cost
// and match count.  Launches are stream-ordered with no host synchronisation.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <climits>

#include "m3s.h"
#include "m3s_internal.h"
#include "m3s_sim3.h"

namespace m3s {

namespace {

constexpr int kThreads = 256;
constexpr int kSolveThreads = 512;
constexpr int kVals = kPoseVals;
constexpr int kStride = 40;         // doubles per edge system
constexpr int kMaxDim = 7 * (M3S_MAX_KEYFRAMES - 1);  // largest reduced system
constexpr int kPatWords = (M3S_MAX_KEYFRAMES + 31) / 32;  // bit words of a set of keyframes

// The factor's block structure (backend_start_kernel), in elimination order:
// position k holds keyframe node perm[k] + 1.  Blocks of L are stored by
// column, the diagonal first, so that a level's blocks are consecutive slots.
constexpr int kLdsBlocks = 320;      // blocks of L in LDS: 320 x 392 B = 122.5 KB
constexpr int kMaxBlocks = 2048;     // blocks of L in the workspace
// Block products of the whole factorization.  A factor of at most 320 blocks
// needs at most 320 + 0.4714 * 320^1.5 = 3019 (edges plus triangles of its
// graph, Kruskal-Katona), which the LDS list holds.
constexpr int kLdsUpdates = 3072;
constexpr int kMaxUpdates = 8192;
// How the call's systems are solved (state[2]).
enum { kSolveLds = 0, kSolveGlobal = 1, kSolveDense = 2 };
// Whether a factor that exceeds LDS is solved faster as a dense system.  In the
// workspace a solve takes about 3.9 us a level and 0.092 us a block product (33
// keyframes, all joined: 32 levels, 5,456 products 581 us; 64 with 120 random
// closures: 30, 3,288 420; 128, each joined to its 8 neighbours: 68, 4,368 725),
// the dense one 2.9 us times the square of its tile columns (33 keyframes: 7
// columns, 150 us; 39: 9, 269; 64: 14, 620), and above kPanelRows, where its panel
// leaves LDS, 1.4 ms and more (128: 28, 9.1 ms), which no factor within the limits
// takes.
__device__ __forceinline__ bool dense_is_faster(int np, int nlev, int nupd) {
    const int nt = np / 32;
    return nt <= 14 && 390 * nlev + 9 * nupd > 294 * nt * nt + 210 * nt + 1200;  // in 10 ns
}
struct PatternBuf {
    int32_t nblk, nlev, nupd, pad;
    uint8_t perm[M3S_MAX_KEYFRAMES];          // position -> keyframe - 1
    uint8_t pos[M3S_MAX_KEYFRAMES];           // keyframe - 1 -> position
    uint16_t colstart[M3S_MAX_KEYFRAMES + 2]; // first slot of each column
    uint16_t lvl[M3S_MAX_KEYFRAMES + 2];      // first position of each level
    uint8_t si[kMaxBlocks], sj[kMaxBlocks];   // row and column position of each slot
    uint16_t ustart[kMaxBlocks + 2];          // products of slot s: upd[ustart[s]] ..
    int32_t estart[kMaxBlocks + 2];           // edges of slot s: elist[estart[s]] ..
    uint32_t upd[kMaxUpdates];                // slot of L_xv | slot of L_zv << 16
};

struct BackendArgs {
    int N, HW, E, blocks_per_edge;
    int n, np;                // reduced system size 7(N-1) and its padding to whole tiles
    const float* Xc;          // [N*HW*3]
    const float* Q;           // [N*HW]
    const int32_t* edges;     // [E*2] (i, j)
    const int32_t* idx;       // [E*HW]
    const uint8_t* valid;     // [E*HW]
    ConfGate gate;
    RobustWeights rw;
    double step_tol;
    double* T64;              // [N*12] world poses
    float* Trel;              // [E*12] T_ij = T_WC[i]^-1 T_WC[j] per edge at the current poses (zero out of range)
    double* edge_sys;         // [E*kStride] fp64 relative normal equations per edge
    double* edge_blk;         // [E*kBlk] A^T H_e A (49) and A^T g_e (7) per edge
    float* partials;          // [E*blocks_per_edge*kMomentStride]
    int32_t* state;           // [0] done flag, [1] applied steps, [2] kSolve*, [3] dense assembly ticket
    double* stat;             // [0] last step norm
    double* M;                // [np*np] dense reduced Hessian, factored in place, or the sparse factor's blocks
    double* rhs;              // [np]
    double* dinv;             // [nt*kTile*kTile] inverses of the diagonal tiles
    PatternBuf* pat;          // block structure of the factor
    uint32_t* elist;          // [3*E] edges of every slot: e | flags
    float* T_out;             // [N*12]
    float* info;              // [4] or null
};

constexpr int kGroup = 4;     // neighbouring matches a lane of the accumulation takes at a time
constexpr int kBlk = 56;      // 49 + 7 doubles per edge
constexpr int kMatchesMost = 8;     // matches per lane of the accumulation (amortises the workgroup reduction)
constexpr int kAccumBlocks = 1536;   // workgroups of an accumulation, at least, where there are matches for them
constexpr int kTile = 32;     // tile of the blocked Cholesky
constexpr int kPanelRows = 416;  // panel rows kept in LDS (larger systems read the panel from memory)
static_assert(kPanelRows <= kSolveThreads, "one thread per panel row");
constexpr int kStageRows = 64;   // raw panel rows staged per step of the panel product
constexpr int kPanelStride = kTile + 1;  // odd stride in doubles: rows of a wave fall in different banks

__device__ __forceinline__ bool edge_in_range(int ei, int ej, int N) {
    return ei >= 0 && ei < N && ej >= 0 && ej < N;
}

// T_ij of edge e = (ei, ej) in fp32 from the fp64 world poses (zero for an edge
// out of range); pose(k, j) is element j of keyframe k's pose.
template <class Pose>
__device__ __forceinline__ void write_relative_pose(const BackendArgs& A, int e, int ei, int ej, Pose pose) {
    double Wi[12], Wj[12], Ti[12], Tij[12];
    if (edge_in_range(ei, ej, A.N)) {
        for (int k = 0; k < 12; ++k) Wi[k] = pose(ei, k);
        for (int k = 0; k < 12; ++k) Wj[k] = pose(ej, k);
        sim3_inverse(Wi, Ti);
        sim3_mul(Ti, Wj, Tij);
    } else {
        for (int k = 0; k < 12; ++k) Tij[k] = 0.0;
    }
    for (int k = 0; k < 12; ++k) A.Trel[12 * e + k] = (float)Tij[k];
}

// A lane takes four neighbouring matches at a time: the six vector loads of the
// pixel side replace 24 scalar ones, and only the matched points and their
// confidences are gathered one by one (with
// 8 to 16 matches a lane, 68 to 60 us for 65 edges at 512 x 384 and 45 to 40 us for
// 199 at 224 x 160).
// COST: false = an iteration's accumulation (the system; skipped once the loop
// has ended), true = the final one (cost and count).
template <bool COST>
__global__ void __launch_bounds__(kThreads) backend_accum_kernel(BackendArgs A) {
    __shared__ float red[kThreads / 64][kMomentStride];
    if (!COST && A.state[0]) return;
    const int e = blockIdx.y;
    const int ei = A.edges[2 * e], ej = A.edges[2 * e + 1];
    const bool edge_ok = edge_in_range(ei, ej, A.N);
    float T[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) T[k] = A.Trel[12 * e + k];
    float acc[kMoments];
#pragma unroll
    for (int k = 0; k < kMoments; ++k) acc[k] = 0.f;

    const int32_t* idx = A.idx + (long)e * A.HW;
    const uint8_t* valid = A.valid + (long)e * A.HW;
    const float* Xi = A.Xc + (long)(edge_ok ? ei : 0) * A.HW * 3;
    const float* Xj = A.Xc + (long)(edge_ok ? ej : 0) * A.HW * 3;
    const float* Qi = A.Q + (long)(edge_ok ? ei : 0) * A.HW;
    const float* Qj = A.Q + (long)(edge_ok ? ej : 0) * A.HW;
    // Workgroups are dealt to the 8 XCDs round-robin (b % 8 with the edge's
    // workgroups consecutive); chunk c(b) gives XCD j the j-th contiguous
    // eighth of the chunks, so each XCD's L2 sees one slice of every keyframe
    // and the edges that share a keyframe reuse it there.
    const int bpe = A.blocks_per_edge;
    const int chunk = (bpe % 8 == 0) ? (int)(blockIdx.x % 8) * (bpe / 8) + (int)(blockIdx.x / 8) : (int)blockIdx.x;
    for (int g = edge_ok ? chunk * kThreads + (int)threadIdx.x : A.HW; kGroup * g < A.HW; g += bpe * kThreads) {
        const int n0 = kGroup * g;
        int mm[kGroup];
        bool ok[kGroup];
        float qj[kGroup], xj[kGroup][3];
        if (n0 + kGroup <= A.HW) {
            const uint32_t v4 = *reinterpret_cast<const u32_any*>(valid + n0);
            const i4_any i4 = *reinterpret_cast<const i4_any*>(idx + n0);
            const f4_any q4 = *reinterpret_cast<const f4_any*>(Qj + n0);
            const f4_any* x4 = reinterpret_cast<const f4_any*>(Xj + 3 * n0);
            const f4_any xa = x4[0], xb = x4[1], xc = x4[2];
            const float xs[12] = {xa.x, xa.y, xa.z, xa.w, xb.x, xb.y, xb.z, xb.w, xc.x, xc.y, xc.z, xc.w};
#pragma unroll
            for (int u = 0; u < kGroup; ++u) {
                mm[u] = i4[u];
                ok[u] = ((v4 >> (8 * u)) & 0xffu) != 0u;
                qj[u] = q4[u];
#pragma unroll
                for (int j = 0; j < 3; ++j) xj[u][j] = xs[3 * u + j];
            }
        } else {
#pragma unroll
            for (int u = 0; u < kGroup; ++u) {
                const bool in = n0 + u < A.HW;
                const int n = in ? n0 + u : n0;
                mm[u] = idx[n];
                ok[u] = in && valid[n] != 0;
                qj[u] = Qj[n];
#pragma unroll
                for (int j = 0; j < 3; ++j) xj[u][j] = Xj[3 * n + j];
            }
        }
        float qi[kGroup], xi[kGroup][3];
#pragma unroll
        for (int u = 0; u < kGroup; ++u) {
            ok[u] = ok[u] && (uint32_t)mm[u] < (uint32_t)A.HW;
            const uint32_t m = ok[u] ? (uint32_t)mm[u] : 0u;
            qi[u] = Qi[m];
            const float* x = Xi + 3u * m;
#pragma unroll
            for (int j = 0; j < 3; ++j) xi[u][j] = x[j];
        }
#pragma unroll
        for (int u = 0; u < kGroup; ++u) {
            float q;
            if (ok[u] && confidence_gate(qi[u], qj[u], A.gate, q))
                accumulate_match<COST>(T, xj[u][0], xj[u][1], xj[u][2], xi[u][0], xi[u][1], xi[u][2], q, A.rw, acc);
        }
    }

    block_moments<kThreads>(acc, red, A.partials + ((size_t)e * A.blocks_per_edge + blockIdx.x) * kMomentStride);
}

// One workgroup per edge: fixed-order fp64 sum of the edge's partials; then
// (iterations only) A = Ad(T_WC[i]^-1), A^T H_e A and A^T g_e.  Bound by the
// latency of its chain, so a fifth wave forms A while the other four sum, and
// the product takes two short steps (15, 65 and 198 edges: 5.0 -> 4.3, 6.2 -> 5.0
// and 5.4 -> 4.8 us).
constexpr int kEdgeThreads = kThreads + 64;
__global__ void __launch_bounds__(kEdgeThreads) backend_edge_kernel(BackendArgs A, int final_pass) {
    __shared__ double sys[kStride];
    __shared__ SumLds<kThreads> part;
    __shared__ double Ad[49], HA[49];
    if (!final_pass && A.state[0]) return;
    const int e = blockIdx.x, tid = threadIdx.x;
    const int ei = A.edges[2 * e], ej = A.edges[2 * e + 1];
    const bool in_range = edge_in_range(ei, ej, A.N);
    if (tid == kThreads && !final_pass && in_range) {
        double Ti[12];
        sim3_inverse(A.T64 + 12 * ei, Ti);
        sim3_adjoint(Ti, Ad);
    }
    sum_partials<kThreads>(A.partials + (size_t)e * A.blocks_per_edge * kMomentStride, A.blocks_per_edge, part, sys);
    if (tid < kVals) A.edge_sys[(size_t)e * kStride + tid] = sys[tid];
    if (final_pass || !in_range) return;
    double* out = A.edge_blk + (size_t)e * kBlk;
    const int a = tid / 7, b = tid % 7;
    if (tid < 49) {
        double hk = 0.0;
        for (int l = 0; l < 7; ++l) hk += sys[upper_index(a < l ? a : l, a < l ? l : a)] * Ad[7 * l + b];
        HA[tid] = hk;
    } else if (tid >= 64 && tid < 71) {
        const int c = tid - 64;
        double s = 0.0;
        for (int k = 0; k < 7; ++k) s += Ad[7 * k + c] * sys[28 + k];
        out[49 + c] = s;
    }
    __syncthreads();
    if (tid < 49) {
        double s = 0.0;
        for (int k = 0; k < 7; ++k) s += Ad[7 * k + a] * HA[7 * k + b];
        out[tid] = s;
    }
}

// Dense assembly of one block row of the reduced system (keyframe
// p = row + 1, rows 7(p-1) .. 7(p-1)+6; row N-1 is the padding rows).  The row
// block is summed from the edges' blocks in edge order (thread (a, b) owns the
// entry at offset (a, b) of the diagonal block, thread 64 + (a, b) those of the
// off-diagonal blocks, in LDS, so every entry has one writer, which visits the
// edges in order) and written out whole, zeros included, with its right-hand
// side -g.  The workgroup first lists the row's edges, one test a lane: with two
// waves looking at every edge in turn, a chain of one round trip an edge, the row
// took 104 us at 741 edges, now 11.
constexpr int kMaxNp = (kMaxDim + kTile - 1) / kTile * kTile;
constexpr uint32_t kRowEdge = 0xffffu, kRowOwnI = 1u << 16;  // listed edge; its other keyframe from bit 17
static_assert(M3S_MAX_EDGES <= 0x10000 && M3S_MAX_KEYFRAMES <= 1 << 15, "a listed edge in 32 bits");
struct AssembleLds {
    double rows[7 * kMaxNp];
    uint32_t list[kSolveThreads];
    int count[kSolveThreads / 64];
};

__device__ __forceinline__ void assemble_row(const BackendArgs& A, int row, AssembleLds& S) {
    const int np = A.np, n = A.n, tid = threadIdx.x;
    if (row == A.N - 1) {
        for (int r = n; r < np; ++r)
            for (int c = tid; c < np; c += kSolveThreads) A.M[(long)r * np + c] = r == c ? 1.0 : 0.0;
        for (int r = n + tid; r < np; r += kSolveThreads) A.rhs[r] = 0.0;
        return;
    }
    for (int i = tid; i < 7 * np; i += kSolveThreads) S.rows[i] = 0.0;
    const int P = row + 1, I = 7 * (P - 1);
    const int lane = tid & 63, wave = tid >> 6, a = lane / 7, b = lane % 7;
    const bool entry = lane < 49, rhs = tid >= 49 && tid < 56;
    double own = 0.0;  // thread's entry of the diagonal block, or of the right-hand side
    for (int e0 = 0; e0 < A.E; e0 += kSolveThreads) {
        const int e = min(e0 + tid, A.E - 1);
        const int ei = A.edges[2 * e], ej = A.edges[2 * e + 1];
        // A self edge has T_ij = I whatever the poses: its blocks cancel.
        const bool hit = e0 + tid < A.E && edge_in_range(ei, ej, A.N) && ei != ej && (ei == P || ej == P);
        const uint64_t hits = __ballot(hit);
        if (lane == 0) S.count[wave] = (int)__popcll(hits);
        __syncthreads();
        int at = (int)__popcll(hits & ((1ull << lane) - 1ull)), total = 0;
        for (int w = 0; w < kSolveThreads / 64; ++w) {
            if (w < wave) at += S.count[w];
            total += S.count[w];
        }
        if (hit) S.list[at] = (uint32_t)e | (ei == P ? kRowOwnI : 0u) | ((uint32_t)(ei == P ? ej : ei) << 17);
        __syncthreads();
        constexpr int kAhead = 4;  // reads in flight together
        for (int l0 = 0; tid < 128 && l0 < total; l0 += kAhead) {
            double t[kAhead];
            uint32_t f[kAhead];
#pragma unroll
            for (int j = 0; j < kAhead; ++j) {
                f[j] = S.list[min(l0 + j, total - 1)];
                // The diagonal takes A^T H_e A from either end; H_ij -= A^T H_e A, H_ji -= (A^T H_e A)^T.
                const bool turned = tid >= 64 && !(f[j] & kRowOwnI);
                const int at = rhs ? 49 + (tid - 49) : entry ? (turned ? 7 * b + a : 7 * a + b) : 0;
                t[j] = A.edge_blk[(size_t)(f[j] & kRowEdge) * kBlk + at];
            }
#pragma unroll
            for (int j = 0; j < kAhead; ++j) {
                if (l0 + j >= total) break;
                const int other = (int)(f[j] >> 17);
                if (tid < 64) own += rhs && !(f[j] & kRowOwnI) ? -t[j] : t[j];  // -g: g_i -= A^T g_e, g_j += A^T g_e
                else if (entry && other > 0) S.rows[a * np + 7 * (other - 1) + b] -= t[j];  // keyframe 0 holds the gauge
            }
        }
        __syncthreads();  // the list is done with
    }
    if (tid < 49) S.rows[a * np + I + b] = own;
    if (rhs) A.rhs[I + tid - 49] = own;
    __syncthreads();
    for (int i = tid; i < 7 * np; i += kSolveThreads) {
        const int r = i / np, c = i - r * np;
        A.M[(long)(I + r) * np + c] = S.rows[i];
    }
}

// Tile (ti, tj) of M as kTile x kTile, row-major with leading dimension np.
__device__ __forceinline__ double* tile_ptr(const BackendArgs& A, int ti, int tj) {
    return A.M + (long)ti * kTile * A.np + (long)tj * kTile;
}

// Trailing update of one 32 x 32 tile (ti, tj), tj <= ti, of the lower
// triangle below tile column k: M[R][C] -= L[R] . L[C], a 4 x 4 block per lane
// of one wave.  P points at the panel rows (stride ps doubles): LDS or M.  Tile
// (0, 0) is the next diagonal tile: its lower triangle goes to dl (the LDS tile
// the next factor reads, stride kTile + 1) instead of M.
template <typename PanelPtr>
__device__ __forceinline__ void trailing_tile(const BackendArgs& A, PanelPtr P, int ps, int R0, int ti, int tj,
                                              int lane, double* dl) {
    const int np = A.np;
    const int r0 = (lane >> 3) * 4, c0 = (lane & 7) * 4;
    const int ra = ti * kTile + r0, ca = tj * kTile + c0;
    // The target entries are read first so their latency overlaps the product.
    double cur[4][4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) cur[u][v] = A.M[(long)(R0 + ra + u) * np + R0 + ca + v];
    double acc[4][4] = {};
    for (int t = 0; t < kTile; ++t) {
        double va[4], vb[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            va[u] = P[(long)(ra + u) * ps + t];
            vb[u] = P[(long)(ca + u) * ps + t];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[u][v] += va[u] * vb[v];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (ti != tj || c0 + v <= r0 + u) {
                const double val = cur[u][v] - acc[u][v];
                if (ti == 0 && tj == 0) dl[(r0 + u) * (kTile + 1) + c0 + v] = val;
                else A.M[(long)(R0 + ra + u) * np + R0 + ca + v] = val;
            }
}

// What the end of a solve reads from memory, read before the substitution that
// precedes it: lane k's pose T_WC[k] and its edge of the first NT.
struct StepIn {
    double T[12];
    int ei, ej;
};
__device__ __forceinline__ StepIn read_step(const BackendArgs& A) {
    StepIn in;
    const int k = min((int)threadIdx.x, A.N - 1), e = min((int)threadIdx.x, A.E - 1);
    for (int j = 0; j < 12; ++j) in.T[j] = A.T64[12 * k + j];
    in.ei = A.edges[2 * e];
    in.ej = A.edges[2 * e + 1];
    return in;
}

// The end of a solve: pose updates T_WC[k] <- Exp(tau_k) o T_WC[k] for
// keyframes 1..N-1 from the solution x (LDS; keyframe k's step at
// 7 pos(k - 1)), the relative pose of every edge
// at the new poses (for the next accumulation), and the step norm, which ends
// the loop below step_tol.  All NT lanes of the workgroup call this; the poses
// pass between them in Tl (12 N doubles of LDS that x does not overlap), not
// through memory.  (With the lists' single round trip: the solve of 8, 32 and 96
// keyframes 16.9 -> 16.3, 34.6 -> 33.4 and 66.5 -> 65.1 us.)
template <int NT, class Pos>
__device__ __forceinline__ void apply_step(const BackendArgs& A, const StepIn& in, const double* x, double* Tl,
                                           double* red, Pos pos) {
    static_assert(NT >= M3S_MAX_KEYFRAMES, "one lane per keyframe");
    const int tid = threadIdx.x;
    if (tid < A.N) {
        double Tn[12];
        if (tid > 0) {
            double E[12];
            sim3_exp(x + 7 * pos(tid - 1), E);
            sim3_mul(E, in.T, Tn);
            for (int j = 0; j < 12; ++j) A.T64[12 * tid + j] = Tn[j];
        } else {
            for (int j = 0; j < 12; ++j) Tn[j] = in.T[j];
        }
        for (int j = 0; j < 12; ++j) Tl[12 * tid + j] = Tn[j];
    }
    __syncthreads();
    auto pose = [&](int k, int j) { return Tl[12 * k + j]; };
    if (tid < A.E) write_relative_pose(A, tid, in.ei, in.ej, pose);
    for (int e = tid + NT; e < A.E; e += NT) write_relative_pose(A, e, A.edges[2 * e], A.edges[2 * e + 1], pose);
    double sq = 0.0;
    for (int k = tid; k < A.n; k += NT) sq += x[k] * x[k];
    for (int o = 32; o > 0; o >>= 1) sq += __shfl_xor(sq, o, 64);
    if ((tid & 63) == 0) red[tid >> 6] = sq;
    __syncthreads();
    if (tid == 0) {
        double t = 0.0;
        for (int w = 0; w < NT / 64; ++w) t += red[w];
        const double step = sqrt(t);
        A.stat[0] = step;
        A.state[1] += 1;
        if (step < A.step_tol) A.state[0] = 1;
    }
}

struct DenseLds {
    double D[kTile][kTile + 1];                // diagonal tile being factored
    double Dinv[kTile][kTile + 1];             // its inverse
    double V[kTile][kTile + 1];                // the inverse's rows before scaling
    double panel[kPanelRows * kPanelStride];   // the factored panel below it
    double x[kMaxDim + kTile];                 // right-hand side, then the solution
    double red[kSolveThreads / 64];
    double stage[kStageRows * kPanelStride];   // raw panel rows
};

// One workgroup: factor the assembled dense system (blocked Cholesky), solve
// and update the poses.
__device__ __forceinline__ void dense_solve(const BackendArgs& A, DenseLds& S) {
    auto& D = S.D;
    auto& Dinv = S.Dinv;
    auto& V = S.V;
    auto& panel = S.panel;
    auto& x = S.x;
    auto& stage = S.stage;
    const int tid = threadIdx.x;
    const int n = A.n, np = A.np, nt = np / kTile;
    (void)n;

    for (int k = tid; k < np; k += kSolveThreads) x[k] = A.rhs[k];

    // Blocked right-looking Cholesky, lower triangle, kTile x kTile tiles.
    // Per tile column k: the diagonal tile is factored, its inverse
    // Dinv = L_kk^-1 is formed and kept for the substitutions, the panel below
    // becomes A_ik Dinv^T (a product, no sequential chain) and the trailing
    // lower triangle takes -= L_ik L_jk^T from the panel (in LDS when it fits).
    bool failed = false;  // the same in every thread: decided from LDS values read after a barrier
    for (int k = 0; k < nt; ++k) {
        double* Mk = tile_ptr(A, k, k);
        // Tile 0 comes from M; every later diagonal tile was left in D by the
        // previous trailing update (its lower triangle, the only part read).
        if (k == 0)
            for (int q = tid; q < kTile * kTile; q += kSolveThreads) D[q / kTile][q % kTile] = Mk[(long)(q / kTile) * np + q % kTile];
        for (int q = tid; q < kTile * kTile; q += kSolveThreads) V[q / kTile][q % kTile] = (q / kTile == q % kTile) ? 1.0 : 0.0;
        const int R0 = (k + 1) * kTile;
        const int m = np - R0;
        static_assert(kStageRows * kTile % kSolveThreads == 0, "whole raw values per thread");
        constexpr int kL = kStageRows * kTile / kSolveThreads;
        double raw[kL];
        auto read_stage = [&](int r0) {
#pragma unroll
            for (int j = 0; j < kL; ++j) {
                const int q = tid + j * kSolveThreads;
                const int rr = r0 + q / kTile, t = q % kTile;
                raw[j] = rr < m ? A.M[(long)(R0 + rr) * np + k * kTile + t] : 0.0;
            }
        };
        // The first panel stage's raw rows (below this tile, which the factor
        // does not write) are read before the factor, to arrive during it.
        if (m > 0) read_stage(0);
        __syncthreads();
        // Factor the tile with the whole workgroup, one barrier per step.  Per
        // column c, with d = D[c][c], the entries below take
        // D[r][q] -= D[r][c] D[q][c] / d and the rows of the running inverse
        // V[r][q] -= D[r][c] V[c][q] / d (r > c); the scaled outputs, column c
        // of L (to M) and row c of Dinv = L_kk^-1 = V[c] / sqrt(d), go to other
        // arrays.  A step takes a group of kC columns: every thread reads the
        // group's pivot block and its entries' values in the group's columns,
        // eliminates them through the group itself, and writes only entries
        // right of the group, rows of V below it, Dinv and M, so a step writes
        // nothing it reads.  Every thread forms the same pivots from the same
        // values read after a barrier, so the decision to stop is the same in
        // every thread.
        constexpr int kC = 4;  // columns per step
        static_assert(kTile % kC == 0, "whole column groups");
        for (int c = 0; c < kTile; c += kC) {
            // Two entries per thread.  Their operands (all inside the tile) are
            // read unconditionally together with the pivot block, so one LDS
            // round trip serves the step.
            static_assert(kTile * kTile % kSolveThreads == 0, "whole entries per thread");
            constexpr int kH = kTile * kTile / kSolveThreads;
            // Per entry: x = D[r][q] (entries right of the group) or V[r][q];
            // rc[l] = D[r][c+l]; y[l] = D[q][c+l] or V[c+l][q] to match x.
            double x[kH], rc[kH][kC], y[kH][kC];
#pragma unroll
            for (int h = 0; h < kH; ++h) {
                const int e2 = tid + h * kSolveThreads;
                const int r = e2 / kTile, q = e2 % kTile;
                const bool d_ent = q >= c + kC && q <= r;
                x[h] = d_ent ? D[r][q] : V[r][q];
#pragma unroll
                for (int l = 0; l < kC; ++l) {
                    rc[h][l] = D[r][c + l];
                    y[h][l] = d_ent ? D[q][c + l] : V[c + l][q];
                }
            }
            // The group's pivot block (lower triangle), eliminated by every thread.
            double B[kC][kC];
#pragma unroll
            for (int i = 0; i < kC; ++i)
#pragma unroll
                for (int j = 0; j <= i; ++j) B[i][j] = D[c + i][c + j];
            bool bad = false;
            double isv[kC], sdv[kC];
            double mk[kH], dv[kH];
#pragma unroll
            for (int h = 0; h < kH; ++h) mk[h] = dv[h] = 0.0;
#pragma unroll
            for (int j = 0; j < kC; ++j) {
                const double dj = B[j][j];
                bad = bad || !(dj > 0.0) || !isfinite(dj);
                // 1/sqrt(d): hardware estimate and two Newton steps.
                double is = __builtin_amdgcn_rsq(dj);
                is = is * fma(-0.5 * dj * is, is, 1.5);
                is = is * fma(-0.5 * dj * is, is, 1.5);
                const double idg = is * is;
                isv[j] = is;
                sdv[j] = dj * is;
#pragma unroll
                for (int i = j + 1; i < kC; ++i)
#pragma unroll
                    for (int l = j + 1; l <= i; ++l) B[i][l] -= B[i][j] * B[l][j] * idg;
#pragma unroll
                for (int h = 0; h < kH; ++h) {
                    const int e2 = tid + h * kSolveThreads;
                    const int r = e2 / kTile, q = e2 % kTile;
                    // Outputs of column c + j: L[r][c+j] and row c + j of Dinv.
                    if (q == c + j) mk[h] = rc[h][j] * is;
                    if (r == c + j) dv[h] = y[h][j] * is;
                    x[h] -= rc[h][j] * y[h][j] * idg;
#pragma unroll
                    for (int l = j + 1; l < kC; ++l) {
                        rc[h][l] -= rc[h][j] * B[l][j] * idg;
                        y[h][l] -= y[h][j] * B[l][j] * idg;
                    }
                }
            }
            if (bad) {
                failed = true;
                break;
            }
            // Each entry has at most one LDS output (D, V or a row of Dinv),
            // chosen by selects; the group's columns of L go to memory.
#pragma unroll
            for (int h = 0; h < kH; ++h) {
                const int e2 = tid + h * kSolveThreads;
                const int r = e2 / kTile, q = e2 % kTile;
                const bool d_upd = q >= c + kC && q <= r;
                const bool v_upd = r >= c + kC && q < c + kC;
                const bool i_row = r >= c && r < c + kC && q <= r;
                const double val = i_row ? dv[h] : x[h];
                double* dst = d_upd ? &D[r][q] : (v_upd ? &V[r][q] : &Dinv[r][q]);
                if (d_upd || v_upd || i_row) *dst = val;
                if (q >= c && q < c + kC && r > q) Mk[(long)r * np + q] = mk[h];
            }
            if (tid < kC) Mk[(long)(c + tid) * np + c + tid] = sdv[tid];
            __syncthreads();
        }
        if (failed) break;
        double* inv = A.dinv + (size_t)k * kTile * kTile;
        for (int q = tid; q < kTile * kTile; q += kSolveThreads) {
            const int r = q / kTile, c = q % kTile;
            inv[q] = c <= r ? Dinv[r][c] : 0.0;
        }
        // Forward substitution folded into the factorization: b_k has taken
        // every earlier tile's -L_kj y_j, so y_k = Dinv_k b_k now; the rows
        // below take -L_ik y_k during the trailing update.
        double yk = 0.0;
        if (tid < kTile) {
            for (int t = 0; t <= tid; ++t) yk += Dinv[tid][t] * x[k * kTile + t];
        }
        __syncthreads();
        if (tid < kTile) x[k * kTile + tid] = yk;
        // Panel: L_ik = A_ik Dinv^T, kStageRows rows at a time staged in LDS,
        // four elements per thread.  The raw rows of the next stage are read
        // into registers while the current one is computed (this stage writes
        // only its own rows).
        const bool in_lds = m <= kPanelRows;
        for (int r0 = 0; r0 < m; r0 += kStageRows) {
#pragma unroll
            for (int j = 0; j < kL; ++j) {
                const int q = tid + j * kSolveThreads;
                stage[(q / kTile) * kPanelStride + q % kTile] = raw[j];
            }
            __syncthreads();
            if (r0 + kStageRows < m) read_stage(r0 + kStageRows);
            // Column c of four rows per thread: each Dinv[c][t] is read once for
            // the four rows (same products and order per entry as a row-wise dot).
            const int c = tid % kTile;
            constexpr int kU = kStageRows * kTile / kSolveThreads;
            double acc[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) acc[u] = 0.0;
            for (int t = 0; t <= c; ++t) {
                // (The reads together: with this many registers the scheduler would
                // otherwise wait for each, 3 us a tile column.)
                const double dv = Dinv[c][t];
                double sv[kU];
#pragma unroll
                for (int u = 0; u < kU; ++u) sv[u] = stage[(tid / kTile + u * (kSolveThreads / kTile)) * kPanelStride + t];
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < kU; ++u) acc[u] += sv[u] * dv;
            }
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int rr = r0 + tid / kTile + u * (kSolveThreads / kTile);
                if (rr < m) {
                    A.M[(long)(R0 + rr) * np + k * kTile + c] = acc[u];
                    if (in_lds) panel[rr * kPanelStride + c] = acc[u];
                }
            }
            __syncthreads();
        }
        // Trailing update of the lower triangle, M[R][C] -= L[R] . L[C] for
        // R >= C >= R0: one wave per 32 x 32 tile.
        {
            const int tt = m / kTile;
            const int ntiles = tt * (tt + 1) / 2;
            const int wave = tid >> 6, lane = tid & 63;
            for (int tix = wave; tix < ntiles; tix += kSolveThreads / 64) {
                int ti = 0;
                while ((ti + 1) * (ti + 2) / 2 <= tix) ++ti;
                const int tj = tix - ti * (ti + 1) / 2;
                if (in_lds)
                    trailing_tile(A, (const double*)panel, kPanelStride, R0, ti, tj, lane, &D[0][0]);
                else
                    trailing_tile(A, (const double*)(A.M + (long)R0 * np + k * kTile), np, R0, ti, tj, lane, &D[0][0]);
            }
            // b_i -= L_ik y_k, one thread per panel row.
            auto minus_ly = [&](const double* row, double* b) {
                double sacc = 0.0;
                for (int t = 0; t < kTile; ++t) sacc += row[t] * x[k * kTile + t];
                *b -= sacc;
            };
            if (in_lds) {
                if (tid < m) minus_ly(panel + tid * kPanelStride, x + R0 + tid);
            } else {
                for (int rr = tid; rr < m; rr += kSolveThreads) minus_ly(A.M + (long)(R0 + rr) * np + k * kTile, x + R0 + rr);
            }
        }
        __syncthreads();
    }
    if (failed) {
        if (tid == 0) A.state[0] = 1;
        return;
    }

    // Backward substitution L^T tau = y, tile by tile from the last: tau_k =
    // Dinv_k^T y_k (y_k has taken every later tile's share), then every earlier
    // entry c takes -sum over the tile's rows r of L[r][c] tau_r: reads along
    // rows of L, contiguous across threads.
    // A tile's reads of Dinv and of the L entries of each thread's first
    // column are issued together, before either is needed.
    for (int k = nt - 1; k >= 0; --k) {
        const double* inv = A.dinv + (size_t)k * kTile * kTile;
        constexpr int kI = kTile * kTile / kSolveThreads;
        double dv[kI];
#pragma unroll
        for (int j = 0; j < kI; ++j) dv[j] = inv[tid + j * kSolveThreads];
        const bool first = tid < k * kTile;
        double lr[kTile];
        if (first) {
#pragma unroll
            for (int r = 0; r < kTile; ++r) lr[r] = A.M[(long)(k * kTile + r) * np + tid];
        }
#pragma unroll
        for (int j = 0; j < kI; ++j) {
            const int q = tid + j * kSolveThreads;
            Dinv[q / kTile][q % kTile] = dv[j];
        }
        __syncthreads();
        double y = 0.0;
        if (tid < kTile) {
            for (int t = tid; t < kTile; ++t) y += Dinv[t][tid] * x[k * kTile + t];
        }
        __syncthreads();
        if (tid < kTile) x[k * kTile + tid] = y;
        __syncthreads();
        if (first) {
            double sacc = 0.0;
#pragma unroll
            for (int r = 0; r < kTile; ++r) sacc += lr[r] * x[k * kTile + r];
            x[tid] -= sacc;
        }
        for (int c = tid + kSolveThreads; c < k * kTile; c += kSolveThreads) {
            double sacc = 0.0;
#pragma unroll 8
            for (int r = 0; r < kTile; ++r) sacc += A.M[(long)(k * kTile + r) * np + c] * x[k * kTile + r];
            x[c] -= sacc;
        }
        __syncthreads();
    }

    static_assert(12 * M3S_MAX_KEYFRAMES <= kPanelRows * kPanelStride, "poses in the panel's LDS");
    const StepIn step = read_step(A);
    __syncthreads();
    apply_step<kSolveThreads>(A, step, x, panel, S.red, [](int k) { return k; });
}

// ---------------------------------------------------------------- block-sparse solve
//
// The reduced system has one 7 x 7 block row per keyframe 1..N-1, and block
// (i, j) is non-zero only where an edge joins keyframes i and j.  Its Cholesky
// factor is as sparse, and as parallel, as the elimination order lets it be.
// backend_start_kernel picks the order once per call: level by level, each
// level an independent set of keyframes of nearly the least degree in the
// graph that the earlier levels leave (the chain of a sequence halves at every
// level).  The columns of one level depend on earlier levels only, so a level
// costs the latency of one column.  Eliminated one column at a time in keyframe
// order, a 31-column system (a 32-keyframe sequence with 3 closures) took 31
// steps of about 2.3 us and its factor had 115 blocks: 101 us; here it is 6
// levels, 89 blocks and 31 us.  A 96-keyframe sequence with 8 closures had
// 791 blocks, more than LDS holds, and took the dense solve, 3,578 us; here it
// is 9 levels, 288 blocks and 62 us.

constexpr int kPatThreads = 512;

// Edges of a slot: the edge and how its block enters (PatternBuf, elist).
constexpr uint32_t kEdgeMask = 0xffffu;   // M3S_MAX_EDGES fits 16 bits
constexpr uint32_t kEdgeTransposed = 1u << 16, kEdgeOwnI = 1u << 17;
static_assert(M3S_MAX_EDGES <= 0x10000, "edge index in 16 bits");
static_assert(M3S_MAX_KEYFRAMES <= 128, "two keyframes per lane, positions in a byte");

// Exclusive sums over the workgroup of every thread's v; total in *all.
__device__ __forceinline__ int block_exclusive(int v, int* tmp, int* all) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int inc = v;
    for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(inc, o, 64);
        if (lane >= o) inc += u;
    }
    __syncthreads();  // earlier readers of tmp are done
    if (lane == 63) tmp[wave] = inc;
    __syncthreads();
    int before = 0, sum = 0;
    for (int w = 0; w < kPatThreads / 64; ++w) {
        if (w < wave) before += tmp[w];
        sum += tmp[w];
    }
    *all = sum;
    return before + inc - v;
}

// Smallest value of the wave (every lane active), uniform.
__device__ __forceinline__ int wave_least(int v) {
    v = min(v, __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, false));   // quad_perm [1,0,3,2]
    v = min(v, __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, false));   // quad_perm [2,3,0,1]
    v = min(v, __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, false));  // row_half_mirror
    v = min(v, __builtin_amdgcn_mov_dpp(v, 0x140, 0xF, 0xF, false));  // row_mirror
    return min(min(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
               min(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

// The elimination, in one wave without barriers: lane l holds keyframes l and
// l + 64 of the remaining graph (rows r; adj holds them for the other lanes).  A
// level is a maximal independent set among the keyframes of degree at most
// max(least + 1, 2), found in rounds: a candidate that comes before all its
// candidate neighbours is taken, and its neighbours drop out.  The order is by
// degree, then by the parity of the index among the remaining keyframes (which
// takes every other keyframe of a chain in one round; the parity alternates from
// level to level), then by index.  Eliminating the level joins the neighbours of
// each of its keyframes.  About as many rounds as levels (9 levels in 12 rounds
// for 96 keyframes with 8 closures); taking the keyframes one at a time, least
// degree first, gave the same fill and number of levels in a serial chain of
// 0.27 to 0.43 us a keyframe.  Returns the number of levels.
__device__ __forceinline__ int eliminate(int nb, uint32_t (*adj)[kPatWords], uint32_t (*col)[kPatWords],
                                         uint32_t (*row)[kPatWords], int32_t* keys, uint8_t* perm, uint8_t* pos,
                                         uint16_t* lvl) {
    static_assert(kPatWords == 4, "two keyframes per lane, two words each");
    const int lane = threadIdx.x & 63;
    uint32_t r[2][kPatWords], mine[2][kPatWords];  // neighbours left; positions of the columns that hold the keyframe
    bool alive[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        alive[h] = lane + 64 * h < nb;
#pragma unroll
        for (int w = 0; w < kPatWords; ++w) {
            r[h][w] = alive[h] ? adj[lane + 64 * h][w] : 0u;
            mine[h][w] = 0u;
        }
    }
    auto below = [&](uint64_t m) { return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u)); };
    // Word w of a set held as two 64-bit masks.
    auto word = [](const uint64_t (&m)[2], int w) { return (uint32_t)(m[w >> 1] >> (32 * (w & 1))); };
    int k = 0, nlev = 0;
    while (k < nb) {
        if (lane == 0) lvl[nlev] = (uint16_t)k;
        int deg[2], least = INT_MAX;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            deg[h] = 0;
#pragma unroll
            for (int w = 0; w < kPatWords; ++w) deg[h] += __popc(r[h][w]);
            if (alive[h]) least = min(least, deg[h]);
        }
        const int top = max(wave_least(least) + 1, 2);
        const uint64_t left[2] = {__ballot(alive[0]), __ballot(alive[1])};
        int key[2];
        bool cand[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int rank = (h ? (int)__popcll(left[0]) : 0) + below(left[h]);
            key[h] = deg[h] * 256 + ((rank + nlev) & 1) * 128 + lane + 64 * h;
            cand[h] = alive[h] && deg[h] <= top;
            keys[lane + 64 * h] = key[h];
        }
        uint64_t level[2] = {0ull, 0ull};
        for (;;) {
            const uint64_t cm[2] = {__ballot(cand[0]), __ballot(cand[1])};
            if ((cm[0] | cm[1]) == 0ull) break;
            bool take[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                take[h] = cand[h];
#pragma unroll
                for (int w = 0; w < kPatWords; ++w) {
                    uint32_t m = cand[h] ? r[h][w] & word(cm, w) : 0u;
                    while (m) {
                        take[h] = take[h] && key[h] < keys[32 * w + __builtin_ctz(m)];
                        m &= m - 1u;
                    }
                }
            }
            const uint64_t tm[2] = {__ballot(take[0]), __ballot(take[1])};
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                uint32_t near = 0u;
#pragma unroll
                for (int w = 0; w < kPatWords; ++w) near |= r[h][w] & word(tm, w);
                cand[h] = cand[h] && !take[h] && near == 0u;
                if (take[h]) {
                    const int x = lane + 64 * h, p = k + (h ? (int)__popcll(tm[0]) : 0) + below(tm[h]);
                    perm[p] = (uint8_t)x;
                    pos[x] = (uint8_t)p;
#pragma unroll
                    for (int w = 0; w < kPatWords; ++w) col[p][w] = r[h][w];
                    alive[h] = false;
                }
                level[h] |= tm[h];
            }
            k += (int)(__popcll(tm[0]) + __popcll(tm[1]));
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int x = lane + 64 * h;
#pragma unroll
            for (int w = 0; w < kPatWords; ++w) {
                uint32_t m = alive[h] ? r[h][w] & word(level, w) : 0u;
                while (m) {
                    const int v = 32 * w + __builtin_ctz(m), p = pos[v];
                    m &= m - 1u;
#pragma unroll
                    for (int q = 0; q < kPatWords; ++q) {
                        r[h][q] |= col[p][q];
                        mine[h][q] |= (p >> 5) == q ? 1u << (p & 31) : 0u;
                    }
                }
            }
#pragma unroll
            for (int w = 0; w < kPatWords; ++w)
                r[h][w] = alive[h] ? r[h][w] & ~(word(level, w) | ((x >> 5) == w ? 1u << (x & 31) : 0u)) : 0u;
        }
        ++nlev;
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int w = 0; w < kPatWords; ++w) row[lane + 64 * h][w] = mine[h][w];
    return nlev;
}

// Once per call.  Workgroup 0: elimination order, levels, the factor's blocks,
// and for every block the edges that enter it and the products it takes.  It is
// a chain of short serial parts: 18 us for 32 keyframes and 44 us for
// 96, from 60 and 164 us with the wave minimum through LDS permutes, each slot's
// products found by walking every earlier column and its edges by one lane.  The
// other workgroups: the fp64 poses and the edges' relative poses at T_in.
__global__ void __launch_bounds__(kPatThreads) backend_start_kernel(BackendArgs A, const float* __restrict__ T_in) {
    __shared__ uint32_t adj[M3S_MAX_KEYFRAMES][kPatWords];
    __shared__ uint32_t col[M3S_MAX_KEYFRAMES][kPatWords];  // by position: later keyframes of the column
    __shared__ uint32_t row[M3S_MAX_KEYFRAMES][kPatWords];  // by keyframe: positions of its row's columns
    __shared__ uint8_t perm[M3S_MAX_KEYFRAMES], pos[M3S_MAX_KEYFRAMES];
    __shared__ int32_t cstart[M3S_MAX_KEYFRAMES + 1];
    __shared__ uint16_t lvl[M3S_MAX_KEYFRAMES + 2];
    __shared__ uint8_t si[kMaxBlocks], sj[kMaxBlocks];
    __shared__ int2 chunk[kPatThreads];
    __shared__ int32_t cursor[kMaxBlocks];  // edges of a slot, then where its next one goes
    __shared__ int tmp[kPatThreads / 64];
    __shared__ int nlev_s;
    const int nb = A.N - 1, tid = threadIdx.x, lane = tid & 63;
    if (blockIdx.x > 0) {
        const int t = ((int)blockIdx.x - 1) * kPatThreads + tid;
        if (t < 12 * A.N) A.T64[t] = (double)T_in[t];
        if (t < A.E) write_relative_pose(A, t, A.edges[2 * t], A.edges[2 * t + 1], [&](int k, int j) { return (double)T_in[12 * k + j]; });
        return;
    }
    if (tid < 4 && tid != 2) A.state[tid] = 0;
    if (tid < 2) A.stat[tid] = 0.0;
    PatternBuf& P = *A.pat;
    for (int i = tid; i < nb * kPatWords; i += kPatThreads) (&adj[0][0])[i] = 0u;
    __syncthreads();
    for (int e = tid; e < A.E; e += kPatThreads) {
        const int ei = A.edges[2 * e], ej = A.edges[2 * e + 1];
        if (!edge_in_range(ei, ej, A.N) || ei == ej || ei == 0 || ej == 0) continue;
        atomicOr(&adj[ei - 1][(ej - 1) >> 5], 1u << ((ej - 1) & 31));
        atomicOr(&adj[ej - 1][(ei - 1) >> 5], 1u << ((ei - 1) & 31));
    }
    __syncthreads();
    if (tid < 64) {
        const int nlev = eliminate(nb, adj, col, row, cursor, perm, pos, lvl);
        if (lane == 0) {
            lvl[nlev] = (uint16_t)nb;
            nlev_s = nlev;
        }
    }
    __syncthreads();
    // Column starts and the row and column of every slot.
    int nblk, c = 0;
    if (tid < nb)
        for (int w = 0; w < kPatWords; ++w) c += __popc(col[tid][w]);
    const int c0 = block_exclusive(tid < nb ? c + 1 : 0, tmp, &nblk);
    const bool fits = nblk <= kMaxBlocks;
    if (tid < nb) {
        cstart[tid] = c0;
        if (fits) {
            int s = c0;
            si[s] = sj[s] = (uint8_t)tid;
            ++s;
            for (int w = 0; w < kPatWords; ++w) {
                uint32_t m = col[tid][w];
                while (m) {
                    si[s] = pos[32 * w + __builtin_ctz(m)];
                    sj[s] = (uint8_t)tid;
                    ++s;
                    m &= m - 1u;
                }
            }
        }
    }
    __syncthreads();
    if (!fits) {
        if (tid == 0) A.state[2] = kSolveDense;
        return;
    }
    // Each thread's consecutive slots: products with every earlier column that
    // holds both the slot's row and its column.
    constexpr int kOwn = kMaxBlocks / kPatThreads;
    const int own_n = (nblk + kPatThreads - 1) / kPatThreads;
    auto own_slot = [&](int j) { return j < own_n ? tid * own_n + j : nblk; };
    // Columns that rows x and z of the factor share, before column z itself.
    auto shared_cols = [&](int x, int z, int w) { return row[x][w] & row[z][w]; };
    auto slot_in = [&](int v, int x) {  // slot of (keyframe x, column v)
        int s = cstart[v] + 1;
        for (int w = 0; w < (x >> 5); ++w) s += __popc(col[v][w]);
        return s + __popc(col[v][x >> 5] & ((1u << (x & 31)) - 1u));
    };
    int usum = 0;
    for (int j = 0; j < kOwn; ++j) {
        const int s = own_slot(j);
        if (s >= nblk) break;
        const int x = perm[si[s]], z = perm[sj[s]];
        for (int w = 0; w < kPatWords; ++w) usum += __popc(shared_cols(x, z, w));
    }
    int nupd;
    int u0 = block_exclusive(usum, tmp, &nupd);
    const bool in_lds = nblk <= kLdsBlocks && nupd <= kLdsUpdates;
    if (nupd > kMaxUpdates || (!in_lds && dense_is_faster(A.np, nlev_s, nupd))) {
        if (tid == 0) A.state[2] = kSolveDense;
        return;
    }
    for (int j = 0; j < kOwn; ++j) {
        const int s = own_slot(j);
        if (s >= nblk) break;
        P.ustart[s] = (uint16_t)u0;
        const int x = perm[si[s]], z = perm[sj[s]];
        for (int w = 0; w < kPatWords; ++w) {
            uint32_t m = shared_cols(x, z, w);
            while (m) {
                const int v = 32 * w + __builtin_ctz(m);
                m &= m - 1u;
                P.upd[u0++] = (uint32_t)slot_in(v, x) | ((uint32_t)slot_in(v, z) << 16);
            }
        }
    }
    // Edges of every slot, in edge order, first counted, then listed: eight
    // lanes per slot, each a contiguous eighth of a chunk of edges.
    for (int i = tid; i < nblk; i += kPatThreads) cursor[i] = 0;
    for (int pass = 0; pass < 2; ++pass) {
        for (int b = 0; b < A.E; b += kPatThreads) {
            __syncthreads();
            const int m = min(kPatThreads, A.E - b);
            if (tid < m) {
                const int ei = A.edges[2 * (b + tid)], ej = A.edges[2 * (b + tid) + 1];
                const bool use = edge_in_range(ei, ej, A.N) && ei != ej;
                chunk[tid] = use ? make_int2(ei - 1, ej - 1) : make_int2(-1, -1);
            }
            __syncthreads();
            const int sub = tid & 7, seg = (m + 7) / 8, t0 = min(sub * seg, m), t1 = min(t0 + seg, m);
            for (int s = tid >> 3; s < nblk; s += kPatThreads / 8) {
                const int x = perm[si[s]], z = perm[sj[s]];
                // H_ii, H_jj += blk; H_ij -= blk, H_ji -= blk^T: a row owned by j reads it transposed.
                // (An edge's two keyframes differ; no branches in the test.)
                auto hits = [&](int2 c) { return ((int)(c.x == x) | (int)(c.y == x)) & ((int)(c.x == z) | (int)(c.y == z)); };
                uint64_t hit = 0ull;  // of the at most 64 edges of the lane
#pragma unroll 4
                for (int t = t0; t < t1; ++t) hit |= (uint64_t)hits(chunk[t]) << (t - t0);
                const int c = (int)__popcll(hit);
                int inc = c;
                for (int o = 1; o < 8; o <<= 1) {
                    const int u = __shfl_up(inc, o, 8);
                    if (sub >= o) inc += u;
                }
                const int all = __shfl(inc, 7, 8);
                if (pass) {
                    int at = cursor[s] + inc - c;
                    while (hit) {
                        const int t = t0 + __builtin_ctzll(hit);
                        hit &= hit - 1ull;
                        const bool own = chunk[t].x == x;
                        A.elist[at++] = (uint32_t)(b + t) | (own ? kEdgeOwnI : 0u) |
                                        (x != z && !own ? kEdgeTransposed : 0u);
                    }
                }
                // The eight lanes have read the cursor (they are of one wave).
                if (sub == 7) cursor[s] += all;
            }
        }
        if (pass) break;
        __syncthreads();
        int esum = 0, nedge;
        for (int j = 0; j < kOwn; ++j) {
            const int s = own_slot(j);
            if (s < nblk) esum += cursor[s];
        }
        int base = block_exclusive(esum, tmp, &nedge);
        for (int j = 0; j < kOwn; ++j) {
            const int s = own_slot(j);
            if (s >= nblk) break;
            const int c = cursor[s];
            P.estart[s] = cursor[s] = base;
            base += c;
        }
        if (tid == 0) P.estart[nblk] = nedge;
    }
    for (int i = tid; i < nb; i += kPatThreads) {
        P.perm[i] = perm[i];
        P.pos[i] = pos[i];
        P.colstart[i] = (uint16_t)cstart[i];
    }
    for (int i = tid; i <= nlev_s; i += kPatThreads) P.lvl[i] = lvl[i];
    for (int i = tid; i < nblk; i += kPatThreads) {
        P.si[i] = si[i];
        P.sj[i] = sj[i];
    }
    if (tid == 0) {
        P.nblk = nblk;
        P.nlev = nlev_s;
        P.nupd = nupd;
        P.colstart[nb] = (uint16_t)nblk;
        P.ustart[nblk] = (uint16_t)nupd;
        A.state[2] = in_lds ? kSolveLds : kSolveGlobal;
    }
}

// LDS of the sparse solve.  In LDS mode the blocks take most of it; in global
// mode the longer lists do.
template <bool LDS>
struct SparseLds {
    static constexpr int kBlocks = LDS ? kLdsBlocks : kMaxBlocks;
    static constexpr int kUpdates = LDS ? kLdsUpdates : kMaxUpdates;
    static constexpr int kEntries = LDS ? 1024 : 8192;  // edge entries; the rest are read from memory
    double Lb[LDS ? kLdsBlocks * 49 : 1];
    double xs[kMaxDim];                        // right-hand side, then y, then the solution, by position
    double red[kSolveThreads / 64];
    alignas(8) uint32_t upd[kUpdates];
    uint32_t elist[kEntries];
    int32_t estart[kBlocks + 1];
    uint16_t ustart[kBlocks + 2];
    uint16_t off[kBlocks];                     // slots of the blocks off the diagonal
    uint16_t colstart[M3S_MAX_KEYFRAMES + 2], lvl[M3S_MAX_KEYFRAMES + 2];
    uint8_t pos[M3S_MAX_KEYFRAMES];
    uint8_t si[kBlocks], sj[kBlocks];
    int bad;
};

// Copies the pattern's lists to LDS, as many entries of each as the mode can
// hold (what lies past the pattern's own is not used): with the lengths not
// awaited, this is one round trip to memory instead of four.
template <bool LDS>
__device__ __forceinline__ void read_lists(const BackendArgs& A, SparseLds<LDS>& S) {
    const PatternBuf& P = *A.pat;
    const int tid = threadIdx.x, nb = A.N - 1;
    constexpr int kB = SparseLds<LDS>::kBlocks, kU = SparseLds<LDS>::kUpdates, kE = SparseLds<LDS>::kEntries;
    static_assert(kSolveThreads > M3S_MAX_KEYFRAMES && kU % kSolveThreads == 0 && kE % kSolveThreads == 0, "whole steps");
    uint32_t u[LDS ? kU / kSolveThreads : 1], l[LDS ? kE / kSolveThreads : 1];
    if constexpr (LDS) {
#pragma unroll
        for (int j = 0; j < kU / kSolveThreads; ++j) u[j] = P.upd[tid + j * kSolveThreads];
#pragma unroll
        for (int j = 0; j < kE / kSolveThreads; ++j) l[j] = A.elist[min(tid + j * kSolveThreads, 3 * A.E - 1)];
    }
    const int nblk = P.nblk;
    for (int i = tid; i < kB; i += kSolveThreads) {
        const uint8_t si = P.si[i], sj = P.sj[i];
        S.si[i] = si;
        S.sj[i] = sj;
        // A column's diagonal block comes first, so slot i is
        // the (i - sj - 1)-th other one.  (No pattern, so any value, in dense mode.)
        const int j = i - sj - 1;
        if (i < nblk && si != sj && j >= 0) S.off[j] = (uint16_t)i;
    }
    for (int i = tid; i <= kB; i += kSolveThreads) {
        S.ustart[i] = P.ustart[i];
        S.estart[i] = P.estart[i];
    }
    if (tid <= nb) {
        S.colstart[tid] = P.colstart[tid];
        if (tid < nb) S.pos[tid] = P.pos[tid];
        S.lvl[tid] = P.lvl[tid];
    }
    if constexpr (LDS) {
#pragma unroll
        for (int j = 0; j < kU / kSolveThreads; ++j) S.upd[tid + j * kSolveThreads] = u[j];
#pragma unroll
        for (int j = 0; j < kE / kSolveThreads; ++j) S.elist[tid + j * kSolveThreads] = l[j];
    } else {
        for (int i = tid; i < P.nupd; i += kSolveThreads) S.upd[i] = P.upd[i];
        for (int i = tid; i < min(3 * A.E, kE); i += kSolveThreads) S.elist[i] = A.elist[i];
    }
    if (tid == 0) S.bad = 0;
    __syncthreads();
}

// The blocks of the reduced system, each the sum of its edges' blocks in edge
// order, to Lb: one lane per entry and one wave per block.  A step of a wave
// takes QD diagonal blocks, of which the reads of each one's first four edges
// (a sequence's) are issued together without branches between them, and QO
// others with two (both directions of a pair); they come from memory that other
// XCDs wrote.  With four reads for every block, eight blocks a step and the
// right-hand side after them the gather took 3.3, 6.4 and 14.2 us for 8, 32 and
// 96 keyframes, now 2.2, 4.3 and 11.1; steps of 4 + 8 blocks the same, of 6 + 12
// and 12 + 24 slower (96 keyframes 1,177 and 1,462 us a call, not 1,172).
template <bool LDS, int QD, int QO>
__device__ __forceinline__ void gather_blocks(const BackendArgs& A, SparseLds<LDS>& S, double* __restrict__ Lb, int nb,
                                              int nblk) {
    constexpr int kD = 4, kO = 2, kWaves = kSolveThreads / 64;
    const int tid = threadIdx.x, wave = tid >> 6, en = min(tid & 63, 48), et = 7 * (en % 7) + en / 7;
    const int noff = nblk - nb;
    auto read = [&](int l, double& t) {
        const uint32_t f = S.elist[min(l, (int)S.kEntries - 1)];
        // Past the block's edges (or beyond the listed ones): some edge's block, not used.
        const uint32_t e = min(f & kEdgeMask, (uint32_t)(A.E - 1));
        t = A.edge_blk[(size_t)e * kBlk + ((f & kEdgeTransposed) ? et : en)];
    };
    auto sum = [&](const double* t, int most, int l0, int l1) {
        double v = 0.0;
        const int n0 = min(l0 + most, min(l1, (int)S.kEntries));
#pragma unroll
        for (int j = 0; j < kD; ++j)
            if (j < most) v += l0 + j < n0 ? t[j] : 0.0;
        for (int l = max(n0, l0); l < l1; ++l) {
            const uint32_t f = l < S.kEntries ? S.elist[l] : A.elist[l];
            v += A.edge_blk[(size_t)(f & kEdgeMask) * kBlk + ((f & kEdgeTransposed) ? et : en)];
        }
        return v;
    };
    const bool lane = (tid & 63) < 49;
    for (int d0 = wave, o0 = wave; d0 < nb || o0 < noff; d0 += kWaves * QD, o0 += kWaves * QO) {
        double td[QD][kD], to[QO][kD];
        int sd[QD], so[QO], l0[QD + QO], l1[QD + QO];
#pragma unroll
        for (int i = 0; i < QD; ++i) sd[i] = S.colstart[min(d0 + i * kWaves, nb - 1)];
#pragma unroll
        for (int i = 0; i < QO; ++i) so[i] = min((int)S.off[max(min(o0 + i * kWaves, noff - 1), 0)], nblk - 1);
#pragma unroll
        for (int i = 0; i < QD; ++i) {
            l0[i] = S.estart[sd[i]];
            l1[i] = S.estart[sd[i] + 1];
        }
#pragma unroll
        for (int i = 0; i < QO; ++i) {
            l0[QD + i] = S.estart[so[i]];
            l1[QD + i] = S.estart[so[i] + 1];
        }
#pragma unroll
        for (int i = 0; i < QD; ++i)
#pragma unroll
            for (int j = 0; j < kD; ++j) read(l0[i] + j, td[i][j]);
#pragma unroll
        for (int i = 0; i < QO; ++i)
#pragma unroll
            for (int j = 0; j < kO; ++j) read(l0[QD + i] + j, to[i][j]);
#pragma unroll
        for (int i = 0; i < QD; ++i) {
            if (d0 + i * kWaves >= nb) break;
            const double v = sum(td[i], kD, l0[i], l1[i]);
            if (lane) Lb[49 * sd[i] + en] = v;
        }
#pragma unroll
        for (int i = 0; i < QO; ++i) {
            if (o0 + i * kWaves >= noff) break;
            const double v = sum(to[i], kO, l0[QD + i], l1[QD + i]);
            if (lane) Lb[49 * so[i] + en] = -v;
        }
    }
}

// One workgroup: the block-sparse Cholesky over the pattern, left looking and
// level by level, the forward substitution folded in, the backward substitution
// (levels in reverse), and the pose updates.  Per level:
//   1. one lane per entry of the level's blocks: A_xz -= sum_v L_xv L_zv^T over
//      the listed products, and b_z -= sum_v L_zv y_v (ascending v: one writer
//      per entry in a fixed order);
//   2. sixteen lanes per column: every lane factors L_zz = chol(A_zz) and forms
//      L_zz^-1 in registers, y_z <- L_zz^-1 b_z, then one lane per row a of the
//      column's blocks: L_xz[a] <- A_xz[a] L_zz^-T.  L_zz^-1 replaces L_zz.
// LDS: the blocks are in LDS (Lb = S.Lb), else in the workspace.
template <bool LDS>
__device__ __forceinline__ void sparse_solve(const BackendArgs& A, SparseLds<LDS>& S, double* __restrict__ Lb) {
    const int nb = A.N - 1, tid = threadIdx.x;
    const int nblk = A.pat->nblk, nlev = A.pat->nlev;
    // The right-hand side -g (g_i -= A^T g_e, g_j += A^T g_e): the reads of each
    // entry's first kR edges, summed below.
    constexpr int kR = 4, kRounds = (kMaxDim + kSolveThreads - 1) / kSolveThreads;
    double g[kRounds][kR];
    auto rhs_entry = [&](int l, int a) {
        return A.edge_blk[(size_t)min(S.elist[min(l, (int)S.kEntries - 1)] & kEdgeMask, (uint32_t)(A.E - 1)) * kBlk + 49 + a];
    };
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int q = min(tid + r * kSolveThreads, 7 * nb - 1), l0 = S.estart[S.colstart[q / 7]];
        if (r * kSolveThreads < 7 * nb)
#pragma unroll
            for (int j = 0; j < kR; ++j) g[r][j] = rhs_entry(l0 + j, q % 7);
    }
    gather_blocks<LDS, 2, 4>(A, S, Lb, nb, nblk);
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int q = tid + r * kSolveThreads;
        if (q >= 7 * nb) break;
        const int s = S.colstart[q / 7], l0 = S.estart[s], l1 = S.estart[s + 1];
        double v = 0.0;
        for (int l = l0; l < l1; ++l) {
            const int j = l - l0;
            const uint32_t f = l < S.kEntries ? S.elist[l] : A.elist[l];
            double t;
            if (j < kR && l < S.kEntries) t = j == 0 ? g[r][0] : j == 1 ? g[r][1] : j == 2 ? g[r][2] : g[r][3];
            else t = A.edge_blk[(size_t)(f & kEdgeMask) * kBlk + 49 + q % 7];
            v += (f & kEdgeOwnI) ? t : -t;
        }
        S.xs[q] = v;
    }
    __syncthreads();
    const int grp = tid >> 4, gl = tid & 15;
    constexpr int kGroups = kSolveThreads / 16;
    for (int lv = 0; lv < nlev; ++lv) {
        const int k0 = S.lvl[lv], k1 = S.lvl[lv + 1];
        const int s0 = S.colstart[k0], s1 = S.colstart[k1];
        // 1. Products of earlier levels (the first level has none).
        if (lv > 0) {
            const int nb49 = 49 * (s1 - s0), nall = nb49 + 7 * (k1 - k0);
            for (int q = tid; q < nall; q += kSolveThreads) {
                if (q < nb49) {
                    const int s = s0 + q / 49, e = q % 49, a = e / 7, b = e - 7 * a;
                    const int u1 = S.ustart[s + 1];
                    int u = S.ustart[s];
                    if (u == u1) continue;
                    double v = Lb[49 * s + e];
                    for (; u < u1; ++u) {
                        const uint32_t f = S.upd[u];
                        const double* lx = Lb + 49 * (f & 0xffffu) + 7 * a;
                        const double* lz = Lb + 49 * (f >> 16) + 7 * b;
                        double t = 0.0;
#pragma unroll
                        for (int c = 0; c < 7; ++c) t += lx[c] * lz[c];
                        v -= t;
                    }
                    Lb[49 * s + e] = v;
                } else {
                    const int k = k0 + (q - nb49) / 7, a = (q - nb49) % 7, s = S.colstart[k];
                    const int u1 = S.ustart[s + 1];
                    double v = S.xs[7 * k + a];
                    for (int u = S.ustart[s]; u < u1; ++u) {
                        const int sz = (int)(S.upd[u] & 0xffffu);
                        const double* lz = Lb + 49 * sz + 7 * a;
                        const double* y = S.xs + 7 * S.sj[sz];
                        double t = 0.0;
#pragma unroll
                        for (int c = 0; c < 7; ++c) t += lz[c] * y[c];
                        v -= t;
                    }
                    S.xs[7 * k + a] = v;
                }
            }
            __syncthreads();
        }
        // 2. The level's columns.
        for (int k = k0 + grp; k < k1; k += kGroups) {
            double* Dk = Lb + 49 * S.colstart[k];
            double L[7][7], Li[7][7], yk[7], isd[7];
            bool bad = false;
#pragma unroll
            for (int j = 0; j < 7; ++j) {
                double d = Dk[7 * j + j];
#pragma unroll
                for (int m = 0; m < j; ++m) d -= L[j][m] * L[j][m];
                bad = bad || !(d > 0.0) || !isfinite(d);
                // 1/sqrt(d): hardware estimate and two Newton steps (no fp64
                // division or square root in the chain).
                double is = __builtin_amdgcn_rsq(d);
                is = is * fma(-0.5 * d * is, is, 1.5);
                is = is * fma(-0.5 * d * is, is, 1.5);
                L[j][j] = d * is;
                isd[j] = is;
#pragma unroll
                for (int i = j + 1; i < 7; ++i) {
                    double v = Dk[7 * i + j];
#pragma unroll
                    for (int m = 0; m < j; ++m) v -= L[i][m] * L[j][m];
                    L[i][j] = v * is;
                }
            }
            if (bad) {
                S.bad = 1;
                break;
            }
#pragma unroll
            for (int i = 0; i < 7; ++i) {
                Li[i][i] = isd[i];
#pragma unroll
                for (int j = 0; j < i; ++j) {
                    double v = 0.0;
#pragma unroll
                    for (int m = j; m < i; ++m) v += L[i][m] * Li[m][j];
                    Li[i][j] = -v * Li[i][i];
                }
            }
#pragma unroll
            for (int i = 0; i < 7; ++i) {
                double v = 0.0;
#pragma unroll
                for (int m = 0; m <= i; ++m) v += Li[i][m] * S.xs[7 * k + m];
                yk[i] = v;
            }
            // Panel rows: each lane reads its row before it writes it.
            const int nrow = 7 * (S.colstart[k + 1] - S.colstart[k] - 1);
            for (int q = gl; q < nrow; q += 16) {
                double* row = Dk + 49 + 7 * q;  // the column's blocks follow its diagonal
                double r[7], out[7];
#pragma unroll
                for (int c = 0; c < 7; ++c) r[c] = row[c];
#pragma unroll
                for (int b = 0; b < 7; ++b) {
                    double v = 0.0;
#pragma unroll
                    for (int c = 0; c <= b; ++c) v += r[c] * Li[b][c];
                    out[b] = v;
                }
#pragma unroll
                for (int b = 0; b < 7; ++b) row[b] = out[b];
            }
            // Every lane of the column (one wave holds it) has read the
            // diagonal block and b_k by now.
            if (gl == 0) {
#pragma unroll
                for (int i = 0; i < 7; ++i) {
#pragma unroll
                    for (int j = 0; j <= i; ++j) Dk[7 * i + j] = Li[i][j];
                    S.xs[7 * k + i] = yk[i];
                }
            }
        }
        __syncthreads();
        if (S.bad) {
            if (tid == 0) A.state[0] = 1;
            return;
        }
    }
    const StepIn step = read_step(A);
    // Backward substitution x_z = L_zz^-T (y_z - sum_x L_xz^T x_x): sixteen
    // lanes per column, lane 8 h + c summing component c over every other block.
    for (int lv = nlev - 1; lv >= 0; --lv) {
        const int k0 = S.lvl[lv], k1 = S.lvl[lv + 1];
        for (int kb = k0; kb < k1; kb += kGroups) {
            const int k = kb + grp;
            const bool on = k < k1;
            const int c = gl & 7, h = gl >> 3;
            const int sd = on ? S.colstart[k] : 0, n = on ? S.colstart[k + 1] - sd - 1 : 0;
            double t = 0.0;
            if (c < 7) {
                for (int j = h; j < n; j += 2) {
                    const double* blk = Lb + 49 * (sd + 1 + j) + c;
                    const double* xx = S.xs + 7 * S.si[sd + 1 + j];
#pragma unroll
                    for (int a = 0; a < 7; ++a) t += blk[7 * a] * xx[a];
                }
            }
            t += __shfl_xor(t, 8, 64);
            const double w = on && c < 7 ? S.xs[7 * k + c] - t : 0.0;
            double x = 0.0;
#pragma unroll
            for (int b = 0; b < 7; ++b) {
                const double wb = __shfl(w, (tid & 48) + b, 64);
                if (on && c <= b) x += Lb[49 * sd + 7 * b + min(c, 6)] * wb;
            }
            if (on && h == 0 && c < 7) S.xs[7 * k + c] = x;
        }
        __syncthreads();
    }
    // (The blocks, or in global mode the products, are done with.)
    double* Tl = LDS ? S.Lb : reinterpret_cast<double*>(S.upd);
    static_assert(12 * M3S_MAX_KEYFRAMES * 8 <= (LDS ? sizeof(S.Lb) : sizeof(S.upd)), "poses in LDS");
    apply_step<kSolveThreads>(A, step, S.xs, Tl, S.red, [&](int k) { return (int)S.pos[k]; });
}

// One launch per iteration, N workgroups.  Sparse: workgroup 0 solves and the
// others return.  Dense: every workgroup assembles its block row, and the last
// one to finish solves (its ticket tells; it resets the ticket for the next
// iteration).
__global__ void __launch_bounds__(kSolveThreads) backend_solve_kernel(BackendArgs A) {
    constexpr size_t kSparse = sizeof(SparseLds<true>) > sizeof(SparseLds<false>) ? sizeof(SparseLds<true>) : sizeof(SparseLds<false>);
    constexpr size_t kBytes = sizeof(DenseLds) > kSparse ? sizeof(DenseLds) : kSparse;
    static_assert(sizeof(AssembleLds) <= kBytes && kBytes <= 163328, "LDS of a CU");
    __shared__ __align__(16) char lds[kBytes];
    __shared__ int last;
    // (The lists of the usual mode are on their way while the state is read.)
    if (blockIdx.x == 0) read_lists<true>(A, *reinterpret_cast<SparseLds<true>*>(lds));
    if (A.state[0]) return;
    const int mode = A.state[2];
    if (mode != kSolveDense) {
        if (blockIdx.x != 0) return;
        if (mode == kSolveLds) {
            SparseLds<true>& S = *reinterpret_cast<SparseLds<true>*>(lds);
            sparse_solve<true>(A, S, S.Lb);
        } else {
            SparseLds<false>& S = *reinterpret_cast<SparseLds<false>*>(lds);
            __syncthreads();
            read_lists<false>(A, S);
            sparse_solve<false>(A, S, A.M);
        }
        return;
    }
    __syncthreads();
    assemble_row(A, (int)blockIdx.x, *reinterpret_cast<AssembleLds*>(lds));
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) last = atomicAdd(A.state + 3, 1) == (int)gridDim.x - 1 ? 1 : 0;
    __syncthreads();
    if (!last) return;
    __threadfence();
    if (threadIdx.x == 0) A.state[3] = 0;
    dense_solve(A, *reinterpret_cast<DenseLds*>(lds));
}

__global__ void __launch_bounds__(256) backend_finish_kernel(BackendArgs A) {
    const int t = threadIdx.x + blockIdx.x * blockDim.x;
    if (t < 12 * A.N) A.T_out[t] = (float)A.T64[t];
    if (blockIdx.x == 0 && A.info) {
        // Cost and count: every 256th edge per thread, then the threads in a fixed tree.
        __shared__ double part[2][256];
        double cost = 0.0, count = 0.0;
        for (int e = threadIdx.x; e < A.E; e += 256) {
            if (!edge_in_range(A.edges[2 * e], A.edges[2 * e + 1], A.N)) continue;
            cost += A.edge_sys[(size_t)e * kStride + 35];
            count += A.edge_sys[(size_t)e * kStride + 36];
        }
        part[0][threadIdx.x] = cost;
        part[1][threadIdx.x] = count;
        for (int o = 128; o > 0; o >>= 1) {
            __syncthreads();
            if ((int)threadIdx.x < o) {
                part[0][threadIdx.x] += part[0][threadIdx.x + o];
                part[1][threadIdx.x] += part[1][threadIdx.x + o];
            }
        }
        if (threadIdx.x == 0) {
            A.info[0] = (float)part[0][0];
            A.info[1] = (float)part[1][0];
            A.info[2] = (float)A.state[1];
            A.info[3] = (float)A.stat[0];
        }
    }
}

// Workspace layout.
struct BackendLayout {
    size_t T64, Trel, edge_sys, edge_blk, partials, state, stat, M, rhs, dinv, pat, elist, total;
};

int padded_dim(int N) { return (7 * (N - 1) + kTile - 1) / kTile * kTile; }

// Workgroups of one edge with `per` matches a lane.
int accum_blocks(int HW, int per) {
    const int b = (HW + kThreads * per - 1) / (kThreads * per);
    return b < 1 ? 1 : (b > 1024 ? 1024 : b);
}

// Rows of partials: enough for every problem with fewer edges or smaller frames as
// well, so that a workspace kept for a program's largest graph serves them all.
// (The split into more, shorter workgroups is taken below kAccumBlocks workgroups
// and at most doubles them.)
size_t partial_rows(int HW, int E) {
    const size_t most = (size_t)accum_blocks(HW, kMatchesMost) * E, split = (size_t)accum_blocks(HW, kGroup) * E;
    const size_t cap = 2 * (size_t)kAccumBlocks;
    static_assert(kMatchesMost == 2 * kGroup, "one halving");
    return std::max(most, std::min(split, cap));
}

BackendLayout backend_layout(int N, int HW, int E) {
    auto al = [](size_t v) { return (v + 255) / 256 * 256; };
    const size_t np = padded_dim(N);
    BackendLayout L;
    size_t o = 0;
    L.T64 = o;      o = al(o + sizeof(double) * 12 * N);
    L.Trel = o;     o = al(o + sizeof(float) * 12 * E);
    L.edge_sys = o; o = al(o + sizeof(double) * kStride * E);
    L.edge_blk = o; o = al(o + sizeof(double) * kBlk * E);
    L.partials = o; o = al(o + sizeof(float) * kMomentStride * partial_rows(HW, E));
    L.state = o;    o = al(o + sizeof(int32_t) * 4);
    L.stat = o;     o = al(o + sizeof(double) * 2);
    L.M = o;        o = al(o + sizeof(double) * np * np);
    L.rhs = o;      o = al(o + sizeof(double) * np);
    L.dinv = o;     o = al(o + sizeof(double) * np * kTile);
    L.pat = o;      o = al(o + sizeof(PatternBuf));
    L.elist = o;    o = al(o + sizeof(uint32_t) * 3 * (size_t)E);
    L.total = o;
    return L;
}

}  // namespace

// Workgroups of one edge: 8 matches a lane, or 4 where that leaves fewer than
// 6 workgroups a CU.  For 65 edges at 512 x 384 a 10-iteration solve takes 1,174 us with 32
// a lane, 1,127 with 16 and 1,085 with 8; for 15 edges at 160 x 120 the accumulation
// takes 18.4 us with 16 (75 workgroups) and 6.9 with 4 (285).
int backend_blocks_per_edge(int HW, int E) {
    const int most = accum_blocks(HW, kMatchesMost);
    return (int64_t)most * E < kAccumBlocks ? accum_blocks(HW, kGroup) : most;
}

size_t backend_workspace_bytes(int N, int HW, int E) { return backend_layout(N, HW, E).total; }

hipError_t launch_backend(int N, int HW, int E, const float* Xc, const float* Q, const int32_t* edges,
                          const int32_t* idx, const uint8_t* valid, float q_min, float sigma_ray, float sigma_dist,
                          float huber, int iters, double step_tol, float* T, float* info, void* ws, hipStream_t s) {
    const BackendLayout L = backend_layout(N, HW, E);
    char* w = reinterpret_cast<char*>(ws);
    BackendArgs A;
    A.N = N; A.HW = HW; A.E = E;
    A.blocks_per_edge = backend_blocks_per_edge(HW, E);
    A.n = 7 * (N - 1);
    A.np = padded_dim(N);
    A.Xc = Xc; A.Q = Q; A.edges = edges; A.idx = idx; A.valid = valid;
    A.gate = conf_gate(q_min);
    A.rw = robust_weights(sigma_ray, sigma_dist, huber);
    A.step_tol = step_tol;
    A.T64 = reinterpret_cast<double*>(w + L.T64);
    A.Trel = reinterpret_cast<float*>(w + L.Trel);
    A.edge_sys = reinterpret_cast<double*>(w + L.edge_sys);
    A.edge_blk = reinterpret_cast<double*>(w + L.edge_blk);
    A.partials = reinterpret_cast<float*>(w + L.partials);
    A.state = reinterpret_cast<int32_t*>(w + L.state);
    A.stat = reinterpret_cast<double*>(w + L.stat);
    A.M = reinterpret_cast<double*>(w + L.M);
    A.rhs = reinterpret_cast<double*>(w + L.rhs);
    A.dinv = reinterpret_cast<double*>(w + L.dinv);
    A.pat = reinterpret_cast<PatternBuf*>(w + L.pat);
    A.elist = reinterpret_cast<uint32_t*>(w + L.elist);
    A.T_out = T;
    A.info = info;
    const dim3 grid(A.blocks_per_edge, E);
    backend_start_kernel<<<1 + (max(12 * N, E) + kPatThreads - 1) / kPatThreads, kPatThreads, 0, s>>>(A, T);
    for (int it = 0; it <= iters; ++it) {
        const int final_pass = it == iters ? 1 : 0;
        timer_begin("backend_accum", s);
        if (final_pass) backend_accum_kernel<true><<<grid, kThreads, 0, s>>>(A);
        else backend_accum_kernel<false><<<grid, kThreads, 0, s>>>(A);
        timer_end(s);
        timer_begin("backend_edge", s);
        backend_edge_kernel<<<E, kEdgeThreads, 0, s>>>(A, final_pass);
        timer_end(s);
        if (final_pass) break;
        timer_begin("backend_solve", s);
        backend_solve_kernel<<<N, kSolveThreads, 0, s>>>(A);
        timer_end(s);
    }
    backend_finish_kernel<<<(12 * N + 255) / 256, 256, 0, s>>>(A);
    return hipGetLastError();
}

}  // namespace m3s
