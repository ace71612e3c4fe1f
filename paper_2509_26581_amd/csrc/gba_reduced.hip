// The explicit reduced camera system of small problems: S = Hcc_lambda -
// sum_j W_j Hpp_lambda,j^-1 W_j^T formed once per damped step as a dense
// matrix, and the whole preconditioned conjugate-gradient solve on it in one
// workgroup per problem, or (one larger problem) the products of launched
// iterations.  The implicit products (gba_kernels.hip) stream the
// stored Jacobian once per PCG iteration and take two or three launches for
// it; with few cameras S is smaller than that Jacobian, and an iteration on it
// needs no launch.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "gba.h"
#include "gba_device.h"
#include "gba_internal.h"
#include "gba_pcg.h"

namespace gba {

// ==========================================================================
// Rank bitmaps, once per device graph: per camera one bit per point of its
// problem (set when the camera observes the point) in 64-bit words, each with
// the camera-major position of the word's first edge, so that the edge of
// (camera, point) is found by one 16-byte load and a population count.
// ==========================================================================
__global__ __launch_bounds__(256) void k_rank_set(DeviceGraph g) {
    for (int e = blockIdx.x * (int)blockDim.x + (int)threadIdx.x; e < g.ne;
         e += (int)(gridDim.x * blockDim.x)) {
        const int a = g.e_cam[e], prob = g.cam_prob[a];
        if (g.xs_off[prob] < 0) continue;
        const int p0 = g.prob_pt_off[prob], nw = rank_words(g.prob_pt_off[prob + 1] - p0);
        const int j = g.e_pt[e] - p0;
        RankWord* w = g.xs_rank + g.xs_rank_off[prob] + (size_t)(a - g.prob_cam_off[prob]) * nw + (j >> 6);
        atomicOr((unsigned long long*)&w->mask, 1ull << (j & 63));
    }
}

__global__ __launch_bounds__(64) void k_rank_clear(DeviceGraph g, size_t words) {
    for (size_t k = blockIdx.x * (size_t)blockDim.x + threadIdx.x; k < words;
         k += (size_t)gridDim.x * blockDim.x)
        g.xs_rank[k] = RankWord{0ull, 0, 0};
}

// first camera-major edge of camera a
__device__ __forceinline__ int cam_edge_begin(const DeviceGraph& g, int a) {
    return g.cm_run_off[g.chunk_run_off[g.cam_chunk_off[a]]];
}

// One wavefront per camera: the words' first edges, a running sum of their
// population counts.
__global__ __launch_bounds__(64) void k_rank_base(DeviceGraph g) {
    const int a = blockIdx.x, prob = g.cam_prob[a];
    if (g.xs_off[prob] < 0) return;
    const int nw = rank_words(g.prob_pt_off[prob + 1] - g.prob_pt_off[prob]);
    RankWord* w = g.xs_rank + g.xs_rank_off[prob] + (size_t)(a - g.prob_cam_off[prob]) * nw;
    int base = cam_edge_begin(g, a);
    const int l = lane_id();
    for (int k0 = 0; k0 < nw; k0 += kWave) {
        const int c = k0 + l < nw ? __popcll(w[k0 + l].mask) : 0;
        int s = c;
        for (int off = 1; off < kWave; off <<= 1) {
            const int t = __shfl_up(s, off, kWave);
            if (l >= off) s += t;
        }
        if (k0 + l < nw) w[k0 + l].base = base + s - c;
        base += __shfl(s, kWave - 1, kWave);
    }
}

// ==========================================================================
// Off-diagonal blocks of S: S_ik = -sum over the points j that cameras i and
// k both observe of W_ij Hpp_lambda,j^-1 W_kj^T = J_c,i^T (J_p,i Hpp^-1
// J_p,k^T) J_c,k, one workgroup per camera pair i < k (three of them for three
// rows of the block each look the edges up and load the Jacobians three times:
// FP64, 110,000 edges of 18 and 28 cameras, 98 and 114 us a step where whole
// blocks take 48 and 60).  Its four wavefronts share camera i's edges;
// each looks its edges' points up in camera k's rank bitmap and queues the matches, so that
// every lane of the arithmetic holds a common point; per match it reads both
// edges' stored Jacobians (camera-major copy) and the point's inverse block,
// and keeps the block's sums in registers: no atomics, and an order that
// depends on the problem alone.  Terms, sums and S are FP64 in the mixed modes
// too, as the launched products' camera sums are.  Bound by the gathers of the
// two Jacobians (192 B a match in FP32, mostly from the L2).  The diagonal
// blocks come with the preconditioner (k_cam_finalize).
// ==========================================================================

// one match's J_c,i^T (J_p,i Hpp^-1 J_p,k^T) J_c,k added to acc; ea, eb: the
// camera-major edges of both cameras
template <typename T, typename JS>
__device__ __forceinline__ void reduced_term(const DeviceGraph& g, int ea, int eb, double (&acc)[81]) {
    T ja[2][9], jb[2][9], pat[2][3], pbt[2][3];
    jac_load<JS>(g.jst_cm, ea, ja, pat);
    jac_load<JS>(g.jst_cm, eb, jb, pbt);
    const T* H = (const T*)g.hpp_inv + kHinvStride * (size_t)g.cm_pt[ea];
    const double h[6] = {(double)H[0], (double)H[1], (double)H[2], (double)H[3], (double)H[4], (double)H[5]};
    double A[2][2], pa[2][3], pb[2][3];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            pa[r][c] = (double)pat[r][c];
            pb[r][c] = (double)pbt[r][c];
        }
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const double t0 = pa[r][0] * h[0] + pa[r][1] * h[1] + pa[r][2] * h[2];
        const double t1 = pa[r][0] * h[1] + pa[r][1] * h[3] + pa[r][2] * h[4];
        const double t2 = pa[r][0] * h[2] + pa[r][1] * h[4] + pa[r][2] * h[5];
#pragma unroll
        for (int c = 0; c < 2; ++c) A[r][c] = t0 * pb[c][0] + t1 * pb[c][1] + t2 * pb[c][2];
    }
    double m[2][9];
#pragma unroll
    for (int c = 0; c < 9; ++c) {
        m[0][c] = A[0][0] * (double)jb[0][c] + A[0][1] * (double)jb[1][c];
        m[1][c] = A[1][0] * (double)jb[0][c] + A[1][1] * (double)jb[1][c];
    }
#pragma unroll
    for (int r = 0; r < 9; ++r) {
        const double u0 = (double)ja[0][r], u1 = (double)ja[1][r];
#pragma unroll
        for (int c = 0; c < 9; ++c) acc[9 * r + c] += u0 * m[0][c] + u1 * m[1][c];
    }
}

template <typename T, typename JS>
__global__ __launch_bounds__(256) void k_reduced_blocks(DeviceGraph g) {
    const int a = blockIdx.x, prob = g.cam_prob[a];
    const long long off = g.xs_off[prob];
    if (off < 0 || g.lam[prob] < 0.0) return;
    if ((sizeof(T) == 8) != (g.mode == kModeFP64) || sizeof(JS) != (size_t)g.jac_bytes) return;
    constexpr int kSums = 81, kRegsOut = (kSums + kWave - 1) / kWave;
    __shared__ int qa_s[4][2 * kWave], qb_s[4][2 * kWave];
    __shared__ double red[4][kRegsOut * kWave];
    const int l = lane_id(), w = (int)threadIdx.x >> 6;
    const int c0 = g.prob_cam_off[prob], nc = g.prob_cam_off[prob + 1] - c0, i = a - c0;
    const int p0 = g.prob_pt_off[prob], nw = rank_words(g.prob_pt_off[prob + 1] - p0);
    const int n = 9 * nc, ld = reduced_ld(n);
    const int q0 = cam_edge_begin(g, a), q1 = cam_edge_begin(g, a + 1);
    T* __restrict__ S = (T*)g.xs_S + off;
    int* qa = qa_s[w];
    int* qb = qb_s[w];
    for (int k = i + 1 + (int)blockIdx.y; k < nc; k += (int)gridDim.y) {   // uniform
        const RankWord* __restrict__ rank = g.xs_rank + g.xs_rank_off[prob] + (size_t)k * nw;
        double acc[kSums];
#pragma unroll
        for (int u = 0; u < kSums; ++u) acc[u] = 0.0;
        auto add = [&](int ea, int eb) { reduced_term<T, JS>(g, ea, eb, acc); };
        int queued = 0;   // uniform per wavefront
        for (int base = q0 + w * kWave; base < q1; base += 4 * kWave) {
            const int q = base + l;
            bool hit = false;
            int other = 0;
            if (q < q1) {
                const int j = g.cm_pt[q] - p0;
                const RankWord r = rank[j >> 6];
                hit = (r.mask >> (j & 63)) & 1ull;
                other = r.base + __popcll(r.mask & ((1ull << (j & 63)) - 1ull));
            }
            const uint64_t hits = __ballot(hit);
            if (!hits) continue;
            if (hit) {
                const int at = queued + __popcll(hits & ((1ull << l) - 1ull));
                qa[at] = q;
                qb[at] = other;
            }
            queued += __popcll(hits);
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            if (queued >= kWave) {
                const int ea = qa[l], eb = qb[l];
                const bool more = l < queued - kWave;
                const int na = more ? qa[kWave + l] : 0, nb = more ? qb[kWave + l] : 0;
                add(ea, eb);
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                if (more) {
                    qa[l] = na;
                    qb[l] = nb;
                }
                queued -= kWave;
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            }
        }
        if (l < queued) add(qa[l], qb[l]);
        __builtin_amdgcn_wave_barrier();
        wave_sum_scatter(acc);   // sum u in lane rev6(u % 64), register u / 64
        __syncthreads();         // the previous block's sums have been read
#pragma unroll
        for (int v = 0; v < kRegsOut; ++v) red[w][v * kWave + rev6(l)] = acc[v];
        __syncthreads();
        for (int u = (int)threadIdx.x; u < kSums; u += (int)blockDim.x) {
            const T sum = (T)(-((red[0][u] + red[1][u]) + (red[2][u] + red[3][u])));
            const int row = 9 * i + u / 9, col = 9 * k + u % 9;
            S[(size_t)col * ld + row] = sum;
            S[(size_t)row * ld + col] = sum;
        }
    }
}

// ==========================================================================
// The common points of every camera pair of a larger problem, once per device
// graph (the lookups above in every step would take 180 us at 203 cameras).
// One wavefront per pair: counts, then (after the scan) the matches in point
// order.
// ==========================================================================
template <bool kFill>
__global__ __launch_bounds__(256) void k_pair_lists(DeviceGraph g) {
    const int l = lane_id(), i = (int)blockIdx.x;
    const int k = (int)blockIdx.y * 4 + ((int)threadIdx.x >> 6);
    if (k >= g.nc) return;
    const size_t at = (size_t)i * g.nc + k;
    if (k <= i) {
        if (!kFill && l == 0) g.xs_pair_off[at] = 0;
        return;
    }
    const int nw = rank_words(g.np);
    const RankWord* __restrict__ rank = g.xs_rank + (size_t)k * nw;
    const int q0 = cam_edge_begin(g, i), q1 = cam_edge_begin(g, i + 1);
    int n = 0;
    const int first = kFill ? g.xs_pair_off[at] : 0;
    for (int base = q0; base < q1; base += kWave) {
        const int q = base + l;
        bool hit = false;
        int other = 0;
        if (q < q1) {
            const int j = g.cm_pt[q];
            const RankWord r = rank[j >> 6];
            hit = (r.mask >> (j & 63)) & 1ull;
            other = r.base + __popcll(r.mask & ((1ull << (j & 63)) - 1ull));
        }
        const uint64_t hits = __ballot(hit);
        if (kFill && hit) g.xs_pairs[first + n + __popcll(hits & ((1ull << l) - 1ull))] = make_int2(q, other);
        n += __popcll(hits);
    }
    if (!kFill && l == 0) g.xs_pair_off[at] = n;
}

// counts -> offsets (exclusive, the total last), one workgroup
__global__ __launch_bounds__(1024) void k_pair_scan(DeviceGraph g) {
    __shared__ int wsum[16];
    const int tid = (int)threadIdx.x, l = tid & 63, w = tid >> 6, n = g.nc * g.nc;
    int base = 0;
    for (int k0 = 0; k0 < n; k0 += 1024) {
        const int c = k0 + tid < n ? g.xs_pair_off[k0 + tid] : 0;
        int s = c;
        for (int off = 1; off < 64; off <<= 1) {
            const int t = __shfl_up(s, off, 64);
            if (l >= off) s += t;
        }
        if (l == 63) wsum[w] = s;
        __syncthreads();
        int before = base;
        for (int v = 0; v < 16; ++v) {
            if (v < w) before += wsum[v];
            base += wsum[v];
        }
        if (k0 + tid < n) g.xs_pair_off[k0 + tid] = before + s - c;
        __syncthreads();
    }
    if (tid == 0) g.xs_pair_off[n] = base;
}

// One record per camera-major edge, contiguous (128 bytes in the mixed modes):
// J_p Hpp^-1, two pads, J_c, J_p.  The matches of a pair are a few of its
// cameras' edges, and from the stored Jacobian's tiles each 16 bytes of one
// came with a line of their own.  A match takes J_p Hpp^-1 of one edge and J_p
// of the other, so that the blocks hold the same point inverses as the diagonal
// ones (a factor L L^T of an inverse rounded to FP32 is off by up to thousands
// of roundings where its condition passes 1e8: points far away for their
// baseline, at a small damping).
template <typename T, typename JS>
__global__ __launch_bounds__(256) void k_reduced_edges(DeviceGraph g) {
    if ((sizeof(T) == 8) != (g.mode == kModeFP64) || sizeof(JS) != (size_t)g.jac_bytes) return;
    const int e = (int)(blockIdx.x * 256 + threadIdx.x);
    if (e >= g.ne) return;
    T jc[2][9], jp[2][3];
    jac_load<JS>(g.jst_cm, e, jc, jp);
    T out[kEdgeRec];
    point_side(jp, (const T*)g.hpp_inv + kHinvStride * (size_t)g.cm_pt[e], out);
    out[6] = out[7] = (T)0;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
#pragma unroll
        for (int c = 0; c < 9; ++c) out[8 + 9 * r + c] = jc[r][c];
#pragma unroll
        for (int c = 0; c < 3; ++c) out[26 + 3 * r + c] = jp[r][c];
    }
    typedef T V __attribute__((ext_vector_type(16 / sizeof(T))));
    constexpr int kV = 16 / (int)sizeof(T);
    V* dst = (V*)((T*)g.xs_edge + kEdgeRec * (size_t)e);
#pragma unroll
    for (int k = 0; k < kEdgeRec / kV; ++k) {
        V v;
#pragma unroll
        for (int u = 0; u < kV; ++u) v[u] = out[kV * k + u];
        dst[k] = v;
    }
}

// entries kFirst .. kFirst + kN - 1 of edge e's record (whole 16-byte groups)
template <int kFirst, int kN, typename T>
__device__ __forceinline__ void edge_record(const DeviceGraph& g, int e, T (&v)[kN]) {
    typedef T V __attribute__((ext_vector_type(16 / sizeof(T))));
    constexpr int kV = 16 / (int)sizeof(T);
    static_assert(kFirst % kV == 0 && kN % kV == 0 && kFirst + kN <= kEdgeRec, "whole groups of the record");
    const V* src = (const V*)((const T*)g.xs_edge + kEdgeRec * (size_t)e + kFirst);
#pragma unroll
    for (int k = 0; k < kN / kV; ++k) {
        const V x = src[k];
#pragma unroll
        for (int u = 0; u < kV; ++u) v[kV * k + u] = x[u];
    }
}

// Off-diagonal blocks of S from the lists, kLanes lanes per camera pair (about
// a pair's mean number of common points, as the sums over the lanes cost more
// than the terms of one match); pairs without a common point keep the zeros of
// the build.  203 cameras, 0.4M pairs of edges: 39 us a step (mixed), 68 (FP64;
// 98 with three lane groups for three rows of a block each).
template <typename T, int kLanes>
__global__ __launch_bounds__(256) void k_reduced_pairs(DeviceGraph g) {
    if ((sizeof(T) == 8) != (g.mode == kModeFP64)) return;
    constexpr int kSums = 81, kGroups = 256 / kLanes;
    const int l = (int)threadIdx.x % kLanes, i = (int)blockIdx.x;
    const int k = i + 1 + (int)blockIdx.y * kGroups + (int)threadIdx.x / kLanes;
    if (i + 1 + (int)blockIdx.y * kGroups >= g.nc || g.lam[0] < 0.0) return;   // uniform
    int m0 = 0, m1 = 0;
    if (k < g.nc) {
        const size_t at = (size_t)i * g.nc + k;
        m0 = g.xs_pair_off[at];
        m1 = g.xs_pair_off[at + 1];
    }
    if (__ballot(m0 < m1) == 0) return;   // whole wavefronts
    double acc[kSums];
#pragma unroll
    for (int u = 0; u < kSums; ++u) acc[u] = 0.0;
    for (int m = m0 + l; m < m1; m += kLanes) {
        const int2 e = g.xs_pairs[m];
        T a[28], b[24];
        edge_record<0, 28>(g, e.x, a);   // J_p Hpp^-1, the pads, J_c (and two entries of J_p)
        edge_record<8, 24>(g, e.y, b);   // J_c, J_p
        const T* ja = a + 8;
        double A[2][2], M[2][9];
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int c = 0; c < 2; ++c)
                A[r][c] = (double)a[3 * r] * (double)b[18 + 3 * c] + (double)a[3 * r + 1] * (double)b[19 + 3 * c] +
                          (double)a[3 * r + 2] * (double)b[20 + 3 * c];
#pragma unroll
        for (int c = 0; c < 9; ++c) {
            M[0][c] = A[0][0] * (double)b[c] + A[0][1] * (double)b[9 + c];
            M[1][c] = A[1][0] * (double)b[c] + A[1][1] * (double)b[9 + c];
        }
#pragma unroll
        for (int r = 0; r < 9; ++r) {
            const double u0 = (double)ja[r], u1 = (double)ja[9 + r];
#pragma unroll
            for (int c = 0; c < 9; ++c) acc[9 * r + c] += u0 * M[0][c] + u1 * M[1][c];
        }
    }
    group_sum_scatter<kLanes>(acc);   // sum u in lane group_rev(u % kLanes), register u / kLanes
    if (m0 == m1) return;
    const int ld = reduced_ld(9 * g.nc);
    T* __restrict__ S = (T*)g.xs_S;
#pragma unroll
    for (int v = 0; v < (kSums + kLanes - 1) / kLanes; ++v) {
        const int u = v * kLanes + group_rev<kLanes>(l);
        if (u < kSums) {
            const int row = 9 * i + u / 9, col = 9 * k + u % 9;
            S[(size_t)col * ld + row] = (T)-acc[v];
            S[(size_t)row * ld + col] = (T)-acc[v];
        }
    }
}

// ==========================================================================
// PCG on the explicit S, one workgroup of four or eight wavefronts per problem
// from the start to the stop.  The product: a wavefront takes 128 rows (two per
// lane) of one column group and keeps the first kRegs columns of the group in
// registers (the rest are read from the L2 every iteration); the direction is
// read from LDS four columns at a time, each value used for two rows, which
// balances the LDS reads (2 cycles a value and wavefront) with the products.
// The products, their sums and the vectors are FP64 in every mode; the mixed
// modes have FP32 in S's off-diagonal blocks (summed in FP64; the diagonal
// blocks stay FP64) and where the launched iterations have it in what goes in
// and out (right-hand side, preconditioner, solution).  With FP32 sums a damped
// step of five cameras with 16,000 common points was 5.7e-5 of its norm from the
// FP64 one, where it is 1.8e-5 now (FP64 blocks: 1.4e-5; launched products:
// 1.2e-4), and over 120 served requests of 5 to 40 keyframes the points of
// whole solves are 0.90 times as far from a 64-bit solve as the launched
// products' (geometric mean; FP64 blocks: 0.88).
// The vectors live in the registers of the row owners (63 rows, whole
// cameras, per wavefront, so that the preconditioner's exchange stays inside
// a wavefront) and an iteration is three workgroup barriers: direction,
// partial products with p^T q, residual dots.  Arithmetic and decisions are
// those of the launched kernels (pcg_decision, apply_body); q = S p is formed
// directly.  The order of every sum depends on the problem alone.  Bound by
// the latency of its serial chain (LDS exchanges, cross-lane sums, two FP64
// divisions): 1.3 us an iteration at 90 rows, where the launched iteration
// takes 14.2 us (two kernels).
// ==========================================================================
// four columns of the product for the two rows of a lane
template <typename T>
__device__ __forceinline__ void fma4(const double* __restrict__ p4, const T* __restrict__ a,
                                     const T* __restrict__ b, double (&qa)[4], double (&qb)[4]) {
    const double4 v = *(const double4*)p4;   // 16-byte aligned: columns start at multiples of four
    qa[0] = fma((double)a[0], v.x, qa[0]);
    qb[0] = fma((double)b[0], v.x, qb[0]);
    qa[1] = fma((double)a[1], v.y, qa[1]);
    qb[1] = fma((double)b[1], v.y, qb[1]);
    qa[2] = fma((double)a[2], v.z, qa[2]);
    qb[2] = fma((double)b[2], v.z, qb[2]);
    qa[3] = fma((double)a[3], v.w, qa[3]);
    qb[3] = fma((double)b[3], v.w, qb[3]);
}

// One problem's PCG in the first kWaves wavefronts of the workgroup (the
// others have returned): kR row wavefronts (128 kR rows at least n), kWaves /
// kR column groups.  kStream: groups may be wider than kRegs columns.
template <typename T, int kWaves, int kR, int kRegs, bool kStream>
__device__ __forceinline__ void pcg_reduced_body(const DeviceGraph& g, const int prob, double tol, int relative) {
    static_assert(kRegs % 4 == 0 && kWaves <= 16, "columns are taken four at a time");
    constexpr int kG = kWaves / kR, kRows = kR * 2 * kWave;
    constexpr int kOwners = (kRows + kOwnRows - 1) / kOwnRows < kWaves ? (kRows + kOwnRows - 1) / kOwnRows : kWaves;
    __shared__ __align__(32) double p_s[kRows + kRegs + 4];
    __shared__ double r_s[kOwners * kWave], x_s[kOwners * kWave];
    __shared__ double part[kG][kRows];
    __shared__ __align__(16) double red_q[16], red_z[16], red_r[16];
    const int c0 = g.prob_cam_off[prob], n = 9 * (g.prob_cam_off[prob + 1] - c0);
    const int ld = reduced_ld(n);
    const int W = (n + kOwnRows - 1) / kOwnRows;   // owner wavefronts, at most kOwners
    const int tid = (int)threadIdx.x, l = lane_id();
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform, and known to be
    const int grp = w / kR, row0 = (w % kR) * 2 * kWave + l, row1 = row0 + kWave;
    // columns of this wavefront's group, four at a time: columns past n are
    // column n - 1 against zeros of the direction, rows past n are row n - 1
    // and their sums meet zeros of the direction and no owner
    const int cpg = ((n + kG - 1) / kG + 3) & ~3;
    const int cb = min(grp * cpg, (n + 3) & ~3), ce = grp < kG ? min(n, cb + cpg) : cb;
    const T* __restrict__ S = (const T*)g.xs_S + g.xs_off[prob];
    // byte offsets of the lane's rows in a column, whose address is uniform
    const unsigned o0 = (unsigned)(min(row0, n - 1) * sizeof(T)), o1 = (unsigned)(min(row1, n - 1) * sizeof(T));
    auto entry = [&](int c, unsigned o) {
        return *(const T*)((const char*)(S + (size_t)(min(c, n - 1) * ld)) + o);
    };
    double s0[kRegs], s1[kRegs];
#pragma unroll
    for (int u = 0; u < kRegs; u += 4) {
        if (cb + u < ce) {
#pragma unroll
            for (int v = u; v < u + 4; ++v) {
                s0[v] = entry(cb + v, o0);
                s1[v] = entry(cb + v, o1);
            }
        }
    }
    const int own = w * kOwnRows + l;
    const bool owner = w < W && l < kOwnRows && own < n;
    const int a9 = l % 9, base9 = w * kWave + own_first(l);
    double m[9];
    double h[9];   // the owner's row of its camera's diagonal block
    double r = 0, p = 0, z = 0;
    T* __restrict__ best = (T*)g.v_best + 9 * (size_t)c0 + own;   // the owner's entry
#pragma unroll
    for (int b = 0; b < 9; ++b) {
        m[b] = 0;
        h[b] = 0.0;
    }
    if (owner) {
        const T* __restrict__ Minv = (const T*)g.minv + 45 * (size_t)(c0 + own / 9);
#pragma unroll
        for (int b = 0; b < 9; ++b) m[b] = (double)Minv[sym9(a9, b)];
        const double* __restrict__ D = g.xs_diag + 45 * (size_t)(c0 + own / 9);
#pragma unroll
        for (int b = 0; b < 9; ++b) h[b] = D[sym9(a9, b)];
        r = ((const T*)g.v_r)[9 * (size_t)c0 + own];
        *best = 0;
    }
    if (w < kOwners) x_s[tid] = 0;
    for (int k = tid; k < kRows + kRegs + 4; k += kWaves * kWave) p_s[k] = 0.0;
    if (grp < kG && cb >= ce) part[grp][row0] = part[grp][row1] = 0.0;   // a group without columns
    if (tid < 16) red_q[tid] = red_z[tid] = red_r[tid] = 0.0;
    __syncthreads();
    // sum of the wavefronts' values (of 16, by rotations inside a row of 16
    // lanes)
    auto sum_waves = [&](const double* v) {
        if constexpr (kWaves == 4) return (v[0] + v[1]) + (v[2] + v[3]);
        double t = v[l & 15];
        t += SegScan::move<0x128, 0xF>(t);
        t += SegScan::move<0x124, 0xF>(t);
        t += SegScan::move<0x122, 0xF>(t);
        t += SegScan::move<0x121, 0xF>(t);
        return lane63(t);
    };
    // z = M^-1 r and the dots r.z, r.r over the owners
    double rz = 0.0, rr = 0.0;
    auto precondition = [&]() {
        if (w < W) {
            r_s[tid] = r;
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            double z0 = 0, z1 = 0, z2 = 0;
#pragma unroll
            for (int b = 0; b < 9; b += 3) {   // (lane 63 reads the last camera's against m = 0)
                z0 += m[b] * r_s[base9 + b];
                z1 += m[b + 1] * r_s[base9 + b + 1];
                z2 += m[b + 2] * r_s[base9 + b + 2];
            }
            z = (z0 + z1) + z2;
            // both dots in one chain: the low half of the lanes goes on with
            // r.z, the high half with r.r
            double d = swap_add<32>(r * z, r * r);
            d += SegScan::move<0x128, 0xF>(d);
            d += SegScan::move<0x124, 0xF>(d);
            d += SegScan::move<0x122, 0xF>(d);
            d += SegScan::move<0x121, 0xF>(d);
            d = swap_add<16>(d, d);   // rows 0 and 1 (2 and 3) added
            if (l == 0) red_z[w] = d;
            if (l == 32) red_r[w] = d;
        }
        __syncthreads();
        rz = sum_waves(red_z);
        rr = sum_waves(red_r);
    };
    precondition();
    const double rr0 = rr, thresh = relative ? tol * tol * rr : tol * tol, ratio = g.pcg_ratio;
    const bool track = ratio > 0.0 && isfinite(ratio);
    double min_rr = rr, beta = 0.0;
    int iters = 0, use_best = 0;
    // every thread holds the same scalars; the decisions are made uniform
    auto yes = [](bool b) { return __builtin_amdgcn_readfirstlane((int)b) != 0; };
    int done = yes(g.lam[prob] < 0.0) ? 5 : (yes(rr <= thresh || !(rz > 0.0)) ? 1 : 0);
    while (!done) {
        p = iters ? fma(beta, p, z) : z;
        if (owner) p_s[own] = p;
        __syncthreads();
        double pq_part = 0.0;
        if (cb < ce) {
            const double p0 = p_s[row0], p1 = p_s[row1];
            double qa[4] = {0, 0, 0, 0}, qb[4] = {0, 0, 0, 0};
#pragma unroll
            for (int u = 0; u < kRegs; u += 4)
                if (cb + u < ce) fma4(p_s + cb + u, s0 + u, s1 + u, qa, qb);   // uniform per wavefront
#pragma unroll 1
            for (int c = cb + kRegs; kStream && c < ce; c += 4) {
                T a[4], b[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    a[u] = entry(c + u, o0);
                    b[u] = entry(c + u, o1);
                }
                fma4(p_s + c, a, b, qa, qb);
            }
            const double ta = (qa[0] + qa[1]) + (qa[2] + qa[3]), tb = (qb[0] + qb[1]) + (qb[2] + qb[3]);
            part[grp][row0] = ta;
            part[grp][row1] = tb;
            // p^T q from the partial products
            pq_part = p0 * ta + p1 * tb;
        }
        double q = 0;
        if (w < W && owner) {
            const int b0 = own - a9;
#pragma unroll
            for (int b = 0; b < 9; ++b) q += h[b] * p_s[b0 + b];
            pq_part += p * q;
        }
        {
            const double d = wave_sum(pq_part);
            if (l == 0) red_q[w] = d;
        }
        __syncthreads();
        if (w < W) {
            double t[kG];
#pragma unroll
            for (int k = 0; k < kG; ++k) t[k] = part[k][min(own, kRows - 1)];
#pragma unroll
            for (int k = 0; k < kG; ++k) q += t[k];
        }
        const double pq = sum_waves(red_q);
        if (yes(!(pq > 0.0 && isfinite(pq)))) {   // breakdown: x stays the last iterate
            done = 3;
            break;
        }
        const double alpha = rz / pq;
        if (owner) {
            x_s[tid] = fma(alpha, p, x_s[tid]);
            r = fma(-alpha, q, r);
        }
        const double rz_old = rz;
        precondition();
        iters += 1;
        if (track) {
            if (yes(rr < min_rr)) {
                min_rr = rr;
                use_best = 1;
                if (owner) *best = (T)x_s[tid];
            } else if (yes(rr > ratio * ratio * min_rr)) {
                done = 4;
                if (owner) x_s[tid] = *best;
            }
        }
        if (!done && yes(rr <= thresh)) done = 1;
        if (!done && iters >= g.pcg_max_iters) done = 2;
        beta = rz_old > 0.0 ? rz / rz_old : 0.0;
    }
    if (owner) ((T*)g.v_x)[9 * (size_t)c0 + own] = (T)x_s[tid];
    if (tid == 0) {
        PcgState st;
        st.rz = rz;
        st.rr = rr;
        st.rr0 = rr0;
        st.min_rr = min_rr;
        st.thresh = thresh;
        st.iters = iters;
        st.done = done;
        st.use_best = use_best;
        st.act = 0;
        st.beta = beta;
        st.fresh = iters == 0 ? 1 : 0;
        st.pad_ = 0;
        g.pcg[prob] = st;
        g.pcg_dec[prob] = st;
        if (g.pcg_host) g.pcg_host[prob] = st;
    }
}

// A problem's class follows its own size: up to 128 rows four wavefronts
// (one per SIMD: the scalar steps between the products, which every wavefront
// repeats, then issue once per SIMD), above that eight, with 32 columns of a
// group (of at most 64 up to 256 rows, of 128 to 256 above, FP32 S only) in
// registers, as FP64 in every mode, and the rest streamed from the L2.  More or
// fewer registers and FP32 in them were slower: FP64, 16 and 24 cameras, whole
// solves of 4,800 points, 24 and 40 columns 1.01 and 1.27, 1.05 and 1.25 ms
// against 0.90 and 1.18; mixed, whole solves of a window of 40 cameras, 24, 32,
// 40 and 48 columns 10.5, 10.2, 11.0 and 12.3 ms; of 18 cameras, whose products
// then convert every entry in every iteration, FP32 registers 4.9 against 2.6.  kBig:
// the batch holds a problem above the first class.
constexpr int kBigWaves = 8;
template <typename T, bool kBig>
__global__ __launch_bounds__(kBig ? kBigWaves * kWave : 4 * kWave) void k_pcg_reduced(DeviceGraph g, double tol,
                                                                                      int relative) {
    const int prob = blockIdx.x;
    if (g.xs_off[prob] < 0 || (sizeof(T) == 8) != (g.mode == kModeFP64)) return;
    const int n = 9 * (g.prob_cam_off[prob + 1] - g.prob_cam_off[prob]);
    if (n <= 2 * kWave) {
        if (kBig && threadIdx.x >= 4 * kWave) return;
        pcg_reduced_body<T, 4, 1, 32, false>(g, prob, tol, relative);
    } else if constexpr (kBig) {
        if (n <= 4 * kWave) pcg_reduced_body<T, kBigWaves, 2, 32, true>(g, prob, tol, relative);
        else if constexpr (sizeof(T) == 4) pcg_reduced_body<T, kBigWaves, 4, 32, true>(g, prob, tol, relative);
    }
}

// ==========================================================================
// A launched PCG iteration's product on S (one problem): the iteration's
// decision, then q = S p = S z + beta q_old, p = z + beta p_old and partial
// p^T q, kReducedRows rows per workgroup.  Four wavefronts share the columns
// (16 bytes a lane and row, every row's loads in flight together), the fifth
// takes the decision and the rows' other operands meanwhile.  Sums in FP64.
// Bound by the reads of S: 5.0 us at 203 cameras in FP32 (13 MB), 7.4 at 320
// (33 MB), where the point pass and its reduction take 12.6 and 14; 16 rows a
// workgroup and half the bytes in flight took 9.5 at 203.
// ==========================================================================
constexpr int kReducedProductBlock = 5 * kWave;
template <typename T>
__global__ __launch_bounds__(kReducedProductBlock) void k_reduced_product(KernelGraph g,
                                                                          const void* __restrict__ Sv,
                                                                          const double* __restrict__ D) {
    if ((sizeof(T) == 8) != (g.mode == kModeFP64)) return;
    constexpr int kWaves = 4;
    __shared__ double tot_s[kWaves][kReducedRows];
    const int n = 9 * g.nc, ld = reduced_ld(n), k0 = (int)blockIdx.x * kReducedRows;
    const int l = lane_id(), w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const T* __restrict__ z = (const T*)g.v_z;
    if (w == kWaves) {
        // lanes l < kReducedRows own a row each
        const int k = k0 + l, i = k / 9, r = k % 9;
        const bool own = l < kReducedRows && k < n;
        double diag = 0.0;
        T zk = 0, pold = 0, qold = 0;
        if (own) {
            zk = z[k];
            pold = ((const T*)g.v_p)[k];
            qold = ((const T*)g.v_q)[k];
#pragma unroll
            for (int c = 0; c < 9; ++c) diag += D[45 * (size_t)i + sym9(r, c)] * (double)z[9 * i + c];
        }
        const PcgState d = pcg_decision(g, 0);
        if (blockIdx.x == 0 && l == 0) g.pcg_dec[0] = d;
        __syncthreads();   // the products
        if (!(d.act & kActStep)) return;
        double dot = 0.0;
        if (own) {
            double s = diag;
#pragma unroll
            for (int v = 0; v < kWaves; ++v) s += tot_s[v][l];
            const T beta = (T)d.beta, sz = (T)s;
            const T q = (d.act & kActRun) ? fma(beta, qold, sz) : sz;
            const T p = (d.act & kActRun) ? fma(beta, pold, zk) : zk;
            ((T*)g.v_q)[k] = q;
            ((T*)g.v_p)[k] = p;
            dot = (double)p * (double)q;
        }
        dot = wave_sum(dot);
        if (l == 0) g.pq_partial[blockIdx.x] = dot;
        return;
    }
    constexpr int kV = 16 / (int)sizeof(T);
    typedef T V __attribute__((ext_vector_type(kV)));
    const T* __restrict__ S = (const T*)Sv;
    double acc[kReducedRows];
#pragma unroll
    for (int u = 0; u < kReducedRows; ++u) acc[u] = 0.0;
    if (!g.pcg[0].done) {   // (uniform; a stopped PCG only takes the decision)
        for (int c = kV * (int)threadIdx.x; c < n; c += kV * kWaves * kWave) {
            V s[kReducedRows];
#pragma unroll
            for (int u = 0; u < kReducedRows; ++u)   // rows are padded to whole vectors
                s[u] = *(const V*)(S + (size_t)min(k0 + u, n - 1) * ld + c);
#pragma unroll
            for (int v = 0; v < kV; ++v) {
                const bool in = c + v < n;
                const double zv = in ? (double)z[c + v] : 0.0;
#pragma unroll
                for (int u = 0; u < kReducedRows; ++u) acc[u] += (in ? (double)s[u][v] : 0.0) * zv;
            }
        }
    }
    wave_sum_scatter(acc);   // row u in lane rev6(u)
    if (rev6(l) < kReducedRows) tot_s[w][rev6(l)] = acc[0];
    __syncthreads();
}

// ==========================================================================
// launchers
// ==========================================================================
hipError_t launch_reduced_build(const DeviceGraph& g, size_t rank_total, size_t s_total, hipStream_t s) {
    if (!g.xs_on) return hipSuccess;
    const int eg = std::max(1, std::min(4096, (g.ne + 255) / 256));
    hipLaunchKernelGGL(k_rank_clear, dim3((unsigned)std::min<size_t>(4096, (rank_total + 63) / 64)), dim3(64),
                       0, s, g, rank_total);
    hipLaunchKernelGGL(k_rank_set, dim3(eg), dim3(256), 0, s, g);
    hipLaunchKernelGGL(k_rank_base, dim3(g.nc), dim3(64), 0, s, g);
    if (g.xs_wide) {
        const dim3 grid(g.nc, (unsigned)((g.nc + 3) / 4));
        hipLaunchKernelGGL(k_pair_lists<false>, grid, dim3(256), 0, s, g);
        hipLaunchKernelGGL(k_pair_scan, dim3(1), dim3(1024), 0, s, g);
        hipLaunchKernelGGL(k_pair_lists<true>, grid, dim3(256), 0, s, g);
        // (an even number of FP32 entries: whole padded columns)
        const hipError_t e = launch_fill_f64((double*)g.xs_S, 0.0, g.mode == kModeFP64 ? s_total : s_total / 2, s);
        if (e != hipSuccess) return e;
    }
    return hipGetLastError();
}

template <typename T, typename JS>
static void reduced_pairs(const DeviceGraph& g, hipStream_t s) {
    const long long mean = g.xs_pair_total / std::max(1LL, (long long)g.nc * (g.nc - 1) / 2);
    auto grid = [&](int lanes) {
        const int groups = 256 / lanes;
        return dim3(g.nc, (unsigned)std::max(1, (g.nc - 1 + groups - 1) / groups));
    };
    hipLaunchKernelGGL((k_reduced_edges<T, JS>), dim3((unsigned)((g.ne + 255) / 256)), dim3(256), 0, s, g);
    if (mean > 40) hipLaunchKernelGGL((k_reduced_pairs<T, 64>), grid(64), dim3(256), 0, s, g);
    else if (mean > 12) hipLaunchKernelGGL((k_reduced_pairs<T, 32>), grid(32), dim3(256), 0, s, g);
    else hipLaunchKernelGGL((k_reduced_pairs<T, 16>), grid(16), dim3(256), 0, s, g);
}

hipError_t launch_reduced_form(const DeviceGraph& g, hipStream_t s) {
    if (!g.xs_on || g.nc == 0) return hipSuccess;
    if (g.xs_wide) {
        if (g.mode == kModeFP64) reduced_pairs<double, double>(g, s);
        else if (g.mode == kModeFP32) reduced_pairs<float, float>(g, s);
        else reduced_pairs<float, bf16>(g, s);
        return hipGetLastError();
    }
    // one workgroup per block of the longest row
    const dim3 grid(g.nc, (unsigned)std::max(1, g.xs_cams - 1));
    if (g.mode == kModeFP64)
        hipLaunchKernelGGL((k_reduced_blocks<double, double>), grid, dim3(256), 0, s, g);
    else if (g.mode == kModeFP32)
        hipLaunchKernelGGL((k_reduced_blocks<float, float>), grid, dim3(256), 0, s, g);
    else
        hipLaunchKernelGGL((k_reduced_blocks<float, bf16>), grid, dim3(256), 0, s, g);
    return hipGetLastError();
}

hipError_t launch_reduced_product(const DeviceGraph& g0, hipStream_t s, int max_iters, double ratio) {
    KernelGraph g = g0;
    g.pcg_max_iters = max_iters;
    g.pcg_ratio = ratio;
    // (one problem: its S is the whole of xs_S)
    const dim3 grid(g0.xs_rows), block(kReducedProductBlock);
    const void* S = g0.xs_S;
    const double* D = g0.xs_diag;
    if (g.mode == kModeFP64) hipLaunchKernelGGL(k_reduced_product<double>, grid, block, 0, s, g, S, D);
    else hipLaunchKernelGGL(k_reduced_product<float>, grid, block, 0, s, g, S, D);
    return hipGetLastError();
}

// The problems with a one-workgroup PCG are stopped ones to launched iterations
// that run beside it (their decision reads `done` alone, which stays nonzero).
__global__ __launch_bounds__(64) void k_pcg_reduced_mark(DeviceGraph g) {
    const int prob = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (prob >= g.n_probs || g.xs_off[prob] < 0) return;
    g.pcg[prob].done = 1;
    g.pcg[prob].act = 0;
    g.pcg_dec[prob].act = 0;
}

hipError_t launch_pcg_reduced_mark(const DeviceGraph& g, hipStream_t s) {
    if (!g.xs_on) return hipSuccess;
    hipLaunchKernelGGL(k_pcg_reduced_mark, dim3((g.n_probs + 63) / 64), dim3(64), 0, s, g);
    return hipGetLastError();
}

hipError_t launch_pcg_reduced(const DeviceGraph& g0, hipStream_t s, double tol, int relative, int max_iters,
                              double ratio) {
    if (!g0.xs_on) return hipSuccess;
    DeviceGraph g = g0;
    g.pcg_max_iters = max_iters;
    g.pcg_ratio = ratio;
    const bool big = 9 * g.xs_cams > 2 * kWave;
    const dim3 grid(g.n_probs), block(!big ? 256 : 64 * kBigWaves);
    if (g.mode == kModeFP64) {
        if (big) hipLaunchKernelGGL((k_pcg_reduced<double, true>), grid, block, 0, s, g, tol, relative);
        else hipLaunchKernelGGL((k_pcg_reduced<double, false>), grid, block, 0, s, g, tol, relative);
    } else {
        if (big) hipLaunchKernelGGL((k_pcg_reduced<float, true>), grid, block, 0, s, g, tol, relative);
        else hipLaunchKernelGGL((k_pcg_reduced<float, false>), grid, block, 0, s, g, tol, relative);
    }
    return hipGetLastError();
}

}  // namespace gba
