// Orders of the visual-inertial solve's observations, made on the device from
// the caller's arrays: points renumbered by the first keyframe that observes
// them, observations in padded point order (by point, then keyframe) and in
// keyframe order (by keyframe, then point).  Every order is a stable sort, so
// it depends on the input alone.
#pragma once

#include <hip/hip_runtime.h>

#include "gba_device.h"

namespace gba {
namespace vi {

// ---- stable counting sort of item indices by a key's digit, `per` items per
// workgroup, at most kSortBins digits
constexpr int kSortBits = 12, kSortBins = 1 << kSortBits;

__device__ __forceinline__ int sort_digit(const int* __restrict__ key, int item, int shift) {
    const int k = key[item];
    return k < 0 ? -1 : (k >> shift) & (kSortBins - 1);   // negative keys are left out
}

// counts per (digit, workgroup); in: the items in order (null: 0, 1, ...)
__global__ __launch_bounds__(256) void k_sort_count(int n, int per, const int* __restrict__ in,
                                                   const int* __restrict__ key, int shift, int nb, int* __restrict__ counts) {
    __shared__ int hist[kSortBins];
    for (int b = (int)threadIdx.x; b < nb; b += 256) hist[b] = 0;
    __syncthreads();
    const int i0 = (int)blockIdx.x * per, i1 = (int)min((long long)n, i0 + (long long)per);
    for (int i = i0 + (int)threadIdx.x; i < i1; i += 256) {
        const int b = sort_digit(key, in ? in[i] : i, shift);
        if (b >= 0) atomicAdd(&hist[b], 1);
    }
    __syncthreads();
    for (int b = (int)threadIdx.x; b < nb; b += 256) counts[(size_t)b * gridDim.x + blockIdx.x] = hist[b];
}

// one wavefront per digit: its counts become offsets within the digit
__global__ __launch_bounds__(64) void k_sort_rows(int nblk, int* __restrict__ counts, int* __restrict__ total) {
    int* row = counts + (size_t)blockIdx.x * nblk;
    const int l = lane_id();
    int base = 0;
    for (int k0 = 0; k0 < nblk; k0 += 64) {
        const int c = k0 + l < nblk ? row[k0 + l] : 0;
        int s = c;
        for (int off = 1; off < 64; off <<= 1) {
            const int t = __shfl_up(s, off, 64);
            if (l >= off) s += t;
        }
        if (k0 + l < nblk) row[k0 + l] = base + s - c;
        base += __shfl(s, 63, 64);
    }
    if (l == 0) total[blockIdx.x] = base;
}

// the digits' totals become their first positions (one wavefront)
__global__ __launch_bounds__(64) void k_sort_base(int nb, int* __restrict__ total) {
    const int l = lane_id();
    int base = 0;
    for (int k0 = 0; k0 < nb; k0 += 64) {
        const int c = k0 + l < nb ? total[k0 + l] : 0;
        int s = c;
        for (int off = 1; off < 64; off <<= 1) {
            const int t = __shfl_up(s, off, 64);
            if (l >= off) s += t;
        }
        if (k0 + l < nb) total[k0 + l] = base + s - c;
        base += __shfl(s, 63, 64);
    }
}

// the items to their places: one wavefront per `per` items, 64 at a time
// in order; lanes of one digit are ranked by ballots
__global__ __launch_bounds__(64) void k_sort_place(int n, int per, const int* __restrict__ in,
                                                  const int* __restrict__ key, int shift, int nb, const int* __restrict__ offset,
                                                  const int* __restrict__ base, int* __restrict__ out) {
    __shared__ int at[kSortBins];
    const int l = lane_id();
    for (int b = l; b < nb; b += 64) at[b] = base[b] + offset[(size_t)b * gridDim.x + blockIdx.x];
    __syncthreads();
    const int i0 = (int)blockIdx.x * per, i1 = (int)min((long long)n, i0 + (long long)per);
    for (int i = i0 + l; i - l < i1; i += 64) {
        const int item = i < i1 ? (in ? in[i] : i) : 0;
        const int b = i < i1 ? sort_digit(key, item, shift) : -1;
        uint64_t left = __ballot(b >= 0);
        while (left) {   // one digit at a time
            const int lead = __ffsll((long long)left) - 1;
            const int d = __builtin_amdgcn_readlane(b, lead);
            const uint64_t same = __ballot(b == d);
            if (b == d) out[at[d] + __popcll(same & ((1ull << l) - 1ull))] = item;
            __builtin_amdgcn_wave_barrier();
            if (l == lead) at[d] += __popcll(same);
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
            left &= ~same;
        }
    }
}

// ---- the orders
__global__ __launch_bounds__(256) void k_vo_fill(long long n, int* __restrict__ a, int v) {
    const long long i = blockIdx.x * 256LL + threadIdx.x;
    if (i < n) a[i] = v;
}

// 32-bit indices; per point the first keyframe and the observation count;
// unknown is set by an id outside [0, K) or [0, N)
__global__ __launch_bounds__(256) void k_vo_raw(long long n, int K, int N, const long long* __restrict__ kf64,
                                               const long long* __restrict__ pt64, int* __restrict__ kf,
                                               int* __restrict__ pt, int* __restrict__ first,
                                               int* __restrict__ cnt, int* __restrict__ unknown) {
    const long long e = blockIdx.x * 256LL + threadIdx.x;
    if (e >= n) return;
    if (kf64[e] < 0 || kf64[e] >= K || pt64[e] < 0 || pt64[e] >= N) {
        *unknown = 1;
        return;
    }
    const int k = (int)kf64[e], j = (int)pt64[e];
    kf[e] = k;
    pt[e] = j;
    atomicMin(first + j, k);
    atomicAdd(cnt + j, 1);
}

// points in their new order: counts, positions and the inverse map
__global__ __launch_bounds__(256) void k_vo_points(int n, const int* __restrict__ old, const int* __restrict__ cnt,
                                                  const double* __restrict__ Xraw, int* __restrict__ renum,
                                                  int* __restrict__ cnt_new, double* __restrict__ X) {
    const int q = (int)(blockIdx.x * 256 + threadIdx.x);
    if (q >= n) return;
    const int j = old[q];
    renum[j] = q;
    cnt_new[q] = cnt[j];
    for (int c = 0; c < 3; ++c) X[3 * (size_t)q + c] = Xraw[3 * (size_t)j + c];
}

__global__ __launch_bounds__(256) void k_vo_points_out(int n, const int* __restrict__ old, const double* __restrict__ X,
                                                      double* __restrict__ Xraw) {
    const int q = (int)(blockIdx.x * 256 + threadIdx.x);
    if (q >= n) return;
    for (int c = 0; c < 3; ++c) Xraw[3 * (size_t)old[q] + c] = X[3 * (size_t)q + c];
}

// observations into their point's run (in any order); qpt is -1 elsewhere
__global__ __launch_bounds__(256) void k_vo_place(long long n, const int* __restrict__ pt, const int* __restrict__ renum,
                                                 const int* __restrict__ at, int* __restrict__ used,
                                                 int* __restrict__ qe, int* __restrict__ qpt) {
    const long long e = blockIdx.x * 256LL + threadIdx.x;
    if (e >= n) return;
    const int j = renum[pt[e]];
    const int s = at[j] + atomicAdd(used + j, 1);
    qe[s] = (int)e;
    qpt[s] = j;
}

// each run of at most 64 observations by keyframe, then input order: a slot's
// place is the number of smaller ones in its run (the work grows with the square
// of a run: longer ones are sorted, k_vo_long_keys)
__global__ __launch_bounds__(256) void k_vo_rank(long long np, const int* __restrict__ qpt, const int* __restrict__ at,
                                                const int* __restrict__ cnt, const int* __restrict__ kf,
                                                const int* __restrict__ qe, int* __restrict__ qs) {
    const long long i = blockIdx.x * 256LL + threadIdx.x;
    if (i >= np) return;
    const int j = qpt[i];
    if (j < 0) {
        qs[i] = -1;
        return;
    }
    if (cnt[j] > 64) return;   // k_vo_long_place's
    const int lo = at[j], hi = lo + cnt[j], e = qe[i], k = kf[e];
    int r = 0;
    for (int u = lo; u < hi; ++u) {
        const int f = qe[u], m = kf[f];
        r += (m < k || (m == k && f < e)) ? 1 : 0;
    }
    qs[lo + r] = e;
}

// The observations of the longer runs are sorted by keyframe, then by point
// (both stable, so a run ends by keyframe, then input order).  keys: an
// observation's keyframe and its point's number among the long ones, -1 for the
// others; long_of: that number per point (-1: not long)
__global__ __launch_bounds__(256) void k_vo_long_keys(long long n, const int* __restrict__ kf, const int* __restrict__ pt,
                                                     const int* __restrict__ renum, const int* __restrict__ long_of,
                                                     int* __restrict__ key_kf, int* __restrict__ key_pt) {
    const long long e = blockIdx.x * 256LL + threadIdx.x;
    if (e >= n) return;
    const int l = long_of[renum[pt[e]]];
    key_kf[e] = l < 0 ? -1 : kf[e];
    key_pt[e] = l;
}

// sorted observations to the slots of the long runs (in the same order)
__global__ __launch_bounds__(256) void k_vo_long_place(int n, const int* __restrict__ sorted, const int* __restrict__ slot,
                                                      int* __restrict__ qs) {
    const int i = (int)(blockIdx.x * 256 + threadIdx.x);
    if (i < n) qs[slot[i]] = sorted[i];
}

// the point-order arrays; twice is set when a keyframe observes a point more
// than once; qkey: the slot's keyframe, -1 in a pad
__global__ __launch_bounds__(256) void k_vo_slots(long long np, const int* __restrict__ qs, const int* __restrict__ qpt,
                                                 const int* __restrict__ kf, const double* __restrict__ obs,
                                                 int* __restrict__ qkf, int* __restrict__ qkey,
                                                 double* __restrict__ qobs, int* __restrict__ twice) {
    const long long i = blockIdx.x * 256LL + threadIdx.x;
    if (i >= np) return;
    const int e = qs[i];
    const int k = e < 0 ? 0 : kf[e];
    qkf[i] = k;
    qkey[i] = e < 0 ? -1 : k;
    for (int c = 0; c < 3; ++c) qobs[3 * i + c] = e < 0 ? 0.0 : obs[3 * (size_t)e + c];
    if (e >= 0 && i > 0 && qpt[i - 1] == qpt[i] && kf[qs[i - 1]] == k) *twice = 1;
}

// the keyframe-order arrays, the slots' places in them and each keyframe's
// range
__global__ __launch_bounds__(256) void k_vo_kf(int n, int K, const int* __restrict__ kslot, const int* __restrict__ qkf,
                                              const int* __restrict__ qpt, const double* __restrict__ qobs,
                                              int* __restrict__ kf, int* __restrict__ pt, double* __restrict__ obs,
                                              int* __restrict__ kinv, int* __restrict__ kfoff) {
    const int e = (int)(blockIdx.x * 256 + threadIdx.x);
    if (e >= n) return;
    const int s = kslot[e], k = qkf[s];
    kf[e] = k;
    pt[e] = qpt[s];
    kinv[s] = e;
    for (int c = 0; c < 3; ++c) obs[3 * (size_t)e + c] = qobs[3 * (size_t)s + c];
    const int before = e == 0 ? -1 : qkf[kslot[e - 1]];
    for (int m = before + 1; m <= k; ++m) kfoff[m] = e;
    if (e == n - 1)
        for (int m = k + 1; m <= K; ++m) kfoff[m] = n;
}

}  // namespace vi
}  // namespace gba
