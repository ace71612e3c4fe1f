// The decision of a launched PCG iteration, taken by its product kernel.
#pragma once

#include "gba_device.h"
#include "gba_internal.h"

namespace gba {

// Sum of part[stride * q + off] over the workgroups q of a problem, by one
// wavefront (every lane gets the result).
__device__ __forceinline__ double wave_sum_blocks(const double* part, int stride, int off, int q0,
                                                  int q1, int sub = 0, int parts = 1) {
    // this wavefront is number `sub` of `parts` sharing the range; four
    // independent partial sums keep four loads in flight per lane
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    const int step = kWave * parts;
    int q = q0 + sub * kWave + lane_id();
    for (; q + 3 * step < q1; q += 4 * step) {
        s0 += part[stride * q + off];
        s1 += part[stride * (q + step) + off];
        s2 += part[stride * (q + 2 * step) + off];
        s3 += part[stride * (q + 3 * step) + off];
    }
    for (; q < q1; q += step) s0 += part[stride * q + off];
    return wave_sum((s0 + s1) + (s2 + s3));
}

// ==========================================================================
// PCG decisions.  The step taken by iteration i of the PCG is decided at its
// start, from the state (g.pcg) and the dot products r^T z, r^T r left by
// iteration i-1 (per camera-aligned workgroup in dot_partial): convergence,
// iteration limit, rejection ratio, beta = r^T z / (r^T z)_old.  The product
// kernel takes the decision (every workgroup from the same sums, so all agree;
// the problem's first workgroup stores it in g.pcg_dec for the later kernels
// of the iteration) and multiplies z, not the direction: by linearity
// S p = S z + beta S p_old, so the q reduction forms q = S z + beta q_old and
// p = z + beta p_old itself, and the apply kernel stores the state.  An
// iteration is three kernels with no separate scalar pass, and the product
// gathers one vector.
// ==========================================================================
__device__ __forceinline__ PcgState pcg_decision(const KernelGraph& g, int prob) {
    PcgState st = g.pcg[prob];
    const int q0 = g.dc_cam.prob_blk[prob], q1 = g.dc_cam.prob_blk[prob + 1];
    double rz = wave_sum_blocks(g.dot_partial, 2, 0, q0, q1);
    double rr = wave_sum_blocks(g.dot_partial, 2, 1, q0, q1);
    if (g.full) {   // the point parts of the full system's vectors
        const int p0 = g.dc_pts.prob_blk[prob], p1 = g.dc_pts.prob_blk[prob + 1];
        rz += wave_sum_blocks(g.pdot_partial, 2, 0, p0, p1);
        rr += wave_sum_blocks(g.pdot_partial, 2, 1, p0, p1);
    }
    if (st.done) {   // stopped earlier: nothing to do
        st.act = 0;
        return st;
    }
    if (st.fresh) {  // first step: p = z, r^T z from the start
        st.fresh = 0;
        st.beta = 0.0;
        st.act = kActFresh | kActState;
        return st;
    }
    int done = 0, keep_best = 0;
    st.iters += 1;
    st.rr = rr;
    const double ratio = g.pcg_ratio;
    const bool track = ratio > 0.0 && isfinite(ratio);
    if (track && rr < st.min_rr) {
        st.min_rr = rr;
        keep_best = 1;
    } else if (track && rr > ratio * ratio * st.min_rr) {
        done = 4;
    }
    if (!done && rr <= st.thresh) done = 1;
    if (!done && st.iters >= g.pcg_max_iters) done = 2;
    st.beta = st.rz > 0.0 ? rz / st.rz : 0.0;
    st.rz = rz;
    st.done = done;
    if (keep_best) st.use_best = 1;
    st.act = kActState | (done ? 0 : kActRun) | (keep_best ? kActKeepBest : 0) |
             (done == 4 ? kActRestore : 0);
    return st;
}

// One entry of the direction: z + beta p_old rounded to the vector type, or z
// on the first step.
template <typename VT>
__device__ __forceinline__ VT dir_entry(VT z, VT pold, int act, VT beta) {
    return (act & kActRun) ? fma(beta, pold, z) : z;
}

}  // namespace gba
