// fmm_far.h -- far boxes through the targets' interval, for the eigenvector-side FMM kernels.
#pragma once

#include "fmm.h"

namespace sdc {

// ---------------------------------------------------------------------------------------
// The far field of one work item (64 neighbouring targets) as a function on the targets'
// interval.  Instead of meeting every target, a far box's 16 equivalent sources meet the 16
// Chebyshev nodes of the interval, and each target interpolates the boxes' sum there: a
// quarter of the Cauchy entries plus one 16-term series.  Only boxes at least FV_SEP_T interval
// widths away take part -- interpolating 1/(s - x) at that distance converges like
// (4 + sqrt 15)^-16 = 5e-15, the separation at which a box's own sources stand for its poles --
// the others stay with the direct sums (entries per row, level of 4096 problems: 541 -> 387;
// evaluation 3.25 -> 2.60 ms, b 1.75 -> 1.54 ms).  Node positions are kept as offsets from the
// interval's centre, so a difference s - x_m = (s - centre) - offset_m is as accurate as the
// shifted differences of the targets themselves.  Against long double, with and without the
// expansion: single entries of Q (5 problems of 8192, 40 of 2048) 1.0e-14 and 9.9e-15 off at most,
// what the boxes' own nodes leave; b of the last root, whose far field is all of it, 8.8e-16 and
// 6.7e-16; a last root with all but 1e-9 of its weight in boxes 1.5 intervals away and more 3.8e-16
// and 5.7e-16.
constexpr double FV_SEP_T = 1.5;
constexpr double FV_SEP_BWD = 3.0;  // the adjoint's, as its lists' (1/t^2 and 1/t^3 lose more)
constexpr int FV_MIN_EXP = 4;  // fewer boxes: the interpolation costs more than it saves
// A launch uses the expansion once its items give every CU two workgroups: from there the
// FP64 pipe is the bound (1024 items, one problem of 65536 with 64 columns: 232 -> 173 us with
// the expansion), below the latency of one item, which it lengthens (16 items, n = 1024: 17
// -> 20 us for 16 columns, 13 -> 18 us for b).
constexpr int FV_EXPAND_PER_CU = 2;

// cos((2q + 1) pi / 32) and (-1)^q sin((2q + 1) pi / 32): the nodes and barycentric weights
__constant__ double FV_NODE[FMM_P] = {
    0.99518472667219693, 0.95694033573220882, 0.88192126434835505, 0.77301045336273699,
    0.63439328416364549, 0.47139673682599781, 0.29028467725446233, 0.09801714032956077,
    -0.098017140329560645, -0.29028467725446216, -0.4713967368259977, -0.63439328416364538,
    -0.77301045336273699, -0.88192126434835494, -0.95694033573220882, -0.99518472667219682
};
__constant__ double FV_BARY[FMM_P] = {
    0.098017140329560604, -0.29028467725446233, 0.47139673682599764, -0.63439328416364549,
    0.77301045336273699, -0.88192126434835494, 0.95694033573220894, -0.99518472667219682,
    0.99518472667219693, -0.95694033573220894, 0.88192126434835505, -0.7730104533627371,
    0.63439328416364549, -0.47139673682599786, 0.29028467725446239, -0.098017140329560826
};

// centre and half-width of an item's targets, rows r0 .. r1 of the problem's n (targets are
// ascending: roots d_K + eta, or with trans 0 the poles); hw = 0: no expansion (one target, or
// targets so close together that the centre's rounding would show)
__device__ __forceinline__ double2 fv_interval(const FmmVec &v, int64_t base, int n, int r0, int r1) {
    double da = v.d[base + r0], db = v.d[base + r1], ea = 0.0, eb = 0.0;
    if (v.trans) {
        da = v.d[base + clamp_idx(v.origin[base + r0], n)];
        db = v.d[base + clamp_idx(v.origin[base + r1], n)];
        ea = v.eta[base + r0];
        eb = v.eta[base + r1];
    }
    const double c = 0.5 * ((da + ea) + (db + eb)), h = 0.5 * ((db - da) + (eb - ea));
    return make_double2(c, h >= 0x1p-44 * fabs(c) ? h : 0.0);
}

// The far boxes of leaf L (nl left, nr right ones) into fbox: those summed directly from the
// front, those of the expansion from the back; returns how many of the latter (none with
// expand false).  One wavefront, all lanes.
__device__ __forceinline__ int fv_split_far(const FmmArgs &f, const FmmVec &v, int L, int nl, int nr,
                                            double2 iv, bool expand, int *fbox) {
    const int lane = lane_id();
    int nd = 0, ne = 0;
    for (int e0 = 0; e0 < nl + nr; e0 += WAVE) {
        const int e = e0 + lane;
        const bool in = e < nl + nr;
        int g = 0;
        bool ex = false;
        if (in) {
            g = e < nl ? f.far_l[(int64_t)L * FMM_FAR_MAX + e]
                       : f.far_r[(int64_t)L * FMM_FAR_MAX + e - nl];
            // the box's end sources: its nodes descend (a leaf of few poles keeps them
            // ascending instead, but that is a problem's last leaf, whose nearest is the first)
            const double *nd2 = v.vnode + (int64_t)g * FMM_P;
            const double c = v.vcen ? v.vcen[g] - iv.x : -iv.x;
            const double dist = fmin(fabs(nd2[0] + c), fabs(nd2[FMM_P - 1] + c)) - iv.y;
            ex = expand && iv.y > 0.0 && dist >= v.sep_t * 2.0 * iv.y;
        }
        const unsigned long long md = __ballot(in && !ex), me = __ballot(ex);
        auto rank = [&](unsigned long long mk) {
            return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(mk >> 32),
                                                  __builtin_amdgcn_mbcnt_lo((unsigned)mk, 0u));
        };
        if (ex) fbox[2 * FMM_FAR_MAX - 1 - (ne + rank(me))] = g;
        else if (in) fbox[nd + rank(md)] = g;
        nd += __popcll(md);
        ne += __popcll(me);
    }
    if (ne > 0 && ne < FV_MIN_EXP) {  // too few: back among the direct ones
        if (lane < ne) {
            const int g = fbox[2 * FMM_FAR_MAX - 1 - lane];
            fbox[nd + lane] = g;
        }
        ne = 0;
    }
    return wave_uniform(ne);
}

}  // namespace sdc
