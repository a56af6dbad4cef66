// fmm.h -- triangular far-field compression of the secular sums (internal).
#pragma once

#include <vector>

#include "common.h"

namespace sdc {

constexpr int FMM_P = 16;          // Chebyshev nodes per box (equivalent sources)
constexpr int FMM_NEAR_MAX = 24;   // near leaves (and so near ranges) per target leaf
constexpr int FMM_FAR_MAX = 64;    // far boxes per side per target leaf
constexpr int FMM_PL = 20;         // Chebyshev terms of a target leaf's local expansion
constexpr int FMM_LOC = 4 * FMM_PL; // local expansion of a target leaf: psi, psi', phi, phi'
                                    // far fields, FMM_PL Chebyshev coefficients each

// Chebyshev nodes (first kind) of a P-point grid on [-1, 1], cos((2q + 1) pi / 2P), and the
// barycentric weights of the first FMM_P of them, (-1)^q sin((2q + 1) pi / 2P)
__device__ __forceinline__ double cheb_node(int q, int P = FMM_P) {
    return cos((2.0 * q + 1.0) * 3.14159265358979323846 / (2.0 * P));
}
__device__ __forceinline__ double cheb_bary(int q) {
    return ((q & 1) ? -1.0 : 1.0) * sin((2.0 * q + 1.0) * 3.14159265358979323846 / (2.0 * FMM_P));
}
// Per batch: the problems that use the FMM, their trees, and per-leaf interaction lists.
// Problem q (in FMM numbering) owns boxes [box_off[q], box_off[q+1]) in heap order over its
// leaves (level h has 2^h boxes; box (h, i) covers leaves [i 2^(H-h), (i+1) 2^(H-h))), and
// leaves [leaf_off[q], leaf_off[q+1]).
struct FmmArgs {
    const int64_t *off;
    int leaf;                 // poles per leaf
    double sep;               // separation ratio for the far field (times the box's width)
    double sep_loc;           // separation from the target interval, times its width, of the
                              // sources that enter a target leaf's local expansion
    const int32_t *fmm_prob;  // [nfmm] batch problem index
    const int32_t *fmm_of;    // [nprob] FMM index of a problem, -1 for direct
    const int32_t *box_off;   // [nfmm + 1]
    const int32_t *leaf_off;  // [nfmm + 1]
    const int32_t *height;    // [nfmm] tree height H (levels 0..H)
    const double2 *dw;        // (d_j, w_j) of the batch (from validation); .x alone for geometry
    const double *pos;        // when set, the points' positions (instead of dw's .x)
    const double *tail;       // [nprob] bound of the last root above d_{n-1}; nullptr: taken
    const double *teta;       // from the last root itself (its gap and origin; the poles are
    const int32_t *torg;      // pos)
    const int32_t *status;
    int32_t *used;            // [nboxes] == gen if some target leaf of the current lists lists
                              // the box as far field
    int gen;                  // the current lists' number: the lists kernel tags the boxes it
                              // uses with it, so no pass clears the flags between builds
    double2 *eq;              // [boxes][FMM_P] equivalent sources (node, weight)
    int32_t *near_lo, *near_hi;   // [leaves][FMM_NEAR_MAX] pole ranges: runs of adjacent near leaves
    int32_t *near_lf;             // [leaves][FMM_NEAR_MAX] 1: the range lies sep_loc target widths
                                  // (and a tile of indices) from the target interval, so its
                                  // poles enter the local expansion instead of the solver's
                                  // direct sums (the other consumers sum every near range)
    int32_t *far_l, *far_r;       // [leaves][FMM_FAR_MAX] far box ids (global)
    int32_t *cnt;             // [leaves][3] counts (near, far left, far right); -1 = direct
    // Far boxes also separated from the whole target interval (by sep_loc times its width)
    // enter the leaf's local expansion instead of being summed per root and iteration.
    int32_t *far_ld, *far_rd;       // [leaves][FMM_FAR_MAX] the far boxes summed directly
                                    // from the front, those in the expansion from the back
    int32_t *cntd;                  // [leaves][2] counts of the direct ones (left, right)
    double2 *loc_ab;          // [leaves] (centre, half-width) of the target interval
    double *loc;              // [leaves][FMM_LOC] Chebyshev coefficients on that interval
    int nboxes, nleaves;
    const int32_t *box_fmm;   // [nboxes] owning FMM problem of each box
    const int32_t *leaf_fmm;  // [nleaves] owning FMM problem of each leaf
    const int32_t *leaf_box;  // [nleaves] global box id of each leaf
    const int32_t *upper_box; // [nupper] global ids of the boxes above the leaves that hold
                              // poles, the largest (most leaves below) first
    int nupper;
    // Small upper boxes share a wavefront or a workgroup: of the first upper_cls[c] boxes none has
    // 2^(6-c) leaves or fewer (c = 0 .. 5; with c = 0 those of more than 64)
    int upper_cls[7];         // ([6]: nupper)
    // the eigenvector-side sources of the upper boxes in parts of at most FMMV_PART_PTS
    // points: items (box, part, parts, partial slot or -1), largest boxes first; the boxes
    // cut into several parts (box, first slot) and their partial weights
    const int4 *upper_item;   // [nupper_item]
    int nupper_item;
    int nitem_big;            // those of boxes with more than 4 leaves (the first ones)
    const int2 *split_box;    // [nsplit]
    int nsplit;
    double *vpart;            // [slots][column groups][FMM_P][FMMV_MAX_M]
    // targets of the lists: nullptr, the roots of the solver (a target leaf's roots lie in
    // [d_first, d_next]); else the positions of the target points themselves (the poles, for
    // sums over the roots), a leaf spanning [tpos[first], tpos[last]]
    const double *tpos;
};

// interaction lists of one set of targets (see FmmArgs) and the number of their last build
struct FmmLists {
    int32_t *near_lo = nullptr, *near_hi = nullptr, *near_lf = nullptr;
    int32_t *far_l = nullptr, *far_r = nullptr, *far_ld = nullptr, *far_rd = nullptr;
    int32_t *cnt = nullptr, *cntd = nullptr, *used = nullptr;
    double2 *loc_ab = nullptr;
    int gen = 0;
};

// Host side: the FMM layout of one batch for one leaf size.  The device arrays, those
// of the layout and those written on every call, are owned here.
struct FmmPlan {
    int leaf = 0;
    int crossover = 0;               // problems with n >= crossover use the FMM
    int nfmm = 0, nboxes = 0, nleaves = 0;
    int max_dir = 0;                 // most poles of a problem that does not use the FMM
    int lds_chunk = 64;              // roots per work item of the direct solver in LDS
    std::vector<int32_t> fmm_prob_h, fmm_of_h, box_off_h, leaf_off_h;
    int32_t *fmm_prob = nullptr, *fmm_of = nullptr, *box_off = nullptr, *leaf_off = nullptr;
    int32_t *height = nullptr, *box_fmm = nullptr, *leaf_fmm = nullptr;
    int32_t *leaf_box = nullptr, *upper_box = nullptr;
    int nupper = 0;
    int4 *upper_item = nullptr;
    int2 *split_box = nullptr;
    int nupper_item = 0, nitem_big = 0, nsplit = 0, nslot = 0;
    int upper_cls[7] = {0};          // see FmmArgs
    double2 *eq = nullptr;           // per-call arrays (fmm_arrays)
    double *loc = nullptr, *vnode = nullptr, *vcen = nullptr;
    double *vw[2] = {nullptr}, *vpart[2] = {nullptr};  // passes of up to 16 columns; wider ones
    double2 *lgeo = nullptr;
    double *lmom = nullptr;
    FmmLists own;                    // lists of the poles' targets
    FmmLists roots;                  // of the sums over the roots (Y = Qhat X), kept apart from
                                     // the solver's, which later calls on the same poles reuse
    // work items: 64-root pieces of the target leaves (a piece never crosses a leaf)
    int sub = TILE;                    // roots per work item
    int nitems = 0;
    int split = 1;                     // wavefronts per work item (they share its lists)
    std::vector<int32_t> item_off_h;   // FMM problem q owns items [item_off[q], item_off[q+1])
    Tile *leaf_lpt = nullptr;          // work items, longest problems first
    Tile *leaf_nat = nullptr;          // ... in problem order
    // the solver's work items: ssub roots of a leaf, shared by ssplit wavefronts (the solver in LDS
    // gives each its own roots, the ablations' its share of every root's sources)
    int ssub = TILE;
    int snitems = 0;
    int ssplit = 1;
    std::vector<int32_t> sitem_off_h;
    Tile *sitem_lpt = nullptr;
    Tile *sitem_nat = nullptr;
    // direct chunks of the other problems, by cut length (those in use)
    Tile *dir_lpt[kNumChunks] = {nullptr};
    int32_t dir_count[kNumChunks] = {0};
    bool dir_built[kNumChunks] = {false};
    void *mem = nullptr;               // the arrays above that hold the layout
    void *work = nullptr;              // the per-call arrays
    size_t work_cap = 0;
    std::vector<void *> allocs;        // direct chunks added later
};

// Eigenvector-side FMM (Sec. 4.3-4.4 with local shifting): sums over the poles i of a
// problem for every root j, sum_i src_i,c K(d_i - lambda_j), with K = 1/t (the apply
// Y = Qhat^T X: src = zhat_i X_i,c, scaled by b_j) or K = 1/t^2 (b: src = zhat_i^2);
// with trans = 0, sums over the roots j for every pole i, sum_j src_j,c / (d_i - lambda_j)
// (the apply Y = Qhat X: src = b_j X_j,c, scaled by zhat_i), sources at the roots.
struct FmmVec {
    int m;                    // weight columns (<= FMMV_MAX_PASS), in groups of FMMV_MAX_M
    int kern;                 // 1: 1/t, 2: 1/t^2; 3 and 4: the adjoint's sums over the poles and
                              // over the roots (several kernels of two and three columns)
    int trans;                // 1: sums over the poles (targets the roots); 0: over the roots
                              // (source positions lambda_j = d_{K_j} + eta_j, written by
                              // launch_fmmv_pos)
    // The sources' weights are read from X itself, src_s,c = scale_s X_s,c (kern 2: scale_s^2;
    // scale: zhat, or b for trans 0): X is column-major, so 64 sources of a column are one
    // 512-byte run, and no packed copy of it has to be written and read back
    const double *X;
    int64_t ldx;
    const double *scale;
    double *vnode;            // [boxes][FMM_P] equivalent source nodes
    double *vcen;             // when set (the adjoint), [boxes] their boxes' centres, and the nodes
                              // are held as offsets from those
    double *vw;               // [boxes][FMM_P][m] equivalent source weights
    const double *d;          // poles
    const int32_t *origin;    // roots' origins (local indices)
    const double *eta;        // roots' offsets
    const double2 *ke;        // trans 0: (d_{K_j}, eta_j) per root (launch_fmmv_pos)
    const double *post;       // kern 1: per-root scale (b); unused for kern 2
    double *Y;                // kern 1: output columns, ld ldy
    int64_t ldy;
    double *bout;             // kern 2: b_j = (sum)^(-1/2)
    int fuse_b;               // kern 1 on the MFMA: the last of the m weight columns is zhat^2;
                              // the evaluation forms b from it with the kernel 1/t^2, writes
                              // it to bout and scales the other m - 1 columns by it
    int expand;               // VALU evaluation: far boxes through the targets' interval (set
                              // by launch_fmmv_eval)
    double sep_t;             // interval widths from which a far box goes through it (set there)
    const double *zh;         // fuse_b: zhat, for b's near terms (zhat / t)^2
    const double *u;          // kern 3: u (scale: z)
    const double4 *rk;        // kern 4: (d_K, eta, alpha, beta) per root
    const double *gk;         // ... and gamma
    unsigned long long *work; // kernel timing on: algorithmic flops of the launch (set by
                              // launch_fmmv_eval): (2m + 3) per near pole or far source of a
                              // root for kern 1, 6 for kern 2, plus the output scaling
};
constexpr int FMMV_MAX_M = 16;       // columns per group (the MFMA tile)
constexpr int FMMV_MAX_PASS = 64;    // columns per set of launches
constexpr int FMMV_PART_PTS = 512;   // points per part of an upper box's sources (2 chunks)

// Loewner far field (Sec. 4.3, eqs. lowner2 and logv with local shifting): for a far box B
// and a pole x outside it,
//     G_B(x) = sum_{j in B} log((lambda_j - x) / (d_j - x))
//            = sum_{k >= 1} (-1)^(k+1) M_k r^k / k,   r = hw / (c - x),
// with the box's centre c and half-width hw (its span covers its poles and roots) and the
// moments M_k = sum_j ((t_j + D_j)^k - t_j^k), t_j = (d_j - c) / hw, D_j = delta_j / hw,
// delta_j = lambda_j - d_j.  Every moment is a sum of terms proportional to delta_j, so no
// cancellation: P_1 = D, P_{k+1} = (t + D) P_k + D t^k.
constexpr int FMML_K = 28;  // moments per box (|r| <= 1/4 at separation 1.5: 0.25^28 ~ 1e-17)

struct FmmlArgs {
    double2 *pd;              // (d_j, delta_j) per entry (pole and its root's offset)
    double2 *geo;             // [boxes] (c, hw)
    double *mom;              // [boxes][FMML_K] coefficients (-1)^(k+1) M_k / k, k = 1 .. K
    // pack != 0: the leaves' launch packs its poles' (d_j, delta_j) into pd itself (when the lists
    // already exist, as the separate packing launch would)
    int pack;
    const double *d, *eta;
    const int32_t *origin;
};
hipError_t launch_fmml_moments(const FmmArgs &f, const FmmlArgs &l, hipStream_t s);

// per-entry packing for the FMM problems: launch_fmml_pack the (d_j, delta_j) pairs of the
// Loewner far field, launch_fmmv_pos the roots' positions and (d_K, eta)
struct FmmvPackArgs {
    const int64_t *off;
    const Tile *tiles;   // 64-entry tiles of the FMM problems
    int ntiles;
    const double *d, *eta;
    const int32_t *origin;
    double2 *pairs;
    double *pos;         // launch_fmmv_pos: lambda_j = d_{K_j} + eta_j
    double2 *ke;         // (d_{K_j}, eta_j) per root; Loewner packing: when every problem of
                         // the batch uses the FMM (else nullptr)
};
hipError_t launch_fmmv_pos(const FmmvPackArgs &a, hipStream_t s);
// Loewner far field: (d_j, delta_j) pairs and the last roots' offsets, then the products
hipError_t launch_fmml_pack(const FmmvPackArgs &a, hipStream_t s);
hipError_t launch_loewner_fmm(const VecArgs &a, const FmmArgs &f, const FmmlArgs &l, int split,
                              hipStream_t s);


hipError_t launch_fmm_build(const FmmArgs &f, hipStream_t s);
// interaction lists only (no secular equivalent sources)
hipError_t launch_fmm_lists(const FmmArgs &f, hipStream_t s);
hipError_t launch_fmmv_sources(const FmmArgs &f, const FmmVec &v, hipStream_t s);
hipError_t launch_fmmv_eval(const SolveArgs &items, const FmmArgs &f, const FmmVec &v, int split,
                            int num_cu, hipStream_t s);
hipError_t launch_secular_fmm(const SolveArgs &a, const FmmArgs &f, int split,
                              hipStream_t s);
// one pass of the adjoint (kern 3: the roots' sums over the poles, kern 4: the poles' over the
// roots) for the FMM problems
hipError_t launch_backward_fmm(const BwdArgs &a, const FmmArgs &f, const FmmVec &v, int split,
                               int num_cu, hipStream_t s);

}  // namespace sdc
