// fmm_vec.hip -- eigenvector-side triangular FMM on gfx950 (Sec. 4.3, "Structured
// eigenvectors via FMM with local shifting", and the Z-update of Alg. 3).
//
// For the roots j of a large problem the sums over its poles i
//     apply:  Y_j,c = b_j sum_i r_ij (zhat_i X_i,c)        (Y = Qhat^T X, eqs. eigvecs, qk)
//     b:      b_j   = (sum_i zhat_i^2 r_ij^2)^(-1/2)      (eq. b)
// with r_ij = 1/(d_i - lambda_j) are evaluated on the same pole tree and interaction
// lists as the secular sums: near leaves directly in the shifted form
// (d_i - d_{K_j}) - eta_j, far boxes through equivalent sources in lambda-form.  The
// equivalent sources of a box are its Chebyshev nodes and the weights
// W_q,c = sum_{i in box} src_i,c L_q(d_i), one column per right-hand side.  Plain sums
// need no psi/phi split, but the lists are the directional ones of the solver and the
// near field keeps the local shifting, as the paper prescribes for these products.
#include "fmm_far.h"

namespace sdc {

typedef double v4d_f __attribute__((ext_vector_type(4)));

// compile-time flags for generic lambdas
struct fv_true { static constexpr bool value = true; };
struct fv_false { static constexpr bool value = false; };


// lambda_j = d_{K_j} + eta_j, the positions of the sums over the roots, and (d_{K_j}, eta_j)
// for their near sources; one lane per root
__global__ __launch_bounds__(64) void k_fmmv_pos(FmmvPackArgs a) {
    const Tile t = a.tiles[blockIdx.x];
    const int64_t base = a.off[t.prob];
    const int n = (int)(a.off[t.prob + 1] - base);
    const int j = t.row0 + lane_id();
    if (j >= n) return;
    const double dK = a.d[base + clamp_idx(a.origin[base + j], n)], e = a.eta[base + j];
    a.pos[base + j] = dK + e;
    a.ke[base + j] = make_double2(dK, e);
}

// Equivalent sources, one workgroup (256 threads) per box, in two launches: LEAVES = true
// compresses every leaf box from its poles; LEAVES = false compresses every used box above
// the leaves from the equivalent sources of its leaves (16 per leaf instead of up to
// n/4 poles: the far field of a leaf's sources equals that of its poles to the
// interpolation accuracy, and the box's nodes interpolate it again).  Points are taken a
// chunk at a time: each of the chunk's threads forms the 16 Lagrange values of one point in
// LDS, then W_q,c += sum_k L_q(x_k) w_k,c over the chunk runs on the FP64 MFMA, its weight
// operands loaded straight from memory before the Lagrange values are formed: a leaf's from
// the columns of X (each lane the 16 consecutive points of one column that it feeds), an
// upper box's from the leaves' weights (point-major: the 4 points x 16 columns of one step
// are 128-byte runs).  blockIdx.y is the group of FMMV_MAX_M columns.  Up to four columns (b,
// the adjoint) are added on the VALU instead: lane (node, quarter of the points), the weights
// from the lanes that loaded them; a 16-column step costs as much as 16 columns of that
// (boxes and leaves of a level of 4096 problems, b: 780 -> 690 us; with boxes of at most four
// leaves on a wavefront instead of a workgroup 450).
template <int C>
__device__ __forceinline__ double row_lane(double v) {  // lane C of each row of 16
    return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), 0x150 + C, 0xf, 0xf, true),
                            __builtin_amdgcn_mov_dpp(__double2loint(v), 0x150 + C, 0xf, 0xf, true));
}
template <bool LEAVES, bool FEW>
__global__ __launch_bounds__(LEAVES ? 64 : 256, LEAVES ? 1 : 4) void k_fmmv_sources(FmmArgs f, FmmVec v) {
    // leaves: one wavefront, 64 points per chunk; upper boxes (up to 16 sources per leaf
    // below): four wavefronts, 256 points per chunk
    constexpr int NW = LEAVES ? 1 : 4;
    constexpr int FV_CHUNK = 64 * NW;
    __shared__ double Lq[FV_CHUNK][FMM_P + 1];
    // leaves in the first launch; in the second the parts of the upper boxes with poles
    // (used ones): (box, part, parts, partial slot); boxes of at most 4 leaves, 64 points, four to
    // a workgroup, a wavefront each (`one`)
    const bool one = LEAVES || (int)blockIdx.x >= f.nitem_big;
    const int wv = LEAVES ? 0 : wave_uniform((int)(threadIdx.x / WAVE));
    const int item = !LEAVES && one ? f.nitem_big + ((int)blockIdx.x - f.nitem_big) * 4 + wv
                                    : (int)blockIdx.x;
    if (!LEAVES && item >= f.nupper_item) return;
    const int4 it = LEAVES ? make_int4(f.leaf_box[item], 0, 1, -1) : f.upper_item[item];
    const int g = it.x;
    if (!LEAVES && f.used[g] != f.gen) return;
    const int qf = f.box_fmm[g];
    const int p = f.fmm_prob[qf];
    const int64_t base = f.off[p];
    const int n = (int)(f.off[p + 1] - base);
    const int hidx = g - f.box_off[qf];
    const int H = f.height[qf];
    int h = 0;
    while ((2 << h) - 1 <= hidx) ++h;
    if (f.status[p] & ~SUPERDC_ST_NOCONV) return;
    const int bi = hidx - ((1 << h) - 1);
    const int64_t span = (int64_t)f.leaf << (H - h);
    const int lo = (int)min((int64_t)n, bi * span), hi = (int)min((int64_t)n, (bi + 1) * span);
    if (lo >= hi) return;  // empty box (never listed)
    const int lane = lane_id();
    const int row0 = wv * WAVE;                    // the wavefront's rows of Lq
    const int tid = one ? lane : (int)threadIdx.x; // thread of the box
    const int chunk = one ? WAVE : FV_CHUNK;
    auto sync = [&]() {
        if (one) wave_sync();
        else __syncthreads();
    };
    const int m = v.m;
    const int g0 = blockIdx.y * FMMV_MAX_M;       // this group's columns [g0, g0 + mg)
    const int mg = min(FMMV_MAX_M, m - g0);
    const int mx = v.kern >= 2 ? 0 : min(mg, m - v.fuse_b - g0);  // those that are X's
    const double *d = f.pos + base;               // the points' positions (poles, or roots)
    const double *sc = v.scale + base;
    const double *X = v.kern >= 2 ? nullptr : v.X + base + (int64_t)g0 * v.ldx;
    // column c of the group: scale X, or scale^2 for the b sum's; the adjoint's z^2 and u z of a
    // pole (kern 3), alpha, beta and gamma of a root (kern 4, no scale)
    auto column = [&](int c, int &stride) -> const double * {
        stride = v.kern == 4 && c < 2 ? 4 : 1;
        if (v.kern == 4)
            return c < 2 ? reinterpret_cast<const double *>(v.rk + base) + 2 + c : v.gk + base;
        if (c < mx) return X + (int64_t)c * v.ldx;
        return v.kern == 3 && c == 1 ? v.u + base : sc;
    };
    const double a = d[lo], b = d[hi - 1];
    const double cc = 0.5 * (a + b), hw = 0.5 * (b - a);
    // the adjoint's nodes are offsets from cc (rounded as positions, they would lie eps |d| off
    // their place, which shows at a distance of 64 poles), its points' from the roots' own pairs
    const bool rel = v.vcen != nullptr;
    const double nc = rel ? 0.0 : cc;
    const double lim = rel ? 1.0 + 0x1p-20 : 1.0;  // the ends were rounded as positions
    auto point = [&](int k) {  // pole or root k of a leaf, from cc
        if (v.kern != 4) return d[k] - cc;
        const double4 r = v.rk[base + k];
        return (r.x - cc) + r.y;
    };
    double *node = v.vnode + (int64_t)g * FMM_P;
    double *w = v.vw + (int64_t)g * FMM_P * m + g0;
    if (LEAVES && hi - lo <= FMM_P) {  // few poles: they are their own equivalent sources
        if (tid < FMM_P) {
            const bool in = lo + tid < hi;
            if (blockIdx.y == 0) {
                node[tid] = !in ? nc : rel ? point(lo + tid) : d[lo + tid];
                if (rel && tid == 0) v.vcen[g] = cc;
            }
            for (int c = 0; c < mg; ++c) {
                int st;
                const double *wc = column(c, st);
                w[tid * m + c] = !in ? 0.0 : v.kern == 4 ? wc[(lo + tid) * st] : sc[lo + tid] * wc[lo + tid];
            }
        }
        return;
    }
    // the points: poles of a leaf, or the sources of the box's leaves
    const int leaf0 = (1 << H) - 1 + bi * (1 << (H - h));      // heap index of the first leaf
    const int nleaf = (int)((hi - lo + f.leaf - 1) / f.leaf);  // leaves with poles
    const int npts = LEAVES ? hi - lo : nleaf * FMM_P;
    // this part's points [pk0, pk1)
    const int pk0 = LEAVES ? 0 : min(npts, it.y * FMMV_PART_PTS);
    const int pk1 = LEAVES ? npts : (it.z == 1 ? npts : min(npts, pk0 + FMMV_PART_PTS));
    double tq[FMM_P], lam[FMM_P];
#pragma unroll
    for (int r = 0; r < FMM_P; ++r) {
        tq[r] = cheb_node(r);
        lam[r] = cheb_bary(r);
    }
    const double ihw = 1.0 / hw;
    v4d_f acc = v4d_f{0.0, 0.0, 0.0, 0.0};  // FEW: columns 0 .. 3 of node lane % 16
    // an upper box's points' weights, m per point: the sources of the box's leaves
    const double *wsrc = v.vw + (int64_t)(f.box_off[qf] + leaf0) * FMM_P * m + g0;
    for (int k0 = pk0; k0 < pk1; k0 += chunk) {
        // W (16 nodes x 16 columns) += L (16 x chunk) S (chunk x 16) on the FP64 MFMA: each
        // wavefront takes 64 points of the chunk, 4 per step (A lane l = L[l % 16][point],
        // B lane l = S[point][l % 16]): step st of lane l takes point 16 (l / 16) + st for a
        // leaf, 4 st + l / 16 for an upper box
        double bs[16];
        const int c = lane & 15;
        if (LEAVES) {
            const int p0 = k0 + 16 * (lane >> 4);
            int stride;
            const double *xc = column(min(c, mg - 1), stride) + (int64_t)(lo + p0) * stride;
            const double *sp = sc + lo + p0;
            if (c < mg && p0 + 16 <= pk1) {
                if (v.kern == 4) {
#pragma unroll
                    for (int st = 0; st < 16; ++st) bs[st] = xc[st * stride];
                } else {
#pragma unroll
                    for (int st = 0; st < 16; ++st) bs[st] = sp[st] * xc[st];
                }
            } else {
#pragma unroll
                for (int st = 0; st < 16; ++st)
                    bs[st] = p0 + st < pk1 && c < mg
                                 ? (v.kern == 4 ? 1.0 : sp[st]) * xc[st * stride] : 0.0;
            }
        } else {
#pragma unroll
            for (int st = 0; st < 16; ++st) {
                const int pt = k0 + (one ? 0 : row0) + 4 * st + (lane >> 4);
                bs[st] = pt < pk1 && c < mg ? wsrc[(int64_t)pt * m + c] : 0.0;
            }
        }
        const int k = k0 + tid;
        if (k < pk1) {
            double x;  // the point from cc
            if (LEAVES) {
                x = point(lo + k);
            } else {
                const int64_t b0 = f.box_off[qf] + leaf0;
                x = v.vnode[b0 * FMM_P + k];
                x = rel ? (v.vcen[b0 + k / FMM_P] - cc) + x : x - cc;
            }
            // (a box of one position: ihw is infinite, and every node lies there)
            const double t = fmin(lim, fmax(-lim, x * ihw));
            int hit = -1;
            double inv[FMM_P], den = 0.0;
#pragma unroll
            for (int r = 0; r < FMM_P; ++r) {
                const double dlt = t - tq[r];
                if (dlt == 0.0) hit = r;
                inv[r] = lam[r] * rcp_nr(dlt);
                den += inv[r];
            }
            const double iden = 1.0 / den;
#pragma unroll
            for (int r = 0; r < FMM_P; ++r)
                Lq[row0 + lane][r] = hit >= 0 ? (r == hit ? 1.0 : 0.0) : inv[r] * iden;
        } else {
#pragma unroll
            for (int r = 0; r < FMM_P; ++r) Lq[row0 + lane][r] = 0.0;
        }
        sync();
#pragma unroll
        for (int st = 0; st < 16; ++st) {
            const int kk = LEAVES ? 16 * (lane >> 4) + st : row0 + 4 * st + (lane >> 4);
            const double l = Lq[kk][lane & 15];
            if (FEW) {
                acc[0] = __builtin_fma(l, row_lane<0>(bs[st]), acc[0]);
                if (mg > 1) acc[1] = __builtin_fma(l, row_lane<1>(bs[st]), acc[1]);
                if (mg > 2) acc[2] = __builtin_fma(l, row_lane<2>(bs[st]), acc[2]);
                if (mg > 3) acc[3] = __builtin_fma(l, row_lane<3>(bs[st]), acc[3]);
            } else {
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(l, bs[st], acc, 0, 0, 0);
            }
        }
        sync();
    }
    double *red = &Lq[0][0];
    if (FEW) {
        // the four quarters' sums, column c of node q to lane 16 c + q, then the wavefronts'
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            acc[c] += __shfl_xor(acc[c], 16);
            acc[c] += __shfl_xor(acc[c], 32);
        }
        const int qn = lane & 15, cn = lane >> 4;
        double s2 = cn < 2 ? (cn ? acc[1] : acc[0]) : (cn == 2 ? acc[2] : acc[3]);
        if (!one) {
            if (wv > 0) red[(wv - 1) * WAVE + lane] = s2;
            __syncthreads();
        }
        if (one || wv == 0) {
            if (!one)
                for (int u = 0; u < NW - 1; ++u) s2 += red[u * WAVE + lane];
            if (it.w >= 0)
                f.vpart[(((int64_t)it.w * gridDim.y + blockIdx.y) * FMM_P + qn) * FMMV_MAX_M + cn] = s2;
            else if (cn < mg)
                w[qn * m + cn] = s2;
        }
        if (it.y == 0 && blockIdx.y == 0 && tid < FMM_P) {
            node[tid] = nc + hw * tq[tid];
            if (rel && tid == 0) v.vcen[g] = cc;
        }
        return;
    }
    mfma_drain();
    // the four wavefronts' partial W added in wavefront order (through the staging LDS);
    // accumulator r of lane l holds W[4 r + l / 16][l % 16]
    if (!one && wv > 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r) red[((wv - 1) * 4 + r) * WAVE + lane] = acc[r];
    }
    if (!one) __syncthreads();
    if (one || wv == 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            double s2 = acc[r];
            for (int u = 0; u < (one ? 0 : NW - 1); ++u) s2 += red[(u * 4 + r) * WAVE + lane];
            const int qn = 4 * r + (lane >> 4), cn = lane & 15;
            if (it.w >= 0)  // one part of several: its partial weights, summed afterwards
                f.vpart[(((int64_t)it.w * gridDim.y + blockIdx.y) * FMM_P + qn) * FMMV_MAX_M + cn] = s2;
            else if (cn < mg)
                w[qn * m + cn] = s2;
        }
    }
    if (it.y == 0 && blockIdx.y == 0 && tid < FMM_P) node[tid] = cc + hw * tq[tid];
}

// The weights of the upper boxes computed in several parts: the parts' partial weights
// added in part order.  One workgroup per such box and column group, thread (node q, column c).
__global__ __launch_bounds__(FMM_P * FMMV_MAX_M) void k_fmmv_sources_sum(FmmArgs f, FmmVec v) {
    const int2 sb = f.split_box[blockIdx.x];
    const int g = sb.x;
    if (f.used[g] != f.gen) return;
    const int qf = f.box_fmm[g];
    const int p = f.fmm_prob[qf];
    if (f.status[p] & ~SUPERDC_ST_NOCONV) return;
    const int n = (int)(f.off[p + 1] - f.off[p]);
    const int hidx = g - f.box_off[qf];
    const int H = f.height[qf];
    int h = 0;
    while ((2 << h) - 1 <= hidx) ++h;
    const int bi = hidx - ((1 << h) - 1);
    const int64_t span = (int64_t)f.leaf << (H - h);
    const int lo = (int)min((int64_t)n, bi * span), hi = (int)min((int64_t)n, (bi + 1) * span);
    const int nleaf = (hi - lo + f.leaf - 1) / f.leaf;
    const int parts = (nleaf * FMM_P + FMMV_PART_PTS - 1) / FMMV_PART_PTS;
    const int q = threadIdx.x / FMMV_MAX_M, c = threadIdx.x % FMMV_MAX_M;
    const int gy = blockIdx.y, col = gy * FMMV_MAX_M + c;
    if (col >= v.m) return;
    double s = 0.0;
    for (int u = 0; u < parts; ++u)
        s += f.vpart[(((int64_t)(sb.y + u) * gridDim.y + gy) * FMM_P + q) * FMMV_MAX_M + c];
    v.vw[((int64_t)g * FMM_P + q) * v.m + col] = s;
}

// Evaluation at the roots: work items are 64-root pieces of the target leaves; S
// wavefronts per item split the near ranges and the far boxes, and their partial sums are
// added in wavefront order.  NC columns, an accumulator each per lane.  In the expansion a lane holds
// node lane % 16 and every fourth source of a box.
template <int NC>
struct FvEvalShared {
    int fbox[2 * FMM_FAR_MAX];
    int nexp;
    double gsum[8][NC][FMM_P];  // far field at the nodes, per wavefront (at most 8)
};

template <int KERN, int NC>
__device__ void fmmv_item(const SolveArgs &it, const FmmArgs &f, const FmmVec &v, Tile t,
                          FvEvalShared<NC> &sh, double *red) {
    const int p = t.prob;
    const int64_t base = it.off[p];
    const int n = (int)(it.off[p + 1] - base);
    const int lane = lane_id();
    const int S = blockDim.x / WAVE, wv = wave_uniform((int)(threadIdx.x / WAVE));
    const int j = t.row0 + lane;
    const bool active = j < n;
    constexpr int m = NC;  // the columns
    if (f.status[p] & ~SUPERDC_ST_NOCONV) {
        if (active && wv == 0) {
            const double nan = __builtin_nan("");
            if (KERN == 1)
                for (int c = 0; c < m; ++c) v.Y[base + j + (int64_t)c * v.ldy] = nan;
            else
                v.bout[base + j] = nan;
        }
        return;
    }
    const int jj = active ? j : n - 1;
    const double dK = v.d[base + clamp_idx(v.origin[base + jj], n)];
    const double eta = v.eta[base + jj];
    const double x = dK + eta;
    const int qf = f.fmm_of[p];
    const int L = wave_uniform(f.leaf_off[qf] + t.row0 / f.leaf);
    int nn = wave_uniform(f.cnt[3 * (int64_t)L]);
    const int nl = wave_uniform(f.cnt[3 * (int64_t)L + 1]);
    const int nr = wave_uniform(f.cnt[3 * (int64_t)L + 2]);
    const const_double_ptr dd = as_const(v.d + base);
    const const_double_ptr sc = as_const(v.scale + base);  // zhat
    const const_double_ptr X = as_const(KERN == 1 ? v.X + base : v.d + base);
    double acc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[c] = 0.0;
    int64_t ent = 0;  // pole or source entries this wavefront sums per root (kernel timing)
    // one near range [lo, hi) of poles, shifted form, two Newton steps; two poles share one
    // reciprocal (it issues at a quarter of the FMA rate), as in the direct b kernel, while
    // every |t| of the wavefront's roots lies inside [2^-300, 2^300]: the smallest is |eta| (a
    // root's origin is its nearest pole), the largest at an end of the problem (b of a level of
    // 4096 problems: 1.54 -> 1.45 ms)
    const bool pair = __ballot(fabs(eta) < 0x1p-300 ||
                               fmax(fabs((dd[0] - dK) - eta), fabs((dd[n - 1] - dK) - eta)) > 0x1p300) == 0ull;
    auto near = [&](int lo, int hi) {
        ent += hi > lo ? hi - lo : 0;
        int i = lo;
        if (pair) {
#pragma unroll 2
            for (; i + 2 <= hi; i += 2) {
                const double t0 = (dd[i] - dK) - eta, t1 = (dd[i + 1] - dK) - eta;
                const double R = rcp_nr(t0 * t1);
                // scale_i / t_i, divided before any further product: scale times t can leave the
                // range where the quotient does not
                const double q0 = sc[i] * t1 * R, q1 = sc[i + 1] * t0 * R;
                if (KERN == 1) {
#pragma unroll
                    for (int c = 0; c < NC; ++c) {
                        const const_double_ptr x = X + i + (int64_t)c * v.ldx;
                        acc[c] = __builtin_fma(q0, x[0], __builtin_fma(q1, x[1], acc[c]));
                    }
                } else {
                    acc[0] = __builtin_fma(q0, q0, __builtin_fma(q1, q1, acc[0]));
                }
            }
        }
        for (; i < hi; ++i) {
            const double r = rcp_nr((dd[i] - dK) - eta);
            const double qv = r * sc[i];
            if (KERN == 1) {
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    acc[c] = __builtin_fma(qv, X[i + (int64_t)c * v.ldx], acc[c]);
            } else {  // (zhat / t)^2, squared after the division (r^2 zhat^2 can leave range)
                acc[0] = __builtin_fma(qv, qv, acc[0]);
            }
        }
    };
    if (nn < 0) {  // lists overflowed: every pole directly, split over the wavefronts
        near(wave_uniform((int)(((int64_t)n * wv) / S)), wave_uniform((int)(((int64_t)n * (wv + 1)) / S)));
    } else {
        for (int e = 0; e < nn; ++e) {
            const int lo0 = wave_uniform(f.near_lo[(int64_t)L * FMM_NEAR_MAX + e]);
            const int hi0 = wave_uniform(f.near_hi[(int64_t)L * FMM_NEAR_MAX + e]);
            near(lo0 + (int)(((int64_t)(hi0 - lo0) * wv) / S),
                 lo0 + (int)(((int64_t)(hi0 - lo0) * (wv + 1)) / S));
        }
        // far boxes of both sides, lambda-form, one Newton step
        const double2 iv = fv_interval(v, base, n, t.row0, min(t.row0 + WAVE, n) - 1);
        if (wv == 0) {
            const int k = fv_split_far(f, v, L, nl, nr, iv, v.expand != 0, sh.fbox);
            if (lane == 0) sh.nexp = k;
        }
        __syncthreads();
        const int ne = wave_uniform(sh.nexp);
        if (ne > 0) {
            const double off = iv.y * FV_NODE[lane & 15];
            double gs[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) gs[c] = 0.0;
            for (int e = wv; e < ne; e += S) {
                const int64_t g = sh.fbox[2 * FMM_FAR_MAX - 1 - e];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int64_t sq = g * FMM_P + 4 * k + (lane >> 4);
                    const double r = rcp_nr1((v.vnode[sq] - iv.x) - off);
                    if (KERN == 1) {
#pragma unroll
                        for (int c = 0; c < NC; ++c)
                            gs[c] = __builtin_fma(r, v.vw[sq * m + c], gs[c]);
                    } else {
                        gs[0] = __builtin_fma(r * r, v.vw[sq], gs[0]);
                    }
                }
            }
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                gs[c] += __shfl_xor(gs[c], 16);
                gs[c] += __shfl_xor(gs[c], 32);
                if (lane < FMM_P) sh.gsum[wv][c][lane] = gs[c];
            }
            wave_sync();
            // this wavefront's share of the far field at the targets
            const double tau = ((dK - iv.x) + eta) / iv.y;
            double num[NC], den = 0.0;
#pragma unroll
            for (int c = 0; c < NC; ++c) num[c] = 0.0;
            for (int q = 0; q < FMM_P; ++q) {
                const double dl = tau - FV_NODE[q];
                // a target on a node: that node's term outweighs the others
                const double b = FV_BARY[q] * rcp_nr(dl == 0.0 ? 0x1p-200 : dl);
                den += b;
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    num[c] = __builtin_fma(b, sh.gsum[wv][c][q], num[c]);
            }
            const double iden = 1.0 / den;
#pragma unroll
            for (int c = 0; c < NC; ++c) acc[c] = __builtin_fma(num[c], iden, acc[c]);
            if (v.work && lane == 0) {  // kernel timing: the expansion's algorithmic flops
                const unsigned long long per = KERN == 1 ? 2 * (unsigned long long)m + 3 : 6;
                atomicAdd(v.work, (unsigned long long)((ne - wv + S - 1) / S) * FMM_P * FMM_P * per +
                                      (unsigned long long)(WAVE * FMM_P * 2 * m));
            }
        }
        for (int e = wv; e < nl + nr - ne; e += S) {
            const int g = wave_uniform(sh.fbox[e]);
            const const_double_ptr nd = as_const(v.vnode + (int64_t)g * FMM_P);
            const const_double_ptr ww = as_const(v.vw + (int64_t)g * FMM_P * m);
            ent += FMM_P;
#pragma unroll 4
            for (int q = 0; q < FMM_P; ++q) {
                const double r = rcp_nr1(nd[q] - x);
                if (KERN == 1) {
#pragma unroll
                    for (int c = 0; c < NC; ++c)
                        acc[c] = __builtin_fma(r, ww[q * m + c], acc[c]);
                } else {
                    acc[0] = __builtin_fma(r * r, ww[q], acc[0]);
                }
            }
        }
    }
    const unsigned long long rows = (unsigned long long)__popcll(__ballot(active));
    if (v.work && lane == 0) {  // kernel timing: algorithmic flops of this wavefront's share
        const unsigned long long per = KERN == 1 ? 2 * (unsigned long long)m + 3 : 6;
        atomicAdd(v.work, rows * (unsigned long long)ent * per +
                              (wv == 0 && KERN == 1 ? rows * (unsigned long long)m : 0));
    }
    if (S > 1) {
        if (wv > 0)
#pragma unroll
            for (int c = 0; c < NC; ++c) red[((wv - 1) * NC + c) * WAVE + lane] = acc[c];
        __syncthreads();
        if (wv == 0)
            for (int w = 1; w < S; ++w)
#pragma unroll
                for (int c = 0; c < NC; ++c) acc[c] += red[((w - 1) * NC + c) * WAVE + lane];
        __syncthreads();
    }
    if (active && wv == 0) {
        if (KERN == 1) {
            const double post = v.post[base + j];
#pragma unroll
            for (int c = 0; c < NC; ++c)
                v.Y[base + j + (int64_t)c * v.ldy] = post * acc[c];
        } else {
            v.bout[base + j] = 1.0 / sqrt(acc[0]);
        }
    }
}

// blockDim.x = 64 S; dynamic LDS: (S - 1) NC doubles per lane
template <int KERN, int NC>
__global__ __launch_bounds__(512) void k_fmmv_eval(SolveArgs it, FmmArgs f, FmmVec v) {
    extern __shared__ double red[];
    __shared__ FvEvalShared<NC> sh;
    fmmv_item<KERN, NC>(it, f, v, it.tiles[xcd_item()], sh, red);
}

// ---------------------------------------------------------------------------------------
// Y = Qhat^T X (or Qhat X, sums over the roots) through the FMM on MFMA: for a 64-row work
// item the near sources and the far boxes' equivalent sources form one gathered reduction
// dimension, and the product
//     Y_j,c = b_j sum_k 1/((s_k - d_{K_j}) - eta_j) W_k,c
// (s_k a pole or a Chebyshev node, W_k,c its weight) is the dense contraction of the direct
// apply: each wavefront generates its 16 x 4 slices of the Cauchy block and feeds
// v_mfma_f64_16x16x4f64.  Every source uses the shifted difference, never less accurate than
// the lambda-form.
//
// The bound is the FP64 pipe: on gfx950 the FP64 MFMA (72 cycles each, measured) and FP64 VALU
// instructions share it and do not overlap (two wavefronts of each on one SIMD took the sum of
// their times), so a step of 4 sources x 16 rows x 16 columns costs 72 cycles and about 36 for
// its Cauchy entries, and a 65536-root launch (1024 items, about 20 chunks each) 62 us.  What
// kept the kernel from it (it took 95 us) was waiting, so a chunk goes through two LDS buffers with one
// barrier, its loads issued before the previous chunk is multiplied and used only when it is
// stored; every lane loads (indices clamped to the chunk's own sources, padding set to zero
// at the store), so that the loads of a chunk are one run without branches; and the values
// loaded once per item are taken before the loop, since a first use inside it made the
// compiler wait there for the next chunk's loads as well: 80 us, and in a level of 4096 problems
// (16 columns) 4.08 -> 3.25 ms.  The far boxes go through the targets' interval (fv_split_far),
// which left 5 chunks and 41 boxes an item on average: 73 us, and 2.60 ms.  A launch with too few items to give every CU two workgroups
// gives each item TEAMS teams of four wavefronts, which take the chunks in turn and add their
// sums in team order (n = 1024, 16 items: 23 -> 12 us).
// ---------------------------------------------------------------------------------------
constexpr int FV_K = 64;            // sources per chunk
// Two blocks of 16 columns an item (one generates the Cauchy entries and builds the lists of both)
// from so many items per CU on.  Measured, one -> two blocks, us a launch, Q^T X: 64 columns of
// 65536 roots (8 a CU) 142 -> 126 (four blocks: 133, two workgroups a CU by LDS), of 16384 (2 a CU)
// 40.0 -> 38.5, 32 columns of 16384 (1 a CU) 27.3 -> 29.3.  With three blocks a quarter of the
// matrix work is padding: 48 columns, 2 a CU 32 -> 37.5, 8 a CU 110 -> 125, 64 a CU 685 -> 609.
constexpr int FV_WIDE_PER_CU = 2;
constexpr int FV_WIDE3_PER_CU = 32;
constexpr int FV_LD = FV_K + 4;     // LDS row: the 16 columns x 4 sources of a step fall on
                                    // different banks

// The chunks of an item (built once per item in LDS): near ranges in 64-source chunks, then
// the far boxes 4 at a time (64 equivalent sources).  x = 0: sources [y, y + z); x = 1: far
// boxes fbox[y .. y + z).
// (at most FMM_NEAR_MAX near leaves of at most 1024 poles, the largest leaf the options
// allow; a run of adjacent leaves has no more chunks than its leaves, since every leaf but
// a problem's last holds a multiple of 64 poles)
constexpr int FV_MAXCH = FMM_NEAR_MAX * (1024 / FV_K) + (2 * FMM_FAR_MAX + 3) / 4;

static_assert(FV_K * 16 == 4 * 256, "a chunk's 64 sources x 16 columns: four per thread");
static_assert(FMM_NEAR_MAX <= WAVE, "a lane per near range");

// A chunk's data on its way from memory to LDS, raw: masks and scales are applied at the
// store.  Near sources: thread t holds source t % 64 in columns t / 64 + 4 i (a wavefront
// reads 64 consecutive entries of a column of X) and its scale; far sources: source t / 16 of
// box i in column t % 16 (their weights are source-major: 16 threads read a source's row).
template <int NC>
struct FvStage {
    double2 sd;    // (first wavefront) source position and, with b formed beside the columns,
                   // zhat (near) or the weight of zhat^2 (far); TRANS 0: (d_K, eta) (near) or
                   // (node, 0) (far)
    double w[4 * NC];
    double sc;
};

template <int TRANS, bool FB, int NC>
__device__ __forceinline__ void fv_fetch(const FmmVec &v, int64_t base, const int *fbox, int4 ch,
                                         int tid, int g0, int mg, int mx, FvStage<NC> &st) {
    const int m = v.m;
    const bool first = wave_uniform(tid / WAVE) == 0;
    if (ch.x == 0) {
        const int64_t j = base + ch.y + min(tid & (FV_K - 1), ch.z - 1);
        const double *xs = v.X + j + (int64_t)g0 * v.ldx;
        st.sc = v.scale[j];
#pragma unroll
        for (int i = 0; i < 4 * NC; ++i)
            st.w[i] = xs[(int64_t)min(tid / FV_K + 4 * i, mx - 1) * v.ldx];
        if (first) {
            if (TRANS == 0) st.sd = v.ke[j];
            else st.sd = make_double2(v.d[j], FB ? v.zh[j] : 0.0);
        }
    } else {
        // far chunk: box i of the chunk holds its FMM_P = 16 sources r16
        const int r16 = tid >> 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t sq = (int64_t)fbox[ch.y + min(i, ch.z - 1)] * FMM_P + r16;
#pragma unroll
            for (int b = 0; b < NC; ++b)
                st.w[4 * b + i] = v.vw[sq * m + g0 + min(16 * b + (tid & 15), mg - 1)];
        }
        if (first) {
            const int64_t sq = (int64_t)fbox[ch.y + min(tid / FMM_P, ch.z - 1)] * FMM_P + tid % FMM_P;
            st.sd = make_double2(v.vnode[sq], FB ? v.vw[sq * m + m - 1] : 0.0);
        }
    }
}

// Padding (past a partial chunk's sources or the group's columns) is stored as weight zero at
// the position of one of the chunk's own sources.
template <bool FB, int NC>
__device__ __forceinline__ void fv_store(int4 ch, int tid, int mg, int mx, const FvStage<NC> &st,
                                         double *Xs, double2 *Sd) {
    const int cnt = ch.x == 0 ? ch.z : ch.z * FMM_P;
    if (ch.x == 0) {
        const int sl = tid & (FV_K - 1), c0 = tid / FV_K;
#pragma unroll
        for (int i = 0; i < 4 * NC; ++i)
            Xs[(c0 + 4 * i) * FV_LD + sl] =
                sl < ch.z && c0 + 4 * i < mx ? st.sc * st.w[i] : 0.0;
    } else {
        const int c = tid & 15, r16 = tid >> 4;
#pragma unroll
        for (int b = 0; b < NC; ++b)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                Xs[(16 * b + c) * FV_LD + r16 + 16 * i] =
                    i < ch.z && 16 * b + c < mg ? st.w[4 * b + i] : 0.0;
    }
    if (wave_uniform(tid / WAVE) == 0)
        Sd[tid] = make_double2(st.sd.x, FB && tid >= cnt ? 0.0 : st.sd.y);
}

template <int NC>
struct FvTeam {
    double Xs[2][16 * NC * FV_LD];
    double2 Sd[2][FV_K];
};

template <int TEAMS, int NC>
struct FvShared {
    FvTeam<NC> team[TEAMS];
    int4 ctab[FV_MAXCH];
    int fbox[2 * FMM_FAR_MAX];
    int nch, nexp;
    double node[FMM_P], bary[FMM_P];  // FV_NODE and FV_BARY (read by lane)
};

// gi: the group of NC blocks of FMMV_MAX_M columns of the pass.  FEW: the last block has one to three
// columns, which are as exact as fmmv_item's, that takes so few alone
template <int TRANS, bool FB, int TEAMS, int NC, bool FEW>
__device__ void fmmv_item_mfma(const SolveArgs &it, const FmmArgs &f, const FmmVec &v, Tile t,
                               int gi, FvShared<TEAMS, NC> &sh) {
    static_assert(NC == 1 || (TEAMS == 1 && !FB), "one block of columns for teams and b");
    const int p = t.prob;
    const int64_t base = it.off[p];
    const int n = (int)(it.off[p + 1] - base);
    const int lane = lane_id();
    const int wave = wave_uniform((int)(threadIdx.x / WAVE));
    const int tm = wave >> 2, wv = wave & 3;      // team, wavefront of the team
    const int tid = threadIdx.x & 255;            // thread of the team
    const int o0 = t.row0;
    const int g0 = gi * (NC * FMMV_MAX_M);
    const int mg = min(NC * FMMV_MAX_M, v.m - g0);  // columns of the group
    const int mo = mg - (FB ? 1 : 0);          // output columns
    if (f.status[p] & ~SUPERDC_ST_NOCONV) {
        const double nan = __builtin_nan("");
        for (int e = threadIdx.x; e < FV_K * mo; e += blockDim.x) {
            const int r = o0 + (e % FV_K), c = g0 + e / FV_K;
            if (r < n) v.Y[base + r + (int64_t)c * v.ldy] = nan;
        }
        if (FB && threadIdx.x < FV_K && o0 + (int)threadIdx.x < n)
            v.bout[base + o0 + threadIdx.x] = nan;
        return;
    }
    const int qf = f.fmm_of[p];
    const int L = wave_uniform(f.leaf_off[qf] + t.row0 / f.leaf);
    const int nn = wave_uniform(f.cnt[3 * (int64_t)L]);
    const bool direct = nn < 0;  // overflowed lists: every source, 64 at a time
    double2 iv = fv_interval(v, base, n, o0, min(o0 + FV_K, n) - 1);
    if (!direct) {
        if (wave == 0) {  // a lane per near range, its chunks after those of the lanes below
            const int nl = wave_uniform(f.cnt[3 * (int64_t)L + 1]);
            const int nr = wave_uniform(f.cnt[3 * (int64_t)L + 2]);
            int lo = 0, hi = 0;
            if (lane < nn) {
                lo = f.near_lo[(int64_t)L * FMM_NEAR_MAX + lane];
                hi = f.near_hi[(int64_t)L * FMM_NEAR_MAX + lane];
            }
            const int ne = fv_split_far(f, v, L, nl, nr, iv, TEAMS == 1, sh.fbox), nd = nl + nr - ne;
            int end = (hi - lo + FV_K - 1) / FV_K;
            const int mine = end;
            for (int o = 1; o < FMM_NEAR_MAX; o *= 2) {
                const int up = __shfl_up(end, o);
                if (lane >= o) end += up;
            }
            int c = end - mine;
            for (int a = lo; a < hi; a += FV_K) sh.ctab[c++] = make_int4(0, a, min(FV_K, hi - a), 0);
            const int near = __shfl(end, FMM_NEAR_MAX - 1), far = (nd + 3) / 4;
            for (int e = lane; e < far; e += WAVE)
                sh.ctab[near + e] = make_int4(1, 4 * e, min(4, nd - 4 * e), 0);
            if (lane == 0) {
                sh.nch = near + far;
                sh.nexp = ne;
            }
        }
    } else if (threadIdx.x == 0) {
        sh.nch = (n + FV_K - 1) / FV_K;
        sh.nexp = 0;
    }
    __syncthreads();
    const int nch = wave_uniform(sh.nch), nexp = wave_uniform(sh.nexp);
    auto chunk = [&](int ci) -> int4 {
        if (direct) return make_int4(0, ci * FV_K, min(FV_K, n - ci * FV_K), 0);
        const int4 ch = sh.ctab[ci];
        return make_int4(wave_uniform(ch.x), wave_uniform(ch.y), wave_uniform(ch.z), 0);
    };
    // the target of the Cauchy rows this lane generates: row o0 + 16 wv + lane%16, a root
    // (d_K, eta) or (TRANS 0) a pole d_i.  A row past the end only feeds its own output row,
    // never written.
    const int oc = min(o0 + wv * 16 + (lane & 15), n - 1);
    double ra = TRANS ? v.d[base + clamp_idx(v.origin[base + oc], n)] : v.d[base + oc];
    double rb = TRANS ? v.eta[base + oc] : 0.0;
    v4d_f acc[NC];
#pragma unroll
    for (int b = 0; b < NC; ++b) acc[b] = v4d_f{0.0, 0.0, 0.0, 0.0};
    // FB: this lane's share of b's sum for its Cauchy row (the sources it generates entries
    // for), on the VALU beside the multiply: one column does not need the MFMA
    double bsum = 0.0;
    FvStage<NC> st;
    const int rounds = (nch + TEAMS - 1) / TEAMS;
    int4 cur = make_int4(0, 0, 0, 0);
    if (tm < nch) {
        cur = chunk(tm);
        fv_fetch<TRANS, FB, NC>(v, base, sh.fbox, cur, tid, g0, mg, mo, st);
    }
    asm volatile("" : "+v"(ra), "+v"(rb), "+v"(iv.x), "+v"(iv.y));  // loaded here, not in the loop
    for (int rd = 0; rd < rounds; ++rd) {
        double *Xs = sh.team[tm].Xs[rd & 1];
        double2 *Sd = sh.team[tm].Sd[rd & 1];
        const int ci = rd * TEAMS + tm;
        const bool live = ci < nch;
        if (live) fv_store<FB, NC>(cur, tid, mg, mo, st, Xs, Sd);
        __syncthreads();
        const bool near = cur.x == 0;
        if (ci + TEAMS < nch) {  // the next chunk's loads, in flight during the multiply
            cur = chunk(ci + TEAMS);
            fv_fetch<TRANS, FB, NC>(v, base, sh.fbox, cur, tid, g0, mg, mo, st);
        }
        if (!live) continue;
        // a step of 4 sources: the Cauchy entry of this lane's row (one reciprocal with a
        // Newton step, FEW: with two) into the MFMA
        auto multiply = [&](auto is_near) {
#pragma unroll 4
            for (int kk = 0; kk < FV_K; kk += 4) {
                const int sl = kk + (lane >> 4);
                const double2 sd = Sd[sl];
                const double t = TRANS ? (sd.x - ra) - rb : (ra - sd.x) - sd.y;
                const double av = FEW ? rcp_nr(t) : rcp_nr1(t);
#pragma unroll
                for (int b = 0; b < NC; ++b) {
                    const double bv = Xs[(16 * b + (lane & 15)) * FV_LD + sl];
                    acc[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc[b], 0, 0, 0);
                }
                if (FB) {
                    if (is_near.value) {  // (zhat / t)^2: squared after the division
                        const double qv = av * sd.y;
                        bsum = fma(qv, qv, bsum);
                    } else {  // far sources: weights of zhat^2, t bounded away from 0
                        bsum = fma(av * av, sd.y, bsum);
                    }
                }
            }
        };
        if (!FB || near) multiply(fv_true{});
        else multiply(fv_false{});
        mfma_drain();  // before any copy of the accumulators between chunks
    }
    if (TEAMS == 1 && nexp > 0) {
        // The expansion: the Cauchy rows are the interval's nodes.  Wavefront w takes the boxes
        // w, w + 4, ..., their operands straight from memory (step s of a box: source
        // 4 s + lane / 16, column lane % 16), the next box's in flight.
        const double off = iv.y * sh.node[lane & 15];
        v4d_f g[NC];
#pragma unroll
        for (int b = 0; b < NC; ++b) g[b] = v4d_f{0.0, 0.0, 0.0, 0.0};
        double gb = 0.0;  // FB: sum of W / t^2 at this lane's node over its sources
        struct Box {
            double w[4 * NC], x[4], b[4];
        };
        auto fetch = [&](int e, Box &o) {
            const int64_t s0 = (int64_t)sh.fbox[2 * FMM_FAR_MAX - 1 - e] * FMM_P + (lane >> 4);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                o.x[k] = v.vnode[s0 + 4 * k];
#pragma unroll
                for (int b = 0; b < NC; ++b)
                    o.w[4 * b + k] =
                        v.vw[(s0 + 4 * k) * v.m + g0 + min(16 * b + (lane & 15), mg - 1)];
                if (FB) o.b[k] = v.vw[(s0 + 4 * k) * v.m + v.m - 1];
            }
        };
        auto add = [&](const Box &o) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const double t = (o.x[k] - iv.x) - off;
                const double av = rcp_nr1(TRANS ? t : -t);
#pragma unroll
                for (int b = 0; b < NC; ++b)
                    g[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, o.w[4 * b + k], g[b], 0, 0, 0);
                if (FB) gb = fma(av * av, o.b[k], gb);
            }
            mfma_drain();
        };
        Box b0, b1;  // in turn: one in flight while the other is added
        if (wv < nexp) fetch(wv, b0);
        for (int e = wv; e < nexp; e += 8) {
            if (e + 4 < nexp) fetch(e + 4, b1);
            add(b0);
            if (e + 4 >= nexp) break;
            if (e + 8 < nexp) fetch(e + 8, b0);
            add(b1);
        }
        // the wavefronts add their sums through the buffer that the last round left free;
        // accumulator s of lane l (node 4 s + l / 16, column l % 16) is the operand that step s
        // of the interpolation feeds
        double *part = sh.team[0].Xs[rounds & 1];
        double *pb = (double *)sh.team[0].Sd[rounds & 1];
        static_assert(4 * 4 * WAVE <= 16 * FV_LD && 4 * FMM_P <= 2 * FV_K, "the sums fit the buffer");
#pragma unroll
        for (int b = 0; b < NC; ++b)
#pragma unroll
            for (int k = 0; k < 4; ++k) part[((b * 4 + wv) * 4 + k) * WAVE + lane] = g[b][k];
        if (FB) {
            gb += __shfl_xor(gb, 16);
            gb += __shfl_xor(gb, 32);
            if (lane < FMM_P) pb[wv * FMM_P + lane] = gb;
        }
        __syncthreads();
        // Lagrange values of this lane's row at the nodes 4 k + lane / 16 (barycentric form; a
        // target on a node: that node's term outweighs the others)
        const double tau = ((ra - iv.x) + rb) / iv.y;
        double lq[4], den = 0.0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double dl = tau - sh.node[4 * k + (lane >> 4)];
            lq[k] = sh.bary[4 * k + (lane >> 4)] * rcp_nr(dl == 0.0 ? 0x1p-200 : dl);
            den += lq[k];
        }
        den += __shfl_xor(den, 16);
        den += __shfl_xor(den, 32);
        const double iden = 1.0 / den;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
#pragma unroll
            for (int b = 0; b < NC; ++b) {
                double gk = part[(b * 16 + k) * WAVE + lane];
#pragma unroll
                for (int u = 1; u < 4; ++u) gk += part[((b * 4 + u) * 4 + k) * WAVE + lane];
                acc[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(lq[k] * iden, gk, acc[b], 0, 0, 0);
            }
            if (FB) {
                const int q = 4 * k + (lane >> 4);
                double bk = pb[q];
#pragma unroll
                for (int u = 1; u < 4; ++u) bk += pb[u * FMM_P + q];
                bsum = fma(lq[k] * iden, bk, bsum);
            }
        }
    }
    if (FB) {  // the four lanes of a Cauchy row (lane % 16) hold its partial sums
        bsum += __shfl_xor(bsum, 16);
        bsum += __shfl_xor(bsum, 32);
    }
    if (v.work && threadIdx.x == 0) {  // kernel timing: the item's algorithmic flops
        unsigned long long ent = 0;  // near and far sources summed per row
        for (int ci = 0; ci < nch; ++ci) {
            const int4 ch = chunk(ci);
            ent += ch.x == 0 ? ch.z : ch.z * FMM_P;
        }
        const unsigned long long rows = (unsigned long long)min(FV_K, n - o0);
        const unsigned long long per = 2 * (unsigned long long)mg + 3;
        atomicAdd(v.work, rows * ent * per + 2 * rows * (unsigned long long)mo +
                              (nexp > 0 ? FMM_P * (nexp * FMM_P * per + rows * 2 * mg) : 0));
    }
    mfma_drain();
    if (TEAMS > 1) {  // the teams' sums through their own buffers, added in team order
        double *mine = &sh.team[tm].Xs[0][0] + wv * 5 * WAVE;
        static_assert(4 * 5 * WAVE <= 2 * 16 * FV_LD, "a team's sums fit its buffers");
        __syncthreads();
        if (tm > 0) {
#pragma unroll
            for (int r = 0; r < 4; ++r) mine[r * WAVE + lane] = acc[0][r];
            if (FB) mine[4 * WAVE + lane] = bsum;
        }
        __syncthreads();
        if (tm > 0) return;
        for (int u = 1; u < TEAMS; ++u) {
            const double *o = &sh.team[u].Xs[0][0] + wv * 5 * WAVE;
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[0][r] += o[r * WAVE + lane];
            if (FB) bsum += o[4 * WAVE + lane];
        }
    }
    // v_mfma_f64_16x16x4f64 returns D[4 r + lane/16][lane % 16] in accumulator r
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = o0 + wv * 16 + 4 * r + (lane >> 4);
        double post;
        if (FB) {  // b's sum of this row is held by the lanes that generated its entries
            post = 1.0 / sqrt(__shfl(bsum, 4 * r + (lane >> 4)));
            if (row < n && (lane & 15) == 0) v.bout[base + row] = post;
        } else {
            post = row < n ? v.post[base + row] : 0.0;
        }
#pragma unroll
        for (int b = 0; b < NC; ++b) {
            const int col = 16 * b + (lane & 15);
            if (row < n && col < mo)
                v.Y[base + row + (int64_t)(g0 + col) * v.ldy] = post * acc[b][r];
        }
    }
}

template <int TRANS, bool FB, int TEAMS, int NC, bool FEW>
__global__ __launch_bounds__(256 * TEAMS, NC == 1 ? 4 : 3) void k_fmmv_eval_mfma(SolveArgs it,
                                                                                 FmmArgs f,
                                                                                 FmmVec v) {
    __shared__ FvShared<TEAMS, NC> sh;
    if (TEAMS == 1 && threadIdx.x < FMM_P) {
        sh.node[threadIdx.x] = FV_NODE[threadIdx.x];
        sh.bary[threadIdx.x] = FV_BARY[threadIdx.x];
    }
    // the column groups of a tile are neighbouring items: they read the same lists and poles
    const int ng = (v.m + NC * FMMV_MAX_M - 1) / (NC * FMMV_MAX_M);
    const int item = xcd_item();
    fmmv_item_mfma<TRANS, FB, TEAMS, NC, FEW>(it, f, v, it.tiles[item / ng], item % ng, sh);
}

// ---------------------------------------------------------------------------------------
// Loewner far field: box moments.  LEAVES = true: every leaf from its poles and roots;
// LEAVES = false: every used box above the leaves from its leaves' moments, translated to
// the box's centre and half-width (t_box = alpha + beta t_leaf):
//     M_k = sum_m C(k, m) alpha^(k-m) beta^m M_m(leaf)
// (M_0 = 0: each pole-root pair carries opposite unit charges).  One workgroup per box; the
// per-thread partial moments are added in a fixed order through LDS.

// binomial coefficient C(k, m) for k <= FMML_K (integers below 2^53: exact in double); used
// with constant arguments only, so every coefficient is a literal of the unrolled loops
__host__ __device__ constexpr double binom(int k, int m) {
    double c = 1.0;
    for (int j = 1; j <= m; ++j) c = c * (k - m + j) / j;
    return c;
}
// ---------------------------------------------------------------------------------------
// moments are stored as the series' coefficients (-1)^(k+1) M_k / k
__host__ __device__ constexpr double mom_scale(int k) { return k & 1 ? (double)k : -(double)k; }

// the range of box g; false: invalid problem, or an empty box
struct MomBox {
    int H, n, lo, hi, leaf0;  // leaf0: its first leaf's box
    int64_t base;
    double c, hw, ihw;
};
__device__ __forceinline__ bool mom_box(const FmmArgs &f, int g, MomBox &b) {
    const int qf = f.box_fmm[g];
    const int p = f.fmm_prob[qf];
    b.base = f.off[p];
    b.n = (int)(f.off[p + 1] - b.base);
    const int hidx = g - f.box_off[qf];
    b.H = f.height[qf];
    int h = 0;
    while ((2 << h) - 1 <= hidx) ++h;
    const int bi = hidx - ((1 << h) - 1);
    const int64_t span = (int64_t)f.leaf << (b.H - h);
    b.lo = (int)min((int64_t)b.n, bi * span);
    b.hi = (int)min((int64_t)b.n, (bi + 1) * span);
    b.leaf0 = f.box_off[qf] + (1 << b.H) - 1 + bi * (1 << (b.H - h));
    return !(f.status[p] & ~SUPERDC_ST_NOCONV) && b.lo < b.hi;
}
__device__ __forceinline__ void mom_span(const FmmlArgs &l, MomBox &b) {
    const double2 *pd = l.pd + b.base;
    // its poles and roots, without the problem's last root: that one lies rho |z|^2 above its
    // pole, as far as the others spread, and would widen the box until most poles are too
    // close for its expansion (they multiply the last pair's factor themselves)
    const double x0 = pd[b.lo].x, x1 = pd[b.hi - 1].x + (b.hi < b.n ? pd[b.hi - 1].y : 0.0);
    b.c = 0.5 * (x0 + x1);
    b.hw = 0.5 * (x1 - x0);
    b.ihw = b.hw > 0.0 ? 1.0 / b.hw : 0.0;
}
// leaf gl's moments translated to the box's centre and half-width, added to M
__device__ __forceinline__ void mom_translate(const FmmlArgs &l, int gl, double c, double ihw,
                                              double (&M)[FMML_K]) {
    const double2 gc = l.geo[gl];
    const double al = (gc.x - c) * ihw, be = gc.y * ihw;
    const double *Ml = l.mom + (int64_t)gl * FMML_K;
    // moment m of the leaf spread over k >= m: C(k, m) alpha^(k-m) beta^m M_m, the
    // power of alpha built up along k (no row of coefficients kept: few registers)
    double bm = 1.0;
#pragma unroll
    for (int m = 1; m <= FMML_K; ++m) {
        bm *= be;
        double q = Ml[m - 1] * (bm * mom_scale(m));  // alpha^(k-m) beta^m M_m
#pragma unroll
        for (int k = m; k <= FMML_K; ++k) {
            M[k - 1] = __builtin_fma(binom(k, m), q, M[k - 1]);
            q *= al;
        }
    }
}

// every leaf, one wavefront each
__global__ __launch_bounds__(WAVE) void k_fmml_moments(FmmArgs f, FmmlArgs l) {
    __shared__ double part[WAVE][FMML_K + 1];
    const int g = f.leaf_box[blockIdx.x], tid = threadIdx.x;
    MomBox b;
    if (!mom_box(f, g, b)) return;
    if (l.pack) {  // the leaf's poles packed here (the same arithmetic as k_fmml_pack)
        for (int j = b.lo + tid; j < b.hi; j += WAVE) {
            const double dj = l.d[b.base + j];
            const double dK = l.d[b.base + clamp_idx(l.origin[b.base + j], b.n)];
            const double ej = l.eta[b.base + j];
            const double delta = (dK - dj) + ej;
            l.pd[b.base + j] = make_double2(dj, delta);
        }
        __syncthreads();
    }
    mom_span(l, b);
    const double2 *pd = l.pd + b.base;
    double M[FMML_K];
#pragma unroll
    for (int k = 0; k < FMML_K; ++k) M[k] = 0.0;
    for (int j = b.lo + tid; j < min(b.hi, b.n - 1); j += WAVE) {
        const double t = (pd[j].x - b.c) * b.ihw, D = pd[j].y * b.ihw, tD = t + D;
        double P = D, tk = 1.0;
#pragma unroll
        for (int k = 0; k < FMML_K; ++k) {
            M[k] += P;  // P = (t + D)^(k+1) - t^(k+1)
            tk *= t;
            P = __builtin_fma(tD, P, D * tk);
        }
    }
    // lane k adds column k over the 64 lanes in order
#pragma unroll
    for (int k = 0; k < FMML_K; ++k) part[tid][k] = M[k];
    __syncthreads();
    if (tid < FMML_K) {
        double sk = 0.0;
        for (int u = 0; u < WAVE; ++u) sk += part[u][tid];
        l.mom[(int64_t)g * FMML_K + tid] = sk / mom_scale(tid + 1);
    }
    if (tid == 0) l.geo[g] = make_double2(b.c, b.hw);
}

// Used boxes above the leaves from their leaves' moments.  More than 64 leaves: a workgroup.
// Others: 2^c lanes, one a leaf, 2^(6-c) boxes to a wavefront -- most upper boxes have two or
// four leaves, and with a workgroup each they took 500 us of a level of 4096 problems (now 36).
constexpr int MOM_HALF = FMML_K / 2;
static_assert(2 * MOM_HALF == FMML_K, "moments go through LDS in two halves");
__global__ __launch_bounds__(256, 4) void k_fmml_moments_up(FmmArgs f, FmmlArgs l) {
    __shared__ double lds[4 * WAVE * (MOM_HALF + 1)];
    static_assert(2 * WAVE * (FMML_K + 1) <= 4 * WAVE * (MOM_HALF + 1), "a large box's two buffers");
    const int tid = threadIdx.x, wv = wave_uniform(tid / WAVE), ln = tid % WAVE;
    double M[FMML_K];
#pragma unroll
    for (int k = 0; k < FMML_K; ++k) M[k] = 0.0;
    MomBox b;
    const int nbig = f.upper_cls[0];
    if ((int)blockIdx.x >= nbig) {
        // this wavefront's boxes: class c of at most 2^c leaves
        int w = ((int)blockIdx.x - nbig) * 4 + wv, c = 6;
        for (; c >= 1; --c) {
            const int waves = (f.upper_cls[7 - c] - f.upper_cls[6 - c] + (64 >> c) - 1) / (64 >> c);
            if (w < waves) break;
            w -= waves;
        }
        if (c < 1) return;
        const int first = f.upper_cls[6 - c] + w * (64 >> c);
        const int i = first + (ln >> c);
        const bool in = i < f.upper_cls[7 - c];
        const int g = in ? f.upper_box[i] : 0;
        const bool ok = in && f.used[g] == f.gen && mom_box(f, g, b);
        if (ok) {
            mom_span(l, b);
            const int e = ln & ((1 << c) - 1), nleaf = (b.hi - b.lo + f.leaf - 1) / f.leaf;
            if (e < nleaf) mom_translate(l, b.leaf0 + e, b.c, b.ihw, M);
            if (e == 0) l.geo[g] = make_double2(b.c, b.hw);
        }
        const unsigned long long live = __ballot(ok);
        // sums over each box's lanes, in leaf order
        double *part = lds + wv * WAVE * (MOM_HALF + 1);
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int k = 0; k < MOM_HALF; ++k)
                part[ln * (MOM_HALF + 1) + k] = h ? M[MOM_HALF + k] : M[k];
            wave_sync();
            for (int e = ln; e < (64 >> c) * MOM_HALF; e += WAVE) {
                const int u = e / MOM_HALF, k = e % MOM_HALF;
                if (!(live >> (u << c) & 1)) continue;
                double s = 0.0;
                for (int r = 0; r < 1 << c; ++r) s += part[((u << c) + r) * (MOM_HALF + 1) + k];
                l.mom[(int64_t)f.upper_box[first + u] * FMML_K + h * MOM_HALF + k] =
                    s / mom_scale(h * MOM_HALF + k + 1);
            }
            wave_sync();
        }
        return;
    }
    double(*part)[FMML_K + 1] = reinterpret_cast<double(*)[FMML_K + 1]>(lds);
    double(*part2)[FMML_K + 1] = part + WAVE;
    const int g = f.upper_box[blockIdx.x];
    if (f.used[g] != f.gen || !mom_box(f, g, b)) return;
    mom_span(l, b);
    const int nleaf = (b.hi - b.lo + f.leaf - 1) / f.leaf;
    for (int e = tid; e < nleaf; e += blockDim.x) mom_translate(l, b.leaf0 + e, b.c, b.ihw, M);
    // the four wavefronts are folded onto the first, (w0 + w2) + (w1 + w3), through two 64-row
    // buffers; then lane k adds column k over the rows, in order (one pass, no barrier per level
    // of a tree)
    if (wv >= 2) {
#pragma unroll
        for (int k = 0; k < FMML_K; ++k) (wv == 2 ? part : part2)[ln][k] = M[k];
    }
    __syncthreads();
    if (wv < 2) {
#pragma unroll
        for (int k = 0; k < FMML_K; ++k) M[k] += (wv == 0 ? part : part2)[ln][k];
    }
    __syncthreads();
    if (wv == 1) {
#pragma unroll
        for (int k = 0; k < FMML_K; ++k) part[ln][k] = M[k];
    }
    __syncthreads();
    if (wv == 0) {
#pragma unroll
        for (int k = 0; k < FMML_K; ++k) M[k] += part[ln][k];
    }
    __syncthreads();
    if (wv == 0) {
#pragma unroll
        for (int k = 0; k < FMML_K; ++k) part[ln][k] = M[k];
    }
    __syncthreads();
    if (tid < FMML_K) {
        double sk = 0.0;
        for (int u = 0; u < WAVE; ++u) sk += part[u][tid];
        l.mom[(int64_t)g * FMML_K + tid] = sk / mom_scale(tid + 1);
    }
    if (tid == 0) l.geo[g] = make_double2(b.c, b.hw);
}

hipError_t launch_fmml_moments(const FmmArgs &f, const FmmlArgs &l, hipStream_t s) {
    if (f.nboxes <= 0) return hipSuccess;
    SDC_LAUNCH(KID_FMML_MOMENTS, k_fmml_moments, dim3(f.nleaves), dim3(WAVE), 0, s, f, l);
    int waves = 0;
    for (int c = 1; c <= 6; ++c)
        waves += (f.upper_cls[7 - c] - f.upper_cls[6 - c] + (64 >> c) - 1) / (64 >> c);
    const int blocks = f.upper_cls[0] + (waves + 3) / 4;
    if (blocks > 0)
        SDC_LAUNCH(KID_FMML_MOMENTS, k_fmml_moments_up, dim3(blocks), dim3(256), 0, s, f, l);
    return hipGetLastError();
}

// (d_j, delta_j) with delta_j = lambda_j - d_j = (d_{K_j} - d_j) + eta_j; one lane per entry
__global__ __launch_bounds__(64) void k_fmml_pack(FmmvPackArgs a) {
    const Tile t = a.tiles[blockIdx.x];
    const int64_t base = a.off[t.prob];
    const int n = (int)(a.off[t.prob + 1] - base);
    const int j = t.row0 + lane_id();
    if (j >= n) return;
    const double dj = a.d[base + j];
    const double dK = a.d[base + clamp_idx(a.origin[base + j], n)];
    const double ej = a.eta[base + j];
    const double delta = (dK - dj) + ej;
    a.pairs[base + j] = make_double2(dj, delta);
    if (a.ke) a.ke[base + j] = make_double2(dK, ej);
}

hipError_t launch_fmml_pack(const FmmvPackArgs &a, hipStream_t s) {
    if (a.ntiles <= 0) return hipSuccess;
    SDC_LAUNCH(KID_FMML_PACK, k_fmml_pack, dim3(a.ntiles), dim3(64), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_fmmv_pos(const FmmvPackArgs &a, hipStream_t s) {
    if (a.ntiles <= 0) return hipSuccess;
    SDC_LAUNCH(KID_FMMV_PACK, k_fmmv_pos, dim3(a.ntiles), dim3(64), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_fmmv_sources(const FmmArgs &f, const FmmVec &v, hipStream_t s) {
    if (f.nboxes <= 0) return hipSuccess;
    const int ng = (v.m + FMMV_MAX_M - 1) / FMMV_MAX_M;
    const dim3 gl(f.nleaves, ng), gu(f.nitem_big + (f.nupper_item - f.nitem_big + 3) / 4, ng);
    if (v.m <= 4) {
        SDC_LAUNCH(KID_FMMV_SOURCES, (k_fmmv_sources<true, true>), gl, dim3(64), 0, s, f, v);
        if (f.nupper_item > 0)
            SDC_LAUNCH(KID_FMMV_SOURCES, (k_fmmv_sources<false, true>), gu, dim3(256), 0, s, f, v);
    } else {
        SDC_LAUNCH(KID_FMMV_SOURCES, (k_fmmv_sources<true, false>), gl, dim3(64), 0, s, f, v);
        if (f.nupper_item > 0)
            SDC_LAUNCH(KID_FMMV_SOURCES, (k_fmmv_sources<false, false>), gu, dim3(256), 0, s, f, v);
    }
    if (f.nsplit > 0)
        SDC_LAUNCH(KID_FMMV_SOURCES, k_fmmv_sources_sum, dim3(f.nsplit, ng),
                   dim3(FMM_P * FMMV_MAX_M), 0, s, f, v);
    return hipGetLastError();
}

hipError_t launch_fmmv_eval(const SolveArgs &it, const FmmArgs &f, const FmmVec &v0, int split,
                            int num_cu, hipStream_t s) {
    if (it.ntiles <= 0) return hipSuccess;
    FmmVec v = v0;
    v.sep_t = FV_SEP_T;
    // the MFMA for a dense enough block of columns, and for every sum over the roots
    const bool mfma = v.kern == 1 && (v.m >= 4 || v.fuse_b || v.trans == 0);
    v.work = trace_work(mfma ? KID_FMMV_EVAL_MFMA : KID_FMMV_EVAL);
    if (mfma) {
        const int groups = (v.m + FMMV_MAX_M - 1) / FMMV_MAX_M, items = it.ntiles * groups;
        const int wide = (groups + 1) / 2;
        const bool few = v.trans && !v.fuse_b && (v.m - 1) % FMMV_MAX_M < 3;
#define SDC_FV(T, FB, K, N, FEW)                                                                   \
    SDC_LAUNCH(KID_FMMV_EVAL_MFMA, (k_fmmv_eval_mfma<T, FB, K, N, FEW>), g, dim3(256 * K), 0, s, it, f, v)
        if (!v.fuse_b && groups > 1 &&
            it.ntiles * wide >= (groups == 3 ? FV_WIDE3_PER_CU : FV_WIDE_PER_CU) * num_cu) {
            const dim3 g(it.ntiles * wide);
            if (v.trans == 0) SDC_FV(0, false, 1, 2, false);
            else if (few) SDC_FV(1, false, 1, 2, true);
            else SDC_FV(1, false, 1, 2, false);
            return hipGetLastError();
        }
        const int teams = items >= FV_EXPAND_PER_CU * num_cu ? 1 : items >= num_cu ? 2 : 4;
        const dim3 g(items);
#define SDC_FV_TEAMS(T, FB, FEW)                     \
    {                                                \
        if (teams == 1) SDC_FV(T, FB, 1, 1, FEW);    \
        else if (teams == 2) SDC_FV(T, FB, 2, 1, FEW); \
        else SDC_FV(T, FB, 4, 1, FEW);               \
    }
        if (v.trans == 0) SDC_FV_TEAMS(0, false, false)
        else if (v.fuse_b) SDC_FV_TEAMS(1, true, false)
        else if (few) SDC_FV_TEAMS(1, false, true)
        else SDC_FV_TEAMS(1, false, false)
#undef SDC_FV_TEAMS
#undef SDC_FV
        return hipGetLastError();
    }
    if (v.trans == 0 || v.m >= 4) return hipErrorInvalidValue;
    v.expand = it.ntiles >= FV_EXPAND_PER_CU * num_cu;
    const dim3 g(it.ntiles), blk(WAVE * split);
    // a kernel per column count: with the count tested in the loops one column took twice as long
    // (34,000 items: 510 -> 315 us)
    const size_t lds = sizeof(double) * WAVE * (split - 1) * v.m;
    if (v.kern == 2) SDC_LAUNCH(KID_FMMV_EVAL, (k_fmmv_eval<2, 1>), g, blk, lds, s, it, f, v);
    else if (v.m == 1) SDC_LAUNCH(KID_FMMV_EVAL, (k_fmmv_eval<1, 1>), g, blk, lds, s, it, f, v);
    else if (v.m == 2) SDC_LAUNCH(KID_FMMV_EVAL, (k_fmmv_eval<1, 2>), g, blk, lds, s, it, f, v);
    else SDC_LAUNCH(KID_FMMV_EVAL, (k_fmmv_eval<1, 3>), g, blk, lds, s, it, f, v);
    return hipGetLastError();
}

}  // namespace sdc
