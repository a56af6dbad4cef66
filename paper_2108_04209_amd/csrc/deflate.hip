// deflate.hip -- deflation of the rank-one problems of a batch (Remark 1) on gfx950, and
// the orthogonal factor it leaves in the eigenvector matrix.
//
// For A = diag(d) + v v^T, v = sqrt(rho) z, d non-decreasing, and a user tolerance tau:
//   rule 1: pole k deflates if |v_k| < tau (eigenpair (d_k, e_k));
//   rule 2: scanning the other poles left to right, the current pole a and the next pole b
//           rotate together if |(d_a - d_b) v_a v_b| < (v_a^2 + v_b^2) tau (z can stand
//           for v: both sides scale by rho).  G = [c -s; s c] with c = z_b / r,
//           s = z_a / r, r = |(z_a, z_b)| takes (z_a, z_b) to (0, r); the off-diagonal
//           entry cs (d_a - d_b) of G diag(d_a, d_b) G^T is below tau and is dropped.  Pole a
//           deflates with eigenvalue c^2 d_a + s^2 d_b; pole b goes on with
//           d_b' = s^2 d_a + c^2 d_b (held in [d_a, d_b]) and z_b' = r.
// A = G^T (diag(d') + v' v'^T) G up to the dropped entries, so the eigenvector matrix is
// Q = G^T P (Qhat (+) I), with P placing the reduced problem's eigenvectors and the deflated
// unit vectors at their poles.
//
// The scan is sequential only through runs of rotations.  One wavefront owns a problem and
// takes its poles 64 at a time: the poles that survive rule 1 are packed into lanes, every
// lane tests its pair (left neighbour, itself) at once, and only the lane after a rotation
// is re-tested with the rotated values.  A window of 64 poles costs one pass plus one per
// rotation in it.
//
// Decisions are taken with the same expressions in the same order as a plain sequential
// implementation, without contraction into fused multiply-adds, so they do not depend on
// how the lanes split the work.
#include <algorithm>

#include "common.h"

namespace sdc {

// Poles per segment of the parallel scan (a multiple of 64): short enough to spread a problem over
// wavefronts, but a boundary that rotates costs a second scan of its segment (18 rank-one
// steps of a tridiagonal matrix of 65536 rows, which rotate at most boundaries, us a step for
// 64, 128, 256, 512, 1024 poles: 59 46 36 28 31).  Problems of up to 8 segments (DEFL_WG) take
// one launch with the joins and the placement.  Longer segments where the records (problems
// x segments of the largest) would grow past 64 MB, or past 256 to a problem.
constexpr int DEFL_SEG = 512, DEFL_SEG_MAX = 2048;
constexpr int DEFL_WAVES = 8, DEFL_WG = DEFL_WAVES * DEFL_SEG;

static int defl_seg(int nprob, int max_n) {
    int seg = DEFL_SEG;
    while (seg < DEFL_SEG_MAX && (max_n > 256 * seg || (int64_t)nprob * ((max_n + seg - 1) / seg) > (1 << 21)))
        seg *= 2;
    return seg;
}

struct DeflArgs {
    const int64_t *off;
    const double *d, *z, *rho;
    double tau;
    double *dout, *zout;
    int32_t *perm, *rright, *rleft;
    double *rc, *rs;
    int32_t *kept, *status;
    double2 *val;    // workspace: final (d, z) of each pole by pole index
    int8_t *flag;    // workspace: 1 kept, 0 deflated
    int4 *seg_i;     // workspace [nprob][maxseg]: current pole, first survivor, status, kept
    double2 *seg_d;  // workspace [nprob][maxseg]: the current pole's (d, z)
    int seg, maxseg; // poles per segment, segments of the largest problem
};

// the rule-2 test and the rotation (evaluated exactly as written)
__device__ __forceinline__ bool defl_test(double da, double za, double db, double zb,
                                          double tau) {
#pragma clang fp contract(off)
    const double r2 = za * za + zb * zb;
    const double lhs = fabs(((da - db) * za) * zb);
    return lhs < r2 * tau;
}

__device__ __forceinline__ void defl_rotate(double da, double za, double db, double zb,
                                            double &c, double &s, double &dl, double &dr,
                                            double &r) {
#pragma clang fp contract(off)
    const double r2 = za * za + zb * zb;
    r = sqrt(r2);
    c = zb / r;
    s = za / r;
    const double cc = c * c, ss = s * s;
    dl = cc * da + ss * db;
    dr = ss * da + cc * db;
    if (dr < da) dr = da;
    if (dr > db) dr = db;
}

// read a double / int from lane l (l wave-uniform)
__device__ __forceinline__ double lane_get(double v, int l) {
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffff), l);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ int lane_get(int v, int l) { return __builtin_amdgcn_readlane(v, l); }

// The scan over poles [lo, hi) of a problem, a window of 64 at a time, with the incoming
// current pole (ca, cd, cz) (ca < 0: none yet): rule 1, the packing of the survivors into
// lanes and the rule-2 tests, writing the outcome of every pole of the range and of the
// incoming pole once it is decided.  On return (ca, cd, cz) is the current pole, still
// undecided; `first` is the range's first pole that survives rule 1 (-1: none).  Returns
// the number of poles decided kept.
__device__ int defl_scan(const DeflArgs &a, int64_t base, int lo, int hi, double sv, int &ca,
                         double &cd, double &cz, int &first, double *sd, double *sz, int *si) {
    const int lane = lane_id();
    const double tau = a.tau;
    const double *d = a.d + base, *z = a.z + base;
    double2 *val = a.val + base;
    int8_t *flag = a.flag + base;
    int32_t *rright = a.rright + base, *rleft = a.rleft + base;
    double *rc = a.rc + base, *rs = a.rs + base;
    int nkept = 0;
    first = -1;
    // the next window's loads are issued before this one is worked on
    double ndi = lo + lane < hi ? d[lo + lane] : 0.0, nzi = lo + lane < hi ? z[lo + lane] : 0.0;
    for (int c0 = lo; c0 < hi; c0 += WAVE) {
        const int i = c0 + lane;
        const bool valid = i < hi;
        const double di = ndi, zi = nzi;
        if (i + WAVE < hi) {
            ndi = d[i + WAVE];
            nzi = z[i + WAVE];
        }
        const bool r1 = valid && fabs(sv * zi) < tau;  // rule 1
        if (valid) {
            rright[i] = -1;
            rleft[i] = -1;
            rc[i] = 1.0;
            rs[i] = 0.0;
            if (r1) {
                val[i] = make_double2(di, 0.0);
                flag[i] = 0;
            }
        }
        // pack the poles that survive rule 1 into lanes 0 .. cnt-1, in order
        const unsigned long long cm = __ballot(valid && !r1);
        const int cnt = __popcll(cm);
        const int rank = __builtin_amdgcn_mbcnt_hi((unsigned)(cm >> 32),
                                                   __builtin_amdgcn_mbcnt_lo((unsigned)cm, 0u));
        if (valid && !r1) {
            sd[rank] = di;
            sz[rank] = zi;
            si[rank] = i;
        }
        wave_sync();
        const bool live = lane < cnt;
        const double bd = live ? sd[lane] : 0.0, bz = live ? sz[lane] : 0.0;
        const int bi = live ? si[lane] : -1;
        wave_sync();
        if (cnt == 0) continue;
        if (first < 0) first = lane_get(bi, 0);
        // left neighbour of every lane's pair: the previous lane's pole, the current pole
        // of the scan for lane 0
        double ld = __shfl_up(bd, 1), lz = __shfl_up(bz, 1);
        int li = __shfl_up(bi, 1);
        int start = 0;
        if (lane == 0) {
            ld = cd;
            lz = cz;
            li = ca;
        }
        if (ca < 0) start = 1;  // the first surviving pole has no left neighbour
        int rot_lane = -1;      // lane of the last rotation in this window
        double md = 0.0, mz = 0.0;
        for (;;) {
            const bool test = live && lane >= start;
            const bool F = test && defl_test(ld, lz, bd, bz, tau);
            const unsigned long long fm = __ballot(F);
            const int j = fm ? (int)__builtin_ctzll(fm) : cnt;
            // pairs start .. j-1 do not rotate: their left poles are kept as they stand
            if (lane >= start && lane < j && live) {
                val[li] = make_double2(ld, lz);
                flag[li] = 1;
            }
            nkept += max(0, j - start);
            if (!fm) break;
            // pair j rotates: its left pole deflates, its right pole goes on rotated
            double c = 0.0, s = 0.0, dl = 0.0, dr = 0.0, r = 0.0;
            if (lane == j) {
                defl_rotate(ld, lz, bd, bz, c, s, dl, dr, r);
                val[li] = make_double2(dl, 0.0);
                flag[li] = 0;
                rright[li] = bi;
                rleft[bi] = li;
                rc[li] = c;
                rs[li] = s;
            }
            md = lane_get(dr, j);
            mz = lane_get(r, j);
            rot_lane = j;
            if (lane == j + 1) {
                ld = md;
                lz = mz;
            }
            start = j + 1;
            if (start >= cnt) break;
        }
        // the window's last pole becomes the current pole of the scan
        if (rot_lane == cnt - 1) {
            cd = md;
            cz = mz;
        } else {
            cd = lane_get(bd, cnt - 1);
            cz = lane_get(bz, cnt - 1);
        }
        ca = lane_get(bi, cnt - 1);
    }
    return nkept;
}

// validation of poles [lo, hi) of problem p: finite, non-decreasing (across the range's
// end as well), rho > 0
__device__ int defl_check(const DeflArgs &a, int p, int64_t base, int lo, int hi, int n) {
    const int lane = lane_id();
    const double *d = a.d + base, *z = a.z + base;
    int st = 0;
    for (int i = lo + lane; i < hi; i += WAVE) {
        const double di = d[i], zi = z[i];
        if (!isfinite(di) || !isfinite(zi)) st |= SUPERDC_ST_NONFINITE;
        if (i + 1 < n && d[i + 1] < di) st |= SUPERDC_ST_UNSORTED;
    }
    for (int o = WAVE / 2; o > 0; o >>= 1) st |= __shfl_xor(st, o);
    const double rho = a.rho[p];
    if (!isfinite(rho)) st |= SUPERDC_ST_NONFINITE;
    else if (!(rho > 0.0)) st |= SUPERDC_ST_RHO;
    return st;
}

// Segments are scanned in parallel, one wavefront each, as if no pole came before them; their
// records keep the undecided current pole at the end, the first pole that survives rule 1,
// the status bits and the number of poles decided kept.
__device__ void defl_segment(const DeflArgs &a, int p, int64_t base, int n, int sg, int4 *rec_i,
                             double2 *rec_d, double *sd, double *sz, int *si) {
    const int lo = sg * a.seg;
    if (lo >= n) return;
    const int hi = min(n, lo + a.seg);
    const int st = defl_check(a, p, base, lo, hi, n);
    int ca = -1, first = -1, nk = 0;
    double cd = 0.0, cz = 0.0;
    if (!st) nk = defl_scan(a, base, lo, hi, sqrt(a.rho[p]), ca, cd, cz, first, sd, sz, si);
    if (lane_id() == 0) {
        rec_i[sg] = make_int4(ca, first, st, nk);
        rec_d[sg] = make_double2(cd, cz);
    }
}

// The joins of a problem, in order, by one wavefront.  The scan entering segment s holds the
// current pole of everything before it.  If that pole and the segment's first survivor do
// not rotate, the pole is kept and the segment's own scan stands exactly (it started from
// that survivor); if they do, the segment is scanned again from the incoming pole (which
// deflates).  The records of 64 segments and their first survivors are loaded at once, so
// that the chain runs in registers.  Returns the status; on 0 the records' counts are final
// and kept is the problem's.
__device__ int defl_join(const DeflArgs &a, int p, int64_t base, int n, int4 *rec_i,
                         const double2 *rec_d, int &kept, double *sd, double *sz, int *si) {
    const int lane = lane_id();
    const int nseg = (n + a.seg - 1) / a.seg;
    int st = 0;
    for (int sg = lane; sg < nseg; sg += WAVE) st |= rec_i[sg].z;
    for (int o = WAVE / 2; o > 0; o >>= 1) st |= __shfl_xor(st, o);
    kept = 0;
    if (st) return st;
    const double sv = sqrt(a.rho[p]);
    int ca = -1, nk = 0;
    double cd = 0.0, cz = 0.0;
    auto keep = [&]() {  // the current pole is kept
        if (lane == 0) {
            a.val[base + ca] = make_double2(cd, cz);
            a.flag[base + ca] = 1;
            atomicAdd(&rec_i[ca / a.seg].w, 1);
        }
        ++nk;
    };
    for (int s0 = 0; s0 < nseg; s0 += WAVE) {
        const int mine = min(s0 + lane, nseg - 1);
        const int4 ri = rec_i[mine];
        const double2 rd = rec_d[mine];
        const int fi = max(ri.y, 0);
        const double fd = a.d[base + fi], fz = a.z[base + fi];
        for (int u = 0; u < min(WAVE, nseg - s0); ++u) {
            const int f = lane_get(ri.y, u);
            if (f < 0) continue;  // nothing survives rule 1 here: the current pole passes on
            if (ca >= 0 && defl_test(cd, cz, lane_get(fd, u), lane_get(fz, u), a.tau)) {
                int first;
                const int lo = (s0 + u) * a.seg;
                const int k = defl_scan(a, base, lo, min(n, lo + a.seg), sv, ca, cd, cz, first, sd,
                                        sz, si);
                if (lane == 0) rec_i[s0 + u].w = k;
                nk += k;
                continue;
            }
            if (ca >= 0) keep();  // and the segment's scan stands
            ca = lane_get(ri.x, u);
            cd = lane_get(rd.x, u);
            cz = lane_get(rd.y, u);
            nk += lane_get(ri.w, u);
        }
    }
    if (ca >= 0) keep();
    kept = nk;
    return 0;
}

// placement of a segment: kept poles first, deflated ones after, each in pole order
__device__ void defl_place(const DeflArgs &a, int64_t base, int n, int sg, const int4 *rec_i,
                           int kept) {
    const int lo = sg * a.seg;
    if (lo >= n) return;
    const int hi = min(n, lo + a.seg);
    const int lane = lane_id();
    int pk = 0;  // kept poles before this segment
    for (int u = lane; u < sg; u += WAVE) pk += rec_i[u].w;
    for (int o = WAVE / 2; o > 0; o >>= 1) pk += __shfl_xor(pk, o);
    int pd = kept + (lo - pk);
    const double2 *val = a.val + base;
    const int8_t *flag = a.flag + base;
    int8_t nfl = lo + lane < hi ? flag[lo + lane] : 0;
    double2 nv = lo + lane < hi ? val[lo + lane] : make_double2(0.0, 0.0);
    for (int c0 = lo; c0 < hi; c0 += WAVE) {
        const int i = c0 + lane;
        const bool valid = i < hi;
        const int8_t fl = nfl;
        const double2 v = nv;
        if (i + WAVE < hi) {  // the next window's loads in flight
            nfl = flag[i + WAVE];
            nv = val[i + WAVE];
        }
        const bool k = valid && fl != 0;
        const unsigned long long km = __ballot(k), dm = __ballot(valid && !k);
        const unsigned long long mm = k ? km : dm;
        const int rank = __builtin_amdgcn_mbcnt_hi((unsigned)(mm >> 32),
                                                   __builtin_amdgcn_mbcnt_lo((unsigned)mm, 0u));
        if (valid) {
            const int j = (k ? pk : pd) + rank;
            a.dout[base + j] = v.x;
            a.zout[base + j] = k ? v.y : 0.0;
            a.perm[base + j] = i;
        }
        pk += __popcll(km);
        pd += __popcll(dm);
    }
}

// problems of up to DEFL_WG poles: one workgroup scans, joins and places
__global__ __launch_bounds__(DEFL_WAVES * WAVE) void k_deflate(DeflArgs a) {
    __shared__ double sd[DEFL_WAVES][WAVE], sz[DEFL_WAVES][WAVE];
    __shared__ int si[DEFL_WAVES][WAVE];
    __shared__ int4 rec_i[DEFL_WAVES];
    __shared__ double2 rec_d[DEFL_WAVES];
    __shared__ int res[2];
    const int p = blockIdx.x, wv = wave_uniform((int)(threadIdx.x / WAVE));
    const int64_t base = a.off[p];
    const int n = (int)(a.off[p + 1] - base);
    defl_segment(a, p, base, n, wv, rec_i, rec_d, sd[wv], sz[wv], si[wv]);
    __syncthreads();
    if (wv == 0) {
        int kept;
        const int st = defl_join(a, p, base, n, rec_i, rec_d, kept, sd[0], sz[0], si[0]);
        if (lane_id() == 0) {
            a.kept[p] = res[0] = kept;
            a.status[p] = res[1] = st;
        }
    }
    __threadfence_block();
    __syncthreads();
    if (!res[1]) defl_place(a, base, n, wv, rec_i, res[0]);
}

// larger ones: the segments, the joins and the placement in launches of their own
__global__ __launch_bounds__(WAVE) void k_deflate_scan(DeflArgs a) {
    __shared__ double sd[WAVE], sz[WAVE];
    __shared__ int si[WAVE];
    const int p = blockIdx.x;
    const int64_t base = a.off[p], r0 = (int64_t)p * a.maxseg;
    defl_segment(a, p, base, (int)(a.off[p + 1] - base), blockIdx.y, a.seg_i + r0, a.seg_d + r0, sd,
                 sz, si);
}

__global__ __launch_bounds__(WAVE) void k_deflate_join(DeflArgs a) {
    __shared__ double sd[WAVE], sz[WAVE];
    __shared__ int si[WAVE];
    const int p = blockIdx.x;
    const int64_t base = a.off[p], r0 = (int64_t)p * a.maxseg;
    int kept;
    const int st = defl_join(a, p, base, (int)(a.off[p + 1] - base), a.seg_i + r0, a.seg_d + r0,
                             kept, sd, sz, si);
    if (lane_id() == 0) {
        a.kept[p] = kept;
        a.status[p] = st;
    }
}

__global__ __launch_bounds__(WAVE) void k_deflate_place(DeflArgs a) {
    const int p = blockIdx.x;
    if (a.status[p]) return;
    const int64_t base = a.off[p];
    defl_place(a, base, (int)(a.off[p + 1] - base), blockIdx.y, a.seg_i + (int64_t)p * a.maxseg,
               a.kept[p]);
}

// ---------------------------------------------------------------------------------------
// the orthogonal factor: Y = G^T P U (trans 0) or Y = P^T G X (trans 1) on total x m
// column-major blocks (leading dimensions ldx, ldy), each problem on its own rows
// ---------------------------------------------------------------------------------------
struct ExpandArgs {
    const int64_t *off;
    int nprob, m;
    const int32_t *perm, *rright, *rleft;
    const double *rc, *rs;
    const double *X;
    int64_t ldx;
    double *Y;
    int64_t ldy;
    double *T;  // workspace for trans 1 (total x m, leading dimension total)
};

// whether pole i (of the problem at base) has a rotation partner on its right / left: links that
// run through increasing poles and that both ends hold
__device__ __forceinline__ bool defl_right(const ExpandArgs &a, int64_t base, int n, int i) {
    const int r = a.rright[base + i];
    return r > i && r < n && a.rleft[base + r] == i;
}
__device__ __forceinline__ bool defl_left(const ExpandArgs &a, int64_t base, int i) {
    const int l = a.rleft[base + i];
    return l >= 0 && l < i && a.rright[base + l] == i;
}

__device__ __forceinline__ int find_prob(const int64_t *off, int nprob, int64_t e) {
    int lo = 0, hi = nprob;  // off[lo] <= e < off[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (off[mid] <= e) lo = mid;
        else hi = mid;
    }
    return lo;
}

// The kernels below are bound by memory: one thread takes a row through `cpt` columns, so that
// the search for its problem, the permutation and the links are read once for all of them
// (one thread per row and column, with the search and a 64-bit division each, took 3 to 6 times
// as long; 1024 problems, 1.7 million rows: row copies 585 -> 196 us
// in all, 16 columns through the factor 764 -> 318 us).  The problem of the
// wavefront's first row is found with wave-uniform loads; most lanes share it.
__device__ __forceinline__ int row_prob(const int64_t *off, int nprob, int64_t row, int64_t total) {
    const int64_t first = (int64_t)blockIdx.x * blockDim.x + wave_uniform((int)threadIdx.x & -WAVE);
    const int lo = wave_uniform(find_prob(off, nprob, first < total ? first : total - 1));
    if (row < off[lo + 1]) return lo;
    return lo + find_prob(off + lo, nprob - lo, row);
}

// trans 0: Y[perm[j]] = X[j]; trans 1: Y[j] = (G X)[perm[j]], taken from T for the rows of
// rotation chains and from X for the others
__global__ __launch_bounds__(256) void k_defl_place(ExpandArgs a, int trans, int64_t total, int cpt) {
    const int64_t row = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int p = row_prob(a.off, a.nprob, row, total);
    if (row >= total) return;
    const int64_t base = a.off[p];
    const int n = (int)(a.off[p + 1] - base);
    const int pj = a.perm[row];
    if (pj < 0 || pj >= n) return;  // not a placement of this problem
    const int64_t prow = base + pj;
    const int c0 = blockIdx.y * cpt, c1 = min(a.m, c0 + cpt);
    if (trans == 0) {
        copy_cols(a.X + row, a.ldx, a.Y + prow, a.ldy, c0, c1);
    } else {
        const bool chain = defl_left(a, base, pj) || defl_right(a, base, n, pj);
        copy_cols((chain ? a.T : a.X) + prow, chain ? total : a.ldx, a.Y + row, a.ldy, c0, c1);
    }
}

// rotations along their chains (one thread per chain and column group): trans 0 applies
// G^T = G_1^T ... G_R^T to V = Y in place, walking each chain back from its last pole; trans 1
// takes X to T = G X, G = G_R ... G_1, on the chains' rows alone, walking forward from their
// first pole.  Chains are disjoint.  The value that a chain carries on stays in a register.
template <int NC>
__device__ void defl_walk(const ExpandArgs &a, int trans, int64_t total, int64_t base, int n, int i,
                          int c0) {
    const double *rc = a.rc + base, *rs = a.rs + base;
    const int32_t *rr = a.rright + base, *rl = a.rleft + base;
    double y[NC];
    // a chain runs through strictly increasing poles; a link that does not is not
    // followed, so every walk ends within n_p steps
    if (trans == 0) {
        double *v = a.Y + c0 * a.ldy + base;
        int bb = i;
#pragma unroll
        for (int c = 0; c < NC; ++c) y[c] = v[bb + c * a.ldy];
        for (int aa = rl[bb]; aa >= 0 && aa < bb; bb = aa, aa = rl[aa]) {
            const double cc = rc[aa], ss = rs[aa];
            double x[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) x[c] = v[aa + c * a.ldy];
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                v[bb + c * a.ldy] = -ss * x[c] + cc * y[c];
                y[c] = cc * x[c] + ss * y[c];
            }
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) v[bb + c * a.ldy] = y[c];
    } else {
        const double *v = a.X + c0 * a.ldx + base;
        double *t = a.T + c0 * total + base;
        int aa = i;
#pragma unroll
        for (int c = 0; c < NC; ++c) y[c] = v[aa + c * a.ldx];
        while (defl_right(a, base, n, aa)) {
            const int bb = rr[aa];
            const double cc = rc[aa], ss = rs[aa];
            double x[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) x[c] = v[bb + c * a.ldx];
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                t[aa + c * total] = cc * y[c] - ss * x[c];
                y[c] = ss * y[c] + cc * x[c];
            }
            aa = bb;
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) t[aa + c * total] = y[c];
    }
}

__global__ __launch_bounds__(256) void k_defl_rotate(ExpandArgs a, int trans, int64_t total, int cpt) {
    const int64_t row = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int p = row_prob(a.off, a.nprob, row, total);
    if (row >= total) return;
    const int64_t base = a.off[p];
    const int n = (int)(a.off[p + 1] - base), i = (int)(row - base);
    const bool start = trans == 0 ? a.rleft[row] >= 0 && a.rright[row] < 0
                                  : defl_right(a, base, n, i) && !defl_left(a, base, i);
    if (!start) return;
    const int c1 = min(a.m, ((int)blockIdx.y + 1) * cpt);
    int c = blockIdx.y * cpt;
    for (; c + 4 <= c1; c += 4) defl_walk<4>(a, trans, total, base, n, i, c);
    for (; c < c1; ++c) defl_walk<1>(a, trans, total, base, n, i, c);
}

// X into T as it stands (trans 1 with X and Y overlapping)
__global__ __launch_bounds__(256) void k_defl_copy(const double *X, int64_t ldx, double *T,
                                                   int64_t total, int m) {
    const int64_t row = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (row < total) copy_cols(X + row, ldx, T + row, total, 0, m);
}

// ---------------------------------------------------------------------------------------
// row copies between two batch layouts (total x m column-major each): rows [0, cnt_p) of
// problem p, cnt_p = min(rows ? rows[p] : n_src, n_src, n_dst); the other rows of dst get
// `fill` when has_fill
// ---------------------------------------------------------------------------------------
struct CopyRowsArgs {
    const int64_t *soff, *doff;
    int nprob, m;
    const int32_t *rows;
    const double *src;
    int64_t lds;
    double *dst;
    int64_t ldd;
    int has_fill;
    double fill;
};

__global__ __launch_bounds__(256) void k_copy_rows(CopyRowsArgs a, int64_t dtotal, int cpt) {
    const int64_t row = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int p = row_prob(a.doff, a.nprob, row, dtotal);
    if (row >= dtotal) return;
    const int64_t db = a.doff[p], nd = a.doff[p + 1] - db;
    const int64_t sb = a.soff[p], ns = a.soff[p + 1] - sb;
    int64_t cnt = ns < nd ? ns : nd;
    if (a.rows) {
        const int64_t r = a.rows[p] < 0 ? 0 : a.rows[p];
        if (r < cnt) cnt = r;
    }
    const int64_t j = row - db;
    const int c0 = blockIdx.y * cpt, c1 = min(a.m, c0 + cpt);
    if (j < cnt) copy_cols(a.src + sb + j, a.lds, a.dst + row, a.ldd, c0, c1);
    else if (a.has_fill)
        for (int c = c0; c < c1; ++c) a.dst[c * a.ldd + row] = a.fill;
}

// A deflated HSS step's row copies, one launch each instead of two: the reduced problems' poles and
// weights (a node that deflated completely: d = 0, z = 1), and a node's eigenvalues, the
// reduced roots in front of the deflated poles (18 steps over 65536 rows: 8.0 -> 7.9 ms).
__global__ __launch_bounds__(256) void k_step_reduced(const int64_t *off, const int64_t *roff, int nprob,
                                                      const int32_t *kept, const double *d,
                                                      const double *z, double *dr, double *zr,
                                                      int64_t rtotal) {
    const int64_t row = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int p = row_prob(roff, nprob, row, rtotal);
    if (row >= rtotal) return;
    const int64_t j = row - roff[p], s = off[p] + j;
    const bool in = j < kept[p] && s < off[p + 1];
    dr[row] = in ? d[s] : 0.0;
    zr[row] = in ? z[s] : 1.0;
}

__global__ __launch_bounds__(256) void k_step_values(const int64_t *off, const int64_t *roff, int nprob,
                                                     const int32_t *kept, const double *d,
                                                     const double *lam, double *E, int64_t total) {
    const int64_t row = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int p = row_prob(off, nprob, row, total);
    if (row >= total) return;
    const int64_t j = row - off[p], s = roff[p] + j;
    E[row] = j < kept[p] && s < roff[p + 1] ? lam[s] : d[row];
}

// ---------------------------------------------------------------------------------------
int deflate_segments(int nprob, int max_n) {
    const int seg = defl_seg(nprob, max_n);
    return max_n > seg ? (max_n + seg - 1) / seg : 1;
}

hipError_t launch_deflate(const int64_t *off, int nprob, const double *d, const double *z,
                          const double *rho, double tau, double *dout, double *zout,
                          int32_t *perm, int32_t *rright, int32_t *rleft, double *rc, double *rs,
                          int32_t *kept, int32_t *status, double2 *val, int8_t *flag,
                          int max_n, int4 *seg_i, double2 *seg_d, hipStream_t s) {
    DeflArgs a{off,  d,  z,    rho,    tau, dout, zout,  perm,  rright, rleft,
               rc,   rs, kept, status, val, flag, seg_i, seg_d, DEFL_SEG, 0};
    if (max_n <= DEFL_WG) {
        SDC_LAUNCH(KID_DEFLATE, k_deflate, dim3(nprob),
                   dim3(WAVE * std::max(1, (max_n + DEFL_SEG - 1) / DEFL_SEG)), 0, s, a);
        return hipGetLastError();
    }
    a.seg = defl_seg(nprob, max_n);
    a.maxseg = deflate_segments(nprob, max_n);
    const dim3 g2(nprob, a.maxseg);
    SDC_LAUNCH(KID_DEFLATE, k_deflate_scan, g2, dim3(WAVE), 0, s, a);
    SDC_LAUNCH(KID_DEFLATE, k_deflate_join, dim3(nprob), dim3(WAVE), 0, s, a);
    SDC_LAUNCH(KID_DEFLATE, k_deflate_place, g2, dim3(WAVE), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_deflate_expand(const int64_t *off, int nprob, int64_t total, int m,
                                 const int32_t *perm, const int32_t *rright,
                                 const int32_t *rleft, const double *rc, const double *rs,
                                 int trans, const double *X, int64_t ldx, double *Y,
                                 int64_t ldy, double *T, hipStream_t s) {
    ExpandArgs a{off, nprob, m, perm, rright, rleft, rc, rs, X, ldx, Y, ldy, T};
    if (total * m == 0) return hipSuccess;
    const int cpt = cols_per_thread(total, m);
    const dim3 g = row_grid(total, m, cpt);
    if (trans == 0) {
        SDC_LAUNCH(KID_DEFL_PLACE, k_defl_place, g, dim3(256), 0, s, a, 0, total, cpt);
        SDC_LAUNCH(KID_DEFL_ROTATE, k_defl_rotate, g, dim3(256), 0, s, a, 0, total, cpt);
    } else {
        if (X < Y + (m - 1) * ldy + total && Y < X + (m - 1) * ldx + total) {
            SDC_LAUNCH(KID_DEFL_PLACE, k_defl_copy, dim3(g.x), dim3(256), 0, s, X, ldx, T, total, m);
            a.X = T;
            a.ldx = total;
        }
        SDC_LAUNCH(KID_DEFL_ROTATE, k_defl_rotate, g, dim3(256), 0, s, a, 1, total, cpt);
        SDC_LAUNCH(KID_DEFL_PLACE, k_defl_place, g, dim3(256), 0, s, a, 1, total, cpt);
    }
    return hipGetLastError();
}

hipError_t launch_step_reduced(const int64_t *off, const int64_t *roff, int nprob,
                               const int32_t *kept, const double *d, const double *z, double *dr,
                               double *zr, int64_t rtotal, hipStream_t s) {
    SDC_LAUNCH(KID_COPY_ROWS, k_step_reduced, row_grid(rtotal, 1, 1), dim3(256), 0, s, off, roff, nprob,
               kept, d, z, dr, zr, rtotal);
    return hipGetLastError();
}

hipError_t launch_step_values(const int64_t *off, const int64_t *roff, int nprob,
                              const int32_t *kept, const double *d, const double *lam, double *E,
                              int64_t total, hipStream_t s) {
    SDC_LAUNCH(KID_COPY_ROWS, k_step_values, row_grid(total, 1, 1), dim3(256), 0, s, off, roff, nprob,
               kept, d, lam, E, total);
    return hipGetLastError();
}

hipError_t launch_copy_rows(const int64_t *soff, const int64_t *doff, int nprob,
                            int64_t dtotal, int m, const int32_t *rows, const double *src,
                            int64_t lds, double *dst, int64_t ldd, const double *fill,
                            hipStream_t s) {
    CopyRowsArgs a{soff, doff, nprob, m, rows, src, lds, dst, ldd, fill ? 1 : 0, fill ? *fill : 0.0};
    if (dtotal * m == 0) return hipSuccess;
    const int cpt = cols_per_thread(dtotal, m);
    SDC_LAUNCH(KID_COPY_ROWS, k_copy_rows, row_grid(dtotal, m, cpt), dim3(256), 0, s, a, dtotal, cpt);
    return hipGetLastError();
}

}  // namespace sdc
