// vectors.hip -- Loewner update vector and eigenvector normalisation for gfx950.
//
//   rho zhat_i^2 = prod_j (lambda_j - d_i) / prod_{j != i} (d_j - d_i)    (eq. lowner)
//   b_j          = (sum_i zhat_i^2 / (d_i - lambda_j)^2)^(-1/2)             (eq. b)
// Every lambda_j - d_i is formed from the solver's shifted representation as
// (d_{K_j} - d_i) + eta_j (eq. qk), so nearby roots keep their relative accuracy.
//
// The paper evaluates the Loewner products as exponentials of log sums through an FMM
// (eqs. lowner2, logv).  Here each lane keeps the numerator and denominator products of
// one pole as separate running products (two interleaved chains each) and strips their
// binary exponents every 8 factors per chain (frexp), accumulating the exponents in an
// integer; one division and one ldexp finish the pole.  No logarithms, and the 8-factor
// blocks cannot over- or underflow for factors between 2^-120 and 2^120.  Both products are
// homogeneous in the scale of the problem (n factors over n - 1), so a problem whose span
// s = d_{n-1} - d_0 + eta_{n-1} lies outside [2^-32, 2^32] has every factor multiplied by
// 2^-e (e the binary exponent of s, an exact scaling) and e added back at the end: the
// factors are then at most 2 in magnitude, and the result is the same, bit for bit, as for
// the problem scaled into range.  Factors below 2^-120 s (relative gaps or eta_k below
// about 7.5e-37 of the span) can still underflow a block.
#include "common.h"
#include "fmm.h"

namespace sdc {

// ke_j = (d_{K_j}, eta_j) for every root (origin indices are local to the problem)
__global__ __launch_bounds__(64) void k_pack_ke(VecArgs a) {
    const Tile t = a.tiles[blockIdx.x];
    const int64_t base = a.off[t.prob];
    const int n = (int)(a.off[t.prob + 1] - base);
    const int k = t.row0 + lane_id();
    if (k < n) {
        const int K = clamp_idx(a.origin[base + k], n);
        a.ke[base + k] = make_double2(a.d[base + K], a.eta[base + k]);
    }
}

__device__ __forceinline__ void renorm(double &num, double &den, int &E) {
    E += __builtin_amdgcn_frexp_exp(num) - __builtin_amdgcn_frexp_exp(den);
    num = __builtin_amdgcn_frexp_mant(num);
    den = __builtin_amdgcn_frexp_mant(den);
}

// products over roots j in [j0, j1); SKIP drops the denominator factor j == i.
// Two independent product chains (even and odd roots) keep the multiplies from waiting
// on each other; each strips its exponents after every 8 factors.  Roots come in blocks of 4
// through the scalar cache, into two register sets that alternate, so the next block's loads
// are in flight while this block is multiplied: 16 roots to a turn of the loop without a
// branch in it (a loop that tested for the end after each block spent more scalar
// instructions on moving the sets about than vector instructions on the factors).
// SC: every factor is multiplied by sg (a power of two) before it enters its product.
struct LwSet {
    double k[8], d[4];  // (d_K, eta) pairs and poles
};
__device__ __forceinline__ void lw_load(LwSet &s, const_double_ptr kp, const_double_ptr dp) {
#pragma unroll
    for (int u = 0; u < 8; ++u) s.k[u] = kp[u];
#pragma unroll
    for (int u = 0; u < 4; ++u) s.d[u] = dp[u];
}

template <bool SKIP, bool SC>
__device__ __forceinline__ void loewner_range(const_double2_ptr ke, const_double_ptr dd,
                                              int j0, int j1,
                                              int i, double di, double &num, double &den,
                                              int &E, double sg) {
    if (j0 >= j1) return;
    double na = 1.0, da = 1.0, nb = 1.0, db = 1.0;
    auto scl = [&](double f) { return SC ? f * sg : f; };
    auto block = [&](const LwSet &s, int j) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double fn = scl((s.k[2 * u] - di) + s.k[2 * u + 1]), fd = scl(s.d[u] - di);
            const double fk = SKIP && j + u == i ? 1.0 : fd;
            if (u & 1) {
                nb *= fn;
                db *= fk;
            } else {
                na *= fn;
                da *= fk;
            }
        }
    };
    auto strip = [&]() {
        renorm(na, da, E);
        renorm(nb, db, E);
    };
    int j = j0;
    if (j + 16 <= j1) {
        LwSet s0, s1;
        lw_load(s0, ke.p + 2 * (int64_t)j, dd + j);
        do {
            const const_double_ptr kp = ke.p + 2 * (int64_t)j, dp = dd + j;
            lw_load(s1, kp + 8, dp + 4);
            block(s0, j);
            lw_load(s0, kp + 16, dp + 8);
            block(s1, j + 4);
            lw_load(s1, kp + 24, dp + 12);
            block(s0, j + 8);
            const int jn = min(j + 16, j1 - 4);  // past the last turn: within the range, not used
            lw_load(s0, ke.p + 2 * (int64_t)jn, dd + jn);
            block(s1, j + 12);
            strip();
            j += 16;
        } while (j + 16 <= j1);
    }
    for (; j + 4 <= j1; j += 4) {
        LwSet s;
        lw_load(s, ke.p + 2 * (int64_t)j, dd + j);
        block(s, j);
    }
    strip();  // at most 6 factors per chain since the last one
    for (; j < j1; ++j) {  // at most 3 more factors per chain after the strip above
        const double2 kv = ke[j];
        na *= scl((kv.x - di) + kv.y);
        da *= SKIP && j == i ? 1.0 : scl(dd[j] - di);
    }
    num *= na * nb;  // mantissas in [0.5, 1) times at most 3 factors: no over- or underflow
    den *= da * db;
    renorm(num, den, E);
}

// The binary exponent e used to scale a problem's factors (0 when its span is in range):
// the span of poles and roots, d_{n-1} - d_0 + eta_{n-1}, read from the packed pairs.
__device__ __forceinline__ int loewner_scale(const_double2_ptr ke, const_double_ptr dd, int n) {
    const double2 kl = ke[n - 1];
    const double span = (kl.x - dd[0]) + kl.y;
    const int e = __builtin_amdgcn_frexp_exp(span);
    return (e < -32 || e > 32) ? e : 0;
}

// With S = blockDim.x / 64 > 1 wavefronts per tile, wavefront w takes the roots
// [n w / S, n (w+1) / S) and the partial results are combined in wavefront order.
__device__ __forceinline__ void split_range(int n, int &p0, int &p1) {
    const int S = blockDim.x / WAVE, wv = threadIdx.x / WAVE;
    p0 = wave_uniform((int)(((int64_t)n * wv) / S));
    p1 = wave_uniform((int)(((int64_t)n * (wv + 1)) / S));
}

__device__ void loewner_tile(const VecArgs &a, Tile t, double4 *red) {
    const int p = t.prob;
    const int64_t base = a.off[p];
    const int n = (int)(a.off[p + 1] - base);
    const int i = t.row0 + lane_id();
    const bool active = i < n;
    const int S = blockDim.x / WAVE, wv = threadIdx.x / WAVE;
    if (a.status[p] & ~SUPERDC_ST_NOCONV) {
        if (active && wv == 0) {
            const double nan = __builtin_nan("");
            a.zhat[base + i] = nan;
            a.dz[base + i] = make_double2(a.d[base + i], nan);
        }
        return;
    }
    const int ii = active ? i : n - 1;
    const_double2_ptr ke = as_const(a.ke + base);  // written by k_pack_ke
    const_double_ptr dd = as_const(a.d + base);
    const double di = a.d[base + ii];
    double num = 1.0, den = 1.0;
    int E = 0;
    int p0, p1;
    split_range(n, p0, p1);
    const int t1 = wave_uniform(min(t.row0 + TILE, n));
    const int es = wave_uniform(loewner_scale(ke, dd, n));
    if (es == 0) {
        loewner_range<false, false>(ke, dd, p0, min(t.row0, p1), ii, di, num, den, E, 1.0);
        loewner_range<true, false>(ke, dd, max(t.row0, p0), min(t1, p1), ii, di, num, den, E, 1.0);
        loewner_range<false, false>(ke, dd, max(t1, p0), p1, ii, di, num, den, E, 1.0);
    } else {  // every factor scaled by 2^-es; the ratio gains 2^-es, added back below
        const double sg = __builtin_ldexp(1.0, -es);
        loewner_range<false, true>(ke, dd, p0, min(t.row0, p1), ii, di, num, den, E, sg);
        loewner_range<true, true>(ke, dd, max(t.row0, p0), min(t1, p1), ii, di, num, den, E, sg);
        loewner_range<false, true>(ke, dd, max(t1, p0), p1, ii, di, num, den, E, sg);
        if (wv == 0) E += es;
    }
    if (S > 1) {
        red[wv * WAVE + lane_id()] = make_double4(num, den, (double)E, 0.0);
        __syncthreads();
        if (wv == 0) {
            for (int w = 1; w < S; ++w) {
                const double4 v = red[w * WAVE + lane_id()];
                num *= v.x;
                den *= v.y;
                E += (int)v.z;
                renorm(num, den, E);
            }
        }
        __syncthreads();
    }
    if (active && wv == 0) {
        const double R = ldexp(num / den, E);
        const double zi = a.z[base + i];
        const double zh = copysign(sqrt(R / a.rho[p]), zi);
        a.zhat[base + i] = zh;
        a.dz[base + i] = make_double2(di, zh);
    }
}

// ---------------------------------------------------------------------------------------
// Loewner products of the FMM problems: the near leaves of the lists exactly (the same
// renormalised products), the far boxes through their moment expansions
//     sum_{j in B} log((lambda_j - d_i) / (d_j - d_i)) = sum_k (-1)^(k+1) M_k r^k / k,
//     r = hw / (c - d_i),
// with a direct product over the box for the rare pole where |r| > 0.35.  Work items are
// 64-pole pieces of the target leaves; S wavefronts split the lists.
// ---------------------------------------------------------------------------------------
// M: coefficients (-1)^(k+1) M_k / k, as the moments are stored
__device__ __forceinline__ double lw_series(const_double_ptr M, double r) {
    double acc = 0.0;
#pragma unroll
    for (int k = FMML_K; k >= 1; --k) acc = __builtin_fma(acc, r, M[k - 1]);
    return acc * r;
}

// Poles and boxes are the same for the whole wavefront, so both come through the scalar cache
// and cost the vector units nothing but their arithmetic.  (Staged in LDS they cost three LDS
// reads a pole and 28 a box, which bound the launch, and an item ran in rounds of loads and
// barriers; the coefficients were formed per lane.  Measured, LDS -> scalar loads, us: a
// level of 4096 problems 2640 -> 2210; with the last root out of the boxes 1110.)
__device__ void loewner_fmm_tile(const VecArgs &a, const FmmArgs &f, const FmmlArgs &l, Tile t,
                                 double4 *red) {
    const int p = t.prob;
    const int64_t base = a.off[p];
    const int n = (int)(a.off[p + 1] - base);
    const int lane = lane_id();
    const int i = t.row0 + lane;
    const bool active = i < n;
    const int S = blockDim.x / WAVE, wv = wave_uniform((int)(threadIdx.x / WAVE));
    if (a.status[p] & ~SUPERDC_ST_NOCONV) {
        if (active && wv == 0) {
            const double nan = __builtin_nan("");
            a.zhat[base + i] = nan;
            a.dz[base + i] = make_double2(a.d[base + i], nan);
        }
        return;
    }
    const int ii = active ? i : n - 1;
    const_double2_ptr ke = as_const(a.ke + base);  // written by k_pack_ke
    const_double_ptr dd = as_const(a.d + base);
    const double di = a.d[base + ii];
    double num = 1.0, den = 1.0, far = 0.0;
    int E = 0;
    const int qf = f.fmm_of[p];
    const int L = wave_uniform(f.leaf_off[qf] + t.row0 / f.leaf);
    const int nn = wave_uniform(f.cnt[3 * (int64_t)L]);
    const int nl = wave_uniform(f.cnt[3 * (int64_t)L + 1]);
    const int nr = wave_uniform(f.cnt[3 * (int64_t)L + 2]);
    const int t0 = t.row0, t1 = wave_uniform(min(t.row0 + TILE, n));
    // a problem out of range has every factor scaled by sg = 2^-es (added back below)
    const int es = wave_uniform(loewner_scale(ke, dd, n));
    const double sg = __builtin_ldexp(1.0, -es);
    // far boxes: lane e holds the e-th (two registers: up to 2 FMM_FAR_MAX of them)
    static_assert(FMM_FAR_MAX == WAVE, "a lane per far box of a side");
    int gl = 0, gr = 0;
    if (lane < nl) gl = f.far_l[(int64_t)L * FMM_FAR_MAX + lane];
    if (lane < nr) gr = f.far_r[(int64_t)L * FMM_FAR_MAX + lane];
    // exact products over the near ranges (overflowed lists, rare: every pole), each split over
    // the wavefronts, the poles of this item dropping their own factor
    int top = 0;  // end of the near poles
    for (int e = 0; e < (nn < 0 ? 1 : nn); ++e) {
        const int lo0 = nn < 0 ? 0 : wave_uniform(f.near_lo[(int64_t)L * FMM_NEAR_MAX + e]);
        const int hi0 = nn < 0 ? n : wave_uniform(f.near_hi[(int64_t)L * FMM_NEAR_MAX + e]);
        top = hi0;
        const int lo = wave_uniform(lo0 + (int)(((int64_t)(hi0 - lo0) * wv) / S));
        const int hi = wave_uniform(lo0 + (int)(((int64_t)(hi0 - lo0) * (wv + 1)) / S));
        if (es == 0) {
            loewner_range<false, false>(ke, dd, lo, min(hi, t0), ii, di, num, den, E, 1.0);
            loewner_range<true, false>(ke, dd, max(lo, t0), min(hi, t1), ii, di, num, den, E, 1.0);
            loewner_range<false, false>(ke, dd, max(lo, t1), hi, ii, di, num, den, E, 1.0);
        } else {
            loewner_range<false, true>(ke, dd, lo, min(hi, t0), ii, di, num, den, E, sg);
            loewner_range<true, true>(ke, dd, max(lo, t0), min(hi, t1), ii, di, num, den, E, sg);
            loewner_range<false, true>(ke, dd, max(lo, t1), hi, ii, di, num, den, E, sg);
        }
    }
    // the last pole and its root are in no box's moments
    if (top < n && wv == 0) {
        const double2 kv = ke[n - 1];
        num *= ((kv.x - di) + kv.y) * sg;
        den *= (dd[n - 1] - di) * sg;
        renorm(num, den, E);
    }
    for (int e = wv; e < nl + nr && nn >= 0; e += S) {
        const int g = e < nl ? __builtin_amdgcn_readlane(gl, e) : __builtin_amdgcn_readlane(gr, e - nl);
        const const_double2_ptr geo = as_const(l.geo + g);
        const double2 gc = geo[0];
        const double r = gc.y * rcp_nr(gc.x - di);
        if (fabs(r) <= 0.35) {
            far += lw_series(as_const(l.mom + (int64_t)g * FMML_K), r);
        } else {  // too close for the expansion: the box's exact products for this lane
            const int hidx = g - f.box_off[qf];
            const int H = f.height[qf];
            int h = 0;
            while ((2 << h) - 1 <= hidx) ++h;
            const int bi = hidx - ((1 << h) - 1);
            const int64_t span = (int64_t)f.leaf << (H - h);
            const int lo = (int)min((int64_t)n, bi * span);
            const int hi = (int)min((int64_t)n - 1, (bi + 1) * span);
            for (int j = lo; j < hi; ++j) {  // j != i: a far box never holds pole i
                const double2 kv = ke[j];
                num *= ((kv.x - di) + kv.y) * sg;  // as many factors on both sides
                den *= (dd[j] - di) * sg;
                if ((j & 7) == 7) renorm(num, den, E);
            }
            renorm(num, den, E);
        }
    }
    if (es != 0 && wv == 0) E += es;
    if (S > 1) {
        red[wv * WAVE + lane_id()] = make_double4(num, den, (double)E, far);
        __syncthreads();
        if (wv == 0) {
            for (int w = 1; w < S; ++w) {
                const double4 v = red[w * WAVE + lane_id()];
                num *= v.x;
                den *= v.y;
                E += (int)v.z;
                far += v.w;
                renorm(num, den, E);
            }
        }
        __syncthreads();
    }
    if (active && wv == 0) {
        const double R = ldexp((num / den) * exp(far), E);
        const double zi = a.z[base + i];
        const double zh = copysign(sqrt(R / a.rho[p]), zi);
        a.zhat[base + i] = zh;
        a.dz[base + i] = make_double2(di, zh);
    }
}

__device__ void bnorm_tile(const VecArgs &a, Tile t, double4 *red) {
    const int p = t.prob;
    const int64_t base = a.off[p];
    const int n = (int)(a.off[p + 1] - base);
    const int j = t.row0 + lane_id();
    const bool active = j < n;
    const int S = blockDim.x / WAVE, wv = threadIdx.x / WAVE;
    if (a.status[p] & ~SUPERDC_ST_NOCONV) {
        if (active && wv == 0) a.bnorm[base + j] = __builtin_nan("");
        return;
    }
    const_double2_ptr dz = as_const(a.dz + base);  // written by k_loewner
    const double2 kv = a.ke[base + (active ? j : n - 1)];
    int p0, p1;
    split_range(n, p0, p1);
    // two poles share one reciprocal (the FP64 reciprocal issues at a quarter of the FMA
    // rate): zhat0/t0 = zhat0 t1 R and zhat1/t1 = zhat1 t0 R with R = 1/(t0 t1), squared after
    // the division (zhat^2 t^2 leaves the range where the quotient does not).  The products need
    // every |t| inside [2^-300, 2^300] (the range the solver's shared reciprocals use);
    // the smallest |t| of a root is |eta| (its origin is its nearest pole) and the largest
    // is at an end of the pole range.  A wavefront with a root outside takes one
    // reciprocal per pole.
    double s0 = 0.0, s1 = 0.0;
    int i = p0;
    bool paired = false;
    if (p0 < p1) {
        const double tmax = fmax(fabs((dz[p0].x - kv.x) - kv.y), fabs((dz[p1 - 1].x - kv.x) - kv.y));
        const bool ok = fabs(kv.y) >= 0x1p-300 && tmax <= 0x1p300;
        paired = __ballot(!ok) == 0ull;
    }
    if (paired) {
        for (; i + 2 <= p1; i += 2) {
            const double2 q0v = dz[i], q1v = dz[i + 1];
            const double t0 = (q0v.x - kv.x) - kv.y, t1 = (q1v.x - kv.x) - kv.y;
            const double R = rcp_nr(t0 * t1);
            const double q0 = q0v.y * t1 * R, q1 = q1v.y * t0 * R;
            s0 = __builtin_fma(q0, q0, s0);
            s1 = __builtin_fma(q1, q1, s1);
        }
    }
    for (; i + 2 <= p1; i += 2) {
        const double2 q0v = dz[i], q1v = dz[i + 1];
        const double q0 = q0v.y * rcp_nr((q0v.x - kv.x) - kv.y);
        const double q1 = q1v.y * rcp_nr((q1v.x - kv.x) - kv.y);
        s0 = __builtin_fma(q0, q0, s0);
        s1 = __builtin_fma(q1, q1, s1);
    }
    if (i < p1) {
        const double2 q0v = dz[i];
        const double q0 = q0v.y * rcp_nr((q0v.x - kv.x) - kv.y);
        s0 = __builtin_fma(q0, q0, s0);
    }
    double sum = s0 + s1;
    if (S > 1) {
        red[wv * WAVE + lane_id()] = make_double4(sum, 0.0, 0.0, 0.0);
        __syncthreads();
        if (wv == 0)
            for (int w = 1; w < S; ++w) sum += red[w * WAVE + lane_id()].x;
        __syncthreads();
    }
    if (active && wv == 0) a.bnorm[base + j] = 1.0 / sqrt(sum);
}

// zhat and b of a whole problem of at most VS_N poles in one workgroup, for batches of such
// problems: the packed roots, the poles and zhat stay in LDS.  Four wavefronts (eight beyond
// 128 poles), in as many shares of the factors (terms) as there are wavefronts to a tile of 64
// poles (roots).  The three launches it replaces took longer to issue than to run: one problem
// of 100 poles 16.7 -> 12.7 us a call, 512 of 128 19.4 -> 12.1, 4096 of 128 95 -> 56; at 256
// poles a single problem is slower this way (16 -> 18), so the line is below.
constexpr int VS_W = 8;  // wavefronts, at most
__global__ __launch_bounds__(WAVE * VS_W) void k_vectors_small(VecArgs a) {
    __shared__ double2 ke[VS_N];
    __shared__ double dd[VS_N], zh[VS_N];
    __shared__ double3 red[VS_W][WAVE];
    const int p = blockIdx.x, tid = threadIdx.x, lane = lane_id();
    const int64_t base = a.off[p];
    const int n = (int)(a.off[p + 1] - base);
    if (a.status[p] & ~SUPERDC_ST_NOCONV) {
        for (int j = tid; j < n; j += blockDim.x) a.zhat[base + j] = a.bnorm[base + j] = __builtin_nan("");
        return;
    }
    for (int j = tid; j < n; j += blockDim.x) {
        dd[j] = a.d[base + j];
        ke[j] = make_double2(a.d[base + clamp_idx(a.origin[base + j], n)], a.eta[base + j]);
    }
    __syncthreads();
    const int tiles = (n + WAVE - 1) / WAVE, S = (int)(blockDim.x / WAVE) / tiles;
    const int wv = wave_uniform(tid / WAVE), tile = wv / S, sh = wv % S;
    const int i = tile * WAVE + lane, ii = min(i, n - 1);
    const int j0 = n * sh / S, j1 = tile < tiles ? n * (sh + 1) / S : 0;
    // Loewner products (as loewner_tile; a problem in range has es = 0 and sg = 1, exact)
    const double2 kl = ke[n - 1];
    const int ex = __builtin_amdgcn_frexp_exp((kl.x - dd[0]) + kl.y);
    const int es = wave_uniform(ex < -32 || ex > 32 ? ex : 0);
    const double sg = __builtin_ldexp(1.0, -es);
    const double di = dd[ii];
    double na = 1.0, da = 1.0, nb = 1.0, db = 1.0;
    int E = 0, j = j0;
    auto factor = [&](int u, double &nu, double &de) {
        const double2 k = ke[u];
        nu *= ((k.x - di) + k.y) * sg;
        de *= u == ii ? 1.0 : (dd[u] - di) * sg;
    };
    for (; j + 16 <= j1; j += 16) {
#pragma unroll
        for (int u = 0; u < 16; u += 2) {
            factor(j + u, na, da);
            factor(j + u + 1, nb, db);
        }
        renorm(na, da, E);
        renorm(nb, db, E);
    }
    for (; j + 2 <= j1; j += 2) {  // at most 7 factors more per chain
        factor(j, na, da);
        factor(j + 1, nb, db);
    }
    if (j < j1) factor(j, na, da);
    renorm(na, da, E);
    renorm(nb, db, E);
    double num = na * nb, den = da * db;
    renorm(num, den, E);
    if (S > 1) {
        red[wv][lane] = make_double3(num, den, (double)E);
        __syncthreads();
        if (sh == 0)
            for (int w = 1; w < S; ++w) {
                const double3 v = red[wv + w][lane];
                num *= v.x;
                den *= v.y;
                E += (int)v.z;
                renorm(num, den, E);
            }
    }
    if (sh == 0 && i < n) {
        const double R = ldexp(num / den, E + es);
        const double v = copysign(sqrt(R / a.rho[p]), a.z[base + i]);
        a.zhat[base + i] = v;
        zh[i] = v;
    }
    __syncthreads();
    // b_i = (sum_j zhat_j^2 / (d_j - lambda_i)^2)^(-1/2) (as bnorm_tile)
    const double2 kv = ke[ii];
    double s0 = 0.0, s1 = 0.0;
    j = j0;
    const double tmax = fmax(fabs((dd[0] - kv.x) - kv.y), fabs((dd[n - 1] - kv.x) - kv.y));
    if (__ballot(!(fabs(kv.y) >= 0x1p-300 && tmax <= 0x1p300)) == 0ull) {
#pragma unroll 4
        for (; j + 2 <= j1; j += 2) {
            const double t0 = (dd[j] - kv.x) - kv.y, t1 = (dd[j + 1] - kv.x) - kv.y;
            const double R = rcp_nr(t0 * t1);
            const double q0 = zh[j] * t1 * R, q1 = zh[j + 1] * t0 * R;
            s0 = __builtin_fma(q0, q0, s0);
            s1 = __builtin_fma(q1, q1, s1);
        }
    }
    for (; j < j1; ++j) {
        const double q = zh[j] * rcp_nr((dd[j] - kv.x) - kv.y);
        s1 = __builtin_fma(q, q, s1);
    }
    double sum = s0 + s1;
    if (S > 1) {
        red[wv][lane] = make_double3(sum, 0.0, 0.0);
        __syncthreads();
        if (sh == 0)
            for (int w = 1; w < S; ++w) sum += red[wv + w][lane].x;
    }
    if (sh == 0 && i < n) a.bnorm[base + i] = 1.0 / sqrt(sum);
}

hipError_t launch_vectors_small(const VecArgs &a, int nprob, int max_n, hipStream_t s) {
    if (max_n > VS_N) return hipErrorInvalidValue;
    SDC_LAUNCH(KID_LOEWNER, k_vectors_small, dim3(nprob), dim3(WAVE * (max_n <= 128 ? 4 : VS_W)), 0, s, a);
    return hipGetLastError();
}

// blockDim.x = 64 S; dynamic LDS: one double4 per thread when S > 1
__global__ __launch_bounds__(1024) void k_loewner(VecArgs a) {
    extern __shared__ double4 red4[];
    loewner_tile(a, a.tiles[xcd_item()], red4);
}

__global__ __launch_bounds__(1024) void k_bnorm(VecArgs a) {
    extern __shared__ double4 red4[];
    bnorm_tile(a, a.tiles[xcd_item()], red4);
}

__global__ __launch_bounds__(1024) void k_loewner_fmm(VecArgs a, FmmArgs f, FmmlArgs l) {
    extern __shared__ double4 red4[];
    loewner_fmm_tile(a, f, l, a.tiles[xcd_item()], red4);
}

hipError_t launch_pack_ke(const VecArgs &a, hipStream_t s) {
    if (a.ntiles <= 0) return hipSuccess;
    SDC_LAUNCH(KID_PACK, k_pack_ke, dim3(a.ntiles), dim3(64), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_loewner_fmm(const VecArgs &a, const FmmArgs &f, const FmmlArgs &l, int split,
                              hipStream_t s) {
    if (a.ntiles <= 0) return hipSuccess;
    const size_t lds = split > 1 ? sizeof(double4) * WAVE * split : 0;
    SDC_LAUNCH(KID_LOEWNER_FMM, k_loewner_fmm, dim3(a.ntiles), dim3(WAVE * split), lds,
               s, a, f, l);
    return hipGetLastError();
}

hipError_t launch_loewner(const VecArgs &a, int split, hipStream_t s) {
    if (a.ntiles <= 0) return hipSuccess;
    const size_t lds = split > 1 ? sizeof(double4) * WAVE * split : 0;
    SDC_LAUNCH(KID_LOEWNER, k_loewner, dim3(a.ntiles), dim3(WAVE * split), lds, s, a);
    return hipGetLastError();
}

hipError_t launch_bnorm(const VecArgs &a, int split, hipStream_t s) {
    if (a.ntiles <= 0) return hipSuccess;
    const size_t lds = split > 1 ? sizeof(double4) * WAVE * split : 0;
    SDC_LAUNCH(KID_BNORM, k_bnorm, dim3(a.ntiles), dim3(WAVE * split), lds, s, a);
    return hipGetLastError();
}

}  // namespace sdc
