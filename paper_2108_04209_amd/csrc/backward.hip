// backward.hip -- adjoint of the rank-one eigensolver on gfx950 (not in the paper).
//
// With r_ik = 1/((d_i - d_{K_k}) - eta_k) (the solver's shifted form), S_k = sum_i z_i^2 r_ik^2,
// b_k = S_k^(-1/2), q_ik = b_k z_i r_ik and p_k = q_k^T u = b_k h_k, h_k = sum_i u_i z_i r_ik,
// implicit differentiation of f(lambda_k) = 1 + rho sum_i z_i^2/(d_i - lambda_k) = 0 gives
//   dlambda_k/dd_i = z_i^2 r_ik^2 / S_k, dlambda_k/dz_i = -2 z_i r_ik / S_k,
//   dlambda_k/drho = 1/(rho^2 S_k),
// and the explicit derivatives of p_k follow from those of h_k and b_k.  Collecting terms,
//   lbar_k  = g_lam_k + g_p_k (b_k H2_k - h_k b_k^3 S3_k),  H2 = sum u z r^2, S3 = sum z^2 r^3
//   alpha_k = lbar_k b_k^2,  beta_k = g_p_k b_k,  gamma_k = g_p_k h_k b_k^3
//   g_d_i   = z_i^2 sum_k alpha_k r^2 - u_i z_i sum_k beta_k r^2 + z_i^2 sum_k gamma_k r^3
//   g_z_i   = -2 z_i sum_k alpha_k r + u_i sum_k beta_k r - z_i sum_k gamma_k r^2
//   g_rho   = sum_k alpha_k / rho^2
// Pass 1 (one lane per root) forms the root sums over poles; pass 2 (one lane per pole)
// forms the six Cauchy-like sums over roots; pass 3 reduces g_rho per problem.
#include "fmm_far.h"

namespace sdc {

// a root's cotangents from its sums
template <bool PROJ>
__device__ __forceinline__ void bwd_root_out(const BwdArgs &a, int64_t k, double dK, double eta,
                                             double S, double S3, double h, double H2) {
    const double b = 1.0 / sqrt(S);
    const double b2 = b * b;
    double lbar = a.g_lam ? a.g_lam[k] : 0.0;
    double beta = 0.0, gamma = 0.0;
    if (PROJ) {
        const double gp = a.g_proj[k];
        lbar += gp * (b * H2 - h * b2 * b * S3);
        beta = gp * b;
        gamma = gp * h * b2 * b;
    }
    a.rk[k] = make_double4(dK, eta, lbar * b2, beta);
    a.gk[k] = gamma;
}

// a pole's gradients from its sums
template <bool PROJ>
__device__ __forceinline__ void bwd_pole_out(const BwdArgs &a, int64_t i, double A1, double A2,
                                             double A3, double B1, double B2, double B3) {
    const double zi = a.z[i];
    double gd = zi * zi * (A1 + A3);
    double gz = -2.0 * zi * B1 - zi * B3;
    if (PROJ) {
        const double ui = a.u[i];
        gd -= ui * zi * A2;
        gz += ui * B2;
    }
    a.g_d[i] = gd;
    a.g_z[i] = gz;
}

template <bool PROJ>
__device__ void bwd_roots_tile(const BwdArgs &a, Tile t, double4 *red) {
    const int p = t.prob;
    const int64_t base = a.off[p];
    const int n = (int)(a.off[p + 1] - base);
    const int k = t.row0 + lane_id();
    const bool active = k < n;
    const int kk = active ? k : n - 1;
    const bool bad = (a.status[p] & ~SUPERDC_ST_NOCONV) != 0;
    const double dK = a.d[base + clamp_idx(a.origin[base + kk], n)];
    const double eta = a.eta[base + kk];
    const_double_ptr d = as_const(a.d + base);
    const_double_ptr z = as_const(a.z + base);
    const_double_ptr u = as_const(PROJ ? a.u + base : a.z + base);
    double S = 0.0, S3 = 0.0, h = 0.0, H2 = 0.0;
    const int SW = blockDim.x / WAVE, wv = threadIdx.x / WAVE;
    const int i0 = wave_uniform((int)(((int64_t)n * wv) / SW));
    const int i1 = wave_uniform((int)(((int64_t)n * (wv + 1)) / SW));
    if (!bad) {
        for (int i = i0; i < i1; ++i) {
            const double r = rcp_nr((d[i] - dK) - eta);
            const double zr = z[i] * r;
            const double t2 = zr * zr;
            S += t2;
            S3 = __builtin_fma(t2, r, S3);
            if (PROJ) {
                const double uzr = u[i] * zr;
                h += uzr;
                H2 = __builtin_fma(uzr, r, H2);
            }
        }
    }
    if (SW > 1) {  // combine the wavefronts' partial sums in order
        red[wv * WAVE + lane_id()] = make_double4(S, S3, h, H2);
        __syncthreads();
        if (wv == 0)
            for (int w = 1; w < SW; ++w) {
                const double4 v = red[w * WAVE + lane_id()];
                S += v.x;
                S3 += v.y;
                h += v.z;
                H2 += v.w;
            }
        __syncthreads();
    }
    if (!active || wv != 0) return;
    const double nan = __builtin_nan("");
    if (bad) {
        a.rk[base + k] = make_double4(dK, eta, nan, nan);
        a.gk[base + k] = nan;
        return;
    }
    bwd_root_out<PROJ>(a, base + k, dK, eta, S, S3, h, H2);
}

template <bool PROJ>
__device__ void bwd_poles_tile(const BwdArgs &a, Tile t, double4 *red) {
    const int p = t.prob;
    const int64_t base = a.off[p];
    const int n = (int)(a.off[p + 1] - base);
    const int i = t.row0 + lane_id();
    const bool active = i < n;
    const int ii = active ? i : n - 1;
    const int SW = blockDim.x / WAVE, wv = threadIdx.x / WAVE;
    if (a.status[p] & ~SUPERDC_ST_NOCONV) {
        if (active && wv == 0) {
            a.g_d[base + i] = __builtin_nan("");
            a.g_z[base + i] = __builtin_nan("");
        }
        return;
    }
    const int k0 = wave_uniform((int)(((int64_t)n * wv) / SW));
    const int k1 = wave_uniform((int)(((int64_t)n * (wv + 1)) / SW));
    const double di = a.d[base + ii];
    const_double4_ptr rk = as_const(a.rk + base);  // written by the roots pass
    const_double_ptr gk = as_const(a.gk + base);
    double A1 = 0.0, A2 = 0.0, A3 = 0.0, B1 = 0.0, B2 = 0.0, B3 = 0.0;
    for (int k = k0; k < k1; ++k) {
        const double4 v = rk[k];
        const double r = rcp_nr((di - v.x) - v.y);
        const double r2 = r * r;
        A1 = __builtin_fma(v.z, r2, A1);
        B1 = __builtin_fma(v.z, r, B1);
        if (PROJ) {
            const double g = gk[k];
            A2 = __builtin_fma(v.w, r2, A2);
            B2 = __builtin_fma(v.w, r, B2);
            A3 = __builtin_fma(g * r2, r, A3);
            B3 = __builtin_fma(g, r2, B3);
        }
    }
    if (SW > 1) {  // combine the wavefronts' partial sums in order
        red[2 * (wv * WAVE + lane_id())] = make_double4(A1, A2, A3, B1);
        red[2 * (wv * WAVE + lane_id()) + 1] = make_double4(B2, B3, 0.0, 0.0);
        __syncthreads();
        if (wv == 0)
            for (int w = 1; w < SW; ++w) {
                const double4 u0 = red[2 * (w * WAVE + lane_id())];
                const double4 u1 = red[2 * (w * WAVE + lane_id()) + 1];
                A1 += u0.x;
                A2 += u0.y;
                A3 += u0.z;
                B1 += u0.w;
                B2 += u1.x;
                B3 += u1.y;
            }
        __syncthreads();
    }
    if (!active || wv != 0) return;
    bwd_pole_out<PROJ>(a, base + i, A1, A2, A3, B1, B2, B3);
}

// blockDim.x = 64 S; dynamic LDS: two double4 per thread when S > 1
template <bool PROJ, int PASS>
__global__ __launch_bounds__(1024) void k_bwd(BwdArgs a) {
    extern __shared__ double4 red4[];
    if (PASS == 1) bwd_roots_tile<PROJ>(a, a.tiles[xcd_item()], red4);
    else bwd_poles_tile<PROJ>(a, a.tiles[xcd_item()], red4);
}

// ---------------------------------------------------------------------------------------
// The same sums through the FMM, for the large problems: near sources directly in the shifted
// form, far boxes through equivalent sources.  The equivalent weights of a box don't depend on
// the kernel, so those of (z^2, u z) serve the roots' four sums and those of (alpha, beta,
// gamma) the poles' six.  One lane per target, S wavefronts per item of 64 targets; the far
// field of the boxes away from the targets' interval goes through its nodes (fmm_far.h).
// Bound by the FP64 pipe, as the direct sums: 1024 problems of 256 to 4096 roots with
// projections took those 7.7 ms at 93 % of it; here 1.4 ms, 0.3 ms for the weights of the boxes
// and 0.3 ms for the problems below the crossover.  The boxes lie 3 widths away and their nodes
// are offsets from their centres, so that the far field is as exact as the direct sums: gradients
// of single eigenvalues of 2048 to 8192 roots, entry by entry against long double, g_d off by
// 2.4e-15 at most and 5.2e-16 rms (direct 3.2e-15 and 6.8e-16), g_z 2.2e-15 and 4.9e-16 (3.0e-15
// and 6.6e-16); with boxes from 1.5 widths on, 2.0e-13 and 8.9e-15 at most.
// ---------------------------------------------------------------------------------------
template <bool PROJ, int PASS>
struct BwdFar {
    static constexpr int NF = PASS == 1 ? (PROJ ? 4 : 1) : (PROJ ? 6 : 2);  // sums
    static constexpr int NW = PASS == 1 ? (PROJ ? 2 : 1) : (PROJ ? 3 : 1);  // weights
    // a source's terms with reciprocal difference r and weights w
    static __device__ __forceinline__ void add(double r, const double (&w)[NW], double (&acc)[NF]) {
        const double r2 = r * r;
        if constexpr (PASS == 1) {  // S, S3, h, H2
            const double t2 = w[0] * r2;
            acc[0] += t2;
            if constexpr (PROJ) {
                acc[1] = __builtin_fma(t2, r, acc[1]);
                const double t1 = w[1] * r;
                acc[2] += t1;
                acc[3] = __builtin_fma(t1, r, acc[3]);
            }
        } else {  // A1, B1, A2, B2, A3, B3
            acc[0] = __builtin_fma(w[0], r2, acc[0]);
            acc[1] = __builtin_fma(w[0], r, acc[1]);
            if constexpr (PROJ) {
                acc[2] = __builtin_fma(w[1], r2, acc[2]);
                acc[3] = __builtin_fma(w[1], r, acc[3]);
                const double g2 = w[2] * r2;
                acc[4] = __builtin_fma(g2, r, acc[4]);
                acc[5] += g2;
            }
        }
    }
    int fbox[2 * FMM_FAR_MAX];
    int nexp;
    double gsum[8][NF][FMM_P];  // far field at the nodes, per wavefront (at most 8)
};

template <bool PROJ, int PASS>
__device__ void bwd_fmm_item(const BwdArgs &a, const FmmArgs &f, const FmmVec &v, Tile t,
                             BwdFar<PROJ, PASS> &sh, double *red) {
    using Far = BwdFar<PROJ, PASS>;
    constexpr int NF = Far::NF, NW = Far::NW;
    const int p = t.prob;
    const int64_t base = a.off[p];
    const int n = (int)(a.off[p + 1] - base);
    const int lane = lane_id();
    const int S = blockDim.x / WAVE, wv = wave_uniform((int)(threadIdx.x / WAVE));
    const int j = t.row0 + lane;
    const bool active = j < n;
    const int jj = active ? j : n - 1;
    const bool bad = (a.status[p] & ~SUPERDC_ST_NOCONV) != 0;
    // the target x = x0 + x1 (a root's d_K + eta, or a pole)
    const double x0 = PASS == 1 ? a.d[base + clamp_idx(a.origin[base + jj], n)] : a.d[base + jj];
    const double x1 = PASS == 1 ? a.eta[base + jj] : 0.0;
    if (bad) {
        const double nan = __builtin_nan("");
        if (active && wv == 0) {
            if (PASS == 1) {
                a.rk[base + j] = make_double4(x0, x1, nan, nan);
                a.gk[base + j] = nan;
            } else {
                a.g_d[base + j] = nan;
                a.g_z[base + j] = nan;
            }
        }
        return;
    }
    const int L = wave_uniform(f.leaf_off[f.fmm_of[p]] + t.row0 / f.leaf);
    const int nn = wave_uniform(f.cnt[3 * (int64_t)L]);
    const int nl = wave_uniform(f.cnt[3 * (int64_t)L + 1]);
    const int nr = wave_uniform(f.cnt[3 * (int64_t)L + 2]);
    const const_double_ptr d = as_const(a.d + base), z = as_const(a.z + base);
    const const_double_ptr u = as_const(PROJ ? a.u + base : a.z + base);
    const const_double4_ptr rk = as_const(a.rk + base);  // PASS 2: written by the roots' pass
    const const_double_ptr gk = as_const(a.gk + base);
    double acc[NF];
#pragma unroll
    for (int c = 0; c < NF; ++c) acc[c] = 0.0;
    int64_t ent = 0;  // sources this wavefront sums per target (kernel timing)
    // roots: two poles with one reciprocal while every |t| lies inside [2^-300, 2^300] (the
    // smallest is |eta|, the largest at an end of the problem)
    const bool pair = PASS == 1 &&
                      __ballot(fabs(x1) < 0x1p-300 ||
                               fmax(fabs((d[0] - x0) - x1), fabs((d[n - 1] - x0) - x1)) > 0x1p300) == 0ull;
    auto near = [&](int lo, int hi) {
        lo = wave_uniform(lo);
        hi = wave_uniform(hi);
        ent += hi > lo ? hi - lo : 0;
        if constexpr (PASS == 1) {
            // squared after the division (z^2 r^2 can leave the range)
            auto pole = [&](int i, double r) {
                const double zr = z[i] * r;
                const double t2 = zr * zr;
                acc[0] += t2;
                if constexpr (PROJ) {
                    acc[1] = __builtin_fma(t2, r, acc[1]);
                    const double t1 = u[i] * zr;
                    acc[2] += t1;
                    acc[3] = __builtin_fma(t1, r, acc[3]);
                }
            };
            int i = lo;
            if (pair) {
#pragma unroll 2
                for (; i + 2 <= hi; i += 2) {
                    const double t0 = (d[i] - x0) - x1, t1 = (d[i + 1] - x0) - x1;
                    const double R = rcp_nr(t0 * t1);
                    pole(i, t1 * R);
                    pole(i + 1, t0 * R);
                }
            }
            for (; i < hi; ++i) pole(i, rcp_nr((d[i] - x0) - x1));
        } else {
            // four roots to a set of scalar loads, the next set's in flight
            struct Set {
                double4 q[4];
                double g[4];
            };
            auto load = [&](Set &s, int k) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    s.q[u] = rk[k + u];
                    s.g[u] = PROJ ? gk[k + u] : 0.0;
                }
            };
            auto root = [&](const double4 &q, double g) {
                double w[NW];
                w[0] = q.z;
                if constexpr (PROJ) {
                    w[1] = q.w;
                    w[2] = g;
                }
                Far::add(rcp_nr((x0 - q.x) - q.y), w, acc);
            };
            int k = lo;
            if (k + 8 <= hi) {
                Set s0, s1;
                load(s0, k);
                do {
                    load(s1, k + 4);
#pragma unroll
                    for (int u = 0; u < 4; ++u) root(s0.q[u], s0.g[u]);
                    load(s0, min(k + 8, hi - 4));  // past the last turn: in the range, not used
#pragma unroll
                    for (int u = 0; u < 4; ++u) root(s1.q[u], s1.g[u]);
                    k += 8;
                } while (k + 8 <= hi);
            }
            for (; k < hi; ++k) root(rk[k], PROJ ? gk[k] : 0.0);
        }
    };
    if (nn < 0) {  // lists overflowed: every source directly, split over the wavefronts
        near((int)(((int64_t)n * wv) / S), (int)(((int64_t)n * (wv + 1)) / S));
    } else {
        for (int e = 0; e < nn; ++e) {
            const int lo0 = wave_uniform(f.near_lo[(int64_t)L * FMM_NEAR_MAX + e]);
            const int hi0 = wave_uniform(f.near_hi[(int64_t)L * FMM_NEAR_MAX + e]);
            near(lo0 + (int)(((int64_t)(hi0 - lo0) * wv) / S),
                 lo0 + (int)(((int64_t)(hi0 - lo0) * (wv + 1)) / S));
        }
        constexpr double sg = PASS == 1 ? 1.0 : -1.0;  // t: source - root, pole - source
        const double2 iv = fv_interval(v, base, n, t.row0, min(t.row0 + WAVE, n) - 1);
        if (wv == 0) {
            const int k = fv_split_far(f, v, L, nl, nr, iv, v.expand != 0, sh.fbox);
            if (lane == 0) sh.nexp = k;
        }
        __syncthreads();
        const int ne = wave_uniform(sh.nexp);
        if (ne > 0) {
            // lane: node lane % 16, every fourth source of a box
            const double off = iv.y * FV_NODE[lane & 15];
            double gs[NF];
#pragma unroll
            for (int c = 0; c < NF; ++c) gs[c] = 0.0;
            for (int e = wv; e < ne; e += S) {
                const int64_t g = sh.fbox[2 * FMM_FAR_MAX - 1 - e];
                const double c = v.vcen[g] - iv.x;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int64_t sq = g * FMM_P + 4 * k + (lane >> 4);
                    double w[NW];
#pragma unroll
                    for (int c = 0; c < NW; ++c) w[c] = v.vw[sq * NW + c];
                    Far::add(sg * rcp_nr((c + v.vnode[sq]) - off), w, gs);
                }
            }
#pragma unroll
            for (int c = 0; c < NF; ++c) {
                gs[c] += __shfl_xor(gs[c], 16);
                gs[c] += __shfl_xor(gs[c], 32);
                if (lane < FMM_P) sh.gsum[wv][c][lane] = gs[c];
            }
            wave_sync();
            // this wavefront's share of the far field at the targets
            const double tau = ((x0 - iv.x) + x1) / iv.y;
            double num[NF], den = 0.0;
#pragma unroll
            for (int c = 0; c < NF; ++c) num[c] = 0.0;
            for (int q = 0; q < FMM_P; ++q) {
                const double dl = tau - FV_NODE[q];
                // a target on a node: that node's term outweighs the others
                const double b = FV_BARY[q] * rcp_nr(dl == 0.0 ? 0x1p-200 : dl);
                den += b;
#pragma unroll
                for (int c = 0; c < NF; ++c) num[c] = __builtin_fma(b, sh.gsum[wv][c][q], num[c]);
            }
            const double iden = 1.0 / den;
#pragma unroll
            for (int c = 0; c < NF; ++c) acc[c] = __builtin_fma(num[c], iden, acc[c]);
            if (v.work && lane == 0)
                atomicAdd(v.work, (unsigned long long)((ne - wv + S - 1) / S) * FMM_P * FMM_P * (3 * NF) +
                                      (unsigned long long)(WAVE * FMM_P * 2 * NF));
        }
        for (int e = wv; e < nl + nr - ne; e += S) {
            const int g = wave_uniform(sh.fbox[e]);
            const const_double_ptr nd = as_const(v.vnode + (int64_t)g * FMM_P);
            const const_double_ptr ww = as_const(v.vw + (int64_t)g * FMM_P * NW);
            const double c = (v.vcen[g] - x0) - x1;
            ent += FMM_P;
#pragma unroll 4
            for (int q = 0; q < FMM_P; ++q) {
                double w[NW];
#pragma unroll
                for (int c = 0; c < NW; ++c) w[c] = ww[q * NW + c];
                Far::add(sg * rcp_nr(c + nd[q]), w, acc);
            }
        }
    }
    if (v.work && lane == 0)  // kernel timing: algorithmic flops of this wavefront's share
        atomicAdd(v.work, (unsigned long long)__popcll(__ballot(active)) * (unsigned long long)ent *
                              (3 * NF));
    if (S > 1) {
        if (wv > 0)
#pragma unroll
            for (int c = 0; c < NF; ++c) red[((wv - 1) * NF + c) * WAVE + lane] = acc[c];
        __syncthreads();
        if (wv == 0)
            for (int w = 1; w < S; ++w)
#pragma unroll
                for (int c = 0; c < NF; ++c) acc[c] += red[((w - 1) * NF + c) * WAVE + lane];
    }
    if (!active || wv != 0) return;
    if constexpr (PASS == 1) {
        if constexpr (PROJ) bwd_root_out<true>(a, base + j, x0, x1, acc[0], acc[1], acc[2], acc[3]);
        else bwd_root_out<false>(a, base + j, x0, x1, acc[0], 0.0, 0.0, 0.0);
    } else {
        if constexpr (PROJ)
            bwd_pole_out<true>(a, base + j, acc[0], acc[2], acc[4], acc[1], acc[3], acc[5]);
        else
            bwd_pole_out<false>(a, base + j, acc[0], 0.0, 0.0, acc[1], 0.0, 0.0);
    }
}

// blockDim.x = 64 S; dynamic LDS: S - 1 wavefronts' sums
template <bool PROJ, int PASS>
__global__ __launch_bounds__(512) void k_bwd_fmm(BwdArgs a, FmmArgs f, FmmVec v) {
    extern __shared__ double red[];
    __shared__ BwdFar<PROJ, PASS> sh;
    bwd_fmm_item<PROJ, PASS>(a, f, v, a.tiles[xcd_item()], sh, red);
}

// g_rho[p] = sum_k alpha_k / rho_p^2, fixed-order block reduction
__global__ __launch_bounds__(256) void k_bwd_rho(BwdArgs a, int prob_first) {
    const int p = prob_first + blockIdx.x;
    const int64_t base = a.off[p];
    const int n = (int)(a.off[p + 1] - base);
    double s = 0.0;
    for (int k = threadIdx.x; k < n; k += blockDim.x) s += a.rk[base + k].z;
    for (int o = WAVE / 2; o > 0; o >>= 1) s += __shfl_xor(s, o);
    __shared__ double sw[4];
    if (lane_id() == 0) sw[threadIdx.x / WAVE] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < (int)(blockDim.x / WAVE); ++w) t += sw[w];
        const double rho = a.rho[p];
        a.g_rho[p] = (a.status[p] & ~SUPERDC_ST_NOCONV) ? __builtin_nan("") : t / (rho * rho);
    }
}

hipError_t launch_backward(const BwdArgs &a, int split, hipStream_t s) {
    if (a.ntiles <= 0) return hipSuccess;
    const bool proj = a.g_proj != nullptr;
    const dim3 g(a.ntiles), blk(WAVE * split);
    const size_t lds = split > 1 ? 2 * sizeof(double4) * WAVE * split : 0;
    if (proj) {
        SDC_LAUNCH(KID_BWD, (k_bwd<true, 1>), g, blk, lds, s, a);
        SDC_LAUNCH(KID_BWD, (k_bwd<true, 2>), g, blk, lds, s, a);
    } else {
        SDC_LAUNCH(KID_BWD, (k_bwd<false, 1>), g, blk, lds, s, a);
        SDC_LAUNCH(KID_BWD, (k_bwd<false, 2>), g, blk, lds, s, a);
    }
    return hipGetLastError();
}

hipError_t launch_backward_fmm(const BwdArgs &a, const FmmArgs &f, const FmmVec &v0, int split,
                               int num_cu, hipStream_t s) {
    if (a.ntiles <= 0) return hipSuccess;
    const bool proj = a.g_proj != nullptr;
    FmmVec v = v0;
    if (v.m != (v.kern == 3 ? (proj ? 2 : 1) : (proj ? 3 : 1)) || split > 8) return hipErrorInvalidValue;
    v.work = trace_work(KID_BWD_FMM);
    v.sep_t = FV_SEP_BWD;
    v.expand = a.ntiles >= FV_EXPAND_PER_CU * num_cu;
    const dim3 g(a.ntiles), blk(WAVE * split);
#define SDC_BWD(P, K)                                                                   \
    {                                                                                   \
        constexpr int nf = (BwdFar<P, K>::NF);                                          \
        SDC_LAUNCH(KID_BWD_FMM, (k_bwd_fmm<P, K>), g, blk,                              \
                   sizeof(double) * WAVE * (split - 1) * nf, s, a, f, v);               \
    }
    if (v.kern == 3) {
        if (proj) SDC_BWD(true, 1)
        else SDC_BWD(false, 1)
    } else {
        if (proj) SDC_BWD(true, 2)
        else SDC_BWD(false, 2)
    }
#undef SDC_BWD
    return hipGetLastError();
}

hipError_t launch_backward_rho(const BwdArgs &a, int prob_first, int nprob, hipStream_t s) {
    if (nprob <= 0) return hipSuccess;
    SDC_LAUNCH(KID_BWD_RHO, k_bwd_rho, dim3(nprob), dim3(256), 0, s, a, prob_first);
    return hipGetLastError();
}

}  // namespace sdc
