// apply.hip -- Y = Qhat X or Qhat^T X for the Cauchy-like eigenvector matrix on gfx950.
//
//   Qhat = diag(zhat) C diag(b),  C_ij = 1/((d_i - d_{K_j}) - eta_j)     (eqs. qscale, qk)
//   Y = Qhat X   : Y_i = zhat_i sum_j C_ij (b_j X_j)       (Alg. 4, untransposed branch)
//   Y = Qhat^T X : Y_j = b_j    sum_i C_ij (zhat_i X_i)    (Alg. 3 Z-update, Alg. 4)
//
// The product is a dense contraction whose left factor is generated, never stored.
// MFMA kernel: a team of 4 wavefronts owns 64 output rows (16 per wavefront) and a pass of 16,
// 32 or 64 columns; in small launches four teams share an item's reduction.  The reduction runs over 64-entry chunks:
// the scaled right-hand sides (b_s X_s or zhat_s X_s) and the per-entry pole data are
// staged in LDS, then each wavefront generates its 16x4 slice of C with one reciprocal
// per lane and feeds v_mfma_f64_16x16x4f64 against 4x16 slices of the staged block.
// VALU kernel (few right-hand sides): one output row per lane, the same staging, and
// plain FMAs; four wavefronts share a tile's reduction range.
#include "common.h"

namespace sdc {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int AP_ROWS = 64;   // output rows per workgroup
constexpr int AP_K = 64;      // reduction chunk
constexpr int AP_LD = AP_K + 4;  // the 16 columns x 4 rows of an MFMA step on different banks

// per-entry data of the reduction index s
template <int TRANS>
__device__ __forceinline__ void stage_entry(const ApplyArgs &a, int64_t base, int n, int s,
                                            double2 &sd, double &scale) {
    if (s < n) {
        if (TRANS == 0) {  // s runs over roots: (d_{K_s}, eta_s), scale b_s
            sd = make_double2(a.d[base + clamp_idx(a.origin[base + s], n)], a.eta[base + s]);
            scale = a.bnorm[base + s];
        } else {           // s runs over poles: (d_s, zhat_s), scale zhat_s
            sd = make_double2(a.d[base + s], a.zhat[base + s]);
            scale = a.zhat[base + s];
        }
    } else {
        sd = make_double2(0.0, 0.0);
        scale = 0.0;
    }
}

// raw data of one reduction chunk, held in registers while the previous chunk is
// multiplied: the first wavefront's threads hold the pole data of entry s0 + tid; every
// thread holds NCT * 4 right-hand-side values, element e = tid + 256 i (row e % 64 of the
// chunk, column e / 64 of the pass), and the scale of their row.  Every lane loads (rows and
// columns clamped into the problem and the pass), so that a chunk's loads are one run without
// branches, and nothing uses them before the chunk is stored: padding is set to zero and the
// scale multiplied in there.
template <int NCT>
struct ApplyStage {
    double2 sd;
    double sc;
    double x[NCT * 4];
};

template <int TRANS, int NCT>
__device__ __forceinline__ void apply_fetch(const ApplyArgs &a, int64_t base, int n, int s0,
                                            int c0, int ncols, int tid, ApplyStage<NCT> &st) {
    const int64_t s = base + min(s0 + tid % AP_K, n - 1);
    const double *x = a.X + s + (int64_t)c0 * a.ldx;
    st.sc = (TRANS == 0 ? a.bnorm : a.zhat)[s];
#pragma unroll
    for (int i = 0; i < NCT * 4; ++i)
        st.x[i] = x[(int64_t)min(tid / AP_K + 4 * i, ncols - 1) * a.ldx];
    if (wave_uniform(tid / WAVE) == 0) {
        if (TRANS == 0)  // s runs over roots: (d_{K_s}, eta_s)
            st.sd = make_double2(a.d[base + clamp_idx(a.origin[s], n)], a.eta[s]);
        else             // s runs over poles: (d_s, zhat_s)
            st.sd = make_double2(a.d[s], st.sc);
    }
}

template <int TRANS, int NCT>
__device__ __forceinline__ void apply_store(int n, int s0, int ncols, int tid,
                                            const ApplyStage<NCT> &st, double *Xs, double2 *Sd) {
    const bool in = s0 + tid % AP_K < n;
    if (wave_uniform(tid / WAVE) == 0)
        Sd[tid] = make_double2(st.sd.x, TRANS && !in ? 0.0 : st.sd.y);
#pragma unroll
    for (int i = 0; i < NCT * 4; ++i) {
        const int e = tid + 256 * i;
        Xs[(e / AP_K) * AP_LD + e % AP_K] =
            in && tid / AP_K + 4 * i < ncols ? st.sc * st.x[i] : 0.0;
    }
}

// FEW: one to three columns, as exact as the VALU kernel that takes them in larger launches.
// NCT: 16-column blocks per pass (the pass width is 16 NCT columns); this item's pass starts
// at column c0.  FB: form b beside the columns.  TEAMS teams of four wavefronts take the
// reduction's chunks in turn and add their sums in team order, for launches with too few items
// to fill the chip, up to two per CU (the levels of a 1024-row HSS conquer: 6.2 -> 5.3 us a
// launch on average; 8192 rows of 64 columns, 512 items: problems of 128 to 1024, 23 -> 21)
template <int NCT>
struct ApplyTeam {
    double Xs[2][16 * NCT * AP_LD];
    double2 Sd[2][AP_K];
};

template <int TRANS, int NCT, bool FB, int TEAMS, bool FEW>
__device__ void apply_tile_mfma(const ApplyArgs &a, Tile t, int c0, ApplyTeam<NCT> *sh) {
    const int p = t.prob;
    const int64_t base = a.off[p];
    const int n = (int)(a.off[p + 1] - base);
    const int lane = lane_id();
    const int wave = wave_uniform((int)(threadIdx.x / WAVE));
    const int tm = wave >> 2, wv = wave & 3;  // team, wavefront of the team
    const int tid = threadIdx.x & 255;        // thread of the team
    const int o0 = t.row0;
    const int ncols = min(16 * NCT, a.m - c0);
    if (a.status[p] & ~SUPERDC_ST_NOCONV) {
        const double nan = __builtin_nan("");
        for (int e = threadIdx.x; e < AP_ROWS * ncols; e += blockDim.x) {
            const int r = o0 + (e % AP_ROWS), c = c0 + e / AP_ROWS;
            if (r < n) a.Y[base + r + (int64_t)c * a.ldy] = nan;
        }
        if (FB && threadIdx.x < AP_ROWS && o0 + (int)threadIdx.x < n)
            a.bout[base + o0 + threadIdx.x] = nan;
        return;
    }
    // row data for the entries of C this lane generates: row o = o0 + 16 wv + lane%16 (a row
    // past the end only feeds its own output row, never written)
    const int oc = min(o0 + wv * 16 + (lane & 15), n - 1);
    double ra = TRANS ? a.d[base + clamp_idx(a.origin[base + oc], n)] : a.d[base + oc];
    double rb = TRANS ? a.eta[base + oc] : 0.0;
    v4d acc[NCT];
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) acc[ct] = v4d{0.0, 0.0, 0.0, 0.0};
    // FB (one pass of at most 15 columns): b = sum (zhat_s / t)^2, each term squared
    // after the division as the b kernel does (zhat^2 and 1/t^2 apart can leave the
    // exponent range); each lane sums the terms of the entries it generates, on the
    // VALU beside the multiply (one column does not need the MFMA)
    double bsum = 0.0;
    ApplyStage<NCT> st;
    const int nch = (n + AP_K - 1) / AP_K, rounds = (nch + TEAMS - 1) / TEAMS;
    if (tm < nch) apply_fetch<TRANS, NCT>(a, base, n, tm * AP_K, c0, ncols, tid, st);
    asm volatile("" : "+v"(ra), "+v"(rb));  // loaded here, not inside the loop
    // one barrier per chunk: a buffer is stored again two chunks later, behind the barrier
    // that every wavefront reaches after its last read of it
    for (int rd = 0; rd < rounds; ++rd) {
        double *Xb = sh[tm].Xs[rd & 1];
        double2 *Sb = sh[tm].Sd[rd & 1];
        const int ci = rd * TEAMS + tm;
        const bool live = ci < nch;
        if (live) apply_store<TRANS, NCT>(n, ci * AP_K, ncols, tid, st, Xb, Sb);
        __syncthreads();
        // the next chunk's loads are in flight while this one is multiplied
        if (ci + TEAMS < nch)
            apply_fetch<TRANS, NCT>(a, base, n, (ci + TEAMS) * AP_K, c0, ncols, tid, st);
        if (!live) continue;
        // one step of 4 sources: this lane's Cauchy entry (one reciprocal with a Newton
        // step, FEW: with two) into the MFMA of every column tile; padding entries have weight
        // zero at the position of the problem's last source
#pragma unroll 4
        for (int kk = 0; kk < AP_K; kk += 4) {
            const int sl = kk + (lane >> 4);
            const double2 sd = Sb[sl];
            const double t = TRANS ? (sd.x - ra) - rb : (ra - sd.x) - sd.y;
            const double av = FEW ? rcp_nr(t) : rcp_nr1(t);
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct) {
                const double bv = Xb[(ct * 16 + (lane & 15)) * AP_LD + sl];
                acc[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc[ct], 0, 0, 0);
            }
            if (FB) {
                const double qv = av * sd.y;
                bsum = fma(qv, qv, bsum);
            }
        }
        mfma_drain();  // before any copy of the accumulators between chunks
    }
    if (FB) {  // the four lanes of a Cauchy row (lane % 16) hold its partial sums
        bsum += __shfl_xor(bsum, 16);
        bsum += __shfl_xor(bsum, 32);
    }
    if (a.work && threadIdx.x == 0) {  // kernel timing: this pass's algorithmic flops
        const unsigned long long rows = (unsigned long long)min(AP_ROWS, n - o0);
        const unsigned long long me = (unsigned long long)(ncols + (FB ? 1 : 0));
        atomicAdd(a.work, rows * (unsigned long long)n * (2 * me + 3) + 2 * rows * me);
    }
    mfma_drain();
    if (TEAMS > 1) {  // the teams' sums through their own buffers, added in team order
        static_assert(NCT == 1 || TEAMS == 1, "one column tile per team");
        double *mine = &sh[tm].Xs[0][0] + wv * 5 * WAVE;
        static_assert(4 * 5 * WAVE <= 2 * 16 * AP_LD, "a team's sums fit its buffers");
        __syncthreads();
        if (tm > 0) {
#pragma unroll
            for (int v = 0; v < 4; ++v) mine[v * WAVE + lane] = acc[0][v];
            if (FB) mine[4 * WAVE + lane] = bsum;
        }
        __syncthreads();
        if (tm > 0) return;
        for (int u = 1; u < TEAMS; ++u) {
            const double *o = &sh[u].Xs[0][0] + wv * 5 * WAVE;
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[0][v] += o[v * WAVE + lane];
            if (FB) bsum += o[4 * WAVE + lane];
        }
    }
    // v_mfma_f64_16x16x4f64 returns D[4 v + lane/16][lane % 16] in accumulator v
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int row = o0 + wv * 16 + 4 * v + (lane >> 4);
        double postb = 0.0;
        if (FB) {  // b's sum of this row is held by the lanes that generated its entries
            postb = 1.0 / sqrt(__shfl(bsum, 4 * v + (lane >> 4)));
            if (row < n && (lane & 15) == 0) a.bout[base + row] = postb;
        }
        if (row < n) {
            const double post = FB ? postb : (TRANS ? a.bnorm[base + row] : a.zhat[base + row]);
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct) {
                const int col = ct * 16 + (lane & 15);
                if (col < ncols)
                    a.Y[base + row + (int64_t)(c0 + col) * a.ldy] = post * acc[ct][v];
            }
        }
    }
}

template <int TRANS, int NCT, bool FB, int TEAMS, bool FEW>
__global__ __launch_bounds__(256 * TEAMS) void k_apply_mfma(ApplyArgs a) {
    __shared__ ApplyTeam<NCT> sh[TEAMS];
    const int np = (a.m + 16 * NCT - 1) / (16 * NCT);  // passes of a tile: neighbouring items
    const int item = xcd_item();
    apply_tile_mfma<TRANS, NCT, FB, TEAMS, FEW>(a, a.tiles[item / np], item % np * (16 * NCT), sh);
}

// ---------------------------------------------------------------------------------------
// VALU variant: one output row per lane, up to 8 right-hand sides per pass.  AV_W
// wavefronts share a tile: wavefront w takes the reduction chunks w, w + AV_W, ... (each
// stages its own chunk), and the partial sums are added in wavefront order at the end.
// ---------------------------------------------------------------------------------------
constexpr int AV_C = 8;
constexpr int AV_W = 4;

template <int TRANS>
__device__ void apply_tile_valu(const ApplyArgs &a, Tile t, double *Xs, double2 *Sd,
                                double *red) {
    const int p = t.prob;
    const int64_t base = a.off[p];
    const int n = (int)(a.off[p + 1] - base);
    const int lane = lane_id();
    const int wv = threadIdx.x / WAVE;
    const int o = t.row0 + lane;
    const bool ovalid = o < n;
    if (a.status[p] & ~SUPERDC_ST_NOCONV) {
        if (ovalid && wv == 0)
            for (int c = 0; c < a.m; ++c) a.Y[base + o + (int64_t)c * a.ldy] = __builtin_nan("");
        return;
    }
    const int oc = ovalid ? o : n - 1;
    double ra, rb = 0.0;
    if (TRANS == 0) {
        ra = a.d[base + oc];
    } else {
        ra = a.d[base + clamp_idx(a.origin[base + oc], n)];
        rb = a.eta[base + oc];
    }
    const double post = TRANS ? a.bnorm[base + oc] : a.zhat[base + oc];
    double *Xw = Xs + wv * WAVE * AV_C;
    double2 *Sw = Sd + wv * WAVE;
    const int nchunk = (n + WAVE - 1) / WAVE;
    const int rounds = (nchunk + AV_W - 1) / AV_W;  // the same count for every wavefront
    for (int c0 = 0; c0 < a.m; c0 += AV_C) {
        const int ncols = min(AV_C, a.m - c0);
        double acc[AV_C];
#pragma unroll
        for (int c = 0; c < AV_C; ++c) acc[c] = 0.0;
        for (int rd = 0; rd < rounds; ++rd) {
            const int s0 = (rd * AV_W + wv) * WAVE;
            __syncthreads();
            {
                double2 sd;
                double sc;
                const int s = s0 + lane;
                stage_entry<TRANS>(a, base, n, s, sd, sc);
                Sw[lane] = sd;
#pragma unroll
                for (int c = 0; c < AV_C; ++c)
                    Xw[lane * AV_C + c] =
                        (s < n && c < ncols) ? sc * a.X[base + s + (int64_t)(c0 + c) * a.ldx] : 0.0;
            }
            __syncthreads();
            const int cnt = max(0, min(WAVE, n - s0));
            for (int sl = 0; sl < cnt; ++sl) {
                const double2 sd = Sw[sl];
                const double tt = TRANS ? (sd.x - ra) - rb : (ra - sd.x) - sd.y;
                const double r = rcp_nr(tt);
#pragma unroll
                for (int c = 0; c < AV_C; ++c)
                    if (c < ncols) acc[c] = __builtin_fma(r, Xw[sl * AV_C + c], acc[c]);
            }
        }
        // partial sums of wavefronts 1.. through LDS, added in wavefront order by wavefront 0
        __syncthreads();
        if (wv > 0)
#pragma unroll
            for (int c = 0; c < AV_C; ++c) red[((wv - 1) * AV_C + c) * WAVE + lane] = acc[c];
        __syncthreads();
        if (wv == 0) {
            for (int w = 1; w < AV_W; ++w)
#pragma unroll
                for (int c = 0; c < AV_C; ++c) acc[c] += red[((w - 1) * AV_C + c) * WAVE + lane];
            if (ovalid)
                for (int c = 0; c < ncols; ++c)
                    a.Y[base + o + (int64_t)(c0 + c) * a.ldy] = post * acc[c];
        }
        if (a.work && threadIdx.x == 0) {  // kernel timing: this pass's algorithmic flops
            const unsigned long long rows = (unsigned long long)min(WAVE, n - t.row0);
            const unsigned long long me = (unsigned long long)ncols;
            atomicAdd(a.work, rows * (unsigned long long)n * (2 * me + 3) + 2 * rows * me);
        }
    }
}

template <int TRANS>
__global__ __launch_bounds__(WAVE * AV_W) void k_apply_valu(ApplyArgs a) {
    // the partial-sum exchange reuses the staging area (it follows a barrier that ends
    // every read of it)
    static_assert((AV_W - 1) * AV_C * WAVE <= AV_W * WAVE * AV_C, "reduction area");
    __shared__ double Xs[AV_W * WAVE * AV_C];
    __shared__ double2 Sd[AV_W * WAVE];
    double *red = Xs;
    apply_tile_valu<TRANS>(a, a.tiles[blockIdx.x], Xs, Sd, red);
}

hipError_t launch_apply(const ApplyArgs &a0, int use_mfma, int max_n, int num_cu, hipStream_t s) {
    if (a0.ntiles <= 0) return hipSuccess;
    ApplyArgs a = a0;
    a.work = trace_work(use_mfma ? KID_APPLY_MFMA : KID_APPLY_VALU);
    if (use_mfma) {
        // the pass width: 16, 32 or 64 columns, the smallest that covers m (64 beyond), and
        // narrower while the items (64 rows x a pass) are fewer than two per CU
        int nct = a.m <= 16 ? 1 : (a.m <= 32 ? 2 : 4);
        auto items = [&] { return a.ntiles * ((a.m + 16 * nct - 1) / (16 * nct)); };
        while (nct > 1 && items() < 2 * num_cu) nct /= 2;
        const dim3 g(items());
        const bool teams = nct == 1 && items() <= 2 * num_cu && max_n > 2 * AP_K;
#define SDC_APPLY_MFMA(T, C, FB, K)                                                         \
    SDC_LAUNCH(KID_APPLY_MFMA, (k_apply_mfma<T, C, FB, K, false>), g, dim3(256 * K), 0, s, a)
#define SDC_APPLY_FEW(T, K) \
    SDC_LAUNCH(KID_APPLY_MFMA, (k_apply_mfma<T, 1, false, K, true>), g, dim3(256 * K), 0, s, a)
        if (a.m < 4 && !a.fuse_b) {
            if (a.trans) {
                if (teams) SDC_APPLY_FEW(1, 4);
                else SDC_APPLY_FEW(1, 1);
            } else {
                if (teams) SDC_APPLY_FEW(0, 4);
                else SDC_APPLY_FEW(0, 1);
            }
            return hipGetLastError();
        }
        if (a.trans) {
            if (a.fuse_b && teams) SDC_APPLY_MFMA(1, 1, true, 4);
            else if (a.fuse_b) SDC_APPLY_MFMA(1, 1, true, 1);
            else if (teams) SDC_APPLY_MFMA(1, 1, false, 4);
            else if (nct == 1) SDC_APPLY_MFMA(1, 1, false, 1);
            else if (nct == 2) SDC_APPLY_MFMA(1, 2, false, 1);
            else SDC_APPLY_MFMA(1, 4, false, 1);
        } else {
            if (teams) SDC_APPLY_MFMA(0, 1, false, 4);
            else if (nct == 1) SDC_APPLY_MFMA(0, 1, false, 1);
            else if (nct == 2) SDC_APPLY_MFMA(0, 2, false, 1);
            else SDC_APPLY_MFMA(0, 4, false, 1);
        }
#undef SDC_APPLY_FEW
#undef SDC_APPLY_MFMA
    } else {
        const dim3 g(a.ntiles);
        if (a.trans)
            SDC_LAUNCH(KID_APPLY_VALU, k_apply_valu<1>, g, dim3(WAVE * AV_W), 0, s, a);
        else
            SDC_LAUNCH(KID_APPLY_VALU, k_apply_valu<0>, g, dim3(WAVE * AV_W), 0, s, a);
    }
    return hipGetLastError();
}

}  // namespace sdc
