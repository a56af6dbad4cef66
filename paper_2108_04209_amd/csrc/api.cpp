// api.cpp -- C ABI of the gfx950 conquering-stage library (declared in include/superdc.h).
//
// Host responsibilities only: argument checks, batch plans (work tiles ordered
// longest-problem-first for the batched launches), grow-only workspace, and the choice
// between one launch per phase and one launch per problem.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <new>
#include <numeric>
#include <vector>

#include "common.h"
#include "fmm.h"

using namespace sdc;

namespace {

thread_local int g_last_hip_error = 0;

int hip_fail(hipError_t e) {
    g_last_hip_error = (int)e;
    return e == hipErrorOutOfMemory ? SUPERDC_ENOMEM : SUPERDC_EHIP;
}

#define SDC_HIP(call)                                  \
    do {                                               \
        hipError_t e_ = (call);                        \
        if (e_ != hipSuccess) return hip_fail(e_);     \
    } while (0)

}  // namespace

namespace sdc {
int opts_check(const superdc_opts *o) {
    if (!(o->stop_c > 0.0) || o->max_iter < 1 || o->max_iter > 200) return SUPERDC_EINVAL;
    if (o->method < 0 || o->method > 2) return SUPERDC_EINVAL;
    if (o->fmm_order != FMM_P) return SUPERDC_EINVAL;
    if (o->fmm_leaf < 64 || o->fmm_leaf > 1024 || o->fmm_leaf % 64) return SUPERDC_EINVAL;
    if (o->persistent != 0 && o->persistent != 1) return SUPERDC_EINVAL;
    if (o->apply_kernel < 0 || o->apply_kernel > 2) return SUPERDC_EINVAL;
    if (o->fmm_crossover < 0) return SUPERDC_EINVAL;
    if (o->unshifted != 0 && o->unshifted != 1) return SUPERDC_EINVAL;
    if (o->interp != 0 && o->interp != 1) return SUPERDC_EINVAL;
    if (!std::isfinite(o->hss_tau) || o->hss_tau < 0.0) return SUPERDC_EINVAL;
    return SUPERDC_OK;
}

// Small batches by direct sums: the FMM's chain of set-up launches takes as long as
// DIRECT_PAIRS pole-root pairs (n = 1024 .. 4096, whole pipelines with 16 columns, direct
// against FMM: 1 problem of 1024 roots 75 and 175 us, 1 of 4096 205 and 275, 8 of 2048
// 168 and 218, 32 of 1024 164 and 223, 64 of 1024 270 and 268, 128 of 1024 493 and 391).  An
// apply alone crosses earlier, for its FMM has fewer launches and the direct product all
// columns' pairs (8 problems of 1024 roots, 64 columns: 39 and 41 us; 4 of 2048: 70 and 42).
constexpr double DIRECT_PAIRS = 4e7;
constexpr double DIRECT_APPLY_PAIRS = 9e6;
// The adjoint's direct sums take longer the longer the largest problem is (few tiles, each
// through all its poles), its FMM eleven launches more: direct against FMM, 16 problems of 1024
// roots 40 and 72 us, 4 of 2048 62 and 77, 1 of 4096 108 and 84, 64 of 1024 172 and 113, 1 of
// 8192 202 and 97, 128 of 1024 435 and 192.  The line lies where the FMM also gains on a
// program that issues the calls itself (30 us of launches more).  It lies there for every method,
// since the adjoint's results don't depend on the solver's: with larger leaves, which leave more
// to sum directly, in proportion (leaves of 256, direct against FMM: 1 problem of 4097 112 and
// 135 us, 20 of 1100 83 and 120; 1 of 600 roots and leaves of 64 56 and 75).
constexpr double DIRECT_BWD_PAIRS = 7e7;
constexpr int DIRECT_BWD_LEAVES = 64;  // 4096 roots in leaves of 64

int fmm_crossover_of(const superdc_batch *b, const superdc_opts &o, double pairs) {
    if (o.method == 1) return 0x7fffffff;
    if (o.method == 2) return 2 * o.fmm_leaf;
    if (o.fmm_crossover > 0) return o.fmm_crossover;
    const bool direct = b->max_n <= SECL_MAX_N &&
                        b->big_pairs <= (pairs > 0.0 ? pairs : DIRECT_PAIRS) &&
                        !o.unshifted && !o.interp && o.persistent;
    return direct ? 0x7fffffff : b->ctx->fmm_crossover;
}

namespace {
// whether the adjoint of the batch goes through the FMM where the options allow it
bool bwd_by_fmm(const superdc_batch *b, const superdc_opts &o) {
    if (b->max_n > DIRECT_BWD_LEAVES * o.fmm_leaf) return true;
    double pairs = 0.0;
    for (int p = 0; p < b->nprob; ++p) {
        const double n = (double)(b->off_h[p + 1] - b->off_h[p]);
        if (n >= DIRECT_BWD_LEAVES / 4 * o.fmm_leaf) pairs += n * n;
    }
    return pairs > DIRECT_BWD_PAIRS * o.fmm_leaf / 64;
}

int largest_below(const superdc_batch *b, const superdc_opts &o, int crossover) {
    if (b->max_n < crossover) return b->max_n;
    int64_t most = 0;
    for (int p = 0; p < b->nprob; ++p) {
        const int64_t n = b->off_h[p + 1] - b->off_h[p];
        if (n < crossover || n < 2 * o.fmm_leaf) most = std::max(most, n);
    }
    return (int)most;
}
}  // namespace

int largest_direct(const superdc_batch *b, const superdc_opts &o) {
    return largest_below(b, o, fmm_crossover_of(b, o));
}
int largest_direct_bwd(const superdc_batch *b, const superdc_opts &o) {
    return bwd_by_fmm(b, o) ? largest_below(b, o, fmm_crossover_of(b, o, 1.0)) : b->max_n;
}
bool solve_in_lds(int max_dir, const superdc_opts &o) {
    return max_dir <= SECL_MAX_N && !o.unshifted && !o.interp;
}
bool vectors_in_one(const superdc_batch *b, const superdc_opts &o) {
    return o.persistent && b->max_n <= VS_N && b->max_n < fmm_crossover_of(b, o);
}

int chunk_slot(int chunk) {
    for (int i = 0; i < kNumChunks; ++i)
        if (chunk == MIN_CHUNK << i) return i;
    return -1;
}

namespace {
// Host arrays gathered into one device allocation with one copy: a batch and its FMM layout
// hold some thirty small arrays, and a deflated pass makes new ones for its reduced
// problems (an allocation and a synchronous copy each: 2.6 ms of a pass over 1024
// problems, 0.6 ms now).
class Upload {
  public:
    template <typename T>
    void add(T **dst, const std::vector<T> &v) {
        const size_t at = (buf_.size() + 255) & ~(size_t)255;
        buf_.resize(at + std::max<size_t>(1, sizeof(T) * v.size()));
        fix_.push_back({(void **)dst, at});
        if (!v.empty()) std::memcpy(buf_.data() + at, v.data(), sizeof(T) * v.size());
    }
    // the device memory that holds them all (nullptr on failure; *err: why)
    void *commit(superdc_ctx *ctx, hipError_t *err) {
        void *mem = nullptr;
        *err = dev_alloc(ctx, &mem, buf_.size());
        if (*err != hipSuccess) return nullptr;
        *err = hipMemcpy(mem, buf_.data(), buf_.size(), hipMemcpyHostToDevice);
        if (*err != hipSuccess) {
            (void)hipFree(mem);
            return nullptr;
        }
        for (const auto &f : fix_) *f.first = (char *)mem + f.second;
        return mem;
    }

  private:
    std::vector<char> buf_;
    std::vector<std::pair<void **, size_t>> fix_;
};

// Arrays laid out one behind the other in a block that is not initialised
class Layout {
  public:
    template <typename T>
    void add(T **dst, size_t count) {
        fix_.push_back({(void **)dst, size_});
        size_ += (sizeof(T) * std::max<size_t>(1, count) + 255) & ~(size_t)255;
    }
    size_t size() const { return size_; }
    void place(void *mem) const {
        for (const auto &f : fix_) *f.first = (char *)mem + f.second;
    }

  private:
    size_t size_ = 0;
    std::vector<std::pair<void **, size_t>> fix_;
};

// the items of a cut length added to an upload
void list_add(superdc_batch *b, int chunk, Upload &up) {
    TileList &l = b->lists[chunk_slot(chunk)];
    if (l.count) return;
    std::vector<Tile> nat, lpt;
    l.begin.resize(b->nprob + 1);
    for (int p = 0; p < b->nprob; ++p) {
        l.begin[p] = (int32_t)nat.size();
        const int64_t n = b->off_h[p + 1] - b->off_h[p];
        for (int64_t r = 0; r < n; r += chunk) nat.push_back(Tile{p, (int32_t)r});
    }
    l.begin[b->nprob] = (int32_t)nat.size();
    lpt.reserve(nat.size());
    for (int p : b->order)
        for (int32_t t = l.begin[p]; t < l.begin[p + 1]; ++t) lpt.push_back(nat[t]);
    l.count = (int32_t)nat.size();
    up.add(&l.nat, nat);
    up.add(&l.lpt, lpt);
}
}  // namespace

const TileList *tile_list(superdc_batch *b, int chunk) {
    const int slot = chunk_slot(chunk);
    if (slot < 0) return nullptr;
    TileList &l = b->lists[slot];
    if (l.nat) return &l;
    Upload up;
    list_add(b, chunk, up);
    hipError_t e;
    void *mem = up.commit(b->ctx, &e);
    if (!mem) {
        l.count = 0;
        return nullptr;
    }
    b->mem.push_back(mem);
    return &l;
}
}  // namespace sdc

namespace {
// fewest poles each wavefront of a split sums: in the scalar-fetch solver, whose wavefronts all
// repeat the step, and in the Loewner, b and adjoint kernels, which only add up (16 against 128
// poles: 512 problems of 1 to 300 roots 37 -> 19 us for both, a conquer step of 1024 roots
// 14.6 -> 8.0 us, the adjoint of 16 small problems 25 -> 9 us)
constexpr int MIN_SPLIT_POLES = 128;
constexpr int MIN_VEC_POLES = 16;

// Launch shape for problems of the given sizes: the fewest wavefronts per work item
// (split S, a power of two <= 16) and the longest chunk (<= max_chunk) whose work items
// still give every CU 16 wavefronts, keeping >= min_poles summed entries per wavefront.
LaunchShape shape_for(const superdc_ctx *ctx, const int64_t *sizes, int count, int max_chunk,
                      int min_poles) {
    const long target = (long)ctx->num_cu * 16;
    int64_t nmax = 0;
    for (int i = 0; i < count; ++i) nmax = std::max(nmax, sizes[i]);
    for (int S = 1; S <= 16; S *= 2) {
        if (S > 1 && nmax / S < min_poles) break;
        for (int C = max_chunk; C >= TILE; C /= 2) {
            long wg = 0;
            for (int i = 0; i < count; ++i) wg += (sizes[i] + C - 1) / C;
            if (wg * S >= target) return LaunchShape{C, S};
        }
    }
    int S = 1;
    while (S < 16 && nmax / (2 * S) >= min_poles) S *= 2;
    return LaunchShape{TILE, S};
}

}  // namespace

namespace sdc {
LaunchShape plain_shape(const superdc_ctx *ctx, int64_t n) {
    return shape_for(ctx, &n, 1, TILE, MIN_SPLIT_POLES);
}
}  // namespace sdc

namespace {
LaunchShape choose_shape(const superdc_ctx *ctx, const superdc_batch *b, int max_chunk,
                         int min_poles) {
    std::vector<int64_t> sizes(b->nprob);
    for (int p = 0; p < b->nprob; ++p) sizes[p] = b->off_h[p + 1] - b->off_h[p];
    return shape_for(ctx, sizes.data(), b->nprob, max_chunk, min_poles);
}

// Roots per work item of the direct solver in LDS for the problems of fewer than `below` roots,
// from the lanes g that hold a root at first.  Measured over batches of 1 to 4096 problems and
// 64 to 4096 roots (g = 1 .. 64), a launch takes about the batch's work on all SIMDs,
// 4.8 passes a root of (52 n + 1100 g) / 64 cycles (its pairs, and the step that every lane of
// its team repeats; 10 % more at g = 1, where a wavefront waits for the slowest of 64 roots), and
// 0.6 of the longest root, 9 passes of 30 n / g + 4400 cycles.  The g of the smallest sum is
// taken: few large problems spread a root over many lanes (one of 1000 roots: 140 us at g = 1, 20
// at g = 64), many small ones keep it to two (512 of 128 roots: 34 us at g = 2, 183 at 64).
int lds_chunk(const superdc_batch *b, int64_t below) {
    double roots = 0.0, pairs = 0.0, nmax = 0.0;
    for (int p = 0; p < b->nprob; ++p) {
        const double n = (double)(b->off_h[p + 1] - b->off_h[p]);
        if (n >= (double)below) continue;
        roots += n;
        pairs += n * n;
        nmax = std::max(nmax, n);
    }
    const double simds = 4.0 * b->ctx->num_cu;
    int best = 1;
    double cost = 1e300;
    for (int g = 1; g <= WAVE; g *= 2) {
        const double t = 4.8 * (52.0 * pairs + 1100.0 * g * roots) / 64.0 / simds * (1.0 + 0.1 / g) +
                         0.6 * 9.0 * (30.0 * nmax / g + 4400.0);
        if (t < cost) {
            cost = t;
            best = g;
        }
    }
    return secl_waves((int)std::min(nmax, (double)SECL_MAX_N)) * WAVE / best;
}

// far-field separation: a box is far from a target leaf when the gap is >= FMM_SEP times
// the box's width (Chebyshev order 16 then interpolates both kernels to ~1e-14); a source
// enters a target leaf's local expansion when its gap to the target interval is >=
// FMM_SEP_LOC times the interval's width (order 20 then interpolates a source's 1/(s - x)
// to 5e-14 relative and its derivative, which only steers the step, to 2e-12; the stopping
// test's tolerance is n eps (1 + |psi| + |phi|) >= 1.1e-13 relative for the FMM's n >= 1024)
constexpr double FMM_SEP = 1.5;
constexpr double FMM_SEP_LOC = 0.75;
// The adjoint's sums run over 1/t, 1/t^2 and 1/t^3, which nodes at a distance of 1.5 widths
// interpolate to 9e-15, 2e-13 and worse (gradients of single eigenvalues, entry by entry: g_d off by
// 2.0e-13, by direct sums 1.3e-15); 3 widths leave less than the rounding of the terms (8 boxes of
// poles a target instead of 5: 1024 problems with their gradients 4.75 -> 5.1 ms).
constexpr double FMM_SEP_BWD = 3.0;

// synced: the current device has been waited for
void fmm_free(FmmPlan *fp, superdc_batch *b, bool synced) {
    if (!fp) return;
    if (fp->mem) (void)hipFree(fp->mem);
    if (fp->work) b->spare->give(fp->work, fp->work_cap, synced);
    for (void *p : fp->allocs) (void)hipFree(p);
    delete fp;
}

// direct chunks of length C of the problems that don't use the FMM, added to an upload
void dir_add(const superdc_batch *b, FmmPlan *fp, int C, Upload &up) {
    const int slot = chunk_slot(C);
    if (fp->dir_built[slot]) return;
    std::vector<Tile> v;
    for (int p : b->order) {
        if (fp->fmm_of_h[p] >= 0) continue;
        const int64_t n = b->off_h[p + 1] - b->off_h[p];
        for (int64_t r = 0; r < n; r += C) v.push_back(Tile{p, (int32_t)r});
    }
    fp->dir_count[slot] = (int32_t)v.size();
    fp->dir_built[slot] = true;
    up.add(&fp->dir_lpt[slot], v);
}

// the tiles and count of the direct chunks of length C (a length that the autotuner chose after
// the layout was made is added on its first use); false: out of memory
bool dir_list(const superdc_batch *b, FmmPlan *fp, int C, SolveArgs &a) {
    const int slot = chunk_slot(C);
    if (!fp->dir_built[slot]) {
        Upload up;
        dir_add(b, fp, C, up);
        hipError_t e;
        void *mem = up.commit(b->ctx, &e);
        if (!mem) {
            fp->dir_built[slot] = false;
            return false;
        }
        fp->allocs.push_back(mem);
    }
    a.tiles = fp->dir_lpt[slot];
    a.ntiles = fp->dir_count[slot];
    return true;
}

// Columns per set of launches: in small batches up to FMMV_MAX_PASS at once, so that the
// 16-column groups fill the chip together (one 8192-root problem has 128 items for 256 CUs: 64
// columns in four sets of launches took 264 us, in one 73 us; of one 65536-root problem, 560 and
// 317 us); 16 where the wider pass's equivalent weights (2 KiB a box and group) would exceed 64
// MiB -- such a batch has items enough for every CU.
int fmmv_max_pass(const FmmPlan *fp) {
    const int64_t groups = ((int64_t)64 << 20) / ((int64_t)std::max(1, fp->nboxes) * FMM_P * FMMV_MAX_M * 8);
    return FMMV_MAX_M * (int)std::min<int64_t>(FMMV_MAX_PASS / FMMV_MAX_M, std::max<int64_t>(1, groups));
}

// The per-call arrays of a layout: equivalent sources, lists, moments, and the equivalent weights
// of up to 16 columns.  They are the layout's own: a captured call holds their addresses, and
// stays valid while the batch does, whatever other batches of the context run afterwards.  Every
// call writes what it reads, but for the lists that a solve leaves to the Loewner and apply
// calls that follow it inside the library on the same batch, and for the use flags, which start
// below every number of a lists build.  False: out of memory (*err: why).
bool fmm_arrays(FmmPlan *fp, superdc_batch *b, hipError_t *err) {
    Layout up;
    const size_t nb = fp->nboxes, nl = fp->nleaves;
    up.add(&fp->eq, nb * FMM_P);
    up.add(&fp->vnode, nb * FMM_P);
    up.add(&fp->vcen, nb);
    up.add(&fp->lgeo, nb);
    up.add(&fp->lmom, nb * FMML_K);
    up.add(&fp->loc, nl * FMM_LOC);
    up.add(&fp->vw[0], nb * FMM_P * FMMV_MAX_M);
    up.add(&fp->vpart[0], (size_t)fp->nslot * FMM_P * FMMV_MAX_M);
    for (FmmLists *l : {&fp->own, &fp->roots}) {
        up.add(&l->near_lo, nl * FMM_NEAR_MAX);
        up.add(&l->near_hi, nl * FMM_NEAR_MAX);
        up.add(&l->near_lf, nl * FMM_NEAR_MAX);
        up.add(&l->far_l, nl * FMM_FAR_MAX);
        up.add(&l->far_r, nl * FMM_FAR_MAX);
        up.add(&l->far_ld, nl * FMM_FAR_MAX);
        up.add(&l->far_rd, nl * FMM_FAR_MAX);
        up.add(&l->cnt, nl * 3);
        up.add(&l->cntd, nl * 2);
        up.add(&l->loc_ab, nl);
    }
    fp->work = b->spare->take(up.size(), &fp->work_cap);
    if (!fp->work) {
        *err = dev_alloc(b->ctx, &fp->work, up.size());
        if (*err != hipSuccess) {
            fp->work = nullptr;
            return false;
        }
        fp->work_cap = up.size();
    }
    up.place(fp->work);
    return true;
}

// The FMM layout of a batch: which problems use it, their leaf trees and work lists.
// Rebuilt only when the leaf size or the crossover changes.
FmmPlan *fmm_plan(superdc_batch *b, int leaf, int crossover) {
    if (b->fmm && b->fmm->leaf == leaf && b->fmm->crossover == crossover) return b->fmm;
    fmm_free(b->fmm, b, hipDeviceSynchronize() == hipSuccess);
    b->fmm = nullptr;
    FmmPlan *fp = new (std::nothrow) FmmPlan();
    if (!fp) return nullptr;
    fp->leaf = leaf;
    fp->crossover = crossover;
    fp->fmm_of_h.assign(b->nprob, -1);
    std::vector<int32_t> height, box_fmm, leaf_fmm;
    fp->box_off_h.push_back(0);
    fp->leaf_off_h.push_back(0);
    for (int p = 0; p < b->nprob; ++p) {
        const int64_t n = b->off_h[p + 1] - b->off_h[p];
        if (n < crossover || n < 2 * leaf) {
            fp->max_dir = std::max(fp->max_dir, (int)n);
            continue;
        }
        const int q = fp->nfmm++;
        fp->fmm_prob_h.push_back(p);
        fp->fmm_of_h[p] = q;
        const int nl = (int)((n + leaf - 1) / leaf);
        int H = 0;
        while ((1 << H) < nl) ++H;
        height.push_back(H);
        const int nb = (2 << H) - 1;
        fp->box_off_h.push_back(fp->box_off_h.back() + nb);
        fp->leaf_off_h.push_back(fp->leaf_off_h.back() + nl);
        box_fmm.insert(box_fmm.end(), nb, q);
        leaf_fmm.insert(leaf_fmm.end(), nl, q);
    }
    fp->lds_chunk = lds_chunk(b, (int64_t)fp->max_dir + 1);
    fp->nboxes = fp->box_off_h.back();
    fp->nleaves = fp->leaf_off_h.back();
    // the boxes the source kernels visit, so that their grids hold no workgroup without a
    // box: every leaf (all hold poles), and every upper box with poles, largest first
    std::vector<int32_t> leaf_box, upper_box;
    std::vector<int4> upper_item;
    std::vector<int2> split_box;
    int nslot = 0;
    {
        std::vector<std::pair<int, int32_t>> up;  // (leaves below, global box id)
        for (int q = 0; q < fp->nfmm; ++q) {
            const int H = height[q];
            const int nl = fp->leaf_off_h[q + 1] - fp->leaf_off_h[q];
            const int32_t b0 = fp->box_off_h[q];
            for (int l = 0; l < nl; ++l) leaf_box.push_back(b0 + (1 << H) - 1 + l);
            for (int h = 0; h < H; ++h)
                for (int i = 0; i < (1 << h); ++i) {
                    const int first = i << (H - h);
                    if (first < nl)
                        up.emplace_back(std::min(1 << (H - h), nl - first), b0 + (1 << h) - 1 + i);
                }
        }
        std::stable_sort(up.begin(), up.end(),
                         [](const std::pair<int, int32_t> &x, const std::pair<int, int32_t> &y) {
                             return x.first > y.first;
                         });
        for (const auto &e : up) {
            upper_box.push_back(e.second);
            for (int c = 0; c < 6; ++c) fp->upper_cls[c] += e.first > (64 >> c);
        }
        fp->upper_cls[6] = (int)up.size();
        for (const auto &e : up) {
            const int parts = (e.first * FMM_P + FMMV_PART_PTS - 1) / FMMV_PART_PTS;
            if (parts == 1) {
                if (e.first > 4) fp->nitem_big = (int)upper_item.size() + 1;
                upper_item.push_back(make_int4(e.second, 0, 1, -1));
                continue;
            }
            split_box.push_back(make_int2(e.second, nslot));
            for (int u = 0; u < parts; ++u)
                upper_item.push_back(make_int4(e.second, u, parts, nslot + u));
            nslot += parts;
            fp->nitem_big = (int)upper_item.size();
        }
    }
    fp->nupper = (int)upper_box.size();
    fp->nupper_item = (int)upper_item.size();
    fp->nsplit = (int)split_box.size();
    fp->nslot = nslot;
    // work items (64-root pieces of the target leaves) in problem order and longest-first
    std::vector<Tile> lnat, llpt;
    fp->item_off_h.push_back(0);
    for (int q = 0; q < fp->nfmm; ++q) {
        const int p = fp->fmm_prob_h[q];
        const int64_t n = b->off_h[p + 1] - b->off_h[p];
        for (int64_t r = 0; r < n; r += fp->sub) lnat.push_back(Tile{p, (int32_t)r});
        fp->item_off_h.push_back((int32_t)lnat.size());
    }
    fp->nitems = (int)lnat.size();
    for (int p : b->order) {
        const int q = fp->fmm_of_h[p];
        if (q < 0) continue;
        for (int t = fp->item_off_h[q]; t < fp->item_off_h[q + 1]; ++t) llpt.push_back(lnat[t]);
    }
    // wavefronts per item: enough to give the launch ~16 wavefronts per CU
    fp->split = 1;
    while (fp->split < 8 && (long)fp->nitems * fp->split * 2 <= (long)b->ctx->num_cu * 16)
        fp->split *= 2;
    // the solver's items (pieces of ssub roots that never cross a leaf)
    std::vector<Tile> snat, slpt;
    fp->sitem_off_h.push_back(0);
    for (int q = 0; q < fp->nfmm; ++q) {
        const int p = fp->fmm_prob_h[q];
        const int64_t n = b->off_h[p + 1] - b->off_h[p];
        for (int64_t r = 0; r < n; r += fp->ssub) snat.push_back(Tile{p, (int32_t)r});
        fp->sitem_off_h.push_back((int32_t)snat.size());
    }
    fp->snitems = (int)snat.size();
    for (int p : b->order) {
        const int q = fp->fmm_of_h[p];
        if (q < 0) continue;
        for (int t = fp->sitem_off_h[q]; t < fp->sitem_off_h[q + 1]; ++t) slpt.push_back(snat[t]);
    }
    // wavefronts per item of the solver: fewer repeat less of a root's step and window, more
    // fill the chip (batches of 4096 to 65536 roots a problem, us a solve with 1, 2, 4, 8:
    // 128 items 104 77 66 64, 1024 items 134 117 110 127, 4096 items 289 248 256 329, 32768
    // items 1556 1583 1745 2328); a larger leaf takes more, for the LDS it is staged in
    const long cu = b->ctx->num_cu;
    fp->ssplit = fp->snitems <= cu        ? 8
                 : fp->snitems <= 12 * cu ? 4
                 : fp->snitems <= 64 * cu ? 2
                                          : 1;
    while (fp->ssplit < 8 && fp->ssplit * 64 < leaf) fp->ssplit *= 2;
    Upload up;
    up.add(&fp->fmm_prob, fp->fmm_prob_h);
    up.add(&fp->fmm_of, fp->fmm_of_h);
    up.add(&fp->box_off, fp->box_off_h);
    up.add(&fp->leaf_off, fp->leaf_off_h);
    up.add(&fp->height, height);
    up.add(&fp->box_fmm, box_fmm);
    up.add(&fp->leaf_fmm, leaf_fmm);
    up.add(&fp->leaf_box, leaf_box);
    up.add(&fp->upper_box, upper_box);
    up.add(&fp->upper_item, upper_item);
    up.add(&fp->split_box, split_box);
    up.add(&fp->leaf_nat, lnat);
    up.add(&fp->leaf_lpt, llpt);
    up.add(&fp->sitem_nat, snat);
    up.add(&fp->sitem_lpt, slpt);
    // direct chunks of the other problems: the cut lengths in use now
    for (int C : {(int)TILE, fp->lds_chunk, b->sec.chunk}) dir_add(b, fp, C, up);
    for (FmmLists *l : {&fp->own, &fp->roots}) up.add(&l->used, std::vector<int32_t>(fp->nboxes, 0));
    hipError_t e;
    if (!(fp->mem = up.commit(b->ctx, &e)) || !fmm_arrays(fp, b, &e)) {
        fmm_free(fp, b, true);
        return nullptr;
    }
    b->fmm = fp;
    return fp;
}

void set_lists(FmmArgs &f, const FmmLists &l) {
    f.near_lo = l.near_lo;
    f.near_hi = l.near_hi;
    f.near_lf = l.near_lf;
    f.far_l = l.far_l;
    f.far_r = l.far_r;
    f.cnt = l.cnt;
    f.far_ld = l.far_ld;
    f.far_rd = l.far_rd;
    f.cntd = l.cntd;
    f.loc_ab = l.loc_ab;
    f.used = l.used;
    f.gen = l.gen;
}

FmmArgs fmm_args(const FmmPlan *fp, const superdc_batch *b, const SolveArgs &a) {
    FmmArgs f{};
    f.off = b->off_d;
    f.leaf = fp->leaf;
    f.sep = FMM_SEP;
    f.sep_loc = FMM_SEP_LOC;
    f.fmm_prob = fp->fmm_prob;
    f.fmm_of = fp->fmm_of;
    f.box_off = fp->box_off;
    f.leaf_off = fp->leaf_off;
    f.height = fp->height;
    f.dw = a.dw;
    f.tail = a.z2;  // the last root lies below d_{n-1} + sum_j w_j
    f.status = a.status;
    set_lists(f, fp->own);
    f.eq = fp->eq;
    f.loc = fp->loc;
    f.nboxes = fp->nboxes;
    f.nleaves = fp->nleaves;
    f.box_fmm = fp->box_fmm;
    f.leaf_fmm = fp->leaf_fmm;
    f.leaf_box = fp->leaf_box;
    f.upper_box = fp->upper_box;
    f.nupper = fp->nupper;
    f.upper_item = fp->upper_item;
    f.nupper_item = fp->nupper_item;
    f.nitem_big = fp->nitem_big;
    std::copy(fp->upper_cls, fp->upper_cls + 7, f.upper_cls);
    f.split_box = fp->split_box;
    f.nsplit = fp->nsplit;
    return f;
}
// The eigenvector-side FMM of one call: the list geometry comes from this call's poles and
// its last roots.
FmmArgs fmm_vec_args(const FmmPlan *fp, const superdc_batch *b, const double *d,
                     const double *eta, const int32_t *origin, const int32_t *status) {
    SolveArgs a{};
    a.status = const_cast<int32_t *>(status);
    FmmArgs f = fmm_args(fp, b, a);
    f.pos = d;
    f.tail = nullptr;
    f.teta = eta;
    f.torg = origin;
    return f;
}

// The FMM of the sums over the roots (Y = Qhat X): its own lists and use flags, the
// sources' positions in `pos` (the roots), the targets at the poles d.
FmmArgs fmm_roots_args(const FmmPlan *fp, const superdc_batch *b, const double *pos,
                       const int32_t *status, const double *d) {
    FmmArgs f = fmm_vec_args(fp, b, pos, nullptr, nullptr, status);
    f.tpos = d;
    set_lists(f, fp->roots);
    return f;
}

// the FMM plan that applies to this call, or nullptr (rc = ENOMEM on allocation failure)
FmmPlan *fmm_for(superdc_batch *b, const superdc_opts &o, int &rc, double pairs = 0.0) {
    rc = SUPERDC_OK;
    const int crossover = fmm_crossover_of(b, o, pairs);
    if (b->max_n < crossover) return nullptr;
    FmmPlan *fp = fmm_plan(b, o.fmm_leaf, crossover);
    if (!fp) {
        rc = SUPERDC_ENOMEM;
        return nullptr;
    }
    return fp->nfmm > 0 ? fp : nullptr;
}

// the arrays for the equivalent weights of a pass of `cols` columns: those of wide passes are
// allocated, for the widest, by the batch's first such call; false: out of memory
bool fmmv_space(superdc_ctx *ctx, FmmPlan *fp, int cols, FmmArgs &f, FmmVec &v) {
    const int wide = cols > FMMV_MAX_M;
    if (wide && !fp->vw[1]) {
        const int most = fmmv_max_pass(fp);
        Layout w;
        w.add(&fp->vw[1], (size_t)fp->nboxes * FMM_P * most);
        w.add(&fp->vpart[1], (size_t)fp->nslot * FMM_P * most);
        void *mem = nullptr;
        if (dev_alloc(ctx, &mem, w.size()) != hipSuccess) {
            fp->vw[1] = fp->vpart[1] = nullptr;
            return false;
        }
        fp->allocs.push_back(mem);
        w.place(mem);
    }
    v.vnode = fp->vnode;
    v.vw = fp->vw[wide];
    f.vpart = fp->vpart[wide];
    return true;
}

// Run the eigenvector-side FMM over every FMM problem of the batch for the v.m columns of
// v.X: build the lists (first pass only), compress the used boxes, evaluate at the targets
// (one launch, or one launch per problem).
hipError_t fmmv_run(superdc_ctx *ctx, const superdc_batch *b, const FmmPlan *fp,
                    const FmmArgs &f, const FmmVec &v, bool lists, bool persistent,
                    hipStream_t s) {
    hipError_t e = lists ? launch_fmm_lists(f, s) : hipSuccess;
    if (e == hipSuccess) e = launch_fmmv_sources(f, v, s);
    if (e != hipSuccess) return e;
    SolveArgs it{};
    it.off = b->off_d;
    if (persistent) {
        it.tiles = fp->leaf_lpt;
        it.ntiles = fp->nitems;
        return launch_fmmv_eval(it, f, v, fp->split, ctx->num_cu, s);
    }
    for (int q = 0; q < fp->nfmm && e == hipSuccess; ++q) {
        it.tiles = fp->leaf_nat + fp->item_off_h[q];
        it.ntiles = fp->item_off_h[q + 1] - fp->item_off_h[q];
        e = launch_fmmv_eval(it, f, v, fp->split, ctx->num_cu, s);
    }
    return e;
}
}  // namespace

namespace sdc {
hipError_t dev_alloc(superdc_ctx *ctx, void **p, size_t bytes) {
    const hipError_t e = hipMalloc(p, bytes > ctx->alloc_limit ? (size_t)1 << 60 : bytes);
    if (e != hipSuccess) (void)hipGetLastError();
    return e;
}

void *SpareBlock::take(size_t bytes, size_t *cap) {
    std::lock_guard<std::mutex> g(mu_);
    int dev = -1;
    if (!p_ || cap_ < bytes || hipGetDevice(&dev) != hipSuccess || dev != device_) return nullptr;
    void *p = p_;
    *cap = cap_;
    p_ = nullptr;
    cap_ = 0;
    return p;
}

void SpareBlock::give(void *p, size_t cap, bool synced) {
    {
        std::lock_guard<std::mutex> g(mu_);
        int dev = -1;
        if (synced && !closed_ && cap <= SPARE_MAX && cap > cap_ && hipGetDevice(&dev) == hipSuccess &&
            dev == device_) {
            std::swap(p, p_);
            cap_ = cap;
        }
    }
    if (p) (void)hipFree(p);
}

void SpareBlock::close() {
    std::lock_guard<std::mutex> g(mu_);
    if (p_) (void)hipFree(p_);
    p_ = nullptr;
    cap_ = 0;
    closed_ = true;
}

void *ws_get(superdc_ctx *ctx, int slot, size_t bytes) {
    if (bytes == 0) bytes = 256;
    if (ctx->ws_cap[slot] >= bytes) return ctx->ws[slot];
    if (ctx->ws[slot]) {
        if (hipDeviceSynchronize() != hipSuccess) return nullptr;
        (void)hipFree(ctx->ws[slot]);
        ctx->ws[slot] = nullptr;
        ctx->ws_cap[slot] = 0;
    }
    size_t cap = std::max(bytes, ctx->ws_cap[slot] + ctx->ws_cap[slot] / 2);
    void *p = nullptr;
    if (dev_alloc(ctx, &p, cap) != hipSuccess) return nullptr;
    ctx->ws[slot] = p;
    ctx->ws_cap[slot] = cap;
    return p;
}
}  // namespace sdc

#define SDC_OPTS(o, opts)                       \
    superdc_opts o;                             \
    if (opts) o = *(opts);                      \
    else superdc_opts_default(&o);              \
    {                                           \
        int rc_ = opts_check(&o);               \
        if (rc_) return rc_;                    \
    }

namespace sdc {
// Loewner/b and the Cauchy apply.  reuse_lists: right before, a solve of the same problems
// left their FMM interaction lists and (d_K, eta) pairs in the workspace (internal callers only).
int loewner_run(superdc_ctx *ctx, const superdc_batch *b, const double *d, const double *z,
                const double *rho, const double *eta, const int32_t *origin,
                const int32_t *status, double *zhat, double *bnorm, const superdc_opts *opts,
                void *stream, bool reuse_lists, bool fmm_b) {
    if (!ctx || !b || b->ctx != ctx || !d || !z || !rho || !eta || !origin || !status || !zhat ||
        !bnorm)
        return SUPERDC_EINVAL;
    SDC_OPTS(o, opts);
    hipStream_t s = (hipStream_t)stream;
    VecArgs a{};
    a.off = b->off_d;
    a.d = d;
    a.z = z;
    a.rho = rho;
    a.eta = eta;
    a.origin = origin;
    a.status = status;
    a.ke = (double2 *)ws_get(ctx, WS_KE, sizeof(double2) * b->total);
    a.dz = (double2 *)ws_get(ctx, WS_DZ, sizeof(double2) * b->total);
    if (!a.ke || !a.dz) return SUPERDC_ENOMEM;
    a.zhat = zhat;
    a.bnorm = bnorm;
    superdc_batch *bm = const_cast<superdc_batch *>(b);
    if (fmm_b && vectors_in_one(b, o)) {
        SDC_HIP(launch_vectors_small(a, b->nprob, b->max_n, s));
        return SUPERDC_OK;
    }
    const TileList *L = tile_list(bm, TILE);
    if (!L) return SUPERDC_ENOMEM;
    // large problems: zhat and b through the FMM (far boxes by moment expansions of the
    // Loewner log-sums and by equivalent sources for b), the others by direct products/sums
    int rc;
    FmmPlan *fp = fmm_for(bm, o, rc);
    if (rc) return rc;
    FmmvPackArgs pk{};
    FmmVec v{};
    v.trans = 1;
    FmmArgs f{};
    FmmlArgs lf{};
    if (fp) {
        double2 *pairs = (double2 *)ws_get(ctx, WS_VPAIR, sizeof(double2) * b->total);
        if (!pairs) return SUPERDC_ENOMEM;
        pk.off = b->off_d;
        pk.tiles = fp->leaf_nat;
        pk.ntiles = fp->nitems;
        pk.d = d;
        pk.eta = eta;
        pk.origin = origin;
        pk.pairs = pairs;
        // every problem uses the FMM: the Loewner packing writes ke as well
        pk.ke = fp->nfmm == b->nprob ? a.ke : nullptr;
        v.m = 1;
        v.kern = 2;
        v.scale = zhat;
        v.d = d;
        v.origin = origin;
        v.eta = eta;
        v.bout = bnorm;
        v.zh = zhat;
        f = fmm_vec_args(fp, b, d, eta, origin, status);
        if (fmm_b && !fmmv_space(ctx, fp, 1, f, v)) return SUPERDC_ENOMEM;
        lf.pd = pairs;
        lf.geo = fp->lgeo;
        lf.mom = fp->lmom;
        // (d_j, delta_j) pairs, the lists of these poles (unless the solve left them), the
        // Loewner moments of every leaf and used box; with the lists left by the solve the
        // leaves' launch packs the pairs itself
        if (!reuse_lists) {
            SDC_HIP(launch_fmml_pack(pk, s));
            f.gen = ++fp->own.gen;
            SDC_HIP(launch_fmm_lists(f, s));
        } else {
            lf.pack = 1;
            lf.d = d;
            lf.eta = eta;
            lf.origin = origin;
        }
        SDC_HIP(launch_fmml_moments(f, lf, s));
    }
    a.tiles = L->lpt;
    a.ntiles = L->count;
    // a solve right before (reuse_lists) left ke as well
    if (!pk.ke && !reuse_lists) SDC_HIP(launch_pack_ke(a, s));
    if (o.persistent) {
        const int S = b->vec.split;
        if (fp) {
            a.tiles = fp->dir_lpt[chunk_slot(TILE)];
            a.ntiles = fp->dir_count[chunk_slot(TILE)];
        }
        SDC_HIP(launch_loewner(a, S, s));
        if (fp) {
            VecArgs af = a;
            af.tiles = fp->leaf_lpt;
            af.ntiles = fp->nitems;
            SDC_HIP(launch_loewner_fmm(af, f, lf, fp->split, s));
        }
        if (fmm_b)
            SDC_HIP(launch_bnorm(a, S, s));
        if (fp && fmm_b) SDC_HIP(fmmv_run(ctx, b, fp, f, v, false, true, s));
    } else {
        for (int p = 0; p < b->nprob; ++p) {
            const int64_t np = b->off_h[p + 1] - b->off_h[p];
            const int S = shape_for(ctx, &np, 1, TILE, MIN_VEC_POLES).split;
            if (fp && fp->fmm_of_h[p] >= 0) {
                const int q = fp->fmm_of_h[p];
                VecArgs af = a;
                af.tiles = fp->leaf_nat + fp->item_off_h[q];
                af.ntiles = fp->item_off_h[q + 1] - fp->item_off_h[q];
                SDC_HIP(launch_loewner_fmm(af, f, lf, fp->split, s));
                continue;
            }
            a.tiles = L->nat + L->begin[p];
            a.ntiles = L->begin[p + 1] - L->begin[p];
            SDC_HIP(launch_loewner(a, S, s));
            if (fmm_b) SDC_HIP(launch_bnorm(a, S, s));
        }
        if (fp && fmm_b) SDC_HIP(fmmv_run(ctx, b, fp, f, v, false, false, s));
    }
    return SUPERDC_OK;
}

int apply_run(superdc_ctx *ctx, const superdc_batch *b, const double *d, const double *zhat,
              const double *bnorm, const double *eta, const int32_t *origin,
              const int32_t *status, int trans, int32_t m, const double *X, int64_t ldx,
              double *Y, int64_t ldy, const superdc_opts *opts, void *stream, bool reuse_lists,
              bool fuse_b) {
    if (!ctx || !b || b->ctx != ctx || !d || !zhat || !bnorm || !eta || !origin || !status ||
        !X || !Y)
        return SUPERDC_EINVAL;
    if (fuse_b && (trans != 1 || m + 1 > FMMV_MAX_M)) return SUPERDC_EINVAL;
    if ((trans != 0 && trans != 1) || m < 1 || ldx < b->total || ldy < b->total)
        return SUPERDC_EINVAL;
    SDC_OPTS(o, opts);
    // X and Y must not overlap
    const char *x0 = (const char *)X, *x1 = (const char *)(X + (ldx * (m - 1) + b->total));
    const char *y0 = (const char *)Y, *y1 = (const char *)(Y + (ldy * (m - 1) + b->total));
    if (x0 < y1 && y0 < x1) return SUPERDC_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    ApplyArgs a{};
    a.off = b->off_d;
    a.d = d;
    a.zhat = zhat;
    a.bnorm = bnorm;
    a.eta = eta;
    a.origin = origin;
    a.status = status;
    a.trans = trans;
    a.m = m;
    a.X = X;
    a.ldx = ldx;
    a.Y = Y;
    a.ldy = ldy;
    a.fuse_b = fuse_b ? 1 : 0;
    a.bout = const_cast<double *>(bnorm);  // written only with fuse_b
    superdc_batch *bm = const_cast<superdc_batch *>(b);
    const TileList *L = tile_list(bm, TILE);
    if (!L) return SUPERDC_ENOMEM;
    // few columns: the VALU kernel does less work, but in launches of less than two tiles a CU a
    // wavefront's chain of sources bounds it, and the MFMA kernel's teams are the faster up to the
    // line whatever the sizes (VALU against MFMA, one column, us a call: one problem of 100
    // roots 11.7 and 9.2, 511 of 64 12.4 and 9.4, 100 of 300 20.7 and 13.7, 31 of 1000 45 and 32,
    // 7 of 4096 168 and 109)
    const int use_mfma = fuse_b || o.apply_kernel == 2 ||
                         (o.apply_kernel == 0 && (m >= 4 || L->count < 2 * ctx->num_cu));
    // Y = Qhat^T X of the large problems by the eigenvector-side FMM (the sums run over the
    // poles for every root, the layout of the solver's lists), Y = Qhat X by the FMM of the
    // sums over the roots (sources at the roots, targets at the poles, lists of their own);
    // the other problems by the direct kernels
    int rc;
    FmmPlan *fp = fmm_for(bm, o, rc, DIRECT_APPLY_PAIRS);
    if (rc) return rc;
    // the solve left lists only if it used the FMM as well
    if (fmm_crossover_of(b, o) == 0x7fffffff) reuse_lists = false;
    if (o.persistent) {
        a.tiles = fp ? fp->dir_lpt[chunk_slot(TILE)] : L->lpt;
        a.ntiles = fp ? fp->dir_count[chunk_slot(TILE)] : L->count;
        SDC_HIP(launch_apply(a, use_mfma, fp ? fp->max_dir : b->max_n, ctx->num_cu, s));
    } else {
        for (int p = 0; p < b->nprob; ++p) {
            if (fp && fp->fmm_of_h[p] >= 0) continue;
            a.tiles = L->nat + L->begin[p];
            a.ntiles = L->begin[p + 1] - L->begin[p];
            const int np = (int)(b->off_h[p + 1] - b->off_h[p]);
            SDC_HIP(launch_apply(a, use_mfma, np, ctx->num_cu, s));
        }
    }
    if (!fp) return SUPERDC_OK;
    FmmVec v{};
    v.trans = trans;
    v.kern = 1;
    v.ldx = ldx;
    v.scale = trans ? zhat : bnorm;
    v.d = d;
    v.origin = origin;
    v.eta = eta;
    v.post = trans ? bnorm : zhat;
    v.ldy = ldy;
    v.fuse_b = fuse_b ? 1 : 0;
    v.zh = zhat;
    v.bout = const_cast<double *>(bnorm);  // written only with fuse_b
    bool lists = !reuse_lists;
    FmmArgs f{};
    if (trans == 0) {
        double *pos = (double *)ws_get(ctx, WS_VPAIR, sizeof(double2) * b->total);
        double2 *ke = (double2 *)ws_get(ctx, WS_KE, sizeof(double2) * b->total);
        if (!pos || !ke) return SUPERDC_ENOMEM;
        FmmvPackArgs pk{};
        pk.off = b->off_d;
        pk.tiles = fp->leaf_nat;
        pk.ntiles = fp->nitems;
        pk.d = d;
        pk.eta = eta;
        pk.origin = origin;
        pk.pos = pos;
        pk.ke = ke;
        v.ke = ke;
        SDC_HIP(launch_fmmv_pos(pk, s));
        f = fmm_roots_args(fp, b, pos, status, d);
        f.gen = ++fp->roots.gen;  // built with the first columns below
        lists = true;
    } else {
        f = fmm_vec_args(fp, b, d, eta, origin, status);
        if (lists) f.gen = ++fp->own.gen;  // built with the first columns below
    }
    const int pass = std::min(m + v.fuse_b, fmmv_max_pass(fp));  // one pass when fused
    if (!fmmv_space(ctx, fp, pass, f, v)) return SUPERDC_ENOMEM;
    for (int c0 = 0; c0 < m; c0 += pass) {
        v.m = std::min(pass, m + v.fuse_b - c0);
        v.X = X + (int64_t)c0 * ldx;
        v.Y = Y + (int64_t)c0 * ldy;
        SDC_HIP(fmmv_run(ctx, b, fp, f, v, lists, o.persistent != 0, s));
        lists = false;
    }
    return SUPERDC_OK;
}

}  // namespace sdc

extern "C" {

void superdc_opts_default(superdc_opts *o) {
    if (!o) return;
    std::memset(o, 0, sizeof(*o));
    o->stop_c = 1.0;
    o->max_iter = 40;
    o->method = 0;
    o->fmm_order = 16;
    o->fmm_leaf = 64;
    o->persistent = 1;
    o->apply_kernel = 0;
}

// for tests (not in the header): device allocations of more than `bytes` fail on this context
void superdc_test_alloc_limit(superdc_ctx *ctx, size_t bytes) { ctx->alloc_limit = bytes; }

const char *superdc_strerror(int code) {
    switch (code) {
        case SUPERDC_OK: return "success";
        case SUPERDC_EINVAL: return "invalid argument";
        case SUPERDC_ENOMEM: return "device allocation failed";
        case SUPERDC_EHIP: return "HIP runtime error";
        case SUPERDC_ENODEV: return "no gfx950 device";
        default: return "unknown error";
    }
}

int superdc_last_hip_error(void) { return g_last_hip_error; }

int superdc_create(superdc_ctx **out) {
    if (!out) return SUPERDC_EINVAL;
    *out = nullptr;
    int dev = 0, count = 0;
    if (hipGetDeviceCount(&count) != hipSuccess || count < 1) return SUPERDC_ENODEV;
    SDC_HIP(hipGetDevice(&dev));
    hipDeviceProp_t prop;
    SDC_HIP(hipGetDeviceProperties(&prop, dev));
    if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0) return SUPERDC_ENODEV;
    superdc_ctx *ctx = new (std::nothrow) superdc_ctx();
    if (!ctx) return SUPERDC_ENOMEM;
    ctx->device = dev;
    ctx->num_cu = prop.multiProcessorCount;
    try {
        ctx->spare = std::make_shared<SpareBlock>(dev);
    } catch (const std::bad_alloc &) {
        delete ctx;
        return SUPERDC_ENOMEM;
    }
    {
        const int rc = noalloc_init(dev);
        if (rc != SUPERDC_OK) {
            delete ctx;
            return rc;
        }
    }
    *out = ctx;
    return SUPERDC_OK;
}

void superdc_destroy(superdc_ctx *ctx) {
    if (!ctx) return;
    (void)hipDeviceSynchronize();
    for (int i = 0; i < kNumWs; ++i)
        if (ctx->ws[i]) (void)hipFree(ctx->ws[i]);
    ctx->spare->close();
    delete ctx;
}

int superdc_batch_create(superdc_ctx *ctx, int32_t nprob, const int64_t *off_host,
                         superdc_batch **out) {
    if (!ctx || !off_host || !out || nprob < 1) return SUPERDC_EINVAL;
    *out = nullptr;
    if (off_host[0] != 0) return SUPERDC_EINVAL;
    int32_t max_n = 0;
    for (int p = 0; p < nprob; ++p) {
        const int64_t n = off_host[p + 1] - off_host[p];
        if (n < 1 || n > (int64_t)1 << 30) return SUPERDC_EINVAL;
        max_n = std::max<int32_t>(max_n, (int32_t)n);
    }
    superdc_batch *b = new (std::nothrow) superdc_batch();
    if (!b) return SUPERDC_ENOMEM;
    b->ctx = ctx;
    b->spare = ctx->spare;
    b->nprob = nprob;
    b->total = off_host[nprob];
    b->max_n = max_n;
    for (int p = 0; p < nprob; ++p) {
        const double n = (double)(off_host[p + 1] - off_host[p]);
        if (n >= ctx->fmm_crossover) b->big_pairs += n * n;
    }
    b->off_h.assign(off_host, off_host + nprob + 1);
    b->order.resize(nprob);
    std::iota(b->order.begin(), b->order.end(), 0);
    std::stable_sort(b->order.begin(), b->order.end(), [&](int x, int y) {
        return off_host[x + 1] - off_host[x] > off_host[y + 1] - off_host[y];
    });
    // problems of 16384 entries and more are validated in slices of about 4096
    b->vsplit = max_n >= 16384 ? std::min(16, max_n / 4096) : 1;
    // launch shapes for the batched launches (the autotuner may replace them); the solver's
    // tile lists for them are built now, so that a later solve (the allocation-free entry
    // point in particular) finds them ready
    b->sec = choose_shape(ctx, b, SEC_CHUNK, MIN_SPLIT_POLES);
    b->lds_chunk = lds_chunk(b, (int64_t)1 << 31);
    b->vec = choose_shape(ctx, b, TILE, MIN_VEC_POLES);
    b->bwd = b->vec;
    Upload up;
    up.add(&b->off_d, b->off_h);
    for (int C : {(int)TILE, b->sec.chunk, b->lds_chunk}) list_add(b, C, up);
    if (b->vsplit > 1) {
        up.add(&b->vsum, std::vector<double>((size_t)nprob * b->vsplit));
        up.add(&b->vst, std::vector<int32_t>((size_t)nprob * b->vsplit));
    }
    hipError_t e;
    void *mem = up.commit(ctx, &e);
    if (!mem) {
        superdc_batch_destroy(b);
        return hip_fail(e);
    }
    b->mem.push_back(mem);
    *out = b;
    return SUPERDC_OK;
}

void superdc_batch_destroy(superdc_batch *b) {
    if (!b) return;
    fmm_free(b->fmm, b, hipDeviceSynchronize() == hipSuccess);
    for (void *p : b->mem) (void)hipFree(p);
    delete b;
}

int64_t superdc_batch_total(const superdc_batch *b) { return b ? b->total : -1; }

int superdc_secular_solve(superdc_ctx *ctx, const superdc_batch *b, const double *d,
                          const double *z, const double *rho, double *lam, double *eta,
                          int32_t *origin, int32_t *iters, int32_t *status,
                          const superdc_opts *opts, void *stream) {
    if (!ctx || !b || b->ctx != ctx || !d || !z || !rho || !lam || !eta || !origin || !status)
        return SUPERDC_EINVAL;
    SDC_OPTS(o, opts);
    hipStream_t s = (hipStream_t)stream;
    SolveArgs a{};
    a.off = b->off_d;
    a.d = d;
    a.z = z;
    a.rho = rho;
    a.dw = (double2 *)ws_get(ctx, WS_DW, sizeof(double2) * b->total);
    a.z2 = (double *)ws_get(ctx, WS_Z2, sizeof(double) * b->nprob);
    a.ke = (double2 *)ws_get(ctx, WS_KE, sizeof(double2) * b->total);
    if (!a.dw || !a.z2 || !a.ke) return SUPERDC_ENOMEM;
    a.lam = lam;
    a.eta = eta;
    a.origin = origin;
    a.iters = iters;
    a.status = status;
    a.stop_c = o.stop_c;
    a.max_iter = o.max_iter;
    a.unshifted = o.unshifted;
    a.hybrid = o.interp;
    superdc_batch *bm = const_cast<superdc_batch *>(b);
    // problems at or above the crossover size use the triangular FMM (method 2: every
    // problem large enough to have two leaves; method 1: none)
    const int crossover = fmm_crossover_of(b, o);
    FmmPlan *fp = nullptr;
    if (b->max_n >= crossover) {
        fp = fmm_plan(bm, o.fmm_leaf, crossover);
        if (!fp) return SUPERDC_ENOMEM;
        if (fp->nfmm == 0) fp = nullptr;
    }
    FmmArgs f{};
    if (fp) {
        f = fmm_args(fp, b, a);
        f.gen = ++fp->own.gen;  // the lists this solve builds
    }
    if (o.persistent) {
        // one launch over the chunks of the direct problems, longest first,
        // and one over the target leaves of the FMM problems
        const LaunchShape sh = b->sec;
        const int max_dir = fp ? fp->max_dir : b->max_n;  // largest direct problem
        const bool lds = solve_in_lds(max_dir, o);
        a.chunk = !lds ? sh.chunk : fp ? fp->lds_chunk : b->lds_chunk;
        if (fp) {
            if (!dir_list(b, fp, a.chunk, a)) return SUPERDC_ENOMEM;
        } else {
            const TileList *L = tile_list(bm, a.chunk);
            if (!L) return SUPERDC_ENOMEM;
            a.tiles = L->lpt;
            a.ntiles = L->count;
        }
        SDC_HIP(launch_validate(a, 0, b->nprob, b->max_n, s, b->vsplit, b->vsum, b->vst));
        if (fp) SDC_HIP(launch_fmm_build(f, s));
        a.work = trace_work(KID_SECULAR);
        if (lds) SDC_HIP(launch_secular_lds(a, max_dir, s));
        else SDC_HIP(launch_secular(a, sh.split, s));
        if (fp) {
            SolveArgs af = a;
            af.tiles = fp->sitem_lpt;
            af.ntiles = fp->snitems;
            af.chunk = fp->ssub;
            af.work = trace_work(KID_SECULAR_FMM);
            const int ss = b->fmm_ssplit > 0 ? b->fmm_ssplit : fp->ssplit;  // tuned or heuristic
            SDC_HIP(launch_secular_fmm(af, f, ss, s));
        }
    } else {
        // one launch per problem, cut into 64-root chunks (split if the problem is large),
        // or its target leaves for an FMM problem
        if (fp) {
            SDC_HIP(launch_validate(a, 0, b->nprob, b->max_n, s, b->vsplit, b->vsum, b->vst));
            SDC_HIP(launch_fmm_build(f, s));
        }
        for (int p = 0; p < b->nprob; ++p) {
            const int64_t np = b->off_h[p + 1] - b->off_h[p];
            if (!fp) SDC_HIP(launch_validate(a, p, 1, (int)np, s));
            if (fp && fp->fmm_of_h[p] >= 0) {
                const int q = fp->fmm_of_h[p];
                SolveArgs af = a;
                af.tiles = fp->sitem_nat + fp->sitem_off_h[q];
                af.ntiles = fp->sitem_off_h[q + 1] - fp->sitem_off_h[q];
                af.chunk = fp->ssub;
                af.work = trace_work(KID_SECULAR_FMM);
                SDC_HIP(launch_secular_fmm(af, f, fp->ssplit, s));
                continue;
            }
            const LaunchShape sh = plain_shape(ctx, np);
            const TileList *L = tile_list(bm, sh.chunk);
            if (!L) return SUPERDC_ENOMEM;
            a.tiles = L->nat + L->begin[p];
            a.ntiles = L->begin[p + 1] - L->begin[p];
            a.chunk = sh.chunk;
            a.work = trace_work(KID_SECULAR);
            SDC_HIP(launch_secular(a, sh.split, s));
        }
    }
    return SUPERDC_OK;
}

int superdc_loewner(superdc_ctx *ctx, const superdc_batch *b, const double *d, const double *z,
                    const double *rho, const double *eta, const int32_t *origin,
                    const int32_t *status, double *zhat, double *bnorm,
                    const superdc_opts *opts, void *stream) {
    return loewner_run(ctx, b, d, z, rho, eta, origin, status, zhat, bnorm, opts, stream, false);
}

int superdc_cauchy_apply(superdc_ctx *ctx, const superdc_batch *b, const double *d,
                         const double *zhat, const double *bnorm, const double *eta,
                         const int32_t *origin, const int32_t *status, int trans, int32_t m,
                         const double *X, int64_t ldx, double *Y, int64_t ldy,
                         const superdc_opts *opts, void *stream) {
    return apply_run(ctx, b, d, zhat, bnorm, eta, origin, status, trans, m, X, ldx, Y, ldy, opts,
                     stream, false);
}

int superdc_secular_backward(superdc_ctx *ctx, const superdc_batch *b, const double *d,
                             const double *z, const double *rho, const double *eta,
                             const int32_t *origin, const int32_t *status,
                             const double *g_lam, const double *g_proj, const double *u,
                             double *g_d, double *g_z, double *g_rho,
                             const superdc_opts *opts, void *stream) {
    if (!ctx || !b || b->ctx != ctx || !d || !z || !rho || !eta || !origin || !status || !g_d ||
        !g_z || !g_rho)
        return SUPERDC_EINVAL;
    if ((g_proj == nullptr) != (u == nullptr)) return SUPERDC_EINVAL;
    SDC_OPTS(o, opts);
    hipStream_t s = (hipStream_t)stream;
    BwdArgs a{};
    a.off = b->off_d;
    a.nprob = b->nprob;
    a.d = d;
    a.z = z;
    a.rho = rho;
    a.eta = eta;
    a.origin = origin;
    a.status = status;
    a.g_lam = g_lam;
    a.g_proj = g_proj;
    a.u = u;
    a.g_d = g_d;
    a.g_z = g_z;
    a.g_rho = g_rho;
    a.rk = (double4 *)ws_get(ctx, WS_BK, sizeof(double4) * b->total);
    a.gk = (double *)ws_get(ctx, WS_BP, sizeof(double) * b->total);
    if (!a.rk || !a.gk) return SUPERDC_ENOMEM;
    superdc_batch *bm = const_cast<superdc_batch *>(b);
    const TileList *L = tile_list(bm, TILE);
    if (!L) return SUPERDC_ENOMEM;
    if (o.persistent) {
        // the large problems through the FMM; all of them directly where its workspace does
        // not fit
        int rc;
        FmmPlan *fp = bwd_by_fmm(b, o) ? fmm_for(bm, o, rc, 1.0) : nullptr;
        const int nw = g_proj ? 2 : 1;  // weights of a pole; of a root one more with projections
        double *pos = nullptr;
        double2 *ke = nullptr;
        FmmArgs f{};
        FmmVec v{};
        if (fp) {
            pos = (double *)ws_get(ctx, WS_VPAIR, sizeof(double2) * b->total);
            ke = (double2 *)ws_get(ctx, WS_KE, sizeof(double2) * b->total);
            if (!pos || !ke || !fmmv_space(ctx, fp, g_proj ? 3 : 1, f, v)) fp = nullptr;
        }
        a.tiles = fp ? fp->dir_lpt[chunk_slot(TILE)] : L->lpt;
        a.ntiles = fp ? fp->dir_count[chunk_slot(TILE)] : L->count;
        SDC_HIP(launch_backward(a, b->bwd.split, s));
        if (fp) {
            a.tiles = fp->leaf_lpt;
            a.ntiles = fp->nitems;
            v.d = d;
            v.origin = origin;
            v.eta = eta;
            v.scale = z;
            v.u = u;
            v.rk = a.rk;
            v.gk = a.gk;
            v.vcen = fp->vcen;
            double *const part = f.vpart;
            // the roots' sums over the poles
            v.kern = 3;
            v.m = nw;
            v.trans = 1;
            f = fmm_vec_args(fp, b, d, eta, origin, status);
            f.sep = FMM_SEP_BWD;
            f.vpart = part;
            f.gen = ++fp->own.gen;
            SDC_HIP(launch_fmm_lists(f, s));
            SDC_HIP(launch_fmmv_sources(f, v, s));
            SDC_HIP(launch_backward_fmm(a, f, v, fp->split, ctx->num_cu, s));
            // the poles' sums over the roots
            FmmvPackArgs pk{};
            pk.off = b->off_d;
            pk.tiles = fp->leaf_nat;
            pk.ntiles = fp->nitems;
            pk.d = d;
            pk.eta = eta;
            pk.origin = origin;
            pk.pos = pos;
            pk.ke = ke;
            SDC_HIP(launch_fmmv_pos(pk, s));
            v.kern = 4;
            v.m = g_proj ? 3 : 1;
            v.trans = 0;
            f = fmm_roots_args(fp, b, pos, status, d);
            f.sep = FMM_SEP_BWD;
            f.vpart = part;
            f.gen = ++fp->roots.gen;
            SDC_HIP(launch_fmm_lists(f, s));
            SDC_HIP(launch_fmmv_sources(f, v, s));
            SDC_HIP(launch_backward_fmm(a, f, v, fp->split, ctx->num_cu, s));
        }
        SDC_HIP(launch_backward_rho(a, 0, b->nprob, s));
    } else {
        for (int p = 0; p < b->nprob; ++p) {
            const int64_t np = b->off_h[p + 1] - b->off_h[p];
            const int S = shape_for(ctx, &np, 1, TILE, MIN_VEC_POLES).split;
            a.tiles = L->nat + L->begin[p];
            a.ntiles = L->begin[p + 1] - L->begin[p];
            SDC_HIP(launch_backward(a, S, s));
            SDC_HIP(launch_backward_rho(a, p, 1, s));
        }
    }
    return SUPERDC_OK;
}

}  // extern "C"
