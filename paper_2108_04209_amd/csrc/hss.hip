// hss.hip -- kernels of the HSS conquering pass (Alg. 3) on gfx950, besides the rank-one
// solver: leaf eigendecompositions, merging of the children's spectra (the sort with
// permutation P_p of Sec. 4.4), assembly of the update columns and of the basis
// recursion, and the permutations and leaf products used to apply the structured
// eigenmatrix Q (Lemma 2, Alg. 4).
//
// Layout: one tree level covers all n entries, node q of level l owning rows
// [q n_l, (q+1) n_l), n_l = leaf 2^(depth-l).  Per-level column blocks (update columns Z,
// basis columns W) are column-major with leading dimension n.  Small generators are
// row-major r x r, stored per node in level order (heap index 2^l - 1 + q).
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "hss.h"

namespace sdc {

// ---------------------------------------------------------------------------------------
// leaf eigendecomposition: cyclic Jacobi in three kernels:
//   k_leaf_jacobi  rotates A -- kept by position, its upper triangle in lines of two rows
//                  (66 KB for a leaf of 128) -- in LDS, two such leaves to a CU (the rounds are
//                  short and end in a barrier: a second leaf's waves fill the first one's
//                  waits), and logs every round's rotations to HBM as (cos, signed sin) by
//                  position;
//   k_leaf_vectors replays the log on V = I with V in registers: a lane holds 16
//                  consecutive positions of 4 rows, so a round is static register code;
//   k_leaf_w       W = Q^T U from the stored eigenvectors.
// The pairs follow the odd-even ordering over positions: round A pairs positions
// (2k, 2k+1), round B pairs (2k+1, 2k+2), and after every round the two indices of a pair
// trade positions.  Over L rounds every pair of indices meets once (the network ends on
// the reversed order, so a sweep reverses the positions), and a pair's rotation only ever
// touches two neighbouring positions.
// ---------------------------------------------------------------------------------------
constexpr int LJ_TILE = 4;  // rows and columns of a thread's tile: two pairs of each
// Tile rows a and T-1-a together have T-1 tiles right of the diagonal: they go to one group of
// lanes.  Threads: the first wavefront and one tile a lane, but at most 8 wavefronts, so that
// two leaves of 128 share a CU at 128 registers (nine had left one leaf to a CU); the last four
// then take the groups left over as well, a 2 x 2 block of each of their tiles per wavefront
constexpr int lj_rows(int L) { return (L + LJ_TILE - 1) / LJ_TILE; }
constexpr int lj_group(int L) { return lj_rows(L) > 16 ? 32 : lj_rows(L) > 8 ? 16 : 8; }
constexpr int lj_waves(int L) {
    return ((lj_rows(L) + 1) / 2 * lj_group(L) + WAVE - 1) / WAVE;
}
constexpr int lj_threads(int L) { return WAVE * (1 + (lj_waves(L) < 7 ? lj_waves(L) : 7)); }
static_assert(lj_waves(LEAF_MAX) <= 8, "at most 64 tiles left over");
constexpr int LV_SEG = 16;                          // positions a lane holds
constexpr int LV_NSEG = LEAF_MAX / LV_SEG;          // segments of a row (8)
constexpr int LV_RPL = 4;                           // rows a lane holds
constexpr int LV_WROWS = WAVE / LV_NSEG * LV_RPL;   // rows per wavefront (32)
constexpr int LV_PAIRS = LEAF_MAX / 2;              // log entries a round is staged with
constexpr int LV_SP = LV_SEG / 2;                   // pairs of a segment in round A (8)
constexpr int LV_CLD = LV_PAIRS + LV_NSEG;          // staged entry k sits at k + k / LV_SP,
                                                    // so the segments' reads hit distinct banks
constexpr int LV_RB = 4;                            // rounds per staged block
static_assert(LEAF_MAX / 2 <= WAVE, "a round's pairs must fit one wavefront");
static_assert(LEAF_MAX <= 128, "columns in four planes of 32");
static_assert(LV_PAIRS == WAVE, "one staged log entry per lane");
static_assert(LV_NSEG * LV_SEG == LEAF_MAX && LV_NSEG <= 16 && 16 % LV_NSEG == 0,
              "a row's segments are neighbouring lanes of one 16-lane DPP row");
static_assert(LV_RB == 4, "a staged block starts on a round A, and two padding rounds negate\n"
              "every position but the first");

// Entry (i, j), i <= j, of an m x m matrix.  Rows i and m-1-i share a line above the diagonal,
// row i < m/2 from its column on and the other from the front; the diagonal lies behind the
// lines, at diag.  A line is four planes of PW words by column mod 4, one word per bank (PW =
// 32; 16 for leaves up to 64): the lanes of a group read one column of tile row a (banks from
// a + 1 on) and of tile row T-1-a (banks up to a) without conflicts.  With planes of 16, the
// next group's lines have theirs swapped, so that two groups share the banks; the lines
// are skewed by a bank every few, which spreads the entries near the diagonal.
template <int PW>
__device__ __forceinline__ int ut(int i, int j, int m, int diag) {
    if (i == j) return diag + i;
    const int line = min(i, m - 1 - i);
    const int x = i == line ? j : j - i - 1;
    const int plane = PW == 32 ? x & 3 : (x & 3) ^ ((line >> 2) & 1);
    return (line * 4 + plane) * PW + (((x >> 2) + (line >> (PW == 32 ? 2 : 3))) & (PW - 1));
}

// cos and sin of the rotation with tangent t
__device__ __forceinline__ double2 rot_cs(double t) {
    const double c = rcp_nr(sqrt(t * t + 1.0));
    return make_double2(c, t * c);
}

// 1 / sqrt(t) for t well inside the exponent range, to about an ulp
__device__ __forceinline__ double rsqrt_nr(double t) {
    double r = __builtin_amdgcn_rsq(t);
    double g = t * r, h = 0.5 * r;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const double e = __builtin_fma(-h, g, 0.5);
        g = __builtin_fma(g, e, g);
        h = __builtin_fma(h, e, h);
    }
    return 2.0 * h;
}

// The matrix is kept by position: entry (i, j) of the stored upper triangle is the entry
// of the two indices at positions i and j.  A round's rotation of pair k then acts on the
// positions (l, r) of the pair by the reflection [[sigma, c], [c, -sigma]] -- the rotation
// followed by the trade of positions -- with theta = (A(r,r) - A(l,l)) / (2 A(l,r)) taken
// at the positions (the sign of sigma then comes out right whichever of the two indices is
// the smaller), and the round is A <- R A R with R the direct sum of the reflections (the
// identity on the two positions that sit out round B).  Every 2 x 2 block (rows of pair P1,
// columns of pair P2) depends only on its own four entries, so a round is a single pass over
// the blocks P1 <= P2 at addresses fixed for each round type.  Diagonal blocks take
// (x, w; w, y) to (y + t w, 0; 0, x - t w), or to (y, w; w, x) when there is no rotation.
//
// The first wavefront owns the blocks that the next round's rotations read: the diagonal
// blocks, the blocks (k, k+1) of neighbouring pairs and the block (0, m/2 - 1).  A pair of
// the next round joins one position of pair k and one of pair k+1 of this round (or a
// position that sits the round out), so its three entries all lie in those blocks.  That
// wavefront therefore computes the next round's rotations right after its own blocks,
// while the other wavefronts still update theirs, and a round ends in a single barrier;
// the rotation data is double-buffered by round parity.  The other blocks are cut into
// tiles of two pairs by two, one to a thread, with the addresses of a tile's 16 entries per
// round type in registers; entries that are not the thread's (the first wavefront's blocks,
// pairs past the last) go to a spare word of the bank that is free.
//
// What bounded a round of two leaves of 128 on a CU was the issue of instructions (75 to a
// 2 x 2 block, 16 of them in FP64, with the blocks dealt one by one over 16 wavefronts) and,
// for small leaves, the first wavefront's chain of three square roots and three reciprocals.
// Measured: 512 leaves of 128 2580 -> 1900 us with tiles and two reciprocal square roots, the
// LDS then busy two thirds of the time -> 1640 with the tiles in registers (RES) -> 1350 with the
// tiles left over spread over four wavefronts instead of one; 32 leaves of 32 330 -> 132 us.
// What is left is the chain of a round (32 leaves of 128, one to a CU, take 820 us).
//
// RES: a tile's entries off the rows and columns 0 mod 4 belong to the same thread in both round
// types (a round B takes the tile one row and column further on), and stay in its registers
// from round to round: 8 words each way through the LDS instead of 16.  Two of them change
// hands all the same, where a tile touches the first wavefront's blocks: entry (3, 2) or, in
// round B, (1, 0) beside the diagonal, (2, 3) and (0, 1) in the tile of the block (0, m/2 - 1).
// Leaves of whole tiles only (a multiple of 4), with those two kinds of tile apart (12 and more).
template <int LP, bool RES>
__global__ __launch_bounds__(lj_threads(LP), 4) void k_leaf_jacobi(LeafArgs a) {
    // upper triangle by position, its diagonal, and PW spare words, one per bank
    constexpr int PW = LP > 64 ? 32 : 16, DIAG = LP / 2 * 4 * PW, SPARE = DIAG + LP;
    __shared__ double A[SPARE + PW];
    // (c, sigma) of each pair, by round type; even pairs, then odd ones (a tile takes one of
    // each, so neighbouring lanes read neighbouring entries)
    __shared__ double2 cs[2][2][LP / 4];
    __shared__ double tt[2][LP / 2];   // tangent of each pair's rotation (0: none)
    __shared__ double red[lj_threads(LP) / WAVE];
    __shared__ int swept[2];       // per sweep parity: the sweep rotated something
    __shared__ int swbig[2];       // per sweep parity: some tangent was at least 1e-6

    const int leafid = blockIdx.x;
    const int L = a.leaf;
    const int tid = threadIdx.x, nt = blockDim.x;
    const double *D = a.D + (size_t)leafid * L * L;
    // Frobenius norm (of the whole block) for the absolute part of the rotation threshold
    double fro = 0.0;
    for (int e = tid; e < L * L; e += nt) {
        const int i = e / L, j = e - i * L;
        const double v = D[e];
        if (i <= j) A[ut<PW>(i, j, L, DIAG)] = v;
        fro += v * v;
    }
    for (int o = WAVE / 2; o > 0; o >>= 1) fro += __shfl_xor(fro, o);
    if (lane_id() == 0) red[tid / WAVE] = fro;
    const int m = L;  // even
    const int half = m / 2;
    constexpr int spare = SPARE;
    if (tid < PW) A[spare + tid] = 0.0;
    __syncthreads();
    double tot = 0.0;
    for (int w = 0; w < nt / WAVE; ++w) tot += red[w];
    const double absfloor = 1e-18 * sqrt(tot);
    // squares of the entries stay in range (see rotations)
    const bool plain = __builtin_amdgcn_readfirstlane(tot >= 0x1p-800 && tot <= 0x1p800);
    const int total = a.max_sweeps * m;     // rounds the log has room for
    double2 *log = reinterpret_cast<double2 *>(a.rot) + (size_t)leafid * total * half;
    const bool first = tid < WAVE;
    // pair P's v-th position in a round of type p; in round B the last pair is (m - 1, 0), which
    // sits the round out
    auto position = [&](int P, int v, int p) { return 2 * P + v + p == m ? 0 : 2 * P + v + p; };
    auto entry = [&](int i, int j) { return i <= j ? ut<PW>(i, j, m, DIAG) : ut<PW>(j, i, m, DIAG); };
    // the blocks of a round that are not the first wavefront's
    auto tiled = [&](int P1, int P2) {
        return P2 < half && P2 - P1 > 1 && !(P1 == 0 && P2 == half - 1);
    };

    // Addresses in this thread's registers, two to a word, per round type.  First wavefront,
    // lane k (in edge): words 0 and 1 the diagonal block of pair k (left, right, between them), words
    // 2 and 3 a block of neighbours, (k, k+1) in round A and (k-1, k) in round B, or, in the
    // lane left over, the block (0, m/2 - 1).  Others: entries (v, 2h), (v, 2h+1) of the tile in
    // word 2v + h.
    struct Tile4 {
        int ad[2][8];
        int P1, P2;        // first row and column pair (first wavefront: of its block, round A)
        int out;           // bit h: column pair P2 + h sits round B out
    };
    Tile4 t0;
    double x[4][4];        // RES: the tile
    int edge[2][4];        // RES: two addresses to a word: entries 0 .. 3 of the tile's row 0 (round
                           // B: 3), the other three of its column 0 (3), the one that changes hands
    bool beside = false, corner = false;  // beside the diagonal; with the block (0, m/2 - 1)
    int Q1 = 0, Q2 = 0;  // first wavefront: the pairs of its block in round B
    bool sits = false;   // whose column pair sits the round out
    int &P1 = t0.P1, &P2 = t0.P2;
    P1 = P2 = 0;
    const int T = (half + 1) / 2, G = lj_group(m);
    auto take = [&](int e, Tile4 &t) {
        int ta = e / G, tb = ta + 1 + e % G;
        const int row = min(ta, T - 1);  // the group's first tile row
        if (2 * ta >= T) {
            tb = half;  // past the tiles: nothing valid
        } else if (tb >= T) {  // the group's second tile row
            const int other = T - 1 - ta;
            tb = other > ta && tb - T < ta ? tb - T + other + 1 : half;
            ta = other;
        }
        ta = max(min(ta, T - 2), 0);
        t.P1 = 2 * ta;
        t.P2 = min(2 * tb, (half - 1) & ~1);
        t.out = 2 * tb == half - 1 ? 1 : 2 * tb == half - 2 ? 2 : 0;  // the last pair
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int R = 2 * ta + (v >> 1), S = 2 * tb + h;
                    int w[2];
                    for (int u = 0; u < 2; ++u) {
                        if (tb < T && S < half) {
                            w[u] = entry(position(R, v & 1, p), position(S, u, p));
                            if (!tiled(R, S)) w[u] = spare + w[u] % PW;  // the same bank
                        } else {  // a lane without a tile: the bank that its group leaves free
                            const int line = 4 * row + v + p;
                            const int free = 2 * h + u <= v ? row : 0;
                            w[u] = spare + (free + (line >> (PW == 32 ? 2 : 3))) % PW;
                        }
                    }
                    t.ad[p][2 * v + h] = w[0] | w[1] << 16;
                }
    };
    // block (mi, mh) of a tile left over: its addresses, pairs and whether its columns sit round B out
    const bool more = LP > 64 && tid >= 4 * WAVE && lj_waves(m) > 7;
    const int mi = (wave_uniform(tid / WAVE) >> 1) & 1, mh = wave_uniform(tid / WAVE) & 1;
    int mad[2][2], mP = 0, mS = 0;
    bool mout = false;
    if (first) {
        const int k = tid;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const bool diag = k < half && !(p && k == half - 1);
            const int l = 2 * k + p;
            (RES ? edge[p] : t0.ad[p])[0] = diag ? ut<PW>(l, l, m, DIAG) | ut<PW>(l + 1, l + 1, m, DIAG) << 16 : spare | spare << 16;
            (RES ? edge[p] : t0.ad[p])[1] = diag ? ut<PW>(l, l + 1, m, DIAG) : spare;
            const int left = p ? 0 : half - 1;  // the lane left over
            int R = p ? k - 1 : k, S = R + 1;
            bool has = k < half && k != left;
            if (k == left && half >= 3) {
                R = 0;
                S = half - 1;
                has = true;
            }
            if (!has) R = S = 0;
            if (p) {
                Q1 = R;
                Q2 = S;
            } else {
                P1 = R;
                P2 = S;
            }
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                const int r = position(R, v, p);
                (RES ? edge[p] : t0.ad[p])[2 + v] = has ? entry(r, position(S, 0, p)) | entry(r, position(S, 1, p)) << 16
                                   : spare | spare << 16;
            }
            if (p) sits = has && S == half - 1;
        }
    } else {
        take(tid - WAVE, t0);
        if (RES) {
            beside = P2 == P1 + 2;
            corner = P1 == 0 && P2 == half - 2;
            auto at = [&](int p, int v, int u) {
                const int w = t0.ad[p][2 * v + (u >> 1)];
                return u & 1 ? (int)((unsigned)w >> 16) : w & 0xffff;
            };
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int e = p ? 3 : 0, f = p ? 0 : 1;  // the edge, the first entry off it
                const int hand = p ? (corner ? at(1, 0, 1) : at(1, 1, 0))
                                   : (corner ? at(0, 2, 3) : at(0, 3, 2));
                edge[p][0] = at(p, e, 0) | at(p, e, 1) << 16;
                edge[p][1] = at(p, e, 2) | at(p, e, 3) << 16;
                edge[p][2] = at(p, f, e) | at(p, f + 1, e) << 16;
                edge[p][3] = at(p, f + 2, e) |
                             (beside || corner ? hand : spare + hand % PW) << 16;
            }
#pragma unroll
            for (int v = 1; v < 4; ++v)
#pragma unroll
                for (int u = 1; u < 4; ++u) x[v][u] = A[at(0, v, u)];
        }
        if (more) {  // past the 7 wavefronts' first tiles
            Tile4 t1;
            take(7 * WAVE + lane_id(), t1);
            mP = t1.P1 >> 1;
            mS = t1.P2 >> 1;
            mout = (t1.out >> mh) & 1;
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int v = 0; v < 2; ++v)
                    mad[p][v] = mi ? (mh ? t1.ad[p][5 + 2 * v] : t1.ad[p][4 + 2 * v])
                                   : (mh ? t1.ad[p][1 + 2 * v] : t1.ad[p][2 * v]);
        }
    }
    auto lo = [](int w) { return w & 0xffff; };
    auto hi = [](int w) { return (int)((unsigned)w >> 16); };
    // rows of a 2 x 2 block by the reflection (c, s) of their pair, and columns; a column pair
    // that sits the round out has (0, 1) and keeps its second column too
    auto rows = [](double2 r, double &x0, double &x1) {
        const double y = fma(r.x, x1, r.y * x0);
        x1 = fma(r.x, x0, -(r.y * x1));
        x0 = y;
    };
    auto cols = [](double2 r, double n, double &x0, double &x1) {
        const double y = fma(r.x, x1, r.y * x0);
        x1 = fma(r.x, x0, n * x1);
        x0 = y;
    };

    // rotations of round g of type p (first wavefront, lane k: pair k) into buffer p, with the
    // log entry; returns the lane's tangent (0: no rotation)
    auto rotations = [&](int g, auto par) -> double {
        constexpr int p = decltype(par)::value;
        const int *const ad = RES ? edge[p] : t0.ad[p];
        const int k = tid;
        double t = 0.0;
        const double x = A[lo(ad[0])], y = A[hi(ad[0])], w = A[ad[1]];
        if (k < half) {
            const bool idle = p && k == half - 1;
            double2 r = make_double2(1.0, 0.0);
            if (plain) {
                // |w| > eps sqrt(|x y|) + absfloor by squares; with d = y - x, r = 1 / sqrt(d^2 +
                // 4 w^2): cos 2 phi = |d| r and c = sqrt((1 + cos 2 phi) / 2), so that two
                // reciprocal square roots give the whole rotation
                const double over = fabs(w) - absfloor;
                const double d = y - x;
                const double ri = rsqrt_nr(fma(d, d, 4.0 * (w * w)));
                const double c2 = fma(0.5 * fabs(d), ri, 0.5);
                const double rc = rsqrt_nr(c2);
                const double ws = d > 0.0 ? w : d < 0.0 ? -w : fabs(w);
                if (!idle && over > 0.0 && over * over > 0x1p-104 * fabs(x * y)) {
                    const double s = ws * ri * rc, c = c2 * rc;
                    t = s * rc;
                    // c and s come from two roots, each an ulp off to one side: bring c^2 + s^2
                    // back to 1 (leaf of 128: ||Q^T Q - I|| 2.7e-13 -> 3.3e-14, with s = t c
                    // 2.3e-13; an HSS conquer of 65536 rows 15.65 -> 15.68 ms)
                    const double h = -0.5 * fma(s, s, fma(c, c, -1.0));
                    r = make_double2(fma(h, c, c), fma(h, s, s));
                }
            } else if (!idle && fabs(w) > 2.220446049250313e-16 * sqrt(fabs(x) * fabs(y)) + absfloor) {
                // the rotation only has to annihilate w to rounding, so reciprocals by
                // Newton-refined estimates stand in for the divisions
                const double theta = (y - x) * (0.5 * rcp_nr(w));
                if (fabs(theta) > 1e150) t = 0.5 * rcp_nr(theta);
                else t = (theta >= 0.0 ? 1.0 : -1.0) * rcp_nr(fabs(theta) + sqrt(theta * theta + 1.0));
                if (t != 0.0) r = rot_cs(t);
            }
            cs[p][k & 1][k >> 1] = idle ? make_double2(0.0, 1.0) : r;
            tt[p][k] = t;
            // the left position's new column is c y + sigma x and the right one's
            // c x - sigma y, for the columns x, y at the two positions before the round
            if (!idle) {
                // the lane's offset through an empty asm, so that the per-lane log address is
                // formed here rather than held in registers through the rounds
                int kk = k;
                asm volatile("" : "+v"(kk));
                log[(size_t)g * half + kk] = r;
            }
        }
        return t;
    };
    // whether some pair (i, j) of the matrix as it stands would pass the rotation test, over
    // all threads (ends in a barrier).  A sweep that rotates nothing leaves the matrix as it
    // is, so when no pair passes, the next sweep would be empty.  It runs about once per
    // leaf: the thread index goes through an empty asm so that none of its index
    // arithmetic is hoisted out of the rounds and held in registers through them.
    auto any_pair_rotates = [&]() -> bool {
        int t = tid;
        asm volatile("" : "+v"(t));
        const int tpr = nt / m;  // threads per row
        const int i = t / tpr;
        bool any = false;
        if (i < m) {
            const double x = fabs(A[ut<PW>(i, i, m, DIAG)]);
            for (int j = i + 1 + t % tpr; j < m; j += tpr)
                any |= fabs(A[ut<PW>(i, j, m, DIAG)]) > 2.220446049250313e-16 * sqrt(x * fabs(A[ut<PW>(j, j, m, DIAG)])) + absfloor;
        }
        return __syncthreads_or(any);
    };

    // first wavefront: whether the current sweep has rotated anything so far, and anything
    // by a tangent of at least 1e-6
    bool rot_acc = false, big_acc = false;
    auto note = [&](double t) {
        rot_acc |= __any(t != 0.0);
        big_acc |= __any(fabs(t) >= 1e-6);
    };
    auto update = [&](const Tile4 &t, auto par) {
        constexpr int p = decltype(par)::value;
        const double2 r0 = cs[p][0][t.P1 >> 1], r1 = cs[p][1][t.P1 >> 1];
        const double2 q0 = cs[p][0][t.P2 >> 1], q1 = cs[p][1][t.P2 >> 1];
        double x[4][4];
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                x[v][2 * h] = A[lo(t.ad[p][2 * v + h])];
                x[v][2 * h + 1] = A[hi(t.ad[p][2 * v + h])];
            }
        const double n0 = p && (t.out & 1) ? q0.y : -q0.y, n1 = p && (t.out & 2) ? q1.y : -q1.y;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            rows(r0, x[0][u], x[1][u]);
            rows(r1, x[2][u], x[3][u]);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            cols(q0, n0, x[v][0], x[v][1]);
            cols(q1, n1, x[v][2], x[v][3]);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                A[lo(t.ad[p][2 * v + h])] = x[v][2 * h];
                A[hi(t.ad[p][2 * v + h])] = x[v][2 * h + 1];
            }
        }
    };
    // the same with the tile in registers
    auto update_res = [&](auto par) {
        constexpr int p = decltype(par)::value;
        const double2 r0 = cs[p][0][P1 >> 1], r1 = cs[p][1][P1 >> 1];
        const double2 q0 = cs[p][0][P2 >> 1], q1 = cs[p][1][P2 >> 1];
        constexpr int e = p ? 3 : 0, f = p ? 0 : 1;
        double y[4][4];
#pragma unroll
        for (int v = 0; v < 3; ++v)
#pragma unroll
            for (int u = 0; u < 3; ++u) y[f + v][f + u] = x[1 + v][1 + u];
        y[e][0] = A[lo(edge[p][0])];
        y[e][1] = A[hi(edge[p][0])];
        y[e][2] = A[lo(edge[p][1])];
        y[e][3] = A[hi(edge[p][1])];
        y[f][e] = A[lo(edge[p][2])];
        y[f + 1][e] = A[hi(edge[p][2])];
        y[f + 2][e] = A[lo(edge[p][3])];
        const double hand = A[hi(edge[p][3])];
        double &b = y[p ? 1 : 3][p ? 0 : 2], &c = y[p ? 0 : 2][p ? 1 : 3];
        b = beside ? hand : b;
        c = corner ? hand : c;
        const double n0 = -q0.y, n1 = p && (t0.out & 2) ? q1.y : -q1.y;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            rows(r0, y[0][u], y[1][u]);
            rows(r1, y[2][u], y[3][u]);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            cols(q0, n0, y[v][0], y[v][1]);
            cols(q1, n1, y[v][2], y[v][3]);
        }
        A[lo(edge[p][0])] = y[e][0];
        A[hi(edge[p][0])] = y[e][1];
        A[lo(edge[p][1])] = y[e][2];
        A[hi(edge[p][1])] = y[e][3];
        A[lo(edge[p][2])] = y[f][e];
        A[hi(edge[p][2])] = y[f + 1][e];
        A[lo(edge[p][3])] = y[f + 2][e];
        A[hi(edge[p][3])] = corner ? c : b;
#pragma unroll
        for (int v = 0; v < 3; ++v)
#pragma unroll
            for (int u = 0; u < 3; ++u) x[1 + v][1 + u] = y[f + v][f + u];
    };
    // the tiles' registers into the matrix, after a round B
    auto flush = [&]() {
        if (!RES || first) return;
        int e = tid - WAVE;
        asm volatile("" : "+v"(e));  // its addresses formed here, not held through the rounds
        Tile4 t;
        take(e, t);
#pragma unroll
        for (int v = 0; v < 3; ++v)
#pragma unroll
            for (int u = 0; u < 3; ++u) {
                const int w = t.ad[1][2 * v + (u >> 1)];
                A[u & 1 ? hi(w) : lo(w)] = x[1 + v][1 + u];
            }
    };
    // round g of type p up to its barrier; next: the first wavefront goes on to the rotations
    // of round g + 1
    auto round = [&](int g, auto par, bool next) {
        constexpr int p = decltype(par)::value;
        const int *const ad = RES ? edge[p] : t0.ad[p];
        if (first) {
            // all loads first: lane k's diagonal block and its block of neighbours
            const double t = tt[p][min(tid, half - 1)];
            const int R = p ? Q1 : P1, S = p ? Q2 : P2;
            const double2 r1 = cs[p][R & 1][R >> 1], r2 = cs[p][S & 1][S >> 1];
            const double x = A[lo(ad[0])], y = A[hi(ad[0])], w = A[ad[1]];
            double x00 = A[lo(ad[2])], x01 = A[hi(ad[2])];
            double x10 = A[lo(ad[3])], x11 = A[hi(ad[3])];
            A[lo(ad[0])] = fma(t, w, y);
            A[hi(ad[0])] = fma(-t, w, x);
            A[ad[1]] = t != 0.0 ? 0.0 : w;
            rows(r1, x00, x10);
            rows(r1, x01, x11);
            const double n = p && sits ? r2.y : -r2.y;
            cols(r2, n, x00, x01);
            cols(r2, n, x10, x11);
            A[lo(ad[2])] = x00;
            A[hi(ad[2])] = x01;
            A[lo(ad[3])] = x10;
            A[hi(ad[3])] = x11;
            if (next) {
                wave_sync();
                note(rotations(g + 1, std::integral_constant<int, 1 - p>{}));
            }
        } else {
            if (RES) update_res(par);
            else update(t0, par);
            if (more) {
                const double2 r = cs[p][mi][mP], q = cs[p][mh][mS];
                const double n = p && mout ? q.y : -q.y;
                double x00 = A[lo(mad[p][0])], x01 = A[hi(mad[p][0])];
                double x10 = A[lo(mad[p][1])], x11 = A[hi(mad[p][1])];
                rows(r, x00, x10);
                rows(r, x01, x11);
                cols(q, n, x00, x01);
                cols(q, n, x10, x11);
                A[lo(mad[p][0])] = x00;
                A[hi(mad[p][0])] = x01;
                A[lo(mad[p][1])] = x10;
                A[hi(mad[p][1])] = x11;
            }
        }
        __syncthreads();
    };
    const std::integral_constant<int, 0> roundA{};
    const std::integral_constant<int, 1> roundB{};
    if (first) {
        wave_priority(3);  // the other wavefronts wait for its chain at every barrier
        note(rotations(0, roundA));
    }
    __syncthreads();
    int sweep = 0;
    bool converged = false, reversed = false;  // reversed: an empty sweep ran
    for (int g = 0, left = half;; g += 2) {  // left: round pairs of the sweep
        round(g, roundA, true);
        if (--left == 0 && first) {  // the sweep's last round is decided
            if (tid == 0) {
                swept[sweep & 1] = rot_acc;
                swbig[sweep & 1] = big_acc;
            }
            rot_acc = big_acc = false;
        }
        round(g + 1, roundB, g + 2 < total);
        if (left == 0) {  // the end of a sweep
            left = half;
            if (!swept[sweep & 1]) {  // a sweep without rotations: nothing of it needs replaying
                converged = reversed = true;
                break;
            }
            const bool big = swbig[sweep & 1];
            ++sweep;
            // once the sweep's rotations are all tiny, the next one may well be empty: test
            // every pair now instead of running it to find out (the same decision)
            if (!big) {
                flush();
                __syncthreads();
                if (!any_pair_rotates()) {
                    converged = true;
                    break;
                }
            }
            if (sweep == a.max_sweeps) break;
        }
    }
    // ascending order of the eigenvalues (ties broken by position).  A sweep reverses the
    // positions, and the replay stops short of a last sweep without rotations, so position j
    // here is position m-1-j of the replayed vectors when that sweep ran
    if (tid < L) {
        const double v = A[ut<PW>(tid, tid, L, DIAG)];
        int r = 0;
        for (int j = 0; j < L; ++j) {
            const double w = A[ut<PW>(j, j, L, DIAG)];
            r += (w < v) || (w == v && j < tid);
        }
        a.rank[(size_t)leafid * L + (reversed ? L - 1 - tid : tid)] = r;
        a.lam[(size_t)leafid * L + r] = v;
    }
    if (tid == 0) {
        a.sweeps[leafid] = sweep;
        a.status[leafid] = converged ? 0 : SUPERDC_ST_NOCONV;
    }
}

// value of the neighbouring lane (lane + 1 for UP, lane - 1 otherwise) within a row of 16
// lanes; the lanes at a row's end get their own value back
template <bool UP>
__device__ __forceinline__ double lane_shift(double x) {
    constexpr int ctrl = UP ? 0x101 : 0x111;  // DPP row_shl:1 / row_shr:1
    const long long b = __double_as_longlong(x);
    const int lo = (int)(b & 0xffffffffll), hi = (int)(b >> 32);
    const int l2 = __builtin_amdgcn_update_dpp(lo, lo, ctrl, 0xf, 0xf, false);
    const int h2 = __builtin_amdgcn_update_dpp(hi, hi, ctrl, 0xf, 0xf, false);
    return __longlong_as_double(((long long)h2 << 32) | (unsigned int)l2);
}

// the LV_RB rounds of a staged block, whose first round is a round A (static code with no
// exit between the rounds, so V keeps its registers through the block)
__device__ __forceinline__ void replay_block(double (&v)[LV_RPL][LV_SEG], const double2 (*c)[LV_CLD],
                                             int sg, bool has_left) {
#pragma unroll
    for (int u = 0; u < LV_RB; ++u) {
        const double2 *cu = c[u] + sg * (LV_SP + 1);  // entries 8 sg .. 8 sg + 7
        if ((u & 1) == 0) {
            // round A: pairs (2j, 2j+1) of the segment
#pragma unroll
            for (int j = 0; j < LV_SP; ++j) {
                const double2 e = cu[j];
#pragma unroll
                for (int r = 0; r < LV_RPL; ++r) {
                    const double x = v[r][2 * j], y = v[r][2 * j + 1];
                    v[r][2 * j] = fma(e.x, y, e.y * x);
                    v[r][2 * j + 1] = fma(e.x, x, -(e.y * y));
                }
            }
        } else {
            // round B: pairs (2j+1, 2j+2) inside the segment, and the pairs across its
            // ends: (16 sg + 15, 16 sg + 16) with entry 8 sg + 7 on the right, and
            // (16 sg - 1, 16 sg) with entry 8 sg - 1 on the left
            // the last segment's entry 8 sg + 7 is past the round's pairs, so (0, 1) keeps
            // its last position; the first segment has no left pair, and (0, -1) keeps
            // its first position (the neighbours' values are finite either way)
            const double2 er = cu[LV_SP - 1];
            double2 el = cu[has_left ? -2 : 0];
            if (!has_left) el = make_double2(0.0, -1.0);
#pragma unroll
            for (int r = 0; r < LV_RPL; ++r) {
                const double y = lane_shift<true>(v[r][0]);             // right neighbour's first
                const double x = lane_shift<false>(v[r][LV_SEG - 1]);  // left neighbour's last
                const double xs = v[r][LV_SEG - 1], ys = v[r][0];
                v[r][LV_SEG - 1] = fma(er.x, y, er.y * xs);
                v[r][0] = fma(el.x, x, -(el.y * ys));
            }
#pragma unroll
            for (int j = 0; j < LV_SP - 1; ++j) {
                const double2 e = cu[j];
#pragma unroll
                for (int r = 0; r < LV_RPL; ++r) {
                    const double x = v[r][2 * j + 1], y = v[r][2 * j + 2];
                    v[r][2 * j + 1] = fma(e.x, y, e.y * x);
                    v[r][2 * j + 2] = fma(e.x, x, -(e.y * y));
                }
            }
        }
    }
}

// Replay of the rotation log on V = I.  Rows of V J are independent and a round's
// rotations touch neighbouring positions only, so V stays in registers: wavefront w of a
// leaf owns rows [32 w, 32 w + 32); lane 8 g + s holds rows 32 w + 4 g .. + 3 at positions
// [16 s, 16 s + 16) (positions past the leaf are zero padding).  Each round is static code:
// pairs inside a segment from registers, the pairs across segments (round B) with the
// neighbouring lane's value.  The log streams through LDS a block of rounds at a time, the
// next block's loads in flight; only this wavefront touches its LDS, so no barrier is
// needed.  A log entry (c, sigma) takes the columns x, y at the pair's positions to
// (c y + sigma x, c x - sigma y); entries past a round's real pairs are (0, 1), which keeps
// x in place and only negates the padding.
__global__ __launch_bounds__(WAVE, 2) void k_leaf_vectors(LeafArgs a) {
    __shared__ double2 cf[2][LV_RB][LV_CLD];
    const int L = a.leaf, half = L / 2;
    const int nwl = (L + LV_WROWS - 1) / LV_WROWS;
    const int leafid = blockIdx.x / nwl, w = blockIdx.x - leafid * nwl;
    const int lane = threadIdx.x;
    const int sg = lane % LV_NSEG;
    const int row0 = w * LV_WROWS + (lane / LV_NSEG) * LV_RPL, pos0 = sg * LV_SEG;
    const bool has_left = sg > 0;
    double v[LV_RPL][LV_SEG];
#pragma unroll
    for (int r = 0; r < LV_RPL; ++r)
#pragma unroll
        for (int j = 0; j < LV_SEG; ++j) v[r][j] = (row0 + r == pos0 + j) ? 1.0 : 0.0;

    const double2 *log = reinterpret_cast<const double2 *>(a.rot) + (size_t)leafid * a.max_sweeps * L * half;
    const int nsw = a.sweeps[leafid];
    const int rounds = nsw * L;  // L is even: round rd is a round A when rd is even
    // whole blocks only: when the rounds end half-way through a block, its last two rounds
    // run on (0, 1) entries, which keep x and negate y -- over a round A and a round B that
    // negates every position but 0, undone when the vectors are written
    const int nblk = (rounds + LV_RB - 1) / LV_RB;
    const bool padded = rounds % LV_RB != 0;
    const int slot = lane + lane / LV_SP;  // where this lane stages its entry
    double2 nx[LV_RB];
#pragma unroll
    for (int u = 0; u < LV_RB; ++u)
        nx[u] = (u < rounds && lane < half - (u & 1)) ? log[(size_t)u * half + lane] : make_double2(0.0, 1.0);
    for (int b = 0; b < nblk; ++b) {
        double2(*c)[LV_CLD] = cf[b & 1];
#pragma unroll
        for (int u = 0; u < LV_RB; ++u) c[u][slot] = nx[u];
        wave_sync();
#pragma unroll
        for (int u = 0; u < LV_RB; ++u) {
            const int rr = (b + 1) * LV_RB + u;
            nx[u] = (rr < rounds && lane < half - (u & 1)) ? log[(size_t)rr * half + lane]
                                                          : make_double2(0.0, 1.0);
        }
        replay_block(v, c, sg, has_left);
        wave_sync();
    }
    // the column at position pos is the eigenvector whose ascending rank the Jacobi kernel
    // stored for that position
    const int32_t *rank = a.rank + (size_t)leafid * L;
    double *Q = a.Q + (size_t)leafid * L * L;  // eigenvector k contiguous
#pragma unroll
    for (int j = 0; j < LV_SEG; ++j) {
        const int pos = pos0 + j;
        if (pos >= L) continue;
        const size_t k = (size_t)rank[pos];
        const bool flip = padded && pos != 0;
#pragma unroll
        for (int r = 0; r < LV_RPL; ++r)
            if (row0 + r < L) Q[k * L + row0 + r] = flip ? -v[r][j] : v[r][j];
    }
}

// W = Q^T U (L x r) per leaf, column-major with leading dimension ldw over the whole level
__global__ __launch_bounds__(256) void k_leaf_w(LeafArgs a) {
    __shared__ double Us[LEAF_MAX * LEAF_RANK_MAX];
    const int leafid = blockIdx.x;
    const int L = a.leaf, r = a.r, tid = threadIdx.x;
    const double *U = a.U + (size_t)leafid * L * r;
    for (int e = tid; e < L * r; e += blockDim.x) Us[e] = U[e];
    __syncthreads();
    const double *Q = a.Q + (size_t)leafid * L * L;
    for (int e = tid; e < L * r; e += blockDim.x) {
        const int k = e % L, c = e / L;
        const double *q = Q + (size_t)k * L;
        double acc = 0.0;
        for (int i = 0; i < L; ++i) acc = __builtin_fma(q[i], Us[i * r + c], acc);
        a.W[(int64_t)c * a.ldw + (int64_t)leafid * L + k] = acc;
    }
}

// ---------------------------------------------------------------------------------------
// merge of the two sorted child spectra of every node of a level, with the permutation
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ int count_less(const double *x, int n, double v) {
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (x[mid] < v) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

__device__ __forceinline__ int count_leq(const double *x, int n, double v) {
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (x[mid] <= v) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

__global__ __launch_bounds__(256) void k_merge(const double *lam_children, double *d_out,
                                               int32_t *perm, int nc, int64_t total) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    const int64_t node = e / (2 * nc);
    const int loc = (int)(e % (2 * nc));
    const int64_t base = node * 2 * nc;
    const double *A = lam_children + base, *B = A + nc;
    int pos;
    double v;
    if (loc < nc) {
        v = A[loc];
        pos = loc + count_less(B, nc, v);
    } else {
        v = B[loc - nc];
        pos = (loc - nc) + count_leq(A, nc, v);
    }
    d_out[base + pos] = v;
    perm[base + pos] = loc;
}

// Runs of SORT_RUN keys of every segment of nl, sorted in LDS (one workgroup a run): the first
// passes of the merge sort below, without a launch each (a segment of 65536 keys took 16; the
// 18 steps of a deflated HSS pass over 65536 rows 8.73 -> 8.54 ms in all).
constexpr int SORT_RUN = 2048;
__global__ __launch_bounds__(1024) void k_sort_runs(const double *kin, double *kout, int32_t *vout,
                                                    int nl, int nrun) {
    __shared__ double key[2][SORT_RUN];
    __shared__ uint16_t idx[2][SORT_RUN];
    const int r0 = (blockIdx.x % nrun) * SORT_RUN;  // the run's place in its segment
    const int len = min(SORT_RUN, nl - r0);
    const int64_t base = (int64_t)(blockIdx.x / nrun) * nl + r0;
    for (int i = threadIdx.x; i < len; i += blockDim.x) {
        key[0][i] = kin[base + i];
        idx[0][i] = (uint16_t)i;
    }
    int b = 0;
    for (int w = 1; w < len; w <<= 1, b ^= 1) {
        __syncthreads();
        for (int i = threadIdx.x; i < len; i += blockDim.x) {
            const int ps = i & ~(2 * w - 1);
            const int mid = min(ps + w, len), end = min(ps + 2 * w, len);
            const double v = key[b][i];
            int pos = i;
            if (mid < end && key[b][mid] < key[b][mid - 1])  // else the pair is in order
                pos = i < mid ? i + count_less(key[b] + mid, end - mid, v)
                              : i - mid + ps + count_leq(key[b] + ps, mid - ps, v);
            key[b ^ 1][pos] = v;
            idx[b ^ 1][pos] = idx[b][i];
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < len; i += blockDim.x) {
        kout[base + i] = key[b][i];
        vout[base + i] = r0 + idx[b][i];
    }
}

// One pass of a bottom-up merge sort inside every segment of nl keys: runs of w (the last
// one ragged) are merged pairwise.  An element's place is its index in its run plus the
// number of keys of the partner run that go before it (strictly smaller for the left run,
// smaller or equal for the right one), so equal keys keep their order and every place lies
// inside the pair of runs whatever the keys hold.
__global__ __launch_bounds__(256) void k_sort_pass(const double *kin, const int32_t *vin,
                                                   double *kout, int32_t *vout, int nl, int w,
                                                   int64_t total) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    const int64_t base = (e / nl) * nl;
    const int i = (int)(e - base);
    const int ps = (i / (2 * w)) * (2 * w);
    const int mid = min(ps + w, nl), end = min(ps + 2 * w, nl);
    const double v = kin[e];
    const int32_t idx = vin[e];
    int pos;
    if (mid >= end || !(kin[base + mid] < kin[base + mid - 1])) pos = i - ps;  // in order as they are
    else if (i < mid) pos = (i - ps) + count_less(kin + base + mid, end - mid, v);
    else pos = (i - mid) + count_leq(kin + base + ps, mid - ps, v);
    kout[base + ps + pos] = v;
    vout[base + ps + pos] = idx;
}

// ---------------------------------------------------------------------------------------
// update columns Z = P [W_c1 B_p / sqrt(beta_p) ; sqrt(beta_p) W_c2] and basis columns
// V = P [W_c1 R_c1 ; W_c2 R_c2] of every node of a level
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_assemble(AssembleArgs a) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= a.n) return;
    const int nl = a.nl, nc = nl / 2, r = a.r;
    const int64_t node = e / nl;
    const int64_t base = node * nl;
    const int pos = (int)(e - base);
    // the merge writes a permutation only when the children's spectra are sorted and free of
    // NaN (a failed child solve returns NaN): clamp, so that such a node stays in bounds and
    // only its status reports it
    const int src = min(max(a.perm[e], 0), nl - 1);
    const int child = src < nc ? 0 : 1;
    const int64_t hp = ((int64_t)1 << a.level) - 1 + node;                 // parent heap index
    const int64_t hc = ((int64_t)1 << (a.level + 1)) - 1 + 2 * node + child;  // child heap index
    double w[LEAF_RANK_MAX];
    for (int c = 0; c < r; ++c) w[c] = a.Wprev[(int64_t)c * a.n + base + src];
    const double beta = a.beta[hp];
    const double sb = sqrt(beta);
    const double *B = a.B + hp * r * r;
    for (int c2 = 0; c2 < r; ++c2) {
        double z;
        if (child == 0) {
            double acc = 0.0;
            for (int c = 0; c < r; ++c) acc = __builtin_fma(w[c], B[c * r + c2], acc);
            z = acc / sb;
        } else {
            z = sb * w[c2];
        }
        a.M[(int64_t)c2 * a.n + base + pos] = z;
    }
    if (a.with_basis) {
        const double *R = a.R + hc * r * r;
        for (int c2 = 0; c2 < r; ++c2) {
            double acc = 0.0;
            for (int c = 0; c < r; ++c) acc = __builtin_fma(w[c], R[c * r + c2], acc);
            a.M[(int64_t)(r + c2) * a.n + base + pos] = acc;
        }
    }
}

// ---------------------------------------------------------------------------------------
// applying the structured eigenmatrix: permutations of a level and the leaf products
// ---------------------------------------------------------------------------------------
// scatter (P^T): y[node rows perm[pos]] = x[pos];  gather (P): y[pos] = x[perm[pos]]
// (a thread takes a row through `cpt` columns: one to all of them left most of the chip idle,
// 8192 rows of 64 columns 17 -> 3 us)
__global__ __launch_bounds__(256) void k_permute(const int32_t *perm, int nl, int64_t n, int m,
                                                 const double *X, int64_t ldx, double *Y,
                                                 int64_t ldy, int scatter, int cpt) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    const int64_t base = (e / nl) * nl;
    const int64_t src = base + min(max(perm[e], 0), nl - 1);  // in bounds for any perm (k_assemble)
    const int c0 = blockIdx.y * cpt, c1 = min(m, c0 + cpt);
    if (scatter) copy_cols(X + e, ldx, Y + src, ldy, c0, c1);
    else copy_cols(X + src, ldx, Y + e, ldy, c0, c1);
}

// Y_leaf = Q_leaf X_leaf (trans 0) or Q_leaf^T X_leaf (trans 1), all leaves of the level: a
// thread's row of Q against LEAF_COLS columns of X, the columns beside one another in the
// grid.  Every element of Q is read once per LEAF_COLS columns (once per column, it came
// through L2 268 MB for 64 columns of 128 leaves of 64: 66 us, with this 21); the
// products of one entry are added in the same order, k ascending.
constexpr int LEAF_COLS = 8;
__global__ __launch_bounds__(WAVE) void k_leaf_apply(const double *Q, int L, int64_t n, int m,
                                                     int nrow, const double *X, int64_t ldx,
                                                     double *Y, int64_t ldy, int trans) {
    const int64_t row = (int64_t)(blockIdx.x % nrow) * WAVE + threadIdx.x;
    if (row >= n) return;
    const int64_t leafid = row / L;
    const int i = (int)(row % L), c0 = blockIdx.x / nrow * LEAF_COLS;
    const double *q = Q + leafid * L * L + (trans ? (int64_t)i * L : i);
    const int dq = trans ? 1 : L;
    const double *x = X + leafid * L;
    int64_t at[LEAF_COLS];  // past the last column: that one again, not stored
    double acc[LEAF_COLS];
#pragma unroll
    for (int c = 0; c < LEAF_COLS; ++c) {
        at[c] = (int64_t)min(c0 + c, m - 1) * ldx;
        acc[c] = 0.0;
    }
#pragma unroll 4
    for (int k = 0; k < L; ++k) {
        const double w = q[(int64_t)k * dq];
#pragma unroll
        for (int c = 0; c < LEAF_COLS; ++c) acc[c] = __builtin_fma(w, x[at[c] + k], acc[c]);
    }
#pragma unroll
    for (int c = 0; c < LEAF_COLS; ++c)
        if (c0 + c < m) Y[(int64_t)(c0 + c) * ldy + row] = acc[c];
}

__global__ void k_status_or(const int32_t *st, int cnt, int32_t *out) {
    int v = 0;
    for (int i = threadIdx.x; i < cnt; i += blockDim.x) v |= st[i];
    for (int o = WAVE / 2; o > 0; o >>= 1) v |= __shfl_xor(v, o);
    __shared__ int red[4];
    if (lane_id() == 0) red[threadIdx.x / WAVE] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0;
        for (int w = 0; w < (int)(blockDim.x / WAVE); ++w) t |= red[w];
        out[0] = t;
    }
}

__global__ void k_fill(double *x, int64_t n, double v) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n) x[e] = v;
}

static inline dim3 grid_for(int64_t n, int b = 256) { return dim3((unsigned)((n + b - 1) / b)); }

hipError_t launch_leaf_jacobi(const LeafArgs &a, hipStream_t s) {
    // the smallest LDS that holds the leaf, so that small leaves share a CU
    const dim3 nt(lj_threads(a.leaf));
    const bool res = a.leaf % LJ_TILE == 0 && a.leaf >= 3 * LJ_TILE;
#define SDC_LJ(LP)                                                                               \
    {                                                                                            \
        if (res) SDC_LAUNCH(KID_LEAF, (k_leaf_jacobi<LP, true>), dim3(a.nleaf), nt, 0, s, a);    \
        else SDC_LAUNCH(KID_LEAF, (k_leaf_jacobi<LP, false>), dim3(a.nleaf), nt, 0, s, a);       \
    }
    if (a.leaf <= 32) SDC_LJ(32)
    else if (a.leaf <= 64) SDC_LJ(64)
    else SDC_LJ(LEAF_MAX)
#undef SDC_LJ
    SDC_LAUNCH(KID_LEAF_VECTORS, k_leaf_vectors, dim3(a.nleaf * ((a.leaf + LV_WROWS - 1) / LV_WROWS)),
               dim3(WAVE), 0, s, a);
    SDC_LAUNCH(KID_LEAF_VECTORS, k_leaf_w, dim3(a.nleaf), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_merge(const double *lam_children, double *d_out, int32_t *perm, int nc,
                        int64_t n, hipStream_t s) {
    SDC_LAUNCH(KID_MERGE, k_merge, grid_for(n), dim3(256), 0, s, lam_children, d_out, perm, nc, n);
    return hipGetLastError();
}

hipError_t launch_seg_sort(const double *keys, int nl, int64_t n, double *kout, int32_t *vout,
                           double *kbuf, int32_t *vbuf, hipStream_t s) {
    // runs in LDS, then the passes that merge them; the last one writes the outputs
    const int nrun = (nl + SORT_RUN - 1) / SORT_RUN;
    int passes = 0;
    while ((SORT_RUN << passes) < nl) ++passes;
    double *ko = passes & 1 ? kbuf : kout;
    int32_t *vo = passes & 1 ? vbuf : vout;
    const int bs = std::min(1024, std::max(WAVE, (nl + 2 * WAVE - 1) / (2 * WAVE) * WAVE));
    SDC_LAUNCH(KID_SORT, k_sort_runs, dim3((unsigned)(n / nl * nrun)), dim3(bs), 0, s, keys, ko, vo,
               nl, nrun);
    for (int q = 0; q < passes; ++q) {
        const double *kin = ko;
        const int32_t *vin = vo;
        ko = ko == kout ? kbuf : kout;
        vo = vo == vout ? vbuf : vout;
        SDC_LAUNCH(KID_SORT, k_sort_pass, grid_for(n), dim3(256), 0, s, kin, vin, ko, vo, nl,
                   SORT_RUN << q, n);
    }
    return hipGetLastError();
}

hipError_t launch_assemble(const AssembleArgs &a, hipStream_t s) {
    SDC_LAUNCH(KID_ASSEMBLE, k_assemble, grid_for(a.n), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_permute(const int32_t *perm, int nl, int64_t n, int m, const double *X,
                          int64_t ldx, double *Y, int64_t ldy, int scatter, hipStream_t s) {
    const int cpt = cols_per_thread(n, m);
    SDC_LAUNCH(KID_PERMUTE, k_permute, row_grid(n, m, cpt), dim3(256), 0, s, perm, nl, n, m, X, ldx,
               Y, ldy, scatter, cpt);
    return hipGetLastError();
}

hipError_t launch_leaf_apply(const double *Q, int L, int64_t n, int m, const double *X,
                             int64_t ldx, double *Y, int64_t ldy, int trans, hipStream_t s) {
    const int nrow = (int)((n + WAVE - 1) / WAVE);
    SDC_LAUNCH(KID_LEAF_APPLY, k_leaf_apply, dim3((unsigned)nrow * ((m + LEAF_COLS - 1) / LEAF_COLS)),
               dim3(WAVE), 0, s, Q, L, n, m, nrow, X, ldx, Y, ldy, trans);
    return hipGetLastError();
}

hipError_t launch_status_or(const int32_t *st, int cnt, int32_t *out, hipStream_t s) {
    SDC_LAUNCH(KID_STATUS_OR, k_status_or, dim3(1), dim3(256), 0, s, st, cnt, out);
    return hipGetLastError();
}

hipError_t launch_fill(double *x, int64_t n, double v, hipStream_t s) {
    SDC_LAUNCH(KID_FILL, k_fill, grid_for(n), dim3(256), 0, s, x, n, v);
    return hipGetLastError();
}

}  // namespace sdc
