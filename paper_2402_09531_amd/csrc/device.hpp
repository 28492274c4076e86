// Device-side data of a tree and an operator, and the launchers of the HIP
// kernels that make up one matvec and the CG solver.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <utility>
#include <vector>

namespace dwfmm {

// Everything the kernels read about the geometry (device pointers).
struct DevTree {
    int n, d, J, dpad;
    int nleaf, ncl, leaf_first;   // leaf_first = 2^J - 1
    int max_leaf;                 // largest leaf size
    int min_far_level;            // J+1 when there is no farfield
    const double *Xs;             // [dpad][n] coordinates in tree order (rows k >= d are zero)
    const int32_t *perm;          // [n] tree position -> original index
    const int32_t *cbeg, *cend;   // [ncl]
    const int32_t *Fptr, *Fsrc;   // farfield CSR over clusters
    const int32_t *Nptr, *Nsrc;   // nearfield CSR over leaves (leaf-local indices)
    // Symmetric nearfield: every unordered leaf pair {t, s}, t != s, is owned by one of
    // its two leaves (balanced); the owner evaluates the block once and applies it both
    // ways.  own: CSR over owner leaves of partner leaves, block id = CSR position.
    // inc: CSR over partner leaves of the block ids whose column sums they receive.
    int nblk;                     // number of owned blocks of the symmetric nearfield (self blocks included)
    const int32_t *own_ptr, *own_src, *inc_ptr, *inc_blk;
    const double *center;         // [nleaf][dpad] leaf box midpoints (coordinate shift)
    // Order in which the symmetric nearfield launches take the owner leaves: workgroup q runs on
    // XCD q % 8, and XCD k gets the k-th of 8 contiguous leaf segments of equal nearfield work,
    // costliest leaf first; -1 pads the shorter segments.  NULL for trees without a symmetric nearfield.
    const int32_t *leaf_order;
    int n_order;
    // The same for the several-rhs nearfield, which sweeps each target leaf's whole nearfield list:
    // segments of equal list entries, costliest leaf first; near_order_seq has the same segments in
    // leaf order (the launches that read stored BF16 tiles, whose sources then stay in L2).
    // Leaves of more than 128 points are taken as ppl = ceil(max_leaf / 128) pieces each: an entry is
    // ppl * leaf + piece (ppl = 1 otherwise).
    int ppl;
    const int32_t *near_order;
    const int32_t *near_order_seq;
    int n_near_order;
};

struct DevOp {
    int kind;
    double ell;
    int nx, max_nrhs;
    const double *nodes;          // [ncl][nx][dpad] interpolation nodes of every box
    const double *E;              // [ncl][nx][nx] Lagrange transfer matrices (row a, column b)
    const double *Lb;             // [nx][n] Lagrange basis l_a(a_leaf^-1 x_i), tree order
    double *xt;                   // [n][max_nrhs] x in tree order
    __bf16 *xtb;                  // [n][nrhs] the same charges rounded to BF16 through FP32 (max_nrhs > 1)
    double *M, *L;                // [ncl][nx][max_nrhs] moments and locals
    int nxp;                      // nx rounded up to a multiple of 16
    const double *nodesT;         // [ncl][dk][nxp] nodes (shifted: node_shift), axis-major, zero padded (dk = d rounded up to 4)
    const double *nnorm;          // [ncl][nxp] their squared norms, zero padded
    double *rowbuf;               // [nleaf][128] owner-side nearfield row sums (one rhs)
    double *colbuf;               // [nblk][128] column sums of owned blocks (one rhs)
    // Gaussian only: every nearfield exponent |x - c|^2 / ell, |y - c|^2 / ell, 2 (x - c).(y - c) / ell
    // (c the owner leaf's midpoint) is at most 600 in magnitude, so the symmetric FP64 nearfield may
    // evaluate exp(-|x-y|^2/ell) = exp(-|x-c|^2/ell) exp(-|y-c|^2/ell) exp(2 (x-c).(y-c)/ell).
    int gauss_split;
    int gauss_split32;            // the same with every exponent within 80 (the FP32 nearfield)
    // Matern only: sqrt(3) max|x - y| / ell log2(e) <= 1000 over the nearfield (from the host's reach
    // bound), so the FP64 nearfield's 2^-s log2(e) needs no underflow clamp
    int matern_in_range;
    int exp_in_range;             // exponential only: the same for max|x - y| / ell log2(e)
    int gram_close;               // Matern: the same bound within 24 ell; Gaussian: its square within 300 ell (mrhs_near)
    // Power of two 2^-e with every centred nearfield coordinate (a point minus its target leaf's
    // midpoint) at most 1 in magnitude after scaling (e from the host's reach bound): the BF16
    // several-rhs nearfield forms its FP16 Gram operands from the scaled coordinates
    float hscale;
    // Tile cache of the BF16 several-rhs nearfield (NULL when off): column tile t of target leaf l
    // (16 stream columns x 8 row tiles of 16 targets, 64 lanes x 4 BF16 each, 4 KiB) sits at
    // near_tiles + (near_tile_off[l] + t) * 512; near_filled points at a host flag set once a
    // launch has written the tiles; near_cache_mode is chosen per launch (0 off, 1 compute and
    // write, 2 read).
    uint2 *near_tiles;
    const int64_t *near_tile_off;
    int *near_filled;
    int near_cache_mode;
};

// Optional HIP events recorded around the nearfield (P2P) and coupling (M2L)
// launches, on the stream they run on.
struct KernelTimer {
    hipEvent_t p2p_start = nullptr, p2p_stop = nullptr, m2l_start = nullptr, m2l_stop = nullptr;
};

// A second stream and two events with which the farfield (M2M, M2L, L2L) of a one-rhs matvec
// runs beside the symmetric nearfield: forked after P2M, joined before the combine.
struct StreamFork {
    hipStream_t side = nullptr;
    hipEvent_t forked = nullptr, joined = nullptr;
};

// One matvec (or parts of it) on `stream` (with `fork`, partly on its side stream; the result
// is ordered on `stream` as without it).  parts: bit0 nearfield, bit1 farfield.
hipError_t launch_matvec(const DevTree &T, const DevOp &O, const double *x, double *y, int nrhs, int parts,
                         int precision, hipStream_t stream, const KernelTimer *timer = nullptr,
                         const StreamFork *fork = nullptr);

// Evaluation at new points: y (targets, caller order) = K~(targets, sources) x (sources, caller
// order).  Tt/Ot: the target tree (cross farfield/nearfield lists naming source clusters and
// leaves) and the target side (box nodes, transfer matrices, basis at the targets, locals);
// Ts/Os: the source tree and operator, whose charge and moment workspace it uses.
hipError_t launch_eval(const DevTree &Tt, const DevOp &Ot, const DevTree &Ts, const DevOp &Os, const double *x,
                       double *y, int nrhs, hipStream_t stream);

// Parts of the two above that are compiled apart (kernels.hip).  launch_pieces: FP64 nearfield of
// targets T/O over sources Ts/xs (charges in source tree order) in pieces of at most 128 targets,
// any nrhs, with L2P if far; launch_m2l_wide: FP64 coupling of up to 128 nodes, any nrhs;
// launch_m2l_mrhs, launch_mrhs_lp: the several-rhs coupling (n_x <= 32) and the FP32/BF16
// several-rhs nearfield of the matvec.  Radial kernels, d <= 32.
hipError_t launch_pieces(const DevTree &T, const DevOp &O, const DevTree &Ts, const double *xs, double *y, int nrhs,
                         int near, int far, hipStream_t stream);
hipError_t launch_m2l_wide(const DevTree &T, const DevOp &Ot, const DevOp &Os, int first, int cnt, int nrhs,
                           hipStream_t stream);
hipError_t launch_m2l_mrhs(const DevTree &T, const DevOp &O, int first, int cnt, int nrhs, int precision,
                           hipStream_t stream);
hipError_t launch_mrhs_lp(const DevTree &T, const DevOp &O, double *y, int nrhs, int near, int far, int precision,
                          hipStream_t stream);

// Lagrange basis cache Lb from the boxes and the index set (setup).
hipError_t launch_basis(const DevTree &T, int nx, const double *clo, const double *csc, const double *coff,
                        const int32_t *lidx, int nnz_max, const double *Vinv, int nleg, const int32_t *leg_axis,
                        const int32_t *leg_deg, double *Lb, hipStream_t stream);

// ---- batches of independent problems (one rhs each) ----
struct BatchItem {
    DevTree T;
    DevOp O;
    int far;        // the problem has a farfield
    int precision;  // 0 FP64, 1/2 FP32 nearfield and coupling
    // levels of the M2M (up) and L2L groups by the level of their root, 0 where no group starts
    uint8_t up_depth[32], down_depth[32];
};

// M2M (up) and L2L passes: consecutive tree levels run by one launch, one workgroup per cluster of
// level `root`, each over the `depth` levels of its subtree (M2M: the deepest first).
struct XferGroup {
    int root, depth;
};
struct XferGroups {
    int n = 0;
    XferGroup g[32];  // a tree has at most 32 levels
    const XferGroup *begin() const { return g; }
    const XferGroup *end() const { return g + n; }
};
// The launches of M2M over levels hi, ..., lo (up) or L2L over levels lo, ..., hi, in order.  A
// launch costs about 5 us however little it does and a level inside one about 1 us, so levels are
// joined while a workgroup's subtree stays within 4000 cycles of products (1.7 us), or where the
// launch has 2048 workgroups (8 per CU) anyhow.  Cycles of one CU per cluster: one rhs about 24
// terms a cycle over its threads; several rhs 64 per FP64 MFMA on four SIMDs.
inline XferGroups xfer_groups(bool up, int nx, int nrhs, int lo, int hi)
{
    const int64_t src = up ? 2 : 1, nxt = (nx + 15) / 16, rb = (nrhs + 15) / 16;
    const int64_t cyc = nrhs == 1 ? std::max<int64_t>(1, src * nx * nx / 24) : src * nxt * rb * ((nx + 3) / 4) * 16;
    auto join = [&](int root, int depth) { return cyc * (((int64_t)1 << depth) - 1) <= 4000 || root >= 11; };
    XferGroups g;
    if (up) {
        for (int j = hi; j >= lo;) {
            int r = j;
            while (r > lo && join(r - 1, j - r + 2)) --r;
            g.g[g.n++] = {r, j - r + 1};
            j = r - 1;
        }
    } else {
        for (int j = lo; j <= hi;) {
            int depth = 1;
            while (j + depth <= hi && join(j, depth + 1)) ++depth;
            g.g[g.n++] = {j, depth};
            j += depth;
        }
    }
    return g;
}

// One launch of a templated kernel over a slice of the work list.  wpc (M2L only): waves per
// target cluster, 4, 2 or 1; every choice gives bitwise the same locals.
struct BatchLaunch {
    int kind, dk, nxt, prec, off, cnt;
    int wpc = 4;
    int grid = 0;  // M2L: 0 = one workgroup per 4 / wpc list entries; > 0 = a persistent grid of
                   // this many workgroups striding over the list
};
constexpr int kM2lPersistentGrid = 1024;  // 4 workgroups per CU on 256 CUs

// Work list entries are (item, local block); entries with item < 0 are padding.
struct BatchPlan {
    const BatchItem *items = nullptr;
    const double *const *xs = nullptr;
    double *const *ys = nullptr;
    const int2 *work = nullptr;
    int leaf_off = 0, leaf_cnt = 0;
    // (offset, count) per launch: entries (item, root cluster)
    std::vector<std::pair<int, int>> m2m, l2l;
    std::vector<BatchLaunch> m2l, p2p;
};

// With `fork`, the farfield stages run on its side stream beside the nearfield (same bits).
hipError_t launch_batch_matvec(const BatchPlan &P, hipStream_t stream, const StreamFork *fork = nullptr);
// Waves per cluster compiled for an M2L launch with nxt node tiles: 1 only up to two tiles
// (its per-lane accumulators grow with 4 / wpc x nxt).
inline bool m2l_wpc_available(int nxt, int wpc) { return wpc == 4 || wpc == 2 || (wpc == 1 && nxt <= 2); }
// One M2L launch of the plan on its own (the tile-shape tuner times these).
hipError_t launch_batch_m2l(const BatchPlan &P, const BatchLaunch &L, hipStream_t stream);

// ---- CG building blocks (FP64, deterministic fixed-order reductions) ----
// partial[b][c] for b < kDotBlocks (the grid grows with n nrhs up to that); out[c] = sum_b partial[b][c]
// by a fixed-order tree, so a result depends only on n, nrhs and the inputs.
constexpr int kDotBlocks = 1024;
hipError_t launch_dot(const double *a, const double *b, int n, int nrhs, double *partial, double *out,
                      hipStream_t stream);
// Several-rhs CG passes with the inner product that follows (in launch_dot's order):
// q += lambda p, out = p.q;  x += a p, r -= a q, out = r.r (a, out per column)
hipError_t launch_cg_cols_ridge(double *q, const double *p, double lambda, int n, int nrhs, double *partial, double *out,
                                hipStream_t stream);
hipError_t launch_cg_cols_step(double *x, double *r, const double *p, const double *q, const double *a, int n, int nrhs,
                               double *partial, double *out, hipStream_t stream);

// ---- FP64 CG for problems with one right-hand side, any number of them per launch ----
// One problem of a CG launch: CG on (K~ + lambda I) x = b, with A p (or A x) already in q when
// a step needs it.  The inner products of a problem are taken over nblk blocks of chunk rows
// (nblk = min(kDotBlocks, ceil(n / 4096)), the grid launch_dot uses for one column) and summed in
// the same fixed order as launch_dot, so a problem's iterates do not depend on what else the
// launch carries.  scal: [0] |r|^2, [1] |b|^2, [2] p.Ap, [3] new |r|^2, [4] step, [5] beta,
// [8] |out|^2 of the residual step; state: [0] 0 active, 1 converged, 2 breakdown, 3 frozen,
// [1] iterations, [2] steps with p.Ap < 0.
struct CgItem {
    double *x, *r, *p, *q;
    const double *b;
    // residual step: out = f - (out + lambda v) with K~ v already in out; add step: acc += x
    const double *f, *v;
    double *out, *acc;
    double *partial;          // [2][kDotBlocks]
    double *scal;
    int32_t *state;
    double lambda, rtol;
    int n, nblk, chunk, blk0;  // blk0: first block of the problem in the launch's block numbering
    int max_it;                // the problem takes no step once state[1] reaches max_it
    int frozen;                // start: the problem starts frozen; residual and add steps skip it
    int zero_x;                // start: x = 0 and q = 0 (= K~ 0) instead of reading them
    double *mirror;            // mirror step: state[0..2], scal[0], scal[1], scal[8], scal[9] (8 doubles)
};
enum CgStep {
    CG_START,      // blocks: q += lambda x, r = b - q, p = r; partial |r|^2 and |b|^2
    CG_START_SUM,  // problems: |r|^2, |b|^2, state (frozen or active), convergence check
    CG_PQ,         // blocks: q += lambda p, p.q; the last block: step a = |r|^2 / p.q (breakdown,
                   // negative curvature).  A problem of one block runs its whole iteration here.
    CG_XR,         // blocks: x += a p, r -= a q, |r|^2; the last block: beta, count, convergence check
    CG_P,          // blocks: p = r + beta p
    CG_RES,        // blocks: out = f - (out + lambda v); partial |out|^2
    CG_RES_SUM,    // problems: |out|^2 into scal[8]
    CG_ADD,        // blocks: acc += x
    CG_SUB,        // blocks: acc -= x
    CG_MIRROR      // problems: copy state and scalars to mirror, for one host read of many problems
};
inline int cg_blocks(int n) { return (int)std::max<int64_t>(1, std::min<int64_t>(kDotBlocks, ((int64_t)n + 4095) / 4096)); }
// One step for `nitems` problems (device array `items`, blk0 ascending, nblocks blocks in all),
// or, with items == nullptr, for the single problem `one` passed by value.
hipError_t launch_cg(int step, const CgItem *items, int nitems, int nblocks, const CgItem &one, hipStream_t stream);

// The vector steps of one iteration, after its matvec (A p in q): one launch if every problem has one
// block, else three.  They are latency: with a launch for each step's sums too (five), rows read one
// by one, an iteration of N = 4096 spent 25.5 us in these kernels, 11.6 us now.
hipError_t launch_cg_iteration(const CgItem *items, int nitems, int nblocks, const CgItem &one, hipStream_t stream);

}  // namespace dwfmm
