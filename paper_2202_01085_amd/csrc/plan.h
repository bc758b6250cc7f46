// The plan object: everything of Algorithm 1 that does not depend on b.
#pragma once
#include <memory>

#include "common.h"

struct f3m_level {
    int64_t nb = 0;                     // occupied boxes
    int64_t max_box = 0;
    f3m::DevBuf<uint32_t> key;          // [nb]   box key at this depth, ascending
    f3m::DevBuf<uint32_t> start;        // [nb+1] index interval into the box-ordered points
    f3m::DevBuf<uint32_t> parent;       // [nb]   rank of the parent one depth up
    f3m::DevBuf<uint32_t> cstart;       // [nb+1] rank interval of the children one depth down
    f3m::DevBuf<int32_t> cell;          // [nb*D] integer cell coordinates
    f3m::DevBuf<uint64_t> near_ptr, far_ptr;   // [nb+1]
    f3m::DevBuf<uint32_t> near_col, far_col;
    f3m::DevBuf<uint32_t> far_ord;      // [far_sz] the far rows in the order of the partners' row-major cell index (grouped M2L)
    int64_t near_sz = 0, far_sz = 0;
    int64_t far_point_pairs = 0;        // sum of |p||q| over the far pairs of this depth
    // small field (Sec. 4.2): pairs summed directly at this depth, and the target tiles of their rows
    f3m::DevBuf<uint64_t> small_ptr;    // [nb+1]
    f3m::DevBuf<uint32_t> small_col;
    int64_t small_sz = 0, small_point_pairs = 0;
    int64_t sm_ntiles = 0;
    f3m::DevBuf<uint32_t> sm_tile_box, sm_tile_first;
    // P2M work split: a chunk is a run of at most P2M_CHUNK points of one box
    int64_t nchunks = 0;
    int chunk = 256;                    // points of a chunk: P2M_CHUNK, or P2M_LONG where boxes are large
    f3m::DevBuf<uint32_t> chunk_box;    // [nchunks]
    f3m::DevBuf<uint32_t> chunk_first;  // [nb+1] first chunk of each box
    // boxes with very many chunks (few, huge boxes): a slice is a run of at most P2M_SLICE chunks of one
    // box, and the partial node weights are added slice by slice first
    int64_t nslices = 0;
    f3m::DevBuf<uint32_t> slice_box, slice_first;
    // D = 3, 4 nodes/dim, far ratio 2: the M2L enumerates the far partners on the candidate grid
    // around the parent (m2l.hip); far_ptr keeps the row lengths, far_col stays empty
    bool far_implicit = false;
    // ... and, without a small field, per box of the depth ABOVE: the rank of the candidate at each of the 216
    // positions of the grid around it and its child of each parity (~0: none)
    f3m::DevBuf<uint32_t> st_cand, st_child;
    // boxes with few points, more than three dimensions: the far field of the depth goes from point to point
    // (points.hip), by runs of targets of the boxes of the depth ABOVE; far_col stays empty
    bool far_points = false;
    f3m::DevBuf<float> fp_loc;                         // [n][8] local coordinates and child bits of every point
    int64_t fp_ntiles = 0;
    f3m::DevBuf<uint32_t> fp_tile_box, fp_tile_first;
    // Sec. 4.3: nodes per dimension used at this depth (interp_nodes, 3 under the adaptive rule, or 0 =
    // the far pairs of the depth are dropped), r = p^D, and whether every pair of the depth is interpolated
    int p = 0, r = 0;
    bool smooth = false;
    // 1-D factors of the node-to-node kernel matrix, [2*omax+1][p][p]
    struct { float *p = nullptr; } gtab;   // (part of the plan's tables)
    int gtab_omax = 0;
    // node weights / node potentials kept per depth when they are passed between depths
    f3m::DevBuf<float> Wl, Vl;          // [(nb + 1) * 64], [nb * 64]; at depth near_weighted the same again behind
                                        // them for the weighted near pairs
};

// Tables of the permutation in one, two or three passes between the caller's order and the box order of one point set
// (route.hip): per pass the place of every value in the LDS copy of its tile, per tile the first place of each
// digit and where the tile's run of each digit lies in the next order.
struct f3m_route {
    int64_t n = 0, ntiles = 0;
    int ipt = 32;           // values of a tile and of a window: 1024 ipt (two: 8, 20 or 28)
    bool two = false;       // two passes: tiles dealt to the windows directly (512 digits a tile)
    bool grouped = false;   // one pass: the points grouped by the boxes of one depth, in each of them in the caller's order
                            // (slot1, dstart1 and gofs1 of 512 digits a tile; tiles of the caller's order)
    int s2 = 0, B1 = 1, B2 = 1;
    f3m::DevBuf<uint16_t> slot1, slot2, off3;      // [n] each
    f3m::DevBuf<uint32_t> dstart1, dstart2;        // [ntiles][257]
    f3m::DevBuf<uint32_t> gofs1, gofs2;            // [ntiles][256]
};

// The partition of the source set Y of a two-set plan, v = K(X, Y) b (Sec. 3 states the method for
// two data matrices; Algorithm 1 keeps one treecode per set).  Both sets are divided by cubes of
// the same edge, each anchored at its own per-dimension minimum, so the two grids have equal box
// edges at every depth and are shifted against each other.  A one-set plan has no such object.
struct f3m_source {
    int64_t n = 0;
    float alpha[F3M_MAX_DIM] = {0};
    f3m::DevBuf<uint32_t> keys, perm;   // [n]
    f3m::DevBuf<float> Xs;              // [n*D] coordinates in box order, padded
    std::unique_ptr<f3m_route> route;   // large sets: the right-hand side comes into box order in streaming passes
    f3m_level lev[F3M_MAX_LEVELS + 1];  // box tables and P2M work splits only (no lists)
};

struct f3m_plan_s {
    int64_t n = 0;                              // targets (rows of X); also the sources of a one-set plan
    int D = 0, p = 0, r = 0;
    int Lq = 0, L = 0, T = 4;
    float gamma = 1.f, theta = 2.f;
    float E = 0.f, scale = 0.f;
    float alpha[F3M_MAX_DIM] = {0};
    int leaf_max = 128, max_depth = 0, force_all_near = 0, no_overlap = 0;
    float eta_smooth = 0.f;                     // smooth-field limit of Sec. 4.3 (0 = off)
    int adaptive_far = 0;                       // adaptive far-field node rule of Sec. 4.3
    int64_t rho = 0;                            // small-field limit of Sec. 4.2 (0 = off)
    int smooth_depth = -1;                      // depth whose adjacent pairs are interpolated, or -1
    hipStream_t side = nullptr;                 // second stream for the near field
    hipEvent_t ev_fork = nullptr, ev_join = nullptr, ev_p2p0 = nullptr, ev_p2p1 = nullptr;
    int device = 0;
    int64_t bytes = 0;
    int64_t near_point_pairs = 0;

    f3m::DevBuf<uint32_t> keys;   // [n] keys at depth Lq, box order
    f3m::DevBuf<uint32_t> perm;   // [n]
    // "Box order" of the products is that of perm, except where the points are only grouped by the boxes of depth
    // last_depth() (route->grouped): the boxes of that depth and above have the same intervals in both.
    f3m::DevBuf<float> Xs;        // [n*D] coordinates in box order, row-major
    f3m::DevBuf<float> bs, ys;    // [n] right-hand side / far-field result in box order
    f3m::DevBuf<float> yn;        // [n] near-field result in box order
    f3m::DevBuf<float> multi_bs, multi_yn;   // [4][ns + pad], [4][n]: a group of right-hand sides in box order and its
                                             // near-field results (f3m_kmvm_multi; allocated on first use)
    f3m::DevBuf<float> p2p_part;  // [slices][n] partial near-field sums when target tiles are split (few targets)
    f3m::DevBuf<float> W, V;      // [max_l nb_l * r] node weights / node potentials of one depth
    f3m::DevBuf<float> Wpart;     // [max_l nchunks_l * r] partial node weights
    f3m::DevBuf<double> Wslice;   // [max_l nslices_l * r] sums of the partial node weights of a slice
    // near-field work split: a tile is a run of at most 64 targets of one leaf box (the full runs of 64, and the
    // last run if it is not an overflow tile)
    int64_t ntiles = 0;
    f3m::DevBuf<uint32_t> tile_box, tile_first;   // [ntiles], [nb_L+1]
    // ... and overflow tiles: a last run of a leaf box with so few targets (<= 10, <= 8 above 4-D) that the
    // kernel with the sources on the lanes is cheaper; at most one per box
    int64_t notiles = 0;
    f3m::DevBuf<uint32_t> otile_box, otile_first;
    // ... and pairs of tiles (D = 3, Gram near field, one point set): the first runs of two leaf boxes a, a + 1 with
    // the same parent and cells next to each other are worked by one wavefront, which shares the preparation of
    // the sources near both.  pair_box[i] = a; paired[b] != 0 for both boxes of a pair; rtile_* is the tile list
    // without the first runs of paired boxes (tile_* keeps every run: the products with several right-hand sides
    // and the split near field use it).
    int64_t npairs = 0, nrtiles = 0;
    f3m::DevBuf<uint32_t> pair_box, pair_first;
    f3m::DevBuf<uint8_t> paired;
    f3m::DevBuf<uint32_t> rtile_box, rtile_first;
    f3m_level lev[F3M_MAX_LEVELS + 1];          // boxes of X (targets); lists by target box
    std::unique_ptr<f3m_source> src;            // two-set plan: the partition of Y (sources)
    // the source side of either kind of plan
    const f3m_level &slev(int l) const { return src ? src->lev[l] : lev[l]; }
    f3m_level &slev(int l) { return src ? src->lev[l] : lev[l]; }
    int64_t ns() const { return src ? src->n : n; }
    const float *Ys() const { return src ? src->Xs.p : Xs.p; }
    const uint32_t *sperm() const { return src ? src->perm.p : perm.p; }
    const float *salpha() const { return src ? src->alpha : alpha; }
    // grid shift of a depth in units of its box edge, u_d = ((alpha^Y_d - alpha^X_d) / E) 2^depth: the
    // centre of source cell c' minus the centre of target cell c is ((c' - c) + u) box edges
    void grid_shift(int level, double *u) const {
        for (int d = 0; d < D; ++d) {
            const double diff = (double)salpha()[d] - (double)alpha[d];
            const double q = (src && E > 0.f) ? diff / (double)E : 0.0;
            u[d] = q * (double)(1ull << level);
        }
    }
    int near_depth = 0;                 // > 0: the products work down to this depth only, whose adjacent pairs are
                                        // interpolated too, to within fp32 rounding (near_interp_error)
    int near_weighted = 0;              // > 0: the products end at this depth, whose near pairs are interpolated between
                                        // weighted points, to within fp32 rounding (near_weighted_error)
    bool exact_near() const { return near_depth == 0 && near_weighted == 0; }
    int last_depth() const { return near_depth ? near_depth : near_weighted ? near_weighted : L; }   // of the products
    struct { float *p = nullptr; } near_tab;   // factors of the weighted near pairs: 16 (near_factor_index), or for two sets
                                               // [D][offsets][p][p] like gtab
    f3m_level near_src;                        // two sets: the sources' boxes of depth near_weighted that occur in a near row
                                               // (nb, chunk and slice lists), and their weighted node weights (Wl)
    int tree_lmin = 0, tree_lmax = 0;   // tree_lmin > 0: node weights/potentials are passed between depths
                                        // tree_lmin..tree_lmax (D = 3, 4 nodes/dim); other depths work
                                        // straight from the points
    struct { float *p = nullptr; } transfer;   // [2][4][4] parent basis at the child's nodes
    f3m::DevBuf<float> tables;          // gtab of every depth, near_tab and transfer
    // large n: both permutations of a product run as streaming passes (route.hip); the two work
    // vectors hold max(n, sources) floats each
    int64_t route_min_n = 0;                    // three passes (one: grouped) are used from this many points on
    bool route_given = false;                   // the caller named that number: below it no two passes either
    std::unique_ptr<f3m_route> route;           // of the targets (and of the sources of a one-set plan)
    f3m::DevBuf<float> route_a, route_b;
    const f3m_route *sroute() const { return src ? src->route.get() : route.get(); }

    hipEvent_t ev[16] = {nullptr};
    std::vector<hipEvent_t> plan_events;  // two per depth while the plan is built
    std::vector<float> host_tabs;       // the tables on their way to the device, until the plan is complete
    // Times of a product: an event at every boundary between its stages, in order (marks); the others name them.
    // far_events: 6 per depth, around the far-field kernels of that depth.  t_wait0 .. t_wait1 (if not null): a wait for
    // the near field inside the downward pass of depth tree_lmax.
    std::vector<hipEvent_t> marks, far_events;
    hipEvent_t t_begin = nullptr, t_in = nullptr, t_p2p0 = nullptr, t_p2p1 = nullptr, t_out = nullptr, t_end = nullptr,
               t_wait0 = nullptr, t_wait1 = nullptr;
    bool have_plan_times = false, have_kmvm_times = false, have_far_point_pairs = false;
    f3m_times times = {};
    ~f3m_plan_s();
};

namespace f3m {

constexpr int P2M_CHUNK = 256;
constexpr int P2M_LONG = 2048;   // points of a chunk where boxes hold thousands (3-D, 4 nodes per dimension)
constexpr int P2M_SLICE = 512;   // chunks per slice of the two-stage sum of partial node weights
// largest last run of a leaf box that is treated as an overflow tile (near field with the sources on the lanes):
// beyond about 10 targets a half-filled 64-wide tile is the cheaper of the two (measured at n = 1e9)
constexpr int overflow_targets(int D) { return D <= 4 ? 10 : 8; }
constexpr int PAD_POINTS = 64;   // zero padding behind Xs and bs
constexpr int MAX_NODES = 4096;

int quant_depth(int D);
bool smooth_rule(double E, int depth, int D, double gamma, double eta_smooth);   // Sec. 4.3 smoothness criterion
int adaptive_nodes(double E, int depth, double gamma, int p);                   // Sec. 4.3 node rule (0: dropped)

double near_interp_error(double E, int depth, double gamma);                    // D = 3, 4 nodes per dimension
double near_weighted_error(double E, int depth, double gamma, double reach = 1.0);
void product_depths(int L, int64_t leaf_boxes, bool leaf_far, bool leaf_near, bool two_sets, bool may_group, int weighted,
                    int *near_depth, int *near_weighted, bool *grouped);

// plan.hip
void build_plan(f3m_plan_s &P, const float *X, const float *Y, hipStream_t st);   // Y == nullptr: one set (P.src set otherwise)
void compute_far_point_pairs(f3m_plan_s &P);   // near_point_pairs and lev[].far_point_pairs, once (synchronises)
// route.hip: permutations of large vectors as streaming passes with tables built once per plan
bool route_two_passes(int64_t n);   // sizes below those of the three passes for which two pay
void route_build(f3m_route &R, const uint32_t *perm, int64_t n, bool two, int64_t *tally, hipStream_t st);
// points are grouped by the boxes of a depth of at most this (3-D): its tables have a place for every cell, occupied or not
constexpr int ROUTE_GROUP_DEPTH = 3, ROUTE_GROUP_BOXES = 1 << (3 * ROUTE_GROUP_DEPTH);
void route_group_build(f3m_route &R, const uint32_t *keys, int64_t n, int Lq, int depth, const uint32_t *box_keys, int64_t nb,
                       int64_t *tally, hipStream_t st);
void route_scatter(const f3m_route &R, const float *in, const float *in2, float *out, float *tmp_a, float *tmp_b,
                   hipStream_t st);                                   // out[perm[k]] = in[k] (+ in2[k])
void route_gather(const f3m_route &R, const float *in, float *out, float *tmp_a, float *tmp_b, hipStream_t st);
                                                                      // out[k] = in[perm[k]]
void route_gather_rows3(const f3m_route &R, const float *in, float *out, float *tmp, hipStream_t st);
                                                                      // rows of 3 floats; tmp: 3 n floats
void materialize_far(const f3m_plan_s &P, int level, uint32_t *cols_dev, hipStream_t st);   // far rows of an implicit depth
// kmvm.hip
// box_order: b and y are already in the plan's box order, b with PAD_POINTS zeros behind it (one-set plans only; used by
// the solver)
void run_kmvm(f3m_plan_s &P, const float *b, float *y, hipStream_t st, bool box_order = false);
void run_kmvm_multi(f3m_plan_s &P, const float *B, int64_t ldb, float *Y, int64_t ldy, int m, hipStream_t st);
int p2p_nsplit(const f3m_plan_s &P, int l, int64_t ntiles);   // source slices per target tile of the near field (1: none)
bool p2p_pairs_allowed(const f3m_plan_s &P);                  // the near field of the last depth may work tiles in pairs
void run_zero(float *y, int64_t n, hipStream_t st);   // y = 0 with a fill kernel
// exact sums of targets X (nx rows) against sources Y (ny rows, weights b); X == Y for one set
void run_direct(const float *X, int64_t nx, const float *Y, int64_t ny, int D, float gamma, const float *b, float *y,
                hipStream_t st);
void run_direct_rows_f64(const float *X, const float *Y, int64_t ny, int D, float gamma, const float *b,
                         const int64_t *rows, int64_t m, double *y64, hipStream_t st);
// the same with the partial sums in a static device array: no allocation, no wait (m <= 16384)
void run_direct_rows_f64_static(const float *X, int64_t n, int D, float gamma, const float *b, const int64_t *rows,
                                int64_t m, double *y64, hipStream_t st);
void upload_tables(f3m_plan_s &P, hipStream_t st);              // kernel factors of every far depth, parent basis at child nodes
void build_far_orders(f3m_plan_s &P, hipStream_t st);           // far rows in row-major cell order for the grouped M2L
// solve.hip: conjugate gradients for (K + lambda I) x = b on a one-set plan (synchronises)
void run_cg(f3m_plan_s &P, float lambda, const float *b, float *x, int max_iter, float tol, int *iters_host,
            float *history_host, hipStream_t st);
// points.hip: the far field of a depth between points
constexpr int FP_TT = 16;                                                        // targets of a workgroup
bool far_points_allowed(const f3m_plan_s &P, int level);
bool far_points_pays(const f3m_plan_s &P, int level, int64_t point_pairs);       // point pairs of the near boxes one depth up
void far_points_prepare(f3m_plan_s &P, int level, hipStream_t st);
void run_far_points(f3m_plan_s &P, int level, const float *bs, float *ys, int omin, int no, hipStream_t st);
// m2l.hip
bool m2l_stencil_applies(const f3m_plan_s &P);   // D = 3, 4 nodes per dimension, far ratio 2
void build_stencil_tables(f3m_plan_s &P, int level, hipStream_t st);   // after the lists of the depth exist
bool stencil_tables_alloc(f3m_plan_s &P, int level, hipStream_t st);   // false: the depth has no such tables
// The basis of 4 nodes is evaluated with the weights 2/3 and 4/3 rounded to fp32, both 3e-8 too large, so a product of P2M and L2P is
// 1.8e-7 too large in 3-D whatever the points.  This is what takes it out of a factor of one dimension: the interpolated near pairs
// replace exact sums, which have no such bias.
inline double basis_scale() {
    const double w = 1.5 * (double)(1.f / 1.5f);
    return 1.0 / (w * w);
}
void near_table(const f3m_plan_s &P, float *t);                        // 16 factors of the weighted near pairs
void run_near_weighted(f3m_plan_s &P, const float *W, float *V, hipStream_t st);
bool m2l_stencil_small(const f3m_plan_s &P, int level);                // few parents: several depths may share a launch
void run_m2l_small(f3m_plan_s &P, int from, int to, hipStream_t st);
bool run_m2l_stencil(f3m_plan_s &P, int level, const float *W, float *V, hipStream_t st, bool zero_row = false);  // false: does not apply

}  // namespace f3m
