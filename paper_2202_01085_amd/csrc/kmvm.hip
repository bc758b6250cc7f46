// f3m_kmvm and direct_kmvm: the floating-point passes.
// (arXiv 2202.01085: Sec. 3 eq. (1) near field; Sec. 3 "Interpolating k(x,y)" and Fig. 4
//  for the three far-field passes v1 = L_Y b, v2 = K v1, v = L_X^T v2; Appendix E
//  Algorithm 1 for the order of the passes.)
#include <algorithm>
#include <cmath>

#include <mutex>
#include <type_traits>

#include "plan.h"

// Partial sums of direct_kmvm_rows_f64_static, for callers that may not allocate: up to 256 source
// slices of up to 16384 rows (32 MiB, held on every device the library runs on until the process
// ends).  Host code never uses this name as an address: it asks for the array's address on the
// current device once per device (rows_static_scratch) and passes that pointer to the kernels.
constexpr int ROWS_MAX_SLICES = 256;
constexpr int64_t ROWS_STATIC_MAX_M = 16384;
static __device__ __align__(256) double scratch[(size_t)ROWS_MAX_SLICES * (size_t)ROWS_STATIC_MAX_M];

namespace f3m {

// address of `scratch` on the current device (every device holds its own copy at its own address)
static double *rows_static_scratch() {
    constexpr int MAX_DEVICES = 64;
    static std::mutex mu;
    static double *ptr[MAX_DEVICES] = {};
    int dev = 0;
    F3M_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= MAX_DEVICES) fail(F3M_ERR_UNSUPPORTED, "device ordinal above 63");
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[dev]) {
        double *q = nullptr;
        F3M_HIP(hipGetSymbolAddress((void **)&q, HIP_SYMBOL(scratch)));
        if (!q) fail(F3M_ERR_HIP, "hipGetSymbolAddress gave a null address for the static scratch");
        ptr[dev] = q;
    }
    return ptr[dev];
}

constexpr int P_MAX = 8;  // interpolation nodes per dimension supported by the kernels

// Chebyshev nodes of the second kind s_i = cos(i pi/(p-1)) and the reciprocal denominators
// of the product-form Lagrange basis (Sec. 3 "Lagrange interpolation").
struct NodeArg {
    float s[P_MAX];
    float invden[P_MAX];
};
struct CentreArg {
    double alpha[F3M_MAX_DIM];
    double edge;      // l = E / 2^level
    double inv_half;  // 2 / l
};

// 2-D launch shape for `count` blocks: the runtime limits grid.x * block.x to 32 bits, so
// large block counts are folded over y; kernels recover the index with block_index().
static dim3 grid_for(int64_t count) {
    const int64_t gx = 1 << 16;
    if (count <= gx) return dim3((unsigned)(count > 0 ? count : 1), 1, 1);
    return dim3((unsigned)gx, (unsigned)cdiv(count, gx), 1);
}
__device__ inline int64_t block_index() { return (int64_t)blockIdx.y * gridDim.x + blockIdx.x; }

static NodeArg make_nodes(int p) {
    NodeArg a{};
    double s[P_MAX];
    for (int i = 0; i < p; ++i) s[i] = std::cos((double)i * M_PI / (double)(p - 1));
    for (int i = 0; i < p; ++i) {
        double den = 1.0;
        for (int j = 0; j < p; ++j)
            if (j != i) den *= s[i] - s[j];
        a.s[i] = (float)s[i];
        a.invden[i] = (float)(1.0 / den);
    }
    return a;
}

// box centres of a depth: of the target grid, or of the source grid (its own anchor in a two-set plan)
static CentreArg make_centre(const f3m_plan_s &P, int level, bool source = false) {
    CentreArg c{};
    for (int d = 0; d < P.D; ++d) c.alpha[d] = (double)(source ? P.salpha()[d] : P.alpha[d]);
    c.edge = (double)P.E / std::ldexp(1.0, level);
    c.inv_half = 2.0 / c.edge;
    return c;
}

// ------------------------------------------------------------------------------------
// permutation in and out (the reindexing vector sigma of Sec. 4.2)
// ------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void gather_kernel(const float *__restrict__ b, const uint32_t *__restrict__ perm,
                                                     int64_t n, float *__restrict__ bs) {
    int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k < n) bs[k] = b[perm[k]];
}
// y = far-field part + near-field part (if there is one), back in the caller's order
__global__ __launch_bounds__(256) void scatter_kernel(const float *__restrict__ ys, const float *__restrict__ yn,
                                                      const uint32_t *__restrict__ perm, int64_t n,
                                                      float *__restrict__ y) {
    int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k < n) y[perm[k]] = yn ? ys[k] + yn[k] : ys[k];
}
// the last step for a caller that keeps its vectors in box order (the solver)
__global__ __launch_bounds__(256) void add_kernel(const float *__restrict__ ys, const float *__restrict__ yn, int64_t n,
                                                  float *__restrict__ y) {
    int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k < n) y[k] = yn ? ys[k] + yn[k] : ys[k];
}
__global__ __launch_bounds__(256) void zero_kernel(float *__restrict__ p, int64_t n) {
    int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k < n) p[k] = 0.f;
}

// ------------------------------------------------------------------------------------
// near field (Sec. 3 eq. (1)): one wavefront per run of <= 64 targets of a leaf box, one
// lane per target; the sources of the near boxes are wave-uniform, so they arrive through
// the scalar data path and every vector instruction works on 64 distinct pairs.
//   k(x,y) = exp2( nc2 * |x-y|^2 ),  nc2 = -log2(e) / (2 gamma^2)
// All near-field kernels take the targets as (Xt, startT) and the sources as (Xs, bs, start): the
// box-ordered points and point intervals of the target boxes and of the source boxes.  For one
// point set both are the same arrays; for K(X, Y) the columns of a list are ranks of boxes of Y.
// ------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(64) void p2p_kernel(const float *__restrict__ Xt, const uint32_t *__restrict__ startT,
                                                 const float *__restrict__ Xs, const float *__restrict__ bs,
                                                 const uint32_t *__restrict__ start,
                                                 const uint64_t *__restrict__ near_ptr,
                                                 const uint32_t *__restrict__ near_col,
                                                 const uint32_t *__restrict__ tile_box,
                                                 const uint32_t *__restrict__ tile_first, int64_t ntiles,
                                                 float nc2, float *__restrict__ ys, int accumulate) {
    const int64_t t = block_index();
    if (t >= ntiles) return;
    const uint32_t a = tile_box[t];
    const uint32_t k0 = startT[a] + (uint32_t)(t - tile_first[a]) * 64u;
    const uint32_t kend = startT[a + 1];
    const uint32_t k = k0 + threadIdx.x;
    const bool active = k < kend;
    float xi[D];
#pragma unroll
    for (int d = 0; d < D; ++d) xi[d] = active ? Xt[(int64_t)k * D + d] : 0.f;
    double acc = 0.0;   // the runs are added in fp64 (one addition per 32 sources)
    const uint64_t e1 = near_ptr[a + 1];
    for (uint64_t e = near_ptr[a]; e < e1; ++e) {
        const uint32_t q = near_col[e];
        const uint32_t j1 = start[q + 1];
        // runs of 32 sources are summed on their own and then added in fp64: a long row of terms of
        // mixed sign loses fewer bits than with one running fp32 sum
        for (uint32_t j0 = start[q]; j0 < j1; j0 += 32) {
            const uint32_t je = min(j0 + 32u, j1);
            float run = 0.f;
#pragma unroll 4
            for (uint32_t j = j0; j < je; ++j) {
                float r2 = 0.f;
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    float diff = Xs[(int64_t)j * D + d] - xi[d];
                    r2 = fmaf(diff, diff, r2);
                }
                run = fmaf(__builtin_amdgcn_exp2f(r2 * nc2), bs[j], run);
            }
            acc += (double)run;
        }
    }
    if (active) ys[k] = accumulate ? ys[k] + (float)acc : (float)acc;
}

// ------------------------------------------------------------------------------------
// near field with the Gram matrix on the matrix cores.  In box units, relative to the centre
// of the target box (u = (x - centre)/l for a target, w = (y - centre)/l for a source) and with
// g = log2(e) l^2 / (2 gamma^2):
//   k(x,y) = exp2(-g|u|^2) * exp2( 2g u.w - g|w|^2 ).
// The second exponent for 32 sources x 32 targets is a dense contraction with inner
// dimension D+1: source vector (2g w_1..2g w_D, -g|w|^2), target vector (u_1..u_D, 1).  Each
// component is split into two fp16 numbers (hi = fp16(v), lo = fp16(v - hi): 22 significant
// bits) and the products hi*hi + hi*lo + lo*hi are laid side by side along the inner
// dimension, so one v_mfma_f32_32x32x16_f16 (fp32 accumulation, 8 passes) does the work of
// (D+2)/2 fp32 MFMAs of 16 passes each: 3(D+1) <= 16 terms for D <= 4, two instructions above.
// The dropped lo*lo term and the split are a perturbation of the coordinates by 2^-22 of a box
// edge.  exp2 and one FMA per pair stay on the vector ALU; exp2(-g|u|^2) is applied once per
// target.  A wavefront handles a run of <= 64 targets of one leaf box as two column blocks of
// 32; after the MFMA lane (n,h) holds the 16 sources 8(v/4)+4h+(v%4) of target column n, and
// the two halves are added with one shuffle at the end.
// Sources are cut from runs of rank-consecutive near boxes (contiguous points); rows beyond a
// run get zero coordinates and a norm term of -60000, so that their kernel value is
// exp2(-huge) = 0 whatever right-hand side is read for them.
// Used only while g is small (the caller checks it): the expanded square loses
// (|u|^2+|w|^2) g times the rounding unit in the exponent.
// ------------------------------------------------------------------------------------
typedef float f16v __attribute__((ext_vector_type(16)));
typedef _Float16 h8v __attribute__((ext_vector_type(8)));
struct __attribute__((packed, aligned(4))) float4u { float v[4]; };

// hi/lo fp16 split of NC components and the MFMA operand of one instruction:
//   term t of the inner dimension (t = 16 q + 8 h + e): kind = t / NC, component = t % NC
//   source side: (hi, hi, lo)[kind],  target side: (hi, lo, hi)[kind],  zero beyond 3 NC terms
template <int NC, bool SOURCE>
__device__ inline h8v split_operand(const float (&v)[NC], int q, int h) {
    _Float16 hi[NC], lo[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        hi[i] = (_Float16)v[i];
        lo[i] = (_Float16)(v[i] - (float)hi[i]);
    }
    h8v r;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        _Float16 val[2];
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
            const int t = 16 * q + 8 * hh + e;
            const int kind = t / NC, comp = t % NC;
            const bool use_lo = SOURCE ? kind == 2 : kind == 1;
            val[hh] = kind >= 3 ? (_Float16)0.f : (use_lo ? lo[comp] : hi[comp]);
        }
        r[e] = h ? val[1] : val[0];
    }
    return r;
}

typedef float f2v __attribute__((ext_vector_type(2)));
typedef _Float16 h2v __attribute__((ext_vector_type(2)));
typedef uint32_t u4v __attribute__((ext_vector_type(4)));

__device__ inline uint32_t pack_f16(float a, float b) {
    const h2v h = __builtin_convertvector((f2v){a, b}, h2v);
    return __builtin_bit_cast(uint32_t, h);
}
__device__ inline f2v unpack_f16(uint32_t v) { return __builtin_convertvector(__builtin_bit_cast(h2v, v), f2v); }

// source operand for four components (D = 3): the same layout as split_operand<4, true>,
// built from packed pairs.  Lane half 0 holds (hi, hi), lane half 1 (lo, 0).
__device__ inline h8v split_source4(const float (&w)[4], int h) {
    const uint32_t hi01 = pack_f16(w[0], w[1]), hi23 = pack_f16(w[2], w[3]);
    const f2v b01 = unpack_f16(hi01), b23 = unpack_f16(hi23);
    const uint32_t lo01 = pack_f16(w[0] - b01.x, w[1] - b01.y), lo23 = pack_f16(w[2] - b23.x, w[3] - b23.y);
    u4v r;
    r.x = h ? lo01 : hi01;
    r.y = h ? lo23 : hi23;
    r.z = h ? 0u : hi01;
    r.w = h ? 0u : hi23;
    return __builtin_bit_cast(h8v, r);
}

// target operand for four components (D = 3): the same layout as split_operand<4, false>, built
// from packed pairs.  Lane half 0 holds (hi, lo), lane half 1 (hi, 0).
__device__ inline h8v split_target4(const float (&u)[4], int h) {
    const uint32_t hi01 = pack_f16(u[0], u[1]), hi23 = pack_f16(u[2], u[3]);
    const f2v b01 = unpack_f16(hi01), b23 = unpack_f16(hi23);
    const uint32_t lo01 = pack_f16(u[0] - b01.x, u[1] - b01.y), lo23 = pack_f16(u[2] - b23.x, u[3] - b23.y);
    u4v r;
    r.x = hi01;
    r.y = hi23;
    r.z = h ? 0u : lo01;
    r.w = h ? 0u : lo23;
    return __builtin_bit_cast(h8v, r);
}

template <int D>
__global__ __launch_bounds__(256) void p2p_mfma_kernel(const float *__restrict__ Xt,
                                                       const uint32_t *__restrict__ startT,
                                                       const float *__restrict__ Xs, const float *__restrict__ bs,
                                                       const uint32_t *__restrict__ start,
                                                       const int32_t *__restrict__ cell,
                                                       const uint64_t *__restrict__ near_ptr,
                                                       const uint32_t *__restrict__ near_col,
                                                       const uint32_t *__restrict__ tile_box,
                                                       const uint32_t *__restrict__ tile_first, int64_t ntiles,
                                                       float g, float inv_l, CentreArg C, float *__restrict__ ys,
                                                       int accumulate) {
    constexpr int NC = D + 1;
    constexpr int NQ = (3 * NC + 15) / 16;   // MFMA instructions per 32 x 32 block
    const int lane = threadIdx.x & 63;
    const int64_t t = block_index() * 4 + (threadIdx.x >> 6);
    if (t >= ntiles) return;
    const uint32_t a = __builtin_amdgcn_readfirstlane(tile_box[t]);
    const uint32_t k0 = startT[a] + (uint32_t)(t - tile_first[a]) * 64u;
    const uint32_t kend = startT[a + 1];
    const bool two = __builtin_amdgcn_readfirstlane((int)(kend - k0)) > 32;
    const int nn = lane & 31, kk = lane >> 5;
    float ctr[D];
#pragma unroll
    for (int d = 0; d < D; ++d) ctr[d] = (float)(C.alpha[d] + ((double)cell[(int64_t)a * D + d] + 0.5) * C.edge);

    // B operands: the targets of the two column blocks
    h8v Bop[2][NQ];
    float ni[2];
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
        const uint32_t kt = k0 + cb * 32 + nn;
        // unconditional loads (in bounds: Xs is padded by 64 points), masked by a factor so
        // that they are issued together and not one by one under a branch
        const float valid = kt < kend ? 1.f : 0.f;
        float u[NC];
        float s = 0.f;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            u[d] = (Xt[(int64_t)kt * D + d] - ctr[d]) * inv_l * valid;
            s = fmaf(u[d], u[d], s);
        }
        u[D] = 1.f;
        ni[cb] = -g * s;
#pragma unroll
        for (int q = 0; q < NQ; ++q) Bop[cb][q] = split_operand<NC, false>(u, q, kk);
    }
    float acc0 = 0.f, acc1 = 0.f;
    const float g2l = 2.f * g * inv_l;
    const float nrm = -0.25f / g;

    // the blocks of 32 sources: near boxes with consecutive ranks are one contiguous run of
    // points, and blocks are cut from runs, not from single boxes, which wastes fewer rows.
    // (jb, je) is a block start and the end of its run; e walks the near list.
    uint64_t e = near_ptr[a];
    const uint64_t e1 = near_ptr[a + 1];
    auto next_run = [&](uint32_t &jb, uint32_t &je) {
        uint32_t q = near_col[e];
        jb = start[q];
        ++e;
        while (e < e1 && near_col[e] == q + 1) { ++q; ++e; }
        je = start[q + 1];
    };
    // the loads of a block: one source row per lane (both halves the same) and the right-hand
    // sides of the 16 sources this lane sees after the MFMA.  Always in bounds (64 points of
    // padding behind Xs and bs); rows at or beyond je are masked in block().
    auto load = [&](uint32_t jb, float (&x)[D], float4u (&bq)[4]) {
        const uint32_t j = jb + nn;
#pragma unroll
        for (int d = 0; d < D; ++d) x[d] = Xs[(int64_t)j * D + d];
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) bq[q4] = *reinterpret_cast<const float4u *>(bs + jb + 8 * q4 + 4 * kk);
    };
    auto block = [&](uint32_t jb, uint32_t je, const float (&x)[D], const float4u (&bq)[4]) {
        const bool live = jb + nn < je;
        float w[NC];
        float s = 0.f;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            w[d] = (x[d] - ctr[d]) * (live ? g2l : 0.f);     // 2 g w_d
            s = fmaf(w[d], w[d], s);
        }
        w[D] = live ? s * nrm : -60000.f;              // -g |w|^2
        h8v Aop[NQ];
        if constexpr (NC == 4) {
            Aop[0] = split_source4(w, kk);
        } else {
#pragma unroll
            for (int qq = 0; qq < NQ; ++qq) Aop[qq] = split_operand<NC, true>(w, qq, kk);
        }
        f16v c0 = {0.f};
#pragma unroll
        for (int qq = 0; qq < NQ; ++qq) c0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(Aop[qq], Bop[0][qq], c0, 0, 0, 0);
        if (two) {
            f16v c1 = {0.f};
#pragma unroll
            for (int qq = 0; qq < NQ; ++qq) c1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(Aop[qq], Bop[1][qq], c1, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 16; ++v) acc0 = fmaf(__builtin_amdgcn_exp2f(c0[v]), bq[v >> 2].v[v & 3], acc0);
#pragma unroll
            for (int v = 0; v < 16; ++v) acc1 = fmaf(__builtin_amdgcn_exp2f(c1[v]), bq[v >> 2].v[v & 3], acc1);
        } else {
#pragma unroll
            for (int v = 0; v < 16; ++v) acc0 = fmaf(__builtin_amdgcn_exp2f(c0[v]), bq[v >> 2].v[v & 3], acc0);
        }
    };
    // A row can be empty (with the small field or the smooth field the box's own pair may be
    // handled elsewhere): nothing to add, and next_run must not read past the row.
    if (e == e1) {
        const uint32_t kt = k0 + kk * 32 + nn;
        if (kt < kend) ys[kt] = accumulate ? ys[kt] : 0.f;
        return;
    }
    // two register sets in turn: the loads of the next block are in flight while the current
    // one is worked on.
    float xa[D], xb[D];
    float4u ba[4], bb[4];
    uint32_t jba, jea, jbb, jeb;
    next_run(jba, jea);
    load(jba, xa, ba);
    for (;;) {
        jbb = jba + 32;
        jeb = jea;
        bool more = true;
        if (jbb >= jea) {
            if (e < e1) next_run(jbb, jeb);
            else more = false;
        }
        load(more ? jbb : jba, xb, bb);     // unconditional: a fixed number of loads in flight
        block(jba, jea, xa, ba);
        if (!more) break;
        jba = jbb + 32;
        jea = jeb;
        if (jba >= jeb) {
            if (e < e1) next_run(jba, jea);
            else more = false;
        }
        load(more ? jba : jbb, xa, ba);
        block(jbb, jeb, xb, bb);
        if (!more) break;
    }
    acc0 += __shfl_xor(acc0, 32, 64);
    acc1 += __shfl_xor(acc1, 32, 64);
    const float res = kk ? __builtin_amdgcn_exp2f(ni[1]) * acc1 : __builtin_amdgcn_exp2f(ni[0]) * acc0;
    const uint32_t kt = k0 + kk * 32 + nn;
    if (kt < kend) ys[kt] = accumulate ? ys[kt] + res : res;
}

// The near-field kernel for D = 3.  The sources of a target tile are the points of its near
// boxes, taken as ONE dense sequence: lane r of the wavefront holds (first point, length,
// running offsets) of near box r, and the source at sequence position p is found from that
// table with wave-uniform lane reads, so steps of 64 sources are full except the last one.
// Source operands are prepared for 64 sources at a time: lane l loads the source at position
// w0 + l, splits its four components (2g w_x, 2g w_y, 2g w_z, -g|w|^2) into packed fp16 pairs
// hi01, hi23, lo01, lo23, and one v_permlane32_swap per pair turns (hi, lo) into the operand
// registers of two blocks of 32 sources at once:
//   swap(hi, lo): hi' = [hi of sources 0-31 | lo of sources 0-31]   -> block A, both lane halves
//                 lo' = [hi of sources 32-63 | lo of sources 32-63] -> block B
// Inner dimension of the MFMA (k = 8 half + e): source side half 0 = (hi, hi), half 1 = (lo, lo);
// target side half 0 = (hi, lo), half 1 = (hi, 0): hi*hi + hi*lo + lo*hi, the fourth product
// meets a zero.  The right-hand sides of a step pass through 64 floats of LDS per wavefront
// (written by the lane that owns the source, read as the 16 values a lane needs per block).
// SPLIT: a problem with few target tiles and long rows (few targets against many sources) gives
// every tile to `nsplit` wavefronts; wavefront s of a tile takes the s-th slice (a multiple of 64
// positions) of the source sequence of every round and writes its sums to part[s][target]; they
// are added in ascending s by p2p_split_sum_kernel.
// MB > 1: MB right-hand sides at once (MA.bs[j] -> MA.ys[j]); the exponents and the exponentials of a
// block are formed once and every right-hand side adds its own 16 multiply-adds per lane, so the
// dominant cost of the near field is shared by the columns.
struct MultiArg {
    const float *bs[4];
    float *ys[4];
};

template <bool SPLIT, int MB>
__global__ __launch_bounds__(256) void p2p_gram3_kernel(const float *__restrict__ Xt,
                                                        const uint32_t *__restrict__ startT,
                                                        const float *__restrict__ Xs, const float *__restrict__ bs,
                                                        const uint32_t *__restrict__ start,
                                                        const int32_t *__restrict__ cell,
                                                        const uint64_t *__restrict__ near_ptr,
                                                        const uint32_t *__restrict__ near_col,
                                                        const uint32_t *__restrict__ tile_box,
                                                        const uint32_t *__restrict__ tile_first, int64_t ntiles,
                                                        float g, float inv_l, CentreArg C, float *__restrict__ ys,
                                                        int accumulate, int nsplit, int64_t ntargets,
                                                        float *__restrict__ part, MultiArg MA,
                                                        const uint8_t *__restrict__ paired) {
    constexpr int D = 3, NC = 4;
    static_assert(MB >= 1 && MB <= 4 && !(SPLIT && MB > 1), "unsupported variant");
    __shared__ __attribute__((aligned(16))) float bbuf[4][MB * 64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int64_t t = block_index() * 4 + wv;
    int slice = 0;
    if constexpr (SPLIT) {
        if (t >= ntiles * nsplit) return;
        const int64_t tile = t / nsplit;
        slice = (int)(t - tile * nsplit);
        t = tile;
    } else {
        if (t >= ntiles) return;
    }
    const uint32_t a = __builtin_amdgcn_readfirstlane(tile_box[t]);
    // paired (or null): boxes whose first run of targets is worked by p2p_gram3_pair_kernel; the tile list
    // then starts at their second run
    const uint32_t k0 = startT[a] + ((uint32_t)(t - tile_first[a]) + (paired && paired[a] ? 1u : 0u)) * 64u;
    const uint32_t kend = startT[a + 1];
    const int ntg = __builtin_amdgcn_readfirstlane((int)(kend - k0));   // targets of the tile (wave-uniform)
    const int nn = lane & 31, kk = lane >> 5;
    float ctr[D];
#pragma unroll
    for (int d = 0; d < D; ++d) ctr[d] = (float)(C.alpha[d] + ((double)cell[(int64_t)a * D + d] + 0.5) * C.edge);

    // B operands: the targets of the two column blocks
    h8v Bop[2];
    float ni[2];
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
        const uint32_t kt = k0 + cb * 32 + nn;
        const float valid = kt < kend ? 1.f : 0.f;   // loads are in bounds (padding), masked by a factor
        float u[NC];
        float s = 0.f;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            u[d] = (Xt[(int64_t)kt * D + d] - ctr[d]) * inv_l * valid;
            s = fmaf(u[d], u[d], s);
        }
        u[D] = 1.f;
        ni[cb] = -g * s;
        Bop[cb] = split_target4(u, kk);
    }
    float acc0 = 0.f, acc1 = 0.f;
    float accm0[MB], accm1[MB];   // MB > 1: one pair of accumulators per right-hand side
#pragma unroll
    for (int j = 0; j < MB; ++j) accm0[j] = accm1[j] = 0.f;
    const float g2l = 2.f * g * inv_l;
    const float nrm = -0.25f / g;
    float *bw = bbuf[wv];

    // operands of the two blocks of 32 sources of a step.  A lane whose position lies behind the
    // sequence holds the last source again (a near point like the others: finite exponent) and
    // its right-hand side is zero.
    auto prepare = [&](const float (&x)[D], h8v &opA, h8v &opB) {
        float w[NC];
        float s = 0.f;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            w[d] = (x[d] - ctr[d]) * g2l;                    // 2 g w_d
            s = fmaf(w[d], w[d], s);
        }
        w[D] = s * nrm;                                      // -g |w|^2
        const uint32_t hi01 = pack_f16(w[0], w[1]), hi23 = pack_f16(w[2], w[3]);
        const f2v b01 = unpack_f16(hi01), b23 = unpack_f16(hi23);
        const uint32_t lo01 = pack_f16(w[0] - b01.x, w[1] - b01.y), lo23 = pack_f16(w[2] - b23.x, w[3] - b23.y);
        const auto s01 = __builtin_amdgcn_permlane32_swap(hi01, lo01, false, false);
        const auto s23 = __builtin_amdgcn_permlane32_swap(hi23, lo23, false, false);
        u4v ra, rb;
        ra.x = s01[0]; ra.y = s23[0]; ra.z = s01[0]; ra.w = s23[0];
        rb.x = s01[1]; rb.y = s23[1]; rb.z = s01[1]; rb.w = s23[1];
        opA = __builtin_bit_cast(h8v, ra);
        opB = __builtin_bit_cast(h8v, rb);
    };
    // one block of 32 sources against the tile; bq = right-hand sides at bw[first .. first + 31].
    // (The two column blocks are summed in differently shaped code on purpose: identical
    // sequences get merged by the compiler into one that addresses the accumulators through
    // scratch memory.)
    auto block = [&](const h8v &op, int first) {
        if constexpr (MB > 1) {
            // the exponentials once, then 16 multiply-adds per right-hand side and column block
            f16v e0 = {0.f}, e1 = {0.f};
            e0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(op, Bop[0], e0, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 16; ++v) e0[v] = __builtin_amdgcn_exp2f(e0[v]);
            if (ntg > 32) {
                e1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(op, Bop[1], e1, 0, 0, 0);
#pragma unroll
                for (int v = 0; v < 16; ++v) e1[v] = __builtin_amdgcn_exp2f(e1[v]);
            }
#pragma unroll
            for (int j = 0; j < MB; ++j) {
                float4 bq[4];
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4)
                    bq[q4] = *reinterpret_cast<const float4 *>(bw + j * 64 + first + 8 * q4 + 4 * kk);
                const float *bf = reinterpret_cast<const float *>(bq);
#pragma unroll
                for (int v = 0; v < 16; ++v) accm0[j] = fmaf(e0[v], bf[v], accm0[j]);
                if (ntg > 32) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) accm1[j] = fmaf(e1[v], bf[v], accm1[j]);
                }
            }
            return;
        }
        float4 bq[4];
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) bq[q4] = *reinterpret_cast<const float4 *>(bw + first + 8 * q4 + 4 * kk);
        const float *bf = reinterpret_cast<const float *>(bq);
        f16v c0 = {0.f};
        c0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(op, Bop[0], c0, 0, 0, 0);
        // the test is made on a scalar register at each use: kept as a lane mask across the loop it
        // costs two vector instructions per step
        int nt2 = ntg;
        asm volatile("" : "+s"(nt2));
        if (nt2 > 32) {
            f16v c1 = {0.f};
            c1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(op, Bop[1], c1, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 16; ++v) acc0 = fmaf(__builtin_amdgcn_exp2f(c0[v]), bf[v], acc0);
#pragma unroll
            for (int v = 15; v >= 0; --v) acc1 = fmaf(__builtin_amdgcn_exp2f(c1[v]), bf[v], acc1);
        } else {
#pragma unroll
            for (int v = 0; v < 16; ++v) acc0 = fmaf(__builtin_amdgcn_exp2f(c0[v]), bf[v], acc0);
        }
    };

    const uint64_t e0 = near_ptr[a], e1 = near_ptr[a + 1];
    for (uint64_t er = e0; er < e1; er += 64) {   // rounds of up to 64 near boxes (one round with far ratio 2)
        const int m = (int)(e1 - er < 64 ? e1 - er : 64);
        uint32_t sfirst = 0, slen = 0;
        if (lane < m) {
            const uint32_t q = near_col[er + lane];
            sfirst = start[q];
            slen = start[q + 1] - sfirst;
        }
        const uint32_t cend = wave_incl_scan_u32(slen);   // inclusive running sum of the lengths over the lanes
        const uint32_t cbeg = cend - slen;
        const uint32_t delta = sfirst - cbeg;   // position -> source index inside this lane's box (mod 2^32)
        uint32_t S = __builtin_amdgcn_readlane(cend, 63);   // sources of this round
        uint32_t wbeg = 0;                                   // this wavefront's positions: [wbeg, S)
        if constexpr (SPLIT) {
            const uint32_t per = ((S + (uint32_t)nsplit - 1) / (uint32_t)nsplit + 63u) & ~63u;
            const uint64_t lo = (uint64_t)slice * per;
            wbeg = lo < S ? (uint32_t)lo : S;
            S = (uint64_t)wbeg + per < S ? wbeg + per : S;
            // wave-uniform, but derived from the wavefront's number: kept in scalar registers by force
            wbeg = __builtin_amdgcn_readfirstlane(wbeg);
            S = __builtin_amdgcn_readfirstlane(S);
        }
        if (wbeg >= S) continue;
        int r = 0;   // first near box that reaches into the current window (wave-uniform)
        // Source index of position w0 + lane; positions from S on take the last source of the
        // sequence, so every index is in bounds.  Box r holds w0 (cbeg <= w0 < cend), so it is the
        // box of every position until a later box begins at or before the position; a box without
        // points is overridden by its successor, which begins at the same position.
        auto locate = [&](uint32_t w0) {
            const uint32_t p = min(w0 + (uint32_t)lane, S - 1u);
            while ((uint32_t)__builtin_amdgcn_readlane(cend, r) <= w0) ++r;   // ends: w0 < S <= cend of lane 63
            uint32_t src = p + (uint32_t)__builtin_amdgcn_readlane(delta, r);
            for (int rr = r + 1; rr < m; ++rr) {
                const uint32_t c0 = __builtin_amdgcn_readlane(cbeg, rr);
                if (c0 >= w0 + 64) break;
                const uint32_t dl = __builtin_amdgcn_readlane(delta, rr);
                src = p >= c0 ? p + dl : src;
            }
            return src;
        };
        // Two register sets take turns as "current" and "next" step (no copies at the end of a step): the loads
        // of the next step are in flight during the current one; the last step loads its own sources again,
        // so the number of loads in flight is fixed.
        auto fetch = [&](uint32_t w0, float (&x)[D], float &b1, float (&bm)[MB]) __attribute__((always_inline)) {
            const uint32_t src = locate(w0);
#pragma unroll
            for (int d = 0; d < D; ++d) x[d] = Xs[(int64_t)src * D + d];
            if constexpr (MB > 1) {
#pragma unroll
                for (int j = 0; j < MB; ++j) bm[j] = MA.bs[j][src];
            } else {
                b1 = bs[src];
            }
        };
        auto step = [&](uint32_t w0, const float (&xc)[D], float bc, float (&bcm)[MB], float (&xnext)[D], float &bnext,
                        float (&bnextm)[MB]) __attribute__((always_inline)) {
            fetch(w0 + 64 < S ? w0 + 64 : w0, xnext, bnext, bnextm);
            if (w0 + 64 > S) {   // last step only: the positions behind the sequence get weight zero
                asm volatile("");   // keeps this a branch: as selects it costs every step three instructions
                const bool live = w0 + lane < S;
                bc = live ? bc : 0.f;
#pragma unroll
                for (int j = 0; j < MB; ++j) bcm[j] = live ? bcm[j] : 0.f;
            }
            __builtin_amdgcn_wave_barrier();
            if constexpr (MB > 1) {
#pragma unroll
                for (int j = 0; j < MB; ++j) bw[j * 64 + lane] = bcm[j];
            } else {
                bw[lane] = bc;
            }
            __builtin_amdgcn_wave_barrier();   // LDS operations of a wavefront complete in order
            h8v opA, opB;
            prepare(xc, opA, opB);
            block(opA, 0);
            if (w0 + 32 < S) block(opB, 32);
        };
        float xa[D], xb[D], ba = 0.f, bb = 0.f;
        float bam[MB], bbm[MB];
#pragma unroll
        for (int j = 0; j < MB; ++j) bam[j] = bbm[j] = 0.f;
        fetch(wbeg, xa, ba, bam);
        for (uint32_t w0 = wbeg;;) {
            step(w0, xa, ba, bam, xb, bb, bbm);
            w0 += 64;
            if (w0 >= S) break;
            step(w0, xb, bb, bbm, xa, ba, bam);
            w0 += 64;
            if (w0 >= S) break;
        }
    }
    if constexpr (MB > 1) {
        const uint32_t kt = k0 + kk * 32 + nn;
        const float scale = __builtin_amdgcn_exp2f(kk ? ni[1] : ni[0]);
#pragma unroll
        for (int j = 0; j < MB; ++j) {
            const float a0 = accm0[j] + __shfl_xor(accm0[j], 32, 64), a1 = accm1[j] + __shfl_xor(accm1[j], 32, 64);
            if (kt < kend) MA.ys[j][kt] = scale * (kk ? a1 : a0);
        }
        return;
    }
    acc0 += __shfl_xor(acc0, 32, 64);
    acc1 += __shfl_xor(acc1, 32, 64);
    const float res = kk ? __builtin_amdgcn_exp2f(ni[1]) * acc1 : __builtin_amdgcn_exp2f(ni[0]) * acc0;
    const uint32_t kt = k0 + kk * 32 + nn;
    if constexpr (SPLIT) {
        if (kt < kend) part[(int64_t)slice * ntargets + kt] = res;
    } else {
        if (kt < kend) ys[kt] = accumulate ? ys[kt] + res : res;
    }
}

// The 3-D Gram near field for PAIRS of target tiles.  Two leaf boxes a and a + 1 with the same parent and
// cells next to each other share most of their near boxes (18 of 27 with far ratio 2), and the cost of a step
// of p2p_gram3_kernel that is not exponentials and multiply-adds (finding and loading 64 sources, preparing
// their operands) does not depend on the number of target columns.  One wavefront takes the first run of
// targets of both boxes: coordinates are relative to the midpoint of the two box centres, and the source
// sequence is cut in three segments,
//   [ boxes near both | boxes near a only | boxes near a + 1 only ],
// each walked like the sequence of p2p_gram3_kernel; the first segment is worked against all column blocks.
// The segments come from the two near rows (at most 32 entries each: lanes 0-31 hold the row of a, lanes 32-63
// that of a + 1): an entry of a's row is also near a + 1 iff its squared cell offset from a + 1 is below the
// far threshold T (the integer rule that built the rows), and the copies in the row of a + 1 are dropped.
// Within a segment boxes keep their list order.
__global__ __launch_bounds__(256) void p2p_gram3_pair_kernel(const float *__restrict__ Xs,
                                                             const uint32_t *__restrict__ start,
                                                             const float *__restrict__ bs,
                                                             const int32_t *__restrict__ cell,
                                                             const uint64_t *__restrict__ near_ptr,
                                                             const uint32_t *__restrict__ near_col,
                                                             const uint32_t *__restrict__ pair_box, int64_t npairs,
                                                             int T, float g, float inv_l, CentreArg C,
                                                             float *__restrict__ ys) {
    constexpr int D = 3, NC = 4;
    __shared__ __attribute__((aligned(16))) float bbuf[4][64];
    __shared__ uint32_t tab_first[4][64], tab_len[4][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t t = block_index() * 4 + wv;
    if (t >= npairs) return;
    const uint32_t a = __builtin_amdgcn_readfirstlane(pair_box[t]);   // the pair is (a, a + 1)
    const int nn = lane & 31, kk = lane >> 5;
    int32_t ca[D], eo[D];   // cell of a, and the cell of a + 1 relative to it
    float ctr[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        ca[d] = cell[(int64_t)a * D + d];
        eo[d] = cell[(int64_t)(a + 1) * D + d] - ca[d];
        ctr[d] = (float)(C.alpha[d] + ((double)ca[d] + 0.5 + 0.5 * (double)eo[d]) * C.edge);
    }
    const uint32_t kA = start[a], kB = start[a + 1], kBe = start[a + 2];
    const int ntA = __builtin_amdgcn_readfirstlane((int)min(kB - kA, 64u));    // targets of the two tiles
    const int ntB = __builtin_amdgcn_readfirstlane((int)min(kBe - kB, 64u));

    // Column blocks of 32 targets: those of a, then those of a + 1, at most four.  Where both tiles end in a partly
    // filled block and one block less holds all targets (in memory they follow each other), they are packed: block
    // `mixed` then holds targets of both, and in a segment of sources near one box only, the sums of the other's lanes
    // are put back.  At n = 1e7 (38 targets a box) that is 3 blocks instead of 4 for the sources near both: 2.80 -> 2.63 ms
    // for the product.
    const int cA = (ntA + 31) >> 5, cB = (ntB + 31) >> 5, packed_blocks = (ntA + ntB + 31) >> 5;
    const bool packed = packed_blocks < cA + cB;   // then ntA is no multiple of 32, so box a ends with its tile
    const int nblocks = packed ? packed_blocks : cA + cB;
    const int firstB = packed ? cA - 1 : cA;       // first block with targets of a + 1
    // the target of a lane of a block, and whether there is one
    auto target = [&](int cb, uint32_t &kt) {
        const bool of_a = packed || cb < cA;
        const int idx = 32 * (of_a ? cb : cb - cA) + nn;
        const bool valid = idx < (packed ? ntA + ntB : of_a ? ntA : ntB);
        kt = valid ? (of_a ? kA : kB) + (uint32_t)idx : kA;
        return valid;
    };
    h8v Bop[4];
    float ni[4];
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
        uint32_t kt;
        const float valid = target(cb, kt) ? 1.f : 0.f;
        float u[NC];
        float s = 0.f;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            u[d] = (Xs[(int64_t)kt * D + d] - ctr[d]) * inv_l * valid;
            s = fmaf(u[d], u[d], s);
        }
        u[D] = 1.f;
        ni[cb] = -g * s;
        Bop[cb] = split_target4(u, kk);
    }

    // the table of the source boxes: lane = position in [both | a only | a + 1 only]
    int nboth, nonly_a, m;
    uint32_t sfirst, slen;
    {
        const bool of_a = lane < 32;
        const uint64_t e0 = near_ptr[a], e1 = near_ptr[a + 1], e2 = near_ptr[a + 2];
        const int len = (int)(of_a ? e1 - e0 : e2 - e1);
        const bool have = (lane & 31) < len;
        const uint32_t q = have ? near_col[(of_a ? e0 : e1) + (uint64_t)(lane & 31)] : a;
        int d2 = 0;   // squared cell offset of q from the OTHER box of the pair
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int o = cell[(int64_t)q * D + d] - ca[d] - (of_a ? eo[d] : 0);
            d2 += o * o;
        }
        const bool other = d2 < T;
        const bool is_both = have && of_a && other, is_a = have && of_a && !other, is_b = have && !of_a && !other;
        const uint64_t mboth = __ballot(is_both), ma = __ballot(is_a), mb = __ballot(is_b);
        const uint64_t below = (1ull << lane) - 1ull;
        nboth = __popcll(mboth);
        nonly_a = __popcll(ma);
        m = nboth + nonly_a + __popcll(mb);
        const int slot = is_both ? __popcll(mboth & below)
                       : is_a    ? nboth + __popcll(ma & below)
                                 : nboth + nonly_a + __popcll(mb & below);
        const uint32_t f = start[q], l = start[q + 1] - f;
        tab_first[wv][lane] = 0u;
        tab_len[wv][lane] = 0u;
        __builtin_amdgcn_wave_barrier();   // LDS operations of a wavefront complete in order
        if (is_both || is_a || is_b) {
            tab_first[wv][slot] = f;
            tab_len[wv][slot] = l;
        }
        __builtin_amdgcn_wave_barrier();
        sfirst = tab_first[wv][lane];
        slen = tab_len[wv][lane];
    }
    const uint32_t cend = wave_incl_scan_u32(slen);   // inclusive running sum of the lengths over the lanes
    const uint32_t cbeg = cend - slen;
    const uint32_t delta = sfirst - cbeg;   // position -> source index inside this lane's box (mod 2^32)
    const uint32_t S1 = nboth > 0 ? (uint32_t)__builtin_amdgcn_readlane(cend, nboth - 1) : 0u;
    const uint32_t S2 = nboth + nonly_a > 0 ? (uint32_t)__builtin_amdgcn_readlane(cend, nboth + nonly_a - 1) : 0u;
    const uint32_t S3 = __builtin_amdgcn_readlane(cend, 63);

    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    const float g2l = 2.f * g * inv_l;
    const float nrm = -0.25f / g;
    float *bw = bbuf[wv];
    int r = 0;   // first box of the table that reaches into the current window (wave-uniform, only grows)

    // operands of the two blocks of 32 sources of a step, as in p2p_gram3_kernel
    auto prepare = [&](const float (&x)[D], h8v &opA, h8v &opB) __attribute__((always_inline)) {
        float w[NC];
        float s = 0.f;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            w[d] = (x[d] - ctr[d]) * g2l;                    // 2 g w_d
            s = fmaf(w[d], w[d], s);
        }
        w[D] = s * nrm;                                      // -g |w|^2
        const uint32_t hi01 = pack_f16(w[0], w[1]), hi23 = pack_f16(w[2], w[3]);
        const f2v b01 = unpack_f16(hi01), b23 = unpack_f16(hi23);
        const uint32_t lo01 = pack_f16(w[0] - b01.x, w[1] - b01.y), lo23 = pack_f16(w[2] - b23.x, w[3] - b23.y);
        const auto s01 = __builtin_amdgcn_permlane32_swap(hi01, lo01, false, false);
        const auto s23 = __builtin_amdgcn_permlane32_swap(hi23, lo23, false, false);
        u4v ra, rb;
        ra.x = s01[0]; ra.y = s23[0]; ra.z = s01[0]; ra.w = s23[0];
        rb.x = s01[1]; rb.y = s23[1]; rb.z = s01[1]; rb.w = s23[1];
        opA = __builtin_bit_cast(h8v, ra);
        opB = __builtin_bit_cast(h8v, rb);
    };
    // one block of 32 sources against one or two column blocks (nt: 32 a block)
    auto columns = [&](const h8v &op, const float *bf, const h8v &B0, const h8v &B1, int nt, float &acc0,
                       float &acc1) __attribute__((always_inline)) {
        f16v c0 = {0.f};
        c0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(op, B0, c0, 0, 0, 0);
        int nt2 = nt;
        asm volatile("" : "+s"(nt2));   // the test on a scalar register at each use, not on a kept lane mask
        if (nt2 > 32) {
            f16v c1 = {0.f};
            c1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(op, B1, c1, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 16; ++v) acc0 = fmaf(__builtin_amdgcn_exp2f(c0[v]), bf[v], acc0);
#pragma unroll
            for (int v = 15; v >= 0; --v) acc1 = fmaf(__builtin_amdgcn_exp2f(c1[v]), bf[v], acc1);
        } else {
#pragma unroll
            for (int v = 0; v < 16; ++v) acc0 = fmaf(__builtin_amdgcn_exp2f(c0[v]), bf[v], acc0);
        }
    };
    // the positions [wbeg, S) of the sequence against nt0 / 32 of two column blocks, and nt1 / 32 of two more (`all`)
    auto segment = [&](uint32_t wbeg, uint32_t S, auto all, const h8v &B0, const h8v &B1, int nt0, float &acc0,
                       float &acc1, int nt1) __attribute__((always_inline)) {
        constexpr bool ALL = decltype(all)::value;
        if (wbeg >= S) return;
        // source index of position w0 + lane, as in p2p_gram3_kernel; positions from S on take the last source
        // of the segment (w0 < S <= cend of lane 63 ends the search)
        auto locate = [&](uint32_t w0) __attribute__((always_inline)) {
            const uint32_t p = min(w0 + (uint32_t)lane, S - 1u);
            while ((uint32_t)__builtin_amdgcn_readlane(cend, r) <= w0) ++r;
            uint32_t src = p + (uint32_t)__builtin_amdgcn_readlane(delta, r);
            for (int rr = r + 1; rr < m; ++rr) {
                const uint32_t c0 = __builtin_amdgcn_readlane(cbeg, rr);
                if (c0 >= w0 + 64) break;
                const uint32_t dl = __builtin_amdgcn_readlane(delta, rr);
                src = p >= c0 ? p + dl : src;
            }
            return src;
        };
        // two register sets take turns as current and next step, as in p2p_gram3_kernel
        auto fetch = [&](uint32_t w0, float (&x)[D], float &b1) __attribute__((always_inline)) {
            const uint32_t src = locate(w0);
#pragma unroll
            for (int d = 0; d < D; ++d) x[d] = Xs[(int64_t)src * D + d];
            b1 = bs[src];
        };
        auto step = [&](uint32_t w0, const float (&xc)[D], float bc, float (&xnext)[D], float &bnext)
                        __attribute__((always_inline)) {
            fetch(w0 + 64 < S ? w0 + 64 : w0, xnext, bnext);
            if (w0 + 64 > S) {   // last step only: the positions behind the segment get weight zero
                asm volatile("");
                bc = w0 + lane < S ? bc : 0.f;
            }
            __builtin_amdgcn_wave_barrier();
            bw[lane] = bc;
            __builtin_amdgcn_wave_barrier();   // LDS operations of a wavefront complete in order
            h8v opA, opB;
            prepare(xc, opA, opB);
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                if (half == 1 && w0 + 32 >= S) break;
                float4 bq[4];
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4)
                    bq[q4] = *reinterpret_cast<const float4 *>(bw + 32 * half + 8 * q4 + 4 * kk);
                const float *bf = reinterpret_cast<const float *>(bq);
                const h8v &op = half ? opB : opA;
                columns(op, bf, B0, B1, nt0, acc0, acc1);
                if constexpr (ALL) {
                    int nt2 = nt1;
                    asm volatile("" : "+s"(nt2));   // a scalar test, as in columns
                    if (nt2 > 0) columns(op, bf, Bop[2], Bop[3], nt1, acc[2], acc[3]);
                }
            }
        };
        float xa[D], xb[D], ba, bb;
        fetch(wbeg, xa, ba);
        for (uint32_t w0 = wbeg;;) {
            step(w0, xa, ba, xb, bb);
            w0 += 64;
            if (w0 >= S) break;
            step(w0, xb, bb, xa, ba);
            w0 += 64;
            if (w0 >= S) break;
        }
    };
    segment(0u, S1, std::true_type{}, Bop[0], Bop[1], 32 * min(nblocks, 2), acc[0], acc[1], 32 * (nblocks - 2));
    {
        // near a only: blocks 0 .. cA - 1; in the last one only the lanes with a target of a
        const float old0 = acc[0], old1 = acc[1];
        segment(S1, S2, std::false_type{}, Bop[0], Bop[1], 32 * cA, acc[0], acc[1], 0);
        const bool of_a = 32 * (cA - 1) + nn < ntA;
        if (cA == 1) acc[0] = of_a ? acc[0] : old0;
        else acc[1] = of_a ? acc[1] : old1;
    }
    {
        // near a + 1 only: blocks firstB .., at most two; a packed first one only in the lanes with a target of a + 1
        float s0 = firstB == 0 ? acc[0] : firstB == 1 ? acc[1] : acc[2];
        float s1 = firstB == 0 ? acc[1] : firstB == 1 ? acc[2] : acc[3];
        const float old0 = s0;
        const h8v B0 = firstB == 0 ? Bop[0] : firstB == 1 ? Bop[1] : Bop[2];
        const h8v B1 = firstB == 0 ? Bop[1] : firstB == 1 ? Bop[2] : Bop[3];
        segment(S2, S3, std::false_type{}, B0, B1, 32 * (nblocks - firstB), s0, s1, 0);
        if (packed && 32 * firstB + nn < ntA) s0 = old0;
        if (firstB == 0) { acc[0] = s0; acc[1] = s1; }
        else if (firstB == 1) { acc[1] = s0; acc[2] = s1; }
        else { acc[2] = s0; acc[3] = s1; }
    }

#pragma unroll
    for (int h = 0; h < 2; ++h) {   // lanes 0-31 write blocks 0 and 2, lanes 32-63 blocks 1 and 3
        const float lo = acc[2 * h] + __shfl_xor(acc[2 * h], 32, 64), hi = acc[2 * h + 1] + __shfl_xor(acc[2 * h + 1], 32, 64);
        const float res = kk ? __builtin_amdgcn_exp2f(ni[2 * h + 1]) * hi : __builtin_amdgcn_exp2f(ni[2 * h]) * lo;
        uint32_t kt;
        if (target(2 * h + kk, kt)) ys[kt] = res;
    }
}

// sums of the slices of a split near-field launch, in ascending slice order
__global__ __launch_bounds__(256) void p2p_split_sum_kernel(const float *__restrict__ part, int nsplit, int64_t n,
                                                            float *__restrict__ ys, int accumulate) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= n) return;
    float s = accumulate ? ys[k] : 0.f;
    for (int j = 0; j < nsplit; ++j) s += part[(int64_t)j * n + k];
    ys[k] = s;
}

// Direct sums for the small-field pairs of a depth (Sec. 4.2): both boxes of a pair hold few
// points, so neither a lane per target nor blocks of 32 x 32 would be filled.  Here lane =
// source: the sources of a target box's row are taken as one dense sequence over its boxes
// (the lane-held segment table of p2p_gram3_kernel), 64 per step, and a wavefront handles a run
// of at most SMALL_TT targets of one box, whose coordinates are wave-uniform.  Every lane keeps
// one partial sum per target; they are added across the lanes once, at the end.  Differences
// are formed directly (the pairs may be several boxes apart).  The result is added to ys
// (accumulate) or written.  The same kernel takes the overflow tiles of the near field of the last
// depth (overflow != 0): one tile per listed box, the targets behind its last full run of 64.  MB > 1: that many
// right-hand sides share the exponentials (four columns of 3e6 points: 4.83 -> 4.50 ms for the product).
template <int D>
constexpr int small_tt() { return D <= 4 ? 16 : 8; }

template <int D, int TT, int MB = 1>
__global__ __launch_bounds__(256) void p2p_small_kernel(const float *__restrict__ Xt,
                                                        const uint32_t *__restrict__ startT,
                                                        const float *__restrict__ Xs, const float *__restrict__ bs,
                                                        const uint32_t *__restrict__ start,
                                                        const uint64_t *__restrict__ row_ptr,
                                                        const uint32_t *__restrict__ cols,
                                                        const uint32_t *__restrict__ tile_box,
                                                        const uint32_t *__restrict__ tile_first, int64_t ntiles,
                                                        float nc2, float *__restrict__ ys, int overflow, int accumulate,
                                                         MultiArg MA) {
    const int lane = threadIdx.x & 63;
    const int64_t t = block_index() * 4 + (threadIdx.x >> 6);
    if (t >= ntiles) return;
    const uint32_t a = __builtin_amdgcn_readfirstlane(tile_box[t]);
    const uint32_t kend = startT[a + 1];
    const uint32_t k0 = overflow ? startT[a] + ((kend - startT[a]) & ~63u)
                                 : startT[a] + (uint32_t)(t - tile_first[a]) * (uint32_t)TT;
    const int nt = (int)(kend - k0 < (uint32_t)TT ? kend - k0 : (uint32_t)TT);   // wave-uniform
    float xt[TT][D];   // target coordinates, wave-uniform (rows beyond nt repeat an in-bounds point)
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
        const uint32_t kt = k0 + (uint32_t)(tt < nt ? tt : 0);
#pragma unroll
        for (int d = 0; d < D; ++d) xt[tt][d] = Xt[(int64_t)kt * D + d];
    }
    float acc[TT][MB];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
        for (int j = 0; j < MB; ++j) acc[tt][j] = 0.f;
    auto rhs = [&](int j, uint32_t src) { return MB == 1 ? bs[src] : MA.bs[j][src]; };

    const uint64_t e0 = row_ptr[a], e1 = row_ptr[a + 1];
    for (uint64_t er = e0; er < e1; er += 64) {   // rounds of up to 64 boxes of the row
        const int m = (int)(e1 - er < 64 ? e1 - er : 64);
        uint32_t sfirst = 0, slen = 0;
        if (lane < m) {
            const uint32_t q = cols[er + lane];
            sfirst = start[q];
            slen = start[q + 1] - sfirst;
        }
        const uint32_t cend = wave_incl_scan_u32(slen);   // inclusive running sum of the lengths over the lanes
        const uint32_t cbeg = cend - slen;
        const uint32_t delta = sfirst - cbeg;   // position -> source index inside this lane's box (mod 2^32)
        const uint32_t S = __builtin_amdgcn_readlane(cend, 63);
        if (S == 0) continue;
        int r = 0;
        // source index of position w0 + lane, as in p2p_gram3_kernel (positions from S on take the
        // last source of the sequence)
        auto locate = [&](uint32_t w0) {
            const uint32_t p = min(w0 + (uint32_t)lane, S - 1u);
            while ((uint32_t)__builtin_amdgcn_readlane(cend, r) <= w0) ++r;   // ends: w0 < S = cend of lane 63
            uint32_t src = p + (uint32_t)__builtin_amdgcn_readlane(delta, r);
            for (int rr = r + 1; rr < m; ++rr) {
                const uint32_t c0 = __builtin_amdgcn_readlane(cbeg, rr);
                if (c0 >= w0 + 64) break;
                const uint32_t dl = __builtin_amdgcn_readlane(delta, rr);
                src = p >= c0 ? p + dl : src;
            }
            return src;
        };
        float xn[D], bn[MB];
        {
            const uint32_t src = locate(0);
#pragma unroll
            for (int d = 0; d < D; ++d) xn[d] = Xs[(int64_t)src * D + d];
#pragma unroll
            for (int j = 0; j < MB; ++j) bn[j] = rhs(j, src);
        }
        for (uint32_t w0 = 0; w0 < S; w0 += 64) {
            float x[D];
#pragma unroll
            for (int d = 0; d < D; ++d) x[d] = xn[d];
            float bv[MB];
#pragma unroll
            for (int j = 0; j < MB; ++j) bv[j] = bn[j];
            if (w0 + 64 > S) {      // last step only: positions behind the sequence contribute nothing
                asm volatile("");   // keeps this a branch (as a select it costs every step three instructions)
#pragma unroll
                for (int j = 0; j < MB; ++j) bv[j] = w0 + lane < S ? bv[j] : 0.f;
            }
            // the loads of the next step are in flight during this one (the last step loads its own
            // sources again, so the number of loads in flight is fixed)
            const uint32_t nsrc = locate(w0 + 64 < S ? w0 + 64 : w0);
#pragma unroll
            for (int d = 0; d < D; ++d) xn[d] = Xs[(int64_t)nsrc * D + d];
#pragma unroll
            for (int j = 0; j < MB; ++j) bn[j] = rhs(j, nsrc);
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) {
                if (tt < nt) {
                    float r2 = 0.f;
#pragma unroll
                    for (int d = 0; d < D; ++d) {
                        const float df = x[d] - xt[tt][d];
                        r2 = fmaf(df, df, r2);
                    }
                    const float e = __builtin_amdgcn_exp2f(r2 * nc2);
#pragma unroll
                    for (int j = 0; j < MB; ++j) acc[tt][j] = fmaf(e, bv[j], acc[tt][j]);
                }
            }
        }
    }
    // sums over the lanes; lane tt keeps the total of target tt
#pragma unroll
    for (int j = 0; j < MB; ++j) {
        float res = 0.f;
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
            if (tt < nt) {
                float v = acc[tt][j];
#pragma unroll
                for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
                if (lane == tt) res = v;
            }
        }
        float *out = MB == 1 ? ys : MA.ys[j];
        if (lane < nt) out[k0 + lane] = accumulate ? out[k0 + lane] + res : res;
    }
}

// exact product, all pairs (Sec. 2, KeOps paragraph): targets are the rows of X (nx of them), sources the rows of Y
// (n of them, weights b); X == Y for one point set.  Two kernels (run_direct_d says which one takes a call); both add
// runs of 32 sources in fp32 and the runs in fp64.
//
// Lane = target, the sources wave-uniform (scalar loads).  Bound: the vector ALU with many sources (3-D: 4.5e12 pairs/s),
// the reads of X and writes of y with few (1e7 targets, 1 source, 3-D: 35 us).
template <int D>
__global__ __launch_bounds__(64) void direct_lane_kernel(const float *__restrict__ X, int64_t nx,
                                                         const float *__restrict__ Y, const float *__restrict__ b,
                                                         int64_t n, float nc2, float *__restrict__ y) {
    const int64_t i = (int64_t)blockIdx.x * 64 + threadIdx.x;
    const bool active = i < nx;
    float xi[D];
#pragma unroll
    for (int d = 0; d < D; ++d) xi[d] = active ? X[i * D + d] : 0.f;
    double acc = 0.0;
    for (int64_t j0 = 0; j0 < n; j0 += 32) {
        const int64_t je = min(j0 + 32, n);
        float run = 0.f;
#pragma unroll 4
        for (int64_t j = j0; j < je; ++j) {
            float r2 = 0.f;
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const float diff = Y[j * D + d] - xi[d];
                r2 = fmaf(diff, diff, r2);
            }
            run = fmaf(__builtin_amdgcn_exp2f(r2 * nc2), b[j], run);
        }
        acc += (double)run;
    }
    if (active) y[i] = (float)acc;
}

// A lane per target alone leaves the chip idle below some 1e5 targets (n = 2e4: 313 wavefronts on 1024 SIMDs), so here a
// wavefront is TL target lanes x 64 / TL source lanes, the eight wavefronts of a workgroup share their targets and divide
// the sources, and the sums meet in a fixed order at the end.  Sources pass through LDS in tiles of DT_TILE rows (D
// coordinates and the weight); a lane keeps TPL targets, so that a row read from LDS serves TPL pairs.
// Bound: the vector ALU, nine instructions per 3-D pair (three differences, four for the scaled square, the exponential,
// one multiply-add).  As dependent chains they take 40 cycles of a SIMD (4 each, the exponential 8); the kernel takes 33
// (4.76e12 pairs/s at n = 3e5 and 2.4 GHz): instructions of several wavefronts overlap.
// Measured (3-D): n = 2e4 1003 -> 102 us (1250 workgroups, 1024 of which are resident at once: the second round leaves
// most of the chip idle; 84 us at the rate of n = 3e5), n = 3e5 24.6 -> 18.9 ms; 1e3 .. 5e3 points 9 .. 15 us, the time
// of a launch.
constexpr int DT_NT = 512;
constexpr int DT_TILE = 1024;
template <int D, int TL, int TPL>
__global__ __launch_bounds__(DT_NT) void direct_kernel(const float *__restrict__ X, int64_t nx,
                                                       const float *__restrict__ Y, const float *__restrict__ b,
                                                       int64_t n, float nc2, float *__restrict__ y) {
    constexpr int RS = D == 1 ? 2 : D <= 3 ? 4 : 8;       // floats of a row in LDS: vector reads stay aligned
    constexpr int SL = 64 / TL;                           // source lanes of a wavefront
    constexpr int NG = (DT_NT / 64) * SL;                 // source groups of the workgroup
    constexpr int RUN = 32;                               // sources of a run
    static_assert(DT_TILE % NG == 0, "every group has as many rows of a tile");
    __shared__ __attribute__((aligned(16))) float rows[DT_TILE * RS];
    __shared__ double sums[DT_NT / 64][TL * TPL];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int tl = lane % TL, sl = lane / TL, grp = w * SL + sl;
    const int64_t t0 = block_index() * (TL * TPL), i0 = t0 + tl;
    if (t0 >= nx) return;
    float xi[TPL][D];
    double acc[TPL];
#pragma unroll
    for (int t = 0; t < TPL; ++t) {
        const int64_t i = min(i0 + t * TL, nx - 1);       // a lane behind the last target repeats it
#pragma unroll
        for (int d = 0; d < D; ++d) xi[t][d] = X[i * D + d];
        acc[t] = 0.0;
    }
    for (int64_t j0 = 0; j0 < n; j0 += DT_TILE) {
        __syncthreads();                                  // the previous tile has been read
#pragma unroll
        for (int k = 0; k < DT_TILE / DT_NT; ++k) {
            const int row = k * DT_NT + tid;
            const int64_t j = min(j0 + row, n - 1);       // rows behind the last source repeat it with weight zero
            const float bj = b[j];
#pragma unroll
            for (int d = 0; d < D; ++d) rows[row * RS + d] = Y[j * D + d];
            rows[row * RS + D] = j0 + row < n ? bj : 0.f;
        }
        __syncthreads();
        const int left = (int)min(n - j0, (int64_t)DT_TILE);
        for (int r0 = 0; r0 < left; r0 += NG * RUN) {     // a run of every group: rows r0 + grp, r0 + grp + NG, ...
            float run[TPL];
#pragma unroll
            for (int t = 0; t < TPL; ++t) run[t] = 0.f;
            const int last = min(RUN, (left - r0 + NG - 1) / NG);
#pragma unroll 4
            for (int k = 0; k < last; ++k) {
                const float *row = rows + (r0 + grp + k * NG) * RS;
                float ys[D];
#pragma unroll
                for (int d = 0; d < D; ++d) ys[d] = row[d];
                const float bj = row[D];
#pragma unroll
                for (int t = 0; t < TPL; ++t) {
                    float r2 = 0.f;
#pragma unroll
                    for (int d = 0; d < D; ++d) {
                        const float diff = ys[d] - xi[t][d];
                        r2 = fmaf(diff, diff, r2);
                    }
                    run[t] = fmaf(__builtin_amdgcn_exp2f(r2 * nc2), bj, run[t]);
                }
            }
#pragma unroll
            for (int t = 0; t < TPL; ++t) acc[t] += (double)run[t];
        }
    }
#pragma unroll
    for (int t = 0; t < TPL; ++t) {
#pragma unroll
        for (int off = TL; off < 64; off <<= 1) acc[t] += __shfl_xor(acc[t], off, 64);
        if (sl == 0) sums[w][t * TL + tl] = acc[t];
    }
    __syncthreads();
    if (tid < TL * TPL) {
        const int64_t i = t0 + tid;
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < DT_NT / 64; ++k) s += sums[k][tid];
        if (i < nx) y[i] = (float)s;
    }
}

// 2^(r2 nc2) in fp64 for r2 >= 0, nc2 < 0, to about one unit in the last place: k = the integer next to the exponent
// (the classic shift by 1.5 2^52 leaves it in the low word of the sum), f = exponent - k with |f| <= 1/2 in one fused
// operation, 2^f by 1 + f q(f) with q the polynomial of degree 10 that interpolates (2^f - 1) / f at the Chebyshev
// points of [-1/2, 1/2] (relative error 8.5e-18, formed with 60 digits), and v_ldexp_f64, which also does the
// denormal results.  r2 is cut at `cap`, where the result has long been zero, so that k fits the low word; the minimum
// also turns a NaN into `cap`, so the caller has to see to coordinates that are not numbers.
// The library's exp needs some ten instructions more for arguments of either sign and its special cases.
__device__ inline double exp2_scaled(double r2, double nc2, double cap) {
    constexpr double SHIFT = 6755399441055744.0;
    r2 = fmin(r2, cap);
    const double t = fma(r2, nc2, SHIFT);
    const int k = (int)(uint32_t)__builtin_bit_cast(uint64_t, t);
    const double f = fma(r2, nc2, SHIFT - t);
    double q = 4.4549605981865186e-10;
    q = fma(q, f, 7.072585949269223e-09);
    q = fma(q, f, 1.0178062445845774e-07);
    q = fma(q, f, 1.321544258792169e-06);
    q = fma(q, f, 1.525273382983612e-05);
    q = fma(q, f, 0.0001540353044173605);
    q = fma(q, f, 0.0013333558146416936);
    q = fma(q, f, 0.009618129107606888);
    q = fma(q, f, 0.0555041086648216);
    q = fma(q, f, 0.24022650695910097);
    q = fma(q, f, 0.6931471805599453);
    return __builtin_amdgcn_ldexp(fma(q, f, 1.0), k);
}

// exact rows in fp64: a workgroup of four wavefronts per 64 R rows and slice of the sources (blockIdx.y); the
// wavefronts divide the sources of the slice, lane = R rows.  Partial sums per slice.
// Bound: the fp64 vector ALU (some 25 operations per 3-D pair).  The sources are turned into fp64 once per workgroup
// on their way into LDS (as scalar operands they cost every wavefront D + 1 conversions per source).
// Measured (3-D, 1e4 rows x 1e6 sources): 9.66 -> 7.1 ms, 1.40e12 pairs/s at 23 fp64 instructions each.
// A squared distance that is not a number (a NaN coordinate, or equal infinities) makes the sum NaN, without an
// instruction in the inner loop: a source with a NaN coordinate gets the weight NaN, and a wavefront with a row whose
// coordinates are not all finite goes through its sources a second time.
constexpr int ROWS_TILE = 256;
template <int D, int R>
__global__ __launch_bounds__(256) void rows_f64_kernel(const float *__restrict__ X, const float *__restrict__ Y,
                                                       const float *__restrict__ b, int64_t n,
                                                       const int64_t *__restrict__ rows, int64_t m,
                                                       double nc2, double cap, double *__restrict__ part) {
    constexpr int RS = (D + 2) / 2 * 2;   // doubles of a source in LDS
    __shared__ __attribute__((aligned(16))) double src[ROWS_TILE * RS];
    __shared__ double sums[4][64 * R];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t a0 = (int64_t)blockIdx.x * (64 * R);
    double xi[R][D], acc[R];
#pragma unroll
    for (int t = 0; t < R; ++t) {
        const int64_t i = rows[min(a0 + t * 64 + lane, m - 1)];   // a lane behind the last row repeats it
#pragma unroll
        for (int d = 0; d < D; ++d) xi[t][d] = (double)X[i * D + d];
        acc[t] = 0.0;
    }
    const int64_t per = (n + gridDim.y - 1) / gridDim.y;
    const int64_t j0 = (int64_t)blockIdx.y * per, j1 = min(n, j0 + per);
    for (int64_t jt = j0; jt < j1; jt += ROWS_TILE) {
        __syncthreads();   // the previous tile has been read
        {
            const int64_t j = min(jt + tid, j1 - 1);   // behind the slice: its last source with weight zero
            float bj = b[j];
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const float yj = Y[j * D + d];
                src[tid * RS + d] = (double)yj;
                bj = yj == yj ? bj : yj;
            }
            src[tid * RS + D] = jt + tid < j1 ? (double)bj : 0.0;
        }
        __syncthreads();
        const int cnt = (int)min(j1 - jt, (int64_t)ROWS_TILE);
        double run[R];   // a tile is summed on its own: long slices lose fewer bits than with one running sum
#pragma unroll
        for (int t = 0; t < R; ++t) run[t] = 0.0;
#pragma unroll 2
        for (int k = w; k < cnt; k += 4) {
            const double *row = src + k * RS;
#pragma unroll
            for (int t = 0; t < R; ++t) {
                double r2 = 0.0;
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    const double diff = row[d] - xi[t][d];
                    r2 = fma(diff, diff, r2);
                }
                run[t] = fma(exp2_scaled(r2, nc2, cap), row[D], run[t]);
            }
        }
#pragma unroll
        for (int t = 0; t < R; ++t) acc[t] += run[t];
    }
    bool finite = true;
#pragma unroll
    for (int t = 0; t < R; ++t)
#pragma unroll
        for (int d = 0; d < D; ++d) finite = finite && xi[t][d] - xi[t][d] == 0.0;
    if (__any(!finite)) {
        for (int64_t j = j0 + w; j < j1; j += 4) {
#pragma unroll
            for (int t = 0; t < R; ++t) {
                double r2 = 0.0;
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    const double diff = (double)Y[j * D + d] - xi[t][d];
                    r2 = fma(diff, diff, r2);
                }
                acc[t] = r2 == r2 ? acc[t] : r2;
            }
        }
    }
#pragma unroll
    for (int t = 0; t < R; ++t) sums[w][t * 64 + lane] = acc[t];
    __syncthreads();
    if (tid < 64 * R && a0 + tid < m)
        part[(int64_t)blockIdx.y * m + a0 + tid] = (sums[0][tid] + sums[1][tid]) + (sums[2][tid] + sums[3][tid]);
}
// sums of the slices: a workgroup per 64 rows, every wavefront adds a quarter of the slices in ascending order (one thread
// per row over all of them left 256 slices to 40 workgroups at m = 1e4)
__global__ __launch_bounds__(256) void rows_f64_sum_kernel(const double *__restrict__ part, int64_t m, int slices,
                                                           double *__restrict__ y64) {
    __shared__ double sums[4][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t a = (int64_t)blockIdx.x * 64 + lane;
    double s = 0.0;
    if (a < m) {
#pragma unroll 8
        for (int k = w; k < slices; k += 4) s += part[(int64_t)k * m + a];
    }
    sums[w][lane] = s;
    __syncthreads();
    if (w == 0 && a < m) y64[a] = (sums[0][lane] + sums[1][lane]) + (sums[2][lane] + sums[3][lane]);
}

// ------------------------------------------------------------------------------------
// tensor-product Lagrange weights of one point of a box: for each dimension the local
// coordinate t = (x - centre) / (l/2) is formed in fp64 (centre = alpha + (c + 1/2) l), the
// p basis values in fp32 by the product form.  out[d*p + i] = L_i(t_d).
// ------------------------------------------------------------------------------------
template <int D>
__device__ inline void point_weights(const float *__restrict__ x, const int32_t *__restrict__ cell,
                                     const CentreArg &C, const NodeArg &N, int p, float *out) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
        double centre = C.alpha[d] + ((double)cell[d] + 0.5) * C.edge;
        float t = (float)(((double)x[d] - centre) * C.inv_half);
        for (int i = 0; i < p; ++i) {
            float num = 1.f;
            for (int j = 0; j < p; ++j)
                if (j != i) num *= t - N.s[j];
            out[d * p + i] = num * N.invden[i];
        }
    }
}

// The same with the number of nodes known when compiled, one dimension.
template <int PN>
__device__ inline void dim_weights(float x, int32_t cell, double alpha, const CentreArg &C, const NodeArg &N, float *out) {
    const double centre = alpha + ((double)cell + 0.5) * C.edge;
    const float t = (float)(((double)x - centre) * C.inv_half);
#pragma unroll
    for (int i = 0; i < PN; ++i) {
        float num = 1.f;
#pragma unroll
        for (int j = 0; j < PN; ++j)
            if (j != i) num *= t - N.s[j];
        out[i] = num * N.invden[i];
    }
}

constexpr int ipow(int p, int e) { return e <= 0 ? 1 : p * ipow(p, e - 1); }

// node index -> packed digits (4 bits per dimension)
template <int D>
__device__ inline uint32_t node_code(int i, int p) {
    uint32_t code = 0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        code |= (uint32_t)(i % p) << (4 * d);
        i /= p;
    }
    return code;
}

// ------------------------------------------------------------------------------------
// P2M, v1 = L_Y b (Fig. 4 step 1): W_q[i] = sum_{j in q} L_i(t_j) b_j.
// One block per chunk (a run of <= P2M_CHUNK points of one box); points are staged through LDS as their 1-D basis
// values.  No atomics: a box with several chunks gets partial sums that p2m_reduce_kernel adds in a fixed order.
// At most 64 nodes: a wavefront per chunk, a lane per node; with at most 32 nodes the lanes form groups that share the
// points (16 nodes, 256 points: 64 steps instead of 256).
// ------------------------------------------------------------------------------------
constexpr int FF_TP = 64;  // points staged per step

template <int D>
__global__ __launch_bounds__(64) void p2m_kernel(const float *__restrict__ Xs, const float *__restrict__ bs,
                                                 const uint32_t *__restrict__ start, const int32_t *__restrict__ cell,
                                                 const uint32_t *__restrict__ chunk_box,
                                                 const uint32_t *__restrict__ chunk_first, int64_t nchunks, int p,
                                                 int r, CentreArg C, NodeArg N, float *__restrict__ W,
                                                 float *__restrict__ Wpart) {
    extern __shared__ float lds[];
    const int DP = D * p;
    float *wts = lds;                 // [FF_TP][DP]
    float *bj = lds + FF_TP * DP;     // [FF_TP]
    const int64_t c = block_index();
    if (c >= nchunks) return;
    const uint32_t a = chunk_box[c];
    const uint32_t ci = (uint32_t)(c - chunk_first[a]);
    const uint32_t nch = chunk_first[a + 1] - chunk_first[a];
    const uint32_t k0 = start[a] + ci * (uint32_t)P2M_CHUNK;
    const uint32_t k1 = min(k0 + (uint32_t)P2M_CHUNK, start[a + 1]);
    const int tid = threadIdx.x;
    const int groups = 64 / r, g = tid / r, i = tid - g * r;   // lanes behind the last whole group have no points
    const uint32_t code = node_code<D>(i, p);
    float acc = 0.f;
    for (uint32_t kb = k0; kb < k1; kb += FF_TP) {
        const int cnt = (int)min((uint32_t)FF_TP, k1 - kb);
        __syncthreads();
        if (tid < cnt) {
            const int64_t k = (int64_t)kb + tid;
            point_weights<D>(Xs + k * D, cell + (int64_t)a * D, C, N, p, wts + tid * DP);
            bj[tid] = bs[k];
        }
        __syncthreads();
        if (g < groups) {
            for (int jj = g; jj < cnt; jj += groups) {
                const float *wj = wts + jj * DP;
                float prod = bj[jj];
#pragma unroll
                for (int d = 0; d < D; ++d) prod *= wj[d * p + ((code >> (4 * d)) & 15u)];
                acc += prod;
            }
        }
    }
    __syncthreads();
    bj[tid] = acc;
    __syncthreads();
    if (tid < r) {
        for (int q = 1; q < groups; ++q) acc += bj[q * r + tid];
        float *dst = nch == 1 ? W + (int64_t)a * r : Wpart + c * r;
        dst[tid] = acc;
    }
}

// More than 64 nodes.  The nodes are a tensor grid, so W is a sum over points of outer products: the weights over the lower
// dimensions (RA of them) times those over the upper ones (RB, times b), both made once per point in LDS.  A thread
// owns PN x PN nodes -- the lowest dimension of either half -- so it reads 2 PN values for PN^2 multiply-adds, and where
// that leaves threads over they form groups that share the points.  (A thread per node read D values and multiplied D
// times for each: n = 3e5, D = 7, 3 nodes, both depths 6.1 ms.)
template <int D, int PN>
struct P2mHalves {
    static constexpr int DA = (D + 1) / 2, DB = D - DA;
    static constexpr int RA = ipow(PN, DA), RB = ipow(PN, DB), R = RA * RB;
    static constexpr int TA = RA / PN, TB = RB / PN, ITEMS = TA * TB;
    static constexpr int GROUPS = 256 / ITEMS;
    static constexpr int TP = 32;   // points staged per step
    static_assert(DB >= 1 && ITEMS <= 256, "a thread per PN x PN nodes");
};
template <int D, int PN>
__global__ __launch_bounds__(256) void p2m_halves_kernel(const float *__restrict__ Xs, const float *__restrict__ bs,
                                                         const uint32_t *__restrict__ start,
                                                         const int32_t *__restrict__ cell,
                                                         const uint32_t *__restrict__ chunk_box,
                                                         const uint32_t *__restrict__ chunk_first, int64_t nchunks,
                                                         CentreArg C, NodeArg N, float *__restrict__ W,
                                                         float *__restrict__ Wpart) {
    using H = P2mHalves<D, PN>;
    constexpr int TP = H::TP;
    __shared__ float wts[TP][D * PN];
    __shared__ float half_a[TP][H::RA], half_b[TP][H::RB];
    __shared__ float sums[H::GROUPS > 1 ? H::R : 1];
    const int64_t c = block_index();
    if (c >= nchunks) return;
    const uint32_t a = chunk_box[c];
    const uint32_t ci = (uint32_t)(c - chunk_first[a]);
    const uint32_t nch = chunk_first[a + 1] - chunk_first[a];
    const uint32_t k0 = start[a] + ci * (uint32_t)P2M_CHUNK;
    const uint32_t k1 = min(k0 + (uint32_t)P2M_CHUNK, start[a + 1]);
    const int tid = threadIdx.x;
    const int g = tid / H::ITEMS, item = tid - g * H::ITEMS;
    const int ia = (item % H::TA) * PN, ib = (item / H::TA) * PN;
    float acc[PN][PN];
#pragma unroll
    for (int v = 0; v < PN; ++v)
#pragma unroll
        for (int u = 0; u < PN; ++u) acc[v][u] = 0.f;
    for (uint32_t kb = k0; kb < k1; kb += TP) {
        const int cnt = (int)min((uint32_t)TP, k1 - kb);
        __syncthreads();
        for (int e = tid; e < TP * D; e += 256) {
            const int j = e / D, d = e - j * D;
            if (j < cnt)
                dim_weights<PN>(Xs[((int64_t)kb + j) * D + d], cell[(int64_t)a * D + d], C.alpha[d], C, N, &wts[j][d * PN]);
        }
        __syncthreads();
        for (int e = tid; e < TP * H::RA; e += 256) {
            const int j = e / H::RA;
            int q = e - j * H::RA;
            const int at = q;
            float prod = 1.f;
#pragma unroll
            for (int d = 0; d < H::DA; ++d) {
                prod *= wts[j][d * PN + q % PN];
                q /= PN;
            }
            half_a[j][at] = prod;
        }
        for (int e = tid; e < TP * H::RB; e += 256) {
            const int j = e / H::RB;
            int q = e - j * H::RB;
            const int at = q;
            float prod = j < cnt ? bs[(int64_t)kb + j] : 0.f;
#pragma unroll
            for (int d = 0; d < H::DB; ++d) {
                prod *= wts[j][(H::DA + d) * PN + q % PN];
                q /= PN;
            }
            half_b[j][at] = prod;
        }
        __syncthreads();
        if (g < H::GROUPS) {
            for (int j = g; j < cnt; j += H::GROUPS) {
                float A[PN], B[PN];
#pragma unroll
                for (int u = 0; u < PN; ++u) {
                    A[u] = half_a[j][ia + u];
                    B[u] = half_b[j][ib + u];
                }
#pragma unroll
                for (int v = 0; v < PN; ++v)
#pragma unroll
                    for (int u = 0; u < PN; ++u) acc[v][u] = fmaf(A[u], B[v], acc[v][u]);
            }
        }
    }
    // the groups' sums one after the other, in ascending order
    if constexpr (H::GROUPS > 1) {
        for (int q = H::GROUPS - 1; q >= 1; --q) {
            if (g == q) {
#pragma unroll
                for (int v = 0; v < PN; ++v)
#pragma unroll
                    for (int u = 0; u < PN; ++u) {
                        float *at = &sums[(ia + u) + H::RA * (ib + v)];
                        *at = q == H::GROUPS - 1 ? acc[v][u] : *at + acc[v][u];
                    }
            }
            __syncthreads();
        }
    }
    if (g == 0) {
        float *dst = nch == 1 ? W + (int64_t)a * H::R : Wpart + c * H::R;
#pragma unroll
        for (int v = 0; v < PN; ++v)
#pragma unroll
            for (int u = 0; u < PN; ++u) {
                const int i = (ia + u) + H::RA * (ib + v);
                dst[i] = H::GROUPS > 1 ? acc[v][u] + sums[i] : acc[v][u];
            }
    }
}

// boxes that were split into several chunks: add the partial node weights, chunk by
// chunk in ascending order, in fp64
__global__ __launch_bounds__(256) void p2m_reduce_kernel(const uint32_t *__restrict__ chunk_first, int64_t nb, int r,
                                                         const float *__restrict__ Wpart, float *__restrict__ W) {
    const int64_t a = block_index();
    if (a >= nb) return;
    const uint32_t c0 = chunk_first[a], c1 = chunk_first[a + 1];
    if (c1 - c0 <= 1) return;
    __shared__ double part[4][64];
    const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
    for (int i0 = 0; i0 < r; i0 += 64) {
        const int i = i0 + lane;
        double s = 0.0;
        if (i < r)
            for (uint32_t c = c0 + g; c < c1; c += 4) s += (double)Wpart[(int64_t)c * r + i];
        __syncthreads();
        part[g][lane] = s;
        __syncthreads();
        if (g == 0 && i < r) W[(int64_t)a * r + i] = (float)(((part[0][lane] + part[1][lane]) + part[2][lane]) + part[3][lane]);
    }
}

// Two-stage form for boxes with very many chunks: a block adds the partial node weights of one
// slice (at most P2M_SLICE chunks of one box) in fp64, then a block per box adds its slices,
// both in a fixed order.
__global__ __launch_bounds__(256) void p2m_slice_kernel(const uint32_t *__restrict__ slice_box,
                                                        const uint32_t *__restrict__ slice_first,
                                                        const uint32_t *__restrict__ chunk_first, int64_t nslices, int r,
                                                        const float *__restrict__ Wpart, double *__restrict__ Wslice) {
    const int64_t sidx = block_index();
    if (sidx >= nslices) return;
    const uint32_t a = slice_box[sidx];
    const uint32_t c0 = chunk_first[a] + (uint32_t)(sidx - slice_first[a]) * (uint32_t)P2M_SLICE;
    const uint32_t c1 = min(c0 + (uint32_t)P2M_SLICE, chunk_first[a + 1]);
    __shared__ double part[4][64];
    const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
    for (int i0 = 0; i0 < r; i0 += 64) {
        const int i = i0 + lane;
        double s = 0.0;
        if (i < r)
            for (uint32_t c = c0 + g; c < c1; c += 4) s += (double)Wpart[(int64_t)c * r + i];
        __syncthreads();
        part[g][lane] = s;
        __syncthreads();
        if (g == 0 && i < r) Wslice[sidx * r + i] = ((part[0][lane] + part[1][lane]) + part[2][lane]) + part[3][lane];
    }
}
__global__ __launch_bounds__(256) void p2m_slice_sum_kernel(const uint32_t *__restrict__ slice_first,
                                                            const uint32_t *__restrict__ chunk_first, int64_t nb, int r,
                                                            const double *__restrict__ Wslice, float *__restrict__ W) {
    const int64_t a = block_index();
    if (a >= nb) return;
    if (chunk_first[a + 1] - chunk_first[a] <= 1) return;   // the P2M kernel wrote W itself
    const uint32_t s0 = slice_first[a], s1 = slice_first[a + 1];
    for (int i = threadIdx.x; i < r; i += 256) {
        double s = 0.0;
        for (uint32_t k = s0; k < s1; ++k) s += Wslice[(int64_t)k * r + i];
        W[(int64_t)a * r + i] = (float)s;
    }
}

// ------------------------------------------------------------------------------------
// L2P, v = L_X^T v2 (Fig. 4 step 3): y_a += sum_i L_i(t_a) V_p[i] for the points a of box p.
// One block per chunk, one thread per point; V_p in LDS (every lane reads the same entry).  The sum is nested over the
// dimensions, p + p^2 + ... + p^D multiply-adds; the dimensions of at most 81 nodes are unrolled with their basis values in
// registers, the others are loops that read theirs from LDS.  (One loop over all nodes that multiplied D basis
// values each: n = 3e5, D = 7, 3 nodes, both depths 1.5 ms.)
// ------------------------------------------------------------------------------------
template <int D, int PN>
struct L2pShape {
    static constexpr int inner() {
        int d = 1;
        while (d < D && ipow(PN, d + 1) <= 81) ++d;
        return d;
    }
    static constexpr int IN = inner(), OUT = D - IN;   // unrolled and looped dimensions
};
// sum over the nodes of dimensions 0 .. d
template <int PN, int IN, int d>
__device__ __forceinline__ float l2p_inner(const float (&L)[IN][PN], const float *V) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < PN; ++i) {
        if constexpr (d == 0) s = fmaf(L[0][i], V[i], s);
        else s = fmaf(L[d][i], l2p_inner<PN, IN, (d > 0 ? d - 1 : 0)>(L, V + i * ipow(PN, d)), s);
    }
    return s;
}
// dimensions 0 .. IN - 1 + o, o > 0: wo holds the basis values of the looped dimensions
template <int PN, int IN, int o>
__device__ __forceinline__ float l2p_outer(const float (&L)[IN][PN], const float *wo, const float *V) {
    if constexpr (o == 0) {
        return l2p_inner<PN, IN, IN - 1>(L, V);
    } else {
        float s = 0.f;
#pragma unroll 1
        for (int i = 0; i < PN; ++i)
            s = fmaf(wo[(o - 1) * PN + i], l2p_outer<PN, IN, (o > 0 ? o - 1 : 0)>(L, wo, V + i * ipow(PN, IN + o - 1)), s);
        return s;
    }
}
template <int D, int PN>
__global__ __launch_bounds__(P2M_CHUNK) void l2p_kernel(const float *__restrict__ Xs,
                                                        const uint32_t *__restrict__ start,
                                                        const int32_t *__restrict__ cell,
                                                        const uint64_t *__restrict__ far_ptr,
                                                        const uint32_t *__restrict__ chunk_box,
                                                        const uint32_t *__restrict__ chunk_first, int64_t nchunks,
                                                        CentreArg C, NodeArg N, const float *__restrict__ V,
                                                        float *__restrict__ ys) {
    constexpr int R = ipow(PN, D), IN = L2pShape<D, PN>::IN, OUT = L2pShape<D, PN>::OUT;
    constexpr int STRIDE = (OUT * PN) | 1;
    __shared__ float Vs[R];
    __shared__ float wts[OUT > 0 ? P2M_CHUNK * STRIDE : 1];
    const int64_t c = block_index();
    if (c >= nchunks) return;
    const uint32_t a = chunk_box[c];
    if (far_ptr[a + 1] == far_ptr[a]) return;  // no far partner at this depth: V_p is zero
    const uint32_t ci = (uint32_t)(c - chunk_first[a]);
    const uint32_t k = start[a] + ci * (uint32_t)P2M_CHUNK + threadIdx.x;
    const bool active = k < start[a + 1];
    for (int i = threadIdx.x; i < R; i += P2M_CHUNK) Vs[i] = V[(int64_t)a * R + i];
    float L[IN][PN];
    float *w = wts + (OUT > 0 ? threadIdx.x * STRIDE : 0);
    if (active) {
#pragma unroll
        for (int d = 0; d < IN; ++d)
            dim_weights<PN>(Xs[(int64_t)k * D + d], cell[(int64_t)a * D + d], C.alpha[d], C, N, L[d]);
#pragma unroll
        for (int d = IN; d < D; ++d)
            dim_weights<PN>(Xs[(int64_t)k * D + d], cell[(int64_t)a * D + d], C.alpha[d], C, N, w + (d - IN) * PN);
    }
    __syncthreads();
    if (!active) return;
    ys[k] += l2p_outer<PN, IN, OUT>(L, w, Vs);
}

// f(integral constant of the number of nodes per dimension) for a shape with at most MAX_NODES nodes
template <int D, class F>
static void for_nodes(int p, F &&f) {
    auto at = [&](auto pn) {
        constexpr int PN = decltype(pn)::value;
        if constexpr (ipow(PN, D) <= MAX_NODES) f(pn);
        else fail(F3M_ERR_UNSUPPORTED, "interp_nodes^D exceeds the node cap");
    };
    switch (p) {
        case 2: at(std::integral_constant<int, 2>{}); break;
        case 3: at(std::integral_constant<int, 3>{}); break;
        case 4: at(std::integral_constant<int, 4>{}); break;
        case 5: at(std::integral_constant<int, 5>{}); break;
        case 6: at(std::integral_constant<int, 6>{}); break;
        case 7: at(std::integral_constant<int, 7>{}); break;
        case 8: at(std::integral_constant<int, 8>{}); break;
        default: fail(F3M_ERR_UNSUPPORTED, "interp_nodes must be in [2,8]");
    }
}

// ------------------------------------------------------------------------------------
// P2M and L2P for D = 3 with 4 nodes per dimension (r = 64).  The nodes are {1, 1/2, -1/2, -1}; the product-form basis of one
// coordinate costs 4 subtractions and 10 multiplications.
//   P2M: a quad of lanes per point, the 64 products on the matrix cores (p2m34_kernel); runs of thousands of points
//        of one box: lane = point, the 64 node sums in its registers (p2m34_long_kernel).
//   L2P: lane = point, the tensor contraction nested: 64 + 16 + 4 FMAs per point and set of potentials.
// ------------------------------------------------------------------------------------
__device__ inline void lagrange4(float t, float (&L)[4]) {
    const float d0 = t - 1.f, d1 = t - 0.5f, d2 = t + 0.5f, d3 = t + 1.f;
    const float p01 = d0 * d1, p23 = d2 * d3;
    L[0] = d1 * p23 * (1.f / 1.5f);
    L[1] = d0 * p23 * (-1.f / 0.75f);
    L[2] = p01 * d3 * (1.f / 0.75f);
    L[3] = p01 * d2 * (-1.f / 1.5f);
}

// returns the squared distance from the box centre in units of (l / 2)^2
__device__ inline float weights34(const float *__restrict__ x, const double (&ctr)[3], double inv_half, float (&Lx)[4],
                                  float (&Ly)[4], float (&Lz)[4]) {
    const float tx = (float)(((double)x[0] - ctr[0]) * inv_half), ty = (float)(((double)x[1] - ctr[1]) * inv_half),
                tz = (float)(((double)x[2] - ctr[2]) * inv_half);
    lagrange4(tx, Lx);
    lagrange4(ty, Ly);
    lagrange4(tz, Lz);
    return fmaf(tz, tz, fmaf(ty, ty, tx * tx));
}

// The weighted near pairs (near_weighted_error in plan.hip) need a second set of node weights, of points times
// exp(-|u|^2 / 2 gamma^2) = exp2(kw |u|^2 / (l/2)^2): made together with the plain one (NS = 2 below; dW, dpart: from the plain
// to the weighted arrays), or alone (only).
struct WeightedArg {
    int64_t dW = 0, dpart = 0;
    float kw = 0.f;
    bool only = false;
};

// P2M on the matrix cores: v_mfma_f32_4x4x1 multiplies 16 independent columns of 4 by rows of 4 in fp32.  A quad of lanes is
// one of the 16 and takes one point at a time; its lane i evaluates L_i alone, the three coordinates and the weight
// of the point are made once per point (lane = point) and reach the quad as DPP broadcasts.  With A = L_x L_y[j] (j = 0 .. 3)
// and B = L_z b the node sums of the quad's points stay in 16 registers a lane for each set of weights (v[set][i2][i1], lane
// 4 quad + i3), and are summed over the quads once per box.  What bounds it: vector issue, some 24 instructions
// for 16 points and both sets (the 64-accumulator form, lane = point, took 130 for one lane's point and a sum of 64 x 64 values through
// LDS for each set).
typedef float f4v __attribute__((ext_vector_type(4)));
template <int NS> struct P2mSums { f4v v[NS][4]; };
struct QuadNode { float a, b, c, w; };   // L_i(t) = (t - a) (t - b) (t - c) w, multiplied in the order of lagrange4

__device__ inline QuadNode quad_node(int i) {
    return {i == 0 ? 0.5f : i == 1 ? 1.f : i == 2 ? -1.f : -0.5f, i < 2 ? -0.5f : 1.f, i < 2 ? -1.f : 0.5f,
            i == 0 ? 1.f / 1.5f : i == 1 ? -1.f / 0.75f : i == 2 ? 1.f / 0.75f : -1.f / 1.5f};
}

template <int CTRL, int BANKS> __device__ inline float dpp_into(float old, float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, old), __builtin_bit_cast(int, v), CTRL, 0xF,
                                                                 BANKS, true));
}
template <int R> __device__ inline float quad_bcast(float v) { return dpp_into<R * 0x55, 0xF>(0.f, v); }

// the points in lane R of every quad
template <int NS, int R>
__device__ inline void p2m34_step(P2mSums<NS> &S, const QuadNode &N, float tx, float ty, float tz, float b, float be) {
    auto basis = [&](float t) __attribute__((always_inline)) { return (t - N.a) * ((t - N.b) * (t - N.c)) * N.w; };
    const float Lx = basis(quad_bcast<R>(tx)), Ly = basis(quad_bcast<R>(ty)), Lz = basis(quad_bcast<R>(tz));
    const float A[4] = {Lx * quad_bcast<0>(Ly), Lx * quad_bcast<1>(Ly), Lx * quad_bcast<2>(Ly), Lx * quad_bcast<3>(Ly)};
    const float B = Lz * quad_bcast<R>(b);
#pragma unroll
    for (int j = 0; j < 4; ++j) S.v[0][j] = __builtin_amdgcn_mfma_f32_4x4x1f32(A[j], B, S.v[0][j], 0, 0, 0);
    if constexpr (NS == 2) {
        const float Be = Lz * quad_bcast<R>(be);
#pragma unroll
        for (int j = 0; j < 4; ++j) S.v[NS - 1][j] = __builtin_amdgcn_mfma_f32_4x4x1f32(A[j], Be, S.v[NS - 1][j], 0, 0, 0);
    }
}

// the point that a lane loads: point number i of a run of 64 (HALF: of each half's run of 32) sits in lane i / 16 (i / 8) of quad
// i % 16 (i % 8 of the half), so that a short run needs few steps
template <bool HALF> __device__ inline uint32_t p2m34_point(int lane) {
    return HALF ? 8u * (lane & 3) + ((lane & 31) >> 2) : 16u * (lane & 3) + (lane >> 2);
}

// a run of points, `left` of them or more to come (the same in every lane); points behind the end have b = 0
template <int NS, bool HALF>
__device__ inline void p2m34_run(P2mSums<NS> &S, const QuadNode &N, const float (&x)[3], float b, const double (&ctr)[3],
                                 double inv_half, float kw, bool only, int left) {
    constexpr int PER = HALF ? 8 : 16;
    const float tx = (float)(((double)x[0] - ctr[0]) * inv_half), ty = (float)(((double)x[1] - ctr[1]) * inv_half),
                tz = (float)(((double)x[2] - ctr[2]) * inv_half);
    float be = 0.f;
    if (NS == 2 || only) {
        const float e = __builtin_amdgcn_exp2f(kw * fmaf(tz, tz, fmaf(ty, ty, tx * tx)));
        if (NS == 2) be = b * e;
        else b *= e;
    }
    p2m34_step<NS, 0>(S, N, tx, ty, tz, b, be);
    if (left > PER) p2m34_step<NS, 1>(S, N, tx, ty, tz, b, be);
    if (left > 2 * PER) p2m34_step<NS, 2>(S, N, tx, ty, tz, b, be);
    if (left > 3 * PER) p2m34_step<NS, 3>(S, N, tx, ty, tz, b, be);
}

// sums over the quads of the wavefront (HALF: of each half) to dst (the plain set) and dst + dset: every exchange between lanes
// halves the registers as long as there are some to share out (set, then i2), 16 bytes (i1) a lane at the end
template <int NS, bool HALF> __device__ inline void p2m34_store(const P2mSums<NS> &S, int lane, float *dst, int64_t dset, bool on) {
    auto add32 = [](f4v a, f4v b) __attribute__((always_inline)) {   // lanes 0-31: a, 32-63: b
        f4v r;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const float am = a[m], bm = b[m];
            const auto w = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, am), __builtin_bit_cast(uint32_t, bm), false,
                                                            false);
            r[m] = __builtin_bit_cast(float, (uint32_t)w[0]) + __builtin_bit_cast(float, (uint32_t)w[1]);
        }
        return r;
    };
    auto add16 = [](f4v a, f4v b) __attribute__((always_inline)) {   // even rows of 16 lanes: a, odd rows: b
        f4v r;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const float am = a[m], bm = b[m];
            const auto w = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, am), __builtin_bit_cast(uint32_t, bm), false,
                                                            false);
            r[m] = __builtin_bit_cast(float, (uint32_t)w[0]) + __builtin_bit_cast(float, (uint32_t)w[1]);
        }
        return r;
    };
    auto add8 = [](f4v a, f4v b) __attribute__((always_inline)) {    // lanes 0-7 of a row: a, 8-15: b
        f4v r;
#pragma unroll
        for (int m = 0; m < 4; ++m) r[m] = dpp_into<0x128, 0xC>(a[m], b[m]) + dpp_into<0x128, 0x3>(b[m], a[m]);
        return r;
    };
    auto add4 = [](f4v a, f4v b) __attribute__((always_inline)) {    // even quads of a row: a, odd quads: b
        f4v r;
#pragma unroll
        for (int m = 0; m < 4; ++m) r[m] = dpp_into<0x114, 0xA>(a[m], b[m]) + dpp_into<0x104, 0x5>(b[m], a[m]);
        return r;
    };
    auto fold8 = [](f4v a) __attribute__((always_inline)) {          // lanes 0-7 of a row: a
#pragma unroll
        for (int m = 0; m < 4; ++m) a[m] += dpp_into<0x108, 0xF>(0.f, a[m]);
        return a;
    };
    auto fold4 = [](f4v a) __attribute__((always_inline)) {          // even quads: a (with lane 4 and more to the right)
#pragma unroll
        for (int m = 0; m < 4; ++m) a[m] += dpp_into<0x104, 0xF>(0.f, a[m]);
        return a;
    };
    const auto &v = S.v;
    const int i3 = lane & 3, b2 = (lane >> 2) & 1, b3 = (lane >> 3) & 1, b4 = (lane >> 4) & 1, b5 = lane >> 5;
    f4v r;
    int i2, set = 0;
    if constexpr (HALF && NS == 2) {
        const f4v e = add8(add16(v[0][0], v[1][0]), add16(v[0][2], v[1][2])), o = add8(add16(v[0][1], v[1][1]), add16(v[0][3], v[1][3]));
        r = add4(e, o);
        i2 = 2 * b3 + b2;
        set = b4;
    } else if constexpr (HALF) {
        r = fold4(add8(add16(v[0][0], v[0][2]), add16(v[0][1], v[0][3])));
        i2 = 2 * b4 + b3;
        on = on && b2 == 0;
    } else if constexpr (NS == 2) {
        r = fold4(add8(add16(add32(v[0][0], v[1][0]), add32(v[0][2], v[1][2])), add16(add32(v[0][1], v[1][1]), add32(v[0][3], v[1][3]))));
        i2 = 2 * b4 + b3;
        set = b5;
        on = on && b2 == 0;
    } else {
        r = fold4(fold8(add16(add32(v[0][0], v[0][2]), add32(v[0][1], v[0][3]))));
        i2 = 2 * b5 + b4;
        on = on && b2 == 0 && b3 == 0;
    }
    if (on) *reinterpret_cast<f4v *>(dst + set * dset + 16 * i3 + 4 * i2) = r;
}

template <int NS> __device__ inline void p2m34_zero(P2mSums<NS> &S) {
#pragma unroll
    for (int h = 0; h < NS; ++h)
#pragma unroll
        for (int j = 0; j < 4; ++j) S.v[h][j] = f4v{0.f, 0.f, 0.f, 0.f};
}

// A wavefront per run of up to P2M_CHUNK points of one box (of the chunk list), or, where every box is one run (PAIR), a box
// per HALF wavefront: its sum over the quads covers two boxes at once, and a box of some 40 points fills five steps of 8 instead
// of three of 16.  The loads of two rounds are in flight; they are masked where they are used, and the last rounds load nothing, since a
// branch around a load, or a select right behind it, makes the compiler wait for it there.
// Both sets of 1e7 points in 262144 boxes 100 us (256 by the 64-accumulator form), of 3e6 points in 32768 boxes 27.7 (48), the plain
// set of 2.5e5 points in 4096 boxes 4.2 (9.4).  One pair of boxes to a wavefront: with the loads of four pairs in flight 113,
// 31, 7.5.
template <int NS, bool PERM, bool PAIR>   // PERM: bs is in the caller's order, bs[perm[k]] the right-hand side of point k
__global__ __launch_bounds__(64) void p2m34_kernel(const float *__restrict__ Xs, const float *__restrict__ bs,
                                                   const uint32_t *__restrict__ start, const int32_t *__restrict__ cell,
                                                   const uint32_t *__restrict__ chunk_box,
                                                   const uint32_t *__restrict__ chunk_first, int64_t count, CentreArg C,
                                                   float *__restrict__ W, float *__restrict__ Wpart, WeightedArg A,
                                                   const uint32_t *__restrict__ perm) {
    constexpr int RUN = PAIR ? 32 : 64, AHEAD = 2;
    const int64_t cb = block_index() * (PAIR ? 2 : 1);
    if (cb >= count) return;
    const int lane = threadIdx.x;
    const uint32_t pt = p2m34_point<PAIR>(lane);
    const int64_t c = PAIR ? cb + (lane >> 5) : cb;
    const bool on = c < count;   // PAIR: a box beyond the end repeats the last one, without points
    int64_t a;
    uint32_t k0, k1;
    bool whole = true;
    if constexpr (PAIR) {
        a = on ? c : count - 1;
        k0 = start[a];
        const uint32_t e = start[a + 1];
        k1 = on ? e : k0;
    } else {
        a = (uint32_t)__builtin_amdgcn_readfirstlane(chunk_box[c]);
        const uint32_t c0 = chunk_first[a];
        whole = chunk_first[a + 1] - c0 == 1;
        k0 = start[a] + (uint32_t)(c - c0) * (uint32_t)P2M_CHUNK;
        k1 = min(k0 + (uint32_t)P2M_CHUNK, start[a + 1]);
    }
    double ctr[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) ctr[d] = C.alpha[d] + ((double)cell[a * 3 + d] + 0.5) * C.edge;
    float x[AHEAD][3], bv[AHEAD];
    auto load = [&](int s, uint32_t kb) __attribute__((always_inline)) {   // behind the end: the first point, a valid index
        const uint32_t k = kb + pt, kc = k < k1 ? k : k0;
#pragma unroll
        for (int d = 0; d < 3; ++d) x[s][d] = Xs[(int64_t)kc * 3 + d];
        bv[s] = bs[PERM ? perm[kc] : kc];
    };
#pragma unroll
    for (int s = 0; s < AHEAD; ++s) load(s, k0 + (uint32_t)(RUN * s));
#pragma unroll
    for (int s = 0; s < AHEAD; ++s) {   // else the first loads and the loop's become one, at its top and waited for there
        asm volatile("" : "+v"(bv[s]));
#pragma unroll
        for (int d = 0; d < 3; ++d) asm volatile("" : "+v"(x[s][d]));
    }
    const QuadNode N = quad_node(lane & 3);
    P2mSums<NS> S;
    p2m34_zero(S);
    const int nj = (int)(k1 - k0);   // the wavefront goes on while either half has points left
    int left = PAIR ? max(__builtin_amdgcn_readlane(nj, 0), __builtin_amdgcn_readlane(nj, 32)) : __builtin_amdgcn_readfirstlane(nj);
    uint32_t kb = k0;
    for (; left > RUN * AHEAD; left -= RUN * AHEAD, kb += (uint32_t)(RUN * AHEAD)) {
#pragma unroll
        for (int s = 0; s < AHEAD; ++s) {
            const float xc[3] = {x[s][0], x[s][1], x[s][2]}, b = kb + (uint32_t)(RUN * s) + pt < k1 ? bv[s] : 0.f;
            load(s, kb + (uint32_t)(RUN * (s + AHEAD)));
            p2m34_run<NS, PAIR>(S, N, xc, b, ctr, C.inv_half, A.kw, A.only, RUN);
        }
    }
#pragma unroll
    for (int s = 0; s < AHEAD; ++s) {
        if (left > RUN * s)
            p2m34_run<NS, PAIR>(S, N, x[s], kb + (uint32_t)(RUN * s) + pt < k1 ? bv[s] : 0.f, ctr, C.inv_half, A.kw, A.only, left - RUN * s);
    }
    if (whole) p2m34_store<NS, PAIR>(S, lane, W + a * 64, A.dW, on);
    else p2m34_store<NS, PAIR>(S, lane, Wpart + c * 64, A.dpart, true);
}

constexpr int L2P_NCH = 4;   // chunks per wavefront: their loads are in flight together (a chunk alone is a chain
                             // of dependent loads and the kernel is bound by that latency)
template <bool WEIGHTED, bool PERM>   // Vw: node potentials of the weighted near pairs, evaluated times exp2(kw |u|^2 / (l/2)^2)
__global__ __launch_bounds__(64) void l2p34_kernel(const float *__restrict__ Xs, const uint32_t *__restrict__ start,
                                                   const int32_t *__restrict__ cell,
                                                   const uint64_t *__restrict__ far_ptr,
                                                   const uint32_t *__restrict__ chunk_box,
                                                   const uint32_t *__restrict__ chunk_first, int64_t nchunks, CentreArg C,
                                                   const float *__restrict__ V, const float *base, float *out,
                                                   int one_chunk, const float *__restrict__ Vw, float kw,
                                                   const uint32_t *__restrict__ perm) {
    // out[perm[k]] (PERM; else out[k]) = base (nullptr: zero) + far field
    // one_chunk: every box is a single chunk (chunk index = box rank): two dependent table reads less
    __shared__ __attribute__((aligned(16))) float vbuf[L2P_NCH][64];
    __shared__ __attribute__((aligned(16))) float wbuf[WEIGHTED ? L2P_NCH : 1][64];
    const int64_t c0 = block_index() * L2P_NCH;
    if (c0 >= nchunks) return;
    const int lane = threadIdx.x;
    // chunk j of this wavefront (a chunk beyond the end repeats the last one and is switched off)
    uint32_t a[L2P_NCH], k0[L2P_NCH], k1[L2P_NCH];
    bool on[L2P_NCH];
#pragma unroll
    for (int j = 0; j < L2P_NCH; ++j) {
        const int64_t c = c0 + j < nchunks ? c0 + j : nchunks - 1;
        on[j] = c0 + j < nchunks;
        a[j] = one_chunk ? (uint32_t)c : (uint32_t)__builtin_amdgcn_readfirstlane(chunk_box[c]);
    }
    double ctr[L2P_NCH][3];
    float vrow[L2P_NCH], wrow[L2P_NCH];
#pragma unroll
    for (int j = 0; j < L2P_NCH; ++j) {
        const int64_t c = c0 + j < nchunks ? c0 + j : nchunks - 1;
        // far_ptr given: skip boxes without far partner at this depth (V_p is zero); nullptr: V holds the
        // potentials accumulated over all depths and every box is evaluated
        if (far_ptr && far_ptr[a[j] + 1] == far_ptr[a[j]]) on[j] = false;
        const uint32_t ci = one_chunk ? 0u : (uint32_t)(c - chunk_first[a[j]]);
        k0[j] = start[a[j]] + ci * (uint32_t)P2M_CHUNK;     // a point of the box: always a valid index
        k1[j] = min(k0[j] + (uint32_t)P2M_CHUNK, start[a[j] + 1]);
        if (!on[j]) k1[j] = k0[j];
#pragma unroll
        for (int d = 0; d < 3; ++d) ctr[j][d] = C.alpha[d] + ((double)cell[(int64_t)a[j] * 3 + d] + 0.5) * C.edge;
        vrow[j] = V[(int64_t)a[j] * 64 + lane];             // the node potentials of the box, one per lane
        if constexpr (WEIGHTED) wrow[j] = Vw[(int64_t)a[j] * 64 + lane];
    }
    // The node potentials reach the lanes as LDS broadcasts (every lane reads the same address);
    // as scalar operands they arrive in four dependent batches per box.
#pragma unroll
    for (int j = 0; j < L2P_NCH; ++j) {
        vbuf[j][lane] = vrow[j];
        if constexpr (WEIGHTED) wbuf[j][lane] = wrow[j];
    }
    __builtin_amdgcn_wave_barrier();   // one wavefront per block; its LDS operations complete in order
    // one run of 64 points of a chunk: y += sum_i L_i(t) V[i], nested over the dimensions
    auto run = [&](int j, bool live, uint32_t k, const float (&x)[3], float yold) {
        float Lx[4], Ly[4], Lz[4];
        const float u2 = weights34(x, ctr[j], C.inv_half, Lx, Ly, Lz);
        auto sum = [&](const float *vb) __attribute__((always_inline)) {
            float y = 0.f;
#pragma unroll
            for (int i3 = 0; i3 < 4; ++i3) {
                float sy = 0.f;
#pragma unroll
                for (int i2 = 0; i2 < 4; ++i2) {
                    const float4 v = *reinterpret_cast<const float4 *>(vb + 4 * i2 + 16 * i3);
                    float sx = Lx[0] * v.x;
                    sx = fmaf(Lx[1], v.y, sx);
                    sx = fmaf(Lx[2], v.z, sx);
                    sx = fmaf(Lx[3], v.w, sx);
                    sy = fmaf(Ly[i2], sx, sy);
                }
                y = fmaf(Lz[i3], sy, y);
            }
            return y;
        };
        float y = sum(vbuf[j]);
        if constexpr (WEIGHTED) __builtin_amdgcn_sched_barrier(0);   // one set of potentials at a time in registers: 125, not 176
        if constexpr (WEIGHTED) y = fmaf(__builtin_amdgcn_exp2f(kw * u2), sum(wbuf[WEIGHTED ? j : 0]), y);
        if (live) out[k] = yold + y;
    };
    // Loads are unconditional with the index of a lane beyond the chunk clamped to the chunk's first
    // point (a branch around them would make the compiler wait for every load on its own); the first
    // run of every chunk has all its loads issued before any is used, then what is left of the chunks.
    float x[L2P_NCH][3], yold[L2P_NCH];
    bool live[L2P_NCH];
    uint32_t kk[L2P_NCH], ko[L2P_NCH];
#pragma unroll
    for (int j = 0; j < L2P_NCH; ++j) {
        const uint32_t k = k0[j] + lane;
        live[j] = k < k1[j];
        kk[j] = live[j] ? k : k0[j];
#pragma unroll
        for (int d = 0; d < 3; ++d) x[j][d] = Xs[(int64_t)kk[j] * 3 + d];
        yold[j] = base ? base[kk[j]] : 0.f;
        ko[j] = PERM ? perm[kk[j]] : kk[j];
    }
#pragma unroll
    for (int j = 0; j < L2P_NCH; ++j) {
        run(j, live[j], ko[j], x[j], yold[j]);
        if constexpr (WEIGHTED) __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int j = 0; j < L2P_NCH; ++j) {
        for (uint32_t kb = k0[j] + 64; kb < k1[j]; kb += 64) {
            const uint32_t k = kb + lane;
            const bool lv = k < k1[j];
            const uint32_t kc = lv ? k : k0[j];
            float xr[3];
#pragma unroll
            for (int d = 0; d < 3; ++d) xr[d] = Xs[(int64_t)kc * 3 + d];
            run(j, lv, PERM ? perm[kc] : kc, xr, base ? base[kc] : 0.f);
        }
    }
}

// P2M and L2P of boxes with thousands of points: a wavefront per run of up to P2M_LONG points of one box.  L2P above starts every
// 256 points with the 64 potentials in LDS; here that is 2 % of the work.  P2M above has few registers to sum over the lanes, and
// pays with every factor evaluated four times; with a lane per point and 64 sums in it the sum over the lanes is a few percent of the
// work here, and the multiply-adds cost less than the products of both (two sets of 1e9 points with fp32 sums over a run: 6.0 ms, on
// the matrix cores 6.6; 1e8 points, one set: 0.37, 0.52).  The loads of four rounds are in flight.  WEIGHTED: both sets of node weights / node
// potentials (the weighted near pairs) from one reading of the points.
constexpr int TR_STRIDE = 36;  // floats per lane row in the LDS transpose of 32 accumulators (16-byte aligned, bank-shifted)
constexpr int LONG_AHEAD = 4;
// Points of a run whose node sums stay in fp32: 16 to a lane, then fp64.  With all 2048 points of a run in fp32, over the lanes too,
// sums that cancel were off by three times as much as with runs of 256 points (4.8e-9 of the norm of the weights,
// 1.5e-9; now 1.2e-9).  1e9 points, both sets of weights: 6.28 -> 6.64 ms; 1e8 points, one set, 0.37 as before.
constexpr int LONG_FP32 = 1024;
static_assert(LONG_FP32 % (64 * LONG_AHEAD) == 0, "whole rounds of loads");
template <bool WEIGHTED>
__global__ __launch_bounds__(64) void p2m34_long_kernel(const float *__restrict__ Xs, const float *__restrict__ bs,
                                                        const uint32_t *__restrict__ start, const int32_t *__restrict__ cell,
                                                        const uint32_t *__restrict__ chunk_box,
                                                        const uint32_t *__restrict__ chunk_first, int64_t nchunks,
                                                        CentreArg C, float *__restrict__ W, float *__restrict__ Wpart,
                                                        WeightedArg A) {
    constexpr int NS = WEIGHTED ? 2 : 1;
    __shared__ __attribute__((aligned(16))) float tr[64 * TR_STRIDE];
    const int64_t c = block_index();
    if (c >= nchunks) return;
    const int lane = threadIdx.x;
    const uint32_t a = (uint32_t)__builtin_amdgcn_readfirstlane(chunk_box[c]);
    const uint32_t c0 = chunk_first[a], c1 = chunk_first[a + 1];
    const uint32_t k0 = start[a] + (uint32_t)(c - c0) * (uint32_t)P2M_LONG;
    const uint32_t k1 = min(k0 + (uint32_t)P2M_LONG, start[a + 1]);
    double ctr[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) ctr[d] = C.alpha[d] + ((double)cell[(int64_t)a * 3 + d] + 0.5) * C.edge;
    float x[LONG_AHEAD][3], bv[LONG_AHEAD];
    // unconditional loads, the index behind the end clamped to the last point and its weight zero
    auto load = [&](int s, uint32_t kb) __attribute__((always_inline)) {
        const uint32_t k = kb + (uint32_t)lane, kc = min(k, k1 - 1u);
#pragma unroll
        for (int d = 0; d < 3; ++d) x[s][d] = Xs[(int64_t)kc * 3 + d];
        const float b = bs[kc];
        bv[s] = k < k1 ? b : 0.f;
    };
#pragma unroll
    for (int s = 0; s < LONG_AHEAD; ++s) load(s, k0 + 64u * s);
    // sums over the lanes so far: node 32 q + i in lanes i and 32 + i, half of the rows each
    const int i = lane & 31, part = lane >> 5;
    double sum[NS][2];
#pragma unroll
    for (int h = 0; h < NS; ++h) sum[h][0] = sum[h][1] = 0.0;
    uint32_t kb = k0;
    do {
        float acc[NS][64];
#pragma unroll
        for (int h = 0; h < NS; ++h)
#pragma unroll
            for (int q = 0; q < 64; ++q) acc[h][q] = 0.f;
        const uint32_t ke = min(kb + (uint32_t)LONG_FP32, k1);
        for (; kb < ke; kb += 64u * LONG_AHEAD) {
#pragma unroll
            for (int s = 0; s < LONG_AHEAD; ++s) {
                float Lx[4], Ly[4], Lz[4];
                const float u2 = weights34(x[s], ctr, C.inv_half, Lx, Ly, Lz);
                const float b = bv[s];
                load(s, kb + 64u * (s + LONG_AHEAD));
                float xy[16];
#pragma unroll
                for (int i2 = 0; i2 < 4; ++i2)
#pragma unroll
                    for (int i1 = 0; i1 < 4; ++i1) xy[i1 + 4 * i2] = Lx[i1] * Ly[i2];
#pragma unroll
                for (int h = 0; h < NS; ++h) {
                    const float bh = h ? b * __builtin_amdgcn_exp2f(A.kw * u2) : b;
#pragma unroll
                    for (int i3 = 0; i3 < 4; ++i3) {
                        const float zb = Lz[i3] * bh;
#pragma unroll
                        for (int q = 0; q < 16; ++q) acc[h][q + 16 * i3] = fmaf(xy[q], zb, acc[h][q + 16 * i3]);
                    }
                }
            }
        }
        // sum over the lanes, 32 nodes at a time: a lane writes its row, lane (i, part) adds rows 32 part .. 32 part + 31 of column i
#pragma unroll
        for (int h = 0; h < NS; ++h)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                __syncthreads();
#pragma unroll
                for (int g = 0; g < 8; ++g)
                    *reinterpret_cast<float4 *>(&tr[lane * TR_STRIDE + 4 * g]) = make_float4(
                        acc[h][32 * q + 4 * g], acc[h][32 * q + 4 * g + 1], acc[h][32 * q + 4 * g + 2], acc[h][32 * q + 4 * g + 3]);
                __syncthreads();
                double s0 = 0.0, s1 = 0.0;
#pragma unroll
                for (int row = 0; row < 32; row += 2) {
                    s0 += (double)tr[(32 * part + row) * TR_STRIDE + i];
                    s1 += (double)tr[(32 * part + row + 1) * TR_STRIDE + i];
                }
                sum[h][q] += s0 + s1;
            }
    } while (kb < k1);
#pragma unroll
    for (int h = 0; h < NS; ++h) {
        float *dst = c1 - c0 == 1 ? W + h * A.dW + (int64_t)a * 64 : Wpart + h * A.dpart + c * 64;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const double t = sum[h][q] + __shfl_xor(sum[h][q], 32, 64);
            if (part == 0) dst[32 * q + i] = (float)t;
        }
    }
}

// out = base (nullptr: zero) + far field; far_ptr as in l2p34_kernel
template <bool WEIGHTED>
__global__ __launch_bounds__(64) void l2p34_long_kernel(const float *__restrict__ Xs, const uint32_t *__restrict__ start,
                                                        const int32_t *__restrict__ cell,
                                                        const uint64_t *__restrict__ far_ptr,
                                                        const uint32_t *__restrict__ chunk_box,
                                                        const uint32_t *__restrict__ chunk_first, int64_t nchunks,
                                                        CentreArg C, const float *__restrict__ V, const float *base,
                                                        float *out, const float *__restrict__ Vw, float kw) {
    constexpr int NS = WEIGHTED ? 2 : 1;
    __shared__ __attribute__((aligned(16))) float vb[NS][64];
    const int64_t c = block_index();
    if (c >= nchunks) return;
    const int lane = threadIdx.x;
    const uint32_t a = (uint32_t)__builtin_amdgcn_readfirstlane(chunk_box[c]);
    if (far_ptr && far_ptr[a + 1] == far_ptr[a]) return;
    const uint32_t k0 = start[a] + (uint32_t)(c - chunk_first[a]) * (uint32_t)P2M_LONG;
    const uint32_t k1 = min(k0 + (uint32_t)P2M_LONG, start[a + 1]);
    double ctr[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) ctr[d] = C.alpha[d] + ((double)cell[(int64_t)a * 3 + d] + 0.5) * C.edge;
    vb[0][lane] = V[(int64_t)a * 64 + lane];
    if constexpr (WEIGHTED) vb[NS - 1][lane] = Vw[(int64_t)a * 64 + lane];
    __syncthreads();
    // the potentials of the box in registers of every lane (multiply-adds on registers alone issue fastest)
    float v[NS][64];
#pragma unroll
    for (int h = 0; h < NS; ++h)
#pragma unroll
        for (int q = 0; q < 64; ++q) {
            v[h][q] = vb[h][q];
            asm volatile("" : "+v"(v[h][q]));
        }
    float x[LONG_AHEAD][3], old[LONG_AHEAD];
    auto load = [&](int s, uint32_t kb) __attribute__((always_inline)) {
        const uint32_t kc = min(kb + (uint32_t)lane, k1 - 1u);
#pragma unroll
        for (int d = 0; d < 3; ++d) x[s][d] = Xs[(int64_t)kc * 3 + d];
        old[s] = base ? base[kc] : 0.f;
    };
#pragma unroll
    for (int s = 0; s < LONG_AHEAD; ++s) load(s, k0 + 64u * s);
    for (uint32_t kb = k0; kb < k1; kb += 64u * LONG_AHEAD) {
#pragma unroll
        for (int s = 0; s < LONG_AHEAD; ++s) {
            float Lx[4], Ly[4], Lz[4];
            const float u2 = weights34(x[s], ctr, C.inv_half, Lx, Ly, Lz);
            const float yold = old[s];
            // (base may be out: the entry loaded here is stored by a later round of this lane only)
            load(s, kb + 64u * (s + LONG_AHEAD));
            float y[NS];
#pragma unroll
            for (int h = 0; h < NS; ++h) {
                y[h] = 0.f;
#pragma unroll
                for (int i3 = 0; i3 < 4; ++i3) {
                    float sy = 0.f;
#pragma unroll
                    for (int i2 = 0; i2 < 4; ++i2) {
                        float sx = Lx[0] * v[h][4 * i2 + 16 * i3];
#pragma unroll
                        for (int i1 = 1; i1 < 4; ++i1) sx = fmaf(Lx[i1], v[h][i1 + 4 * i2 + 16 * i3], sx);
                        sy = fmaf(Ly[i2], sx, sy);
                    }
                    y[h] = fmaf(Lz[i3], sy, y[h]);
                }
            }
            if constexpr (WEIGHTED) y[0] = fmaf(__builtin_amdgcn_exp2f(kw * u2), y[NS - 1], y[0]);
            const uint32_t k = kb + 64u * s + (uint32_t)lane;
            if (k < k1) out[k] = yold + y[0];
        }
    }
}

// ------------------------------------------------------------------------------------
// Node weights and node potentials between depths (D = 3, 4 nodes per dimension).
// The basis functions of a parent box are polynomials of degree 3 per coordinate, and the
// 4-node interpolant of a child box reproduces such polynomials exactly.  Hence
//   W_parent[i] = sum_children sum_k L^parent_i(s^child_k) W_child[k]           (upward)
// equals the P2M sum over the parent's points, and evaluating a parent's potential at a
// child's nodes,  V_child[k] += sum_i L^parent_i(s^child_k) V_parent[i]          (downward),
// followed by ONE L2P at the last depth equals the per-depth L2P sums -- both up to
// rounding.  This replaces the streaming passes over all points at every depth (Fig. 4
// steps 1 and 3 per depth) by one pass each at the last depth.
// In parent coordinates the child's node k sits at (s_k -+ 1)/2 (lower / upper half), so the
// 64 x 64 transfer matrix is a tensor product of three 4 x 4 matrices T1[half][i][k].
// ------------------------------------------------------------------------------------
struct TransferArg { float t[2][4][4]; };   // t[half][i][k] = L_i((s_k + (half ? 1 : -1)) / 2)

static TransferArg make_transfer() {
    TransferArg T{};
    double s[4];
    for (int i = 0; i < 4; ++i) s[i] = std::cos((double)i * M_PI / 3.0);
    for (int h = 0; h < 2; ++h)
        for (int k = 0; k < 4; ++k) {
            const double tp = 0.5 * (s[k] + (h ? 1.0 : -1.0));
            for (int i = 0; i < 4; ++i) {
                double num = 1.0, den = 1.0;
                for (int j = 0; j < 4; ++j)
                    if (j != i) { num *= tp - s[j]; den *= s[i] - s[j]; }
                T.t[h][i][k] = (float)(num / den);
            }
        }
    return T;
}

// Both transfers run one wavefront per PARENT with lane = node (ix + 4 iy + 16 iz) and apply the
// three 4 x 4 factors one dimension at a time, 4 multiply-adds each: the other three entries of a
// fibre sit in the lane's quad (x: DPP quad permutations), in its row of 16 lanes (y: DPP row
// rotations by 4, 8, 12) and in the other rows (z: ds_bpermute).  f[k] is the factor entry for the
// fibre element k places further on (cyclically).  All rows of the (at most 8) children are loaded
// before the first is used: one round of memory latency per parent.
template <int CTRL>
__device__ inline float dpp_take(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}

__device__ inline float fibre_x(float v, const float (&f)[4]) {
    float o = f[0] * v;
    o = fmaf(f[1], dpp_take<0x39>(v), o);    // quad_perm [1,2,3,0]
    o = fmaf(f[2], dpp_take<0x4E>(v), o);    // quad_perm [2,3,0,1]
    return fmaf(f[3], dpp_take<0x93>(v), o); // quad_perm [3,0,1,2]
}

__device__ inline float fibre_y(float v, const float (&f)[4]) {
    float o = f[0] * v;
    o = fmaf(f[1], dpp_take<0x12C>(v), o);    // row_ror:12 = the lane 4 further on in the row of 16
    o = fmaf(f[2], dpp_take<0x128>(v), o);    // row_ror:8
    return fmaf(f[3], dpp_take<0x124>(v), o); // row_ror:4
}

__device__ inline float fibre_z(float v, const float (&f)[4], int lane) {
    float o = f[0] * v;
#pragma unroll
    for (int k = 1; k < 4; ++k) o = fmaf(f[k], __shfl(v, (lane + 16 * k) & 63, 64), o);
    return o;
}

// W_parent[i] = sum over children, sum_k T[half][i][k] (per dimension) W_child[k]
__global__ __launch_bounds__(64) void m2m34_kernel(const uint32_t *__restrict__ cstart,
                                                   const uint32_t *__restrict__ child_key, int64_t nparents,
                                                   const float *__restrict__ T, const float *__restrict__ Wchild,
                                                   float *__restrict__ Wparent) {
    __shared__ float tl[32];
    const int64_t P = block_index();
    if (P >= nparents) return;
    const int lane = threadIdx.x, ix = lane & 3, iy = (lane >> 2) & 3, iz = lane >> 4;
    const uint32_t c0 = cstart[P];
    const int nc = min((int)(cstart[P + 1] - c0), 8);   // a box has at most 2^3 children
    if (nc <= 0) {                                      // (boxes are never empty: cannot happen)
        Wparent[P * 64 + lane] = 0.f;
        return;
    }
    if (lane < 32) tl[lane] = T[lane];
    const uint32_t key = child_key[c0 + (uint32_t)min(lane, nc - 1)];
    float w[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) w[j] = Wchild[(int64_t)(c0 + (uint32_t)min(j, nc - 1)) * 64 + lane];
    __syncthreads();
    float f[3][2][4];   // [dimension][half][k]: T[half][i][(i + k) & 3] with i the lane's node index in that dimension
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            f[0][h][k] = tl[h * 16 + ix * 4 + ((ix + k) & 3)];
            f[1][h][k] = tl[h * 16 + iy * 4 + ((iy + k) & 3)];
            f[2][h][k] = tl[h * 16 + iz * 4 + ((iz + k) & 3)];
        }
    float acc = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if (j < nc) {
            const uint32_t par = (uint32_t)__builtin_amdgcn_readlane((int)key, j) & 7u;   // bit d = upper half along d
            float g[3][4];
#pragma unroll
            for (int d = 0; d < 3; ++d)
#pragma unroll
                for (int k = 0; k < 4; ++k) g[d][k] = (par >> d) & 1u ? f[d][1][k] : f[d][0][k];
            acc += fibre_z(fibre_y(fibre_x(w[j], g[0]), g[1]), g[2], lane);
        }
    }
    Wparent[P * 64 + lane] = acc;
}

// V_child[k] += sum_i T[half][i][k] (per dimension) V_parent[i], for every child of the parent
__global__ __launch_bounds__(64) void l2l34_kernel(const uint32_t *__restrict__ cstart,
                                                   const uint32_t *__restrict__ child_key, int64_t nparents,
                                                   const float *__restrict__ T, const float *__restrict__ Vparent,
                                                   float *__restrict__ Vchild) {
    __shared__ float tl[32];
    const int64_t P = block_index();
    if (P >= nparents) return;
    const int lane = threadIdx.x, kx = lane & 3, ky = (lane >> 2) & 3, kz = lane >> 4;
    const uint32_t c0 = cstart[P];
    const int nc = min((int)(cstart[P + 1] - c0), 8);
    if (nc <= 0) return;
    if (lane < 32) tl[lane] = T[lane];
    const uint32_t key = child_key[c0 + (uint32_t)min(lane, nc - 1)];
    const float vp = Vparent[P * 64 + lane];
    float vc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) vc[j] = Vchild[(int64_t)(c0 + (uint32_t)min(j, nc - 1)) * 64 + lane];
    __syncthreads();
    float f[3][2][4];   // [dimension][half][j]: T[half][(k + j) & 3][k] with k the lane's node index in that dimension
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            f[0][h][j] = tl[h * 16 + ((kx + j) & 3) * 4 + kx];
            f[1][h][j] = tl[h * 16 + ((ky + j) & 3) * 4 + ky];
            f[2][h][j] = tl[h * 16 + ((kz + j) & 3) * 4 + kz];
        }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if (j < nc) {
            const uint32_t par = (uint32_t)__builtin_amdgcn_readlane((int)key, j) & 7u;
            float g[3][4];
#pragma unroll
            for (int d = 0; d < 3; ++d)
#pragma unroll
                for (int k = 0; k < 4; ++k) g[d][k] = (par >> d) & 1u ? f[d][1][k] : f[d][0][k];
            Vchild[(int64_t)(c0 + (uint32_t)j) * 64 + lane] = vc[j] + fibre_z(fibre_y(fibre_x(vp, g[0]), g[1]), g[2], lane);
        }
    }
}

// ------------------------------------------------------------------------------------
// M2L for any D and node count (Fig. 4 step 2), V_t += K(s^t, s^q) W_q over the far row of t.
// The Gaussian is a product over dimensions, and so is the tensor grid of nodes, hence the
// node-to-node matrix of a far pair with cell offset o is a Kronecker product,
//   K = G_{o_D} x ... x G_{o_1},   G_o[i][j] = exp(-(l/2)^2 (2 o + s_j - s_i)^2 / (2 gamma^2)),
// of p x p matrices that depend on the offset in one dimension only.  It is applied one
// dimension at a time (D passes of r p multiply-adds instead of r^2 kernel values): the same
// sums as the dense product, in another order.  The table G[o + omax][i][j] is built in fp64
// per depth at plan time.
// Boxes with more than 32 fibres (a fibre = the p entries along one dimension) take
// m2l_kron_grouped_kernel, which also nests the sum over the far partners over the dimensions;
// boxes with fewer take m2l_kron_small_kernel, several far pairs per wavefront.
// For two point sets the grids are shifted by u_d box edges in dimension d, so the factor of
// dimension d depends on o + u_d: the table is kept per dimension, G[d][o - omin_d][i][j] with
// G = exp(-(l/2)^2 (2 (o + u_d) + s_j - s_i)^2 / (2 gamma^2)), `no` offsets per dimension
// (cellT: cells of the target boxes, cellS: of the source boxes; u = 0 and equal tables for one set).
// ------------------------------------------------------------------------------------
struct KronShape {
    int omin[F3M_MAX_DIM];   // smallest tabulated offset (source cell - target cell) per dimension
    int no;                  // tabulated offsets per dimension
};

// ---- far rows in the order of the row-major cell index ------------------------------------------
// The grouped M2L below shares work between far partners whose cells differ in the leading dimensions
// only, so it wants the partners of a target ordered by (c_{D-1}, ..., c_1, c_0), most significant first:
// ascending row-major index beta = sum_d c_d 2^(depth d) (the box index of Sec. 4.2).  The far lists are
// stored ascending in the interleaved key; far_ord holds every row once more in beta order.  A row is
// sorted in pieces of at most FO_CH entries (bitonic network in LDS); the M2L is correct for any
// order, a piece boundary only costs it a few shared sums.
constexpr int FO_CH = 8192;    // 64 KB of keys: two workgroups per compute unit
constexpr int FO_NT = 512;
__global__ __launch_bounds__(FO_NT) void far_order_kernel(const uint64_t *__restrict__ far_ptr,
                                                         const uint32_t *__restrict__ far_col,
                                                         const int32_t *__restrict__ cellS, int D, int depth, int64_t nb,
                                                         uint32_t *__restrict__ far_ord) {
    __shared__ uint64_t key[FO_CH];
    const int64_t a = block_index();
    if (a >= nb) return;
    const int tid = threadIdx.x;
    const uint64_t e0 = far_ptr[a], e1 = far_ptr[a + 1];
    for (uint64_t c0 = e0; c0 < e1; c0 += FO_CH) {
        const int len = (int)(e1 - c0 < (uint64_t)FO_CH ? e1 - c0 : (uint64_t)FO_CH);
        int n2 = 2;
        while (n2 < len) n2 <<= 1;
        for (int i = tid; i < n2; i += FO_NT) {
            uint64_t k = ~0ull;
            if (i < len) {
                const uint32_t q = far_col[c0 + i];
                uint64_t beta = 0;
                for (int d = 0; d < D; ++d) beta |= (uint64_t)(uint32_t)cellS[(int64_t)q * D + d] << (depth * d);
                k = (beta << 32) | q;
            }
            key[i] = k;
        }
        __syncthreads();
        for (int k = 2; k <= n2; k <<= 1)
            for (int j = k >> 1; j > 0; j >>= 1) {
                for (int i = tid; i < n2; i += FO_NT) {
                    const int ixj = i ^ j;
                    if (ixj > i) {
                        const uint64_t x = key[i], y = key[ixj];
                        if ((x > y) == ((i & k) == 0)) {
                            key[i] = y;
                            key[ixj] = x;
                        }
                    }
                }
                __syncthreads();
            }
        for (int i = tid; i < len; i += FO_NT) far_ord[c0 + i] = (uint32_t)key[i];
        __syncthreads();
    }
}

constexpr int ipow_c(int p, int d) { return d <= 0 ? 1 : p * ipow_c(p, d - 1); }

// Grouped M2L: the far partners q of a target t are taken in the order of far_ord, and the sum
//   V_t = sum_q (G_{o_{D-1}(q)} x ... x G_{o_0(q)}) W_q
// is nested over the dimensions,
//   V_t = sum_{o_{D-1}} G_{o_{D-1}} [ sum_{o_{D-2}} G_{o_{D-2}} [ ... sum_{o_0} G_{o_0} W_q ] ]:
// level d keeps a partial sum S_d over the partners that agree in (o_{d+1}, ..., o_{D-1}); when the next
// partner differs in one of those, S_d is multiplied by the factor of dimension d+1 and added to S_{d+1}
// ("flush").  Every partner costs one factor (dimension 0, on data straight from global memory), every
// group of a level one more, instead of D factors per partner: the same sums as the dense products, in
// another order.  For partners in any other order the result is the same (more flushes).
// One workgroup of 256 threads per target; a thread owns up to NFL fibres of every dimension (a fibre =
// the p entries along one dimension) and keeps S_d of its fibres of dimension d in registers; a flush
// passes S_d through LDS (node layout) to the owners of the fibres of dimension d+1, alternating
// between two buffers so that one barrier per flush is enough.
template <int PN, int DD>
__global__ __launch_bounds__(256) void m2l_kron_grouped_kernel(const int32_t *__restrict__ cellT,
                                                               const int32_t *__restrict__ cellS,
                                                               const uint64_t *__restrict__ far_ptr,
                                                               const uint32_t *__restrict__ far_ord, int64_t nb,
                                                               const float *__restrict__ G, KronShape S,
                                                               const float *__restrict__ W, float *__restrict__ V) {
    constexpr int R = ipow_c(PN, DD), NFIB = R / PN, NFL = (NFIB + 255) / 256;
    __shared__ float buf[2][R];
    const int64_t a = block_index();
    if (a >= nb) return;
    const uint64_t e0 = far_ptr[a], e1 = far_ptr[a + 1];
    if (e0 == e1) return;   // no far partner at this depth: the row of V is left alone
    const int tid = threadIdx.x;
    float acc[DD][NFL][PN];
#pragma unroll
    for (int d = 0; d < DD; ++d)
#pragma unroll
        for (int k = 0; k < NFL; ++k)
#pragma unroll
            for (int i = 0; i < PN; ++i) acc[d][k][i] = 0.f;
    int ca[DD], prev[DD];
#pragma unroll
    for (int d = 0; d < DD; ++d) ca[d] = cellT[a * DD + d];
    // factor matrix of dimension d for a source cell coordinate (the index is clamped to the table:
    // every far pair lies inside it by construction)
    auto factor = [&](int d, int cs) __attribute__((always_inline)) {
        int k = cs - ca[d] - S.omin[d];
        k = k < 0 ? 0 : (k >= S.no ? S.no - 1 : k);
        return G + ((int64_t)d * S.no + k) * (PN * PN);
    };
    int flip = 0;
    // S_d, times the factor of dimension d+1 for source cell coordinate cs1, is added to S_{d+1}; S_d = 0
    auto flush = [&](auto dconst, int cs1) __attribute__((always_inline)) {
        constexpr int d = decltype(dconst)::value;
        constexpr int sd = ipow_c(PN, d), sd1 = sd * PN;
        float *B = buf[flip];
        flip ^= 1;
#pragma unroll
        for (int k = 0; k < NFL; ++k) {
            const int f = tid + 256 * k;
            if (f < NFIB) {
                const int hi = f / sd, base = hi * sd1 + (f - hi * sd);
#pragma unroll
                for (int j = 0; j < PN; ++j) {
                    B[base + j * sd] = acc[d][k][j];
                    acc[d][k][j] = 0.f;
                }
            }
        }
        __syncthreads();
        const float *__restrict__ g = factor(d + 1, cs1);
#pragma unroll
        for (int k = 0; k < NFL; ++k) {
            const int f = tid + 256 * k;
            if (f < NFIB) {
                const int hi = f / sd1, base = hi * sd1 * PN + (f - hi * sd1);
                float in[PN];
#pragma unroll
                for (int j = 0; j < PN; ++j) in[j] = B[base + j * sd1];
#pragma unroll
                for (int i = 0; i < PN; ++i) {
                    float t = acc[d + 1][k][i];
#pragma unroll
                    for (int j = 0; j < PN; ++j) t = fmaf(g[i * PN + j], in[j], t);
                    acc[d + 1][k][i] = t;
                }
            }
        }
    };
    // the levels below `upto` end their groups (upto = DD: all of them)
    auto flush_below = [&](int upto) __attribute__((always_inline)) {
        if constexpr (DD > 1) { if (upto > 0) flush(std::integral_constant<int, 0>{}, prev[1]); }
        if constexpr (DD > 2) { if (upto > 1) flush(std::integral_constant<int, 1>{}, prev[2]); }
        if constexpr (DD > 3) { if (upto > 2) flush(std::integral_constant<int, 2>{}, prev[3]); }
        if constexpr (DD > 4) { if (upto > 3) flush(std::integral_constant<int, 3>{}, prev[4]); }
        if constexpr (DD > 5) { if (upto > 4) flush(std::integral_constant<int, 4>{}, prev[5]); }
        if constexpr (DD > 6) { if (upto > 5) flush(std::integral_constant<int, 5>{}, prev[6]); }
    };
    // the fibres of dimension 0 of a partner's node weights: p consecutive floats each
    auto load = [&](uint32_t q, float (&w)[NFL][PN]) __attribute__((always_inline)) {
        const float *Wq = W + (int64_t)q * R;
#pragma unroll
        for (int k = 0; k < NFL; ++k) {
            const int f = tid + 256 * k;
#pragma unroll
            for (int j = 0; j < PN; ++j) w[k][j] = f < NFIB ? Wq[f * PN + j] : 0.f;
        }
    };
    float wn[NFL][PN];
    uint32_t qn = __builtin_amdgcn_readfirstlane(far_ord[e0]);
    load(qn, wn);
    for (uint64_t e = e0; e < e1; ++e) {
        const uint32_t q = qn;
        float wc[NFL][PN];
#pragma unroll
        for (int k = 0; k < NFL; ++k)
#pragma unroll
            for (int j = 0; j < PN; ++j) wc[k][j] = wn[k][j];
        if (e + 1 < e1) {   // the next partner's weights are on their way during this one's sums
            qn = __builtin_amdgcn_readfirstlane(far_ord[e + 1]);
            load(qn, wn);
        }
        int cs[DD];
#pragma unroll
        for (int d = 0; d < DD; ++d) cs[d] = __builtin_amdgcn_readfirstlane(cellS[(int64_t)q * DD + d]);
        if (e > e0) {
            int upto = 0;   // one more than the highest dimension >= 1 in which this partner differs from the last
#pragma unroll
            for (int d = 1; d < DD; ++d) upto = cs[d] != prev[d] ? d : upto;
            flush_below(upto);
        }
        const float *__restrict__ g = factor(0, cs[0]);
#pragma unroll
        for (int k = 0; k < NFL; ++k)
#pragma unroll
            for (int i = 0; i < PN; ++i) {
                float t = acc[0][k][i];
#pragma unroll
                for (int j = 0; j < PN; ++j) t = fmaf(g[i * PN + j], wc[k][j], t);
                acc[0][k][i] = t;
            }
#pragma unroll
        for (int d = 0; d < DD; ++d) prev[d] = cs[d];
    }
    flush_below(DD);
    // S_{D-1} is the row of V: node (fibre f of the last dimension, entry j) = j r/p + f
    float *Va = V + a * R;
#pragma unroll
    for (int k = 0; k < NFL; ++k) {
        const int f = tid + 256 * k;
        if (f < NFIB) {
#pragma unroll
            for (int j = 0; j < PN; ++j) Va[j * NFIB + f] = acc[DD - 1][k][j];
        }
    }
}

// The same for boxes with few fibres (r/p <= 32, e.g. D = 3 with 4 nodes per dimension: 16): one
// fibre per lane would leave most of the wavefront idle, so the lanes form 64 / (r/p) groups and
// every group takes its own far pair of the row (pairs e0 + g, e0 + g + groups, ...), with its
// own LDS buffer and its own accumulators.  The factor matrices then differ between the groups,
// so the table of the depth is staged in LDS once per target.  At the end the accumulators of the
// groups are added in a fixed order.
template <int PN>
__global__ __launch_bounds__(64) void m2l_kron_small_kernel(const int32_t *__restrict__ cellT,
                                                            const int32_t *__restrict__ cellS,
                                                            const uint64_t *__restrict__ far_ptr,
                                                            const uint32_t *__restrict__ far_col, int64_t nb, int D,
                                                            int r, const float *__restrict__ G, KronShape S,
                                                            const float *__restrict__ W, float *__restrict__ V) {
    extern __shared__ float lds[];   // [groups][r] buffers, then the table [D][no][PN][PN]
    const int64_t a = block_index();
    if (a >= nb) return;
    const uint64_t e0 = far_ptr[a], e1 = far_ptr[a + 1];
    if (e0 == e1) return;
    const int lane = threadIdx.x;
    const int nfib = r / PN;
    const int ngrp = 64 / nfib;
    const int g = lane / nfib, f = lane - g * nfib;
    const bool act = g < ngrp;
    float *buf = lds + (act ? g : 0) * r;
    float *tab = lds + ngrp * r;
    const int tab_n = D * S.no * PN * PN;
    for (int i = lane; i < tab_n; i += 64) tab[i] = G[i];
    float acc[PN];
#pragma unroll
    for (int i = 0; i < PN; ++i) acc[i] = 0.f;
    int ca[F3M_MAX_DIM];
    for (int d = 0; d < D; ++d) ca[d] = cellT[a * D + d];
    auto factor = [&](int d, int cs) {
        int k = cs - ca[d] - S.omin[d];
        k = k < 0 ? 0 : (k >= S.no ? S.no - 1 : k);
        return tab + (d * S.no + k) * (PN * PN);
    };
    auto apply = [&](const float *gm, const float (&in)[PN], float (&out)[PN]) {
#pragma unroll
        for (int i = 0; i < PN; ++i) {
            float t = 0.f;
#pragma unroll
            for (int j = 0; j < PN; ++j) t = fmaf(gm[i * PN + j], in[j], t);
            out[i] = t;
        }
    };
    for (uint64_t e = e0; e < e1; e += (uint64_t)ngrp) {   // wave-uniform trip count
        const bool live = act && e + (uint64_t)g < e1;
        const uint32_t q = far_col[live ? e + (uint64_t)g : e];
        const float *Wq = W + (int64_t)q * r;
        __syncthreads();   // the table is in place; the last pass of the previous round has read the buffers
        if (live) {
            float in[PN], out[PN];
#pragma unroll
            for (int j = 0; j < PN; ++j) in[j] = Wq[f * PN + j];
            apply(factor(0, cellS[(int64_t)q * D]), in, out);
            if (D == 1) {
#pragma unroll
                for (int i = 0; i < PN; ++i) acc[i] += out[i];
            } else {
#pragma unroll
                for (int i = 0; i < PN; ++i) buf[f + i * nfib] = out[i];
            }
        }
        int stride = 1;   // of dimension d in the LDS layout (dimensions 1..D-1 fastest first, then 0)
        for (int d = 1; d < D; ++d) {
            __syncthreads();
            if (live) {
                const int hi = (int)(((float)f + 0.5f) * (1.f / (float)stride));   // f / stride
                const int base = hi * stride * PN + (f - hi * stride);
                float in[PN], out[PN];
#pragma unroll
                for (int j = 0; j < PN; ++j) in[j] = buf[base + j * stride];
                apply(factor(d, cellS[(int64_t)q * D + d]), in, out);
                if (d == D - 1) {
#pragma unroll
                    for (int i = 0; i < PN; ++i) acc[i] += out[i];
                } else {
#pragma unroll
                    for (int i = 0; i < PN; ++i) buf[base + i * stride] = out[i];
                }
            }
            stride *= PN;
        }
    }
    // accumulators of every group to its buffer at the flat node index i = sum_d i_d p^d, then the
    // groups are added in ascending order
    __syncthreads();
    if (act) {
        int stride = 1;
        for (int d = 2; d < D; ++d) stride *= PN;
        const int hi = (int)(((float)f + 0.5f) * (1.f / (float)stride));
#pragma unroll
        for (int i = 0; i < PN; ++i) {
            int flat;
            if (D == 1) {
                flat = i;
            } else {
                const int idx = hi * stride * PN + (f - hi * stride) + i * stride;   // LDS layout index
                const int i0 = idx / nfib;
                flat = i0 + PN * (idx - i0 * nfib);
            }
            buf[flat] = acc[i];
        }
    }
    __syncthreads();
    float *Va = V + a * r;
    for (int i = lane; i < r; i += 64) {
        float sum = 0.f;
        for (int gg = 0; gg < ngrp; ++gg) sum += lds[gg * r + i];
        Va[i] = sum;
    }
}

// Offsets (source cell - target cell) a far pair of a depth can have in dimension d.  The parents
// of a far pair are near, |O + U| < theta in every dimension (U the shift at the parents' depth),
// and a child centre lies half a child edge from its parent's: |o + u| < 2 theta + 1.  Depth 1
// has the root pair as parents, which is near whatever its distance: o in {-1, 0, 1}.  One more
// offset on either side is tabulated, and everything is cut to the cells a depth has.
static KronShape kron_shape(const f3m_plan_s &P, int level) {
    KronShape S{};
    double u[F3M_MAX_DIM];
    P.grid_shift(level, u);
    const double reach = 2.0 * (double)P.theta + 2.0, cmax = (double)((1ll << level) - 1);
    S.no = 1;
    for (int d = 0; d < P.D; ++d) {
        double lo = level == 1 ? -1.0 : std::max(-cmax, std::floor(-reach - u[d]));
        double hi = level == 1 ? 1.0 : std::min(cmax, std::ceil(reach - u[d]));
        if (hi < lo) hi = lo = std::min(std::max(lo, -cmax), cmax);   // no far pair can exist here
        S.omin[d] = (int)lo;
        S.no = std::max(S.no, (int)(hi - lo) + 1);
    }
    return S;
}

// Depths whose M2L is the grouped one (more than 32 fibres per box, far rows stored): every far row once more,
// ordered by the row-major cell index of the partner.
void build_far_orders(f3m_plan_s &P, hipStream_t st) {
    for (int l = 1; l <= P.L; ++l) {
        f3m_level &lv = P.lev[l];
        if (lv.far_sz == 0 || lv.p == 0 || lv.far_implicit || lv.far_points || lv.r / lv.p <= 32) continue;
        lv.far_ord.alloc((size_t)lv.far_sz, &P.bytes);
        far_order_kernel<<<grid_for(lv.nb), dim3(FO_NT), 0, st>>>(lv.far_ptr.p, lv.far_col.p, P.slev(l).cell.p, P.D, l, lv.nb,
                                                                lv.far_ord.p);
        F3M_HIP(hipGetLastError());
    }
}

// up to TAB_ARG floats to the device as an argument of a launch: a copy from pageable memory takes the host 20 us
constexpr int TAB_ARG = 960;
struct TabArg { float v[TAB_ARG]; };
__global__ __launch_bounds__(256) void put_table_kernel(float *__restrict__ dst, int n, TabArg A) {
    for (int i = threadIdx.x; i < n; i += 256) dst[i] = A.v[i];
}

// per depth with far pairs: the 1-D factor matrices of the node-to-node kernel matrix, built in fp64; the factors of the weighted
// near pairs and the parent's basis at a child's nodes
void upload_tables(f3m_plan_s &P, hipStream_t st) {
    std::vector<float> &g = P.host_tabs;
    g.clear();
    std::vector<std::pair<float **, size_t>> places;   // where the address of a table goes, and its offset
    auto table = [&](float **at, size_t count) {
        places.emplace_back(at, g.size());
        g.resize(g.size() + count);
        return &g[places.back().second];
    };
    if (P.tree_lmin > 0) {
        const TransferArg T = make_transfer();
        std::copy(&T.t[0][0][0], &T.t[0][0][0] + 32, table(&P.transfer.p, 32));
    }
    if (P.near_weighted && !P.src) near_table(P, table(&P.near_tab.p, 16));
    for (int l = 1; l <= P.L; ++l) {
        f3m_level &lv = P.lev[l];
        if (lv.far_sz == 0 || lv.p == 0 || l > P.last_depth()) continue;
        const int p = lv.p;
        std::vector<double> s(p);
        for (int k = 0; k < p; ++k) s[k] = p > 1 ? std::cos(M_PI * (double)k / (double)(p - 1)) : 0.0;
        const double half = 0.5 * (double)P.E / (double)(1ull << l);
        const double c = half * half / (2.0 * (double)P.gamma * (double)P.gamma);
        KronShape S = kron_shape(P, l);
        if (lv.far_implicit) {
            // the candidate-grid M2L (one point set, far ratio 2) reads one table G[o + 3][i][j], o = -3..3
            S.no = 7;
            S.omin[0] = -3;
            lv.gtab_omax = 3;
        }
        const int ndim = lv.far_implicit ? 1 : P.D;
        if (!lv.far_implicit && !lv.far_points && lv.r / p <= 32) {
            // m2l_kron_small_kernel stages the factor tables of the depth in LDS beside its far-pair buffers
            const size_t lds = (size_t)((64 / (lv.r / p)) * lv.r + P.D * S.no * p * p) * sizeof(float);
            if (lds > 64 * 1024)
                fail(F3M_ERR_UNSUPPORTED, "eta = " + std::to_string(P.theta) + " gives " + std::to_string(S.no) +
                                              " cell offsets per dimension at depth " + std::to_string(l) +
                                              ": the factor tables of the M2L exceed 64 KB of LDS for this D and interp_nodes");
        }
        double u[F3M_MAX_DIM];
        P.grid_shift(l, u);
        float *G = table(&lv.gtab.p, (size_t)ndim * S.no * p * p);
        for (int d = 0; d < ndim; ++d)
            for (int k = 0; k < S.no; ++k)
                for (int i = 0; i < p; ++i)
                    for (int j = 0; j < p; ++j) {
                        // source node minus target node in half box edges: 2 (o + u) + s_j - s_i
                        const double t = 2.0 * ((double)(S.omin[d] + k) + u[d]) + s[j] - s[i];
                        G[(((size_t)d * S.no + k) * p + i) * p + j] = (float)std::exp(-c * t * t);
                    }
        if (P.src && l == P.near_weighted) {   // the factor F of near_weighted_error, for the same offsets
            float *Gn = table(&P.near_tab.p, (size_t)ndim * S.no * p * p);
            for (int d = 0; d < ndim; ++d)
                for (int k = 0; k < S.no; ++k)
                    for (int i = 0; i < p; ++i)
                        for (int j = 0; j < p; ++j) {
                            const double o = (double)(S.omin[d] + k) + u[d];
                            Gn[(((size_t)d * S.no + k) * p + i) * p + j] =
                                (float)(basis_scale() * std::exp(2.0 * c * (s[i] * s[j] + 2.0 * o * (s[i] - s[j] - o))));
                        }
        }
    }
    if (g.empty()) return;
    P.tables.alloc(g.size(), &P.bytes);
    for (auto &t : places) *t.first = P.tables.p + t.second;
    if (g.size() <= 8 * TAB_ARG) {
        for (size_t at = 0; at < g.size(); at += TAB_ARG) {
            TabArg A;
            const int count = (int)std::min<size_t>(TAB_ARG, g.size() - at);
            std::copy(g.data() + at, g.data() + at + count, A.v);
            put_table_kernel<<<dim3(1), dim3(256), 0, st>>>(P.tables.p + at, count, A);
        }
        F3M_HIP(hipGetLastError());
    } else {   // (the host copy stays until the plan has been waited for)
        F3M_HIP(hipMemcpyAsync(P.tables.p, g.data(), g.size() * sizeof(float), hipMemcpyHostToDevice, st));
    }
}


// ------------------------------------------------------------------------------------
// partial node weights of the chunks of a box -> W, in one or two stages
static void reduce_partials(f3m_plan_s &P, f3m_level &lv, int r, float *W, hipStream_t st, int64_t dpart = 0) {
    if (lv.nslices > 0) {
        p2m_slice_kernel<<<grid_for(lv.nslices), dim3(256), 0, st>>>(lv.slice_box.p, lv.slice_first.p, lv.chunk_first.p,
                                                                    lv.nslices, r, P.Wpart.p + dpart, P.Wslice.p);
        p2m_slice_sum_kernel<<<grid_for(lv.nb), dim3(256), 0, st>>>(lv.slice_first.p, lv.chunk_first.p, lv.nb, r,
                                                                   P.Wslice.p, W);
    } else {
        p2m_reduce_kernel<<<grid_for(lv.nb), dim3(256), 0, st>>>(lv.chunk_first.p, lv.nb, r, P.Wpart.p + dpart, W);
    }
}

// every box of the depth is exactly one chunk of the P2M / L2P work split (chunk index = box rank)
static int single_chunks(const f3m_level &lv) { return lv.max_box <= P2M_CHUNK && lv.nchunks == lv.nb ? 1 : 0; }
// the runs of the depth are long ones (D = 3, 4 nodes per dimension)
static bool long_chunks(const f3m_level &lv) { return lv.chunk > P2M_CHUNK; }

// P2M of the runs of lv (3-D, 4 nodes): NS = 2 both sets of node weights, else one.  chunk_box and its like from `list`, boxes of lv.
template <int NS>
static void p2m34(const f3m_plan_s &P, const f3m_level &lv, const f3m_level &list, const float *X, const float *b, const CentreArg &C,
                  float *W, const WeightedArg &A, const uint32_t *perm, hipStream_t st) {
    const bool pairs = &lv == &list && single_chunks(lv);
    const int64_t count = pairs ? lv.nb : list.nchunks;
    if (long_chunks(list)) {
        p2m34_long_kernel<(NS > 1)><<<grid_for(count), dim3(64), 0, st>>>(X, b, lv.start.p, lv.cell.p, list.chunk_box.p, list.chunk_first.p,
                                                                         count, C, W, P.Wpart.p, A);
        F3M_HIP(hipGetLastError());
        return;
    }
    auto run = [&](auto kern) {
        kern<<<grid_for(pairs ? cdiv(count, 2) : count), dim3(64), 0, st>>>(X, b, lv.start.p, lv.cell.p, list.chunk_box.p, list.chunk_first.p,
                                                                            count, C, W, P.Wpart.p, A, perm);
        F3M_HIP(hipGetLastError());
    };
    if (pairs && perm) run(p2m34_kernel<NS, true, true>);
    else if (pairs) run(p2m34_kernel<NS, false, true>);
    else if (perm) run(p2m34_kernel<NS, true, false>);
    else run(p2m34_kernel<NS, false, false>);
}

// g = log2(e) l^2 / (2 gamma^2) of a depth: c l^2 bounds the magnitude of the expanded exponent terms in
// box-local coordinates (|x'|^2 + |y'|^2 <= 7.5 D/3 l^2)
static double gram_exponent_scale(const f3m_plan_s &P, int l) {
    const CentreArg CL = make_centre(P, l);
    const double c = 1.4426950408889634 / (2.0 * (double)P.gamma * (double)P.gamma);
    return c * CL.edge * CL.edge;
}

// the near field of a depth runs on the Gram kernels (expanded square on the matrix cores) while g D <= 6;
// above the limit, and for the root pair of two point sets (near whatever its distance: no bound on the
// coordinates), the difference form is used
static bool gram_near_field(const f3m_plan_s &P, int l) {
    const double gl = gram_exponent_scale(P, l);
    return gl * (double)P.D <= 6.0 && gl > 1e-30 && !P.force_all_near && P.T <= 1024 && !(P.src && l == 0);
}

// Slices that a target tile of the 3-D Gram near field over the near list of depth l is cut into (1: none):
// with few target tiles and long rows several wavefronts share a tile, each on a slice of the sources.
// Tiles of the last depth may be worked in pairs by p2p_gram3_pair_kernel: one point set in 3-D on the Gram
// path.  Coordinates relative to the midpoint of a pair are up to 1.6 times those relative to a box centre in
// the products of the expanded square, so the limit on g D is that of the Gram path divided by 1.6.
bool p2p_pairs_allowed(const f3m_plan_s &P) {
    return P.D == 3 && !P.src && gram_near_field(P, P.L) && gram_exponent_scale(P, P.L) * 3.0 <= 3.75 &&
           p2p_nsplit(P, P.L, P.ntiles) == 1;
}

int p2p_nsplit(const f3m_plan_s &P, int l, int64_t ntiles) {
    const f3m_level &lv = P.lev[l];
    if (!(P.D == 3 && gram_near_field(P, l) && ntiles > 0 && ntiles < 8192 && lv.nb > 0 && P.slev(l).nb > 0)) return 1;
    const double row_sources = (double)lv.near_sz / (double)lv.nb * ((double)P.ns() / (double)P.slev(l).nb);   // per tile
    const int nsplit = (int)std::min<double>(std::min<double>(64.0, (double)cdiv(262144, ntiles)), row_sources / 2048.0);
    return nsplit < 2 ? 1 : nsplit;
}

// box_order: b and y are in the plan's box order (one-set plans; b padded), so there are no permutations.
// bs_in / yn_in (both or neither): the right-hand side already gathered into box order (padded like
// the plan's own buffer) and the near-field result already computed for it; used by the products with
// several right-hand sides, whose near field is evaluated for a group of columns at once.
template <int D>
static void run_kmvm_d(f3m_plan_s &P, const float *b, float *y, hipStream_t st, bool box_order,
                       const float *bs_in = nullptr, const float *yn_in = nullptr) {
    if (box_order) bs_in = b;
    const float *bs = bs_in ? bs_in : P.bs.p;
    // no near field: every pair is interpolated (smooth field, or the products stop above the last depth)
    const bool no_near = !yn_in && P.rho == 0 && (P.lev[P.L].near_sz == 0 || !P.exact_near());
    // the plan's second stream has nothing to do where the near pairs are interpolated on the first one
    const hipStream_t side = P.near_weighted ? nullptr : P.side;
    const float *yn = yn_in ? yn_in : no_near ? nullptr : P.yn.p;
    const int64_t n = P.n;
    const float nc2 = (float)(-1.4426950408889634 / (2.0 * (double)P.gamma * (double)P.gamma));
    // A mark at every boundary between two stages with launches.  An event record is a packet of its own on the stream:
    // one event per boundary, where stages used to record their begin and end each, and no pass that only fills or
    // copies (below), take the product of 2e4 points from 134 us to 85 us.
    size_t nmarks = 0;
    auto mark = [&] {
        if (nmarks == P.marks.size()) {   // (an event that cannot be made leaves the list as it is)
            P.marks.reserve(nmarks + 1);
            P.marks.push_back(event_get());
        }
        F3M_HIP(hipEventRecord(P.marks[nmarks], st));
        return P.marks[nmarks++];
    };
    const unsigned gn = (unsigned)cdiv(n, 256);
    f3m_level &leaf = P.lev[P.L];
    const float *Ys = P.Ys();   // sources in box order (the targets themselves for one point set)

    hipEvent_t now = P.t_begin = mark();   // the last mark: nothing has been launched on the stream since
    // One set whose points are read by the P2M of one depth only: it takes the right-hand side from the caller's order itself
    const uint32_t *perm_in = nullptr;
    if (!bs_in && !P.src && !P.route && no_near && P.tree_lmin > 0 && !long_chunks(P.lev[P.tree_lmax])) {
        perm_in = P.perm.p;
        for (int l = 1; l < P.tree_lmin || l <= P.last_depth(); ++l)
            if ((l < P.tree_lmin || l > P.tree_lmax) && P.lev[l].far_sz > 0 && P.lev[l].p > 0) perm_in = nullptr;
    }
    if (perm_in) bs = b;
    if (!bs_in && !perm_in) {   // else gathered by the caller
        if (P.sroute())
            route_gather(*P.sroute(), b, P.bs.p, P.route_a.p, P.route_b.p, st);
        else
            gather_kernel<<<dim3((unsigned)cdiv(P.ns(), 256)), dim3(256), 0, st>>>(b, P.sperm(), P.ns(), P.bs.p);
        now = mark();
    }
    P.t_in = now;
    // The near field goes to the plan's second stream (vector ALU work) and overlaps the
    // far field (matrix-core work) on the caller's stream; with no_overlap it runs in line.
    hipStream_t sn = side ? side : st;
    if (side) {
        F3M_HIP(hipEventRecord(P.ev_fork, st));
        F3M_HIP(hipStreamWaitEvent(side, P.ev_fork, 0));
        F3M_HIP(hipEventRecord(P.ev_p2p0, sn));
    }
    // exact sums over a CSR list of box pairs of one depth (target tiles given), into yn
    auto direct_pairs = [&](int l, const uint64_t *row_ptr, const uint32_t *cols, const uint32_t *tile_box,
                            const uint32_t *tile_first, int64_t ntiles, int accumulate,
                            const uint8_t *paired = nullptr) {
        f3m_level &lv = P.lev[l];
        const uint32_t *sstart = P.slev(l).start.p;
        const CentreArg CL = make_centre(P, l);
        const double gl = gram_exponent_scale(P, l);
        const bool gram = gram_near_field(P, l);
        // few target tiles with long rows: several wavefronts per tile, each on a slice of the sources
        const int nsplit = cols == lv.near_col.p ? p2p_nsplit(P, l, ntiles) : 1;
        if (nsplit > 1) {
            // the partial sums were sized when the plan was built: nothing is allocated here
            if (P.p2p_part.count < (size_t)nsplit * (size_t)n)
                fail(F3M_ERR_HIP, "internal: the plan holds no room for the split near field");
            p2p_gram3_kernel<true, 1><<<grid_for(cdiv(ntiles * nsplit, 4)), dim3(256), 0, sn>>>(
                P.Xs.p, lv.start.p, Ys, bs, sstart, lv.cell.p, row_ptr, cols, tile_box, tile_first, ntiles, (float)gl,
                (float)(1.0 / CL.edge), CL, P.yn.p, accumulate, nsplit, n, P.p2p_part.p, MultiArg{}, nullptr);
            p2p_split_sum_kernel<<<dim3(gn), dim3(256), 0, sn>>>(P.p2p_part.p, nsplit, n, P.yn.p, accumulate);
        } else if (gram && D == 3) {
            if (ntiles > 0)
                p2p_gram3_kernel<false, 1><<<grid_for(cdiv(ntiles, 4)), dim3(256), 0, sn>>>(
                    P.Xs.p, lv.start.p, Ys, bs, sstart, lv.cell.p, row_ptr, cols, tile_box, tile_first, ntiles,
                    (float)gl, (float)(1.0 / CL.edge), CL, P.yn.p, accumulate, 1, n, nullptr, MultiArg{}, paired);
        }
        else if (gram)
            p2p_mfma_kernel<D><<<grid_for(cdiv(ntiles, 4)), dim3(256), 0, sn>>>(
                P.Xs.p, lv.start.p, Ys, bs, sstart, lv.cell.p, row_ptr, cols, tile_box, tile_first, ntiles, (float)gl,
                (float)(1.0 / CL.edge), CL, P.yn.p, accumulate);
        else
            p2p_kernel<D><<<grid_for(ntiles), dim3(64), 0, sn>>>(P.Xs.p, lv.start.p, Ys, bs, sstart, row_ptr, cols,
                                                                tile_box, tile_first, ntiles, nc2, P.yn.p, accumulate);
        F3M_HIP(hipGetLastError());
    };
    if (yn_in || no_near) {
        // computed by the caller, or nothing to compute
    } else if (leaf.near_sz == 0) {
        // every pair was interpolated (smooth field, Sec. 4.3) or summed at its own depth (small field)
        zero_kernel<<<dim3(gn), dim3(256), 0, sn>>>(P.yn.p, n);
    } else {
        if (P.npairs > 0) {
            // the first runs of paired boxes two at a time, every other big tile on its own
            const CentreArg CL = make_centre(P, P.L);
            p2p_gram3_pair_kernel<<<grid_for(cdiv(P.npairs, 4)), dim3(256), 0, sn>>>(
                P.Xs.p, leaf.start.p, bs, leaf.cell.p, leaf.near_ptr.p, leaf.near_col.p, P.pair_box.p, P.npairs, P.T,
                (float)gram_exponent_scale(P, P.L), (float)(1.0 / CL.edge), CL, P.yn.p);
            F3M_HIP(hipGetLastError());
            direct_pairs(P.L, leaf.near_ptr.p, leaf.near_col.p, P.rtile_box.p, P.rtile_first.p, P.nrtiles, 0,
                         P.paired.p);
        } else {
            direct_pairs(P.L, leaf.near_ptr.p, leaf.near_col.p, P.tile_box.p, P.tile_first.p, P.ntiles, 0);
        }
        // last runs with few targets: sources on the lanes
        if (P.notiles > 0)
            p2p_small_kernel<D, overflow_targets(D)><<<grid_for(cdiv(P.notiles, 4)), dim3(256), 0, sn>>>(
                P.Xs.p, leaf.start.p, Ys, bs, P.slev(P.L).start.p, leaf.near_ptr.p, leaf.near_col.p, P.otile_box.p,
                P.otile_first.p, P.notiles, nc2, P.yn.p, 1, 0, MultiArg{});
    }
    // small-field pairs of every depth (Sec. 4.2), added on top
    for (int l = 1; l <= P.L && !yn_in; ++l) {
        f3m_level &lv = P.lev[l];
        if (lv.small_sz > 0) {
            p2p_small_kernel<D, small_tt<D>()><<<grid_for(cdiv(lv.sm_ntiles, 4)), dim3(256), 0, sn>>>(
                P.Xs.p, lv.start.p, Ys, bs, P.slev(l).start.p, lv.small_ptr.p, lv.small_col.p, lv.sm_tile_box.p,
                lv.sm_tile_first.p, lv.sm_ntiles, nc2, P.yn.p, 0, 1, MultiArg{});
            F3M_HIP(hipGetLastError());
        }
    }
    F3M_HIP(hipGetLastError());
    if (side) {
        F3M_HIP(hipEventRecord(P.ev_p2p1, side));
        F3M_HIP(hipEventRecord(P.ev_join, side));
        P.t_p2p0 = P.ev_p2p0;
        P.t_p2p1 = P.ev_p2p1;
    } else {
        P.t_p2p0 = now;
        if (!yn_in && !no_near) now = mark();
        P.t_p2p1 = now;
    }
    // six marks per depth: [0,1] bracket the upward pass (P2M or M2M), [2,3] the M2L, [4,5] the
    // downward pass (L2L and/or L2P) of that depth
    P.far_events.assign((size_t)(P.L + 1) * 6, nullptr);
    P.t_wait0 = P.t_wait1 = nullptr;
    auto level_events = [&](int l) { return &P.far_events[(size_t)l * 6]; };
    const bool tree = P.tree_lmin > 0;   // D = 3, 4 nodes per dimension on depths tree_lmin..tree_lmax
    // no far pairs, dropped by the adaptive rule (Sec. 4.3), or part of the band of the tree
    auto on_its_own = [&](int l) {
        const f3m_level &lv = P.lev[l];
        return lv.far_sz > 0 && lv.p > 0 && l <= P.last_depth() && !(tree && l >= P.tree_lmin && l <= P.tree_lmax);
    };
    // Where the band holds every far depth its one L2P writes the far field of every point: nothing to preset, and in box
    // order it adds the near field and writes the result.
    bool one_l2p = tree;
    for (int l = 1; l <= P.L; ++l) one_l2p = one_l2p && !on_its_own(l);
    // So it does where the result goes straight to its place in the caller's order (perm_out), by direct stores.
    const uint32_t *perm_out = one_l2p && !box_order && !P.route && !long_chunks(P.lev[P.tree_lmax]) ? P.perm.p : nullptr;
    const bool direct_out = one_l2p && (box_order || perm_out);
    if (!one_l2p) {
        zero_kernel<<<dim3(gn), dim3(256), 0, st>>>(P.ys.p, n);
        F3M_HIP(hipGetLastError());
        now = mark();
    }
    // node weights of the source boxes of a depth, from the points, into P.W (the boxes its chunk list names)
    auto p2m_depth = [&](int l) {
        f3m_level &lv = P.lev[l];
        f3m_level &sv = P.slev(l);
        const int p = lv.p, r = lv.r;
        const NodeArg N = make_nodes(p);
        const CentreArg CS = make_centre(P, l, true);   // source grid
        size_t sh = (size_t)(FF_TP * D * p + FF_TP) * sizeof(float);
        if (D == 3 && p == 4)
            p2m34<1>(P, sv, sv, Ys, bs, CS, P.W.p, WeightedArg{}, nullptr, st);
        else if (r <= 64)
            p2m_kernel<D><<<grid_for(sv.nchunks), dim3(64), sh, st>>>(
                Ys, bs, sv.start.p, sv.cell.p, sv.chunk_box.p, sv.chunk_first.p, sv.nchunks, p, r, CS, N,
                P.W.p, P.Wpart.p);
        else
            for_nodes<D>(p, [&](auto pn) {
                constexpr int PN = decltype(pn)::value;
                if constexpr (ipow(PN, D) > 64)
                    p2m_halves_kernel<D, PN><<<grid_for(sv.nchunks), dim3(256), 0, st>>>(
                        Ys, bs, sv.start.p, sv.cell.p, sv.chunk_box.p, sv.chunk_first.p, sv.nchunks, CS, N, P.W.p, P.Wpart.p);
            });
        F3M_HIP(hipGetLastError());
        if (sv.max_box > sv.chunk)   // some box has several chunks
            reduce_partials(P, sv, r, P.W.p, st);
        F3M_HIP(hipGetLastError());
    };
    // M2L of a depth from its far list, factor by factor; rows of V whose far row is empty are left alone
    auto kron_m2l = [&](int l, const float *W, float *V, bool near_rows = false) {
        f3m_level &lv = P.lev[l];
        f3m_level &sv = P.slev(l);
        const int p = lv.p, r = lv.r;
        const KronShape KS = kron_shape(P, l);
        const int nfib = r / p;
        if (nfib <= 32) {   // several far pairs per wavefront
            const size_t sh = (size_t)((64 / nfib) * r + D * KS.no * p * p) * sizeof(float);
            auto launch = [&](auto kern) {
                kern<<<grid_for(lv.nb), dim3(64), sh, st>>>(
                    lv.cell.p, sv.cell.p, near_rows ? lv.near_ptr.p : lv.far_ptr.p, near_rows ? lv.near_col.p : lv.far_col.p, lv.nb,
                    D, r, near_rows ? P.near_tab.p : lv.gtab.p, KS, W, V);
            };
            switch (p) {
                case 2: launch(m2l_kron_small_kernel<2>); break;
                case 3: launch(m2l_kron_small_kernel<3>); break;
                case 4: launch(m2l_kron_small_kernel<4>); break;
                case 5: launch(m2l_kron_small_kernel<5>); break;
                case 6: launch(m2l_kron_small_kernel<6>); break;
                case 7: launch(m2l_kron_small_kernel<7>); break;
                case 8: launch(m2l_kron_small_kernel<8>); break;
                default: fail(F3M_ERR_UNSUPPORTED, "interp_nodes must be in [2,8]");
            }
        } else {
            if (!lv.far_ord.p) fail(F3M_ERR_HIP, "internal: the far rows of this depth have not been ordered");
            auto launch = [&](auto kern) {
                kern<<<grid_for(lv.nb), dim3(256), 0, st>>>(lv.cell.p, sv.cell.p, lv.far_ptr.p, lv.far_ord.p, lv.nb, lv.gtab.p,
                                                           KS, W, V);
            };
            // every (nodes per dimension, D) with more than 32 fibres and at most 4096 nodes
            switch (p * 8 + D) {
                case 2 * 8 + 7: launch(m2l_kron_grouped_kernel<2, 7>); break;
                case 3 * 8 + 5: launch(m2l_kron_grouped_kernel<3, 5>); break;
                case 3 * 8 + 6: launch(m2l_kron_grouped_kernel<3, 6>); break;
                case 3 * 8 + 7: launch(m2l_kron_grouped_kernel<3, 7>); break;
                case 4 * 8 + 4: launch(m2l_kron_grouped_kernel<4, 4>); break;
                case 4 * 8 + 5: launch(m2l_kron_grouped_kernel<4, 5>); break;
                case 4 * 8 + 6: launch(m2l_kron_grouped_kernel<4, 6>); break;
                case 5 * 8 + 4: launch(m2l_kron_grouped_kernel<5, 4>); break;
                case 5 * 8 + 5: launch(m2l_kron_grouped_kernel<5, 5>); break;
                case 6 * 8 + 3: launch(m2l_kron_grouped_kernel<6, 3>); break;
                case 6 * 8 + 4: launch(m2l_kron_grouped_kernel<6, 4>); break;
                case 7 * 8 + 3: launch(m2l_kron_grouped_kernel<7, 3>); break;
                case 7 * 8 + 4: launch(m2l_kron_grouped_kernel<7, 4>); break;
                case 8 * 8 + 3: launch(m2l_kron_grouped_kernel<8, 3>); break;
                case 8 * 8 + 4: launch(m2l_kron_grouped_kernel<8, 4>); break;
                default: fail(F3M_ERR_UNSUPPORTED, "no M2L kernel for this number of nodes and dimensions");
            }
        }
        F3M_HIP(hipGetLastError());
    };
    // ---- depths that are handled on their own, straight from the points (Fig. 4 steps 1-3)
    for (int l = 1; l <= P.L; ++l) {
        f3m_level &lv = P.lev[l];
        if (!on_its_own(l)) continue;
        const int p = lv.p;
        const NodeArg N = make_nodes(p);
        hipEvent_t *ev = level_events(l);
        const CentreArg C = make_centre(P, l);          // target grid
        ev[0] = now;
        if (lv.far_points) {   // from point to point: no node weights or potentials
            const KronShape KS = kron_shape(P, l);
            ev[1] = ev[2] = now;
            run_far_points(P, l, bs, P.ys.p, KS.omin[0], KS.no, st);
            ev[3] = ev[4] = ev[5] = now = mark();
            continue;
        }
        p2m_depth(l);
        ev[1] = ev[2] = now = mark();
        if (!(lv.far_implicit && run_m2l_stencil(P, l, P.W.p, P.V.p, st))) kron_m2l(l, P.W.p, P.V.p);
        ev[3] = ev[4] = now = mark();
        {
            if (D == 3 && p == 4 && long_chunks(lv))
                l2p34_long_kernel<false><<<grid_for(lv.nchunks), dim3(64), 0, st>>>(
                    P.Xs.p, lv.start.p, lv.cell.p, lv.far_ptr.p, lv.chunk_box.p, lv.chunk_first.p, lv.nchunks, C, P.V.p, P.ys.p,
                    P.ys.p, nullptr, 0.f);
            else if (D == 3 && p == 4)
                l2p34_kernel<false, false><<<grid_for(cdiv(lv.nchunks, L2P_NCH)), dim3(64), 0, st>>>(
                    P.Xs.p, lv.start.p, lv.cell.p, lv.far_ptr.p, lv.chunk_box.p, lv.chunk_first.p, lv.nchunks, C, P.V.p, P.ys.p,
                    P.ys.p, single_chunks(lv), nullptr, 0.f, nullptr);
            else
                for_nodes<D>(p, [&](auto pn) {
                    l2p_kernel<D, decltype(pn)::value><<<grid_for(lv.nchunks), dim3(P2M_CHUNK), 0, st>>>(
                        P.Xs.p, lv.start.p, lv.cell.p, lv.far_ptr.p, lv.chunk_box.p, lv.chunk_first.p, lv.nchunks, C, N,
                        P.V.p, P.ys.p);
                });
            F3M_HIP(hipGetLastError());
        }
        ev[5] = now = mark();
    }
    // ---- depths tree_lmin..tree_lmax: P2M at the last depth of the band, weights passed upward,
    //      M2L per depth, potentials passed downward, one L2P at the last depth of the band
    if (tree) {
        // One point set: node weights from the points at the last depth of the band and upward from
        // there.  Two point sets: only the targets' side uses the tree; the node weights of a depth come
        // from the points of the source boxes that its far rows name (the sources' tree may hold many
        // more boxes than are ever used, and a pass over all of them costs more than it saves).
        const int L = P.tree_lmax;
        const int r = 64;
        f3m_level &lf = P.lev[L];
        // near pairs between weighted points: exp2(kw |u|^2 / (l/2)^2) = exp(-|u|^2 / 2 gamma^2)
        const bool weighted = P.near_weighted == L;
        if (P.near_weighted && !weighted) fail(F3M_ERR_HIP, "internal: weighted near pairs outside the last depth of the tree");
        const double half = 0.5 * (double)P.E / std::ldexp(1.0, L);
        const float kw = (float)(-1.4426950408889634 * half * half / (2.0 * (double)P.gamma * (double)P.gamma));
        if (!P.src) {
            {
                hipEvent_t *ev = level_events(L);
                ev[0] = now;
                const WeightedArg A{(lf.nb + 1) * r, lf.nchunks * r, kw, false};
                if (weighted) p2m34<2>(P, lf, lf, P.Xs.p, bs, make_centre(P, L), lf.Wl.p, A, perm_in, st);
                else p2m34<1>(P, lf, lf, P.Xs.p, bs, make_centre(P, L), lf.Wl.p, A, perm_in, st);
                if (lf.max_box > lf.chunk) {   // some box has several chunks
                    reduce_partials(P, lf, r, lf.Wl.p, st);
                    if (weighted) reduce_partials(P, lf, r, lf.Wl.p + A.dW, st, A.dpart);
                }
                F3M_HIP(hipGetLastError());
                ev[1] = now = mark();
            }
            if (weighted) {   // the near field of this product (two sets: below)
                P.t_p2p0 = now;
                run_near_weighted(P, lf.Wl.p + (lf.nb + 1) * r, lf.Vl.p + lf.nb * r, st);
                P.t_p2p1 = now = mark();
            }
            for (int l = L - 1; l >= P.tree_lmin; --l) {
                f3m_level &lv = P.lev[l], &dn = P.lev[l + 1];
                hipEvent_t *ev = level_events(l);
                ev[0] = now;
                m2m34_kernel<<<grid_for(lv.nb), dim3(64), 0, st>>>(lv.cstart.p, dn.key.p, lv.nb, P.transfer.p, dn.Wl.p, lv.Wl.p);
                F3M_HIP(hipGetLastError());
                ev[1] = now = mark();
            }
        }
        for (int l = P.tree_lmin; l <= L; ++l) {
            f3m_level &lv = P.lev[l];
            hipEvent_t *ev = level_events(l);
            if (P.src) {
                ev[0] = now;
                p2m_depth(l);
                ev[1] = now = mark();
            }
            ev[2] = now;
            if (m2l_stencil_small(P, l)) {
                // with the depths behind it that have few parents too; the time is that of the deepest
                int to = l;
                while (to < L && m2l_stencil_small(P, to + 1)) ++to;
                run_m2l_small(P, l, to, st);
                for (; l < to; ++l) level_events(l)[2] = level_events(l)[3] = now;
                ev = level_events(to);
                ev[2] = now;
            } else if (lv.far_implicit) {
                if (!run_m2l_stencil(P, l, lv.Wl.p, lv.Vl.p, st, true))   // Wl ends with a row of zeros
                    fail(F3M_ERR_HIP, "internal: depth outside the candidate-grid M2L");
            } else {
                // from the far list: the potentials of the boxes without far partners must read zero
                zero_kernel<<<dim3((unsigned)cdiv(lv.nb * (int64_t)r, 256)), dim3(256), 0, st>>>(lv.Vl.p, lv.nb * (int64_t)r);
                kron_m2l(l, P.src ? P.W.p : lv.Wl.p, lv.Vl.p);
            }
            ev[3] = now = mark();
        }
        if (weighted && P.src) {   // the near field of this product
            P.t_p2p0 = now;
            f3m_level &ns = P.near_src;
            if (ns.nchunks > 0) {
                WeightedArg A;
                A.kw = kw;
                A.only = true;
                p2m34<1>(P, P.slev(L), ns, Ys, bs, make_centre(P, L, true), ns.Wl.p, A, nullptr, st);
                if (ns.max_box > ns.chunk) reduce_partials(P, ns, r, ns.Wl.p, st);
            }
            float *Vn = lf.Vl.p + lf.nb * r;
            zero_kernel<<<dim3((unsigned)cdiv(lf.nb * (int64_t)r, 256)), dim3(256), 0, st>>>(Vn, lf.nb * (int64_t)r);
            kron_m2l(L, ns.Wl.p, Vn, true);
            P.t_p2p1 = now = mark();
        }
        for (int l = P.tree_lmin + 1; l <= L; ++l) {
            f3m_level &lv = P.lev[l], &up = P.lev[l - 1];
            hipEvent_t *ev = level_events(l);
            ev[4] = now;
            l2l34_kernel<<<grid_for(up.nb), dim3(64), 0, st>>>(up.cstart.p, lv.key.p, up.nb, P.transfer.p, up.Vl.p, lv.Vl.p);
            F3M_HIP(hipGetLastError());
            if (l < L) ev[5] = now = mark();
        }
        {
            hipEvent_t *ev = level_events(L);
            if (P.tree_lmin == L) ev[4] = now;
            // The L2P adds the near field, so it waits for it; without that it would overlap, and a pass would add and scatter (product of
            // 1e6 points, exact near field on the second stream: 270 us, 277 with the pass; 2e6 normal 1080 and 1109; below 1e4 points the
            // two differ by less than 2 %).
            if (side && direct_out) {   // the near field may be what is waited for: not part of the downward pass
                P.t_wait0 = mark();
                F3M_HIP(hipStreamWaitEvent(st, P.ev_join, 0));
                P.t_wait1 = mark();
            }
            const float *base = direct_out ? yn : one_l2p ? nullptr : P.ys.p;
            auto l2p = [&](auto kern) {
                kern<<<grid_for(cdiv(lf.nchunks, L2P_NCH)), dim3(64), 0, st>>>(
                    P.Xs.p, lf.start.p, lf.cell.p, nullptr, lf.chunk_box.p, lf.chunk_first.p, lf.nchunks, make_centre(P, L), lf.Vl.p,
                    base, direct_out ? y : P.ys.p, single_chunks(lf), weighted ? lf.Vl.p + lf.nb * r : nullptr, kw, perm_out);
            };
            auto l2p_long = [&](auto kern) {
                kern<<<grid_for(lf.nchunks), dim3(64), 0, st>>>(
                    P.Xs.p, lf.start.p, lf.cell.p, nullptr, lf.chunk_box.p, lf.chunk_first.p, lf.nchunks, make_centre(P, L), lf.Vl.p,
                    base, direct_out ? y : P.ys.p, weighted ? lf.Vl.p + lf.nb * r : nullptr, kw);
            };
            if (long_chunks(lf)) {
                if (weighted) l2p_long(l2p34_long_kernel<true>);
                else l2p_long(l2p34_long_kernel<false>);
            } else {
                if (weighted && perm_out) l2p(l2p34_kernel<true, true>);
                else if (weighted) l2p(l2p34_kernel<true, false>);
                else if (perm_out) l2p(l2p34_kernel<false, true>);
                else l2p(l2p34_kernel<false, false>);
            }
            F3M_HIP(hipGetLastError());
            ev[5] = now = mark();
        }
        // the lowest tree depth has no downward pass of its own
        if (P.tree_lmin < L) {
            hipEvent_t *ev = level_events(P.tree_lmin);
            ev[4] = ev[5] = now;
        }
    }
    if (side && !direct_out) {
        F3M_HIP(hipStreamWaitEvent(st, P.ev_join, 0));
        now = mark();
    }
    P.t_out = now;
    if (direct_out) {
        // written by the L2P
    } else if (box_order) {
        add_kernel<<<dim3(gn), dim3(256), 0, st>>>(P.ys.p, yn, n, y);
        F3M_HIP(hipGetLastError());
    } else if (P.route) {
        route_scatter(*P.route, P.ys.p, yn, y, P.route_a.p, P.route_b.p, st);
    } else {
        scatter_kernel<<<dim3(gn), dim3(256), 0, st>>>(P.ys.p, yn, P.perm.p, n, y);
        F3M_HIP(hipGetLastError());
    }
    P.t_end = direct_out ? now : mark();
    // A product that is being captured into a graph has no times: its event records are nodes of the graph, not
    // time stamps the host can read (f3m_stage_times then reports the stages of the plan only).
    hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
    F3M_HIP(hipStreamIsCapturing(st, &capturing));
    P.have_kmvm_times = capturing == hipStreamCaptureStatusNone;
}

// Products with several right-hand sides: column j of B (ns entries from B + j ldb) gives column j of Y
// (n entries at Y + j ldy).  Where the near field runs on the D = 3 Gram kernel, it is evaluated for groups
// of up to 4 columns at once (the exponentials, the dominant cost, are shared); everything else is done
// column by column with the kernels of the single product.  Otherwise: m single products.
void run_kmvm_multi(f3m_plan_s &P, const float *B, int64_t ldb, float *Y, int64_t ldy, int m, hipStream_t st) {
    const int64_t n = P.n, ns = P.ns();
    f3m_level &leaf = P.lev[P.L];
    const CentreArg CL = make_centre(P, P.L);
    const double gl = 1.4426950408889634 / (2.0 * (double)P.gamma * (double)P.gamma) * CL.edge * CL.edge;
    // the conditions under which the single product uses the plain D = 3 Gram kernel for its near field
    const bool fused = m > 1 && P.D == 3 && gl * 3.0 <= 6.0 && gl > 1e-30 && !P.force_all_near && P.T <= 1024 &&
                       !(P.src && P.L == 0) && P.rho == 0 && leaf.near_sz > 0 && P.exact_near() && P.ntiles >= 8192;
    if (!fused) {
        for (int j = 0; j < m; ++j) run_kmvm(P, B + (int64_t)j * ldb, Y + (int64_t)j * ldy, st);
        return;
    }
    const size_t bs_stride = (size_t)ns + PAD_POINTS;
    if (!P.multi_bs.p) {
        P.multi_bs.alloc(4 * bs_stride, &P.bytes);
        P.multi_yn.alloc(4 * (size_t)n, &P.bytes);
        fill_words((uint32_t *)P.multi_bs.p, (int64_t)(4 * bs_stride), nullptr, 0, 0u, st);   // the padding stays zero
    }
    for (int j0 = 0; j0 < m; j0 += 4) {
        const int mb = std::min(4, m - j0);
        if (mb == 1) {
            run_kmvm(P, B + (int64_t)j0 * ldb, Y + (int64_t)j0 * ldy, st);
            break;
        }
        MultiArg MA{};
        for (int j = 0; j < mb; ++j) {
            float *bsj = P.multi_bs.p + (size_t)j * bs_stride;
            if (P.sroute())
                route_gather(*P.sroute(), B + (int64_t)(j0 + j) * ldb, bsj, P.route_a.p, P.route_b.p, st);
            else
                gather_kernel<<<dim3((unsigned)cdiv(ns, 256)), dim3(256), 0, st>>>(B + (int64_t)(j0 + j) * ldb, P.sperm(), ns, bsj);
            MA.bs[j] = bsj;
            MA.ys[j] = P.multi_yn.p + (size_t)j * (size_t)n;
        }
        F3M_HIP(hipGetLastError());
        auto launch = [&](auto kern) {
            kern<<<grid_for(cdiv(P.ntiles, 4)), dim3(256), 0, st>>>(
                P.Xs.p, leaf.start.p, P.Ys(), nullptr, P.slev(P.L).start.p, leaf.cell.p, leaf.near_ptr.p, leaf.near_col.p,
                P.tile_box.p, P.tile_first.p, P.ntiles, (float)gl, (float)(1.0 / CL.edge), CL, nullptr, 0, 1, n, nullptr, MA,
                nullptr);
        };
        if (mb == 2) launch(p2p_gram3_kernel<false, 2>);
        else if (mb == 3) launch(p2p_gram3_kernel<false, 3>);
        else launch(p2p_gram3_kernel<false, 4>);
        F3M_HIP(hipGetLastError());
        if (P.notiles > 0) {
            const float nc2 = (float)(-1.4426950408889634 / (2.0 * (double)P.gamma * (double)P.gamma));
            auto overflow = [&](auto kern) {
                kern<<<grid_for(cdiv(P.notiles, 4)), dim3(256), 0, st>>>(
                    P.Xs.p, leaf.start.p, P.Ys(), nullptr, P.slev(P.L).start.p, leaf.near_ptr.p, leaf.near_col.p,
                    P.otile_box.p, P.otile_first.p, P.notiles, nc2, nullptr, 1, 0, MA);
            };
            if (mb == 2) overflow(p2p_small_kernel<3, overflow_targets(3), 2>);
            else if (mb == 3) overflow(p2p_small_kernel<3, overflow_targets(3), 3>);
            else overflow(p2p_small_kernel<3, overflow_targets(3), 4>);
            F3M_HIP(hipGetLastError());
        }
        for (int j = 0; j < mb; ++j)
            run_kmvm_d<3>(P, nullptr, Y + (int64_t)(j0 + j) * ldy, st, false, MA.bs[j], MA.ys[j]);
    }
}

void run_zero(float *y, int64_t n, hipStream_t st) {
    zero_kernel<<<dim3((unsigned)cdiv(n, 256)), dim3(256), 0, st>>>(y, n);
    F3M_HIP(hipGetLastError());
}

void run_kmvm(f3m_plan_s &P, const float *b, float *y, hipStream_t st, bool box_order) {
    switch (P.D) {
        case 1: run_kmvm_d<1>(P, b, y, st, box_order); break;
        case 2: run_kmvm_d<2>(P, b, y, st, box_order); break;
        case 3: run_kmvm_d<3>(P, b, y, st, box_order); break;
        case 4: run_kmvm_d<4>(P, b, y, st, box_order); break;
        case 5: run_kmvm_d<5>(P, b, y, st, box_order); break;
        case 6: run_kmvm_d<6>(P, b, y, st, box_order); break;
        case 7: run_kmvm_d<7>(P, b, y, st, box_order); break;
        default: fail(F3M_ERR_INVALID_ARG, "D must be in [1,7]");
    }
}

template <int D>
static void run_direct_d(const float *X, int64_t nx, const float *Y, int64_t ny, float gamma, const float *b, float *y,
                         hipStream_t st) {
    const float nc2 = (float)(-1.4426950408889634 / (2.0 * (double)gamma * (double)gamma));
    // A workgroup of direct_kernel has fixed costs (a whole tile of sources loaded, sums met across lanes and wavefronts), so
    // with few sources for the number of targets the lane per target is faster: 1e7 targets x 10 sources 41 against 605
    // us, x 200 438 against 817; 1e6 x 200 52 against 78, x 500 (even), x 1000 244 against 213; 1e5 x 100 even, x 200 13
    // against 11 (3-D).  With all SIMDs full of target lanes it needs no LDS reads and no second sum: above three
    // dimensions it then stays ahead with any number of sources (3e6 targets x 4000, 4-D to 7-D: 2 to 12 %), in fewer
    // dimensions up to some 1100.
    const bool many = nx >= (1 << 21);
    const int64_t few = std::max<int64_t>(128, std::min<int64_t>(nx / 800, D >= 4 ? 700 : many ? 1100 : 400));
    if (ny <= few || (many && D >= 4)) {
        direct_lane_kernel<D><<<dim3((unsigned)cdiv(nx, 64)), dim3(64), 0, st>>>(X, nx, Y, b, ny, nc2, y);
        F3M_HIP(hipGetLastError());
        return;
    }
    // Two targets per lane halve the LDS reads (n = 3e5, 3-D: 4.76e12 against 4.41e12 pairs/s); below 2^16 targets the
    // smaller tiles fill the compute units more evenly (n = 2e4: 8 % faster, at 5e4 1 %).
    if (nx <= 65536)
        direct_kernel<D, 16, 1><<<grid_for(cdiv(nx, 16)), dim3(DT_NT), 0, st>>>(X, nx, Y, b, ny, nc2, y);
    else
        direct_kernel<D, 16, 2><<<grid_for(cdiv(nx, 32)), dim3(DT_NT), 0, st>>>(X, nx, Y, b, ny, nc2, y);
    F3M_HIP(hipGetLastError());
}

void run_direct(const float *X, int64_t nx, const float *Y, int64_t ny, int D, float gamma, const float *b, float *y,
                hipStream_t st) {
    switch (D) {
        case 1: run_direct_d<1>(X, nx, Y, ny, gamma, b, y, st); break;
        case 2: run_direct_d<2>(X, nx, Y, ny, gamma, b, y, st); break;
        case 3: run_direct_d<3>(X, nx, Y, ny, gamma, b, y, st); break;
        case 4: run_direct_d<4>(X, nx, Y, ny, gamma, b, y, st); break;
        case 5: run_direct_d<5>(X, nx, Y, ny, gamma, b, y, st); break;
        case 6: run_direct_d<6>(X, nx, Y, ny, gamma, b, y, st); break;
        case 7: run_direct_d<7>(X, nx, Y, ny, gamma, b, y, st); break;
        default: fail(F3M_ERR_INVALID_ARG, "D must be in [1,7]");
    }
}

static int rows_slices(int64_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>(ROWS_MAX_SLICES, n / 4096)); }

// part: slices * m doubles of scratch, every entry of which the first kernel writes
template <int D>
static void run_rows_d(const float *X, const float *Y, int64_t n, float gamma, const float *b, const int64_t *rows,
                       int64_t m, double *y64, double *part, hipStream_t st) {
    const double nc2 = -1.4426950408889634074 / (2.0 * (double)gamma * (double)gamma);
    const double cap = 4096.0 / -nc2;   // 2^-4096: zero in fp64
    const int slices = rows_slices(n);
    // More rows per lane share the LDS reads of a source (m = 1e4, n = 1e6: 7.64, 7.56, 7.15 ms with 1, 2, 4 rows), but the
    // last workgroup of rows is then emptier (m = 64: 157, 205, 288 us).
    auto launch = [&](auto kern, int64_t per) {
        kern<<<dim3((unsigned)cdiv(m, per), (unsigned)slices), dim3(256), 0, st>>>(X, Y, b, n, rows, m, nc2, cap, part);
    };
    if (m <= 256) launch(rows_f64_kernel<D, 1>, 64);
    else if (m <= 2048) launch(rows_f64_kernel<D, 2>, 128);
    else launch(rows_f64_kernel<D, 4>, 256);
    F3M_HIP(hipGetLastError());
    rows_f64_sum_kernel<<<dim3((unsigned)cdiv(m, 64)), dim3(256), 0, st>>>(part, m, slices, y64);
    F3M_HIP(hipGetLastError());
}

static void run_rows(const float *X, const float *Y, int64_t ny, int D, float gamma, const float *b,
                     const int64_t *rows, int64_t m, double *y64, double *part, hipStream_t st) {
    switch (D) {
        case 1: run_rows_d<1>(X, Y, ny, gamma, b, rows, m, y64, part, st); break;
        case 2: run_rows_d<2>(X, Y, ny, gamma, b, rows, m, y64, part, st); break;
        case 3: run_rows_d<3>(X, Y, ny, gamma, b, rows, m, y64, part, st); break;
        case 4: run_rows_d<4>(X, Y, ny, gamma, b, rows, m, y64, part, st); break;
        case 5: run_rows_d<5>(X, Y, ny, gamma, b, rows, m, y64, part, st); break;
        case 6: run_rows_d<6>(X, Y, ny, gamma, b, rows, m, y64, part, st); break;
        case 7: run_rows_d<7>(X, Y, ny, gamma, b, rows, m, y64, part, st); break;
        default: fail(F3M_ERR_INVALID_ARG, "D must be in [1,7]");
    }
}

void run_direct_rows_f64(const float *X, const float *Y, int64_t ny, int D, float gamma, const float *b,
                         const int64_t *rows, int64_t m, double *y64, hipStream_t st) {
    DevBuf<double> part;
    part.alloc((size_t)rows_slices(ny) * (size_t)m);
    run_rows(X, Y, ny, D, gamma, b, rows, m, y64, part.p, st);
    F3M_HIP(hipStreamSynchronize(st));  // `part` is released on return
}

// The same sums with the partial results in the library's static device array instead of an
// allocation: nothing here allocates or frees, and nothing waits for the device.
void run_direct_rows_f64_static(const float *X, int64_t n, int D, float gamma, const float *b, const int64_t *rows,
                                int64_t m, double *y64, hipStream_t st) {
    if (m > ROWS_STATIC_MAX_M)
        fail(F3M_ERR_UNSUPPORTED, "direct_kmvm_rows_f64_static: m = " + std::to_string(m) + " rows exceed the limit of " +
                                      std::to_string(ROWS_STATIC_MAX_M) + " (the static scratch holds 256 slices of that many)");
    run_rows(X, X, n, D, gamma, b, rows, m, y64, rows_static_scratch(), st);
}

}  // namespace f3m
