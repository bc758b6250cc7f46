// Far field of a depth between POINTS, for depths whose boxes hold few of them.
//
// The interpolated kernel of a far pair of boxes (t, q) with cell offset o is a product over dimensions, and so are
// the Lagrange weights, so L_X K L_Y^T between a target x of t and a source y of q is a product of D scalars,
//   k~(x, y) = prod_d  sum_ij L_i(x_d) G_{o_d}[i][j] L_j(y_d),
// with the 1-D factors G of the node-to-node kernel matrix: the value that P2M, M2L and L2P give, in another
// order of the sums.  It costs about 4 D + 10 instructions per pair of points where the M2L reads r = p^D weights and
// runs through about 2 p r multiply-adds per pair of boxes, so it wins where the boxes of a pair hold few points
// (see far_points_pays below), and it needs no node weights, no node potentials, no far rows.
//
// A workgroup takes up to FP_TT targets of one PARENT box (a box of the depth above) and the sources of all the boxes
// near that parent, whose children are the candidates of the targets' far rows.  For target x the vectors
//   A_d[c][j] = sum_i L_i(x_d) G_o[i][j],  c = 0..5 the source's cell relative to the parent's block of 6 per dimension
// lie in LDS with o^2 as a fourth entry: a lane (= one source) reads the entry of its own c, 16 bytes per dimension,
// multiplies it with its L_j(y_d), and the sum of the o^2 tells whether the pair of boxes is far.  Bound: the LDS reads,
// D x 1 KB per 64 pairs (at D = 7 28 cycles of a compute unit at 256 bytes per cycle), beside 41 vector instructions.
// Measured at n = 1e7, D = 7, 3 nodes: a 128-bit LDS read every 3.98 cycles of a compute unit, their full rate, at a clock
// of 1.98 GHz; 1.0e12 pairs/s at n = 3e5.
#include <algorithm>
#include <cmath>

#include "plan.h"

namespace f3m {
namespace {

constexpr int FP_ROW = 256;   // near boxes of the parent taken at once

struct FpGrid {
    double alpha[F3M_MAX_DIM];
    double edge, inv_half;   // of the boxes of the depth
    int level, shift;        // depth, and bits of a key below it
};

// Per point of the depth, 32 bytes: the local coordinates in its box (formed in fp64, as P2M and L2P form them) and in
// the last word the child bits of its box.
template <int D>
__global__ __launch_bounds__(256) void far_points_prepare_kernel(const float *__restrict__ Xs,
                                                                 const uint32_t *__restrict__ keys, int64_t n, FpGrid C,
                                                                 float4 *__restrict__ loc) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= n) return;
    const uint32_t key = keys[k] >> C.shift;
    float t[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int d = 0; d < D; ++d) {
        int32_t c = 0;
        for (int b = 0; b < C.level; ++b) c |= (int32_t)((key >> (b * D + d)) & 1u) << b;
        const double centre = C.alpha[d] + ((double)c + 0.5) * C.edge;
        t[d] = (float)(((double)Xs[k * D + d] - centre) * C.inv_half);
    }
    t[7] = __uint_as_float(key & ((1u << D) - 1u));
    loc[2 * k] = make_float4(t[0], t[1], t[2], t[3]);
    loc[2 * k + 1] = make_float4(t[4], t[5], t[6], t[7]);
}

// Lagrange basis on the nodes {1, 0, -1} or {1, -1}
template <int PN>
__device__ inline void basis(float t, float (&L)[PN]) {
    if constexpr (PN == 3) {
        L[0] = 0.5f * (t * (t + 1.f));
        L[1] = (1.f - t) * (1.f + t);
        L[2] = 0.5f * (t * (t - 1.f));
    } else {
        L[0] = 0.5f * (1.f + t);
        L[1] = 0.5f * (1.f - t);
    }
}

// ys += far field of the depth.  tile_box: the parent of every tile; G: [D][no][PN][PN]; Tmin: smallest squared cell
// offset of a far pair.
template <int D, int PN>
__global__ __launch_bounds__(256) void far_points_kernel(const float4 *__restrict__ loc, const float *__restrict__ bs,
                                                         const uint32_t *__restrict__ up_start,
                                                         const int32_t *__restrict__ up_cell,
                                                         const uint64_t *__restrict__ up_near_ptr,
                                                         const uint32_t *__restrict__ up_near_col,
                                                         const uint32_t *__restrict__ tile_box,
                                                         const uint32_t *__restrict__ tile_first, int64_t ntiles,
                                                         const float *__restrict__ G, int omin, int no, float Tmin,
                                                         float *__restrict__ ys) {
    __shared__ float4 tab[FP_TT][D][6];
    __shared__ uint32_t rend[FP_ROW], rdelta[FP_ROW], rcode[FP_ROW];
    __shared__ uint32_t wsum[4];
    __shared__ float red[4][FP_TT];
    const int64_t tile = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    if (tile >= ntiles) return;   // uniform over the workgroup
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const uint32_t P = tile_box[tile];
    const uint32_t k0 = up_start[P] + (uint32_t)(tile - tile_first[P]) * (uint32_t)FP_TT;
    const int nt = (int)min((uint32_t)FP_TT, up_start[P + 1] - k0);
    int32_t pc[D];
#pragma unroll
    for (int d = 0; d < D; ++d) pc[d] = up_cell[(int64_t)P * D + d];
    for (int i = tid; i < nt * D * 6; i += 256) {
        const int t = i / (D * 6), d = (i / 6) % D, c = i % 6;
        const float *row = (const float *)(loc + 2 * ((int64_t)k0 + t));
        float L[PN];
        basis<PN>(row[d], L);
        const int o = c - 2 - (int)((__float_as_uint(row[7]) >> d) & 1u);
        const int k = min(max(o - omin, 0), no - 1);   // offsets no pair of cells has are not tabulated
        const float *g = G + ((int64_t)d * no + k) * (PN * PN);
        float v[3] = {0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < PN; ++j) {
            float s = 0.f;
#pragma unroll
            for (int q = 0; q < PN; ++q) s = fmaf(L[q], g[q * PN + j], s);
            v[j] = s;
        }
        tab[t][d][c] = make_float4(v[0], v[1], v[2], (float)(o * o));
    }
    float acc[FP_TT];
#pragma unroll
    for (int t = 0; t < FP_TT; ++t) acc[t] = 0.f;

    const uint64_t e0 = up_near_ptr[P], e1 = up_near_ptr[P + 1];
    for (uint64_t er = e0; er < e1; er += FP_ROW) {
        const int m = (int)(e1 - er < FP_ROW ? e1 - er : FP_ROW);
        uint32_t first = 0, len = 0, code = 0;
        if (tid < m) {
            const uint32_t q = up_near_col[er + tid];
            first = up_start[q];
            len = up_start[q + 1] - first;
#pragma unroll
            for (int d = 0; d < D; ++d) code |= (uint32_t)(up_cell[(int64_t)q * D + d] - pc[d] + 1) << (2 * d);
        }
        const uint32_t incl = wave_incl_scan_u32(len);
        __syncthreads();   // the table is in place, the last round has read its row
        if (lane == 63) wsum[w] = incl;
        __syncthreads();
        uint32_t base = 0, S = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t s = wsum[k];
            base += k < w ? s : 0u;
            S += s;
        }
        rend[tid] = base + incl;
        rdelta[tid] = first - (base + incl - len);   // position in the row -> source (mod 2^32)
        rcode[tid] = code;
        __syncthreads();
        for (uint32_t w0 = 64u * (uint32_t)w; w0 < S; w0 += 256u) {
            const uint32_t p = min(w0 + (uint32_t)lane, S - 1u);
            // first entry with rend > p (it exists: p < S = rend of the last entry)
            int lo = 0;
#pragma unroll
            for (int s = FP_ROW / 2; s > 0; s >>= 1) lo += rend[lo + s - 1] <= p ? s : 0;
            const uint32_t src = p + rdelta[lo];
            const uint32_t qc = rcode[lo];
            const float4 l0 = loc[2 * (int64_t)src], l1 = loc[2 * (int64_t)src + 1];
            const float b = w0 + (uint32_t)lane < S ? bs[src] : 0.f;
            const float x[8] = {l0.x, l0.y, l0.z, l0.w, l1.x, l1.y, l1.z, l1.w};
            const uint32_t bits = __float_as_uint(l1.w);
            float L[D][PN];
            int at[D];
#pragma unroll
            for (int d = 0; d < D; ++d) {
                basis<PN>(x[d], L[d]);
                at[d] = (int)(((qc >> (2 * d)) & 3u) * 2u + ((bits >> d) & 1u));
            }
#pragma unroll
            for (int t = 0; t < FP_TT; ++t) {
                if (t < nt) {   // uniform
                    float prod = 1.f, d2 = 0.f;
#pragma unroll
                    for (int d = 0; d < D; ++d) {
                        const float4 A = tab[t][d][at[d]];
                        float s = A.x * L[d][0];
                        s = fmaf(A.y, L[d][1], s);
                        if constexpr (PN == 3) s = fmaf(A.z, L[d][2], s);
                        prod = d ? prod * s : s;
                        d2 = d ? d2 + A.w : A.w;
                    }
                    acc[t] = fmaf(prod, d2 >= Tmin ? b : 0.f, acc[t]);
                }
            }
        }
    }
#pragma unroll
    for (int t = 0; t < FP_TT; ++t) {
        float v = acc[t];
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
        if (lane == 0) red[w][t] = v;
    }
    __syncthreads();
    if (tid < nt) ys[(int64_t)k0 + tid] += (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]);
}

FpGrid make_grid(const f3m_plan_s &P, int level) {
    FpGrid g{};
    for (int d = 0; d < P.D; ++d) g.alpha[d] = (double)P.alpha[d];
    g.edge = (double)P.E / std::ldexp(1.0, level);
    g.inv_half = 2.0 / g.edge;
    g.level = level;
    g.shift = P.D * (P.Lq - level);
    return g;
}

}  // namespace

// The far pairs of a depth can be taken point by point: one point set, the plain far rule with a ratio of at most 2
// (the boxes near a parent are at most one cell away per dimension: six cells of candidates) or the smooth depth, no
// small field, two or three nodes per dimension, more than three dimensions.
bool far_points_allowed(const f3m_plan_s &P, int level) {
    const f3m_level &lv = P.lev[level];
    return P.D >= 4 && !P.src && P.T <= 4 && P.rho == 0 && !P.force_all_near && (lv.p == 2 || lv.p == 3);
}

// Point pairs (of the near boxes one depth up: what the kernel goes through) against r per far pair of boxes.  Measured on
// clustered points in 4 to 7 dimensions: 0.65 to 1.1 ps a point pair; P2M, M2L and L2P of a depth 0.8 to 1.1 ps a far pair
// and node with more than 512 nodes, 2 to 5 ps with fewer.  At n = 3e5, D = 7, 3 nodes: 4.4e9 point pairs in 4.4 ms where
// 4.3e8 far pairs of boxes took 648 ms, 1.7e10 in 17 ms against 44 ms, and 4.9e10 in 45 ms against 6.4 ms, which stay
// with the boxes.
bool far_points_pays(const f3m_plan_s &P, int level, int64_t point_pairs) {
    const f3m_level &lv = P.lev[level];
    return (lv.r > 512 ? 1.0 : 0.5) * (double)point_pairs <= (double)lv.far_sz * (double)lv.r;
}

void far_points_prepare(f3m_plan_s &P, int level, hipStream_t st) {
    f3m_level &lv = P.lev[level];
    lv.fp_loc.alloc((size_t)P.n * 8, &P.bytes);
    const FpGrid C = make_grid(P, level);
    const dim3 grid((unsigned)cdiv(P.n, 256));
    auto launch = [&](auto kern) { kern<<<grid, dim3(256), 0, st>>>(P.Xs.p, P.keys.p, P.n, C, (float4 *)lv.fp_loc.p); };
    switch (P.D) {
        case 4: launch(far_points_prepare_kernel<4>); break;
        case 5: launch(far_points_prepare_kernel<5>); break;
        case 6: launch(far_points_prepare_kernel<6>); break;
        default: launch(far_points_prepare_kernel<7>); break;
    }
    F3M_HIP(hipGetLastError());
}

void run_far_points(f3m_plan_s &P, int level, const float *bs, float *ys, int omin, int no, hipStream_t st) {
    f3m_level &lv = P.lev[level], &up = P.lev[level - 1];
    const float Tmin = lv.smooth ? -1.f : (float)P.T;
    const int64_t gx = std::min<int64_t>(lv.fp_ntiles, 1 << 16);
    const dim3 grid((unsigned)gx, (unsigned)cdiv(lv.fp_ntiles, gx));
    auto launch = [&](auto kern) {
        kern<<<grid, dim3(256), 0, st>>>((const float4 *)lv.fp_loc.p, bs, up.start.p, up.cell.p, up.near_ptr.p, up.near_col.p,
                                         lv.fp_tile_box.p, lv.fp_tile_first.p, lv.fp_ntiles, lv.gtab.p, omin, no, Tmin, ys);
    };
    switch (lv.p * 8 + P.D) {
        case 2 * 8 + 4: launch(far_points_kernel<4, 2>); break;
        case 2 * 8 + 5: launch(far_points_kernel<5, 2>); break;
        case 2 * 8 + 6: launch(far_points_kernel<6, 2>); break;
        case 2 * 8 + 7: launch(far_points_kernel<7, 2>); break;
        case 3 * 8 + 4: launch(far_points_kernel<4, 3>); break;
        case 3 * 8 + 5: launch(far_points_kernel<5, 3>); break;
        case 3 * 8 + 6: launch(far_points_kernel<6, 3>); break;
        case 3 * 8 + 7: launch(far_points_kernel<7, 3>); break;
        default: fail(F3M_ERR_HIP, "internal: no point-wise far field for this number of nodes and dimensions");
    }
    F3M_HIP(hipGetLastError());
}

}  // namespace f3m
