// M2L, v2 = K v1 (arXiv 2202.01085, Sec. 3 "Interpolating k(x,y)", Fig. 4 step 2), for D = 3
// with 4 nodes per dimension (r = 64 nodes per box) and the paper's far rule (ratio 2).
// Everything else (other D, node counts, far ratios) takes the Kronecker-factor kernels in kmvm.hip.
#include <algorithm>
#include <cmath>

#include "plan.h"

namespace f3m {

static dim3 grid2(int64_t count) {
    const int64_t gx = 1 << 16;
    if (count <= gx) return dim3((unsigned)(count > 0 ? count : 1), 1, 1);
    return dim3((unsigned)gx, (unsigned)cdiv(count, gx), 1);
}
__device__ inline int64_t block_index2() { return (int64_t)blockIdx.y * gridDim.x + blockIdx.x; }

// (one point set only: the candidate grid assumes that targets and sources share a grid)
bool m2l_stencil_applies(const f3m_plan_s &P) {
    return P.D == 3 && P.p == 4 && P.T == 4 && !P.force_all_near && !P.src;
}

// ------------------------------------------------------------------------------------
// M2L by sum factorisation over the candidate grid (D = 3, 4 nodes per dimension, far ratio 2).
//
// The Gaussian is a product over dimensions and the nodes are a tensor grid, so the node-to-node
// matrix of a far pair with cell offset o is G_{o_z} x G_{o_y} x G_{o_x} (Kronecker product of
// 4 x 4 factors, G_o[i][j] = exp(-(l/2)^2 (2 o + s_j - s_i)^2 / (2 gamma^2))).  The candidates
// of a target are the children of the boxes near its parent: a 6 x 6 x 6 grid of cells around
// the parent, of which the 3 x 3 x 3 block around the target is near and the rest far.  Hence
//   V_t = sum_cz G_{o_z} [ sum_cy G_{o_y} [ sum_{cx far} G_{o_x} W_(cx,cy,cz) ] ]
// with the x factor applied once per far candidate (189), the y factor once per line of the
// grid (36) and the z factor once per plane (6): the same sums as 189 dense 64 x 64 products,
// reordered, in 231 x 256 instead of 189 x 4096 multiply-adds.
//
// One workgroup per parent box: its 8 wavefronts first copy the node weights of all
// candidates (<= 216 rows of 64 floats, read once per parent instead of once per target)
// into LDS at their grid position, then wavefront w handles the child with parity w: lane =
// node (ix + 4 iy + 16 iz).  The x factor needs the other three entries of the lane's quad:
// DPP quad permutations; the y and z factors use ds_bpermute.  The factor entries a lane
// needs (6 candidate coordinates x 4 rotations x 3 dimensions) sit in registers.
// ------------------------------------------------------------------------------------
constexpr int ST_CAND = 216;

__global__ __launch_bounds__(512) void m2l_stencil_kernel(const uint64_t *__restrict__ up_near_ptr,
                                                          const uint32_t *__restrict__ up_near_col,
                                                          const uint32_t *__restrict__ up_cstart,
                                                          const int32_t *__restrict__ up_cell,
                                                          const int32_t *__restrict__ cell,
                                                          const uint32_t *__restrict__ key, int64_t nparents,
                                                          int64_t per_xcd, const float *__restrict__ G, int all_far,
                                                          const uint32_t *__restrict__ start, uint32_t rho,
                                                          const float *__restrict__ W, float *__restrict__ V) {
    __shared__ float rows[ST_CAND * 64];
    __shared__ int present[ST_CAND];
    __shared__ uint32_t cand[ST_CAND];      // candidate k of near parent j at [8 j + k]: rank or ~0
    __shared__ int cpos[ST_CAND];           // its position in the 6 x 6 x 6 grid
    __shared__ uint32_t ccnt[ST_CAND];      // points of the candidate at a grid position (small-field rule)
    __shared__ uint32_t qfirst[27], qcount[27];
    __shared__ float gs[7 * 16];            // the factor table
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    // consecutive parents (neighbours in space) on the same XCD, so that its L2 serves the overlap
    const int64_t bi = block_index2();
    const int64_t pb = (bi & 7) * per_xcd + (bi >> 3);
    if ((bi >> 3) >= per_xcd || pb >= nparents) return;
    // the boxes near the parent (at most 27 with far ratio 2) and their child ranges
    if (tid < 27) {
        const uint64_t e = up_near_ptr[pb] + tid;
        uint32_t first = 0, count = 0;
        if (e < up_near_ptr[pb + 1]) {
            const uint32_t q = up_near_col[e];
            first = up_cstart[q];
            count = up_cstart[q + 1] - first;
        }
        qfirst[tid] = first;
        qcount[tid] = count;
    }
    if (tid < ST_CAND) present[tid] = 0;
    if (tid >= 256 && tid < 256 + 7 * 16) gs[tid - 256] = G[tid - 256];
    __syncthreads();
    if (tid < ST_CAND) {
        const int j = tid >> 3, k = tid & 7;
        uint32_t c = 0xFFFFFFFFu;
        if ((uint32_t)k < qcount[j]) {
            c = qfirst[j] + k;
            const int px = cell[(int64_t)c * 3] - 2 * up_cell[pb * 3] + 2,
                      py = cell[(int64_t)c * 3 + 1] - 2 * up_cell[pb * 3 + 1] + 2,
                      pz = cell[(int64_t)c * 3 + 2] - 2 * up_cell[pb * 3 + 2] + 2;
            const int pos = px + 6 * py + 36 * pz;     // in [0, 216): the near box is within one cell of the parent
            cpos[tid] = pos;
            present[pos] = 1;
            if (rho) ccnt[pos] = start[c + 1] - start[c];
        }
        cand[tid] = c;
    }
    __syncthreads();
    // node weights of the candidates into LDS: 27 rows per wavefront, all loads in flight together
    {
        float tmp[27];
#pragma unroll
        for (int i = 0; i < 27; ++i) {
            const uint32_t c = cand[w + 8 * i];
            tmp[i] = W[(int64_t)(c == 0xFFFFFFFFu ? 0u : c) * 64 + lane];
        }
#pragma unroll
        for (int i = 0; i < 27; ++i)
            if (cand[w + 8 * i] != 0xFFFFFFFFu) rows[cpos[w + 8 * i] * 64 + lane] = tmp[i];
    }
    __syncthreads();
    // the child with parity w, if it exists (no barrier below this point)
    uint32_t t = 0xFFFFFFFFu;
    for (uint32_t c = up_cstart[pb]; c < up_cstart[pb + 1]; ++c)
        if ((key[c] & 7u) == (uint32_t)w) t = c;
    if (t == 0xFFFFFFFFu) return;
    const int tx = w & 1, ty = (w >> 1) & 1, tz = w >> 2;
    const uint32_t tcnt = rho ? start[t + 1] - start[t] : 0u;
    // far and present candidates, one bit each: bit cx + 8 (cy + 6 cz), so that the six bits of a
    // line of the grid sit in one byte
    uint64_t mask[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        const int mm = lane + 64 * k, cx = mm & 7, ln = mm >> 3;
        bool ok = false;
        if (cx < 6 && ln < 36) {
            const int cy = ln % 6, cz = ln / 6;
            const int ox = cx - 2 - tx, oy = cy - 2 - ty, oz = cz - 2 - tz;
            // all_far: the smooth depth of Sec. 4.3, where adjacent pairs are interpolated too
            ok = present[cx + 6 * ln] != 0 && (all_far || ox * ox + oy * oy + oz * oz >= 4);
            // small field (Sec. 4.2): a pair with at most rho points is summed directly elsewhere
            if (ok && rho && tcnt + ccnt[cx + 6 * ln] <= rho) ok = false;
        }
        mask[k] = __ballot(ok);
    }
    const int ix = lane & 3, iy = (lane >> 2) & 3, iz = lane >> 4;
    // factor entries: candidate coordinate c (offset c - 2 - t_d), rotation k -> G_o[i][(i + k) % 4]
    float fx[6][4], fy[6][4], fz[6][4];
#pragma unroll
    for (int c = 0; c < 6; ++c)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            fx[c][k] = gs[(c + 1 - tx) * 16 + ix * 4 + ((ix + k) & 3)];
            fy[c][k] = gs[(c + 1 - ty) * 16 + iy * 4 + ((iy + k) & 3)];
            fz[c][k] = gs[(c + 1 - tz) * 16 + iz * 4 + ((iz + k) & 3)];
        }
    int ylane[4], zlane[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        ylane[k] = ix + 4 * ((iy + k) & 3) + 16 * iz;
        zlane[k] = ix + 4 * iy + 16 * ((iz + k) & 3);
    }
    float acc = 0.f;
#pragma unroll
    for (int cz = 0; cz < 6; ++cz) {
        float plane = 0.f;
#pragma unroll
        for (int cy = 0; cy < 6; ++cy) {
            float line = 0.f;
            // the six rows of the line are read unconditionally (rows of absent candidates hold
            // stale data and are skipped below), so one wait covers them
            float v[6];
#pragma unroll
            for (int cx = 0; cx < 6; ++cx) v[cx] = rows[(cx + 6 * cy + 36 * cz) * 64 + lane];
            // line += sum_k fx[cx][k] * (entry k places further in the lane's quad); the row value
            // comes straight from the LDS read, so no vector-ALU write precedes the DPP reads of it
            auto xfactor = [&](int cx) {
                asm("v_fmac_f32 %0, %2, %1\n\t"
                    "v_fmac_f32_dpp %0, %1, %3 quad_perm:[1,2,3,0] row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
                    "v_fmac_f32_dpp %0, %1, %4 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
                    "v_fmac_f32_dpp %0, %1, %5 quad_perm:[3,0,1,2] row_mask:0xf bank_mask:0xf bound_ctrl:1"
                    : "+v"(line)
                    : "v"(v[cx]), "v"(fx[cx][0]), "v"(fx[cx][1]), "v"(fx[cx][2]), "v"(fx[cx][3]));
            };
            const int ln = cy + 6 * cz;
            const uint32_t bits = (uint32_t)(mask[ln >> 3] >> (8 * (ln & 7))) & 0x3Fu;
            if (bits == 0x3Fu) {   // the whole line is far and present: no tests
#pragma unroll
                for (int cx = 0; cx < 6; ++cx) xfactor(cx);
            } else {
#pragma unroll
                for (int cx = 0; cx < 6; ++cx)
                    if ((bits >> cx) & 1u) xfactor(cx);
            }
            // y factor: the lane needs the entries 4, 8, 12 lanes further on in its row of 16
            // lanes (cyclically): row rotations by 12, 8, 4 to the right
            // (`line` was last written by a vector-ALU instruction: the plain multiply-add and
            // the s_nop give the two wait states that a DPP read of it needs)
            asm("v_fmac_f32 %0, %2, %1\n\t"
                "s_nop 0\n\t"
                "v_fmac_f32_dpp %0, %1, %3 row_ror:12 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
                "v_fmac_f32_dpp %0, %1, %4 row_ror:8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
                "v_fmac_f32_dpp %0, %1, %5 row_ror:4 row_mask:0xf bank_mask:0xf bound_ctrl:1"
                : "+v"(plane)
                : "v"(line), "v"(fy[cy][0]), "v"(fy[cy][1]), "v"(fy[cy][2]), "v"(fy[cy][3]));
        }
        acc = fmaf(fz[cz][0], plane, acc);
#pragma unroll
        for (int k = 1; k < 4; ++k) acc = fmaf(fz[cz][k], __shfl(plane, zlane[k], 64), acc);
    }
    V[(int64_t)t * 64 + lane] = acc;
}

// ------------------------------------------------------------------------------------
// The same sums with the work shared between the eight children of a parent (no small field).
// The far sum of a target is the sum over ALL candidates of the 6 x 6 x 6 grid minus the sum over
// the 3 x 3 x 3 block around the target, and the sum over all candidates factorises further: the
// x factor of a candidate depends on the target's x parity only, so the line sums
//   X_tx(cy, cz) = sum_cx G_{cx-2-tx} W_(cx,cy,cz)              2 x 36 lines, 6 applications each
// serve four targets each, the plane sums
//   Y_{tx,ty}(cz) = sum_cy G_{cy-2-ty} X_tx(cy, cz)             4 x 6 planes, 6 applications each
// serve two, and a target needs only
//   V_all = sum_cz G_{cz-2-tz} Y_{tx,ty}(cz)                    6 applications
// from which the same sums over the near block are taken plane by plane.  The near candidates of a line are the first
// three applications of its sum, so they cost nothing; their 4 x 4 plane sums take 3 applications each.
// Per parent 432 + 144 + 48 + 48 = 672 applications of a 4 x 4 factor to a 64-vector instead of 8 x 231.  The rows of
// the candidates go from memory into the registers of the wavefront that sums their line, zeros for absent ones: no
// masks, and with 37 KB of LDS three workgroups share a compute unit (with the rows in LDS, 80 KB, it was two, and
// the kernel waits at its barriers: plan and product of 1e6 normal points
// 2.63 -> 2.35 ms, of 1e7 points the product 2.63 -> 2.45, four columns of 3e6 points 4.51 -> 3.78).  The
// subtraction costs no accuracy that matters: |near part| / |far part| is of order one for wide
// kernels, and for narrow ones both are part of a result dominated by the near field itself.
// all_far (the smooth depth of Sec. 4.3, every candidate interpolated): no subtraction.
// ------------------------------------------------------------------------------------
// tables for it, made once per plan and depth: for every parent the rank of the candidate at each
// position of its 6 x 6 x 6 grid (~0: no such box) and its child of each parity (~0: none), so that a
// workgroup starts with one table read instead of a chain of four dependent ones (near list ->
// child ranges -> cells -> rows), which is what bounded the kernel
__global__ __launch_bounds__(256) void stencil_table_kernel(const uint64_t *__restrict__ up_near_ptr,
                                                            const uint32_t *__restrict__ up_near_col,
                                                            const uint32_t *__restrict__ up_cstart,
                                                            const int32_t *__restrict__ up_cell,
                                                            const int32_t *__restrict__ cell,
                                                            const uint32_t *__restrict__ key, int64_t nparents,
                                                            uint32_t *__restrict__ cand_tab,
                                                            uint32_t *__restrict__ child_tab) {
    const int64_t pb = block_index2();
    if (pb >= nparents) return;
    const int tid = threadIdx.x;
    if (tid < ST_CAND) {
        const int j = tid >> 3, k = tid & 7;
        const uint64_t e = up_near_ptr[pb] + j;
        if (e < up_near_ptr[pb + 1]) {
            const uint32_t q = up_near_col[e];
            const uint32_t first = up_cstart[q], count = up_cstart[q + 1] - first;
            if ((uint32_t)k < count) {
                const uint32_t c = first + k;
                const int px = cell[(int64_t)c * 3] - 2 * up_cell[pb * 3] + 2,
                          py = cell[(int64_t)c * 3 + 1] - 2 * up_cell[pb * 3 + 1] + 2,
                          pz = cell[(int64_t)c * 3 + 2] - 2 * up_cell[pb * 3 + 2] + 2;
                // in [0, 6) each: a near box is within one cell of the parent
                cand_tab[pb * ST_CAND + px + 6 * py + 36 * pz] = c;
            }
        }
    } else if (tid < ST_CAND + 8) {
        const uint32_t w = (uint32_t)(tid - ST_CAND);
        for (uint32_t c = up_cstart[pb]; c < up_cstart[pb + 1]; ++c)
            if ((key[c] & 7u) == w) child_tab[pb * 8 + w] = c;
    }
}

// ZROW: W has a row of zeros behind its last box (index zero_row): an absent candidate (~0 in the table)
// reads that row, which saves the compare-and-select pairs around every load.
// Several depths with few parents share a launch (their M2L do not depend on each other): the workgroups from first[k] on are
// those of entry k.
struct M2lDepths {
    static constexpr int MAX = 6;
    const uint32_t *cand[MAX], *child[MAX];
    const float *G[MAX], *W[MAX];
    float *V[MAX];
    uint32_t first[MAX], nparents[MAX], zero_row[MAX];
    int all_far[MAX];
    int count = 0;
};
template <bool ZROW>
__global__ __launch_bounds__(512) void m2l_stencil_shared_kernel(M2lDepths A) {
    __shared__ float xl[2 * 36 * 64];       // X_tx(cy, cz) at [(tx * 36 + cy + 6 cz) * 64 + node]
    __shared__ float xn[2 * 16 * 64];       // the same over the near candidates only, 1 <= cy, cz <= 4
    __shared__ float yp[4 * 6 * 64];        // Y_{tx,ty}(cz) at [((tx + 2 ty) * 6 + cz) * 64 + node]
    __shared__ float yn[4 * 4 * 64];        // near, 1 <= cz <= 4
    __shared__ float gs[7 * 16];            // the factor table
    // (the wavefront's number in a scalar register: ranks and row addresses are then scalar work)
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    int e = 0;
#pragma unroll
    for (int k = 1; k < M2lDepths::MAX; ++k)
        if (k < A.count && blockIdx.x >= A.first[k]) e = k;
    const uint32_t *__restrict__ cand_tab = A.cand[e], *__restrict__ child_tab = A.child[e];
    const float *__restrict__ W = A.W[e];
    float *__restrict__ V = A.V[e];
    const uint32_t zero_row = A.zero_row[e];
    const int all_far = A.all_far[e];
    // consecutive parents (neighbours in space) on the same XCD, so that its L2 serves the overlap
    const uint32_t bi = blockIdx.x - A.first[e], per_xcd = (A.nparents[e] + 7) / 8;
    const int64_t pb = (int64_t)(bi & 7) * per_xcd + (bi >> 3);
    if ((bi >> 3) >= per_xcd || pb >= (int64_t)A.nparents[e]) return;
    if (tid < 7 * 16) gs[tid] = A.G[e][tid];
    const uint32_t t = child_tab[pb * 8 + w];   // the child with parity w (wave-uniform), or ~0
    // lines w + 8 i of six candidates each, i = 0..4: node weights straight into registers (zeros for absent
    // candidates), all loads in flight together
    constexpr int NL = 5;
    float v[NL][6];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const int ln = min(w + 8 * i, 35);   // (wavefronts 4 to 7 have four lines: the fifth is not used)
        const uint32_t *cand = cand_tab + pb * ST_CAND + 6 * ln;
#pragma unroll
        for (int cx = 0; cx < 6; ++cx) {
            const uint32_t c = cand[cx];
            if constexpr (ZROW) v[i][cx] = W[(int64_t)min(c, zero_row) * 64 + lane];
            else {
                const float val = W[(int64_t)(c == 0xFFFFFFFFu ? 0u : c) * 64 + lane];
                v[i][cx] = c == 0xFFFFFFFFu ? 0.f : val;
            }
        }
    }
    __syncthreads();
    const int tx = w & 1, ty = (w >> 1) & 1, tz = w >> 2;
    const int ix = lane & 3, iy = (lane >> 2) & 3, iz = lane >> 4;
    // out += sum_k f[k] * (entry k places further on in the lane's quad / row of 16 / wavefront).  A DPP operand must not
    // have been written by one of the last two vector instructions: the x factors of both parities are applied in one
    // block that starts with two ordinary multiply-adds, the y factor waits.
    auto xfirst2 = [&](float &out0, float &out1, float v0, float v1, const float (&f)[4]) {   // the same factor, two inputs
        asm("v_mul_f32 %0, %4, %2\n\t"
            "v_mul_f32 %1, %4, %3\n\t"
            "v_fmac_f32_dpp %0, %2, %5 quad_perm:[1,2,3,0] row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %1, %3, %5 quad_perm:[1,2,3,0] row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %0, %2, %6 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %1, %3, %6 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %0, %2, %7 quad_perm:[3,0,1,2] row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %1, %3, %7 quad_perm:[3,0,1,2] row_mask:0xf bank_mask:0xf bound_ctrl:1"
            : "=&v"(out0), "=&v"(out1)
            : "v"(v0), "v"(v1), "v"(f[0]), "v"(f[1]), "v"(f[2]), "v"(f[3]));
    };
    auto xapply2 = [&](float &out0, float &out1, float v0, float v1, const float (&f)[4]) {
        asm("v_fmac_f32 %0, %4, %2\n\t"
            "v_fmac_f32 %1, %4, %3\n\t"
            "v_fmac_f32_dpp %0, %2, %5 quad_perm:[1,2,3,0] row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %1, %3, %5 quad_perm:[1,2,3,0] row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %0, %2, %6 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %1, %3, %6 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %0, %2, %7 quad_perm:[3,0,1,2] row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %1, %3, %7 quad_perm:[3,0,1,2] row_mask:0xf bank_mask:0xf bound_ctrl:1"
            : "+&v"(out0), "+&v"(out1)
            : "v"(v0), "v"(v1), "v"(f[0]), "v"(f[1]), "v"(f[2]), "v"(f[3]));
    };
    auto xapply2d = [&](float &out0, float &out1, float v0, float v1, const float (&f)[4], const float (&h)[4]) {
        asm("v_fmac_f32 %0, %4, %2\n\t"
            "v_fmac_f32 %1, %8, %3\n\t"
            "v_fmac_f32_dpp %0, %2, %5 quad_perm:[1,2,3,0] row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %1, %3, %9 quad_perm:[1,2,3,0] row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %0, %2, %6 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %1, %3, %10 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %0, %2, %7 quad_perm:[3,0,1,2] row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %1, %3, %11 quad_perm:[3,0,1,2] row_mask:0xf bank_mask:0xf bound_ctrl:1"
            : "+&v"(out0), "+&v"(out1)
            : "v"(v0), "v"(v1), "v"(f[0]), "v"(f[1]), "v"(f[2]), "v"(f[3]), "v"(h[0]), "v"(h[1]), "v"(h[2]), "v"(h[3]));
    };
    auto yapply = [&](float &out, float v, const float (&f)[4]) {
        asm("v_fmac_f32 %0, %2, %1\n\t"
            "s_nop 0\n\t"
            "v_fmac_f32_dpp %0, %1, %3 row_ror:12 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %0, %1, %4 row_ror:8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %0, %1, %5 row_ror:4 row_mask:0xf bank_mask:0xf bound_ctrl:1"
            : "+v"(out)
            : "v"(v), "v"(f[0]), "v"(f[1]), "v"(f[2]), "v"(f[3]));
    };
    // the first application of a sum: out = ..., no zeroed accumulator to start from
    auto yfirst = [&](float &out, float v, const float (&f)[4]) {
        asm("v_mul_f32 %0, %2, %1\n\t"
            "s_nop 0\n\t"
            "v_fmac_f32_dpp %0, %1, %3 row_ror:12 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %0, %1, %4 row_ror:8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            "v_fmac_f32_dpp %0, %1, %5 row_ror:4 row_mask:0xf bank_mask:0xf bound_ctrl:1"
            : "=&v"(out)
            : "v"(v), "v"(f[0]), "v"(f[1]), "v"(f[2]), "v"(f[3]));
    };
    int zlane[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) zlane[k] = ix + 4 * iy + 16 * ((iz + k) & 3);
    auto zapply = [&](float &out, float v, const float (&f)[4]) {
        out = fmaf(f[0], v, out);
#pragma unroll
        for (int k = 1; k < 4; ++k) out = fmaf(f[k], __shfl(v, zlane[k], 64), out);
    };
    // factor entries for candidate coordinate c and target parity t: offset c - 2 - t, rotation k
    auto factor = [&](int c, int t, int i, float (&f)[4]) {
#pragma unroll
        for (int k = 0; k < 4; ++k) f[k] = gs[(c + 1 - t) * 16 + i * 4 + ((i + k) & 3)];
    };

    // ---- line sums over x for both parities.  Parity 0 has offset c - 2 from candidate c, parity 1 c - 3: table
    // entries c + 1 and c, so candidate c of parity 0 and c + 1 of parity 1 share a factor.  The near candidates
    // (c = 1..3 and 2..4, entries 2, 3, 4) come first, and their sum is kept where the line is near in y and z.
    {
        float fx[7][4];
#pragma unroll
        for (int e = 0; e < 7; ++e) factor(e, 1, ix, fx[e]);
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int ln = w + 8 * i;
            if (ln < 36) {   // wave-uniform
                float l0, l1;
                xfirst2(l0, l1, v[i][1], v[i][2], fx[2]);
                xapply2(l0, l1, v[i][2], v[i][3], fx[3]);
                xapply2(l0, l1, v[i][3], v[i][4], fx[4]);
                const int cy = ln % 6, cz = ln / 6;
                if (!all_far && cy >= 1 && cy <= 4 && cz >= 1 && cz <= 4) {
                    xn[(cy - 1 + 4 * (cz - 1)) * 64 + lane] = l0;
                    xn[(16 + cy - 1 + 4 * (cz - 1)) * 64 + lane] = l1;
                }
                xapply2(l0, l1, v[i][0], v[i][1], fx[1]);
                xapply2(l0, l1, v[i][4], v[i][5], fx[5]);
                xapply2d(l0, l1, v[i][5], v[i][0], fx[6], fx[0]);
                xl[ln * 64 + lane] = l0;
                xl[(36 + ln) * 64 + lane] = l1;
            }
        }
    }
    __syncthreads();
    // ---- plane sums over y: wavefront w takes the parities (w & 3) and the planes 3 (w >> 2) .. + 2
    {
        float fy[6][4];
#pragma unroll
        for (int c = 0; c < 6; ++c) factor(c, ty, iy, fy[c]);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int cz = 3 * (w >> 2) + i;
            float u[6];
#pragma unroll
            for (int cy = 0; cy < 6; ++cy) u[cy] = xl[(tx * 36 + cy + 6 * cz) * 64 + lane];
            float plane;
            yfirst(plane, u[0], fy[0]);
#pragma unroll
            for (int cy = 1; cy < 6; ++cy) yapply(plane, u[cy], fy[cy]);
            yp[((w & 3) * 6 + cz) * 64 + lane] = plane;
        }
        if (!all_far) {
            // near candidates t_d + 1 .. t_d + 3, offsets -1, 0, 1: entries 2, 3, 4 whatever the parity
            float fn[3][4];
#pragma unroll
            for (int k = 0; k < 3; ++k) factor(k + 1, 0, iy, fn[k]);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int cz = 2 * (w >> 2) + i;   // counted from the first near plane
                float u[3];
#pragma unroll
                for (int k = 0; k < 3; ++k) u[k] = xn[(16 * tx + ty + k + 4 * cz) * 64 + lane];
                float plane;
                yfirst(plane, u[0], fn[0]);
#pragma unroll
                for (int k = 1; k < 3; ++k) yapply(plane, u[k], fn[k]);
                yn[((w & 3) * 4 + cz) * 64 + lane] = plane;
            }
        }
    }
    __syncthreads();
    // ---- the child with parity w, if it exists (no barrier below this point): far = all - near, plane by plane
    if (t == 0xFFFFFFFFu) return;
    float acc = 0.f;
    {
        float u[6];
#pragma unroll
        for (int cz = 0; cz < 6; ++cz) u[cz] = yp[((w & 3) * 6 + cz) * 64 + lane];
        if (!all_far) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {   // near planes tz + 1 .. tz + 3
                const float near = yn[((w & 3) * 4 + k) * 64 + lane];
                if (k >= tz && k <= tz + 2) u[k + 1] -= near;
            }
        }
#pragma unroll
        for (int cz = 0; cz < 6; ++cz) {
            float fz[4];
            factor(cz, tz, iz, fz);
            zapply(acc, u[cz], fz);
        }
    }
    V[(int64_t)t * 64 + lane] = acc;
}

// ------------------------------------------------------------------------------------
// The same sums where parents are many.  A workgroup of twelve wavefronts takes four parents (neighbours in box order); a
// wavefront takes one plane cy of their grids and one x parity of the targets, a quarter of its lanes one parent.  A lane
// holds a fibre: the four entries of a row along x, read from memory as one float4, so the x factor is 16 multiply-adds on
// registers with operands that are the same in every lane.  Two v_permlane32_swap and two v_permlane16_swap exchange the
// register index (ix) with the two highest lane bits (iz), and the z factor is of the same kind; only the finished plane
// sums go through LDS, where the y factor is applied.  The nodes are {1, 1/2, -1/2, -1}, so an entry of a factor depends on
// |2 (2 o + s_j - s_i)| = 0 .. 16 only: 17 numbers, in registers.
// What bounds it: vector issue, 4.1 cycles per instruction and SIMD.  A multiply-add on registers alone takes 3.1 cycles a wavefront
// here, one with a DPP operand 4.4.  Leaf depth of 1e7 uniform points (32768 parents): 306 us by the kernel above, 192 by this
// one; of 1e6 normal points (sparse grids: lines without a candidate are passed over): 397 and 270.  The
// kernel above with a plane per wavefront and two barriers instead of three took 306 us as well; this one with both x
// parities in a wavefront (96 registers, five wavefronts per SIMD) 220.
// ------------------------------------------------------------------------------------
// index into the 17 factor values of entry (i, j) of G_o
__device__ constexpr int factor_index(int o, int i, int j) {
    constexpr int h[4] = {2, 1, -1, -2};   // twice the nodes
    const int k = 4 * o + h[j] - h[i];
    return k < 0 ? -k : k;
}
// out[i] += sum_j G_o[i][j] in[j]
template <int O>
__device__ __forceinline__ void fibre_apply(float (&out)[4], const float (&in)[4], const float (&E)[17]) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) out[i] = fmaf(E[factor_index(O, i, j)], in[j], out[i]);
}
// register index <-> the two highest lane bits (a 4 x 4 transpose)
__device__ __forceinline__ void fibre_swap(float (&r)[4]) {
    uint32_t u[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) u[k] = __builtin_bit_cast(uint32_t, r[k]);
    const auto a = __builtin_amdgcn_permlane32_swap(u[0], u[2], false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(u[1], u[3], false, false);
    const auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
    const auto d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
    r[0] = __builtin_bit_cast(float, (uint32_t)c[0]);
    r[1] = __builtin_bit_cast(float, (uint32_t)c[1]);
    r[2] = __builtin_bit_cast(float, (uint32_t)d[0]);
    r[3] = __builtin_bit_cast(float, (uint32_t)d[1]);
}

// Plane sums of the finished planes in LDS: planes 1 and 4 are near for the lower / the upper children only, so they are
// kept twice.  Row of plane cy for children of y parity ty: the four parities tx + 2 tz of the four parents.
constexpr int PL_ROWS = 8;
constexpr int PL_STRIDE = 80;   // floats a 64-vector takes (the four parents fall on different banks)
constexpr int ST_PAR = 4;       // parents of a workgroup
__device__ inline int plane_row(int cy, int ty) {
    return cy == 0 ? 0 : cy == 1 ? 1 + ty : cy == 4 ? 5 + ty : cy == 5 ? 7 : cy + 1;   // 2 -> 3, 3 -> 4
}

// the children of one y parity: sum over the planes, in a lane the four entries of a y fibre
template <int TY>
__device__ __forceinline__ void planes_to_child(float (&acc)[4], const float *pl, int comb, int lane, const float (&E)[17]) {
    const float *src = pl + comb * (ST_PAR * PL_STRIDE) + (lane >> 4) * PL_STRIDE + 4 * (lane & 15);
    constexpr int ROW = 4 * ST_PAR * PL_STRIDE;
    auto plane = [&](int cy, auto o) __attribute__((always_inline)) {
        const float4 f = *reinterpret_cast<const float4 *>(src + plane_row(cy, TY) * ROW);
        const float in[4] = {f.x, f.y, f.z, f.w};
        fibre_apply<decltype(o)::value>(acc, in, E);
    };
    plane(0, std::integral_constant<int, -2 - TY>{});
    plane(1, std::integral_constant<int, -1 - TY>{});
    plane(2, std::integral_constant<int, 0 - TY>{});
    plane(3, std::integral_constant<int, 1 - TY>{});
    plane(4, std::integral_constant<int, 2 - TY>{});
    plane(5, std::integral_constant<int, 3 - TY>{});
}

// the line and plane sums of one plane cy for children of x parity TX (see m2l_stencil_quad_kernel)
template <bool ZROW, int TX>
__device__ __forceinline__ void plane_sums(const uint32_t (*__restrict__ rank)[36], int w, int lane, int all_far, uint32_t zero_row,
                                           const float *__restrict__ W, const float (&E)[17], float *pl) {
    // lane = iy + 4 (parent) + 16 iz
    const uint2 *cand = reinterpret_cast<const uint2 *>(rank[(lane >> 2) & 3]);
    const float *Wl = W + 4 * ((lane & 3) + 4 * (lane >> 4));
    float p0[4], p1[4], q0[4], q1[4];   // plane sums of the z parities, and the same over the near candidates
#pragma unroll
    for (int i = 0; i < 4; ++i) p0[i] = p1[i] = q0[i] = q1[i] = 0.f;
    const bool near_plane = !all_far && w >= 1 && w <= 4;
    // The rows of a line are loaded while the line before it is worked: each into the registers that the row in the same
    // place has just left.
    float u[6][4];
    uint32_t c[6];
    auto rank_line = [&](int cz) __attribute__((always_inline)) {
        const uint2 r0 = cand[3 * cz], r1 = cand[3 * cz + 1], r2 = cand[3 * cz + 2];
        c[0] = r0.x; c[1] = r0.y; c[2] = r1.x; c[3] = r1.y; c[4] = r2.x; c[5] = r2.y;
        // false: no candidate in the line of any of the parents: it adds nothing
        return __ballot((c[0] & c[1] & c[2] & c[3] & c[4] & c[5]) != ~0u) != 0ull;
    };
    auto load_row = [&](int cx) __attribute__((always_inline)) {
        const bool none = c[cx] == ~0u;
        const uint32_t row = ZROW ? min(c[cx], zero_row) : none ? 0u : c[cx];
        const float4 f = *reinterpret_cast<const float4 *>(Wl + (int64_t)row * 64);
        u[cx][0] = ZROW || !none ? f.x : 0.f;
        u[cx][1] = ZROW || !none ? f.y : 0.f;
        u[cx][2] = ZROW || !none ? f.z : 0.f;
        u[cx][3] = ZROW || !none ? f.w : 0.f;
    };
    bool some = rank_line(0);
#pragma unroll
    for (int cx = 0; cx < 6; ++cx) load_row(cx);
    auto line = [&](auto CZ) __attribute__((always_inline)) {
        constexpr int cz = decltype(CZ)::value;
        bool next = false;
        if constexpr (cz < 5) next = rank_line(cz + 1);
        // offset c - 2 - TX from candidate c; the near candidates (c = TX + 1 .. TX + 3) come first, and their sum is
        // kept where the line is near in y and z
        float l[4] = {0.f, 0.f, 0.f, 0.f};
        if (some) {
            fibre_apply<-1>(l, u[TX + 1], E);
            fibre_apply<0>(l, u[TX + 2], E);
            fibre_apply<1>(l, u[TX + 3], E);
        }
        if constexpr (cz < 5) {
            load_row(TX + 1);
            load_row(TX + 2);
            load_row(TX + 3);
        }
        if (some) {
            if constexpr (cz >= 1 && cz <= 4) {
                if (near_plane) {
                    float n[4] = {l[0], l[1], l[2], l[3]};
                    fibre_swap(n);
                    if constexpr (cz <= 3) fibre_apply<cz - 2>(q0, n, E);   // near the children with tz = 0: cz = 1..3
                    if constexpr (cz >= 2) fibre_apply<cz - 3>(q1, n, E);   // tz = 1: cz = 2..4
                }
            }
            fibre_apply<-2 - TX>(l, u[0], E);
            fibre_apply<3 - TX>(l, u[5], E);
            fibre_apply<TX ? -2 : 2>(l, u[TX ? 1 : 4], E);
        }
        if constexpr (cz < 5) {
            load_row(0);
            load_row(5);
            load_row(TX ? 1 : 4);
        }
        if (some) {
            fibre_swap(l);
            fibre_apply<cz - 2>(p0, l, E);
            fibre_apply<cz - 3>(p1, l, E);
        }
        some = next;
    };
    line(std::integral_constant<int, 0>{});
    line(std::integral_constant<int, 1>{});
    line(std::integral_constant<int, 2>{});
    line(std::integral_constant<int, 3>{});
    line(std::integral_constant<int, 4>{});
    line(std::integral_constant<int, 5>{});
    // far = all - near, where the plane is near the child (planes ty + 1 .. ty + 3).  Now lane = iy + 4 (parent) + 16 ix;
    // entry (ix, iy, iz) of a plane sum goes to place iy + 4 ix + 16 iz.
    const int row0 = plane_row(w, 0), row1 = plane_row(w, 1);   // wave-uniform
    const bool near0 = near_plane && w <= 3, near1 = near_plane && w >= 2;
    float *dst = pl + TX * (ST_PAR * PL_STRIDE) + ((lane >> 2) & 3) * PL_STRIDE + (lane & 3) + 4 * (lane >> 4);
    auto store = [&](int row, bool near) __attribute__((always_inline)) {
        float *d = dst + row * (4 * ST_PAR * PL_STRIDE);
#pragma unroll
        for (int iz = 0; iz < 4; ++iz) {
            d[16 * iz] = near ? p0[iz] - q0[iz] : p0[iz];
            d[2 * ST_PAR * PL_STRIDE + 16 * iz] = near ? p1[iz] - q1[iz] : p1[iz];
        }
    };
    store(row0, near0);
    if (row1 != row0) store(row1, near1);
}

template <bool ZROW>
__global__ __launch_bounds__(768) void m2l_stencil_quad_kernel(const uint32_t *__restrict__ cand_tab,
                                                                 const uint32_t *__restrict__ child_tab,
                                                                 int64_t nparents, int64_t per_xcd,
                                                                 const float *__restrict__ G, int all_far,
                                                                 uint32_t zero_row,
                                                                 const float *__restrict__ W, float *__restrict__ V) {
    __shared__ __attribute__((aligned(16))) float pl[PL_ROWS * 4 * ST_PAR * PL_STRIDE];
    __shared__ float es[17];
    __shared__ __attribute__((aligned(8))) uint32_t ranks[6][ST_PAR][36];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // consecutive parents (neighbours in space) on the same XCD, so that its L2 serves the overlap
    const int64_t bi = block_index2();
    const int64_t p0 = ((bi & 7) * per_xcd + (bi >> 3)) * ST_PAR;
    if ((bi >> 3) >= per_xcd || p0 >= nparents) return;
    if (tid < 17) {   // entry k of the factors: offset o and nodes (i, j) with 4 o + 2 s_j - 2 s_i = k
        const int o = tid >= 12 ? 3 : tid >= 8 ? 2 : tid >= 4 ? 1 : 0, d = tid - 4 * o;   // d = 0 .. 4
        const int i = d == 0 ? 0 : d == 1 ? 1 : d == 2 ? 2 : d == 3 ? 2 : 3;              // h = 2, 1, -1, -2
        const int j = d == 0 ? 0 : d == 1 ? 0 : d == 2 ? 1 : d == 3 ? 0 : 0;
        es[tid] = G[(o + 3) * 16 + i * 4 + j];
    }
    // candidate ranks by plane: place cx + 6 cy + 36 cz of a parent goes to [cy][parent][cx + 6 cz]; a parent behind the
    // last one repeats it, and nothing of it is stored
    for (int e = tid; e < ST_PAR * ST_CAND; e += 768) {
        const int q = e / ST_CAND, k = e - q * ST_CAND;
        const int cz = k / 36, cy = (k - 36 * cz) / 6, cx = k - 36 * cz - 6 * cy;
        ranks[cy][q][cx + 6 * cz] = cand_tab[min(p0 + q, nparents - 1) * ST_CAND + k];
    }
    __syncthreads();
    float E[17];
#pragma unroll
    for (int k = 0; k < 17; ++k) E[k] = es[k];
    if (w < 6) plane_sums<ZROW, 0>(ranks[w], w, lane, all_far, zero_row, W, E, pl);
    else plane_sums<ZROW, 1>(ranks[w - 6], w - 6, lane, all_far, zero_row, W, E, pl);
    __syncthreads();
    // ---- the child of parity w of the four parents, where it exists: lane = ix + 4 iz + 16 (parent)
    if (w >= 8) return;
    const int64_t pb = p0 + (lane >> 4);
    const uint32_t t = pb < nparents ? child_tab[pb * 8 + w] : ~0u;
    if (__ballot(t != ~0u) == 0ull) return;
    const int comb = (w & 1) + 2 * (w >> 2);   // tx + 2 tz
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    if ((w >> 1) & 1) planes_to_child<1>(acc, pl, comb, lane, E);
    else planes_to_child<0>(acc, pl, comb, lane, E);
    if (t != ~0u) {
        float *out = V + (int64_t)t * 64 + (lane & 3) + 16 * ((lane >> 2) & 3);
#pragma unroll
        for (int iy = 0; iy < 4; ++iy) out[4 * iy] = acc[iy];
    }
}

constexpr int64_t M2L_QUAD_PARENTS = 1024;

// ------------------------------------------------------------------------------------
// Near pairs between weighted points (near_weighted_error in plan.hip): V_t = sum over the 27 boxes q around t of
// G'_{o_z} x G'_{o_y} x G'_{o_x} W'_q with G'_o[i][j] = exp((l/2)^2 / gamma^2 (s_i s_j + 2 o s_i - 2 o s_j - 2 o^2)), o = -1, 0, 1.
// G'_{-o} is the transpose of G'_o, and G'_o[i][j] = G'_o[3-j][3-i]: 16 different numbers.  The eight children of a parent share
// their line and plane sums on the inner 4 x 4 x 4 places of its candidate grid, by the scheme of
// m2l_stencil_quad_kernel: eight wavefronts, one per plane cy = 1 .. 4 and x parity of the targets.  1e7 points, 32768
// parents: 67 us (exact sums over these pairs: 1560 us), with the second half of the P2M (117 -> 256 us) and the L2P (81 -> 115).
// ------------------------------------------------------------------------------------
__host__ __device__ constexpr int near_factor_index(int o, int i, int j) {
    if (o < 0) return near_factor_index(-o, j, i);
    const bool far_i = i == 0 || i == 3, far_j = j == 0 || j == 3;   // |s| = 1, else 1/2
    if (o == 0) return (far_i && far_j ? 0 : far_i || far_j ? 1 : 2) + ((i < 2) != (j < 2) ? 3 : 0);
    const int a = i + j <= 3 ? i : 3 - j, b = i + j <= 3 ? j : 3 - i;
    return 6 + (a == 0 ? b : a == 1 ? 4 + b : a == 2 ? 7 + b : 9);
}
template <int O>
__device__ __forceinline__ void near_apply(float (&out)[4], const float (&in)[4], const float (&E)[16]) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) out[i] = fmaf(E[near_factor_index(O, i, j)], in[j], out[i]);
}

template <int TX>
__device__ __forceinline__ void near_plane_sums(const uint32_t (*__restrict__ rank)[16], int plane, int lane, uint32_t zero_row,
                                                const float *__restrict__ W, const float (&E)[16], float *pl) {
    // lane = iy + 4 (parent) + 16 iz; places TX .. TX + 2 of the four along x
    const uint32_t *cand = rank[(lane >> 2) & 3];
    const float *Wl = W + 4 * ((lane & 3) + 4 * (lane >> 4));
    float u[4][3][4];   // every row of the plane that is needed, all loads in flight together
#pragma unroll
    for (int cz = 0; cz < 4; ++cz)
#pragma unroll
        for (int cx = 0; cx < 3; ++cx) {
            const float4 f = *reinterpret_cast<const float4 *>(Wl + (int64_t)min(cand[4 * cz + TX + cx], zero_row) * 64);
            u[cz][cx][0] = f.x;
            u[cz][cx][1] = f.y;
            u[cz][cx][2] = f.z;
            u[cz][cx][3] = f.w;
        }
    float p0[4] = {0.f, 0.f, 0.f, 0.f}, p1[4] = {0.f, 0.f, 0.f, 0.f};   // plane sums of the z parities
    auto line = [&](auto CZ) __attribute__((always_inline)) {
        constexpr int cz = decltype(CZ)::value;
        float l[4] = {0.f, 0.f, 0.f, 0.f};
        near_apply<-1>(l, u[cz][0], E);
        near_apply<0>(l, u[cz][1], E);
        near_apply<1>(l, u[cz][2], E);
        fibre_swap(l);
        if constexpr (cz <= 2) near_apply<cz - 1>(p0, l, E);
        if constexpr (cz >= 1) near_apply<cz - 2>(p1, l, E);
    };
    line(std::integral_constant<int, 0>{});
    line(std::integral_constant<int, 1>{});
    line(std::integral_constant<int, 2>{});
    line(std::integral_constant<int, 3>{});
    // now lane = iy + 4 (parent) + 16 ix; entry (ix, iy, iz) goes to place iy + 4 ix + 16 iz
    float *dst = pl + (plane * 4 + TX) * (ST_PAR * PL_STRIDE) + ((lane >> 2) & 3) * PL_STRIDE + (lane & 3) + 4 * (lane >> 4);
#pragma unroll
    for (int iz = 0; iz < 4; ++iz) {
        dst[16 * iz] = p0[iz];
        dst[2 * ST_PAR * PL_STRIDE + 16 * iz] = p1[iz];
    }
}

__global__ __launch_bounds__(512) void near_weighted_kernel(const uint32_t *__restrict__ cand_tab,
                                                            const uint32_t *__restrict__ child_tab, int64_t nparents,
                                                            int64_t per_xcd, const float *__restrict__ tab,
                                                            uint32_t zero_row, const float *__restrict__ W,
                                                            float *__restrict__ V) {
    __shared__ __attribute__((aligned(16))) float pl[4 * 4 * ST_PAR * PL_STRIDE];   // [plane][tx + 2 tz][parent]
    __shared__ float es[16];
    __shared__ uint32_t ranks[4][ST_PAR][16];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t bi = block_index2();
    const int64_t p0 = ((bi & 7) * per_xcd + (bi >> 3)) * ST_PAR;
    if ((bi >> 3) >= per_xcd || p0 >= nparents) return;
    if (tid < 16) es[tid] = tab[tid];
    if (tid >= 256) {   // the inner places; a parent behind the last one repeats it, and nothing of it is stored
        const int e = tid - 256, q = e >> 6, cx = e & 3, cy = (e >> 2) & 3, cz = (e >> 4) & 3;
        ranks[cy][q][cx + 4 * cz] = cand_tab[min(p0 + q, nparents - 1) * ST_CAND + (cx + 1) + 6 * (cy + 1) + 36 * (cz + 1)];
    }
    __syncthreads();
    float E[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) E[k] = es[k];
    if (w < 4) near_plane_sums<0>(ranks[w], w, lane, zero_row, W, E, pl);
    else near_plane_sums<1>(ranks[w - 4], w - 4, lane, zero_row, W, E, pl);
    __syncthreads();
    // ---- the child of parity w of the four parents, where it exists: lane = ix + 4 iz + 16 (parent)
    const int64_t pb = p0 + (lane >> 4);
    const uint32_t t = pb < nparents ? child_tab[pb * 8 + w] : ~0u;
    if (__ballot(t != ~0u) == 0ull) return;
    const int ty = (w >> 1) & 1;
    const float *src = pl + (4 * ty + (w & 1) + 2 * (w >> 2)) * (ST_PAR * PL_STRIDE) + (lane >> 4) * PL_STRIDE + 4 * (lane & 15);
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    auto plane = [&](auto o) __attribute__((always_inline)) {   // planes ty, ty + 1, ty + 2 of the four
        constexpr int O = decltype(o)::value;
        const float4 f = *reinterpret_cast<const float4 *>(src + (O + 1) * 4 * (ST_PAR * PL_STRIDE));
        const float in[4] = {f.x, f.y, f.z, f.w};
        near_apply<O>(acc, in, E);
    };
    plane(std::integral_constant<int, -1>{});
    plane(std::integral_constant<int, 0>{});
    plane(std::integral_constant<int, 1>{});
    if (t != ~0u) {
        float *out = V + (int64_t)t * 64 + (lane & 3) + 16 * ((lane >> 2) & 3);
#pragma unroll
        for (int iy = 0; iy < 4; ++iy) out[4 * iy] = acc[iy];
    }
}

void near_table(const f3m_plan_s &P, float *t) {
    const double s[4] = {1.0, 0.5, -0.5, -1.0};
    const double half = 0.5 * (double)P.E / (double)(1ull << P.near_weighted);
    const double c = half * half / ((double)P.gamma * (double)P.gamma);
    for (int o = 0; o <= 1; ++o)
        for (int i = 0; i < 4; ++i)
            for (int j = 0; j < 4; ++j)
                t[near_factor_index(o, i, j)] = (float)(basis_scale() * std::exp(c * (s[i] * s[j] + 2.0 * o * (s[i] - s[j] - o))));
}

// W: weighted node weights of depth near_weighted with a row of zeros behind them
void run_near_weighted(f3m_plan_s &P, const float *W, float *V, hipStream_t st) {
    f3m_level &lv = P.lev[P.near_weighted], &up = P.lev[P.near_weighted - 1];
    const int64_t per_xcd = cdiv(cdiv(up.nb, ST_PAR), 8);
    near_weighted_kernel<<<grid2(per_xcd * 8), dim3(512), 0, st>>>(lv.st_cand.p, lv.st_child.p, up.nb, per_xcd, P.near_tab.p,
                                                                  (uint32_t)lv.nb, W, V);
    F3M_HIP(hipGetLastError());
}

// candidate and child tables of a depth whose M2L runs on the candidate grid without a small field
// the tables of a depth, preset to "none"; false: the depth does not use them
bool stencil_tables_alloc(f3m_plan_s &P, int level, hipStream_t st) {
    // (while the depths are built their last one for the products, P.near_weighted, is not yet known)
    if (!m2l_stencil_applies(P) || level < 1 || P.rho != 0 || (P.near_depth && level > P.near_depth) ||
        (P.near_weighted && level > P.near_weighted)) return false;
    f3m_level &lv = P.lev[level], &up = P.lev[level - 1];
    if (!lv.far_implicit || lv.far_sz == 0 || lv.p == 0) return false;
    lv.st_cand.alloc((size_t)up.nb * ST_CAND, &P.bytes);
    lv.st_child.alloc((size_t)up.nb * 8, &P.bytes);
    fill_words(lv.st_cand.p, up.nb * ST_CAND, lv.st_child.p, up.nb * 8, ~0u, st);
    return true;
}

void build_stencil_tables(f3m_plan_s &P, int level, hipStream_t st) {
    if (level >= 1 && P.lev[level].st_cand.p) return;   // written by the list kernel already
    if (!stencil_tables_alloc(P, level, st)) return;
    f3m_level &lv = P.lev[level], &up = P.lev[level - 1];
    stencil_table_kernel<<<grid2(up.nb), dim3(256), 0, st>>>(up.near_ptr.p, up.near_col.p, up.cstart.p, up.cell.p,
                                                            lv.cell.p, lv.key.p, up.nb, lv.st_cand.p, lv.st_child.p);
    F3M_HIP(hipGetLastError());
}

// the M2L of the depth runs on the candidate grid with few parents, and may share a launch with others of its kind
bool m2l_stencil_small(const f3m_plan_s &P, int level) {
    return m2l_stencil_applies(P) && level >= 1 && P.lev[level].far_implicit && P.lev[level].st_cand.p && P.lev[level].gtab.p &&
           P.lev[level - 1].nb < M2L_QUAD_PARENTS;
}

static void add_depth(const f3m_plan_s &P, int level, const float *W, float *V, uint32_t zero_row, M2lDepths &A, uint32_t &blocks) {
    const f3m_level &lv = P.lev[level], &up = P.lev[level - 1];
    const int k = A.count++;
    A.cand[k] = lv.st_cand.p;
    A.child[k] = lv.st_child.p;
    A.G[k] = lv.gtab.p;
    A.W[k] = W;
    A.V[k] = V;
    A.first[k] = blocks;
    A.nparents[k] = (uint32_t)up.nb;
    A.zero_row[k] = zero_row;
    A.all_far[k] = lv.smooth || level == P.near_depth ? 1 : 0;
    blocks += (uint32_t)(cdiv(up.nb, 8) * 8);
}

// depths from .. to (m2l_stencil_small each, node weights with a row of zeros behind them): one launch for up to six.  The three
// depths of 2.5e5 points: 19 us one after the other, 10 together.
void run_m2l_small(f3m_plan_s &P, int from, int to, hipStream_t st) {
    for (int l = from; l <= to;) {
        M2lDepths A;
        uint32_t blocks = 0;
        // the deepest first: it has the most workgroups
        const int last = std::min(to, l + M2lDepths::MAX - 1);
        for (int k = last; k >= l; --k) add_depth(P, k, P.lev[k].Wl.p, P.lev[k].Vl.p, (uint32_t)P.lev[k].nb, A, blocks);
        m2l_stencil_shared_kernel<true><<<dim3(blocks), dim3(512), 0, st>>>(A);
        F3M_HIP(hipGetLastError());
        l = last + 1;
    }
}

bool run_m2l_stencil(f3m_plan_s &P, int level, const float *W, float *V, hipStream_t st, bool zero_row) {
    if (!m2l_stencil_applies(P) || level < 1) return false;
    f3m_level &lv = P.lev[level], &up = P.lev[level - 1];
    if (lv.gtab.p == nullptr || lv.gtab_omax != 3) return false;
    const int64_t per_xcd = cdiv(up.nb, 8);
    const int all_far = lv.smooth || level == P.near_depth ? 1 : 0;
    if (lv.st_cand.p) {   // no small field: the variants that share the line and plane sums between the children
        // Four parents to a workgroup from M2L_QUAD_PARENTS on: below, the chip is not full and the longer chain of a workgroup
        // shows (8, 64, 512, 4096 parents: 5.0, 5.1, 6 to 7, 42 us with one parent to a workgroup, 8.2, 9.3, 9.6, 28 with four).
        if (up.nb < M2L_QUAD_PARENTS) {
            M2lDepths A;
            uint32_t blocks = 0;
            add_depth(P, level, W, V, zero_row ? (uint32_t)lv.nb : 0u, A, blocks);
            if (zero_row) m2l_stencil_shared_kernel<true><<<dim3(blocks), dim3(512), 0, st>>>(A);   // W carries a row of zeros at index nb
            else m2l_stencil_shared_kernel<false><<<dim3(blocks), dim3(512), 0, st>>>(A);
        } else {
            const int64_t per = cdiv(cdiv(up.nb, ST_PAR), 8);
            auto launch = [&](auto kern, uint32_t zr) {
                kern<<<grid2(per * 8), dim3(768), 0, st>>>(lv.st_cand.p, lv.st_child.p, up.nb, per, lv.gtab.p, all_far, zr, W, V);
            };
            if (zero_row) launch(m2l_stencil_quad_kernel<true>, (uint32_t)lv.nb);
            else launch(m2l_stencil_quad_kernel<false>, 0u);
        }
        F3M_HIP(hipGetLastError());
        return true;
    }
    m2l_stencil_kernel<<<grid2(per_xcd * 8), dim3(512), 0, st>>>(up.near_ptr.p, up.near_col.p, up.cstart.p, up.cell.p,
                                                                lv.cell.p, lv.key.p, up.nb, per_xcd, lv.gtab.p,
                                                                all_far, lv.start.p, (uint32_t)P.rho, W, V);
    F3M_HIP(hipGetLastError());
    return true;
}

}  // namespace f3m
