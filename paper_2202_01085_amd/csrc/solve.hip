// f3m_cg_solve: kernel ridge regression, alpha = (k(X,X) + lambda I)^{-1} b, by conjugate gradients with
// the F3M product as the solver's matrix-vector product (arXiv 2202.01085, Sec. 5 "Kernel Ridge
// Regression experiment"; the paper plugs F3M into a conjugate-gradient solver the same way).
// Textbook Hestenes-Stiefel recurrences from x_0 = 0.  Vectors are fp32 in HBM; every inner product
// is accumulated in fp64 in a fixed order (grid-stride partial sums, which every block of the next pass adds up for
// itself), and the step lengths stay on the device, so an iteration costs one f3m_kmvm and three fused vector passes
// (48 n bytes).  The host reads the residual of an iteration from its own memory while the next one runs, as long as the tolerance is far
// (cg_loop.h); should an iteration have been launched that was not needed, the device stops by itself (a flag that keeps x from changing)
// and the solve ends after that iteration's product.  With a pass for every sum and a copy and a wait in every iteration, ten
// iterations of 2.5e5 points took 2.14 ms, now 1.81.
// The solve works in the plan's box order: b is permuted once on the way in and x once on the
// way out (inner products do not depend on the order), so the products inside the loop skip
// both permutations of f3m_kmvm.
#include <cmath>
#include <vector>

#include "cg_loop.h"
#include "plan.h"

namespace f3m {

constexpr int CG_NT = 256;
constexpr int CG_BLOCKS = 2048;

// scalars in device memory: r . r of the iteration and of the next one in turn, p . q, whether the solve has ended
enum { S_RS = 0, S_PQ = 2, S_STOP = 3, S_COUNT = 4 };
// words of the host: r . r at the start; per iteration (in turn) r . r, p . q and whether it was the last
enum { W_RS0 = 0, W_SLOT = 8, W_PER = 4, W_SLOTS = 2 };

__device__ inline void block_sum_to(double v, double *dst) {
    __shared__ double sm[CG_NT / 64];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int k = 0; k < CG_NT / 64; ++k) s += sm[k];
        *dst = s;
    }
}

// sum of partial sums, the same bits in every block (and thread)
__device__ inline double sum_parts(const double *__restrict__ part, int nparts) {
    __shared__ double total;
    double s = 0.0;
    for (int k = threadIdx.x; k < nparts; k += CG_NT) s += part[k];
    block_sum_to(s, &total);
    __syncthreads();
    return total;
}

// box order: x = 0, r = p = b[perm]; partial sums of b . b
__global__ __launch_bounds__(CG_NT) void cg_init_kernel(const float *__restrict__ b, const uint32_t *__restrict__ perm,
                                                        float *__restrict__ x, float *__restrict__ r,
                                                        float *__restrict__ p, int64_t n, double *__restrict__ part) {
    double s = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * CG_NT + threadIdx.x; i < n; i += (int64_t)gridDim.x * CG_NT) {
        const float v = b[perm ? perm[i] : (uint32_t)i];
        x[i] = 0.f;
        r[i] = v;
        p[i] = v;
        s += (double)v * (double)v;
    }
    block_sum_to(s, part + blockIdx.x);
}

// q = K p on entry; q <- q + lambda p; partial sums of p . q
__global__ __launch_bounds__(CG_NT) void cg_shift_dot_kernel(const float *__restrict__ p, float *__restrict__ q,
                                                             float lambda, int64_t n, double *__restrict__ part) {
    double s = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * CG_NT + threadIdx.x; i < n; i += (int64_t)gridDim.x * CG_NT) {
        const float pv = p[i];
        const float qv = fmaf(lambda, pv, q[i]);
        q[i] = qv;
        s += (double)pv * (double)qv;
    }
    block_sum_to(s, part + blockIdx.x);
}

// alpha = r . r / p . q; x += alpha p, r -= alpha q; partial sums of r . r
__global__ __launch_bounds__(CG_NT) void cg_update_kernel(float *__restrict__ x, float *__restrict__ r,
                                                          const float *__restrict__ p, const float *__restrict__ q,
                                                          double *__restrict__ scal, int turn,
                                                          const double *__restrict__ part_pq, int64_t n,
                                                          double *__restrict__ part) {
    if (scal[S_STOP] != 0.0) return;   // (the same for all threads)
    const double pq = sum_parts(part_pq, (int)gridDim.x);
    const float alpha = (float)(scal[S_RS + turn] / pq);
    if (blockIdx.x == 0 && threadIdx.x == 0) scal[S_PQ] = pq;
    double s = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * CG_NT + threadIdx.x; i < n; i += (int64_t)gridDim.x * CG_NT) {
        x[i] = fmaf(alpha, p[i], x[i]);
        const float rv = fmaf(-alpha, q[i], r[i]);
        r[i] = rv;
        s += (double)rv * (double)rv;
    }
    block_sum_to(s, part + blockIdx.x);
}

// beta = r . r / (r . r before); p = r + beta p; the iteration's scalars to the host, and the end of the solve
__global__ __launch_bounds__(CG_NT) void cg_direction_kernel(float *__restrict__ p, const float *__restrict__ r,
                                                             double *__restrict__ scal, int turn,
                                                             const double *__restrict__ part_rr, double limit, int64_t n,
                                                             double *__restrict__ slot) {
    const double rs = sum_parts(part_rr, (int)gridDim.x);
    const float beta = (float)(rs / scal[S_RS + turn]);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const double pq = scal[S_PQ];
        const bool stop = scal[S_STOP] != 0.0 || !(pq > 0.0) || !isfinite(rs) || sqrt(rs) <= limit;
        scal[S_RS + 1 - turn] = rs;
        if (stop) scal[S_STOP] = 1.0;
        slot[0] = rs;
        slot[1] = pq;
        slot[2] = stop ? 1.0 : 0.0;
    }
    for (int64_t i = (int64_t)blockIdx.x * CG_NT + threadIdx.x; i < n; i += (int64_t)gridDim.x * CG_NT)
        p[i] = fmaf(beta, p[i], r[i]);
}

// the solution back in the caller's order
__global__ __launch_bounds__(CG_NT) void cg_unpermute_kernel(const float *__restrict__ xs,
                                                             const uint32_t *__restrict__ perm, int64_t n,
                                                             float *__restrict__ x) {
    for (int64_t i = (int64_t)blockIdx.x * CG_NT + threadIdx.x; i < n; i += (int64_t)gridDim.x * CG_NT)
        x[perm[i]] = xs[i];
}

// r . r of the start, to the device and to the host
__global__ __launch_bounds__(CG_NT) void cg_start_kernel(const double *__restrict__ part, int nparts, double *__restrict__ scal,
                                                         double *__restrict__ rs0) {
    const double s = sum_parts(part, nparts);
    if (threadIdx.x == 0) {
        scal[S_RS] = s;
        *rs0 = s;
    }
}

void run_cg(f3m_plan_s &P, float lambda, const float *b, float *x, int max_iter, float tol, int *iters_host,
            float *history_host, hipStream_t st) {
    const int64_t n = P.n;
    ReleaseScope scope(st);      // one wait for the work vectors, at the end
    DevBuf<float> xs, r, p, q;   // box order
    DevBuf<double> part, part2, scal;
    xs.alloc((size_t)n);
    r.alloc((size_t)n);
    p.alloc((size_t)n + PAD_POINTS);
    q.alloc((size_t)n);
    const int blocks = (int)std::min<int64_t>(CG_BLOCKS, cdiv(n, CG_NT));
    part.alloc((size_t)blocks);
    part2.alloc((size_t)blocks);
    scal.alloc(S_COUNT);
    fill_words((uint32_t *)(p.p + n), PAD_POINTS, (uint32_t *)scal.p, 2 * S_COUNT, 0u, st);
    double *words = (double *)scope_words();
    // grouped points are not in the order of perm
    const bool grouped = P.route && P.route->grouped;
    if (grouped) route_gather(*P.route, b, q.p, nullptr, nullptr, st);
    cg_init_kernel<<<dim3(blocks), dim3(CG_NT), 0, st>>>(grouped ? q.p : b, grouped ? nullptr : P.perm.p, xs.p, r.p, p.p, n, part.p);
    cg_start_kernel<<<dim3(1), dim3(CG_NT), 0, st>>>(part.p, blocks, scal.p, words + W_RS0);
    F3M_HIP(hipGetLastError());
    F3M_HIP(hipStreamSynchronize(st));
    const double nb = std::sqrt(words[W_RS0]);
    int it = 0;   // iterations whose result the host has seen
    if (history_host) history_host[0] = nb > 0.0 ? 1.f : 0.f;
    if (!std::isfinite(nb)) fail(F3M_ERR_NONFINITE, "the right-hand side holds a NaN or an infinity");
    struct Events {
        hipEvent_t e[W_SLOTS] = {nullptr};
        int device;
        explicit Events(int d) : device(d) {}
        ~Events() { for (hipEvent_t v : e) event_put(v, device); }
    } ev(P.device);
    for (hipEvent_t &e : ev.e) e = event_get();
    auto slot = [&](int k) { return words + W_SLOT + W_PER * (k % W_SLOTS); };
    // the result of iteration k: true if it was the last
    auto look = [&](int k, double *residual) {
        F3M_HIP(hipEventSynchronize(ev.e[k % W_SLOTS]));
        const double rs = slot(k)[0], pq = slot(k)[1];
        const bool last = slot(k)[2] != 0.0;
        it = k + 1;
        if (!(pq > 0.0) || !std::isfinite(rs)) {
            if (iters_host) *iters_host = it;
            fail(F3M_ERR_BREAKDOWN,
                 "conjugate gradients broke down: p.(K + lambda I)p is not positive (the approximate operator is not "
                 "positive definite along a search direction; raise lambda or the accuracy of the plan)");
        }
        *residual = std::sqrt(rs);
        if (history_host) history_host[it] = (float)(std::sqrt(rs) / nb);
        return last;
    };
    const double limit = (double)tol * nb;
    auto launch = [&](int k) {
        run_kmvm(P, p.p, q.p, st, true);
        cg_shift_dot_kernel<<<dim3(blocks), dim3(CG_NT), 0, st>>>(p.p, q.p, lambda, n, part.p);
        cg_update_kernel<<<dim3(blocks), dim3(CG_NT), 0, st>>>(xs.p, r.p, p.p, q.p, scal.p, k & 1, part.p, n, part2.p);
        cg_direction_kernel<<<dim3(blocks), dim3(CG_NT), 0, st>>>(p.p, r.p, scal.p, k & 1, part2.p, limit, n, slot(k));
        F3M_HIP(hipGetLastError());
        F3M_HIP(hipEventRecord(ev.e[k % W_SLOTS], st));
    };
    cg_iterate(nb > 0.0 ? max_iter : 0, nb, limit, launch, look);
    if (iters_host) *iters_host = it;
    if (grouped) route_scatter(*P.route, xs.p, nullptr, x, nullptr, nullptr, st);
    else cg_unpermute_kernel<<<dim3(blocks), dim3(CG_NT), 0, st>>>(xs.p, P.perm.p, n, x);
    F3M_HIP(hipGetLastError());
    F3M_HIP(hipStreamSynchronize(st));
}

}  // namespace f3m
