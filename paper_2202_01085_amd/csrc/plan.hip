// f3m_plan: enclosing cube, keys, radix sort, box tables, interaction lists.
// (arXiv 2202.01085: Sec. 3 "Enclosing and partitioning the data", Sec. 4.1, Sec. 4.2,
//  Appendix E Algorithm 1 "Divide", "Calculate interactions left", "Partition".)
#include <algorithm>
#include <cmath>
#include <cstring>

#include "plan.h"

f3m_plan_s::~f3m_plan_s() {
    for (auto &e : ev) f3m::event_put(e, device);
    for (auto &e : plan_events) f3m::event_put(e, device);
    for (auto &e : marks) f3m::event_put(e, device);
    for (hipEvent_t e : {ev_fork, ev_join, ev_p2p0, ev_p2p1}) f3m::event_put(e, device);
    if (side) (void)hipStreamDestroy(side);
}

namespace f3m {

int quant_depth(int D) {
    int q = 32 / D;
    return q > 20 ? 20 : q;
}

// ------------------------------------------------------------------------------------
// enclosing cube: per-dimension min and max (exact in fp32), non-finite detection
// ------------------------------------------------------------------------------------
constexpr int BBOX_BLOCKS = 1024;
constexpr int BBOX_NT = 256;

template <int D>
__global__ __launch_bounds__(BBOX_NT) void bbox_kernel(const float *__restrict__ X, int64_t n,
                                                       float *__restrict__ part) {
    float mn[D], mx[D];
#pragma unroll
    for (int d = 0; d < D; ++d) { mn[d] = INFINITY; mx[d] = -INFINITY; }
    int bad = 0;
    for (int64_t i = (int64_t)blockIdx.x * BBOX_NT + threadIdx.x; i < n; i += (int64_t)gridDim.x * BBOX_NT) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            float v = X[i * D + d];
            bad |= !(fabsf(v) <= 3.402823466e38f);
            mn[d] = fminf(mn[d], v);
            mx[d] = fmaxf(mx[d], v);
        }
    }
    __shared__ float smn[BBOX_NT / 64][D], smx[BBOX_NT / 64][D];
    __shared__ int sbad;
    if (threadIdx.x == 0) sbad = 0;
    __syncthreads();
    int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int d = 0; d < D; ++d) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            mn[d] = fminf(mn[d], __shfl_xor(mn[d], off, 64));
            mx[d] = fmaxf(mx[d], __shfl_xor(mx[d], off, 64));
        }
        if (lane == 0) { smn[w][d] = mn[d]; smx[w][d] = mx[d]; }
    }
    if (bad) atomicOr(&sbad, 1);
    __syncthreads();
    if (threadIdx.x < D) {
        int d = threadIdx.x;
        float a = smn[0][d], b = smx[0][d];
        for (int k = 1; k < BBOX_NT / 64; ++k) { a = fminf(a, smn[k][d]); b = fmaxf(b, smx[k][d]); }
        part[(int64_t)blockIdx.x * (2 * D + 1) + d] = a;
        part[(int64_t)blockIdx.x * (2 * D + 1) + D + d] = b;
    }
    if (threadIdx.x == 0) part[(int64_t)blockIdx.x * (2 * D + 1) + 2 * D] = sbad ? 1.f : 0.f;
}
// the same over the blocks, to words of the host: minima, maxima, whether a value is not finite (one wavefront per word)
__global__ __launch_bounds__(1024) void bbox_final_kernel(const float *__restrict__ part, int nblocks, int D,
                                                          uint64_t *__restrict__ words) {
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, m = 2 * D + 1;
    if (w >= m) return;
    float v = w < D ? INFINITY : -INFINITY;
    for (int k = lane; k < nblocks; k += 64) {
        const float p = part[(int64_t)k * m + w];
        v = w < D ? fminf(v, p) : fmaxf(v, p);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const float o = __shfl_xor(v, off, 64);
        v = w < D ? fminf(v, o) : fmaxf(v, o);
    }
    if (lane == 0) words[w] = __float_as_uint(v);
}

// ------------------------------------------------------------------------------------
// cells and keys (Sec. 4.2 box-index formula).  The cell of a point is fixed once, at the
// quantisation depth Lq, by two separately rounded fp32 operations and a truncation:
//   c_d = min( trunc( (x_d - alpha_d) * s ), 2^Lq - 1 ),   s = fl32(2^Lq / E)
// The cell at depth l is c_d >> (Lq - l).  Key: bit k of c_d -> key bit k*D + d.
// ------------------------------------------------------------------------------------
struct AlphaArg { float a[F3M_MAX_DIM]; };

// bit k of c -> bit k * D (c < 2^(32 / D))
template <int D>
__device__ inline uint32_t spread_bits(uint32_t c) {
    if constexpr (D == 1) {
        return c;
    } else if constexpr (D == 2) {
        c &= 0xFFFFu;
        c = (c | (c << 8)) & 0x00FF00FFu;
        c = (c | (c << 4)) & 0x0F0F0F0Fu;
        c = (c | (c << 2)) & 0x33333333u;
        return (c | (c << 1)) & 0x55555555u;
    } else if constexpr (D == 3) {
        c &= 0x3FFu;
        c = (c | (c << 16)) & 0x030000FFu;
        c = (c | (c << 8)) & 0x0300F00Fu;
        c = (c | (c << 4)) & 0x030C30C3u;
        return (c | (c << 2)) & 0x09249249u;
    } else {
        uint32_t r = 0;
#pragma unroll
        for (int k = 0; k < 32 / D; ++k) r |= ((c >> k) & 1u) << (k * D);
        return r;
    }
}

template <int D>
__global__ __launch_bounds__(256) void keys_kernel(const float *__restrict__ X, int64_t n, AlphaArg alpha, float s,
                                                   int Lq, uint32_t *__restrict__ keys) {
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    uint32_t cmax = (uint32_t)((1ull << Lq) - 1);
    uint32_t key = 0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        float diff = __fsub_rn(X[i * D + d], alpha.a[d]);
        float u = __fmul_rn(diff, s);
        uint32_t c = (uint32_t)u;
        c = c > cmax ? cmax : c;
        key |= spread_bits<D>(c) << d;   // c < 2^Lq and Lq * D <= 32
    }
    keys[i] = key;
}

// ------------------------------------------------------------------------------------
// stable LSD radix sort of (key, index) pairs, 8 bits per pass:
//   histogram per tile -> exclusive scan in digit-major order -> stable scatter.
// This replaces the count / cumulative-sum / atomic-increment grouping of Sec. 4.1: the
// result is deterministic (ascending key, then ascending original index).
// ------------------------------------------------------------------------------------
constexpr int RS_NT = 256;
// Keys of a thread.  A tile of 32 x 256 keys writes runs of 32 keys to a digit, which large n need; with few keys its tiles leave compute
// units idle, and a workgroup takes 21 us alone, a chain of 32 rounds.  Below 2^20 keys tiles of 8 x 256: a scatter pass
// of 1e5 keys 21 -> 7.5 us, of 1e6 23.5 -> 11.6.  Plans of 1.5e6 and 2e6 points take the same time with either, of 6e6 929 us
// with the large tiles and 971 with the small ones.
constexpr int RS_IPT_MANY = 32, RS_IPT_FEW = 8;
constexpr int64_t RS_FEW = 1 << 20;
constexpr int RS_SLACK = RS_NT * RS_IPT_MANY;   // keys that may be read behind the last one

template <int RS_IPT>
__global__ __launch_bounds__(RS_NT) void rs_hist_kernel(const uint32_t *__restrict__ keys, int64_t n, int shift,
                                                        uint32_t *__restrict__ hist, int64_t nblk) {
    __shared__ uint32_t h[256];
    // tiles are dealt to the dies like those of the scatter kernel (the counts of neighbouring tiles share lines)
    const int64_t per_die = (nblk + 7) / 8;
    const int64_t tile = (int64_t)(blockIdx.x & 7u) * per_die + (blockIdx.x >> 3);
    if (tile >= nblk) return;
    h[threadIdx.x] = 0;
    __syncthreads();
    // all loads first, four keys each, without a bounds test (the key buffers carry a tile of slack behind the
    // last key); what lies behind the end is left out of the counts
    constexpr int RS_TILE = RS_NT * RS_IPT;
    const int64_t base = tile * RS_TILE;
    const int64_t left = n - base;
    const int cntile = (int)(left < RS_TILE ? left : RS_TILE);
    const uint4 *kp = reinterpret_cast<const uint4 *>(keys + base);
    uint4 v[RS_IPT / 4];
#pragma unroll
    for (int k = 0; k < RS_IPT / 4; ++k) v[k] = kp[k * RS_NT + threadIdx.x];
#pragma unroll
    for (int k = 0; k < RS_IPT / 4; ++k) {
        const int i0 = (k * RS_NT + (int)threadIdx.x) * 4;
        const uint32_t key4[4] = {v[k].x, v[k].y, v[k].z, v[k].w};
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (i0 + c < cntile) atomicAdd(&h[(key4[c] >> shift) & 255u], 1u);
    }
    __syncthreads();
    hist[(int64_t)threadIdx.x * nblk + tile] = h[threadIdx.x];
}

struct U32In {
    const uint32_t *p;
    __device__ uint64_t operator()(int64_t i) const { return p[i]; }
};
struct U32Out {
    uint32_t *p;
    __device__ void operator()(int64_t i, uint64_t ex, uint64_t) const { p[i] = (uint32_t)ex; }
};

// Stable scatter of one tile of RS_TILE keys.  Tile order = (wave, round, lane): every wave
// ranks its own RS_IPT rounds of 64 keys with a private LDS counter array, with no block barrier
// inside the loop; then the tile is put in digit order in LDS and written out so that
// consecutive threads write consecutive addresses of a digit run.  The buffers must be readable
// for a whole tile behind the last key.
template <bool FIRST, int RS_IPT>   // FIRST: the values are the positions themselves (vals_in is not read)
__global__ __launch_bounds__(RS_NT, 4) void rs_scatter_kernel(const uint32_t *__restrict__ keys_in,
                                                           const uint32_t *__restrict__ vals_in,
                                                           uint32_t *__restrict__ keys_out,
                                                           uint32_t *__restrict__ vals_out, int64_t n, int shift,
                                                           const uint32_t *__restrict__ offs, int64_t nblk) {
    constexpr int NW = RS_NT / 64, RS_TILE = RS_NT * RS_IPT;
    __shared__ uint32_t wcnt[NW][256];      // per wave: keys of each digit seen so far
    __shared__ uint32_t dstart[256];        // first tile-local position of each digit
    __shared__ uint32_t gbase[256];         // global position of the tile's first key of each digit
    __shared__ __attribute__((aligned(8))) uint32_t sbuf[RS_TILE];   // the tile in digit order: first its keys, then its values
    // per wave, while the keys are ranked (sbuf is not in use yet): the lanes that hold each digit in the current round
    uint64_t (*wmask)[256] = reinterpret_cast<uint64_t (*)[256]>(sbuf);
    static_assert(sizeof(uint64_t) * NW * 256 <= sizeof(uint32_t) * RS_TILE, "the lane masks must fit the tile buffer");
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    // Workgroups go to the 8 dies in turn; every die takes a contiguous range of tiles, so that the runs
    // which neighbouring tiles append to the same digit meet in one L2 and leave it as whole lines.
    const int64_t per_die = (nblk + 7) / 8;
    const int64_t tile = (int64_t)(blockIdx.x & 7u) * per_die + (blockIdx.x >> 3);
    if (tile >= nblk) return;
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        wcnt[k][tid] = 0;
        wmask[k][tid] = 0ull;
    }
    gbase[tid] = offs[(int64_t)tid * nblk + tile];
    __syncthreads();
    const int64_t base = tile * RS_TILE + (int64_t)w * (RS_IPT * 64);
    // Registers are what bounds the number of resident workgroups: ranks and positions are kept as 16-bit
    // halves (a tile has at most 8192 places; 0xFFFF = out of range), the digits of the written keys as bytes.
    uint32_t key[RS_IPT], val[RS_IPT], rk[RS_IPT / 2];
    const int64_t left = n - tile * RS_TILE;
    const int cntile = (int)(left < RS_TILE ? left : RS_TILE);   // keys of this tile (the last one may be short)
    const int local = w * (RS_IPT * 64) + lane;                  // tile-local index of this thread's first key
    // loads without branches: the buffers carry a tile of slack, and what is read behind the end is left out of
    // the ranking below
    const uint32_t *kp = keys_in + base + lane, *vp = vals_in + base + lane;
#pragma unroll
    for (int r = 0; r < RS_IPT; ++r) key[r] = kp[r * 64];
    // Rank of a key among the earlier keys of its wave with the same digit.  The lanes of a round that hold the
    // same digit find each other through LDS: every lane ORs its own bit into the 64-bit word of its digit
    // (an atomic OR: the result does not depend on the order), reads the word back, and counts the bits below
    // its own.  The first lane of each group then adds the group to the running count of the digit and clears
    // the word.  (LDS operations of a wave complete in order, and the wave runs in lockstep.)
    const uint64_t mybit = 1ull << lane;
#pragma unroll
    for (int r = 0; r < RS_IPT; ++r) {
        const bool valid = local + r * 64 < cntile;
        const uint32_t digit = (key[r] >> shift) & 255u;
        uint32_t rank = 0xFFFFu;
        if (valid) {
            atomicOr(reinterpret_cast<unsigned long long *>(&wmask[w][digit]), (unsigned long long)mybit);
            __builtin_amdgcn_wave_barrier();
            const uint64_t peers = wmask[w][digit];
            const uint32_t cnt = wcnt[w][digit];
            const uint32_t before = __builtin_amdgcn_mbcnt_hi((uint32_t)(peers >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0u));
            rank = cnt + before;   // within (wave, digit): below 2048
            __builtin_amdgcn_wave_barrier();
            if (before == 0) {
                wcnt[w][digit] = cnt + (uint32_t)__popcll(peers);
                wmask[w][digit] = 0ull;
            }
        }
        rk[r >> 1] = (r & 1) ? (rk[r >> 1] | (rank << 16)) : rank;
        __builtin_amdgcn_wave_barrier();   // keep the rounds' LDS accesses in program order
    }
    __syncthreads();
    // digit totals of the tile, exclusive scan over the 256 digits (one digit per thread)
    {
        uint32_t tot = 0;
#pragma unroll
        for (int k = 0; k < NW; ++k) tot += wcnt[k][tid];
        uint64_t blocktot;
        const uint32_t ex = (uint32_t)block_excl_scan_u64(tot, &blocktot);
        dstart[tid] = ex;
    }
    __syncthreads();
    // keys and values pass through the same LDS (32 KB) one after the other
#pragma unroll
    for (int r = 0; r < RS_IPT; ++r) {
        const uint32_t rank = (rk[r >> 1] >> (16 * (r & 1))) & 0xFFFFu;
        if (rank != 0xFFFFu) {
            const uint32_t digit = (key[r] >> shift) & 255u;
            uint32_t pos = dstart[digit] + rank;
            for (int k = 0; k < w; ++k) pos += wcnt[k][digit];
            rk[r >> 1] = (r & 1) ? ((rk[r >> 1] & 0xFFFFu) | (pos << 16)) : ((rk[r >> 1] & 0xFFFF0000u) | pos);
            sbuf[pos] = key[r];
        }
    }
    // the values are loaded only now, into the registers of the keys (keys, values and ranks together would not
    // fit the register budget of four workgroups per compute unit); they arrive while the keys are written out
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < RS_IPT; ++r) {
        if constexpr (FIRST) val[r] = (uint32_t)(base + r * 64 + lane);
        else val[r] = vp[r * 64];
    }
    __syncthreads();
    uint32_t dig[RS_IPT / 4];   // digit of the tile's entry r * RS_NT + tid
#pragma unroll
    for (int r = 0; r < RS_IPT; ++r) {
        const int pos = r * RS_NT + tid;
        uint32_t digit = 0;
        if (pos < cntile) {
            const uint32_t k = sbuf[pos];
            digit = (k >> shift) & 255u;
            keys_out[gbase[digit] + ((uint32_t)pos - dstart[digit])] = k;
        }
        dig[r >> 2] = (r & 3) ? (dig[r >> 2] | (digit << (8 * (r & 3)))) : digit;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RS_IPT; ++r) {
        const uint32_t pos = (rk[r >> 1] >> (16 * (r & 1))) & 0xFFFFu;
        if (pos != 0xFFFFu) sbuf[pos] = val[r];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RS_IPT; ++r) {
        const int pos = r * RS_NT + tid;
        if (pos < cntile) {
            const uint32_t digit = (dig[r >> 2] >> (8 * (r & 3))) & 255u;
            vals_out[gbase[digit] + ((uint32_t)pos - dstart[digit])] = sbuf[pos];
        }
    }
}

// sorts (keys_a, index) by the low `bits` bits; returns true if the result is in the b buffers.  keys_c (or null): takes the
// place of keys_a from the second pass on, whose input then stays as it was (bits > 8).
static bool radix_sort(uint32_t *keys_a, uint32_t *vals_a, uint32_t *keys_b, uint32_t *vals_b, uint32_t *keys_c, int64_t n,
                       int bits, hipStream_t st) {
    const bool few = n < RS_FEW;
    const int64_t nblk = cdiv(n, RS_NT * (few ? RS_IPT_FEW : RS_IPT_MANY));
    const dim3 grid((unsigned)((nblk + 7) / 8 * 8));   // a whole number of rounds over the dies
    DevBuf<uint32_t> hist;
    hist.alloc((size_t)nblk * 256);
    bool in_b = false, first = true;
    for (int shift = 0; shift < bits; shift += 8) {
        const uint32_t *kin = in_b ? keys_b : first || !keys_c ? keys_a : keys_c;
        const uint32_t *vin = first ? nullptr : (in_b ? vals_b : vals_a);
        uint32_t *kout = in_b ? (keys_c ? keys_c : keys_a) : keys_b;
        uint32_t *vout = in_b ? vals_a : vals_b;
        if (few) rs_hist_kernel<RS_IPT_FEW><<<grid, dim3(RS_NT), 0, st>>>(kin, n, shift, hist.p, nblk);
        else rs_hist_kernel<RS_IPT_MANY><<<grid, dim3(RS_NT), 0, st>>>(kin, n, shift, hist.p, nblk);
        F3M_HIP(hipGetLastError());
        exclusive_scan(U32In{hist.p}, nblk * 256, U32Out{hist.p}, nullptr, st);
        auto scatter = [&](auto kern) { kern<<<grid, dim3(RS_NT), 0, st>>>(kin, vin, kout, vout, n, shift, hist.p, nblk); };
        if (few && first) scatter(rs_scatter_kernel<true, RS_IPT_FEW>);
        else if (few) scatter(rs_scatter_kernel<false, RS_IPT_FEW>);
        else if (first) scatter(rs_scatter_kernel<true, RS_IPT_MANY>);
        else scatter(rs_scatter_kernel<false, RS_IPT_MANY>);
        F3M_HIP(hipGetLastError());
        in_b = !in_b;
        first = false;
    }
    return in_b;
}

__global__ void iota_kernel(uint32_t *p, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = (uint32_t)i;
}

template <int D>
__global__ __launch_bounds__(256) void gather_rows_kernel(const float *__restrict__ X, const uint32_t *__restrict__ perm,
                                                          int64_t n, float *__restrict__ Xs) {
    int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= n) return;
    int64_t j = perm[k];
#pragma unroll
    for (int d = 0; d < D; ++d) Xs[k * D + d] = X[j * D + d];
}

// ------------------------------------------------------------------------------------
// box tables per depth (Algorithm 1 "Divide"; empty boxes never appear, Sec. 4.2)
// ------------------------------------------------------------------------------------
struct HeadIn {
    const uint32_t *keys;
    int shift;
    __device__ uint64_t operator()(int64_t i) const {
        if (i == 0) return 1;
        return ((uint64_t)keys[i] >> shift) != ((uint64_t)keys[i - 1] >> shift);
    }
    // a run of 8 keys (base a multiple of 8, so 32-byte aligned: the arrays come from the pool) in two loads
    __device__ void load_run(int64_t base, uint64_t (&v)[SCAN_IPT]) const {
        static_assert(SCAN_IPT == 8, "two loads of four keys");
        const uint4 *p = reinterpret_cast<const uint4 *>(keys + base);
        const uint4 a = p[0], b = p[1];
        const uint32_t k[9] = {base > 0 ? keys[base - 1] : 0u, a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = ((uint64_t)k[j + 1] >> shift) != ((uint64_t)k[j] >> shift);
        if (base == 0) v[0] = 1;
    }
};
// (the last element also writes the entry behind the last box, in the same way in the outputs below)
struct HeadOut {
    const uint32_t *keys;
    int shift;
    uint32_t *start, *bkey;
    int64_t n;
    __device__ void operator()(int64_t i, uint64_t ex, uint64_t v) const {
        if (v) {
            start[ex] = (uint32_t)i;
            bkey[ex] = (uint32_t)((uint64_t)keys[i] >> shift);
        }
        if (i == n - 1) start[ex + v] = (uint32_t)n;
    }
};
// nup: boxes of the depth above (there is one head per box; a count that disagrees is reported by the host)
struct ParentOut {
    uint32_t *parent, *cstart_up;
    int64_t nb, nup;
    __device__ void operator()(int64_t a, uint64_t ex, uint64_t v) const {
        parent[a] = (uint32_t)(ex + v - 1);
        if (v && (int64_t)ex < nup) cstart_up[ex] = (uint32_t)a;
        if (a == nb - 1) cstart_up[nup] = (uint32_t)nb;
    }
};

// Divide from the depth above (used while boxes are much fewer than points): the children of a
// box are sub-intervals of its sorted interval, found by binary search on the key prefix.
// lb[P * 2^D + c] = first point of parent P whose depth-l key is >= (key_P << D | c).
template <int D>
__global__ __launch_bounds__(256) void child_bounds_kernel(const uint32_t *__restrict__ keys, int shift,
                                                           const uint32_t *__restrict__ up_start, int64_t nslots,
                                                           const uint32_t *__restrict__ up_key, uint32_t *__restrict__ lb,
                                                           uint32_t n) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= nslots) return;
    const int64_t P = idx >> D;
    const uint32_t c = (uint32_t)(idx & ((1 << D) - 1));
    uint32_t lo = up_start[P], hi = up_start[P + 1];
    if (c != 0) {
        const uint64_t want = ((uint64_t)up_key[P] << D) | c;
        while (lo < hi) {
            const uint32_t mid = lo + ((hi - lo) >> 1);
            if (((uint64_t)keys[mid] >> shift) < want) lo = mid + 1;
            else hi = mid;
        }
    }
    lb[idx] = lo;
    if (idx == nslots - 1) lb[nslots] = n;
}
struct ChildIn {
    const uint32_t *lb;   // [nslots + 1]
    __device__ uint64_t operator()(int64_t i) const { return lb[i + 1] != lb[i]; }
};
template <int D>
struct ChildOut {
    const uint32_t *lb, *up_key;
    uint32_t *start, *bkey, *parent, *cstart_up;
    int64_t nslots;
    __device__ void operator()(int64_t i, uint64_t ex, uint64_t v) const {
        const int64_t P = i >> D;
        const uint32_t c = (uint32_t)(i & ((1 << D) - 1));
        if (c == 0) cstart_up[P] = (uint32_t)ex;
        if (v) {
            start[ex] = lb[i];
            bkey[ex] = (uint32_t)(((uint64_t)up_key[P] << D) | c);
            parent[ex] = (uint32_t)P;
        }
        if (i == nslots - 1) {
            start[ex + v] = lb[nslots];
            cstart_up[P + 1] = (uint32_t)(ex + v);
        }
    }
};

// depth 0: one box, near itself
__global__ void root_kernel(uint32_t n, int D, uint32_t *key, uint32_t *start, uint32_t *parent, int32_t *cell) {
    key[0] = 0;
    start[0] = 0;
    start[1] = n;
    parent[0] = 0;
    for (int d = 0; d < D; ++d) cell[d] = 0;
}
__global__ void root_lists_kernel(uint64_t *near_ptr, uint64_t *far_ptr, uint32_t *near_col) {
    near_ptr[0] = 0;
    near_ptr[1] = 1;
    far_ptr[0] = 0;
    far_ptr[1] = 0;
    near_col[0] = 0;
}

// largest box: a partial maximum per block, then one block over the partial maxima (which then are the "sizes")
template <bool SIZES>
__global__ __launch_bounds__(256) void max_count_kernel(const uint32_t *__restrict__ start, int64_t nb,
                                                        uint32_t *__restrict__ part, uint64_t *__restrict__ result) {
    uint32_t m = 0;
    for (int64_t a = (int64_t)blockIdx.x * 256 + threadIdx.x; a < nb; a += (int64_t)gridDim.x * 256)
        m = max(m, SIZES ? start[a] : start[a + 1] - start[a]);
    __shared__ uint32_t sm[256];
    sm[threadIdx.x] = m;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) sm[threadIdx.x] = max(sm[threadIdx.x], sm[threadIdx.x + s]);
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        if (gridDim.x == 1) *result = sm[0];
        else part[blockIdx.x] = sm[0];
    }
}

template <int D>
__global__ __launch_bounds__(256) void cells_kernel(const uint32_t *__restrict__ bkey, int64_t nb, int level,
                                                    int32_t *__restrict__ cell) {
    int64_t a = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (a >= nb) return;
    uint32_t key = bkey[a];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        int32_t c = 0;
        for (int k = 0; k < level; ++k) c |= (int32_t)((key >> (k * D + d)) & 1u) << k;
        cell[a * D + d] = c;
    }
}

// ------------------------------------------------------------------------------------
// interaction lists (Algorithm 1 "Calculate interactions left" and "Partition"):
// the candidates of a box are the children of the boxes near its parent; a candidate is
// far iff the squared integer cell offset is >= T = ceil(theta^2)  (Sec. 3, IsFarField
// := |delta centre| >= 2 l, divided by l).  Rows come out sorted by column rank because the
// parent's row is sorted and children have consecutive ranks (Sec. 4.1 "Ensuring
// interactions are sorted").  pass 0 counts, pass 1 fills.  A null near_col or far_col skips
// that side: depths whose M2L works on the candidate grid keep only the far counts, and their
// far rows are produced on request.
// ------------------------------------------------------------------------------------
struct ListArg {
    int T;                 // a pair is far iff the squared integer cell offset is >= T
    int mode;              // 0: far rule, 1: all near, 2: all far (smooth depth, Sec. 4.3)
    uint32_t rho;          // small field (Sec. 4.2): |p| + |q| <= rho goes on the direct list; 0 = off
    const uint32_t *start; // point intervals of the target boxes of this depth (sizes for the small-field rule)
    // source side of the depth: the same tables as the targets' for one point set, those of Y for two
    const int32_t *cell_src;
    const uint32_t *start_src;
    // two sets: the grids are shifted by u box edges, and a pair is far iff
    // sum_d ((c'_d - c_d) + u_d)^2 >= theta2, every fp64 operation rounded on its own, d ascending
    int shifted;
    double u[F3M_MAX_DIM];
    double theta2;
    uint32_t *cnt_near, *cnt_far, *cnt_small;         // pass 0: row lengths
    const uint64_t *near_ptr, *far_ptr, *small_ptr;   // pass 1: row offsets
    uint32_t *near_col, *far_col, *small_col;         // pass 1: columns (null: that list is not written)
    // pass 1 of the by-parent kernel, D = 3, far ratio 2: the tables of the candidate-grid M2L (or null):
    // [parent][216] rank of the candidate at each position of the 6 x 6 x 6 grid around the parent,
    // [parent][8] the child of each parity (both preset to ~0)
    uint32_t *st_cand, *st_child;
};

// up_cstart: children intervals of the SOURCE-side boxes one depth up
template <int D>
__global__ __launch_bounds__(128) void lists_kernel(int pass, int64_t nb, const uint32_t *__restrict__ parent,
                                                    const int32_t *__restrict__ cell,
                                                    const uint64_t *__restrict__ up_near_ptr,
                                                    const uint32_t *__restrict__ up_near_col,
                                                    const uint32_t *__restrict__ up_cstart, ListArg A) {
    int64_t a = (int64_t)blockIdx.x * 128 + threadIdx.x;
    if (a >= nb) return;
    int32_t ca[D];
#pragma unroll
    for (int d = 0; d < D; ++d) ca[d] = cell[a * D + d];
    uint32_t P = parent[a];
    uint64_t nn = 0, nf = 0, ns = 0;
    const uint64_t nbase = pass && A.near_ptr ? A.near_ptr[a] : 0, fbase = pass && A.far_ptr ? A.far_ptr[a] : 0,
                   sbase = pass && A.small_ptr ? A.small_ptr[a] : 0;
    const uint32_t cnt_a = A.rho ? A.start[a + 1] - A.start[a] : 0u;
    for (uint64_t e = up_near_ptr[P]; e < up_near_ptr[P + 1]; ++e) {
        uint32_t Q = up_near_col[e];
        uint32_t b1 = up_cstart[Q + 1];
        for (uint32_t bq = up_cstart[Q]; bq < b1; ++bq) {
            int d2 = 0;
            int o[D];
#pragma unroll
            for (int d = 0; d < D; ++d) {
                o[d] = A.cell_src[(int64_t)bq * D + d] - ca[d];
                d2 += o[d] * o[d];
            }
            bool far_rule = d2 >= A.T;
            if (A.shifted) {
                double s = 0.0;
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    const double t = __dadd_rn((double)o[d], A.u[d]);
                    s = __dadd_rn(s, __dmul_rn(t, t));
                }
                far_rule = s >= A.theta2;
            }
            const bool is_small = A.rho && A.mode != 1 && cnt_a + (A.start_src[bq + 1] - A.start_src[bq]) <= A.rho;
            const bool is_far = A.mode == 2 || (A.mode == 0 && far_rule);
            if (is_small) {
                if (pass && A.small_col) A.small_col[sbase + ns] = bq;
                ++ns;
            } else if (is_far) {
                if (pass && A.far_col) A.far_col[fbase + nf] = bq;
                ++nf;
            } else {
                if (pass && A.near_col) A.near_col[nbase + nn] = bq;
                ++nn;
            }
        }
    }
    if (!pass) {
        A.cnt_near[a] = (uint32_t)nn;
        A.cnt_far[a] = (uint32_t)nf;
        if (A.cnt_small) A.cnt_small[a] = (uint32_t)ns;
    }
}

// The same lists by parent (one point set, far rule only, D <= 3): the 2^D children of a parent
// share their candidates, so one wavefront per parent enumerates them once, 64 to a step with a lane
// per candidate, and tests them against every child.  The candidates of a round are the children
// of up to 64 boxes near the parent, written into LDS in sequence order (lane = near box, running
// sum of the child counts); ballots keep a child's near and far entries in that order.
template <int D>
__global__ __launch_bounds__(64) void lists_parent_kernel(int pass, int64_t nparents,
                                                          const uint32_t *__restrict__ cstart,
                                                          const int32_t *__restrict__ cell,
                                                          const uint64_t *__restrict__ up_near_ptr,
                                                          const uint32_t *__restrict__ up_near_col, ListArg A) {
    constexpr int NC = 1 << D;   // children of a box, at most
    __shared__ uint32_t cand[64 * NC];
    // workgroups go to the 8 dies in turn; every die takes a contiguous range of parents, whose rows and candidates
    // neighbour each other in memory (whole lines leave one L2, shared candidates are read into one L2)
    const int64_t per_die = (nparents + 7) >> 3;
    const int64_t P = (int64_t)(blockIdx.x & 7u) * per_die + (int64_t)(blockIdx.x >> 3);
    if (P >= nparents) return;
    const int lane = threadIdx.x;
    const uint32_t a0 = cstart[P];
    const int nt = min((int)(cstart[P + 1] - a0), NC);
    if (nt <= 0) return;   // (boxes are never empty: cannot happen)
    // lane t < nt holds the cell and the row offsets of child a0 + t
    const uint32_t at = a0 + (uint32_t)min(lane, nt - 1);
    int32_t tc[D];
#pragma unroll
    for (int d = 0; d < D; ++d) tc[d] = cell[(int64_t)at * D + d];
    uint64_t nbase = 0, fbase = 0;
    if (pass && A.near_ptr) nbase = A.near_ptr[at];
    if (pass && A.far_ptr) fbase = A.far_ptr[at];
    uint32_t nn[NC], nf[NC];   // entries so far per child (wave-uniform)
#pragma unroll
    for (int t = 0; t < NC; ++t) nn[t] = nf[t] = 0;
    const uint64_t e0 = up_near_ptr[P], e1 = up_near_ptr[P + 1];
    for (uint64_t er = e0; er < e1; er += 64) {
        const int m = (int)(e1 - er < 64 ? e1 - er : 64);
        uint32_t b0 = 0, nq = 0;
        if (lane < m) {
            const uint32_t Q = up_near_col[er + lane];
            b0 = cstart[Q];
            nq = min(cstart[Q + 1] - b0, (uint32_t)NC);
        }
        const uint32_t cend = wave_incl_scan_u32(nq);   // inclusive running sum of the child counts over the lanes
        const uint32_t cbeg = cend - nq;
        const uint32_t S = __builtin_amdgcn_readlane(cend, 63);   // candidates of this round, <= 64 NC
        __syncthreads();   // the previous round has been read
        for (uint32_t j = 0; j < nq; ++j) cand[cbeg + j] = b0 + j;
        __syncthreads();
        for (uint32_t w0 = 0; w0 < S; w0 += 64) {
            const bool live = w0 + lane < S;
            const uint32_t bq = live ? cand[w0 + lane] : 0u;   // (a lane beyond the sequence reads box 0, unused)
            int32_t cc[D];
#pragma unroll
            for (int d = 0; d < D; ++d) cc[d] = A.cell_src[(int64_t)bq * D + d];
            if constexpr (D == 3) {
                if (pass && A.st_cand && live) {
                    // grid position of the candidate: its cell minus twice the parent's cell, plus 2 (a box near
                    // the parent is within one cell of it, so every coordinate lies in [0, 6))
                    int pos = 0, mul = 1;
                    bool inside = true;
#pragma unroll
                    for (int d = 0; d < D; ++d) {
                        const int q = cc[d] - 2 * (__builtin_amdgcn_readlane(tc[d], 0) >> 1) + 2;
                        inside = inside && q >= 0 && q < 6;
                        pos += q * mul;
                        mul *= 6;
                    }
                    if (inside) A.st_cand[P * 216 + pos] = bq;
                }
            }
#pragma unroll
            for (int t = 0; t < NC; ++t) {
                if (t < nt) {   // wave-uniform
                    int d2 = 0;
#pragma unroll
                    for (int d = 0; d < D; ++d) {
                        const int o = cc[d] - __builtin_amdgcn_readlane(tc[d], t);
                        d2 += o * o;
                    }
                    const bool is_far = d2 >= A.T;
                    const uint64_t mn = __ballot(live && !is_far), mf = __ballot(live && is_far);
                    if (pass) {
                        const uint64_t below = (1ull << lane) - 1ull;
                        if (A.near_col && live && !is_far) {
                            const uint64_t base = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(nbase >> 32), t) << 32) |
                                                  (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)nbase, t);
                            A.near_col[base + nn[t] + (uint32_t)__popcll(mn & below)] = bq;
                        }
                        if (A.far_col && live && is_far) {
                            const uint64_t base = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(fbase >> 32), t) << 32) |
                                                  (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)fbase, t);
                            A.far_col[base + nf[t] + (uint32_t)__popcll(mf & below)] = bq;
                        }
                    }
                    nn[t] += (uint32_t)__popcll(mn);
                    nf[t] += (uint32_t)__popcll(mf);
                }
            }
        }
    }
    if constexpr (D == 3) {
        if (pass && A.st_child && lane < nt)   // the child of each parity (bit d = upper half along dimension d)
            A.st_child[P * 8 + ((tc[0] & 1) | ((tc[1] & 1) << 1) | ((tc[2] & 1) << 2))] = a0 + (uint32_t)lane;
    }
    if (!pass) {
        uint32_t vn = 0, vf = 0;
#pragma unroll
        for (int t = 0; t < NC; ++t)
            if (lane == t) { vn = nn[t]; vf = nf[t]; }
        if (lane < nt) {
            A.cnt_near[a0 + lane] = vn;
            A.cnt_far[a0 + lane] = vf;
            if (A.cnt_small) A.cnt_small[a0 + lane] = 0u;
        }
    }
}

// The same with a wavefront per target box: 64 candidates at a time, a lane each, ballots keep the entries in candidate
// order.  lists_kernel waits for one dependent read of a cell after the other; with few or long rows (few boxes; up to
// 2^D children of up to 3^D near boxes) there are not enough threads to hide that.
template <int D>
__global__ __launch_bounds__(64) void lists_wave_kernel(int pass, int64_t nb, const uint32_t *__restrict__ parent,
                                                        const int32_t *__restrict__ cell,
                                                        const uint64_t *__restrict__ up_near_ptr,
                                                        const uint32_t *__restrict__ up_near_col,
                                                        const uint32_t *__restrict__ up_cstart, ListArg A) {
    __shared__ uint32_t cend[64], cdelta[64];   // near boxes of the parent: end in the sequence, position -> box rank
    const int64_t a = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    if (a >= nb) return;
    const int lane = threadIdx.x;
    int32_t ca[D];
#pragma unroll
    for (int d = 0; d < D; ++d) ca[d] = cell[a * D + d];
    const uint32_t P = parent[a];
    uint64_t nbase = pass && A.near_ptr ? A.near_ptr[a] : 0, fbase = pass && A.far_ptr ? A.far_ptr[a] : 0,
             sbase = pass && A.small_ptr ? A.small_ptr[a] : 0;
    uint32_t nn = 0, nf = 0, ns = 0;
    const uint32_t cnt_a = A.rho ? A.start[a + 1] - A.start[a] : 0u;
    const uint64_t e0 = up_near_ptr[P], e1 = up_near_ptr[P + 1];
    for (uint64_t er = e0; er < e1; er += 64) {
        const int m = (int)(e1 - er < 64 ? e1 - er : 64);
        uint32_t b0 = 0, nq = 0;
        if (lane < m) {
            const uint32_t Q = up_near_col[er + lane];
            b0 = up_cstart[Q];
            nq = up_cstart[Q + 1] - b0;
        }
        const uint32_t end = wave_incl_scan_u32(nq);
        const uint32_t S = __builtin_amdgcn_readlane(end, 63);   // candidates of this round
        __syncthreads();   // the previous round has been read
        cend[lane] = end;
        cdelta[lane] = b0 - (end - nq);
        __syncthreads();
        for (uint32_t w0 = 0; w0 < S; w0 += 64) {
            const bool live = w0 + lane < S;
            const uint32_t p = min(w0 + (uint32_t)lane, S - 1u);
            int lo = 0;   // first entry with cend > p (the last one has S > p)
#pragma unroll
            for (int s = 32; s > 0; s >>= 1) lo += cend[lo + s - 1] <= p ? s : 0;
            const uint32_t bq = p + cdelta[lo];
            int d2 = 0;
            int o[D];
#pragma unroll
            for (int d = 0; d < D; ++d) {
                o[d] = A.cell_src[(int64_t)bq * D + d] - ca[d];
                d2 += o[d] * o[d];
            }
            bool far_rule = d2 >= A.T;
            if (A.shifted) {
                double s = 0.0;
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    const double t = __dadd_rn((double)o[d], A.u[d]);
                    s = __dadd_rn(s, __dmul_rn(t, t));
                }
                far_rule = s >= A.theta2;
            }
            const bool is_small = live && A.rho && A.mode != 1 && cnt_a + (A.start_src[bq + 1] - A.start_src[bq]) <= A.rho;
            const bool is_far = live && !is_small && (A.mode == 2 || (A.mode == 0 && far_rule));
            const bool is_near = live && !is_small && !is_far;
            const uint64_t mn = __ballot(is_near), mf = __ballot(is_far), ms = __ballot(is_small);
            if (pass) {
                const uint64_t below = (1ull << lane) - 1ull;
                if (A.near_col && is_near) A.near_col[nbase + (uint32_t)__popcll(mn & below)] = bq;
                if (A.far_col && is_far) A.far_col[fbase + (uint32_t)__popcll(mf & below)] = bq;
                if (A.small_col && is_small) A.small_col[sbase + (uint32_t)__popcll(ms & below)] = bq;
                nbase += (uint32_t)__popcll(mn);
                fbase += (uint32_t)__popcll(mf);
                sbase += (uint32_t)__popcll(ms);
            } else {
                nn += (uint32_t)__popcll(mn);
                nf += (uint32_t)__popcll(mf);
                ns += (uint32_t)__popcll(ms);
            }
        }
    }
    if (!pass && lane == 0) {
        A.cnt_near[a] = nn;
        A.cnt_far[a] = nf;
        if (A.cnt_small) A.cnt_small[a] = ns;
    }
}

// the rule of the depth is the plain far rule on one point set: the lists can be built by parent
static bool lists_by_parent(const ListArg &A, int D) { return D <= 3 && !A.shifted && A.rho == 0 && A.mode == 0; }

// the rule part of a list kernel argument for one depth of a plan
static ListArg list_rules(const f3m_plan_s &P, int level) {
    const f3m_level &lv = P.lev[level], &sv = P.slev(level);
    ListArg A{};
    A.T = P.T;
    A.mode = P.force_all_near ? 1 : lv.smooth ? 2 : 0;
    A.rho = (uint32_t)P.rho;
    A.start = lv.start.p;
    A.cell_src = sv.cell.p;
    A.start_src = sv.start.p;
    A.shifted = P.src ? 1 : 0;
    P.grid_shift(level, A.u);
    A.theta2 = (double)P.theta * (double)P.theta;
    return A;
}

// One pass over the candidates of a depth.  By parent where the rule allows it; else a wavefront per box above three
// dimensions, where rows are long (n = 3e5, D = 7: plan and product 48.8 -> 37.2 ms), and for fewer than 2^17 boxes,
// whose threads would not fill the chip (two sets, 1e7 x 1e5: 3.14 -> 2.84 ms); with more boxes of at most 216
// candidates each the thread per box issues a quarter of the instructions.
template <int D>
static void launch_lists(int pass, const f3m_plan_s &P, int level, const ListArg &A, bool by_parent, hipStream_t st) {
    const f3m_level &lv = P.lev[level], &up = P.lev[level - 1];
    const uint32_t *up_cstart = P.slev(level - 1).cstart.p;
    bool done = false;
    if constexpr (D <= 3) {
        if (by_parent) {
            lists_parent_kernel<D><<<dim3((unsigned)((up.nb + 7) / 8 * 8)), dim3(64), 0, st>>>(
                pass, up.nb, up.cstart.p, lv.cell.p, up.near_ptr.p, up.near_col.p, A);
            done = true;
        } else if (lv.nb >= (1 << 17)) {
            lists_kernel<D><<<dim3((unsigned)cdiv(lv.nb, 128)), dim3(128), 0, st>>>(
                pass, lv.nb, lv.parent.p, lv.cell.p, up.near_ptr.p, up.near_col.p, up_cstart, A);
            done = true;
        }
    }
    if (!done) {
        const int64_t gx = std::min<int64_t>(lv.nb, 1 << 20);
        lists_wave_kernel<D><<<dim3((unsigned)gx, (unsigned)cdiv(lv.nb, gx)), dim3(64), 0, st>>>(
            pass, lv.nb, lv.parent.p, lv.cell.p, up.near_ptr.p, up.near_col.p, up_cstart, A);
    }
    F3M_HIP(hipGetLastError());
}

// Point pairs of a CSR interaction list, |p| * sum of |q| over the row of p: a wavefront per row, a partial sum per
// workgroup.
__global__ __launch_bounds__(256) void point_pairs_kernel(const uint32_t *__restrict__ start,
                                                          const uint32_t *__restrict__ start_src,
                                                          const uint64_t *__restrict__ row_ptr,
                                                          const uint32_t *__restrict__ cols, int64_t nb,
                                                          uint64_t *__restrict__ part) {
    __shared__ uint64_t wsum[4];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint64_t total = 0;
    for (int64_t a = (int64_t)blockIdx.x * 4 + w; a < nb; a += (int64_t)gridDim.x * 4) {
        uint64_t s = 0;
        for (uint64_t e = row_ptr[a] + lane; e < row_ptr[a + 1]; e += 64) {
            const uint32_t q = cols[e];
            s += start_src[q + 1] - start_src[q];
        }
        total += s * (uint64_t)(start[a + 1] - start[a]);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) total += __shfl_xor(total, off, 64);
    if (lane == 0) wsum[w] = total;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = wsum[0] + wsum[1] + wsum[2] + wsum[3];
}

// waits for the stream (the thread has an open scope of it)
static int64_t point_pairs(const uint32_t *start, const uint32_t *start_src, const uint64_t *row_ptr, const uint32_t *cols,
                           int64_t nb, hipStream_t st) {
    if (nb <= 0) return 0;
    const int64_t grid = std::min<int64_t>(4096, cdiv(nb, 4));
    DevBuf<uint64_t> part;
    part.alloc((size_t)grid);
    uint64_t *total = scope_words();
    point_pairs_kernel<<<dim3((unsigned)grid), dim3(256), 0, st>>>(start, start_src, row_ptr, cols, nb, part.p);
    scan_block_sums(part.p, grid, total, st);
    F3M_HIP(hipGetLastError());
    F3M_HIP(hipStreamSynchronize(st));
    return (int64_t)*total;
}

// offsets of n items, and the total behind them
struct PtrOut {
    uint64_t *p;
    int64_t n;
    __device__ void operator()(int64_t i, uint64_t ex, uint64_t v) const {
        p[i] = ex;
        if (i == n - 1) p[n] = ex + v;
    }
};
// the same for two lists whose totals are below 2^32, in the halves of one number
struct PairIn {
    const uint32_t *a, *b;
    __device__ uint64_t operator()(int64_t i) const { return (uint64_t)a[i] | ((uint64_t)b[i] << 32); }
};
struct PairOut {
    uint64_t *p, *q;
    int64_t n;
    __device__ void operator()(int64_t i, uint64_t ex, uint64_t v) const {
        p[i] = ex & 0xFFFFFFFFull;
        q[i] = ex >> 32;
        if (i == n - 1) {
            p[n] = (ex + v) & 0xFFFFFFFFull;
            q[n] = (ex + v) >> 32;
        }
    }
};
struct FirstOut {
    uint32_t *p;
    int64_t n;
    __device__ void operator()(int64_t i, uint64_t ex, uint64_t v) const {
        p[i] = (uint32_t)ex;
        if (i == n - 1) p[n] = (uint32_t)(ex + v);
    }
};

// ------------------------------------------------------------------------------------
// work splits: runs of at most `chunk` points inside a box
// ------------------------------------------------------------------------------------
struct ChunkCountIn {
    const uint32_t *start;
    uint32_t chunk;
    __device__ uint64_t operator()(int64_t a) const { return (start[a + 1] - start[a] + chunk - 1) / chunk; }
};

__global__ __launch_bounds__(256) void chunk_box_kernel(const uint32_t *__restrict__ first, int64_t nb, int64_t nchunks,
                                                        uint32_t *__restrict__ chunk_box) {
    int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (c >= nchunks) return;
    // largest a with first[a] <= c   (first is non-decreasing, first[nb] = nchunks > c)
    int64_t lo = 0, hi = nb;
    while (hi - lo > 1) {
        int64_t mid = (lo + hi) >> 1;
        if ((int64_t)first[mid] <= c) lo = mid; else hi = mid;
    }
    chunk_box[c] = (uint32_t)lo;
}

// runs of at most `chunk` points inside the boxes whose row of a CSR list is not empty
struct ChunkCountIfIn {
    const uint32_t *start;
    const uint64_t *row_ptr;
    uint32_t chunk;
    __device__ uint64_t operator()(int64_t a) const {
        return row_ptr[a + 1] > row_ptr[a] ? (start[a + 1] - start[a] + chunk - 1) / chunk : 0;
    }
};

// runs of at most `chunk` points inside the boxes that carry a flag
struct ChunkCountFlagIn {
    const uint32_t *start;
    const uint32_t *flag;
    uint32_t chunk;
    __device__ uint64_t operator()(int64_t a) const { return flag[a] ? (start[a + 1] - start[a] + chunk - 1) / chunk : 0; }
};

// Near-field tiles of the last depth.  A box is cut into runs of 64 targets; a last run of at most `ts`
// targets (the overflow of a box a little above 64 points, or a box with very few points) would leave
// most of a 64-wide tile idle, so it becomes an "overflow tile" for the kernel that puts the SOURCES on
// the lanes instead.  Big tiles: the full runs, and the last run if it has more than ts targets.
struct BigTileCountIn {
    const uint32_t *start;
    uint32_t ts;
    __device__ uint64_t operator()(int64_t a) const {
        const uint32_t cnt = start[a + 1] - start[a];
        return cnt / 64u + ((cnt & 63u) > ts ? 1u : 0u);
    }
};
struct OverflowTileCountIn {
    const uint32_t *start;
    uint32_t ts;
    __device__ uint64_t operator()(int64_t a) const {
        const uint32_t rem = (start[a + 1] - start[a]) & 63u;
        return rem >= 1u && rem <= ts ? 1u : 0u;
    }
};

// Pairs of leaf boxes for the paired near field: one thread per parent walks its children in rank order and
// pairs child i with child i + 1 when their cells differ in one dimension only (by one cell, being siblings),
// both first runs of targets are big tiles (64 targets, or more than ts) and both near rows have at most 32
// entries.  paired[a] = 1 for the first box of a pair, 2 for the second, 0 otherwise.
__global__ __launch_bounds__(256) void pair_flag_kernel(int64_t nparents, const uint32_t *__restrict__ cstart,
                                                        const int32_t *__restrict__ cell,
                                                        const uint32_t *__restrict__ start,
                                                        const uint64_t *__restrict__ near_ptr, uint32_t ts,
                                                        uint8_t *__restrict__ paired) {
    const int64_t P = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (P >= nparents) return;
    const uint32_t c0 = cstart[P], c1 = cstart[P + 1];
    auto fits = [&](uint32_t a) {
        const uint32_t cnt = start[a + 1] - start[a];
        return (cnt >= 64u || cnt > ts) && near_ptr[a + 1] - near_ptr[a] <= 32u;
    };
    uint32_t a = c0;
    while (a < c1) {
        bool pair = false;
        if (a + 1 < c1 && fits(a) && fits(a + 1)) {
            int differ = 0;
            for (int d = 0; d < 3; ++d) differ += cell[(int64_t)a * 3 + d] != cell[(int64_t)(a + 1) * 3 + d];
            pair = differ == 1;
        }
        if (pair) {
            paired[a] = 1;
            paired[a + 1] = 2;
            a += 2;
        } else {
            paired[a] = 0;
            a += 1;
        }
    }
}
struct PairCountIn {
    const uint8_t *paired;
    __device__ uint64_t operator()(int64_t a) const { return paired[a] == 1 ? 1u : 0u; }
};
// the big tiles of a box without the first run of a paired box
struct RestTileCountIn {
    const uint32_t *start;
    uint32_t ts;
    const uint8_t *paired;
    __device__ uint64_t operator()(int64_t a) const {
        const uint32_t cnt = start[a + 1] - start[a];
        return cnt / 64u + ((cnt & 63u) > ts ? 1u : 0u) - (paired[a] ? 1u : 0u);
    }
};

// flag[c] = 1 for every column c of a list (equal values from several threads: plain vector stores)
__global__ __launch_bounds__(256) void mark_cols_kernel(const uint32_t *__restrict__ cols, int64_t count,
                                                        uint32_t *__restrict__ flag) {
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < count; e += (int64_t)gridDim.x * 256)
        flag[cols[e]] = 1u;
}

// Lists of work items counted per box: first[nb+1] (exclusive scan) and the box of every item.  The counts of all the
// lists that are asked for are waited for together (build).
struct ItemLists {
    struct List {
        int64_t nb;
        const uint32_t *first;
        DevBuf<uint32_t> *box;
        int64_t *nitems;
    };
    int64_t *tally;
    hipStream_t st;
    std::vector<List> lists;
    ItemLists(int64_t *tally_, hipStream_t st_) : tally(tally_), st(st_) {}

    template <class CountIn>
    void add(CountIn count, int64_t nb, DevBuf<uint32_t> &first, DevBuf<uint32_t> &box, int64_t &nitems) {
        if ((int)lists.size() >= HOST_WORDS) fail(F3M_ERR_HIP, "internal: too many lists of work items");
        first.alloc((size_t)nb + 1, tally);
        exclusive_scan(count, nb, FirstOut{first.p, nb}, scope_words() + lists.size(), st);
        lists.push_back(List{nb, first.p, &box, &nitems});
    }
    // runs of at most `chunk` points, in every box or in those with a row / a flag
    void chunks(const uint32_t *start, int64_t nb, uint32_t chunk, DevBuf<uint32_t> &first, DevBuf<uint32_t> &box,
                int64_t &nitems, const uint64_t *only_rows = nullptr, const uint32_t *only_flagged = nullptr) {
        if (only_flagged) add(ChunkCountFlagIn{start, only_flagged, chunk}, nb, first, box, nitems);
        else if (only_rows) add(ChunkCountIfIn{start, only_rows, chunk}, nb, first, box, nitems);
        else add(ChunkCountIn{start, chunk}, nb, first, box, nitems);
    }
    void build() {
        if (lists.empty()) return;
        F3M_HIP(hipStreamSynchronize(st));
        const uint64_t *totals = scope_words();
        for (size_t k = 0; k < lists.size(); ++k) {
            const List &W = lists[k];
            const int64_t items = (int64_t)totals[k];
            *W.nitems = items;
            W.box->alloc((size_t)items, tally);
            if (items > 0)
                chunk_box_kernel<<<dim3((unsigned)cdiv(items, 256)), dim3(256), 0, st>>>(W.first, W.nb, items, W.box->p);
            F3M_HIP(hipGetLastError());
        }
        lists.clear();
    }
};

// ------------------------------------------------------------------------------------
// a point set while it is partitioned: the targets X of the plan, or the sources Y of a two-set plan
struct SetRef {
    const float *X;
    int64_t n;
    float *alpha;
    DevBuf<uint32_t> *keys, *perm;
    DevBuf<float> *Xs;
    f3m_level *lev;
};

// per-dimension minimum and the largest extent (one fp32 subtraction per dimension) of a set
template <int D>
static float set_bounds(const SetRef &S, const char *name, hipStream_t st) {
    DevBuf<float> part;
    part.alloc((size_t)BBOX_BLOCKS * (2 * D + 1));
    // (a set that needs fewer blocks leaves no empty ones behind)
    const int blocks = (int)std::min<int64_t>(BBOX_BLOCKS, cdiv(S.n, BBOX_NT));
    uint64_t *words = scope_words();
    bbox_kernel<D><<<dim3(blocks), dim3(BBOX_NT), 0, st>>>(S.X, S.n, part.p);
    bbox_final_kernel<<<dim3(1), dim3(1024), 0, st>>>(part.p, blocks, D, words);
    F3M_HIP(hipGetLastError());
    F3M_HIP(hipStreamSynchronize(st));
    auto value = [&](int k) {
        const uint32_t u = (uint32_t)words[k];
        float f;
        std::memcpy(&f, &u, sizeof(f));
        return f;
    };
    if (value(2 * D) != 0.f) fail(F3M_ERR_NONFINITE, std::string(name) + " holds a NaN or an infinity");
    float E = 0.f;
    for (int d = 0; d < D; ++d) {
        const float mn = value(d), mx = value(D + d);
        volatile float ext = mx - mn;  // one fp32 subtraction
        if (ext > E) E = ext;
        S.alpha[d] = mn;
    }
    return E;
}

// words of the scope's array that a depth leaves its counts in (word 0: scan_prepare)
enum { HW_NEAR = 1, HW_FAR = 2, HW_SMALL = 3, HW_SET = 4 };   // HW_SET + 2 k: largest box of set k, heads counted

// Divide (Algorithm 1): the box table of depth l of one set -- heads of runs of equal depth-l keys,
// from the points or, once the boxes of the depth above are few against the points, from their
// intervals -- with parent ranks, child intervals of the depth above and cells.  The size of the largest box arrives
// in `words` with the next wait for the stream (divide_finish).
template <int D>
static void divide_set(f3m_plan_s &P, const SetRef &S, int l, DevBuf<uint32_t> &part, uint64_t *words, hipStream_t st) {
    int64_t *tally = &P.bytes;
    const int64_t n = S.n;
    f3m_level &lv = S.lev[l];
    const uint32_t *keys = S.keys->p;
    if (l == 0) {
        lv.nb = 1;
        lv.key.alloc(1, tally);
        lv.start.alloc(2, tally);
        lv.parent.alloc(1, tally);
        lv.cell.alloc(D, tally);
        root_kernel<<<1, 1, 0, st>>>((uint32_t)n, D, lv.key.p, lv.start.p, lv.parent.p, lv.cell.p);
        F3M_HIP(hipGetLastError());
        lv.max_box = n;
        return;
    }
    const int shift = D * (P.Lq - l);
    f3m_level &up = S.lev[l - 1];
    up.cstart.alloc((size_t)up.nb + 1, tally);
    words[1] = (uint64_t)up.nb;
    if ((up.nb << D) <= n / 4) {
        const int64_t nslots = up.nb << D;
        DevBuf<uint32_t> lb;
        lb.alloc((size_t)nslots + 1);
        child_bounds_kernel<D><<<dim3((unsigned)cdiv(nslots, 256)), dim3(256), 0, st>>>(keys, shift, up.start.p, nslots,
                                                                                      up.key.p, lb.p, (uint32_t)n);
        F3M_HIP(hipGetLastError());
        ChildIn cin{lb.p};
        ScanState SS;
        scan_prepare(cin, nslots, SS, st);
        lv.nb = (int64_t)SS.total;
        lv.key.alloc((size_t)lv.nb, tally);
        lv.start.alloc((size_t)lv.nb + 1, tally);
        lv.parent.alloc((size_t)lv.nb, tally);
        scan_finish(cin, nslots, SS,
                    ChildOut<D>{lb.p, up.key.p, lv.start.p, lv.key.p, lv.parent.p, up.cstart.p, nslots}, st);
    } else {
        HeadIn hin{keys, shift};
        ScanState SS;
        scan_prepare(hin, n, SS, st);
        lv.nb = (int64_t)SS.total;
        lv.key.alloc((size_t)lv.nb, tally);
        lv.start.alloc((size_t)lv.nb + 1, tally);
        lv.parent.alloc((size_t)lv.nb, tally);
        scan_finish(hin, n, SS, HeadOut{keys, shift, lv.start.p, lv.key.p, n}, st);
        exclusive_scan(HeadIn{lv.key.p, D}, lv.nb, ParentOut{lv.parent.p, up.cstart.p, lv.nb, up.nb}, words + 1, st);
    }
    {
        const int grid = lv.nb <= 16384 ? 1 : (int)std::min<int64_t>(1024, cdiv(lv.nb, 256));
        max_count_kernel<false><<<dim3(grid), dim3(256), 0, st>>>(lv.start.p, lv.nb, part.p, words);
        if (grid > 1) max_count_kernel<true><<<dim3(1), dim3(256), 0, st>>>(part.p, grid, part.p, words);
        F3M_HIP(hipGetLastError());
    }
    lv.cell.alloc((size_t)lv.nb * D, tally);
    cells_kernel<D><<<dim3((unsigned)cdiv(lv.nb, 256)), dim3(256), 0, st>>>(lv.key.p, lv.nb, l, lv.cell.p);
    F3M_HIP(hipGetLastError());
}

// after a wait for the stream
static void divide_finish(const SetRef &S, int l, const uint64_t *words) {
    S.lev[l].max_box = (int64_t)words[0];
    if ((int64_t)words[1] != S.lev[l - 1].nb) fail(F3M_ERR_HIP, "internal: parent count mismatch");
}

// The box tables of ALL depths from the sorted keys at once, for sets of up to BULK_MAX points.  A point is the head of a box at
// depth l iff its key differs from the one before it in the bits of depths <= l, so one number per point, the first
// depth at which it is a head, gives every table: counts per block and depth, a scan of them, and one pass that
// writes start, key, parent, cell and child ranges.  Depth by depth it was six launches and two waits each, and small sets are
// bound by those (plan and product of 1e5 points in 2-D 1.16 -> 1.00 ms, of 1e6 normal points 2.07 -> 1.82).
constexpr int64_t BULK_MAX = (int64_t)1 << 24;
constexpr int BULK_LEVELS = F3M_MAX_LEVELS + 1;
constexpr int BULK_TILE = 2048;   // 256 threads with eight keys each

// first depth at which two keys differ (Lq + 1: equal)
template <int D>
__device__ inline int first_depth(uint32_t a, uint32_t b, int Lq) {
    const uint32_t x = a ^ b;
    return x ? Lq - (31 - __clz((int)x)) / D : Lq + 1;
}

// heads of the eight points from base on: first depths, Lq + 2 behind the end
template <int D>
__device__ inline void head_depths(const uint32_t *__restrict__ keys, int64_t base, int64_t n, int Lq, uint32_t (&k)[9], int (&h)[8]) {
    // (whole tiles may be read: the keys carry slack)
    const uint4 *p = reinterpret_cast<const uint4 *>(keys + base);
    const uint4 a = p[0], b = p[1];
    k[0] = base > 0 ? keys[base - 1] : 0u;
    k[1] = a.x; k[2] = a.y; k[3] = a.z; k[4] = a.w; k[5] = b.x; k[6] = b.y; k[7] = b.z; k[8] = b.w;
#pragma unroll
    for (int j = 0; j < 8; ++j) h[j] = base + j >= n ? Lq + 2 : base + j == 0 ? 0 : first_depth<D>(k[j], k[j + 1], Lq);
}

// counts[l][block]: heads of depth l in the block; *depth: the first depth whose boxes all hold at most zeta points (a box
// of depth l holds more iff some point and the one zeta places further on agree in the bits of depth l)
template <int D>
__global__ __launch_bounds__(256) void levels_count_kernel(const uint32_t *__restrict__ keys, int64_t n, int Lq, int zeta,
                                                           int nlevels, int64_t nblk, uint32_t *__restrict__ counts,
                                                           uint32_t *__restrict__ depth) {
    __shared__ uint32_t wsum[4][BULK_LEVELS];
    __shared__ uint32_t wdeep[4];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t base = (int64_t)blockIdx.x * BULK_TILE + (int64_t)tid * 8;
    uint32_t k[9];
    int h[8];
    head_depths<D>(keys, base, n, Lq, k, h);
    uint32_t deep = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j)
        if (base + j + zeta < n) deep = max(deep, (uint32_t)first_depth<D>(k[j + 1], keys[base + j + zeta], Lq));
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) deep = max(deep, (uint32_t)__shfl_xor((int)deep, off, 64));
    for (int l = 0; l < nlevels; ++l) {
        uint32_t c = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) c += (uint32_t)__popcll(__ballot(h[j] <= l));
        if (lane == 0) wsum[w][l] = c;
    }
    if (lane == 0) wdeep[w] = deep;
    __syncthreads();
    if (tid < nlevels) counts[(int64_t)tid * nblk + blockIdx.x] = wsum[0][tid] + wsum[1][tid] + wsum[2][tid] + wsum[3][tid];
    if (tid == 64) {
        const uint32_t d = max(max(wdeep[0], wdeep[1]), max(wdeep[2], wdeep[3]));
        if (d > *(volatile uint32_t *)depth) atomicMax(depth, d);   // (thousands of blocks, few of which raise it)
    }
}

// counts of a depth -> positions of its blocks (a workgroup per depth); totals and the depth to words of the host
__global__ __launch_bounds__(1024) void levels_scan_kernel(uint32_t *__restrict__ counts, int64_t nblk,
                                                           const uint32_t *__restrict__ depth, uint64_t *__restrict__ words) {
    __shared__ uint32_t wsum[16];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, l = blockIdx.x;
    uint32_t *c = counts + (int64_t)l * nblk;
    uint32_t carry = 0;
    for (int64_t r = 0; r < nblk; r += 1024) {
        const uint32_t v = r + tid < nblk ? c[r + tid] : 0u;
        const uint32_t incl = wave_incl_scan_u32(v);
        __syncthreads();   // the last round has read wsum
        if (lane == 63) wsum[w] = incl;
        __syncthreads();
        uint32_t before = carry;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            before += q < w ? wsum[q] : 0u;
            carry += wsum[q];
        }
        if (r + tid < nblk) c[r + tid] = before + incl - v;
    }
    if (tid == 0) {
        words[l] = carry;
        if (l == 0) words[BULK_LEVELS] = *depth;
    }
}

struct LevelTables {
    uint32_t *start[BULK_LEVELS], *key[BULK_LEVELS], *parent[BULK_LEVELS], *cstart[BULK_LEVELS];
    int32_t *cell[BULK_LEVELS];
    uint32_t nb[BULK_LEVELS];
};
// depths 1 .. L (the root is written by root_kernel)
template <int D>
__global__ __launch_bounds__(256) void levels_apply_kernel(const uint32_t *__restrict__ keys, int64_t n, int Lq, int L,
                                                           int64_t nblk, const uint32_t *__restrict__ counts, LevelTables T) {
    __shared__ uint32_t wsum[2][4];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t base = (int64_t)blockIdx.x * BULK_TILE + (int64_t)tid * 8;
    uint32_t k[9];
    int h[8];
    head_depths<D>(keys, base, n, Lq, k, h);
    uint32_t up[8];   // rank of the box of every point, one depth up
#pragma unroll
    for (int j = 0; j < 8; ++j) up[j] = 0u;
    for (int l = 1; l <= L; ++l) {
        uint32_t c = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) c += h[j] <= l ? 1u : 0u;
        const uint32_t incl = wave_incl_scan_u32(c);
        if (lane == 63) wsum[l & 1][w] = incl;
        __syncthreads();   // (two arrays in turn: one barrier per depth)
        uint32_t r = counts[(int64_t)l * nblk + blockIdx.x] + incl - c;
#pragma unroll
        for (int q = 0; q < 3; ++q) r += q < w ? wsum[l & 1][q] : 0u;
        const int shift = D * (Lq - l);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (h[j] <= l) {
                const uint32_t key = (uint32_t)((uint64_t)k[j + 1] >> shift);
                T.start[l][r] = (uint32_t)(base + j);
                T.key[l][r] = key;
                T.parent[l][r] = up[j];
                if (h[j] < l) T.cstart[l - 1][up[j]] = r;
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    int32_t cc = 0;
                    for (int b = 0; b < l; ++b) cc |= (int32_t)((key >> (b * D + d)) & 1u) << b;
                    T.cell[l][(int64_t)r * D + d] = cc;
                }
                ++r;
            }
            up[j] = r - 1u;   // (wraps for the points before the first head of the block's first box only if none precedes:
                              // point 0 is a head of every depth)
            if (base + j == n - 1) {
                T.start[l][T.nb[l]] = (uint32_t)n;
                T.cstart[l - 1][T.nb[l - 1]] = T.nb[l];
            }
        }
    }
}

// largest box of every depth 1 .. L: gridDim.y depths, a maximum per block; then to words of the host
__global__ __launch_bounds__(256) void levels_max_kernel(LevelTables T, uint32_t *__restrict__ largest) {
    const int l = 1 + (int)blockIdx.y;
    uint32_t m = 0;
    for (uint32_t a = blockIdx.x * 256u + threadIdx.x; a < T.nb[l]; a += gridDim.x * 256u) m = max(m, T.start[l][a + 1] - T.start[l][a]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off, 64));
    if ((threadIdx.x & 63) == 0 && m) atomicMax(&largest[l], m);
}
__global__ __launch_bounds__(64) void levels_max_words_kernel(const uint32_t *__restrict__ largest, int L, uint64_t *__restrict__ words) {
    if ((int)threadIdx.x <= L) words[threadIdx.x] = largest[threadIdx.x];
}

// words of the host that the tables of set k report in: boxes of every depth and the last depth, later the largest boxes
inline uint64_t *bulk_words(size_t k) { return scope_words() + 64 + 64 * k; }

// depths of the tree (first step, ends with a wait) and its tables (second step) for all sets; returns the depth where the
// largest box of one of the sets is at most zeta, or cap
template <int D>
static int bulk_divide(f3m_plan_s &P, const std::vector<SetRef> &sets, int cap, hipStream_t st) {
    int64_t *tally = &P.bytes;
    DevBuf<uint32_t> counts[2], depth;
    depth.alloc(2 + 2 * BULK_LEVELS);   // per set: the depth; the largest boxes
    fill_words(depth.p, 2 + 2 * BULK_LEVELS, nullptr, 0, 0u, st);
    for (size_t k = 0; k < sets.size(); ++k) {
        const int64_t n = sets[k].n, nblk = cdiv(n, BULK_TILE);
        counts[k].alloc((size_t)(cap + 1) * (size_t)nblk);
        levels_count_kernel<D><<<dim3((unsigned)nblk), dim3(256), 0, st>>>(sets[k].keys->p, n, P.Lq, P.leaf_max, cap + 1, nblk,
                                                                          counts[k].p, depth.p + k);
        levels_scan_kernel<<<dim3((unsigned)cap + 1), dim3(1024), 0, st>>>(counts[k].p, nblk, depth.p + k, bulk_words(k));
    }
    F3M_HIP(hipGetLastError());
    F3M_HIP(hipStreamSynchronize(st));
    int L = cap;
    for (size_t k = 0; k < sets.size(); ++k) L = std::min(L, (int)bulk_words(k)[BULK_LEVELS]);
    // the loop over the depths ends at the smooth depth at the latest (Sec. 4.3)
    for (int l = 1; l < L; ++l)
        if (!P.force_all_near && smooth_rule((double)P.E, l, D, (double)P.gamma, (double)P.eta_smooth)) L = l;
    for (size_t k = 0; k < sets.size(); ++k) {
        const SetRef &S = sets[k];
        const int64_t nblk = cdiv(S.n, BULK_TILE);
        LevelTables T{};
        for (int l = 0; l <= L; ++l) {
            f3m_level &lv = S.lev[l];
            lv.nb = l ? (int64_t)bulk_words(k)[l] : 1;
            lv.max_box = S.n;   // (of the root; the others: bulk_finish)
            lv.key.alloc((size_t)lv.nb, tally);
            lv.start.alloc((size_t)lv.nb + 1, tally);
            lv.parent.alloc((size_t)lv.nb, tally);
            lv.cell.alloc((size_t)lv.nb * D, tally);
            if (l < L) lv.cstart.alloc((size_t)lv.nb + 1, tally);
            T.start[l] = lv.start.p;
            T.key[l] = lv.key.p;
            T.parent[l] = lv.parent.p;
            T.cstart[l] = lv.cstart.p;
            T.cell[l] = lv.cell.p;
            T.nb[l] = (uint32_t)lv.nb;
        }
        root_kernel<<<1, 1, 0, st>>>((uint32_t)S.n, D, T.key[0], T.start[0], T.parent[0], T.cell[0]);
        if (L >= 1) {
            uint32_t *largest = depth.p + 2 + k * BULK_LEVELS;
            levels_apply_kernel<D><<<dim3((unsigned)nblk), dim3(256), 0, st>>>(S.keys->p, S.n, P.Lq, L, nblk, counts[k].p, T);
            const unsigned gx = (unsigned)std::min<int64_t>(64, cdiv(S.lev[L].nb, 256));
            levels_max_kernel<<<dim3(gx, (unsigned)L), dim3(256), 0, st>>>(T, largest);
            levels_max_words_kernel<<<dim3(1), dim3(64), 0, st>>>(largest, L, bulk_words(k));
        }
        F3M_HIP(hipGetLastError());
    }
    return L;
}

// after a wait for the stream
static void bulk_finish(const std::vector<SetRef> &sets, int L) {
    for (size_t k = 0; k < sets.size(); ++k)
        for (int l = 1; l <= L; ++l) sets[k].lev[l].max_box = (int64_t)bulk_words(k)[l];
}

template <int D>
static void build_plan_d(f3m_plan_s &P, const float *X, const float *Y, hipStream_t st) {
    const int64_t n = P.n;
    int64_t *tally = &P.bytes;
    for (int k = 0; k < 6; ++k) P.ev[k] = event_get();
    F3M_HIP(hipEventRecord(P.ev[0], st));
    // the set(s) to partition: the targets, and the sources when they are another set
    std::vector<SetRef> sets;
    sets.push_back(SetRef{X, n, P.alpha, &P.keys, &P.perm, &P.Xs, P.lev});
    if (P.src) sets.push_back(SetRef{Y, P.src->n, P.src->alpha, &P.src->keys, &P.src->perm, &P.src->Xs, P.src->lev});

    // ---- enclosing cubes: a common edge, the largest extent of either set (Sec. 3), each set
    //      anchored at its own per-dimension minimum (the alpha of the box-index formula, Sec. 4.2)
    {
        float E = 0.f;
        for (size_t k = 0; k < sets.size(); ++k) E = std::max(E, set_bounds<D>(sets[k], k ? "Y" : "X", st));
        P.E = E;
        P.scale = E > 0.f ? (float)(std::ldexp(1.0, P.Lq) / (double)E) : 0.f;
    }

    // ---- keys, sort, gather
    for (const SetRef &S : sets) {
        // (one tile of slack behind the keys and the indices: the sort reads whole tiles)
        S.keys->alloc((size_t)S.n + RS_SLACK, tally);
        S.perm->alloc((size_t)S.n + RS_SLACK, tally);
        AlphaArg aa;
        for (int d = 0; d < F3M_MAX_DIM; ++d) aa.a[d] = S.alpha[d];
        keys_kernel<D><<<dim3((unsigned)cdiv(S.n, 256)), dim3(256), 0, st>>>(S.X, S.n, aa, P.scale, P.Lq, S.keys->p);
        F3M_HIP(hipGetLastError());
    }
    F3M_HIP(hipEventRecord(P.ev[1], st));
    // Points whose products end at a depth of at most ROUTE_GROUP_DEPTH are only grouped by its boxes (below), for which the keys are
    // needed in the caller's order.  The depth, if the tree gets that far: the smooth one, or that of the weighted near pairs.
    bool may_group = false;
    if (D == 3 && !P.src && n >= P.route_min_n && P.rho == 0 && !P.force_all_near && P.E > 0.f)
        for (int l = 1; l <= ROUTE_GROUP_DEPTH && !may_group; ++l)
            may_group = smooth_rule((double)P.E, l, D, (double)P.gamma, (double)P.eta_smooth) ||
                        (l >= 2 && m2l_stencil_applies(P) && !P.adaptive_far && !(P.eta_smooth > 0.f) &&
                         near_weighted_error((double)P.E, l, (double)P.gamma) <= 0x1p-24);
    DevBuf<uint32_t> keys_in;   // ... in the caller's order (may_group)
    int bits_sorted = 0;
    for (const SetRef &S : sets) {
        DevBuf<uint32_t> keys_b, perm_b;
        if (may_group) keys_in.alloc((size_t)S.n + RS_SLACK);
        keys_b.alloc((size_t)S.n + RS_SLACK);
        perm_b.alloc((size_t)S.n + RS_SLACK);
        int bits = P.E > 0.f ? D * P.Lq : 0;
        bits_sorted = bits;
        bool in_b;
        if (bits == 0) {
            iota_kernel<<<dim3((unsigned)cdiv(S.n, 256)), dim3(256), 0, st>>>(S.perm->p, S.n);
            in_b = false;
        } else {
            in_b = radix_sort(S.keys->p, S.perm->p, keys_b.p, perm_b.p, keys_in.p, S.n, bits, st);
        }
        if (in_b) {
            std::swap(S.keys->p, keys_b.p);
            std::swap(S.perm->p, perm_b.p);
            if (keys_in.p) std::swap(keys_in.p, keys_b.p);   // keys_in: the input of the sort
        } else if (keys_in.p) {
            std::swap(S.keys->p, keys_in.p);
        }
    }
    F3M_HIP(hipEventRecord(P.ev[2], st));
    ZeroList zeros;   // cleared when the plan is otherwise complete
    bool grouped = false;   // the points are only grouped by the boxes of the last depth of the products
    // the points into box order, once that depth is known
    auto order_points = [&](size_t k) {
        const SetRef &S = sets[k];
        // 64 zero points of padding after the last point: kernels may read whole 32-point blocks
        S.Xs->alloc(((size_t)S.n + PAD_POINTS) * D, tally);
        zeros.add(S.Xs->p + (size_t)S.n * D, (size_t)PAD_POINTS * D);
        // A large set goes through the permutation in streaming passes, whose tables also serve every product
        // (route.hip); its points follow the same way when they have three coordinates.
        std::unique_ptr<f3m_route> &route = k ? P.src->route : P.route;
        const int last = P.last_depth();
        if (grouped) {
            route.reset(new f3m_route());
            route_group_build(*route, keys_in.p, S.n, P.Lq, last, P.lev[last].key.p, P.lev[last].nb, tally, st);
        } else if ((S.n >= P.route_min_n || (!P.route_given && route_two_passes(S.n))) && bits_sorted > 0) {
            route.reset(new f3m_route());
            route_build(*route, S.perm->p, S.n, S.n < P.route_min_n, tally, st);
        }
        if (route && D == 3) {
            DevBuf<float> tmp;
            if (!route->grouped) tmp.alloc((size_t)S.n * 3);
            route_gather_rows3(*route, S.X, S.Xs->p, tmp.p, st);
        } else {
            gather_rows_kernel<D><<<dim3((unsigned)cdiv(S.n, 256)), dim3(256), 0, st>>>(S.X, S.perm->p, S.n, S.Xs->p);
            F3M_HIP(hipGetLastError());
        }
    };

    // ---- Algorithm 1 loop: divide, new interactions, partition
    int cap = P.Lq;
    if (P.max_depth > 0 && P.max_depth < cap) cap = P.max_depth;
    if (cap > F3M_MAX_LEVELS) cap = F3M_MAX_LEVELS;
    if (!(P.E > 0.f)) cap = 0;
    DevBuf<uint32_t> part;
    part.alloc(1024);
    hipEvent_t ea = P.ev[4], eb = P.ev[5];
    // per depth: after the division, after the lists
    P.plan_events.resize(2 * (size_t)(cap + 1), nullptr);
    uint64_t *words = scope_words();
    int l = 0, weighted = 0;
    bool bulk = cap > 0;
    for (const SetRef &S : sets) bulk = bulk && S.n <= BULK_MAX;
    const int bulk_depth = bulk ? bulk_divide<D>(P, sets, cap, st) : 0;
    for (;; ++l) {
        f3m_level &lv = P.lev[l];
        for (size_t k = 0; k < sets.size() && !bulk; ++k) divide_set<D>(P, sets[k], l, part, words + HW_SET + 2 * k, st);
        const f3m_level &sv = P.slev(l);
        for (int k = 0; k < 2; ++k) P.plan_events[2 * (size_t)l + k] = event_get();
        F3M_HIP(hipEventRecord(P.plan_events[2 * (size_t)l], st));

        // new interactions + partition
        lv.near_ptr.alloc((size_t)lv.nb + 1, tally);
        lv.far_ptr.alloc((size_t)lv.nb + 1, tally);
        if (l == 0) {
            lv.near_col.alloc(1, tally);
            lv.far_col.alloc(1, tally);
            root_lists_kernel<<<1, 1, 0, st>>>(lv.near_ptr.p, lv.far_ptr.p, lv.near_col.p);
            F3M_HIP(hipGetLastError());
            lv.near_sz = 1;
            lv.far_sz = 0;
        } else {
            f3m_level &up = P.lev[l - 1];
            DevBuf<uint32_t> cn, cf, cs;
            cn.alloc((size_t)lv.nb);
            cf.alloc((size_t)lv.nb);
            if (P.rho > 0) cs.alloc((size_t)lv.nb);
            // Sec. 4.3: once the boxes pass the smoothness criterion every pair left is interpolated
            lv.smooth = !P.force_all_near && smooth_rule((double)P.E, l, D, (double)P.gamma, (double)P.eta_smooth);
            if (lv.smooth) P.smooth_depth = l;
            ListArg A = list_rules(P, l);
            A.cnt_near = cn.p;
            A.cnt_far = cf.p;
            A.cnt_small = cs.p;
            launch_lists<D>(0, P, l, A, lists_by_parent(A, D), st);
            words[HW_SMALL] = 0;
            // up to three dimensions with a far ratio of at most 2 a box has at most 216 candidates: both scans in one
            const bool both = D <= 3 && P.T <= 4 && P.rho == 0 && !P.src && !P.force_all_near && lv.nb < ((int64_t)1 << 24);
            if (both) {
                exclusive_scan(PairIn{cn.p, cf.p}, lv.nb, PairOut{lv.near_ptr.p, lv.far_ptr.p, lv.nb}, words + HW_NEAR, st);
            } else {
                exclusive_scan(U32In{cn.p}, lv.nb, PtrOut{lv.near_ptr.p, lv.nb}, words + HW_NEAR, st);
                exclusive_scan(U32In{cf.p}, lv.nb, PtrOut{lv.far_ptr.p, lv.nb}, words + HW_FAR, st);
            }
            if (P.rho > 0) {
                lv.small_ptr.alloc((size_t)lv.nb + 1, tally);
                exclusive_scan(U32In{cs.p}, lv.nb, PtrOut{lv.small_ptr.p, lv.nb}, words + HW_SMALL, st);
            }
            F3M_HIP(hipStreamSynchronize(st));
            if (bulk && l == 1) bulk_finish(sets, bulk_depth);
            for (size_t k = 0; k < sets.size() && !bulk; ++k) divide_finish(sets[k], l, words + HW_SET + 2 * k);
            const uint64_t tn = both ? words[HW_NEAR] & 0xFFFFFFFFull : words[HW_NEAR];
            const uint64_t tf = both ? words[HW_NEAR] >> 32 : words[HW_FAR], ts = words[HW_SMALL];
            if (P.rho > 0) lv.small_col.alloc((size_t)ts, tally);
            lv.near_sz = (int64_t)tn;
            lv.far_sz = (int64_t)tf;
            lv.small_sz = (int64_t)ts;
            lv.near_col.alloc((size_t)tn, tally);
            lv.p = P.adaptive_far ? adaptive_nodes((double)P.E, l, (double)P.gamma, P.p) : P.p;
            lv.r = 1;
            for (int d = 0; d < D; ++d) lv.r *= lv.p;
            if (tf > 0 && m2l_stencil_applies(P) && (lv.p == 4 || lv.p == 0)) {
                // the M2L of this depth enumerates the far partners itself (candidate grid around the
                // parent): only the row lengths are kept
                lv.far_implicit = true;
                lv.far_col.alloc(0, tally);
                // The first depth at which interpolating a pair of adjacent boxes is off by no more than 2^-24, the rounding
                // unit of fp32 (kernel values are close to 1 there), is the last one the products need: all the pairs
                // left there go through the M2L, and the tree below it only defines the lists that are reported.  Measured at n = 1e9,
                // lengthscale 1 (depth 5 of 8): 314 -> 82 ms for plan and product, the error against the oracle unchanged.
                if (P.near_depth == 0 && l >= 2 && lv.p == 4 && P.rho == 0 && !P.adaptive_far && !(P.eta_smooth > 0.f)) {
                    if (near_interp_error((double)P.E, l, (double)P.gamma) <= 0x1p-24) P.near_depth = l;
                    else if (weighted == 0 && near_weighted_error((double)P.E, l, (double)P.gamma) <= 0x1p-24) weighted = l;
                }
            } else if (tf > 0 && far_points_allowed(P, l)) {
                lv.far_points = far_points_pays(P, l, point_pairs(up.start.p, up.start.p, up.near_ptr.p, up.near_col.p, up.nb, st));
                lv.far_col.alloc(lv.far_points ? 0 : (size_t)tf, tally);
            } else {
                lv.far_col.alloc((size_t)tf, tally);
            }
            // two sets: near pairs between weighted points from the first depth on that allows it, as for one set
            if (P.src && weighted == 0 && D == 3 && l >= 2 && tf > 0 && lv.p == 4 && P.rho == 0 && !P.force_all_near &&
                !P.adaptive_far && !(P.eta_smooth > 0.f) && P.theta <= 4.f &&
                near_weighted_error((double)P.E, l, (double)P.gamma, (double)P.theta) <= 0x1p-24)
                weighted = l;
            A.near_ptr = lv.near_ptr.p;
            A.far_ptr = lv.far_ptr.p;
            A.small_ptr = lv.small_ptr.p;
            A.near_col = lv.near_col.p;
            A.far_col = lv.far_implicit || lv.far_points ? nullptr : lv.far_col.p;
            A.small_col = lv.small_col.p;
            if constexpr (D == 3) {
                // the tables of the candidate-grid M2L come out of the same enumeration
                if (lists_by_parent(A, D) && lv.far_implicit && lv.p != 0 && stencil_tables_alloc(P, l, st)) {
                    A.st_cand = lv.st_cand.p;
                    A.st_child = lv.st_child.p;
                }
            }
            launch_lists<D>(1, P, l, A, lists_by_parent(A, D), st);
        }
        F3M_HIP(hipEventRecord(P.plan_events[2 * (size_t)l + 1], st));
        // while interactions remain and the largest box of either tree is above zeta (Algorithm 1)
        if (!(lv.near_sz > 0 && lv.max_box > P.leaf_max && sv.max_box > P.leaf_max && l < cap)) break;
        if (bulk && l >= bulk_depth) fail(F3M_ERR_HIP, "internal: the tables end above the last depth");
    }
    // (small fields may have left no interactions above the last depth that has tables; they are not part of the plan)
    for (const SetRef &S : sets) {
        for (int k = l + 1; k <= bulk_depth; ++k) {
            f3m_level &lv = S.lev[k];
            for (DevBuf<uint32_t> *t : {&lv.key, &lv.start, &lv.parent, &lv.cstart}) t->release();
            lv.cell.release();
            lv.nb = lv.max_box = 0;
        }
        if (bulk_depth > l) S.lev[l].cstart.release();
    }
    P.L = l;
    product_depths(P.L, P.lev[l].nb, P.lev[l].far_sz > 0, P.lev[l].near_sz > 0, P.src != nullptr, may_group, weighted,
                   &P.near_depth, &P.near_weighted, &grouped);
    for (int k = P.last_depth() + 1; k <= P.L; ++k) {   // not needed: the products end above
        P.lev[k].st_cand.release();
        P.lev[k].st_child.release();
    }
    F3M_HIP(hipEventRecord(P.ev[3], st));
    for (size_t k = 0; k < sets.size(); ++k) order_points(k);
    keys_in.release();

    // ---- work splits and workspaces
    F3M_HIP(hipEventRecord(ea, st));
    // With D = 3 and 4 nodes per dimension node weights and node potentials are passed between
    // depths, so only the last depth streams the points.
    // the band of depths with implicit far rows and 4 nodes per dimension (under the adaptive rule
    // the deepest depths may use 3 nodes and the coarsest may be dropped)
    // (with 4 nodes per dimension in 3-D; the M2L of a depth in the band is the candidate-grid one where
    // that applies, else the one that works from the far list: two point sets, other far ratios)
    auto in_band = [&](int k) {
        return D == 3 && k >= 2 && P.lev[k].far_sz > 0 && P.lev[k].p == 4 && k <= P.last_depth();
    };
    for (int k = P.L; k >= 2 && P.tree_lmax == 0; --k)
        if (in_band(k)) P.tree_lmax = k;
    if (P.tree_lmax > 0) {
        P.tree_lmin = P.tree_lmax;
        while (in_band(P.tree_lmin - 1)) --P.tree_lmin;
    }
    upload_tables(P, st);
    build_far_orders(P, st);
    for (int k = 1; k <= P.L; ++k) build_stencil_tables(P, k, st);
    ItemLists items(tally, st);
    int64_t max_w = 0, max_v = 0;
    for (int k = 1; k <= P.L; ++k) {
        f3m_level &lv = P.lev[k];
        if (lv.far_sz == 0 || lv.p == 0 || k > P.last_depth()) continue;   // nothing to interpolate, or dropped
        if (lv.far_points) {
            far_points_prepare(P, k, st);
            const f3m_level &up = P.lev[k - 1];
            items.chunks(up.start.p, up.nb, FP_TT, lv.fp_tile_first, lv.fp_tile_box, lv.fp_ntiles);
            continue;
        }
        const bool tree = P.tree_lmin > 0 && k >= P.tree_lmin && k <= P.tree_lmax;
        f3m_level &sv = P.slev(k);
        if (tree) {
            // Node potentials are passed down the targets' tree.  One point set: node weights are passed up
            // the same tree, and carry one row of zeros behind the last box (what the candidate-grid M2L reads
            // for an absent candidate).  Two point sets: the node weights of every depth come from the points.
            const size_t twice = k == P.near_weighted ? 2 : 1;
            lv.Vl.alloc(twice * (size_t)lv.nb * lv.r, tally);
            if (!P.src) {
                lv.Wl.alloc(twice * (size_t)(lv.nb + 1) * lv.r, tally);
                for (size_t h = 1; h <= twice; ++h)
                    zeros.add(lv.Wl.p + (h * (size_t)(lv.nb + 1) - 1) * lv.r, (size_t)lv.r);
                if (k < P.tree_lmax) continue;   // only the last depth of the band needs chunks
            }
        }
        // Large boxes: long runs.  From 2048 points a box on: below, most runs would be short ones, and a wavefront per run
        // leaves the chip idle (n = 1e9, 32768 boxes: P2M 5.39 -> 3.66 ms, L2P 5.43 -> 3.63).
        if (D == 3 && lv.p == 4 && n / lv.nb >= P2M_LONG) lv.chunk = P2M_LONG;
        if (D == 3 && lv.p == 4 && P.src && P.ns() / sv.nb >= P2M_LONG) sv.chunk = P2M_LONG;
        // runs of points for the L2P (targets: in the band only its last depth) and the P2M (sources: the
        // same runs for one point set)
        if (!tree || k == P.tree_lmax)
            items.chunks(lv.start.p, lv.nb, (uint32_t)lv.chunk, lv.chunk_first, lv.chunk_box, lv.nchunks);
        if (P.src) {
            // Only the source boxes that occur in a far row of this depth need node weights (the two sets
            // may overlap in a small part of the sources' cube only).
            DevBuf<uint32_t> used;
            used.alloc((size_t)sv.nb);
            fill_words(used.p, sv.nb, nullptr, 0, 0u, st);
            mark_cols_kernel<<<dim3((unsigned)std::min<int64_t>(cdiv(lv.far_sz, 256), 1 << 20)), dim3(256), 0, st>>>(
                lv.far_col.p, lv.far_sz, used.p);
            F3M_HIP(hipGetLastError());
            items.chunks(sv.start.p, sv.nb, (uint32_t)sv.chunk, sv.chunk_first, sv.chunk_box, sv.nchunks, nullptr, used.p);
            if (k == P.near_weighted) {   // the same for the near rows
                f3m_level &ns = P.near_src;
                ns.nb = sv.nb;
                ns.max_box = sv.max_box;
                used.alloc((size_t)sv.nb);
                fill_words(used.p, sv.nb, nullptr, 0, 0u, st);
                mark_cols_kernel<<<dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>(cdiv(lv.near_sz, 256), 1 << 20))), dim3(256), 0, st>>>(
                    lv.near_col.p, lv.near_sz, used.p);
                F3M_HIP(hipGetLastError());
                items.chunks(sv.start.p, sv.nb, P2M_CHUNK, ns.chunk_first, ns.chunk_box, ns.nchunks, nullptr, used.p);
                if (ns.max_box > (int64_t)ns.chunk * P2M_SLICE * 2)
                    items.chunks(ns.chunk_first.p, ns.nb, P2M_SLICE, ns.slice_first, ns.slice_box, ns.nslices);
                ns.Wl.alloc((size_t)ns.nb * lv.r, tally);
            }
        }
        if (sv.max_box > (int64_t)sv.chunk * P2M_SLICE * 2) {
            // a box with more than a thousand chunks: its partial node weights are summed in two stages
            items.chunks(sv.chunk_first.p, sv.nb, P2M_SLICE, sv.slice_first, sv.slice_box, sv.nslices);
        }
        if (!tree || P.src) max_w = std::max(max_w, sv.nb * (int64_t)lv.r);
        if (!tree) max_v = std::max(max_v, lv.nb * (int64_t)lv.r);
    }
    if (P.exact_near()) {
        const f3m_level &lf = P.lev[P.L];
        // Few boxes: rows are long, and the near field splits every tile over several wavefronts; an overflow
        // tile would leave its whole row to one wavefront, so there are none (every run is a tile of its own).
        const uint32_t ts = lf.nb < 8192 ? 0u : (uint32_t)overflow_targets(D);
        items.add(BigTileCountIn{lf.start.p, ts}, lf.nb, P.tile_first, P.tile_box, P.ntiles);
        items.add(OverflowTileCountIn{lf.start.p, ts}, lf.nb, P.otile_first, P.otile_box, P.notiles);
    }
    // target tiles of the small-field rows of every depth (Sec. 4.2)
    for (int k = 1; k <= P.L; ++k) {
        f3m_level &lv = P.lev[k];
        if (lv.small_sz > 0)   // runs of targets as p2p_small_kernel takes them
            items.chunks(lv.start.p, lv.nb, D <= 4 ? 16 : 8, lv.sm_tile_first, lv.sm_tile_box, lv.sm_ntiles, lv.small_ptr.p);
    }
    items.build();
    int64_t max_part = 0, max_slice = 0;
    for (int k = 1; k <= P.L; ++k) {
        const f3m_level &sv = P.slev(k);
        max_part = std::max(max_part, (k == P.near_weighted ? 2 : 1) * sv.nchunks * (int64_t)P.lev[k].r);
        max_slice = std::max(max_slice, sv.nslices * (int64_t)P.lev[k].r);
    }
    if (P.near_weighted && P.src) {
        max_part = std::max(max_part, P.near_src.nchunks * (int64_t)P.lev[P.near_weighted].r);
        max_slice = std::max(max_slice, P.near_src.nslices * (int64_t)P.lev[P.near_weighted].r);
    }
    if (P.exact_near()) {
        const f3m_level &lf = P.lev[P.L];
        const uint32_t ts = lf.nb < 8192 ? 0u : (uint32_t)overflow_targets(D);
        // tiles worked in pairs (the rows must come from the plain far rule: the kernel tells the shared near
        // boxes of a pair by it)
        if (P.L >= 1 && ts > 0 && lf.near_sz > 0 && !lf.smooth && P.rho == 0 && p2p_pairs_allowed(P)) {
            const f3m_level &up = P.lev[P.L - 1];
            P.paired.alloc((size_t)lf.nb, tally);
            pair_flag_kernel<<<dim3((unsigned)cdiv(up.nb, 256)), dim3(256), 0, st>>>(
                up.nb, up.cstart.p, lf.cell.p, lf.start.p, lf.near_ptr.p, ts, P.paired.p);
            F3M_HIP(hipGetLastError());
            items.add(PairCountIn{P.paired.p}, lf.nb, P.pair_first, P.pair_box, P.npairs);
            items.add(RestTileCountIn{lf.start.p, ts, P.paired.p}, lf.nb, P.rtile_first, P.rtile_box, P.nrtiles);
            items.build();
        }
    }
    {
        // partial sums of a near field whose tiles are split over several wavefronts (few targets, long rows)
        const int nsplit = P.exact_near() && P.lev[P.L].near_sz > 0 ? p2p_nsplit(P, P.L, P.ntiles) : 1;
        if (nsplit > 1) P.p2p_part.alloc((size_t)nsplit * (size_t)n, tally);
    }
    if ((P.route && !P.route->grouped) || (P.src && P.src->route)) {
        const size_t m = (size_t)std::max<int64_t>(P.route ? n : 0, (P.src && P.src->route) ? P.src->n : (P.route ? n : 0));
        P.route_a.alloc(m, tally);
        P.route_b.alloc(m, tally);
    }
    P.bs.alloc((size_t)P.ns() + PAD_POINTS, tally);
    zeros.add(P.bs.p + P.ns(), PAD_POINTS);
    zeros.run(st);
    P.ys.alloc((size_t)n, tally);
    P.yn.alloc((size_t)n, tally);
    if (!P.no_overlap) F3M_HIP(hipStreamCreateWithFlags(&P.side, hipStreamNonBlocking));
    if (P.side)
        for (hipEvent_t *e : {&P.ev_fork, &P.ev_join, &P.ev_p2p0, &P.ev_p2p1}) *e = event_get();
    P.W.alloc((size_t)max_w, tally);
    P.V.alloc((size_t)max_v, tally);
    P.Wpart.alloc((size_t)max_part, tally);
    P.Wslice.alloc((size_t)max_slice, tally);
    F3M_HIP(hipEventRecord(eb, st));
    F3M_HIP(hipStreamSynchronize(st));

    float ms = 0.f;
    F3M_HIP(hipEventElapsedTime(&P.times.bbox_keys, P.ev[0], P.ev[1]));
    F3M_HIP(hipEventElapsedTime(&P.times.sort, P.ev[1], P.ev[2]));
    F3M_HIP(hipEventElapsedTime(&P.times.gather, P.ev[3], ea));
    P.host_tabs.clear();
    P.times.boxes = P.times.lists = 0.f;
    for (int k = 0; k <= P.L; ++k) {
        const hipEvent_t before = k ? P.plan_events[2 * (size_t)k - 1] : P.ev[2];
        const hipEvent_t mid = P.plan_events[2 * (size_t)k], after = P.plan_events[2 * (size_t)k + 1];
        F3M_HIP(hipEventElapsedTime(&ms, before, mid));
        P.times.boxes += ms;
        F3M_HIP(hipEventElapsedTime(&ms, mid, after));
        P.times.lists += ms;
    }
    F3M_HIP(hipEventElapsedTime(&P.times.tables, ea, eb));
    F3M_HIP(hipEventElapsedTime(&ms, P.ev[0], eb));
    P.times.plan_total = ms;
    P.have_plan_times = true;
}

// Far rows (CSR columns, ascending) of a depth that keeps only their lengths: the fill pass of
// the list kernel with the near side switched off.  cols_dev holds far_sz entries.
void materialize_far(const f3m_plan_s &P, int level, uint32_t *cols_dev, hipStream_t st) {
    const f3m_level &lv = P.lev[level];
    ListArg A = list_rules(P, level);
    A.far_ptr = lv.far_ptr.p;
    A.far_col = cols_dev;
    switch (P.D) {
        case 1: launch_lists<1>(1, P, level, A, false, st); break;
        case 2: launch_lists<2>(1, P, level, A, false, st); break;
        case 3: launch_lists<3>(1, P, level, A, false, st); break;
        case 4: launch_lists<4>(1, P, level, A, false, st); break;
        case 5: launch_lists<5>(1, P, level, A, false, st); break;
        case 6: launch_lists<6>(1, P, level, A, false, st); break;
        default: launch_lists<7>(1, P, level, A, false, st); break;
    }
    F3M_HIP(hipStreamSynchronize(st));
}

// Point pairs behind the near list of the last depth and the far lists of every depth (for
// reports and the coverage identity near + far = n^2); computed on first request because it
// re-reads every list.
void compute_far_point_pairs(f3m_plan_s &P) {
    if (P.have_far_point_pairs) return;
    ReleaseScope scope((hipStream_t) nullptr);
    auto pairs = [&](int l, const uint64_t *row_ptr, const uint32_t *cols) {
        return point_pairs(P.lev[l].start.p, P.slev(l).start.p, row_ptr, cols, P.lev[l].nb, nullptr);
    };
    P.near_point_pairs = pairs(P.L, P.lev[P.L].near_ptr.p, P.lev[P.L].near_col.p);
    for (int l = 1; l <= P.L; ++l) {
        f3m_level &lv = P.lev[l];
        lv.small_point_pairs = lv.small_sz > 0 ? pairs(l, lv.small_ptr.p, lv.small_col.p) : 0;
        lv.far_point_pairs = 0;
        if (lv.far_sz == 0) continue;
        if (lv.far_implicit || lv.far_points) {
            DevBuf<uint32_t> cols;
            cols.alloc((size_t)lv.far_sz);
            materialize_far(P, l, cols.p, nullptr);
            lv.far_point_pairs = pairs(l, lv.far_ptr.p, cols.p);
        } else {
            lv.far_point_pairs = pairs(l, lv.far_ptr.p, lv.far_col.p);
        }
    }
    P.have_far_point_pairs = true;
}

// Smoothness criterion with the O(1) bound of Sec. 4.3: a box of edge l has an effective variance
// of at most D l^2 / (8 gamma^2), two boxes D l^2 / (4 gamma^2); adjacent pairs are interpolated
// when that is <= eta_smooth.
bool smooth_rule(double E, int depth, int D, double gamma, double eta_smooth) {
    if (!(eta_smooth > 0.0)) return false;
    const double l = E / std::ldexp(1.0, depth);
    return (double)D * l * l / (4.0 * gamma * gamma) <= eta_smooth;
}

// Bound on the error of a kernel value between points of two adjacent (or farther) boxes of a depth, in 3-D with
// 4 Chebyshev nodes of the second kind per dimension: g^2 l^4 (12 / 4!) (1/4) / 16 for one dimension of one of the two
// points (l the box edge, g = 1 / (2 gamma^2); the fourth derivative of the 1-D Gaussian is at most 12 g^2, the node
// polynomial (t^2 - 1)(t^2 - 1/4) at most 1/4, at t = 0), times 1 + L + ... + L^5 for the six of them, L = 5/3 the
// Lebesgue constant of these nodes: 0.2395 (l^2 / (2 gamma^2))^2, which is 2^-24 at l = 0.0316 gamma.
double near_interp_error(double E, int depth, double gamma) {
    const double l = E / std::ldexp(1.0, depth), q = l * l / (2.0 * gamma * gamma), L = 5.0 / 3.0;
    return q * q * (12.0 / 24.0) * 0.25 / 16.0 * (std::pow(L, 6.0) - 1.0) / (L - 1.0);
}

// The same for points that carry the Gaussian of their own place in the box.  With x = c + u and y = c' + w, D = c' - c,
//   exp(-|x - y|^2 / 2 gamma^2) = e(u) e(w) F(u, w),  e(u) = exp(-u^2 / 2 gamma^2),
//   F(u, w) = exp((u w + u D - w D - D^2 / 2) / gamma^2) per dimension,
// only F is interpolated: its fourth derivative is ((u - D) / gamma^2)^4 F, at most (1.5 l / gamma^2)^4 F for adjacent boxes
// (|u| <= l / 2, |D| <= l), times (l / 2)^4, a quarter (the node polynomial) over 4!: (0.75 l^2 / gamma^2)^4 / 96 for one
// interpolation.  (reach: the largest |D| / l of a near pair, 1 for one point set.  The grids of two sets are shifted against
// each other, and |D| goes up to the far ratio: 1.25 instead of 0.75 with ratio 2, 2^-24 at l = 0.128 gamma.)
// e(u) e(w) F is at most exp(l^2 / 8 gamma^2) between the nodes (F is taken at another w than e, and the node values of F
// go without e: three dimensions of either point, at most exp(6 l^2 / 8 gamma^2)), and the six interpolations
// make it 1 + L + ... + L^5 times that.  2^-24 at l = 0.166 gamma.  That is the worst sum of six worst errors: there the largest
// error of a pair is 5e-9 and the root of the mean square 9e-10, a sixtieth of fp32 rounding; the sum over the near boxes of
// evenly spread points with equal weights is off by 5e-10 of itself.
double near_weighted_error(double E, int depth, double gamma, double reach) {
    const double l = E / std::ldexp(1.0, depth), q = l * l / (gamma * gamma), L = 5.0 / 3.0;
    const double one = 0.5 * (reach + 0.5) * q, e1 = one * one * one * one / 96.0;
    return e1 * std::exp(0.75 * q) * (std::pow(L, 6.0) - 1.0) / (L - 1.0);
}

// Weighted near pairs end at the first depth that allows it where the last one has this many boxes at least.
constexpr int64_t WEIGHTED_MIN_BOXES = 8192;

// The depth that the products end at, and whether the points need only be grouped by its boxes.  L: the last depth of the tree,
// with leaf_boxes boxes and, or not, far and near pairs; near_depth, weighted: the first depths at which the near pairs may be
// interpolated as they are and between weighted points (0: none; weighted comes first); may_group: the points may be grouped by the
// boxes of a depth of at most ROUTE_GROUP_DEPTH.
//
// The tree is too coarse for the plain interpolation of near pairs, but not for that between weighted points: near pairs
// are interpolated at the first depth that allows it -- or, where the last depth has few boxes, at the last one, which
// costs nothing more (a few workgroups per depth).  Product of 1e7 points, lengthscale 0.1, depth 6 of 6: 2.36 -> 1.04 ms;
// four columns of 3e6 points, lengthscale 0.3, depth 5 of 6: 3.36 -> 1.14 ms; of 2e4 points, lengthscale 1, depth 3
// of 3: 84 -> 71 us.
// Also instead of the plain interpolation two or three depths further down, where that makes the depth so coarse that the
// points need only be grouped by its boxes: one pass each way instead of three (n = 1e9, lengthscale 1, depth 3 and not 5: 77.6 -> 60.6 ms
// for plan and product).  What counts is the depth, not how many of its boxes hold points: points on a line or in a
// plane, or a few clusters, have few boxes at deep depths, whose keys go beyond the tables of the grouping.
void product_depths(int L, int64_t leaf_boxes, bool leaf_far, bool leaf_near, bool two_sets, bool may_group, int weighted,
                    int *near_depth, int *near_weighted, bool *grouped) {
    const bool group = may_group && weighted > 0 && weighted <= ROUTE_GROUP_DEPTH;
    if (group && *near_depth > ROUTE_GROUP_DEPTH) *near_depth = 0;
    *near_weighted = 0;
    if (*near_depth == 0 && weighted > 0)
        *near_weighted = group || two_sets ? weighted : leaf_boxes < WEIGHTED_MIN_BOXES && leaf_far ? L : weighted;
    const int last = *near_depth ? *near_depth : *near_weighted ? *near_weighted : L;
    *grouped = may_group && last <= ROUTE_GROUP_DEPTH && (!leaf_near || *near_depth || *near_weighted);
}

// Adaptive far-field rule of Sec. 4.3 on q = l^2 / (2 gamma^2): min(p, 3) nodes per dimension if
// q <= 0.01 (the paper's min(r, 3^D) on a tensor grid), p if q <= 5, 0 (dropped) above.
int adaptive_nodes(double E, int depth, double gamma, int p) {
    const double l = E / std::ldexp(1.0, depth);
    const double q = l * l / (2.0 * gamma * gamma);
    if (q <= 0.01) return p < 3 ? p : 3;
    if (q <= 5.0) return p;
    return 0;
}

void build_plan(f3m_plan_s &P, const float *X, const float *Y, hipStream_t st) {
    switch (P.D) {
        case 1: build_plan_d<1>(P, X, Y, st); break;
        case 2: build_plan_d<2>(P, X, Y, st); break;
        case 3: build_plan_d<3>(P, X, Y, st); break;
        case 4: build_plan_d<4>(P, X, Y, st); break;
        case 5: build_plan_d<5>(P, X, Y, st); break;
        case 6: build_plan_d<6>(P, X, Y, st); break;
        case 7: build_plan_d<7>(P, X, Y, st); break;
        default: fail(F3M_ERR_INVALID_ARG, "D must be in [1,7]");
    }
}

}  // namespace f3m
