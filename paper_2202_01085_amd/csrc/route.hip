// Permutations of 1e8 .. 2e9 values between the caller's point order and the plan's box order (the
// reindexing vector sigma of Sec. 4.2; grouping of Sec. 4.1) as three streaming passes through LDS; from 2e6 values on as two,
// and as one where a coarse order is enough.
//
// A plain gather b[perm[k]] (or scatter) of a random permutation touches one 128-byte line per 4-byte value
// once the array is larger than the caches: 130 GB of traffic for 4 GB at n = 1e9.  Here a value travels
//     box order k  --pass 1-->  order p1  --pass 2-->  order p2  --pass 3-->  caller's order i = perm[k]
// where, with windows of T = 32768 consecutive caller indices (w = i >> 15, split as w = d1 * B2 + d2):
//   pass 1  deals every tile of T consecutive k into B1 <= 256 buckets by d1 (bucket d1 holds exactly the
//           2^15 B2 values whose destination lies in its B2 windows, so it starts at d1 2^15 B2);
//   pass 2  deals every tile of T consecutive p1 (a tile lies inside one bucket) into the B2 windows of that
//           bucket (window w receives exactly its T values, at w T ...);
//   pass 3  puts the T values of a window in their places inside LDS and writes the window out in one piece.
// (T = 32768 because 128 KB of the 160 KB of LDS then hold one tile of floats.)
// Every pass reads and writes runs that are contiguous in memory (some hundred values per bucket and tile),
// and the places (the position of a value in the LDS copy of its tile, 16 bits per value and pass) depend on
// perm only: they are computed once per plan by route_build, so a pass moves data and does nothing else.
// The gather direction (caller's order -> box order) runs the same three passes backwards with the same tables.
//
// Up to 512 windows (smaller tiles and windows, 2^21 to 14 680 064 = 512 x 28 x 1024 points) pass 1 deals to the windows directly: two
// passes.  From there to 2^24 points a set goes the direct way (at 1.6e7 points three passes take 220 us off a product and add
// 100 to 160 us to the plan).
//
// Where the products need the points by the boxes of a coarse depth only (at most 512 cells), ONE pass does: a tile of T
// consecutive caller indices is dealt to the boxes, in which the points keep the caller's order (route_group_build).
// n = 1e9, 512 boxes: tables 5.8 -> 3.1 ms (with the counts), points 18.7 -> 7.0, right-hand side in 6.2 -> 2.4, result out 6.6 -> 2.2.
#include "plan.h"

namespace f3m {

constexpr int RT_BITS = 15;
constexpr int RT_TILE = 1 << RT_BITS;    // values per tile and per window of the three passes and of the grouping
constexpr int RT_NT = 1024;              // threads of a workgroup: one tile
constexpr int RT_IPT = RT_TILE / RT_NT;  // 32 values per thread
constexpr int RT_NW = RT_NT / 64;        // 16 wavefronts
// The kernels take the values per thread as a template parameter IPT: 32, or for two passes 20 (two workgroups of 80 KB share a
// compute unit, and 10 million points are one round of them), 8 or 28.
constexpr int RT_NB2 = 512;              // digits of two passes and of the grouping

struct RouteCountIn {
    const uint32_t *p;
    __device__ uint64_t operator()(int64_t i) const { return p[i]; }
};
struct RouteCountOut {
    uint32_t *p;
    __device__ void operator()(int64_t i, uint64_t ex, uint64_t) const { p[i] = (uint32_t)ex; }
};

struct RouteLevel {
    int shift;        // digit of a destination index: (i >> shift) & mask
    uint32_t mask;
    int second;       // 0: pass 1 (buckets over all tiles), 1: pass 2 (windows inside the bucket of the tile)
    int s2;           // B2 = 1 << s2 tiles per bucket of pass 1
    int B;            // digits of this pass
    int64_t ntiles;
};

// Tile of this workgroup.  Workgroups go to the 8 dies (each with its own L2) in turn; every die takes a
// contiguous range of tiles, so that the runs which neighbouring tiles write to (or read from) the same bucket
// meet in one L2 as whole lines.  The grid holds a whole number of rounds over the dies (route_grid); a
// workgroup beyond the last tile returns at once.
template <int IPT>
__device__ inline int64_t route_tile(int64_t n) {
    constexpr int TILE = RT_NT * IPT;
    const int64_t ntiles = (n + TILE - 1) / TILE, per_die = (ntiles + 7) >> 3;
    const int64_t t = (int64_t)(blockIdx.x & 7u) * per_die + (int64_t)(blockIdx.x >> 3);
    return t < ntiles ? t : -1;
}
static unsigned route_grid(int64_t ntiles) { return (unsigned)((ntiles + 7) / 8 * 8); }

// Where the runs of a pass begin.  The buckets of pass 1 and the windows of pass 2 have known sizes (bucket d1
// holds exactly the values bound for its B2 windows, a window its T values), so their first positions need no
// counting: bucket d1 starts at d1 B2 T, window w at w T.  A tile reserves the run of each of its digits by an
// atomic add on the cursor of the bucket (pass 1) or window (pass 2); the order of the runs inside a bucket is
// then the order in which the tiles got there, which is as good as any: the places of the later passes are
// computed from the order that came out, and the values end where perm says whatever the order in between.
__global__ __launch_bounds__(256) void route_cursor_init_kernel(uint32_t *__restrict__ cursor, int64_t count,
                                                                uint32_t step) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < count) cursor[i] = (uint32_t)i * step;
}

// One tile of a pass: the place of every value in the LDS copy of the tile (values of a digit together,
// digits ascending, inside a digit in tile order), the destinations moved along to the next order, and the
// tile's tables (first place of each digit; global position of the tile's first value of each digit, minus
// that place).  Tile order = (wavefront, round, lane); ranking against per-wave LDS counters.
template <int IPT, int NB, bool TWO>   // TWO: digit = window of the destination
__global__ __launch_bounds__(RT_NT) void route_rank_kernel(const uint32_t *__restrict__ dest_in, int64_t n, RouteLevel R,
                                                           uint32_t *__restrict__ cursor,
                                                           uint16_t *__restrict__ slot, uint32_t *__restrict__ dest_out,
                                                           uint16_t *__restrict__ off_out,
                                                           uint32_t *__restrict__ dstart_out,
                                                           uint32_t *__restrict__ gofs_out) {
    constexpr int TILE = RT_NT * IPT;
    const int64_t tb = route_tile<IPT>(n);
    if (tb < 0) return;
    constexpr int SKEY = TILE > 2 * RT_NW * NB ? TILE : 2 * RT_NW * NB;
    __shared__ uint32_t wcnt[RT_NW][NB];   // per wave: values of each digit seen so far; later the wave's offset
    __shared__ uint32_t dstart[NB + 1];        // first place of each digit
    __shared__ uint32_t gbase[NB];         // global position of the tile's first value of each digit
    __shared__ __attribute__((aligned(8))) uint32_t skey[SKEY];
    // per wave, while the values are ranked (skey is not in use yet): the lanes that hold each digit in the current round
    uint64_t (*wmask)[NB] = reinterpret_cast<uint64_t (*)[NB]>(skey);
    auto digit_of = [&](uint32_t dest) __attribute__((always_inline)) -> uint32_t {
        return TWO ? dest / (uint32_t)TILE : (dest >> R.shift) & R.mask;
    };
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if (tid < NB) {
#pragma unroll
        for (int k = 0; k < RT_NW; ++k) {
            wcnt[k][tid] = 0;
            wmask[k][tid] = 0ull;
        }
    }
    __syncthreads();
    const uint64_t mybit = 1ull << lane;
    const int64_t tile0 = tb * TILE;
    const int64_t base = tile0 + (int64_t)w * (IPT * 64);
    constexpr int CH = IPT % 8 == 0 ? 8 : 4;
    uint32_t rk[IPT / 2];   // rank within (wave, digit), below 2048: two per register
#pragma unroll
    for (int r = 0; r < IPT / 2; ++r) rk[r] = 0u;
#pragma unroll
    for (int h = 0; h < IPT; h += CH) {   // CH rounds at a time: their loads are in flight together
        uint32_t key[CH];
#pragma unroll
        for (int r = 0; r < CH; ++r) {
            const int64_t i = base + (h + r) * 64 + lane;
            key[r] = i < n ? dest_in[i] : 0u;
        }
#pragma unroll
        for (int r = 0; r < CH; ++r) {
            const int64_t i = base + (h + r) * 64 + lane;
            const bool valid = i < n;
            const uint32_t digit = digit_of(key[r]);
            // The lanes of the round with the same digit find each other through LDS: every lane ORs its own
            // bit into the 64-bit word of its digit (an atomic OR: the result does not depend on the order),
            // reads the word back and counts the bits below its own; the first lane of each group adds the
            // group to the digit's running count and clears the word.  (The wave runs in lockstep and its
            // LDS operations complete in order.)
            if (valid) {
                atomicOr(reinterpret_cast<unsigned long long *>(&wmask[w][digit]), (unsigned long long)mybit);
                __builtin_amdgcn_wave_barrier();
                const uint64_t peers = wmask[w][digit];
                const uint32_t cnt = wcnt[w][digit];
                const uint32_t before =
                    __builtin_amdgcn_mbcnt_hi((uint32_t)(peers >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0u));
                rk[(h + r) / 2] |= (cnt + before) << (16 * ((h + r) & 1));
                __builtin_amdgcn_wave_barrier();
                if (before == 0) {
                    wcnt[w][digit] = cnt + (uint32_t)__popcll(peers);
                    wmask[w][digit] = 0ull;
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    // per digit: the waves' counts become the waves' offsets; the totals go to dstart
    if (tid < NB) {
        uint32_t run = 0;
#pragma unroll
        for (int k = 0; k < RT_NW; ++k) {
            const uint32_t c = wcnt[k][tid];
            wcnt[k][tid] = run;
            run += c;
        }
        dstart[tid] = run;
    }
    __syncthreads();
    if (w == 0) {   // exclusive prefix sum of the totals
        constexpr int PER = NB / 64;
        uint32_t v[PER], s = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) { v[k] = dstart[lane * PER + k]; s += v[k]; }
        uint32_t ex = wave_incl_scan_u32(s) - s;
#pragma unroll
        for (int k = 0; k < PER; ++k) { dstart[lane * PER + k] = ex; ex += v[k]; }
        if (lane == 63) dstart[NB] = ex;
    }
    __syncthreads();
    // the runs of this tile: digit b takes the next dstart[b + 1] - dstart[b] positions of its bucket (pass 1)
    // or of its window inside the bucket of this tile (pass 2)
    if (tid < NB) {
        uint32_t g = 0;
        if (tid < R.B) {
            const uint32_t count = dstart[tid + 1] - dstart[tid];
            const int64_t c = R.second ? ((tb >> R.s2) << R.s2) + tid : (int64_t)tid;
            if (count > 0) g = atomicAdd(&cursor[c], count);
        }
        gbase[tid] = g;
    }
#pragma unroll
    for (int h = 0; h < IPT; h += CH) {
        uint32_t key[CH];   // read again: keeping the first copy would not fit the registers
#pragma unroll
        for (int r = 0; r < CH; ++r) {
            const int64_t i = base + (h + r) * 64 + lane;
            key[r] = i < n ? dest_in[i] : 0u;
        }
#pragma unroll
        for (int r = 0; r < CH; ++r) {
            const int64_t i = base + (h + r) * 64 + lane;
            if (i < n) {
                const uint32_t digit = digit_of(key[r]);
                const uint32_t pos = dstart[digit] + wcnt[w][digit] + ((rk[(h + r) / 2] >> (16 * ((h + r) & 1))) & 0xFFFFu);
                skey[pos] = key[r];
                slot[i] = (uint16_t)pos;
            }
        }
        __builtin_amdgcn_sched_barrier(0);   // keeps the chunks apart: all 32 loads at once would not fit the registers
    }
    __syncthreads();
    const int64_t left = n - tile0;
    const int cntile = (int)(left < TILE ? left : TILE);
#pragma unroll 4
    for (int r = 0; r < IPT; ++r) {
        const int pos = r * RT_NT + tid;
        if (pos < cntile) {
            const uint32_t k = skey[pos];
            const uint32_t digit = digit_of(k);
            const uint32_t g = gbase[digit] + ((uint32_t)pos - dstart[digit]);
            // the last pass needs no more than the place inside the window
            if (off_out) off_out[g] = (uint16_t)(TWO ? k - digit * (uint32_t)TILE : k & (RT_TILE - 1));
            else dest_out[g] = k;
        }
    }
    if (tid <= NB) dstart_out[tb * (NB + 1) + tid] = dstart[tid];
    if (tid < NB) gofs_out[tb * NB + tid] = gbase[tid] - dstart[tid];
}

// ------------------------------------------------------------------------------------
// the passes.  A source or destination with several components per value (the rows of X) is addressed as
// base[(index) * stride + component]; the orders between the passes hold one array per component.
// ------------------------------------------------------------------------------------
// digit whose run of places [ds[b], ds[b+1]) holds place q (ds ascending, ds[NB] = values of the tile)
template <int NB>
__device__ inline int route_digit_of(const uint32_t *ds, uint32_t q) {
    int b = 0;
#pragma unroll
    for (int step = NB / 2; step >= 1; step >>= 1)
        if (ds[b + step] <= q) b += step;
    return b;
}

// pass 1 or 2 forwards: tile of `in` (tile order, in2 added if given) -> runs of `out`; NB: digits of the tables
template <int NB, int IPT>
__global__ __launch_bounds__(RT_NT) void route_deal_kernel(const float *__restrict__ in, const float *__restrict__ in2,
                                                           float *__restrict__ out, const uint16_t *__restrict__ slot,
                                                           const uint32_t *__restrict__ dstart_tab,
                                                           const uint32_t *__restrict__ gofs_tab, int B, int64_t n) {
    constexpr int TILE = RT_NT * IPT;
    const int64_t tb = route_tile<IPT>(n);
    if (tb < 0) return;
    __shared__ float stage[TILE];
    __shared__ uint32_t ds[NB + 1], go[NB];
    const int tid = threadIdx.x;
    const int64_t tile0 = tb * TILE;
    const int64_t left = n - tile0;
    const int cnt = (int)(left < TILE ? left : TILE);
    if (tid <= NB) ds[tid] = dstart_tab[tb * (NB + 1) + tid];
    if (tid < NB) go[tid] = gofs_tab[tb * NB + tid];
    uint16_t sl[IPT];
    float v[IPT];
#pragma unroll
    for (int r = 0; r < IPT; ++r) {
        const int e = r * RT_NT + tid;
        sl[r] = e < cnt ? slot[tile0 + e] : (uint16_t)0;
        v[r] = e < cnt ? in[tile0 + e] : 0.f;
    }
    if (in2) {
#pragma unroll
        for (int r = 0; r < IPT; ++r) {
            const int e = r * RT_NT + tid;
            if (e < cnt) v[r] += in2[tile0 + e];
        }
    }
#pragma unroll
    for (int r = 0; r < IPT; ++r)
        if (r * RT_NT + tid < cnt) stage[sl[r]] = v[r];
    __syncthreads();
    // a thread per place: consecutive places of a run go to consecutive addresses, and all the stores of a
    // thread are independent (a wavefront per run would wait for one short run after the other)
#pragma unroll
    for (int r = 0; r < IPT; ++r) {
        const uint32_t q = (uint32_t)(r * RT_NT + tid);
        if ((int)q < cnt) out[go[route_digit_of<NB>(ds, q)] + q] = stage[q];
    }
}

// pass 2 or 1 backwards: runs of `in` -> tile of `out` (tile order); NC components, one array each on the
// input side (in + c * in_stride); on the output side one array each (ROWS == false) or rows of NC values
template <int NC, bool ROWS, int NB, int IPT>
__global__ __launch_bounds__(RT_NT) void route_collect_kernel(const float *__restrict__ in, int64_t in_stride,
                                                              float *__restrict__ out, int64_t out_stride,
                                                              const uint16_t *__restrict__ slot,
                                                              const uint32_t *__restrict__ dstart_tab,
                                                              const uint32_t *__restrict__ gofs_tab, int B, int64_t n) {
    constexpr int TILE = RT_NT * IPT;
    const int64_t tb = route_tile<IPT>(n);
    if (tb < 0) return;
    __shared__ float stage[TILE];
    __shared__ uint32_t ds[NB + 1], go[NB];
    const int tid = threadIdx.x;
    const int64_t tile0 = tb * TILE;
    const int64_t left = n - tile0;
    const int cnt = (int)(left < TILE ? left : TILE);
    if (tid <= NB) ds[tid] = dstart_tab[tb * (NB + 1) + tid];
    if (tid < NB) go[tid] = gofs_tab[tb * NB + tid];
    uint32_t sl[IPT / 2];   // two places per register
#pragma unroll
    for (int r = 0; r < IPT; r += 2) {
        const int e0 = r * RT_NT + tid, e1 = e0 + RT_NT;
        const uint32_t a = e0 < cnt ? slot[tile0 + e0] : 0u, b = e1 < cnt ? slot[tile0 + e1] : 0u;
        sl[r / 2] = a | (b << 16);
    }
    __syncthreads();
    float v[ROWS ? NC : 1][IPT];
    // a thread per place (see route_deal_kernel): place q comes from go[digit of q] + q in the order before
    constexpr int FLY = IPT % 8 ? 4 : ROWS || IPT % 16 ? 8 : 16;   // loads in flight per thread (the row variant is short of registers)
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const float *src = in + (int64_t)c * in_stride;
#pragma unroll
        for (int h = 0; h < IPT; h += FLY) {
            float t[FLY];
#pragma unroll
            for (int r = 0; r < FLY; ++r) {
                const uint32_t q = (uint32_t)((h + r) * RT_NT + tid);
                t[r] = (int)q < cnt ? src[go[route_digit_of<NB>(ds, q)] + q] : 0.f;
            }
#pragma unroll
            for (int r = 0; r < FLY; ++r) stage[(h + r) * RT_NT + tid] = t[r];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < IPT; ++r) v[ROWS ? c : 0][r] = stage[(sl[r / 2] >> (16 * (r & 1))) & 0xFFFFu];
        if (!ROWS) {
            float *dst = out + (int64_t)c * out_stride;
#pragma unroll
            for (int r = 0; r < IPT; ++r) {
                const int e = r * RT_NT + tid;
                if (e < cnt) dst[tile0 + e] = v[0][r];
            }
        }
        __syncthreads();
    }
    if (ROWS) {
        // a row leaves as one store of NC values
        struct Row { float v[NC]; };
        Row *rows = reinterpret_cast<Row *>(out);
#pragma unroll
        for (int r = 0; r < IPT; ++r) {
            const int e = r * RT_NT + tid;
            if (e < cnt) {
                Row t;
#pragma unroll
                for (int c = 0; c < NC; ++c) t.v[c] = v[ROWS ? c : 0][r];
                rows[tile0 + e] = t;
            }
        }
    }
}

// pass 3 forwards: the values of a window, each to its place inside the window
template <int IPT>
__global__ __launch_bounds__(RT_NT) void route_place_kernel(const float *__restrict__ in, float *__restrict__ out,
                                                            const uint16_t *__restrict__ off, int64_t n) {
    constexpr int TILE = RT_NT * IPT;
    const int64_t tb = route_tile<IPT>(n);
    if (tb < 0) return;
    __shared__ float stage[TILE];
    const int tid = threadIdx.x;
    const int64_t win0 = tb * TILE;
    const int64_t left = n - win0;
    const int cnt = (int)(left < TILE ? left : TILE);
    uint16_t o[IPT];
    float v[IPT];
#pragma unroll
    for (int r = 0; r < IPT; ++r) {
        const int e = r * RT_NT + tid;
        o[r] = e < cnt ? off[win0 + e] : (uint16_t)0;
        v[r] = e < cnt ? in[win0 + e] : 0.f;
    }
#pragma unroll
    for (int r = 0; r < IPT; ++r)
        if (r * RT_NT + tid < cnt) stage[o[r]] = v[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < IPT; ++r) {
        const int e = r * RT_NT + tid;
        if (e < cnt) out[win0 + e] = stage[e];
    }
}

// pass 3 backwards: a window of the caller's array (NC values per row, row-major) -> order p2, one array per
// component.  A thread reads its rows once, whole (the window of a point set is not read again per coordinate),
// and passes them through the LDS copy one coordinate at a time.
template <int NC, int IPT>
__global__ __launch_bounds__(RT_NT) void route_pick_kernel(const float *__restrict__ in, float *__restrict__ out,
                                                           int64_t out_stride, const uint16_t *__restrict__ off,
                                                           int64_t n) {
    constexpr int TILE = RT_NT * IPT;
    const int64_t tb = route_tile<IPT>(n);
    if (tb < 0) return;
    __shared__ float stage[TILE];
    const int tid = threadIdx.x;
    const int64_t win0 = tb * TILE;
    const int64_t left = n - win0;
    const int cnt = (int)(left < TILE ? left : TILE);
    constexpr int FLY = IPT % 8 ? 4 : 8;   // loads in flight per thread
    struct Row { float v[NC]; };
    Row row[IPT];
    const Row *rows = reinterpret_cast<const Row *>(in);
#pragma unroll
    for (int r = 0; r < IPT; ++r) {
        const int e = r * RT_NT + tid;
        row[r] = rows[win0 + (e < cnt ? e : 0)];
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
#pragma unroll
        for (int r = 0; r < IPT; ++r) stage[r * RT_NT + tid] = row[r].v[c];
        __syncthreads();
        float *dst = out + (int64_t)c * out_stride;
#pragma unroll
        for (int h = 0; h < IPT; h += FLY) {
            uint32_t o[FLY];
#pragma unroll
            for (int r = 0; r < FLY; ++r) {
                const int e = (h + r) * RT_NT + tid;
                o[r] = e < cnt ? off[win0 + e] : 0u;
            }
#pragma unroll
            for (int r = 0; r < FLY; ++r) {
                const int e = (h + r) * RT_NT + tid;
                if (e < cnt) dst[win0 + e] = stage[o[r]];
            }
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------------------------------
// One pass: points grouped by the boxes of one depth.  Digit of a point = rank of its box (lut[key >> shift], with
// key >> shift below RG_NB: depth 3 at most); inside a box the
// points keep the caller's order, tile by tile, so the order depends on nothing but the points.
// ------------------------------------------------------------------------------------
constexpr int RG_NB = ROUTE_GROUP_BOXES;
static_assert(RG_NB == RT_NB2, "tables of 512 digits");
static_assert(RG_NB <= RT_NT / 2, "a thread per digit and one more");

// rank of a box by its key; places of unoccupied boxes are not read
__global__ __launch_bounds__(256) void route_lut_kernel(const uint32_t *__restrict__ key, int64_t nb, uint16_t *__restrict__ lut) {
    const int64_t a = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (a < nb) lut[key[a]] = (uint16_t)a;
}

// points of every box in a tile: hist[digit][tile]
__global__ __launch_bounds__(RT_NT) void route_group_count_kernel(const uint32_t *__restrict__ keys, int64_t n, int shift,
                                                                  const uint16_t *__restrict__ lut_tab, int nb,
                                                                  int64_t ntiles, uint32_t *__restrict__ hist) {
    const int64_t tb = route_tile<RT_IPT>(n);
    if (tb < 0) return;
    __shared__ uint32_t cnt[RG_NB];
    __shared__ uint16_t lut[RG_NB];
    const int tid = threadIdx.x;
    if (tid < RG_NB) {
        cnt[tid] = 0;
        lut[tid] = lut_tab[tid];
    }
    __syncthreads();
    const int64_t tile0 = tb * RT_TILE;
#pragma unroll
    for (int h = 0; h < RT_IPT; h += 16) {
        uint32_t key[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int64_t i = tile0 + (h + r) * RT_NT + tid;
            key[r] = i < n ? keys[i] : 0u;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (tile0 + (h + r) * RT_NT + tid < n) atomicAdd(&cnt[lut[key[r] >> shift]], 1u);
    }
    __syncthreads();
    if (tid < nb) hist[(int64_t)tid * ntiles + tb] = cnt[tid];
}

// places of the values of a tile in its LDS copy (as route_rank_kernel finds them), and the tables of the tile; first:
// the scanned counts, i.e. the position of the tile's first value of each digit
__global__ __launch_bounds__(RT_NT) void route_group_rank_kernel(const uint32_t *__restrict__ keys, int64_t n, int shift,
                                                                 const uint16_t *__restrict__ lut_tab, int nb,
                                                                 int64_t ntiles, const uint32_t *__restrict__ first,
                                                                 uint16_t *__restrict__ slot, uint32_t *__restrict__ dstart_out,
                                                                 uint32_t *__restrict__ gofs_out) {
    const int64_t tb = route_tile<RT_IPT>(n);
    if (tb < 0) return;
    __shared__ uint32_t wcnt[RT_NW][RG_NB];   // per wave: values of each digit seen so far; later the wave's offset
    __shared__ uint64_t wmask[RT_NW][RG_NB];  // per wave: the lanes that hold each digit in the current round
    __shared__ uint32_t dstart[RG_NB + 1];
    __shared__ uint16_t lut[RG_NB];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if (tid < RG_NB) {
#pragma unroll
        for (int k = 0; k < RT_NW; ++k) {
            wcnt[k][tid] = 0;
            wmask[k][tid] = 0ull;
        }
        lut[tid] = lut_tab[tid];
    }
    __syncthreads();
    const uint64_t mybit = 1ull << lane;
    const int64_t tile0 = tb * RT_TILE, base = tile0 + (int64_t)w * (RT_IPT * 64);
    uint32_t rk[RT_IPT / 2], dig[RT_IPT / 2];   // rank within (wave, digit), below 2048, and the digit: two per register
#pragma unroll
    for (int r = 0; r < RT_IPT / 2; ++r) rk[r] = dig[r] = 0u;
#pragma unroll
    for (int h = 0; h < RT_IPT; h += 8) {   // eight rounds at a time: their loads are in flight together
        uint32_t key[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int64_t i = base + (h + r) * 64 + lane;
            key[r] = i < n ? keys[i] : 0u;
        }
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const bool valid = base + (h + r) * 64 + lane < n;
            // (see route_rank_kernel: the lanes with the same digit find each other through LDS)
            if (valid) {
                const uint32_t digit = lut[key[r] >> shift];
                dig[(h + r) / 2] |= digit << (16 * ((h + r) & 1));
                atomicOr(reinterpret_cast<unsigned long long *>(&wmask[w][digit]), (unsigned long long)mybit);
                __builtin_amdgcn_wave_barrier();
                const uint64_t peers = wmask[w][digit];
                const uint32_t cnt = wcnt[w][digit];
                const uint32_t before =
                    __builtin_amdgcn_mbcnt_hi((uint32_t)(peers >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0u));
                rk[(h + r) / 2] |= (cnt + before) << (16 * ((h + r) & 1));
                __builtin_amdgcn_wave_barrier();
                if (before == 0) {
                    wcnt[w][digit] = cnt + (uint32_t)__popcll(peers);
                    wmask[w][digit] = 0ull;
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    if (tid < RG_NB) {   // the waves' counts become the waves' offsets; the totals go to dstart
        uint32_t run = 0;
#pragma unroll
        for (int k = 0; k < RT_NW; ++k) {
            const uint32_t c = wcnt[k][tid];
            wcnt[k][tid] = run;
            run += c;
        }
        dstart[tid] = run;
    }
    __syncthreads();
    if (w == 0) {   // exclusive prefix sum of the totals
        constexpr int PER = RG_NB / 64;
        uint32_t v[PER], s = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) { v[k] = dstart[lane * PER + k]; s += v[k]; }
        uint32_t ex = wave_incl_scan_u32(s) - s;
#pragma unroll
        for (int k = 0; k < PER; ++k) { dstart[lane * PER + k] = ex; ex += v[k]; }
        if (lane == 63) dstart[RG_NB] = ex;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RT_IPT; ++r) {
        const int64_t i = base + r * 64 + lane;
        if (i < n) {
            const uint32_t digit = (dig[r / 2] >> (16 * (r & 1))) & 0xFFFFu;
            slot[i] = (uint16_t)(dstart[digit] + wcnt[w][digit] + ((rk[r / 2] >> (16 * (r & 1))) & 0xFFFFu));
        }
    }
    if (tid <= RG_NB) dstart_out[tb * (RG_NB + 1) + tid] = dstart[tid];
    if (tid < RG_NB) gofs_out[tb * RG_NB + tid] = (tid < nb ? first[(int64_t)tid * ntiles + tb] : 0u) - dstart[tid];
}

// rows of three coordinates: tile of `in` (caller's order) -> runs of `out`.  A thread reads its 32 rows once; the places of the
// tile are filled a quarter at a time (96 KB of LDS), and a quarter leaves as runs of whole rows.  The rows and their places are 112 numbers
// a thread, and a workgroup of 1024 threads has 128 registers for each: 21 do not fit, go to scratch memory once and come back in every
// quarter.  n = 1e9: 39 GB moved where rows and places are 26, 7.4 ms.
__global__ __launch_bounds__(RT_NT) void route_group_rows3_kernel(const float *__restrict__ in, float *__restrict__ out,
                                                                  const uint16_t *__restrict__ slot,
                                                                  const uint32_t *__restrict__ dstart_tab,
                                                                  const uint32_t *__restrict__ gofs_tab, int64_t n) {
    const int64_t tb = route_tile<RT_IPT>(n);
    if (tb < 0) return;
    constexpr int QUARTER = RT_TILE / 4;
    __shared__ float stage[QUARTER * 3];
    __shared__ uint32_t ds[RG_NB + 1], go[RG_NB];
    const int tid = threadIdx.x;
    const int64_t tile0 = tb * RT_TILE;
    const int64_t left = n - tile0;
    const int cnt = (int)(left < RT_TILE ? left : RT_TILE);
    if (tid <= RG_NB) ds[tid] = dstart_tab[tb * (RG_NB + 1) + tid];
    if (tid < RG_NB) go[tid] = gofs_tab[tb * RG_NB + tid];
    struct Row { float v[3]; };
    const Row *rin = reinterpret_cast<const Row *>(in);
    Row *rout = reinterpret_cast<Row *>(out);
    Row row[RT_IPT];
    uint32_t sl[RT_IPT / 2];   // two places per register
#pragma unroll
    for (int r = 0; r < RT_IPT; ++r) {
        const int e = r * RT_NT + tid;
        row[r] = rin[tile0 + (e < cnt ? e : 0)];
        const uint32_t p = slot[tile0 + (e < cnt ? e : 0)];
        sl[r / 2] = (r & 1) ? (sl[r / 2] | (p << 16)) : p;
    }
#pragma unroll 1
    for (int h = 0; h < 4; ++h) {
        __syncthreads();   // the places of the last quarter have been read
#pragma unroll
        for (int r = 0; r < RT_IPT; ++r) {
            const uint32_t at = ((sl[r / 2] >> (16 * (r & 1))) & 0xFFFFu) - (uint32_t)(h * QUARTER);
            if (at < (uint32_t)QUARTER && r * RT_NT + tid < cnt) {
                stage[3 * at] = row[r].v[0];
                stage[3 * at + 1] = row[r].v[1];
                stage[3 * at + 2] = row[r].v[2];
            }
        }
        __syncthreads();
#pragma unroll 4
        for (int r = 0; r < QUARTER / RT_NT; ++r) {
            const uint32_t p = (uint32_t)(r * RT_NT + tid), q = (uint32_t)(h * QUARTER) + p;
            if ((int)q < cnt) {
                const Row t = {{stage[3 * p], stage[3 * p + 1], stage[3 * p + 2]}};
                rout[go[route_digit_of<RG_NB>(ds, q)] + q] = t;
            }
        }
    }
}

// ------------------------------------------------------------------------------------
static RouteLevel route_level(const f3m_route &R, int pass) {
    RouteLevel L{};
    L.second = pass == 2;
    L.s2 = R.s2;
    L.ntiles = R.ntiles;
    if (pass == 1) {
        L.shift = RT_BITS + R.s2;
        L.mask = 0xFFu;
        L.B = R.B1;
    } else {
        L.shift = RT_BITS;
        L.mask = (1u << R.s2) - 1u;
        L.B = R.B2;
    }
    return L;
}

// Two passes win over the plain gather and scatter from 2^21 points on: 1e7 points, right-hand side in 179 -> 50 us, result
// out 135 -> 51, points 213 -> 148 for tables of 51 us; 3e6 points, 39 -> 17 and 38 -> 18.  (Three passes at 1e7: 305 tiles of 32768
// on 256 compute units, a second round that is nearly empty.)
bool route_two_passes(int64_t n) { return n >= ((int64_t)1 << 21) && n <= (int64_t)RT_NB2 * RT_NT * 28; }

template <class F>
static void for_ipt(int ipt, F &&f) {
    if (ipt == 8) f(std::integral_constant<int, 8>{});
    else if (ipt == 20) f(std::integral_constant<int, 20>{});
    else f(std::integral_constant<int, 28>{});
}

// Tables of the two or three passes for the permutation perm (n entries, box order -> caller's index).
void route_build(f3m_route &R, const uint32_t *perm, int64_t n, bool two, int64_t *tally, hipStream_t st) {
    R.n = n;
    if (two) {
        R.two = true;
        R.ipt = n <= (int64_t)RT_NB2 * RT_NT * 8 ? 8 : n <= (int64_t)RT_NB2 * RT_NT * 20 ? 20 : 28;
        const int tile = RT_NT * R.ipt;
        R.ntiles = cdiv(n, tile);
        R.B1 = (int)R.ntiles;
        if (R.ntiles > RT_NB2) fail(F3M_ERR_UNSUPPORTED, "too many points for the two-pass permutation");
        R.slot1.alloc((size_t)n, tally);
        R.off3.alloc((size_t)n, tally);
        R.dstart1.alloc((size_t)R.ntiles * (RT_NB2 + 1), tally);
        R.gofs1.alloc((size_t)R.ntiles * RT_NB2, tally);
        DevBuf<uint32_t> cursor;
        cursor.alloc((size_t)R.ntiles);
        route_cursor_init_kernel<<<dim3((unsigned)cdiv(R.ntiles, 256)), dim3(256), 0, st>>>(cursor.p, R.ntiles, (uint32_t)tile);
        RouteLevel L{};
        L.ntiles = R.ntiles;
        L.B = R.B1;
        for_ipt(R.ipt, [&](auto ipt) {
            route_rank_kernel<decltype(ipt)::value, RT_NB2, true><<<dim3(route_grid(R.ntiles)), dim3(RT_NT), 0, st>>>(
                perm, n, L, cursor.p, R.slot1.p, nullptr, R.off3.p, R.dstart1.p, R.gofs1.p);
        });
        F3M_HIP(hipGetLastError());
        return;
    }
    R.ntiles = cdiv(n, RT_TILE);
    int wbits = 0;
    while (((int64_t)1 << wbits) < R.ntiles) ++wbits;
    R.s2 = (wbits + 1) / 2;
    R.B2 = 1 << R.s2;
    R.B1 = (int)cdiv(R.ntiles, R.B2);
    if (R.B1 > 256 || R.B2 > 256) fail(F3M_ERR_UNSUPPORTED, "too many points for the three-pass permutation");
    R.slot1.alloc((size_t)n, tally);
    R.slot2.alloc((size_t)n, tally);
    R.off3.alloc((size_t)n, tally);
    R.dstart1.alloc((size_t)R.ntiles * 257, tally);
    R.dstart2.alloc((size_t)R.ntiles * 257, tally);
    R.gofs1.alloc((size_t)R.ntiles * 256, tally);
    R.gofs2.alloc((size_t)R.ntiles * 256, tally);
    DevBuf<uint32_t> dest1, cursor;
    dest1.alloc((size_t)n);
    const int64_t nwin = (int64_t)R.B1 * R.B2;   // windows, counting the empty ones behind the last value
    cursor.alloc((size_t)nwin);
    const unsigned grid = route_grid(R.ntiles);
    for (int pass = 1; pass <= 2; ++pass) {
        const RouteLevel L = route_level(R, pass);
        const uint32_t *din = pass == 1 ? perm : dest1.p;
        // first positions: bucket d1 at d1 B2 T, window w at w T
        const int64_t ncur = pass == 1 ? R.B1 : nwin;
        route_cursor_init_kernel<<<dim3((unsigned)cdiv(ncur, 256)), dim3(256), 0, st>>>(
            cursor.p, ncur, pass == 1 ? (uint32_t)R.B2 * (uint32_t)RT_TILE : (uint32_t)RT_TILE);
        route_rank_kernel<RT_IPT, 256, false><<<dim3(grid), dim3(RT_NT), 0, st>>>(din, n, L, cursor.p, pass == 1 ? R.slot1.p : R.slot2.p,
                                                             pass == 1 ? dest1.p : nullptr,
                                                             pass == 1 ? nullptr : R.off3.p,
                                                             pass == 1 ? R.dstart1.p : R.dstart2.p,
                                                             pass == 1 ? R.gofs1.p : R.gofs2.p);
        F3M_HIP(hipGetLastError());
    }
}

// Tables of the one pass that groups the points by the nb boxes of a depth (3-D): keys of the points, of depth Lq, in the caller's
// order; the key of a point's box is one of box_keys (ascending).
void route_group_build(f3m_route &R, const uint32_t *keys, int64_t n, int Lq, int depth, const uint32_t *box_keys, int64_t nb,
                       int64_t *tally, hipStream_t st) {
    // The table of ranks is read at the keys of the boxes: few OCCUPIED boxes of a deeper depth do not fit it.
    if (depth < 0 || depth > ROUTE_GROUP_DEPTH || depth > Lq || nb < 1 || nb > RG_NB)
        fail(F3M_ERR_HIP, "internal: too many boxes for the one-pass grouping");
    const int shift = 3 * (Lq - depth);
    R.n = n;
    R.ntiles = cdiv(n, RT_TILE);
    R.grouped = true;
    R.slot1.alloc((size_t)n, tally);
    R.dstart1.alloc((size_t)R.ntiles * (RG_NB + 1), tally);
    R.gofs1.alloc((size_t)R.ntiles * RG_NB, tally);
    DevBuf<uint16_t> lut;
    lut.alloc(RG_NB);
    fill_words((uint32_t *)lut.p, RG_NB / 2, nullptr, 0, 0u, st);
    route_lut_kernel<<<dim3((unsigned)cdiv(nb, 256)), dim3(256), 0, st>>>(box_keys, nb, lut.p);
    DevBuf<uint32_t> hist;
    hist.alloc((size_t)nb * (size_t)R.ntiles);
    const unsigned grid = route_grid(R.ntiles);
    route_group_count_kernel<<<dim3(grid), dim3(RT_NT), 0, st>>>(keys, n, shift, lut.p, (int)nb, R.ntiles, hist.p);
    F3M_HIP(hipGetLastError());
    exclusive_scan(RouteCountIn{hist.p}, nb * R.ntiles, RouteCountOut{hist.p}, nullptr, st);
    route_group_rank_kernel<<<dim3(grid), dim3(RT_NT), 0, st>>>(keys, n, shift, lut.p, (int)nb, R.ntiles, hist.p, R.slot1.p,
                                                               R.dstart1.p, R.gofs1.p);
    F3M_HIP(hipGetLastError());
}

// out[perm[k]] = in[k] (+ in2[k]); tmp_a, tmp_b: n floats each
void route_scatter(const f3m_route &R, const float *in, const float *in2, float *out, float *tmp_a, float *tmp_b,
                   hipStream_t st) {
    const unsigned grid = route_grid(R.ntiles);
    if (R.grouped) {
        if (in2) fail(F3M_ERR_HIP, "internal: grouped points have no exact near field");
        route_collect_kernel<1, false, RG_NB, RT_IPT><<<dim3(grid), dim3(RT_NT), 0, st>>>(in, 0, out, 0, R.slot1.p, R.dstart1.p,
                                                                                 R.gofs1.p, 0, R.n);
        F3M_HIP(hipGetLastError());
        return;
    }
    if (R.two) {
        for_ipt(R.ipt, [&](auto ipt) {
            constexpr int IPT = decltype(ipt)::value;
            route_deal_kernel<RT_NB2, IPT><<<dim3(grid), dim3(RT_NT), 0, st>>>(in, in2, tmp_a, R.slot1.p, R.dstart1.p, R.gofs1.p, R.B1, R.n);
            route_place_kernel<IPT><<<dim3(grid), dim3(RT_NT), 0, st>>>(tmp_a, out, R.off3.p, R.n);
        });
        F3M_HIP(hipGetLastError());
        return;
    }
    route_deal_kernel<256, RT_IPT><<<dim3(grid), dim3(RT_NT), 0, st>>>(in, in2, tmp_a, R.slot1.p, R.dstart1.p, R.gofs1.p, R.B1, R.n);
    route_deal_kernel<256, RT_IPT><<<dim3(grid), dim3(RT_NT), 0, st>>>(tmp_a, nullptr, tmp_b, R.slot2.p, R.dstart2.p, R.gofs2.p, R.B2,
                                                         R.n);
    route_place_kernel<RT_IPT><<<dim3(grid), dim3(RT_NT), 0, st>>>(tmp_b, out, R.off3.p, R.n);
    F3M_HIP(hipGetLastError());
}

// out[k] = in[perm[k]]; tmp_a, tmp_b: n floats each
void route_gather(const f3m_route &R, const float *in, float *out, float *tmp_a, float *tmp_b, hipStream_t st) {
    const unsigned grid = route_grid(R.ntiles);
    if (R.grouped) {
        route_deal_kernel<RG_NB, RT_IPT><<<dim3(grid), dim3(RT_NT), 0, st>>>(in, nullptr, out, R.slot1.p, R.dstart1.p, R.gofs1.p, 0, R.n);
        F3M_HIP(hipGetLastError());
        return;
    }
    if (R.two) {
        for_ipt(R.ipt, [&](auto ipt) {
            constexpr int IPT = decltype(ipt)::value;
            route_pick_kernel<1, IPT><<<dim3(grid), dim3(RT_NT), 0, st>>>(in, tmp_a, 0, R.off3.p, R.n);
            route_collect_kernel<1, false, RT_NB2, IPT><<<dim3(grid), dim3(RT_NT), 0, st>>>(tmp_a, 0, out, 0, R.slot1.p, R.dstart1.p,
                                                                                         R.gofs1.p, R.B1, R.n);
        });
        F3M_HIP(hipGetLastError());
        return;
    }
    route_pick_kernel<1, RT_IPT><<<dim3(grid), dim3(RT_NT), 0, st>>>(in, tmp_a, 0, R.off3.p, R.n);
    route_collect_kernel<1, false, 256, RT_IPT><<<dim3(grid), dim3(RT_NT), 0, st>>>(tmp_a, 0, tmp_b, 0, R.slot2.p, R.dstart2.p,
                                                                      R.gofs2.p, R.B2, R.n);
    route_collect_kernel<1, false, 256, RT_IPT><<<dim3(grid), dim3(RT_NT), 0, st>>>(tmp_b, 0, out, 0, R.slot1.p, R.dstart1.p,
                                                                      R.gofs1.p, R.B1, R.n);
    F3M_HIP(hipGetLastError());
}

// rows of three coordinates: out[k][0..2] = in[perm[k]][0..2].  `out` (3 n floats) first serves as the
// three component arrays of order p2; tmp: 3 n floats.
void route_gather_rows3(const f3m_route &R, const float *in, float *out, float *tmp, hipStream_t st) {
    const unsigned grid = route_grid(R.ntiles);
    if (R.grouped) {
        route_group_rows3_kernel<<<dim3(grid), dim3(RT_NT), 0, st>>>(in, out, R.slot1.p, R.dstart1.p, R.gofs1.p, R.n);
        F3M_HIP(hipGetLastError());
        return;
    }
    if (R.two) {
        for_ipt(R.ipt, [&](auto ipt) {
            constexpr int IPT = decltype(ipt)::value;
            route_pick_kernel<3, IPT><<<dim3(grid), dim3(RT_NT), 0, st>>>(in, tmp, R.n, R.off3.p, R.n);
            route_collect_kernel<3, true, RT_NB2, IPT><<<dim3(grid), dim3(RT_NT), 0, st>>>(tmp, R.n, out, 0, R.slot1.p, R.dstart1.p,
                                                                                        R.gofs1.p, R.B1, R.n);
        });
        F3M_HIP(hipGetLastError());
        return;
    }
    route_pick_kernel<3, RT_IPT><<<dim3(grid), dim3(RT_NT), 0, st>>>(in, out, R.n, R.off3.p, R.n);
    route_collect_kernel<3, false, 256, RT_IPT><<<dim3(grid), dim3(RT_NT), 0, st>>>(out, R.n, tmp, R.n, R.slot2.p, R.dstart2.p,
                                                                      R.gofs2.p, R.B2, R.n);
    route_collect_kernel<3, true, 256, RT_IPT><<<dim3(grid), dim3(RT_NT), 0, st>>>(tmp, R.n, out, 0, R.slot1.p, R.dstart1.p,
                                                                     R.gofs1.p, R.B1, R.n);
    F3M_HIP(hipGetLastError());
}

}  // namespace f3m
