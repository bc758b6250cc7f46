// Device memory of the library comes from a small caching pool: a buffer that is released goes back
// to the pool and the next request of the same size class gets it again.  A plan for n = 1e9 points
// holds ~57 GB in some sixty buffers; building plan after plan (one per time step of a solver, one per
// benchmark step) otherwise pays hipMalloc / hipFree for all of them every time, and on a device
// whose memory was just given back by another process an allocation can take tens of milliseconds
// per gigabyte.  A release waits for the device before the block is put back (as hipFree would), so a
// block is never handed out again while work that uses it is still in flight, on whatever stream.  A plan
// that is built or destroyed waits once for all of its buffers (ReleaseScope): with a wait per buffer and per
// scan, building a plan for 1e5 points was 12 % kernels and 88 % waiting.
#include <map>
#include <mutex>
#include <vector>

#include "common.h"

namespace f3m {
namespace {

struct Pool {
    std::mutex m;
    std::multimap<std::pair<int, size_t>, void *> blocks;   // (device, class size) -> free block
    size_t held = 0;                                          // bytes of the free blocks
    std::vector<void *> words;                                // free arrays of scope_words (one per plan built at once)
    std::vector<std::pair<int, hipEvent_t>> events;           // (device, event)
};
constexpr size_t EVENTS_MAX = 4096;

// the open scope of a thread
struct Scope {
    bool open = false, idle = false;
    hipStream_t st = nullptr;
    std::multimap<std::pair<int, size_t>, void *> blocks;
    void *words = nullptr;
};
thread_local Scope g_scope;

Pool &pool() {
    static Pool *p = new Pool();   // never destroyed: the HIP runtime may be gone at process exit
    return *p;
}
constexpr size_t POOL_CAP = (size_t)96 << 30;   // free blocks beyond this are given back to the device

// size classes: multiples of 1/16 of the power of two below the size (at most 6.25 % over)
size_t class_size(size_t bytes) {
    if (bytes < 4096) return 4096;
    int lg = 63 - __builtin_clzll((unsigned long long)bytes);
    const size_t g = (size_t)1 << (lg - 4);
    return (bytes + g - 1) / g * g;
}

size_t trim_locked(Pool &P, size_t keep) {
    size_t freed = 0;
    // largest blocks first
    while (P.held > keep && !P.blocks.empty()) {
        auto it = P.blocks.begin(), best = it;
        for (; it != P.blocks.end(); ++it)
            if (it->first.second > best->first.second) best = it;
        (void)hipFree(best->second);
        P.held -= best->first.second;
        freed += best->first.second;
        P.blocks.erase(best);
    }
    return freed;
}

void put_locked(Pool &P, int dev, size_t cs, void *p) {
    P.blocks.insert({{dev, cs}, p});
    P.held += cs;
}

// the scope's blocks go to the pool once the work on them has ended
void scope_flush() {
    Scope &S = g_scope;
    if (S.blocks.empty()) return;
    if (hipStreamSynchronize(S.st) != hipSuccess) {
        (void)hipGetLastError();
        (void)hipDeviceSynchronize();
    }
    Pool &P = pool();
    std::lock_guard<std::mutex> lock(P.m);
    for (auto &b : S.blocks) put_locked(P, b.first.first, b.first.second, b.second);
    S.blocks.clear();
    if (P.held > POOL_CAP) trim_locked(P, POOL_CAP);
}

}  // namespace

ReleaseScope::ReleaseScope(hipStream_t st) {
    if (g_scope.open) fail(F3M_ERR_HIP, "internal: a release scope is already open on this thread");
    owner = g_scope.open = true;
    g_scope.idle = false;
    g_scope.st = st;
}

ReleaseScope::ReleaseScope() noexcept {
    if (g_scope.open) return;
    owner = g_scope.open = true;
    g_scope.idle = true;
}

ReleaseScope::~ReleaseScope() {
    if (!owner) return;
    scope_flush();
    if (g_scope.words) {   // kernels that write to it have ended, also where the scope released no block
        if (hipStreamSynchronize(g_scope.st) != hipSuccess) (void)hipGetLastError();
        Pool &P = pool();
        std::lock_guard<std::mutex> lock(P.m);
        P.words.push_back(g_scope.words);
        g_scope.words = nullptr;
    }
    g_scope.open = false;
}

uint64_t *scope_words() {
    Scope &S = g_scope;
    if (!S.open || S.idle) fail(F3M_ERR_HIP, "internal: no release scope of a stream");
    if (!S.words) {
        Pool &P = pool();
        {
            std::lock_guard<std::mutex> lock(P.m);
            if (!P.words.empty()) {
                S.words = P.words.back();
                P.words.pop_back();
            }
        }
        if (!S.words)
            F3M_HIP(hipHostMalloc(&S.words, HOST_WORDS * sizeof(uint64_t), hipHostMallocPortable | hipHostMallocCoherent));
    }
    return (uint64_t *)S.words;
}

hipEvent_t event_get() {
    int dev = 0;
    F3M_HIP(hipGetDevice(&dev));
    {
        Pool &P = pool();
        std::lock_guard<std::mutex> lock(P.m);
        for (size_t k = P.events.size(); k-- > 0;)
            if (P.events[k].first == dev) {
                const hipEvent_t e = P.events[k].second;
                P.events.erase(P.events.begin() + (std::ptrdiff_t)k);
                return e;
            }
    }
    hipEvent_t e = nullptr;
    F3M_HIP(hipEventCreate(&e));
    return e;
}

void event_put(hipEvent_t e, int device) noexcept {
    if (!e) return;
    try {
        Pool &P = pool();
        std::lock_guard<std::mutex> lock(P.m);
        if (P.events.size() < EVENTS_MAX) {
            P.events.emplace_back(device, e);
            return;
        }
    } catch (...) {   // no room for the list
    }
    (void)hipEventDestroy(e);
}

namespace {
__global__ __launch_bounds__(256) void fill_words_kernel(uint32_t *__restrict__ p, int64_t n, uint32_t *__restrict__ q,
                                                         int64_t m, uint32_t value) {
    const int64_t step = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n + m; i += step) {
        if (i < n) p[i] = value;
        else q[i - n] = value;
    }
}
__global__ __launch_bounds__(256) void zero_list_kernel(ZeroList L) {
    for (uint32_t i = threadIdx.x; i < L.n[blockIdx.x]; i += 256) L.p[blockIdx.x][i] = 0.f;
}
}  // namespace

void fill_words(uint32_t *p, int64_t n, uint32_t *q, int64_t m, uint32_t value, hipStream_t st) {
    if (n + m <= 0) return;
    const int64_t blocks = cdiv(n + m, 256 * 8);
    fill_words_kernel<<<dim3((unsigned)(blocks < 8192 ? blocks : 8192)), dim3(256), 0, st>>>(p, n, q, m, value);
    F3M_HIP(hipGetLastError());
}

void ZeroList::add(float *at, size_t words) {
    if (count == MAX) fail(F3M_ERR_HIP, "internal: too many arrays to clear at once");
    p[count] = at;
    n[count++] = (uint32_t)words;
}

void ZeroList::run(hipStream_t st) {
    if (count > 0) zero_list_kernel<<<dim3((unsigned)count), dim3(256), 0, st>>>(*this);
    F3M_HIP(hipGetLastError());
    count = 0;
}

void *pool_alloc(size_t bytes) {
    const size_t cs = class_size(bytes);
    int dev = 0;
    F3M_HIP(hipGetDevice(&dev));
    if (g_scope.open && !g_scope.blocks.empty()) {
        auto it = g_scope.blocks.find({dev, cs});
        if (it != g_scope.blocks.end()) {
            void *p = it->second;
            g_scope.blocks.erase(it);
            return p;
        }
    }
    Pool &P = pool();
    {
        std::lock_guard<std::mutex> lock(P.m);
        auto it = P.blocks.find({dev, cs});
        if (it != P.blocks.end()) {
            void *p = it->second;
            P.blocks.erase(it);
            P.held -= cs;
            return p;
        }
    }
    void *p = nullptr;
    hipError_t e = hipMalloc(&p, cs);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        if (g_scope.open) scope_flush();
        pool_trim();   // give the cached blocks back and try once more
        e = hipMalloc(&p, cs);
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        fail(F3M_ERR_OOM, "hipMalloc of " + std::to_string(cs) + " bytes failed: " + hipGetErrorString(e));
    }
    return p;
}

void pool_free(void *p, size_t bytes) {
    if (!p) return;
    const size_t cs = class_size(bytes);
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        (void)hipFree(p);
        return;
    }
    if (g_scope.open && !g_scope.idle) {
        g_scope.blocks.insert({{dev, cs}, p});
        return;
    }
    if (!g_scope.open) (void)hipDeviceSynchronize();   // nothing in flight may still use the block
    Pool &P = pool();
    std::lock_guard<std::mutex> lock(P.m);
    put_locked(P, dev, cs, p);
    if (P.held > POOL_CAP) trim_locked(P, POOL_CAP);
}

size_t pool_trim() {
    Pool &P = pool();
    std::lock_guard<std::mutex> lock(P.m);
    for (void *w : P.words) (void)hipHostFree(w);
    P.words.clear();
    for (auto &e : P.events) (void)hipEventDestroy(e.second);
    P.events.clear();
    return trim_locked(P, 0);
}

}  // namespace f3m
