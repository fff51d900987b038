// prims.hip -- allocation, error state, prefix scan and LSD radix sort for gfx950.
//
// The radix sort is the voxel build's dominant step (sorting (leaf key,
// point id) pairs) and also orders reception records for deduplication.
// Design: the digit counts of all passes in one read of the keys, then one
// kernel per pass: each block ranks a tile of 2048 or 8192 keys (stable
// in-wave ranks from 8 ballots per key, running digit counts in LDS), and the
// tiles hand their digit prefixes on to each other in tile order.  A sort that fits
// one tile is one kernel.  Tiles and the keys within them keep their order,
// so the whole sort is stable.
#include "internal.h"

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <unordered_map>
#include <vector>

namespace pcrl {

// ---------------------------------------------------------------------------
// error state
// ---------------------------------------------------------------------------

static thread_local std::string g_err;

void set_error(const char* fmt, ...) {
    char buf[1024];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
}

void clear_error() { g_err.clear(); }

const char* get_error() { return g_err.c_str(); }

// ---------------------------------------------------------------------------
// allocation: a caching device allocator
// ---------------------------------------------------------------------------
//
// Freeing through the runtime's stream-ordered pool costs tens of
// microseconds of host time per call, and one build + launch + collect frees
// about eighty buffers.  Freed blocks are kept instead, per device and size
// class, and handed out again:
//   * to an allocation on the stream that freed the block at once (stream
//     order keeps the old and the new user apart);
//   * to an allocation on another stream once an event recorded at the free
//     has completed.
// Size classes are 512 B, then two per power of two: a request above 2^e
// and at most 2^(e+1) bytes gets 1.5 * 2^e or 2^(e+1) (under 50 % slack).  Cached blocks are returned to the runtime when an allocation
// fails, then the allocation is retried once.

size_t size_class(size_t bytes) {
    if (bytes <= 512) return 512;
    int e = 63 - __builtin_clzll((unsigned long long)(bytes - 1));  // 2^e < bytes <= 2^(e+1)
    const size_t q = (size_t)1 << (e - 1);                           // quarter of 2^(e+1)
    return (bytes + q - 1) / q * q;
}

namespace {

struct FreeBlock {
    void* p;
    hipStream_t stream;
    hipEvent_t ev;
};

struct Pool {
    std::mutex mu;
    std::map<std::pair<int, size_t>, std::vector<FreeBlock>> free_;  // (device, class) -> blocks
    std::unordered_map<void*, std::pair<int, size_t>> live;         // block -> (device, class)
    std::map<int, std::vector<hipEvent_t>> events;                   // spare events per device
};

Pool& pool() {
    static Pool* p = new Pool();  // never destroyed: blocks live until the process ends
    return *p;
}

// Return every cached block whose last use has completed to the runtime.
void trim_locked(Pool& P) {
    for (auto& kv : P.free_) {
        auto& v = kv.second;
        for (size_t i = 0; i < v.size();) {
            if (hipEventQuery(v[i].ev) == hipSuccess) {
                (void)hipFree(v[i].p);
                P.events[kv.first.first].push_back(v[i].ev);
                v[i] = v.back();
                v.pop_back();
            } else {
                ++i;
            }
        }
    }
}

}  // namespace

// A caller's allocator (set_allocator) replaces the pool for new blocks;
// every block remembers the allocator that made it, so switching is safe
// while blocks are alive.  The callbacks run with no lock of the library
// held (they may re-enter it, e.g. a framework's collector releasing a
// scene).
namespace {
struct UserAlloc {
    std::mutex mu;
    PcrlAllocator a{};
    bool on = false;
    std::unordered_map<void*, PcrlAllocator> live;
};
UserAlloc& user_alloc() {
    static UserAlloc* u = new UserAlloc();
    return *u;
}
}  // namespace

namespace {
thread_local Arena* t_arena = nullptr;

int arena_alloc(Arena& A, void** p, size_t bytes) {
    const size_t off = (A.top + 255) & ~(size_t)255;
    const size_t want = bytes == 0 ? 1 : bytes;
    if (A.n == Arena::kMaxBlocks) {
        set_error("scratch memory: more than %d blocks in use at once", Arena::kMaxBlocks);
        return PCRL_ENOMEM;
    }
    if (off > A.cap || want > A.cap - off) {
        set_error("scratch memory exhausted: %zu more bytes needed at offset %zu of %zu", want, off, A.cap);
        return PCRL_ENOMEM;
    }
    A.off[A.n] = off;
    A.end[A.n] = off + want;
    A.freed[A.n] = false;
    ++A.n;
    A.top = off + want;
    A.peak = std::max(A.peak, A.top);
    *p = A.base + off;
    return PCRL_OK;
}

bool arena_free(Arena& A, void* p) {
    char* c = static_cast<char*>(p);
    if (c < A.base || c >= A.base + A.cap) return false;
    const size_t off = (size_t)(c - A.base);
    for (int i = A.n; i-- > 0;) {
        if (A.off[i] == off && !A.freed[i]) {
            A.freed[i] = true;
            break;
        }
    }
    while (A.n > 0 && A.freed[A.n - 1]) --A.n;
    A.top = A.n ? A.end[A.n - 1] : 0;
    return true;
}
}  // namespace

ArenaScope::ArenaScope(void* base, size_t bytes) : prev(t_arena) {
    arena.base = static_cast<char*>(base);
    arena.cap = bytes;
    t_arena = &arena;
}

ArenaScope::~ArenaScope() { t_arena = prev; }

int dalloc(void** p, size_t bytes, hipStream_t s) {
    *p = nullptr;
    if (t_arena) return arena_alloc(*t_arena, p, bytes);
    int dev = 0;
    (void)hipGetDevice(&dev);
    const size_t cls = size_class(bytes == 0 ? 1 : bytes);
    UserAlloc& U = user_alloc();
    PcrlAllocator ua{};
    bool use_user = false;
    {
        std::lock_guard<std::mutex> lock(U.mu);
        use_user = U.on;
        ua = U.a;
    }
    if (use_user) {
        void* q = ua.alloc(cls, (pcrl_stream_t)s, ua.ctx);
        if (!q) {
            set_error("device allocation of %zu bytes failed in the caller's allocator", bytes);
            return PCRL_ENOMEM;
        }
        std::lock_guard<std::mutex> lock(U.mu);
        U.live[q] = ua;
        *p = q;
        return PCRL_OK;
    }
    Pool& P = pool();
    std::lock_guard<std::mutex> lock(P.mu);
    auto it = P.free_.find({dev, cls});
    if (it != P.free_.end()) {
        auto& v = it->second;
        for (size_t i = v.size(); i-- > 0;) {
            if (v[i].stream == s || hipEventQuery(v[i].ev) == hipSuccess) {
                *p = v[i].p;
                P.events[dev].push_back(v[i].ev);
                v[i] = v.back();
                v.pop_back();
                P.live[*p] = {dev, cls};
                return PCRL_OK;
            }
        }
    }
    hipError_t e = hipMalloc(p, cls);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        trim_locked(P);
        e = hipMalloc(p, cls);
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        set_error("device allocation of %zu bytes failed: %s", bytes, hipGetErrorString(e));
        *p = nullptr;
        return e == hipErrorOutOfMemory ? PCRL_ENOMEM : PCRL_EHIP;
    }
    P.live[*p] = {dev, cls};
    return PCRL_OK;
}

void dfree(void* p, hipStream_t s) {
    if (!p) return;
    if (t_arena && arena_free(*t_arena, p)) return;
    {
        UserAlloc& U = user_alloc();
        PcrlAllocator ua{};
        bool found = false;
        {
            std::lock_guard<std::mutex> lock(U.mu);
            auto u = U.live.find(p);
            if (u != U.live.end()) {
                ua = u->second;
                U.live.erase(u);
                found = true;
            }
        }
        if (found) {
            ua.free(p, (pcrl_stream_t)s, ua.ctx);
            return;
        }
    }
    Pool& P = pool();
    std::lock_guard<std::mutex> lock(P.mu);
    auto it = P.live.find(p);
    if (it == P.live.end()) return;  // not ours
    const int dev = it->second.first;
    const size_t cls = it->second.second;
    P.live.erase(it);
    hipEvent_t ev = nullptr;
    auto& spare = P.events[dev];
    if (!spare.empty()) {
        ev = spare.back();
        spare.pop_back();
    } else if (hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) {
        (void)hipGetLastError();
        (void)hipStreamSynchronize(s);  // no event: make the block safe for any stream now
        (void)hipFree(p);
        return;
    }
    if (hipEventRecord(ev, s) != hipSuccess) {
        (void)hipGetLastError();
        (void)hipStreamSynchronize(s);
        (void)hipEventRecord(ev, nullptr);
    }
    P.free_[{dev, cls}].push_back(FreeBlock{p, s, ev});
}

int device_cus() {
    static int cus = 0;
    if (!cus) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
            cus = 256;
    }
    return cus;
}

// ---------------------------------------------------------------------------
// fills
// ---------------------------------------------------------------------------

template <typename T>
__global__ void k_fill(T* p, T v, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = v;
}

__global__ void k_iota(uint32_t* p, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = (uint32_t)i;
}

static unsigned grid_for(int64_t n, int block) {
    int64_t g = (n + block - 1) / block;
    int64_t cap = (int64_t)device_cus() * 16;
    if (g > cap) g = cap;
    if (g < 1) g = 1;
    return (unsigned)g;
}

int fill_u32(uint32_t* p, uint32_t v, int64_t n, hipStream_t s) {
    if (n <= 0) return PCRL_OK;
    hipLaunchKernelGGL(k_fill<uint32_t>, dim3(grid_for(n, 256)), dim3(256), 0, s, p, v, n);
    PCRL_TRY_HIP(hipGetLastError());
    return PCRL_OK;
}

int fill_u64(uint64_t* p, uint64_t v, int64_t n, hipStream_t s) {
    if (n <= 0) return PCRL_OK;
    hipLaunchKernelGGL(k_fill<uint64_t>, dim3(grid_for(n, 256)), dim3(256), 0, s, p, v, n);
    PCRL_TRY_HIP(hipGetLastError());
    return PCRL_OK;
}

int iota_u32(uint32_t* p, int64_t n, hipStream_t s) {
    if (n <= 0) return PCRL_OK;
    hipLaunchKernelGGL(k_iota, dim3(grid_for(n, 256)), dim3(256), 0, s, p, n);
    PCRL_TRY_HIP(hipGetLastError());
    return PCRL_OK;
}

// ---------------------------------------------------------------------------
// exclusive scan (reduce -> scan of tile sums -> apply)
// ---------------------------------------------------------------------------

constexpr int SCAN_BLOCK = 256;
constexpr int SCAN_ITEMS = 16;
constexpr int SCAN_TILE = SCAN_BLOCK * SCAN_ITEMS;  // 4096 values per block

__device__ __forceinline__ uint32_t block_excl_scan(uint32_t x, uint32_t* total) {
    __shared__ uint32_t wsum[SCAN_BLOCK / 64];
    const int w = threadIdx.x >> 6;
    uint32_t incl = wave_incl_scan(x);
    if (lane_id() == 63) wsum[w] = incl;
    __syncthreads();
    uint32_t off = 0, tot = 0;
#pragma unroll
    for (int k = 0; k < SCAN_BLOCK / 64; ++k) {
        uint32_t v = wsum[k];
        off += (k < w) ? v : 0u;
        tot += v;
    }
    __syncthreads();
    *total = tot;
    return off + incl - x;
}

__global__ __launch_bounds__(SCAN_BLOCK) void k_scan_reduce(const uint32_t* in, int64_t n, uint32_t* sums) {
    const int64_t tile = (int64_t)blockIdx.x * SCAN_TILE;
    uint32_t acc = 0;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; ++k) {
        int64_t i = tile + (int64_t)k * SCAN_BLOCK + threadIdx.x;
        if (i < n) acc += in[i];
    }
    uint32_t tot;
    (void)block_excl_scan(acc, &tot);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// Each thread owns SCAN_ITEMS consecutive values of the tile, moved as
// 16-byte vectors when VEC (both arrays 16-byte aligned) and the thread's
// values lie inside the array.
template <bool VEC>
__global__ __launch_bounds__(SCAN_BLOCK) void k_scan_apply(const uint32_t* in, uint32_t* out, int64_t n,
                                                           const uint32_t* offs, uint32_t* total) {
    const int64_t tile = (int64_t)blockIdx.x * SCAN_TILE;
    const int64_t first = tile + (int64_t)threadIdx.x * SCAN_ITEMS;
    const bool whole = VEC && first + SCAN_ITEMS <= n;
    uint32_t v[SCAN_ITEMS];
    uint32_t acc = 0;
    if (whole) {
        const uint4* q = reinterpret_cast<const uint4*>(in + first);
#pragma unroll
        for (int k = 0; k < SCAN_ITEMS / 4; ++k) {
            const uint4 u = q[k];
            v[4 * k] = u.x;
            v[4 * k + 1] = u.y;
            v[4 * k + 2] = u.z;
            v[4 * k + 3] = u.w;
        }
    } else {
#pragma unroll
        for (int k = 0; k < SCAN_ITEMS; ++k) {
            int64_t i = first + k;
            v[k] = (i < n) ? in[i] : 0u;
        }
    }
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; ++k) acc += v[k];
    uint32_t tot;
    uint32_t run = block_excl_scan(acc, &tot) + (offs ? offs[blockIdx.x] : 0u);
    uint32_t r[SCAN_ITEMS];
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; ++k) {
        r[k] = run;
        run += v[k];
    }
    if (whole) {
        uint4* q = reinterpret_cast<uint4*>(out + first);
#pragma unroll
        for (int k = 0; k < SCAN_ITEMS / 4; ++k) q[k] = make_uint4(r[4 * k], r[4 * k + 1], r[4 * k + 2], r[4 * k + 3]);
    } else {
#pragma unroll
        for (int k = 0; k < SCAN_ITEMS; ++k) {
            int64_t i = first + k;
            if (i < n) out[i] = r[k];
        }
    }
    if (total && blockIdx.x == gridDim.x - 1 && threadIdx.x == SCAN_BLOCK - 1) *total = run;
}

static void launch_scan_apply(unsigned grid, const uint32_t* in, uint32_t* out, int64_t n, const uint32_t* offs,
                              uint32_t* total, hipStream_t s) {
    const bool vec = (((uintptr_t)in | (uintptr_t)out) & 15u) == 0;
    if (vec) hipLaunchKernelGGL(k_scan_apply<true>, dim3(grid), dim3(SCAN_BLOCK), 0, s, in, out, n, offs, total);
    else hipLaunchKernelGGL(k_scan_apply<false>, dim3(grid), dim3(SCAN_BLOCK), 0, s, in, out, n, offs, total);
}

int scan_u32(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* total, hipStream_t s) {
    if (n <= 0) {
        if (total) PCRL_TRY(fill_u32(total, 0u, 1, s));
        return PCRL_OK;
    }
    const int64_t nb = (n + SCAN_TILE - 1) / SCAN_TILE;
    if (nb == 1) {
        launch_scan_apply(1, in, out, n, nullptr, total, s);
        PCRL_TRY_HIP(hipGetLastError());
        return PCRL_OK;
    }
    uint32_t* sums = nullptr;
    PCRL_TRY(dalloc((void**)&sums, (size_t)nb * sizeof(uint32_t), s));
    hipLaunchKernelGGL(k_scan_reduce, dim3((unsigned)nb), dim3(SCAN_BLOCK), 0, s, in, n, sums);
    int rc = hipGetLastError() == hipSuccess ? PCRL_OK : PCRL_EHIP;
    if (rc == PCRL_OK) rc = scan_u32(sums, sums, nb, nullptr, s);
    if (rc == PCRL_OK) {
        launch_scan_apply((unsigned)nb, in, out, n, sums, total, s);
        if (hipGetLastError() != hipSuccess) rc = PCRL_EHIP;
    }
    dfree(sums, s);
    if (rc == PCRL_EHIP) set_error("scan kernel launch failed");
    return rc;
}

// ---------------------------------------------------------------------------
// LSD radix sort
// ---------------------------------------------------------------------------

// Digits of 4 to 8 bits: a sort of `bits` key bits takes ceil(bits / 8)
// passes, with the digit width spread evenly over them (fewer digits mean
// longer runs per digit in a tile: better-coalesced scatter writes).
constexpr int SORT_BLOCK = 256;
constexpr int SORT_TILE = 4096;                     // keys that one block sorts whole
constexpr int SORT_R = 256;                         // room for the digits of a pass
constexpr int SORT_PASSES = 8;                      // of at most 8 bits, over 64
constexpr int SORT_LOOK = 4;                        // tiles looked back at at a time
constexpr int SORT_HIST_ITEMS = 8;                  // keys of a thread loaded before any is counted

// Shared by the passes of one sort, zero at its start.
struct SortAux {
    uint32_t hist[SORT_PASSES][SORT_R];  // keys per digit of every pass
    uint32_t ticket[SORT_PASSES];        // tiles taken
    uint64_t first;                      // any one key
};

// Tiles' digit counts on their way to prefixes, one word per (tile, digit):
// the low half a count; the high half 2 p + 1 once the tile has published its
// own count in pass p, 2 p + 2 once the count includes all tiles before it.
__device__ __forceinline__ uint64_t state_load(const uint64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void state_store(uint64_t* p, uint32_t flag, uint32_t count) {
    __hip_atomic_store(p, ((uint64_t)flag << 32) | count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Digit counts of every pass in one read of the keys, and the states cleared.
// Neighbouring keys often share digits, so a block counts into `copies`
// copies by lane.
template <typename K>
__global__ __launch_bounds__(SORT_BLOCK) void k_sort_hist(const K* keys, int64_t n, int lo, int db, int passes, int copies,
                                                          SortAux* aux, uint64_t* state, int64_t n_state) {
    extern __shared__ uint32_t cnt[];  // [pass][digit][copy]
    const uint32_t R = 1u << db, cells = (uint32_t)passes * R;
    for (uint32_t c = threadIdx.x; c < cells * (uint32_t)copies; c += SORT_BLOCK) cnt[c] = 0;
    const int64_t stride = (int64_t)gridDim.x * SORT_BLOCK, me = (int64_t)blockIdx.x * SORT_BLOCK + threadIdx.x;
    for (int64_t i = me; i < n_state; i += stride) state[i] = 0;
    if (me == 0) aux->first = (uint64_t)keys[0];
    __syncthreads();
    const uint32_t copy = threadIdx.x & (uint32_t)(copies - 1);
    for (int64_t b = (int64_t)blockIdx.x * SORT_BLOCK * SORT_HIST_ITEMS; b < n; b += stride * SORT_HIST_ITEMS) {
        K kr[SORT_HIST_ITEMS];
#pragma unroll
        for (int k = 0; k < SORT_HIST_ITEMS; ++k) {
            const int64_t i = b + k * SORT_BLOCK + threadIdx.x;
            kr[k] = i < n ? keys[i] : K(0);
        }
#pragma unroll
        for (int k = 0; k < SORT_HIST_ITEMS; ++k) {
            if (b + k * SORT_BLOCK + threadIdx.x >= n) continue;
            for (int p = 0; p < passes; ++p) {
                const uint32_t d = (uint32_t)(kr[k] >> (lo + p * db)) & (R - 1);
                atomicAdd(&cnt[((uint32_t)p * R + d) * (uint32_t)copies + copy], 1u);
            }
        }
    }
    __syncthreads();
    for (uint32_t c = threadIdx.x; c < cells; c += SORT_BLOCK) {
        uint32_t sum = 0;
        for (int k = 0; k < copies; ++k) sum += cnt[c * (uint32_t)copies + k];
        if (sum) atomicAdd(&aux->hist[c >> db][c & (R - 1)], sum);
    }
}

// Whether pass p would move nothing: all keys share its digit.
__device__ __forceinline__ bool sort_trivial(const SortAux* aux, int64_t n, int lo, int db, int p) {
    return aux->hist[p][(uint32_t)(aux->first >> (lo + p * db)) & ((1u << db) - 1u)] == (uint32_t)n;
}

// Ranks of a wave's keys (rows of 64, in order) among the wave's keys with the
// same digit; cnt: the wave's running digit counts, zero at the start.
template <typename K, int ITEMS>
__device__ __forceinline__ void sort_rank(const K (&kr)[ITEMS], int rows, uint32_t valid_n, int shift, int db,
                                          uint32_t* cnt, uint32_t (&pos)[ITEMS]) {
    const uint32_t lane = lane_id();
    const uint64_t lt = lanemask_lt();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        if (k >= rows) break;
        const bool valid = (uint32_t)k * 64u + lane < valid_n;
        const uint32_t digit = (uint32_t)(kr[k] >> shift) & ((1u << db) - 1u);
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            if (b >= db) break;
            const bool bit = (digit >> b) & 1u;
            const uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        const uint32_t rank = __popcll(peers & lt);
        const uint32_t run = cnt[digit];
        pos[k] = run + rank;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // the highest lane of each digit group advances the digit's running count
        if (valid && (peers >> lane) == 1ull) cnt[digit] = run + rank + 1u;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// One pass over one tile: the keys are ranked stably by digit into LDS (digit
// by digit, input order within a digit), then copied out in that order, so
// that consecutive lanes write consecutive addresses of one digit's run.
// Where a digit's run starts follows from the digit counts of the pass and of
// the tiles before this one, which the tiles hand on to each other: a tile
// publishes its counts, adds up those before it (SORT_LOOK at a time, back to
// one that is already a prefix) and publishes its prefix.  Tiles are numbered in
// the order in which their blocks start, and a block publishes before it
// waits, so every wait is for a block that is already running and ends.
// A pass that would move nothing returns at once; where the keys lie (a or b)
// follows from the number of passes before that did move them.
//
// Bound by memory and by the look back: a key is read and written once a pass
// (and read once more for all counts), a tile reads some 8 KB of states past
// the caches.  182 M packed 64-bit keys, 32 bits: 9.08 ms as histogram, scan
// and scatter kernels per pass; 4.87 ms with tiles of 4096 keys looking back
// eight tiles at a time, 4.62 two at a time; 3.78 and 3.94 ms with 8192 and
// 16384 keys, two at a time, 3.68 with 8192 and four (of 2.7 ms at the rate of
// a copy).  100 k pairs, 64 bits: 284 -> 114 us; 5 M keys, 27 bits: 251 -> 204.
template <typename K, bool V, int BLOCK, int ITEMS>
__global__ __launch_bounds__(BLOCK) void k_sort_sweep(K* ka, uint32_t* va, K* kb, uint32_t* vb, int64_t n, int lo,
                                                           int db, int pass, SortAux* aux, uint64_t* state) {
    constexpr int WAVES = BLOCK / 64, TILE = BLOCK * ITEMS;
    __shared__ K skey[TILE];
    __shared__ uint32_t wcnt[WAVES][SORT_R];
    __shared__ uint32_t gbase[SORT_R], wsum[SORT_R / 64], hsum[SORT_R / 64];
    __shared__ uint32_t tile_sh;
    if (sort_trivial(aux, n, lo, db, pass)) return;
    bool in_b = false;
    for (int p = 0; p < pass; ++p) in_b ^= !sort_trivial(aux, n, lo, db, p);
    const K* const kin = in_b ? kb : ka;
    K* const kout = in_b ? ka : kb;
    const uint32_t tid = threadIdx.x, lane = lane_id(), w = tid >> 6, R = 1u << db;
    if (tid == 0) tile_sh = atomicAdd(&aux->ticket[pass], 1u);
    for (uint32_t c = tid; c < (uint32_t)(WAVES * SORT_R); c += BLOCK) wcnt[c / SORT_R][c % SORT_R] = 0;
    __syncthreads();
    const uint32_t tile = tile_sh;
    const int64_t base = (int64_t)tile * TILE, wbase = base + (int64_t)w * (TILE / WAVES);
    const uint32_t tn = (uint32_t)min((int64_t)TILE, n - base);
    const int shift = lo + pass * db;
    // all of the lane's loads first (one memory round trip per tile)
    K kr[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int64_t i = wbase + k * 64 + lane;
        kr[k] = i < n ? kin[i] : K(0);
    }
    uint32_t vr[V ? ITEMS : 1];
    if (V) {
        const uint32_t* const vin = in_b ? vb : va;
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const int64_t i = wbase + k * 64 + lane;
            vr[k] = i < n ? vin[i] : 0u;
        }
    }
    const uint32_t wn = (uint32_t)min(max(n - wbase, (int64_t)0), (int64_t)(TILE / WAVES));
    uint32_t pos[ITEMS];
    sort_rank(kr, ITEMS, wn, shift, db, wcnt[w], pos);
    __syncthreads();
    // the first four waves: thread = digit
    uint32_t run = 0, before[WAVES], incl = 0, hist = 0, hincl = 0;
    uint64_t* const mine = state + (size_t)tile * SORT_R + tid;
    const uint32_t counted = 2u * (uint32_t)pass + 1u, known = counted + 1u;
    if (tid < (uint32_t)SORT_R) {
#pragma unroll
        for (int k = 0; k < WAVES; ++k) {
            before[k] = run;
            run += wcnt[k][tid];
        }
        if (tid < R) {
            state_store(mine, tile ? counted : known, run);
            hist = aux->hist[pass][tid];
        }
        incl = wave_incl_scan(run);
        hincl = wave_incl_scan(hist);
        if (lane == 63) {
            wsum[w] = incl;
            hsum[w] = hincl;
        }
    }
    __syncthreads();
    if (tid < (uint32_t)SORT_R) {
        uint32_t lstart = incl - run, gstart = hincl - hist;
        for (uint32_t k = 0; k < w; ++k) {
            lstart += wsum[k];
            gstart += hsum[k];
        }
#pragma unroll
        for (int k = 0; k < WAVES; ++k) wcnt[k][tid] = before[k] + lstart;
        uint32_t prefix = 0;
        if (tid < R && tile > 0) {
            int64_t q = (int64_t)tile - 1;
            for (bool done = false; !done;) {
                uint64_t s[SORT_LOOK];
#pragma unroll
                for (int k = 0; k < SORT_LOOK; ++k)
                    s[k] = state_load(state + (size_t)max(q - k, (int64_t)0) * SORT_R + tid);
#pragma unroll
                for (int k = 0; k < SORT_LOOK; ++k) {
                    const uint32_t flag = (uint32_t)(s[k] >> 32);
                    if (done || flag < counted) break;  // not there yet: read again from here
                    prefix += (uint32_t)s[k];
                    done = flag == known;
                    --q;
                }
            }
            state_store(mine, known, prefix + run);
        }
        gbase[tid] = gstart + prefix - lstart;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        pos[k] += wcnt[w][(uint32_t)(kr[k] >> shift) & (R - 1u)];
        if ((uint32_t)k * 64u + lane < wn) skey[pos[k]] = kr[k];
    }
    __syncthreads();
    uint32_t g[V ? ITEMS : 1];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const uint32_t j = (uint32_t)k * BLOCK + tid;
        if (j < tn) {
            const K key = skey[j];
            const uint32_t to = gbase[(uint32_t)(key >> shift) & (R - 1u)] + j;
            kout[to] = key;
            if (V) g[k] = to;
        }
    }
    if (V) {
        uint32_t* const vout = in_b ? va : vb;
        uint32_t* const sval = reinterpret_cast<uint32_t*>(skey);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < ITEMS; ++k)
            if ((uint32_t)k * 64u + lane < wn) sval[pos[k]] = vr[k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const uint32_t j = (uint32_t)k * BLOCK + tid;
            if (j < tn) vout[g[k]] = sval[j];
        }
    }
}

// The sorted keys back in a, if the passes left them in b.
template <typename K>
__global__ __launch_bounds__(SORT_BLOCK) void k_sort_home(K* ka, uint32_t* va, const K* kb, const uint32_t* vb, int64_t n,
                                                          int lo, int db, int passes, const SortAux* aux) {
    bool in_b = false;
    for (int p = 0; p < passes; ++p) in_b ^= !sort_trivial(aux, n, lo, db, p);
    if (!in_b) return;
    const int64_t stride = (int64_t)gridDim.x * SORT_BLOCK;
    for (int64_t i = (int64_t)blockIdx.x * SORT_BLOCK + threadIdx.x; i < n; i += stride) {
        ka[i] = kb[i];
        if (va) va[i] = vb[i];
    }
}

// All passes of a sort that fits one tile, in LDS: each wave holds the same
// number of rows of 64 keys.  3000 pairs, 64 bits: 185 us as kernels per pass,
// 54 with four waves, 34 with sixteen (shorter chains).
constexpr int SORT_TILE_BLOCK = 1024;
template <typename K, bool V>
__global__ __launch_bounds__(SORT_TILE_BLOCK) void k_sort_tile(K* keys, uint32_t* vals, uint32_t n, int lo, int db, int passes) {
    constexpr int ITEMS = SORT_TILE / SORT_TILE_BLOCK, WAVES = SORT_TILE_BLOCK / 64;
    __shared__ K skey[SORT_TILE];
    __shared__ uint32_t wsum[SORT_R / 64];
    __shared__ uint32_t wcnt[WAVES][SORT_R];
    const uint32_t tid = threadIdx.x, lane = lane_id(), w = tid >> 6, R = 1u << db;
    const int rows = (int)((n + SORT_TILE_BLOCK - 1) / SORT_TILE_BLOCK);
    const uint32_t wbase = w * (uint32_t)rows * 64u;
    const uint32_t wn = n > wbase ? min(n - wbase, (uint32_t)rows * 64u) : 0u;
    K kr[ITEMS];
    uint32_t vr[V ? ITEMS : 1];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const uint32_t i = (uint32_t)k * 64u + lane;
        kr[k] = i < wn ? keys[wbase + i] : K(0);
        if (V) vr[k] = i < wn ? vals[wbase + i] : 0u;
    }
    for (int p = 0; p < passes; ++p) {
        const int shift = lo + p * db;
        for (uint32_t c = tid; c < (uint32_t)(WAVES * SORT_R); c += SORT_TILE_BLOCK) wcnt[c / SORT_R][c % SORT_R] = 0;
        __syncthreads();
        uint32_t pos[ITEMS];
        sort_rank(kr, rows, wn, shift, db, wcnt[w], pos);
        __syncthreads();
        // the first four waves: thread = digit
        uint32_t run = 0, before[WAVES], incl = 0;
        if (tid < (uint32_t)SORT_R) {
#pragma unroll
            for (int k = 0; k < WAVES; ++k) {
                before[k] = run;
                run += wcnt[k][tid];
            }
            incl = wave_incl_scan(run);
            if (lane == 63) wsum[w] = incl;
        }
        if (__syncthreads_or(run == n)) continue;  // nothing moves
        if (tid < (uint32_t)SORT_R) {
            uint32_t lstart = incl - run;
            for (uint32_t k = 0; k < w; ++k) lstart += wsum[k];
#pragma unroll
            for (int k = 0; k < WAVES; ++k) wcnt[k][tid] = before[k] + lstart;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            if (k >= rows) break;
            pos[k] += wcnt[w][(uint32_t)(kr[k] >> shift) & (R - 1u)];
            if ((uint32_t)k * 64u + lane < wn) skey[pos[k]] = kr[k];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const uint32_t i = (uint32_t)k * 64u + lane;
            if (i < wn) kr[k] = skey[wbase + i];
        }
        __syncthreads();
        if (V) {
            uint32_t* const sval = reinterpret_cast<uint32_t*>(skey);
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                if (k >= rows) break;
                if ((uint32_t)k * 64u + lane < wn) sval[pos[k]] = vr[k];
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                const uint32_t i = (uint32_t)k * 64u + lane;
                if (i < wn) vr[k] = sval[wbase + i];
            }
            __syncthreads();
        }
    }
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const uint32_t i = (uint32_t)k * 64u + lane;
        if (i < wn) {
            keys[wbase + i] = kr[k];
            if (V) vals[wbase + i] = vr[k];
        }
    }
}

template <typename K, int BLOCK, int ITEMS>
static void launch_sweeps(K* ka, uint32_t* va, K* kb, uint32_t* vb, int64_t n, int lo, int db, int passes, SortAux* aux,
                          uint64_t* state, uint32_t n_tiles, hipStream_t s) {
    for (int p = 0; p < passes; ++p) {
        if (va)
            hipLaunchKernelGGL((k_sort_sweep<K, true, BLOCK, ITEMS>), dim3(n_tiles), dim3(BLOCK), 0, s, ka, va, kb, vb, n, lo,
                               db, p, aux, state);
        else
            hipLaunchKernelGGL((k_sort_sweep<K, false, BLOCK, ITEMS>), dim3(n_tiles), dim3(BLOCK), 0, s, ka, va, kb, vb, n, lo,
                               db, p, aux, state);
    }
}

// Keys up to which a tile holds 2048 keys instead of 8192: too few tiles for
// the GPU's 256 CUs otherwise, each a longer chain.  250 k pairs, 32 bits:
// 81 against 88 us; 100 k, 64 bits: 113 against 118; 2 M: 144 (4096) against
// 133.
constexpr int64_t SORT_SMALL = 1 << 18;

// Keys of a tile of a sort of n > SORT_TILE keys.
static int64_t sort_tile_keys(int64_t n) { return 512 * (n <= SORT_SMALL ? 4 : 16); }

size_t radix_sort_scratch_bytes(int64_t n, size_t item) {
    if (n <= SORT_TILE) return 0;
    const int64_t tile = sort_tile_keys(n), n_tiles = (n + tile - 1) / tile;
    return (size_t)n * item + sizeof(SortAux) + (size_t)n_tiles * SORT_R * sizeof(uint64_t);
}

template <typename K>
static int radix_sort_impl(K* keys, uint32_t* vals, int64_t n, int bits, hipStream_t s, int lo_bit = 0) {
    if (n <= 1 || bits <= 0) return PCRL_OK;
    if (n > (int64_t)0xFFFFFFF0ll) {
        set_error("radix sort of %lld items exceeds the 32-bit index range", (long long)n);
        return PCRL_EINVAL;
    }
    const int passes = (bits + 7) / 8;
    const int db = std::max(4, (bits + passes - 1) / passes);  // 4..8
    if (n <= SORT_TILE) {
        if (vals)
            hipLaunchKernelGGL((k_sort_tile<K, true>), dim3(1), dim3(SORT_TILE_BLOCK), 0, s, keys, vals, (uint32_t)n,
                               lo_bit, db, passes);
        else
            hipLaunchKernelGGL((k_sort_tile<K, false>), dim3(1), dim3(SORT_TILE_BLOCK), 0, s, keys, vals, (uint32_t)n,
                               lo_bit, db, passes);
        if (hipGetLastError() == hipSuccess) return PCRL_OK;
        set_error("radix sort kernel failed");
        return PCRL_EHIP;
    }
    const int64_t tile = sort_tile_keys(n);
    const uint32_t n_tiles = (uint32_t)((n + tile - 1) / tile);
    const int64_t n_state = (int64_t)n_tiles * SORT_R;
    K* k2 = nullptr;
    uint32_t* v2 = nullptr;
    SortAux* aux = nullptr;
    uint64_t* state = nullptr;
    int rc = dalloc((void**)&k2, (size_t)n * sizeof(K), s);
    if (rc == PCRL_OK && vals) rc = dalloc((void**)&v2, (size_t)n * sizeof(uint32_t), s);
    if (rc == PCRL_OK) rc = dalloc((void**)&aux, sizeof(SortAux), s);
    if (rc == PCRL_OK) rc = dalloc((void**)&state, (size_t)n_state * sizeof(uint64_t), s);
    if (rc == PCRL_OK) rc = fill_u32((uint32_t*)aux, 0u, sizeof(SortAux) / 4, s);
    if (rc == PCRL_OK) {
        const int copies = passes > 4 ? 4 : 8;
        const size_t lds = ((size_t)passes << db) * copies * sizeof(uint32_t);  // at most 32 KB
        const unsigned grid = (unsigned)std::min<int64_t>(
            (n + SORT_BLOCK * SORT_HIST_ITEMS - 1) / (SORT_BLOCK * SORT_HIST_ITEMS), (int64_t)device_cus() * 4);
        hipLaunchKernelGGL(k_sort_hist<K>, dim3(grid), dim3(SORT_BLOCK), lds, s, keys, n, lo_bit, db, passes, copies, aux,
                           state, n_state);
        if (n <= SORT_SMALL) launch_sweeps<K, 512, 4>(keys, vals, k2, v2, n, lo_bit, db, passes, aux, state, n_tiles, s);
        else launch_sweeps<K, 512, 16>(keys, vals, k2, v2, n, lo_bit, db, passes, aux, state, n_tiles, s);
        hipLaunchKernelGGL(k_sort_home<K>, dim3(grid_for(n, SORT_BLOCK)), dim3(SORT_BLOCK), 0, s, keys, vals, k2, v2, n,
                           lo_bit, db, passes, aux);
        if (hipGetLastError() != hipSuccess) rc = PCRL_EHIP;
    }
    if (rc == PCRL_EHIP) set_error("radix sort kernel failed: %s", hipGetErrorString(hipGetLastError()));
    dfree(k2, s);
    dfree(v2, s);
    dfree(state, s);
    dfree(aux, s);
    return rc;
}

// ---------------------------------------------------------------------------
// bucket order: items grouped by a 16-bit key, any order inside a bucket
// ---------------------------------------------------------------------------

// Counting pass: one atomic per item (neighbouring keys rarely repeat here);
// pos[j] = the item's position among its bucket's items.
__global__ __launch_bounds__(256) void k_bucket_count(const uint16_t* keys, uint32_t n_max, const uint32_t* n_dev,
                                                      uint32_t* cnt, uint32_t* pos) {
    const uint32_t j = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t n = n_dev ? min(*n_dev, n_max) : n_max;
    if (j < n) pos[j] = atomicAdd(&cnt[keys[j]], 1u);
}

// Exclusive scan of the 65536 bucket counts into start[]: 64 workgroups of
// 1024 buckets, each adding the counts of the buckets before its own range
// (read coalesced from cnt, which nothing writes meanwhile).
constexpr int BUCKET_SCAN_BLOCK = 1024;
__global__ __launch_bounds__(BUCKET_SCAN_BLOCK) void k_bucket_scan(const uint32_t* cnt, uint32_t* start) {
    __shared__ uint32_t wsum[BUCKET_SCAN_BLOCK / 64];
    __shared__ uint32_t wprev[BUCKET_SCAN_BLOCK / 64];
    const uint32_t b = blockIdx.x, t = threadIdx.x, w = t >> 6;
    // the buckets before this range as 16-byte vectors (cnt is 16-byte aligned):
    // at most 16 per thread, eight loads in flight at a time
    const uint4* c4 = reinterpret_cast<const uint4*>(cnt);
    uint32_t prev = 0;
#pragma unroll 8
    for (uint32_t i = t; i < (uint32_t)(BUCKET_SCAN_BLOCK / 4) * b; i += BUCKET_SCAN_BLOCK) {
        const uint4 u = c4[i];
        prev += u.x + u.y + u.z + u.w;
    }
    const uint32_t x = cnt[(size_t)BUCKET_SCAN_BLOCK * b + t];
    const uint32_t incl = wave_incl_scan(x);
    const uint32_t pincl = wave_incl_scan(prev);
    if (lane_id() == 63) {
        wsum[w] = incl;
        wprev[w] = pincl;
    }
    __syncthreads();
    uint32_t off = 0, base = 0;
#pragma unroll
    for (int k = 0; k < BUCKET_SCAN_BLOCK / 64; ++k) {
        off += ((uint32_t)k < w) ? wsum[k] : 0u;
        base += wprev[k];
    }
    start[(size_t)BUCKET_SCAN_BLOCK * b + t] = base + off + incl - x;
}

__global__ __launch_bounds__(256) void k_bucket_scatter(const uint16_t* keys, const uint32_t* pos, uint32_t n_max,
                                                        const uint32_t* n_dev, const uint32_t* start,
                                                        uint32_t* order) {
    const uint32_t j = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t n = n_dev ? min(*n_dev, n_max) : n_max;
    if (j < n) order[start[keys[j]] + pos[j]] = j;
}

int bucket_place_u16(const uint16_t* keys, const uint32_t* pos, int64_t n_max, const uint32_t* n_dev,
                     const uint32_t* cnt, uint32_t* order, hipStream_t s) {
    if (n_max <= 0) return PCRL_OK;
    if ((uintptr_t)cnt & 15u) {
        set_error("bucket counts must be 16-byte aligned");
        return PCRL_EINVAL;
    }
    uint32_t* start = nullptr;
    PCRL_TRY(dalloc((void**)&start, (size_t)65536 * sizeof(uint32_t), s));
    hipLaunchKernelGGL(k_bucket_scan, dim3(65536 / BUCKET_SCAN_BLOCK), dim3(BUCKET_SCAN_BLOCK), 0, s, cnt, start);
    hipLaunchKernelGGL(k_bucket_scatter, dim3((unsigned)((n_max + 255) / 256)), dim3(256), 0, s, keys, pos,
                       (uint32_t)n_max, n_dev, (const uint32_t*)start, order);
    const hipError_t e = hipGetLastError();
    dfree(start, s);
    if (e != hipSuccess) {
        set_error("bucket placement kernel failed: %s", hipGetErrorString(e));
        return PCRL_EHIP;
    }
    return PCRL_OK;
}

int bucket_order_u16(const uint16_t* keys, int64_t n_max, const uint32_t* n_dev, uint32_t* order, hipStream_t s) {
    if (n_max <= 0) return PCRL_OK;
    if (n_max > (int64_t)0xFFFFFFF0ll) {
        set_error("bucket order of %lld items exceeds the 32-bit index range", (long long)n_max);
        return PCRL_EINVAL;
    }
    uint32_t *cnt = nullptr, *pos = nullptr;
    PCRL_TRY(dalloc((void**)&cnt, (size_t)65536 * sizeof(uint32_t), s));
    int rc = dalloc((void**)&pos, (size_t)n_max * sizeof(uint32_t), s);
    if (!rc) rc = fill_u32(cnt, 0u, 65536, s);
    if (!rc) {
        hipLaunchKernelGGL(k_bucket_count, dim3((unsigned)((n_max + 255) / 256)), dim3(256), 0, s, keys,
                           (uint32_t)n_max, n_dev, cnt, pos);
        rc = hipGetLastError() == hipSuccess ? PCRL_OK : PCRL_EHIP;
    }
    if (!rc) rc = bucket_place_u16(keys, pos, n_max, n_dev, cnt, order, s);
    if (rc == PCRL_EHIP) set_error("bucket order kernel failed: %s", hipGetErrorString(hipGetLastError()));
    dfree(pos, s);
    dfree(cnt, s);
    return rc;
}

int radix_sort_u64(uint64_t* keys, uint32_t* vals, int64_t n, int bits, hipStream_t s) {
    return radix_sort_impl<uint64_t>(keys, vals, n, bits > 64 ? 64 : bits, s);
}

int radix_sort_u64_bits(uint64_t* keys, uint32_t* vals, int64_t n, int lo_bit, int bits, hipStream_t s) {
    if (lo_bit < 0 || bits < 0 || lo_bit + bits > 64) {
        set_error("radix sort of bits [%d, %d) of 64-bit keys", lo_bit, lo_bit + bits);
        return PCRL_EINVAL;
    }
    return radix_sort_impl<uint64_t>(keys, vals, n, bits, s, lo_bit);
}

int radix_sort_u32(uint32_t* keys, uint32_t* vals, int64_t n, int bits, hipStream_t s) {
    return radix_sort_impl<uint32_t>(keys, vals, n, bits > 32 ? 32 : bits, s);
}

}  // namespace pcrl

extern "C" const char* last_error(void) { return pcrl::get_error(); }

extern "C" const char* pcrl_version(void) { return "pcrl 0.1.0 (gfx950)"; }

namespace pcrl {

// Small device-to-host reads (sizes the host needs before it can go on)
// through a per-thread pinned buffer: the copy goes straight to host memory
// without a pageable staging step.
int read_back(void* host, const void* dev, size_t bytes, hipStream_t s) {
    static thread_local void* pinned = nullptr;
    static thread_local size_t cap = 0;
    if (t_arena) {  // no allocation of any kind: a pageable copy
        if (hipMemcpyAsync(host, dev, bytes, hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess)
            return PCRL_EHIP;
        return PCRL_OK;
    }
    if (bytes > cap) {
        if (pinned) (void)hipHostFree(pinned);
        pinned = nullptr;
        cap = 0;
        const size_t want = std::max<size_t>(bytes, 4096);
        if (hipHostMalloc(&pinned, want, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            pinned = nullptr;
        } else {
            cap = want;
        }
    }
    if (!pinned) {  // no pinned memory: plain pageable copy
        if (hipMemcpyAsync(host, dev, bytes, hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess)
            return PCRL_EHIP;
        return PCRL_OK;
    }
    if (hipMemcpyAsync(pinned, dev, bytes, hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return PCRL_EHIP;
    std::memcpy(host, pinned, bytes);
    return PCRL_OK;
}

}  // namespace pcrl

extern "C" int set_allocator(const PcrlAllocator* a) {
    pcrl::clear_error();
    if (a && (!a->alloc || !a->free)) {
        pcrl::set_error("set_allocator: alloc and free must both be given");
        return PCRL_EINVAL;
    }
    pcrl::UserAlloc& u = pcrl::user_alloc();
    std::lock_guard<std::mutex> lock(u.mu);
    u.on = a != nullptr;
    u.a = a ? *a : PcrlAllocator{};
    return PCRL_OK;
}
