// trace_core.h -- the per-ray bounce body shared by the single-launch and the
// batched kernels (paper, Section 2.2): hierarchical DDA, surfel intersection,
// RX reception, specular reflection and survivor compaction.  Both kernels
// run exactly this code, so a query gives bitwise the same result alone or
// in a batch.
#pragma once

#include "internal.h"

#include <type_traits>

namespace pcrl {

constexpr int TRACE_BLOCK = 256;
constexpr uint32_t NO_HIT = 0xFFFFFFFFu;

// Statistics of the PCRL_LAUNCH_STATS kernel variant.  ST_BYTES is the exact
// algorithmic traffic of the trace kernels: 8 B per top cell and 16 B per block
// record read (between them 12 B per brick word and 4 B per box), 8 B per leaf range, 32 B per
// surfel tested, 36 B of ray state read per segment after the first, 36 B of
// ray state + 16 B of history per reflection, 16 B per record.
enum StatSlot {
    ST_SEGMENTS = 0, ST_DDA, ST_LEAVES, ST_NODES, ST_TESTS, ST_HITS, ST_BYTES, ST_EMPTY_LEAF, ST_UNIFORM,
    ST_WAVE_DDA, ST_WAVE_TESTS, ST_COUNT
};
typedef unsigned long long stat_t;
static_assert(ST_COUNT <= PCRL_NSTATS, "device statistics buffer too small");

struct TraceArgs {
    SceneView v;
    SceneView ov;           // overlay of dynamic points (valid when has_ov; its top grid may lie deeper than v's)
    int32_t has_ov;
    const float* tx;
    const float* rx;
    const float* dirs;      // [n_rays][3] launch directions (the caller's, or the materialised Fibonacci lattice)
    const uint32_t* perm;   // null, or bounce-0 order of the directions
    const uint32_t* order;  // null, or for bounces >= 1: slot i reads the previous bounce's output order[i]
    uint16_t* okeys;        // with order: coherence bucket of each survivor written by a bounce
    uint32_t* opos;         // with order: the survivor's position among its bucket's survivors
    uint32_t* ocnt;         // with order: [K][65536] survivors per bucket, per bounce
    float3 klo, kscale;     // bucket grid: origin and cells per metre (16 per axis over the grid)
    int32_t n_rx;
    int32_t K;
    uint32_t n_rays;
    uint32_t n_total;
    float sig_c;            // sigma * alpha / sqrt(3)
    float4* buf_o[2];       // ray state (o, L); bounce b writes [b & 1], reads [(b & 1) ^ 1]
    float4* buf_d[2];       // (d, last hit id bits)
    uint32_t* buf_g[2];     // global ray id, NO_HIT for an empty slot
    uint32_t* counters;     // [b] live rays entering bounce b, [K+2] records
    float4* hist;
    uint4* rec;
    uint32_t rec_cap;
    int32_t* hit_id;
    float* hit_t;
    unsigned long long* stats;
};

// Rays a wave traces together when n rays are active.  A wave lasts as long as
// its longest ray and tests its lanes' leaves together, so while the waves do
// not fill the GPU fewer rays per wave end sooner; once they do, every extra
// wave costs its own instructions.  The line is at 8,192 waves (8 per SIMD) for
// 32 rays a wave, and at 4,096 for fewer, which leave most lanes idle.  16 k
// rays in a room, four segments: 0.391 ms with 64 rays a wave, 0.352 with 32,
// 0.318 with 16, 0.304 with 8, 0.357 with 4.  766 k rays in a street: 0.338 ms
// with 64, 0.452 with 32; 196 k: 0.525 and 0.401 ms.  80 k rays, a whole launch:
// of 40 TX in an empty room 338 us with 64 and the walk before this one, 362
// with 16, 293 with 32; in a furnished room 440 and 423, in a street 562 and
// 545.  Every wave culls and tests the receivers once, so many receivers move
// the line down: 200 k rays and 1,024 of them take 0.94 ms by the line moved
// so, 1.02 by the line as it is for few.
constexpr uint32_t RPW_MIN = 8, RPW_WAVES = 8192, RPW_RX = 512;
__host__ __device__ __forceinline__ uint32_t rays_per_wave(uint32_t n, uint32_t n_rx) {
    const uint32_t waves = RPW_WAVES * RPW_RX / (RPW_RX + n_rx);
    uint32_t r = 64;
    while (r > RPW_MIN && n / (r / 2) <= (r > 32 ? waves : waves / 2)) r /= 2;
    return r;
}

// Consecutive blocks that go to one XCD before the next one's turn: an eighth
// of the blocks, or in large launches of an eighth's share in up to 8 turns of
// at least PIECE_BLOCKS: neighbouring blocks need much the same lines, but an
// XCD whose eighth of the directions is dear keeps the others waiting.  Street
// canyon, 16 M rays, five segments: 11.0 ms of kernels in one turn, 10.5 with
// turns of 256 blocks, 10.3 with 64, 10.4 with up to 32 turns; its 300 k rays
// with an overlay lose by turns: 0.84 ms in one, 0.86 and 0.90 with turns of
// 64 and 32 blocks.
constexpr uint32_t PIECES = 8, PIECE_BLOCKS = 256;
__host__ __device__ __forceinline__ uint32_t xcd_piece(uint32_t blocks) {
    const uint32_t per = (blocks + 7) / 8, turns = per / PIECE_BLOCKS;
    const uint32_t n = turns < 1 ? 1 : turns > PIECES ? PIECES : turns;
    return per < n ? 1 : (per + n - 1) / n;  // no block at all: pieces of one
}

// The block that workgroup g of a grid works as when `blocks` are needed (a
// number from `blocks` on: none).
__host__ __device__ __forceinline__ uint32_t xcd_turn(uint32_t blocks, uint32_t g) {
    const uint32_t piece = xcd_piece(blocks), k = g >> 3, turn = k / piece;
    return (8u * turn + (g & 7u)) * piece + (k - turn * piece);
}

// Workgroups that hold whole turns of pieces over the XCDs for any number of
// blocks up to `most`.
__host__ __device__ __forceinline__ uint32_t xcd_groups(uint32_t most) {
    return (most + 7) / 8 * 8 + 8 * xcd_piece(most);
}

// Kernels that trace are specialised on the depths TD and OTD of the top grids
// of the base and of the overlay (NO_OV: none).  An overlay shares the base's
// levels and its top grid is as fine or coarser (build.hip).
constexpr int NO_OV = -2;
template <int N>
using Depth = std::integral_constant<int, N>;

static inline int overlay_depth(const TraceArgs& a) { return a.has_ov ? a.ov.depth : NO_OV; }

template <int TD, typename F>
static void with_overlay_depth(int otd, F&& f) {
    static_assert(PCRL_MAX_LEVELS == 4, "depths reach from -1 to 2");
    if (otd == NO_OV) return f(Depth<TD>{}, Depth<NO_OV>{});
    if constexpr (TD == 0)
        if (otd == 1) return f(Depth<0>{}, Depth<1>{});
    if constexpr (TD == 0 || TD == 1)
        if (otd == 2) return f(Depth<TD>{}, Depth<2>{});
    f(Depth<TD>{}, Depth<TD>{});
}

// f(Depth<TD>, Depth<OTD>) for a base and an overlay of these depths.
template <typename F>
static void with_depths(int td, int otd, F&& f) {
    switch (td) {
    case -1: return with_overlay_depth<-1>(otd, f);
    case 0: return with_overlay_depth<0>(otd, f);
    case 1: return with_overlay_depth<1>(otd, f);
    default: return with_overlay_depth<2>(otd, f);
    }
}

// Ping-pong ray buffers of bounce b, chosen by selects: a runtime index into
// the argument struct's arrays would force the whole struct into scratch.
__device__ __forceinline__ float4* ray_o(const TraceArgs& a, int k) { return (k & 1) ? a.buf_o[1] : a.buf_o[0]; }
__device__ __forceinline__ float4* ray_d(const TraceArgs& a, int k) { return (k & 1) ? a.buf_d[1] : a.buf_d[0]; }
__device__ __forceinline__ uint32_t* ray_g(const TraceArgs& a, int k) { return (k & 1) ? a.buf_g[1] : a.buf_g[0]; }

struct Hit {
    uint32_t id;
    uint32_t lab;
    float t;
    float nx, ny, nz;
};

// Per-wave LDS of a trace: the rays of the wave's lanes (read by every lane in
// the cooperative leaf tests) and their running nearest hits.
struct alignas(16) WaveLds {
    float4 o[64];                  // origin, point the ray left (bits; excluded)
    float4 d[64];                  // unit direction, length travelled before the segment
    uint32_t g[64];                // global ray id
    unsigned long long best[64];   // (t bits << 32) | point id: lexicographic min = nearest, ties by id
    uint32_t entry[64];            // entry that set `best` in this trace
    uint32_t delta[64];            // first entry of the lane's leaf minus its first pair
    int32_t mark[64];              // 1 + the lane whose pairs start at this position of the chunk
};

// Occupancy ahead of a ray in a block of 4 x 4 x 4 leaves: bit j of
// ahead[64 o + i] is set when leaf j lies at or after leaf i along every axis
// in direction octant o (bit a: component a negative).  A ray only moves
// ahead, so a block whose mask has no bit there is crossed in one step.
constexpr int AHEAD_WORDS = 8 * 64;

__device__ __forceinline__ void ahead_init(uint64_t* ahead, uint32_t first, uint32_t stride) {
    for (uint32_t i = first; i < (uint32_t)AHEAD_WORDS; i += stride) {
        const uint32_t o = i >> 6, x = i & 3u, y = (i >> 2) & 3u, z = (i >> 4) & 3u;
        const uint32_t nx = (o & 1u) ? 0xFu >> (3u - x) : (0xFu << x) & 0xFu;
        const uint32_t ny = (o & 2u) ? 0xFu >> (3u - y) : (0xFu << y) & 0xFu;
        const uint32_t nz = (o & 4u) ? 0xFu >> (3u - z) : (0xFu << z) & 0xFu;
        const uint32_t sy = (ny & 1u) | ((ny & 2u) << 3) | ((ny & 4u) << 6) | ((ny & 8u) << 9);
        const uint64_t sz = (uint64_t)(nz & 1u) | ((uint64_t)(nz & 2u) << 15) | ((uint64_t)(nz & 4u) << 30) |
                            ((uint64_t)(nz & 8u) << 45);
        ahead[i] = (uint64_t)(nx * sy) * sz;
    }
}

// LDS of a block of `WAVES` waves.
template <int WAVES>
struct alignas(16) TraceLds {
    uint64_t ahead[AHEAD_WORDS];
    WaveLds w[WAVES];
};

// Orders this wave's LDS accesses in the program; the hardware runs the LDS
// instructions of one wave in order, so no wait is needed.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Inclusive wave64 scans on the VALU through DPP row shifts and row
// broadcasts (no LDS round trips).  Every lane of the wave must be active.
// Lanes shifted in from outside a row read 0, the identity of both scans
// (max is used on non-negative values only).
__device__ __forceinline__ uint32_t wave_scan_add_dpp(uint32_t x) {
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, true);   // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, true);   // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, true);   // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, true);   // row_shr:8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);  // row_bcast:15 -> rows 1, 3
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);  // row_bcast:31 -> rows 2, 3
    return x;
}

__device__ __forceinline__ int wave_scan_max_dpp(int x) {
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false));
    return x;
}

__device__ __forceinline__ uint64_t ballot(bool x) { return __builtin_amdgcn_ballot_w64(x); }

__device__ __forceinline__ unsigned long long hit_word(float t, uint32_t id) {
    return ((unsigned long long)__float_as_uint(t) << 32) | id;
}

// Test the leaves (entries r) of all lanes of the wave together: the wave's
// (lane, entry) pairs are dealt out 64 at a time, so every lane tests a
// surfel in every pass whatever the leaves' sizes, and consecutive lanes read
// consecutive entries of a leaf.  Each pair is tested against its owner
// lane's ray and the owner's nearest hit is the minimum of (t, id) over its
// previous hit and all accepted pairs: the same result as testing the
// leaf's entries one after another in the owner's lane.  Called by every
// lane of the wave (r.y 0: no leaf).
//
// A large scene's reflected rays are bound by what their leaves (four entries
// on average) make HBM read: with an entry's two 16-byte halves in one array
// instead of two, a bounce of 12 M rays in a 20M-point street canyon reads 6.4
// GB instead of 8.5, and the launch's kernels take 8.8 ms instead of 9.1.
template <bool STATS>
__device__ __forceinline__ void leaf_tests(const SceneView& v, WaveLds& W, uint2 r, stat_t* cnt) {
    const uint32_t lane = lane_id();
    const uint32_t n = r.y;
    const uint32_t incl = wave_scan_add_dpp(n);
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    const uint32_t excl = incl - n;
    W.delta[lane] = r.x - excl;
    for (uint32_t base = 0; base < total; base += 64) {
        if (STATS && lane == 0) ++cnt[ST_WAVE_TESTS];
        W.mark[lane] = 0;
        wave_sync();
        if (n && excl < base + 64 && incl > base) W.mark[excl > base ? excl - base : 0] = (int)lane + 1;
        wave_sync();
        const uint32_t own = (uint32_t)max(wave_scan_max_dpp(W.mark[lane]), 1) - 1u;  // the pair at `base` has an owner
        // lanes past the last pair repeat it (same loads, no branch)
        const uint32_t pi = min(base + lane, total - 1u);
        const uint32_t k = W.delta[own] + pi;
        const float4 P = v.surf[2 * (size_t)k];
        const float4 N = v.surf[2 * (size_t)k + 1];
        const float4 O = W.o[own];
        const float4 Dd = W.d[own];
        const uint32_t id = __float_as_uint(P.w);
        const float wx = P.x - O.x, wy = P.y - O.y, wz = P.z - O.z;
        // the fused forms are written out: results must not depend on the compiler's choice
        const float den = fmaf(N.z, Dd.z, fmaf(N.x, Dd.x, N.y * Dd.y));
        const float num = fmaf(N.z, wz, fmaf(N.x, wx, N.y * wy));
        const float t = num * __builtin_amdgcn_rcpf(den);
        const float qx = fmaf(t, Dd.x, -wx), qy = fmaf(t, Dd.y, -wy), qz = fmaf(t, Dd.z, -wz);
        const float dist2 = fmaf(qz, qz, fmaf(qx, qx, qy * qy));
        // no short circuit: the id is then loaded with the position
        const bool ok = ((int)(fabsf(den) > 1e-7f) & (int)(t > v.t_eps) & (int)(id != __float_as_uint(O.w)) &
                         (int)(dist2 <= v.rs2)) != 0;
        const unsigned long long cand = hit_word(t, id);
        if (ok) atomicMin(&W.best[own], cand);
        if (ballot(ok)) {
            wave_sync();
            // the pair that holds the minimum names its entry (pairs with equal
            // (t, id) are the same point: same normal and label)
            if (ok && W.best[own] == cand) W.entry[own] = k;
            wave_sync();
        }
    }
}

__device__ __forceinline__ float clampf(float x, float lo, float hi) { return __builtin_amdgcn_fmed3f(x, lo, hi); }
__device__ __forceinline__ float max3(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }
__device__ __forceinline__ float min3(float a, float b, float c) { return fminf(fminf(a, b), c); }

// Index of a top cell: coordinates below 2^22, rows below 2^32.
__device__ __forceinline__ size_t top_index(const SceneView& v, uint32_t x, uint32_t y, uint32_t z) {
    return (uint64_t)(__umul24(z, (uint32_t)v.tdim[1]) + y) * (uint32_t)v.tdim[0] + x;
}

// Walk every active lane's ray (staged in W) through one hierarchy, testing
// the surfels of the leaves it crosses until no nearer hit can follow.  The
// lane's nearest hit so far is W.best; ANY: a lane stops at its first hit
// nearer than that; t_from: the walk starts at this distance.  Called by every
// lane of the wave.
//
// The walk runs in units of leaves, mirrored along every axis on which the
// ray moves backwards, so it only moves towards larger coordinates: a step
// crosses the box from the lane's cell up to hi, te is the distance at which
// it leaves the box and c the next cell.  Cells are whole numbers below 2^22
// held in floats.
//   - TD < 0: the top grid's cells are leaves.  TD >= 0: they are bricks of
//     r^3 leaves (TD = 0), or TD levels of bricks above those.
//   - an empty top cell holds, per direction octant, the edge of the largest
//     empty box of top cells (of 1, 2, 3, 4, 6, 8, 12, 16) from it onwards;
//   - an occupied one holds its brick and the box of its occupied leaves: the
//     ray goes straight to that box, or past the brick when it misses it;
//   - inside, one 16-byte record per 4 x 4 x 4 leaves holds their occupancy:
//     the lane steps leaf by leaf in registers while occupied leaves lie
//     ahead in the block, else to the block's end.
// Every distance is computed from the ray's origin (no accumulation), and a
// surfel is listed in every leaf within the build's rounding pad of its disk,
// so no leaf holding the nearest hit is passed by.
//
// Bound by latency: a wave's chain of steps, each with one to three dependent
// loads, and by instruction issue.  Against a per-step descent through the
// levels with 64-bit divisions (36 then 16 steps a segment, 250 instructions
// each, spilled scalar registers): street canyon, 4 x 4 M rays, 10.2 steps a
// segment, 21.6 -> 11.1 ms of kernels a launch (8.8 with what came later);
// furnished room, 1 M rays, 9.5 steps, 2.25 -> 1.41 ms; 16 k rays in a room
// 0.74 -> 0.30 ms.  The leaves of a step are tested at once: letting lanes wait
// at their leaves until 8, 24 or 48 of them did (fuller tests) took 1.53, 1.66
// and 1.90 ms in the room against 1.49.
template <bool STATS, int TD, bool ANY = false>
__device__ __forceinline__ void walk(const SceneView& v, const uint64_t* ahead, WaveLds& W, bool active, stat_t* cnt,
                                     float t_from = 0.f) {
    const uint32_t lane = lane_id();
    float og[3], dg[3], ig[3], c[3], te = t_from, ts;
    bool neg[3], walking;
    {
        const float4 O = W.o[lane], Dd = W.d[lane];
        const float o[3] = {O.x, O.y, O.z}, d[3] = {Dd.x, Dd.y, Dd.z};
        float t1 = INFINITY, sum = 0.f;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float x = (o[a] - v.org[a]) * v.inv_h, g = d[a] * v.inv_h;
            neg[a] = g < 0.f;
            og[a] = neg[a] ? v.dimf[a] - x : x;
            dg[a] = fabsf(g);
            ig[a] = dg[a] > 1e-30f ? __builtin_amdgcn_rcpf(dg[a]) : 1e30f;
            te = fmaxf(te, -og[a] * ig[a]);
            t1 = fminf(t1, (v.dimf[a] - og[a]) * ig[a]);
            sum += fabsf(x) + dg[a];
        }
        walking = active && te <= t1 && sum < INFINITY;  // false for a non-finite ray
#pragma unroll
        for (int a = 0; a < 3; ++a) c[a] = clampf(floorf(fmaf(te, dg[a], og[a])), 0.f, v.dim1[a]);
        const float t = __uint_as_float((uint32_t)(W.best[lane] >> 32));
        ts = t + (t * 4e-6f + v.stop_pad);
    }
    const uint32_t oct = (neg[0] ? 1u : 0u) | (neg[1] ? 2u : 0u) | (neg[2] ? 4u : 0u);
    const float r = v.rf, r1 = v.r1;
    float plo[3] = {0.f, 0.f, 0.f}, lhi[3] = {0.f, 0.f, 0.f};  // the brick's low corner, its box's far faces (local)
    uint32_t node = 0, cb = 0xFFFFFFFFu, mbase = 0;
    uint64_t mask = 0;
    bool inb = false;
    while (ballot(walking)) {
        if (STATS && lane == 0) ++cnt[ST_WAVE_DDA];
        uint2 rg = make_uint2(0u, 0u);  // the leaf at c: its surfels are tested in this step
        if (walking) {
            if (STATS) ++cnt[ST_DDA];
            float hi[3] = {c[0] + 1.f, c[1] + 1.f, c[2] + 1.f};
            float l[3] = {c[0] - plo[0], c[1] - plo[1], c[2] - plo[2]};
            if (TD < 0 || !inb || max3(l[0], l[1], l[2]) >= r) {
                // the top cell holding c
                float q[3];
                uint32_t u[3];
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    q[a] = TD < 0 ? c[a] : floorf(fmaf(c[a], v.tinv, v.thalf));
                    u[a] = (uint32_t)(neg[a] ? v.tdim1[a] - q[a] : q[a]);
                }
                const uint2 T = v.top[top_index(v, u[0], u[1], u[2])];
                if (STATS) {
                    ++cnt[ST_NODES];
                    cnt[ST_BYTES] += 8;
                }
                inb = false;
                if ((int32_t)T.x < 0) {
                    // empty: the box of (s + 1)^3 top cells onwards is empty
                    const float s = (float)(((T.y >> (4u * oct)) & 15u) + 1u);
#pragma unroll
                    for (int a = 0; a < 3; ++a) hi[a] = (q[a] + s) * v.tspan;
                } else if (TD < 0) {
                    rg = v.rng[T.x];
                    if (STATS) cnt[ST_BYTES] += 8;
                } else {
                    node = T.x;
                    uint32_t box = T.y;
                    bool found = true;
                    if constexpr (TD > 0) {
                        // down the brick levels between the top grid and the leaves' parents
                        float pq[3] = {q[0], q[1], q[2]};
#pragma unroll
                        for (int i = 0; i < TD; ++i) {
                            float qi[3];
                            uint32_t w[3];
#pragma unroll
                            for (int a = 0; a < 3; ++a) {
                                qi[a] = floorf(fmaf(c[a], v.minv[i], v.mhalf[i]));
                                const float m = qi[a] - pq[a] * v.mratio[i];
                                w[a] = (uint32_t)(neg[a] ? v.mratio[i] - 1.f - m : m);
                            }
                            if (found) {
                                const uint32_t rr = (uint32_t)v.mratio[i];
                                const uint32_t loc = w[0] + rr * (w[1] + rr * w[2]);
                                const size_t wi = (size_t)node * v.mnw[i] + (loc >> 6);
                                const uint64_t m = v.mmask[i][wi];
                                if (STATS) {
                                    ++cnt[ST_NODES];
                                    cnt[ST_BYTES] += 12;
                                }
                                found = (m >> (loc & 63u)) & 1ull;
                                node = v.mbase[i][wi] + (uint32_t)__popcll(m & ((uint64_t(1) << (loc & 63u)) - 1ull));
                                if (!found) {
#pragma unroll
                                    for (int a = 0; a < 3; ++a) hi[a] = (qi[a] + 1.f) * v.mspan_f[i];
                                }
                            }
#pragma unroll
                            for (int a = 0; a < 3; ++a) {
                                pq[a] = qi[a];
                                q[a] = qi[a];
                            }
                        }
                        if (found) {
                            box = v.pbox[node];
                            if (STATS) cnt[ST_BYTES] += 4;
                        }
                    }
                    if (found) {
                        // to the box of the brick's occupied leaves, or past the brick
                        float tn = te, tf = INFINITY, b0[3], b1[3];
#pragma unroll
                        for (int a = 0; a < 3; ++a) {
                            plo[a] = q[a] * r;
                            // box in units of v.bunit leaves, mirrored with the ray
                            const float x0 = (float)((box >> (5 * a)) & 31u) * v.bunit;
                            const float x1 = fminf(fmaf((float)((box >> (15 + 5 * a)) & 31u), v.bunit, v.bunit), r);
                            const float m0 = r - x1, m1 = r - x0;
                            const float y0 = neg[a] ? m0 : x0;
                            lhi[a] = neg[a] ? m1 : x1;
                            b0[a] = plo[a] + y0;
                            b1[a] = plo[a] + lhi[a];
                            tn = fmaxf(tn, (b0[a] - og[a]) * ig[a]);
                            tf = fminf(tf, (b1[a] - og[a]) * ig[a]);
                        }
                        if (tn > tf) {
#pragma unroll
                            for (int a = 0; a < 3; ++a) hi[a] = plo[a] + r;
                        } else {
                            inb = true;
                            cb = 0xFFFFFFFFu;
#pragma unroll
                            for (int a = 0; a < 3; ++a) {
                                const float n = floorf(fmaf(tn, dg[a], og[a]));
                                c[a] = fmaxf(c[a], clampf(n, b0[a], b1[a] - 1.f));
                                l[a] = c[a] - plo[a];
                                hi[a] = c[a] + 1.f;
                            }
                        }
                    }
                }
            }
            if (TD >= 0 && inb) {
                if (max3(l[0] - lhi[0], l[1] - lhi[1], l[2] - lhi[2]) >= 0.f) {
                    // past the box on some axis: the rest of the brick ahead is empty
#pragma unroll
                    for (int a = 0; a < 3; ++a) hi[a] = plo[a] + r;
                    inb = false;
                } else {
                    uint32_t u[3];
#pragma unroll
                    for (int a = 0; a < 3; ++a) u[a] = (uint32_t)(neg[a] ? r1 - l[a] : l[a]);
                    const uint32_t B = (uint32_t)v.nblk;
                    const uint32_t b = __umul24(__umul24(u[2] >> 2, B) + (u[1] >> 2), B) + (u[0] >> 2);
                    if (b != cb) {
                        const uint4 k = v.blk[(uint64_t)node * (uint32_t)v.nblk3 + b];
                        cb = b;
                        mask = ((uint64_t)k.y << 32) | k.x;
                        mbase = k.z;
                        if (STATS) {
                            ++cnt[ST_NODES];
                            cnt[ST_BYTES] += 16;
                        }
                    }
                    const uint32_t bit = (u[0] & 3u) | ((u[1] & 3u) << 2) | ((u[2] & 3u) << 4);
                    const uint64_t m = mask & ahead[64u * oct + bit];
                    if (m == 0) {
#pragma unroll
                        for (int a = 0; a < 3; ++a) {
                            const float lo4 = (float)(u[a] & ~3u);
                            hi[a] = plo[a] + (neg[a] ? r - lo4 : fminf(lo4 + 4.f, r));
                        }
                    } else if ((mask >> bit) & 1ull) {
                        rg = v.rng[mbase + (uint32_t)__popcll(mask & ((uint64_t(1) << bit) - 1ull))];
                        if (STATS) cnt[ST_BYTES] += 8;
                    } else if (STATS) {
                        ++cnt[ST_EMPTY_LEAF];
                    }
                }
            }
            if (STATS && rg.y) {
                ++cnt[ST_LEAVES];
                cnt[ST_TESTS] += rg.y;
                cnt[ST_BYTES] += 32ull * rg.y;
            }
            // leave the box [c, hi): the axis (or axes) left first move to hi
            float ta[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) ta[a] = (hi[a] - og[a]) * ig[a];
            te = min3(ta[0], ta[1], ta[2]);
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const float n = clampf(floorf(fmaf(te, dg[a], og[a])), c[a], hi[a] - 1.f);
                c[a] = ta[a] <= te ? hi[a] : n;
            }
            walking = c[0] <= v.dim1[0] && c[1] <= v.dim1[1] && c[2] <= v.dim1[2];
        }
        const uint64_t at_leaf = ballot(rg.y != 0u);
        if (at_leaf) {
            if (STATS) {
                // leaf visits in which every lane at a leaf is in the same one
                const uint32_t lead = (uint32_t)__builtin_amdgcn_readlane((int)rg.x, __ffsll((long long)at_leaf) - 1);
                if (rg.y && ballot(rg.y && rg.x == lead) == at_leaf) ++cnt[ST_UNIFORM];
            }
            leaf_tests<STATS>(v, W, rg, cnt);
            const float t = __uint_as_float((uint32_t)(W.best[lane] >> 32));
            const float before = ts;
            ts = t + (t * 4e-6f + v.stop_pad);
            if (ANY) walking = walking && !(ts < before);
        }
        walking = walking && te <= ts;  // no later cell holds a nearer hit
    }
}

// The range of entries of leaf (x, y, z) (inside the grid; not mirrored), or
// a count of 0 when it is empty.
template <int TD>
__device__ __forceinline__ uint2 leaf_range(const SceneView& v, int x, int y, int z) {
    const float c[3] = {(float)x, (float)y, (float)z};
    float q[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) q[a] = TD < 0 ? c[a] : floorf(fmaf(c[a], v.tinv, v.thalf));
    const uint2 T = v.top[top_index(v, (uint32_t)q[0], (uint32_t)q[1], (uint32_t)q[2])];
    if ((int32_t)T.x < 0) return make_uint2(0u, 0u);
    if constexpr (TD < 0) return v.rng[T.x];
    uint32_t node = T.x;
    if constexpr (TD > 0) {
#pragma unroll
        for (int i = 0; i < TD; ++i) {
            uint32_t w[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const float qi = floorf(fmaf(c[a], v.minv[i], v.mhalf[i]));
                w[a] = (uint32_t)(qi - q[a] * v.mratio[i]);
                q[a] = qi;
            }
            const uint32_t rr = (uint32_t)v.mratio[i];
            const uint32_t loc = w[0] + rr * (w[1] + rr * w[2]);
            const size_t wi = (size_t)node * v.mnw[i] + (loc >> 6);
            const uint64_t m = v.mmask[i][wi];
            if (!((m >> (loc & 63u)) & 1ull)) return make_uint2(0u, 0u);
            node = v.mbase[i][wi] + (uint32_t)__popcll(m & ((uint64_t(1) << (loc & 63u)) - 1ull));
        }
    }
    uint32_t u[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) u[a] = (uint32_t)(c[a] - q[a] * v.rf);
    const uint32_t B = (uint32_t)v.nblk;
    const uint4 k = v.blk[(uint64_t)node * (uint32_t)v.nblk3 + ((u[2] >> 2) * B + (u[1] >> 2)) * B + (u[0] >> 2)];
    const uint64_t mask = ((uint64_t)k.y << 32) | k.x;
    const uint32_t bit = (u[0] & 3u) | ((u[1] & 3u) << 2) | ((u[2] & 3u) << 4);
    if (!((mask >> bit) & 1ull)) return make_uint2(0u, 0u);
    return v.rng[k.z + (uint32_t)__popcll(mask & ((uint64_t(1) << bit) - 1ull))];
}

__device__ __forceinline__ void stage_ray(WaveLds& W, const float o[3], const float d[3], uint32_t last,
                                          float L = 0.f) {
    const uint32_t lane = lane_id();
    W.o[lane] = make_float4(o[0], o[1], o[2], __uint_as_float(last));
    W.d[lane] = make_float4(d[0], d[1], d[2], L);
}

__device__ __forceinline__ void hit_reset(Hit& hit) {
    hit.id = NO_HIT;
    hit.t = INFINITY;
    hit.lab = 0;
    hit.nx = hit.ny = hit.nz = 0.f;
}

// The launch arguments, read again from where they lie (the kernel's argument
// segment, or a batch's query table): what the segment's end needs is loaded
// after the walk instead of being held in scalar registers through it.
typedef const TraceArgs __attribute__((address_space(4)))* ArgsPtr;
// The same pointer on every lane, as scalar registers (arguments in device
// memory are read by scalar loads then; nothing writes them in the kernel).
__device__ __forceinline__ ArgsPtr uniform_args(const TraceArgs* p) {
    const uint64_t x = (uint64_t)p;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32));
    return (ArgsPtr)(((uint64_t)hi << 32) | lo);
}
// The arguments of a kernel whose first parameter is, or starts with, a
// TraceArgs.
__device__ __forceinline__ ArgsPtr kernel_args() { return (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr(); }
__device__ __forceinline__ const TraceArgs& reread(ArgsPtr p) {
    asm volatile("" : "+s"(p));
    return *(const TraceArgs*)p;
}

// One whole segment of every active lane (lanes with `active` false only
// help with the cooperative leaf tests) through the base hierarchy, or the
// overlay when OVL, from the staged ray and the nearest hit so far.  Called by
// every lane of the wave.
template <bool STATS, int TD, bool OVL, bool ANY = false>
__device__ __forceinline__ void trace_segment(ArgsPtr args, const uint64_t* ahead, WaveLds& W, bool active, Hit& hit,
                                              stat_t* cnt) {
    const TraceArgs& a = reread(args);
    const SceneView& v = OVL ? a.ov : a.v;
    const uint32_t lane = lane_id();
    const unsigned long long before = hit_word(hit.t, hit.id);
    W.best[lane] = before;
    wave_sync();
    walk<STATS, TD, ANY>(v, ahead, W, active, cnt);
    const unsigned long long b = W.best[lane];
    if (active && b != before) {
        const float4 N = v.surf[2 * (size_t)W.entry[lane] + 1];
        hit.t = __uint_as_float((uint32_t)(b >> 32));
        hit.id = (uint32_t)b;
        hit.nx = N.x;
        hit.ny = N.y;
        hit.nz = N.z;
        hit.lab = __float_as_uint(N.w);
    }
    wave_sync();
}

// Load slot i of bounce b: the ray, its global id, polyline length and the
// point it left.  Returns false for an empty slot (left by an in-place
// bounce), which an in-place bounce b < K marks empty in its output too.
template <bool FIRST>
__device__ __forceinline__ bool load_ray(const TraceArgs& a, int b, uint32_t i, bool in_place, float o[3], float d[3],
                                         float& L, uint32_t& last, uint32_t& g) {
    L = 0.f;
    last = NO_HIT;
    if (FIRST) {
        const uint32_t ti = i / a.n_rays;
        const uint32_t jl = i - ti * a.n_rays;
        const uint32_t j = a.perm ? a.perm[jl] : jl;  // direction-coherent order
        g = ti * a.n_rays + j;
        o[0] = a.tx[3 * ti];
        o[1] = a.tx[3 * ti + 1];
        o[2] = a.tx[3 * ti + 2];
        d[0] = a.dirs[3 * (size_t)j];
        d[1] = a.dirs[3 * (size_t)j + 1];
        d[2] = a.dirs[3 * (size_t)j + 2];
        const float inv = 1.0f / sqrtf(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
        d[0] *= inv;
        d[1] *= inv;
        d[2] *= inv;
        return true;
    }
    const uint32_t src = a.order ? a.order[i] : i;  // coherence order (never with in-place bounces)
    g = ray_g(a, b + 1)[src];
    if (g == NO_HIT) {
        // the last bounce (b == K) has no output buffers (they may be unallocated)
        if (in_place && b < a.K) ray_g(a, b)[i] = NO_HIT;
        return false;
    }
    const float4 o4 = ray_o(a, b + 1)[src];
    const float4 d4 = ray_d(a, b + 1)[src];
    o[0] = o4.x; o[1] = o4.y; o[2] = o4.z; L = o4.w;
    d[0] = d4.x; d[1] = d4.y; d[2] = d4.z; last = __float_as_uint(d4.w);
    return true;
}

// Octahedral map of a unit direction onto [-1, 1]^2.
__device__ __forceinline__ void octahedral(float x, float y, float z, float& u, float& w) {
    const float s = fabsf(x) + fabsf(y) + fabsf(z);
    u = s > 0.f ? x / s : 0.f;
    w = s > 0.f ? y / s : 0.f;
    if (z < 0.f) {
        const float uu = (1.f - fabsf(w)) * (u >= 0.f ? 1.f : -1.f);
        const float ww = (1.f - fabsf(u)) * (w >= 0.f ? 1.f : -1.f);
        u = uu;
        w = ww;
    }
}

__device__ __forceinline__ uint32_t cell_of(float u, int cells) {
    return (uint32_t)fminf(fmaxf((u * 0.5f + 0.5f) * (float)cells, 0.f), (float)(cells - 1));
}

__device__ __forceinline__ uint32_t spread_bits4x3(uint32_t x) {
    x &= 15u;
    x = (x | (x << 4)) & 0x0C3u;
    x = (x | (x << 2)) & 0x249u;
    return x;
}

// Coherence bucket of a ray: Morton code of its origin on a 16^3 grid over the
// scene (12 bits), then the 4 x 4 octahedral cell of its direction (4 bits).
// Rays that start close together in similar directions walk the same cells.
__device__ __forceinline__ uint32_t ray_bucket(const TraceArgs& a, const float o[3], const float d[3]) {
    const uint32_t cx = (uint32_t)fminf(fmaxf((o[0] - a.klo.x) * a.kscale.x, 0.f), 15.f);
    const uint32_t cy = (uint32_t)fminf(fmaxf((o[1] - a.klo.y) * a.kscale.y, 0.f), 15.f);
    const uint32_t cz = (uint32_t)fminf(fmaxf((o[2] - a.klo.z) * a.kscale.z, 0.f), 15.f);
    float u, w;
    octahedral(d[0], d[1], d[2], u, w);
    const uint32_t m = spread_bits4x3(cx) | (spread_bits4x3(cy) << 1) | (spread_bits4x3(cz) << 2);
    return (m << 4) | (cell_of(u, 4) << 2) | cell_of(w, 4);
}

// Receptions of the wave's segments (lanes with `done`; o, d, L, t: the
// segment and the length before it).  A lane holds one of up to 64 receivers;
// those that no ray of the wave can reach are culled together.  About the axis
// O + s D (one of the rays) every ray lies within e0 + s e1 at s, so a
// receiver it reaches at s in (0, t] lies within alpha + beta s of O + s D,
// alpha = e0 + sig_c max L, beta = e1 + sig_c: its distance from the axis and
// its place along it are bounded.  (The comparisons keep a receiver when
// anything is not a number.)  The others are tested ray by ray.
//
// Bound by instruction issue: some 25 a 64 receivers to cull, 20 each to test.
// Kernels of a launch, with every receiver tested by every wave and culled:
// street canyon, 64 RX, 16 M rays, five segments, 10.4 and 9.1 ms; room, 1,024
// RX, 200 k rays, three segments, 1.08 and 0.94 ms (the first segment 0.29 and
// 0.23; reflected rays lie too far apart for much culling); up to 16 RX
// within 1 %.
template <bool STATS>
__device__ __forceinline__ void receive(const TraceArgs& a, int b, bool done, uint32_t g, const float o[3],
                                        const float d[3], float L, float t, stat_t* cnt) {
    const int n_rx = a.n_rx;
    const uint64_t live = ballot(done);
    if (n_rx == 0 || !live) return;
    const uint32_t lane = lane_id();
    uint32_t* rec_counter = &a.counters[PCRL_CNT_REC(a.K)];
    const int src = (live >> 32) & 1ull ? 32 : __ffsll((long long)live) - 1;
    float O[3], D[3], e0 = 0.f, e1 = 0.f;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        O[k] = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(o[k]), src));
        D[k] = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(d[k]), src));
        const float x = o[k] - O[k], y = d[k] - D[k];
        e0 = fmaf(x, x, e0);
        e1 = fmaf(y, y, e1);
    }
    // non-negative floats order as integers (NaN above all)
    auto largest = [&](float x) {
        const int m = wave_scan_max_dpp(done ? (int)(__float_as_uint(x) & 0x7FFFFFFFu) : 0);
        return __uint_as_float((uint32_t)__builtin_amdgcn_readlane(m, 63));
    };
    const float alpha = 1.0001f * (sqrtf(largest(e0)) + a.sig_c * largest(L));
    const float beta = 1.0001f * (sqrtf(largest(e1)) + a.sig_c);
    const float far = largest(t), inv = 1.0f / (1.0f - beta);
    const bool cull = beta < 0.99f;
    for (int j0 = 0; j0 < n_rx; j0 += 64) {
        const int j = min(j0 + (int)lane, n_rx - 1);
        const float r0 = a.rx[3 * j], r1 = a.rx[3 * j + 1], r2 = a.rx[3 * j + 2];
        bool in = j0 + (int)lane < n_rx;
        if (cull) {
            const float x = r0 - O[0], y = r1 - O[1], z = r2 - O[2];
            const float along = fmaf(z, D[2], fmaf(y, D[1], x * D[0]));
            const float px = fmaf(-along, D[0], x), py = fmaf(-along, D[1], y), pz = fmaf(-along, D[2], z);
            const float off = alpha + 1e-5f * (fabsf(x) + fabsf(y) + fabsf(z));
            const float reach = fmaf(beta, fminf(far, (along + off) * inv), off);
            in = in && !(along < -off) && !(along > far + fmaf(beta, far, off)) &&
                 !(fmaf(pz, pz, fmaf(py, py, px * px)) > reach * reach);
        }
        uint64_t todo = ballot(in);
        while (todo) {
            const int k = __ffsll((long long)todo) - 1;
            todo &= todo - 1ull;
            const float rx0 = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(r0), k));
            const float rx1 = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(r1), k));
            const float rx2 = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(r2), k));
            const float vx = rx0 - o[0], vy = rx1 - o[1], vz = rx2 - o[2];
            // the fused forms are written out: results must not depend on the compiler's choice
            const float s = fmaf(vz, d[2], fmaf(vx, d[0], vy * d[1]));
            bool got = false;
            if (done && s > 0.f && s <= t) {
                const float cx = fmaf(-d[0], s, vx), cy = fmaf(-d[1], s, vy), cz = fmaf(-d[2], s, vz);
                const float rho = a.sig_c * (L + s);
                got = fmaf(cz, cz, fmaf(cx, cx, cy * cy)) <= rho * rho;
            }
            const uint64_t m = ballot(got);
            if (m) {
                const int leader = __ffsll((long long)m) - 1;
                uint32_t slot = 0;
                if ((int)lane == leader) slot = atomicAdd(rec_counter, (uint32_t)__popcll(m));
                slot = __shfl(slot, leader, 64) + (uint32_t)__popcll(m & lanemask_lt());
                if (STATS && got) cnt[ST_BYTES] += 16;
                if (got && slot < a.rec_cap) {
                    const float lp = L + sqrtf(fmaf(vz, vz, fmaf(vx, vx, vy * vy)));
                    a.rec[slot] = make_uint4(g, (uint32_t)(j0 + k) | ((uint32_t)b << 16), __float_as_uint(lp),
                                             __float_as_uint(L + s));
                }
            }
        }
    }
}

// End of the segments of lanes with `done`: log the hit, test every RX on
// [0, t_hit] (rho grows with the unfolded length), reflect at the hit and
// write the survivor (at its own slot i when `in_place`, else compacted with
// one atomic per wave); an in-place bounce marks a dead slot empty.  Called
// by every lane of the wave (ballots).
template <bool FIRST, bool STATS>
__device__ __forceinline__ void finish_segment(const TraceArgs& a, int b, bool done, bool in_place, uint32_t i,
                                               uint32_t g, float o[3], float d[3], float L, uint32_t last,
                                               const Hit& hit, stat_t cnt[ST_COUNT]) {
    const uint32_t lane = lane_id();
    const uint64_t lt = lanemask_lt();
    if (done) {
        if (STATS) {
            ++cnt[ST_SEGMENTS];
            if (hit.id != NO_HIT) ++cnt[ST_HITS];
            if (!FIRST) cnt[ST_BYTES] += 36;
        }
        if (a.hit_id) {
            const size_t idx = (size_t)g * (a.K + 1) + b;
            a.hit_id[idx] = hit.id == NO_HIT ? -1 : (int32_t)hit.id;
            a.hit_t[idx] = hit.id == NO_HIT ? NAN : hit.t;
        }
    }
    receive<STATS>(a, b, done, g, o, d, L, hit.t, cnt);
    // reflect and keep survivors
    const bool surv = done && hit.id != NO_HIT && b < a.K;
    if (surv) {
        const float qx = o[0] + hit.t * d[0], qy = o[1] + hit.t * d[1], qz = o[2] + hit.t * d[2];
        a.hist[(size_t)b * a.n_total + g] = make_float4(qx, qy, qz, __uint_as_float(hit.lab));
        L += hit.t;
        const float dn2 = 2.f * fmaf(d[2], hit.nz, fmaf(d[1], hit.ny, d[0] * hit.nx));
        const float ex = fmaf(-hit.nx, dn2, d[0]), ey = fmaf(-hit.ny, dn2, d[1]), ez = fmaf(-hit.nz, dn2, d[2]);
        const float inv = 1.0f / sqrtf(fmaf(ez, ez, fmaf(ex, ex, ey * ey)));
        d[0] = ex * inv; d[1] = ey * inv; d[2] = ez * inv;
        o[0] = qx; o[1] = qy; o[2] = qz;
        last = hit.id;
    }
    if (b >= a.K) return;
    const uint64_t m = __ballot(surv);
    uint32_t slot = i;
    if (m) {
        const int leader = __ffsll((long long)m) - 1;
        uint32_t first = 0;
        if ((int)lane == leader) first = atomicAdd(&a.counters[b + 1], (uint32_t)__popcll(m));
        first = __shfl(first, leader, 64);
        if (!in_place) slot = first + (uint32_t)__popcll(m & lt);
    }
    if (STATS && surv) cnt[ST_BYTES] += 52;
    if (surv) {
        ray_o(a, b)[slot] = make_float4(o[0], o[1], o[2], L);
        ray_d(a, b)[slot] = make_float4(d[0], d[1], d[2], __uint_as_float(last));
        ray_g(a, b)[slot] = g;
    } else if (done && in_place) {
        ray_g(a, b)[i] = NO_HIT;
    }
    if (a.okeys && m) {  // compacted survivors only (never in place)
        const uint32_t key = surv ? ray_bucket(a, o, d) : 0u;
        const uint32_t pos = wave_bucket_add(a.ocnt + (size_t)b * 65536, key, surv);
        if (surv) {
            a.okeys[slot] = (uint16_t)key;
            a.opos[slot] = pos;
        }
    }
}

// `rpw` (1..64) consecutive slots from `base` of bounce b of one query, one
// per lane, traced in lockstep (base hierarchy, then the overlay).  Slots at
// or past `range` are idle; a slot whose ray id is NO_HIT (left by an
// in-place bounce) is idle too.  Every lane of the wave must call this
// (ballots).
template <bool FIRST, bool STATS, int TD, int OTD>
__device__ __forceinline__ void trace_chunk(ArgsPtr args, const uint64_t* ahead, WaveLds& W, int b, uint32_t base,
                                            uint32_t rpw, uint32_t range, bool in_place, stat_t* cnt) {
    const uint32_t i = base + lane_id();
    bool act;
    {
        float o[3] = {0.f, 0.f, 0.f}, d[3] = {1.f, 0.f, 0.f}, L = 0.f;
        uint32_t last = NO_HIT, g = NO_HIT;
        act = lane_id() < rpw && i < range && load_ray<FIRST>(reread(args), b, i, in_place, o, d, L, last, g);
        stage_ray(W, o, d, last, L);
        W.g[lane_id()] = g;
    }
    Hit hit;
    hit_reset(hit);
    trace_segment<STATS, TD, false>(args, ahead, W, act, hit, cnt);
    // dynamic points: the nearest hit over base and overlay is the nearest
    // hit of the union (ties again by point id); the overlay shares the
    // base's frame and levels
    if constexpr (OTD != NO_OV) trace_segment<STATS, OTD, true>(args, ahead, W, act, hit, cnt);
    const float4 O = W.o[lane_id()], Dd = W.d[lane_id()];
    float o[3] = {O.x, O.y, O.z}, d[3] = {Dd.x, Dd.y, Dd.z};
    finish_segment<FIRST, STATS>(reread(args), b, act, in_place, i, W.g[lane_id()], o, d, Dd.w, __float_as_uint(O.w), hit,
                                 cnt);
}

template <bool STATS>
__device__ __forceinline__ void flush_stats(stat_t cnt[ST_COUNT], unsigned long long* stats) {
    if (!STATS) return;
#pragma unroll
    for (int k = 0; k < ST_COUNT; ++k) {
        const uint64_t sum = wave_sum_u64(cnt[k]);
        if (stats && lane_id() == 0 && sum) atomicAdd(&stats[k], (unsigned long long)sum);
        cnt[k] = 0;
    }
}

// The same for a whole block, whose waves add up in LDS first: a launch of few
// rays per wave has many waves, and one atomic per counter and wave to the same
// few addresses took more than its trace (200 k rays in an empty room, four
// segments: 2.60 ms, 0.78 so).  Called by every thread of the block.
template <bool STATS>
__device__ __forceinline__ void flush_stats_block(stat_t cnt[ST_COUNT], unsigned long long* stats) {
    if constexpr (STATS) {
        __shared__ unsigned long long total[ST_COUNT];
        if (threadIdx.x < (uint32_t)ST_COUNT) total[threadIdx.x] = 0;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < ST_COUNT; ++k) {
            const uint64_t sum = wave_sum_u64(cnt[k]);
            if (lane_id() == 0 && sum) atomicAdd(&total[k], (unsigned long long)sum);
        }
        __syncthreads();
        if (threadIdx.x < (uint32_t)ST_COUNT && stats && total[threadIdx.x])
            atomicAdd(&stats[threadIdx.x], total[threadIdx.x]);
    }
}

// A launch whose segments end at the implicit surface of Eq. 1 instead of the
// surfels (PCRL_LAUNCH_SDF; sdf.hip): runs every segment of every ray.
int sdf_launch_run(PcrlLaunch* L, const TraceArgs& t);

}  // namespace pcrl
