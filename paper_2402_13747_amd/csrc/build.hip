// build.hip -- voxelisation of a labeled point cloud (paper, Section 2.1).
//
// The paper keeps a low-resolution voxel grid for traversal and divides each
// voxel by an integer factor into subvoxels that localise the geometry.  Here
// that becomes a hierarchy of 1..4 levels, each level dividing the previous
// one by an integer ratio:
//
//   top grid         dense, over the cells of the leaves' parents (or a coarser
//                    level when that grid would be too large): the node of an
//                    occupied cell with the box of its leaves, or the empty
//                    boxes that start at an empty one, per direction octant
//   blocks           per leaves' parent one 16-byte record per 4 x 4 x 4 leaves
//   bricks           per occupied cell of every level a bitmask over its
//                    ratio^3 children (linear order)
//   leaves           (first entry, count) ranges into leaf-ordered surfels, in
//                    key order and once more block by block
//   surfels          two 16-byte halves per entry, together, in leaf order:
//                    (x, y, z, point id) and (unit normal, label rank)
//
// A point is listed in EVERY leaf that the axis-aligned box of its disk
// (radius r_s, its own normal) overlaps, padded by a rounding margin, so a
// traversal that tests the leaves it passes finds every disk it crosses.
//
// Pipeline: ingest (normalise normals, validate, AABB, max label) -> sync ->
// label ranks -> per-point leaf counts -> scan -> sync -> emit (key, id) ->
// radix sort -> per-tile node-start counts + their scan -> sync -> bricks,
// leaf ranges, occupied top cells (one pass over the sorted keys) -> skip
// codes of the top grid, blocks -> surfel gather.
#include "internal.h"

#include <algorithm>
#include <cmath>
#include <cstring>

namespace pcrl {

constexpr int BUILD_BLOCK = 256;

static unsigned blocks_for(int64_t n, int block = BUILD_BLOCK) {
    int64_t g = (n + block - 1) / block;
    return (unsigned)std::max<int64_t>(1, g);
}

static int bits_for(uint64_t max_value) {
    int b = 1;
    while (b < 64 && (max_value >> b) != 0) ++b;
    return b;
}

// ---------------------------------------------------------------------------
// ingest
// ---------------------------------------------------------------------------

struct IngestOut {
    float lo[3];
    float hi[3];
    uint32_t max_label;
    uint32_t bad;  // bit0 non-finite position, bit1 bad normal
};

__global__ __launch_bounds__(BUILD_BLOCK) void k_ingest(const float* xyz, const float* nrm, const uint32_t* label,
                                                        int64_t n, float4* unit_nrm, IngestOut* partial) {
    float lo[3] = {INFINITY, INFINITY, INFINITY};
    float hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    uint32_t ml = 0, bad = 0;
    for (int64_t i = (int64_t)blockIdx.x * BUILD_BLOCK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BUILD_BLOCK) {
        const float x = xyz[3 * i], y = xyz[3 * i + 1], z = xyz[3 * i + 2];
        if (!isfinite(x) || !isfinite(y) || !isfinite(z)) bad |= 1u;
        lo[0] = fminf(lo[0], x); lo[1] = fminf(lo[1], y); lo[2] = fminf(lo[2], z);
        hi[0] = fmaxf(hi[0], x); hi[1] = fmaxf(hi[1], y); hi[2] = fmaxf(hi[2], z);
        const float a = nrm[3 * i], b = nrm[3 * i + 1], c = nrm[3 * i + 2];
        const float l2 = a * a + b * b + c * c;
        float inv = 0.f;
        if (!(l2 > 0.f) || !isfinite(l2))
            bad |= 2u;
        else
            inv = 1.0f / sqrtf(l2);
        unit_nrm[i] = make_float4(a * inv, b * inv, c * inv, 0.f);
        ml = max(ml, label[i]);
    }
    // block reduction through LDS
    __shared__ float s_lo[3][BUILD_BLOCK / 64], s_hi[3][BUILD_BLOCK / 64];
    __shared__ uint32_t s_ml[BUILD_BLOCK / 64], s_bad[BUILD_BLOCK / 64];
    for (int off = 32; off > 0; off >>= 1) {
        for (int a = 0; a < 3; ++a) {
            lo[a] = fminf(lo[a], __shfl_xor(lo[a], off, 64));
            hi[a] = fmaxf(hi[a], __shfl_xor(hi[a], off, 64));
        }
        ml = max(ml, __shfl_xor(ml, off, 64));
        bad |= __shfl_xor(bad, off, 64);
    }
    const int w = threadIdx.x >> 6;
    if (lane_id() == 0) {
        for (int a = 0; a < 3; ++a) { s_lo[a][w] = lo[a]; s_hi[a][w] = hi[a]; }
        s_ml[w] = ml;
        s_bad[w] = bad;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        IngestOut o;
        for (int a = 0; a < 3; ++a) { o.lo[a] = INFINITY; o.hi[a] = -INFINITY; }
        o.max_label = 0;
        o.bad = 0;
        for (int k = 0; k < BUILD_BLOCK / 64; ++k) {
            for (int a = 0; a < 3; ++a) { o.lo[a] = fminf(o.lo[a], s_lo[a][k]); o.hi[a] = fmaxf(o.hi[a], s_hi[a][k]); }
            o.max_label = max(o.max_label, s_ml[k]);
            o.bad |= s_bad[k];
        }
        partial[blockIdx.x] = o;
    }
}

// One block of BUILD_BLOCK threads folds the per-block partials.
__global__ __launch_bounds__(BUILD_BLOCK) void k_ingest_final(const IngestOut* partial, int nb, IngestOut* out) {
    float lo[3] = {INFINITY, INFINITY, INFINITY};
    float hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    uint32_t ml = 0, bad = 0;
    for (int k = threadIdx.x; k < nb; k += BUILD_BLOCK) {
        const IngestOut p = partial[k];
        for (int a = 0; a < 3; ++a) { lo[a] = fminf(lo[a], p.lo[a]); hi[a] = fmaxf(hi[a], p.hi[a]); }
        ml = max(ml, p.max_label);
        bad |= p.bad;
    }
    for (int off = 32; off > 0; off >>= 1) {
        for (int a = 0; a < 3; ++a) {
            lo[a] = fminf(lo[a], __shfl_xor(lo[a], off, 64));
            hi[a] = fmaxf(hi[a], __shfl_xor(hi[a], off, 64));
        }
        ml = max(ml, __shfl_xor(ml, off, 64));
        bad |= __shfl_xor(bad, off, 64);
    }
    __shared__ IngestOut s[BUILD_BLOCK / 64];
    const int w = threadIdx.x >> 6;
    if (lane_id() == 0) {
        for (int a = 0; a < 3; ++a) { s[w].lo[a] = lo[a]; s[w].hi[a] = hi[a]; }
        s[w].max_label = ml;
        s[w].bad = bad;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        IngestOut o = s[0];
        for (int k = 1; k < BUILD_BLOCK / 64; ++k) {
            for (int a = 0; a < 3; ++a) { o.lo[a] = fminf(o.lo[a], s[k].lo[a]); o.hi[a] = fmaxf(o.hi[a], s[k].hi[a]); }
            o.max_label = max(o.max_label, s[k].max_label);
            o.bad |= s[k].bad;
        }
        *out = o;
    }
}

// ---------------------------------------------------------------------------
// dilated keys
// ---------------------------------------------------------------------------

struct KeyParams {
    SceneView v;
    float r_s;
    float pad;
    int32_t id_bits;   // packed 64-bit items: bits of the point index below the key
    uint8_t* occ0;     // k_key_count: level-0 cells that a point's leaf box reaches (set to 1)
    const uint32_t* c0;  // k_key_emit: rank of each such level-0 cell (the key's level-0 part)
};

// Hierarchical key of leaf (x, y, z) with level 0 numbered by `c0` (rank of
// the level-0 cell among the occupied ones) or by its linear index (c0
// null); the quotients use magic divisions.
__host__ __device__ __forceinline__ uint64_t leaf_key_fast(const SceneView& v, const uint32_t* c0, int x, int y, int z) {
    int p[3] = {span_div(x, v.mspan[0]), span_div(y, v.mspan[0]), span_div(z, v.mspan[0])};
    const uint32_t cell0 = (uint32_t)p[0] + (uint32_t)v.dim0[0] * ((uint32_t)p[1] + (uint32_t)v.dim0[1] * (uint32_t)p[2]);
    uint64_t k = c0 ? (uint64_t)c0[cell0] : (uint64_t)cell0;
#pragma unroll
    for (int i = 1; i < PCRL_MAX_LEVELS; ++i) {
        if (i >= v.nlev) break;
        const int q[3] = {span_div(x, v.mspan[i]), span_div(y, v.mspan[i]), span_div(z, v.mspan[i])};
        const int r = v.ratio[i - 1];
        const int loc = (q[0] - r * p[0]) + r * ((q[1] - r * p[1]) + r * (q[2] - r * p[2]));
        k = (k << v.lbits[i]) | (uint64_t)loc;
        p[0] = q[0];
        p[1] = q[1];
        p[2] = q[2];
    }
    return k;
}

__device__ __forceinline__ void disk_leaf_box(const KeyParams& kp, const float* xyz, const float4* un, int64_t i,
                                              int lo[3], int hi[3]) {
    const float p[3] = {xyz[3 * i], xyz[3 * i + 1], xyz[3 * i + 2]};
    const float4 nn = un[i];
    const float nv[3] = {nn.x, nn.y, nn.z};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float e = kp.r_s * sqrtf(fmaxf(0.f, 1.f - nv[a] * nv[a])) + kp.pad;
        int l = (int)floorf((p[a] - e - kp.v.org[a]) * kp.v.inv_h);
        int u = (int)floorf((p[a] + e - kp.v.org[a]) * kp.v.inv_h);
        lo[a] = min(max(l, 0), kp.v.dim[a] - 1);
        hi[a] = min(max(u, 0), kp.v.dim[a] - 1);
    }
}

// Whether the disk of point i (radius r_s) may meet leaf (x, y, z), the leaf
// grown by the rounding pad: both the disk's sphere and its plane must reach
// the box.  Both are necessary conditions of an intersection, so no leaf the
// disk touches is dropped; the corner leaves of the disk's bounding box
// (sphere test) and, for tilted disks, off-plane leaves (plane test) are.
__device__ __forceinline__ bool disk_meets_leaf(const KeyParams& kp, const float p[3], const float nv[3], int x, int y,
                                                int z) {
    const float hh = 0.5f * kp.v.h + kp.pad;
    const int c[3] = {x, y, z};
    float d2 = 0.f, pr = 0.f, dn = 0.f;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float ca = kp.v.org[a] + ((float)c[a] + 0.5f) * kp.v.h;  // leaf centre
        const float q = fabsf(p[a] - ca) - hh;
        if (q > 0.f) d2 += q * q;
        pr += fabsf(nv[a]) * hh;
        dn += nv[a] * (ca - p[a]);
    }
    const float r = kp.r_s + kp.pad;
    return d2 <= r * r && fabsf(dn) <= pr + kp.pad;
}

// Keys of one wave staged in LDS before a coalesced copy out (entries past
// the stage are written directly).
constexpr int EMIT_STAGE = 2048;

template <bool EMIT, typename K>
__device__ __forceinline__ uint32_t disk_leaves(const KeyParams& kp, const float* xyz, const float4* un, int64_t i,
                                                K* keys, uint32_t* ids, uint32_t o, K* stage = nullptr,
                                                uint32_t base = 0) {
    int lo[3], hi[3];
    disk_leaf_box(kp, xyz, un, i, lo, hi);
    const float p[3] = {xyz[3 * i], xyz[3 * i + 1], xyz[3 * i + 2]};
    const float4 nn = un[i];
    const float nv[3] = {nn.x, nn.y, nn.z};
    uint32_t k = 0;
    for (int z = lo[2]; z <= hi[2]; ++z)
        for (int y = lo[1]; y <= hi[1]; ++y)
            for (int x = lo[0]; x <= hi[0]; ++x) {
                // a disk inside a single leaf keeps it without the test
                const bool one = lo[0] == hi[0] && lo[1] == hi[1] && lo[2] == hi[2];
                if (!one && !disk_meets_leaf(kp, p, nv, x, y, z)) continue;
                if (EMIT) {
                    const uint64_t key = leaf_key_fast(kp.v, kp.c0, x, y, z);
                    if (ids) {
                        keys[o + k] = (K)key;
                        ids[o + k] = (uint32_t)i;
                    } else {
                        // packed: the key above the point index (one 8-byte item to sort)
                        const K item = (K)((key << kp.id_bits) | (uint64_t)i);
                        const uint32_t at = o + k;
                        if (stage && at - base < (uint32_t)EMIT_STAGE) stage[at - base] = item;
                        else keys[at] = item;
                    }
                }
                ++k;
            }
    return k;
}

// Per point, the number of leaves its disk meets; the level-0 cells its leaf
// box reaches are marked in occ0 (a superset of those of its leaves).
__global__ __launch_bounds__(BUILD_BLOCK) void k_key_count(KeyParams kp, const float* xyz, const float4* un, int64_t n,
                                                           uint32_t* cnt) {
    int64_t i = (int64_t)blockIdx.x * BUILD_BLOCK + threadIdx.x;
    if (i >= n) return;
    cnt[i] = disk_leaves<false, uint64_t>(kp, xyz, un, i, nullptr, nullptr, 0);
    if (kp.occ0) {
        int lo[3], hi[3];
        disk_leaf_box(kp, xyz, un, i, lo, hi);
        const SceneView& v = kp.v;
        for (int cz = span_div(lo[2], v.mspan[0]); cz <= span_div(hi[2], v.mspan[0]); ++cz)
            for (int cy = span_div(lo[1], v.mspan[0]); cy <= span_div(hi[1], v.mspan[0]); ++cy)
                for (int cx = span_div(lo[0], v.mspan[0]); cx <= span_div(hi[0], v.mspan[0]); ++cx)
                    kp.occ0[(size_t)cx + (size_t)v.dim0[0] * ((size_t)cy + (size_t)v.dim0[1] * cz)] = 1;
    }
}

// Ranks of the marked level-0 cells (exclusive scan of occ0, widened to 32
// bits first) and the inverse map rank -> cell.
__global__ void k_occ0_widen(const uint8_t* occ0, int64_t n, uint32_t* out) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c < n) out[c] = occ0[c];
}

__global__ void k_occ0_unmap(const uint8_t* occ0, const uint32_t* rank, int64_t n, uint32_t* unmap) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c < n && occ0[c]) unmap[rank[c]] = (uint32_t)c;
}

// The counts' sum in 64 bits, for inputs whose 32-bit scan might wrap: a
// grid-stride sum per thread, one atomic per wave.
__global__ __launch_bounds__(BUILD_BLOCK) void k_count_total(const uint32_t* cnt, int64_t n, unsigned long long* total) {
    unsigned long long acc = 0;
    for (int64_t i = (int64_t)blockIdx.x * BUILD_BLOCK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BUILD_BLOCK)
        acc += cnt[i];
    acc = wave_sum_u64(acc);
    if (lane_id() == 0 && acc) atomicAdd(total, acc);
}

// The (key, point) items of every point's leaves at its offset.  Packed items
// (ids null) of a one-wave block are contiguous from its first point's
// offset: they are staged in LDS and copied out with coalesced stores.
template <typename K>
__global__ __launch_bounds__(64) void k_key_emit(KeyParams kp, const float* xyz, const float4* un, int64_t n,
                                                 const uint32_t* off, K* keys, uint32_t* ids) {
    const int64_t i = (int64_t)blockIdx.x * 64 + threadIdx.x;
    const bool in = i < n;
    if (ids) {
        if (in) (void)disk_leaves<true, K>(kp, xyz, un, i, keys, ids, off[i]);
        return;
    }
    __shared__ K stage[EMIT_STAGE];
    const uint32_t o = in ? off[i] : 0u;
    const uint32_t base = __builtin_amdgcn_readfirstlane(o);  // lane 0 holds the block's first point
    const uint32_t cnt = in ? disk_leaves<true, K>(kp, xyz, un, i, keys, nullptr, o, stage, base) : 0u;
    uint32_t end = in ? o + cnt : base;
#pragma unroll
    for (int sh = 32; sh >= 1; sh >>= 1) end = max(end, (uint32_t)__shfl_xor((int)end, sh, 64));
    const uint32_t total = min(end - base, (uint32_t)EMIT_STAGE);
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < total; j += 64) keys[(size_t)base + j] = stage[j];
}

// ---------------------------------------------------------------------------
// hierarchy from sorted keys
// ---------------------------------------------------------------------------

struct LevelShifts {
    int32_t nlev;
    int32_t sh[PCRL_MAX_LEVELS];  // node key of level i = key >> sh[i]
};

struct HierOut {
    const uint32_t* unmap0;   // rank of an occupied level-0 cell -> the cell (null: keys hold the cell)
    int32_t g_sh0;            // bits below the level-0 part of a key (without the packed point index)
    int32_t* map0;            // or null
    uint64_t* mask[PCRL_MAX_LEVELS - 1];
    uint32_t* first_child[PCRL_MAX_LEVELS - 1];
    uint2* leaf;
    uint64_t* leaf_key;
    int32_t F;                // level of the top grid
    int32_t words;            // 64-bit words per row of `occ`
    uint2* top;
    uint64_t* occ;            // occupied top cells, one bit each, rows along x
    uint32_t* tcell;          // top cell of every level-F node
};

// Node starts of every level from the sorted keys: an entry opens a node of
// level l when its key differs from the previous entry's above bit sh[l].
// A wave owns a tile of 64 ROUNDS consecutive entries, read in coalesced
// rounds of 64 (lane j of round r: entry tile + 64 r + j), up to LINK_BATCH of
// them before any is used.  Few entries are dealt out in tiles of two rounds:
// the waves' chains of rounds are what counts there: 60 k entries take 34 us
// in k_link and 9.5 in k_link_count with 16 rounds, 7.4 and 3.7 with two (3 M:
// 31 and 10 us with 16; two would need three kernels to scan the counts).
constexpr int LINK_ROUNDS = 16, LINK_ROUNDS_FEW = 2, LINK_BATCH = 8;
constexpr int64_t LINK_FEW = 64 * LINK_ROUNDS_FEW * 4096;  // whose tiles' counts one block scans

// The keys of a batch's rounds r0, r0 + 1, ..: entries from e0 on, 0 past m.
template <int B>
__device__ __forceinline__ void link_load(const uint64_t* keys, int64_t m, int64_t e0, uint64_t (&k)[B]) {
#pragma unroll
    for (int r = 0; r < B; ++r) {
        const int64_t e = e0 + 64 * r + lane_id();
        k[r] = e < m ? keys[e] : 0ull;
    }
}

// The key before this lane's in round r of a batch (`last`: before the batch).
template <int B>
__device__ __forceinline__ uint64_t link_prev(const uint64_t (&k)[B], int r, uint64_t last) {
    const uint64_t up = __shfl_up((unsigned long long)k[r], 1, 64);
    const uint64_t before = r > 0 ? (uint64_t)__shfl((unsigned long long)k[r > 0 ? r - 1 : 0], 63, 64) : last;
    return lane_id() == 0 ? before : up;
}

__device__ __forceinline__ uint32_t link_flags(uint64_t k, uint64_t prev, int64_t e, const LevelShifts& ls) {
    uint32_t f = 0;
#pragma unroll
    for (int l = 0; l < PCRL_MAX_LEVELS; ++l)
        if (l < ls.nlev && (e == 0 || ((k ^ prev) >> ls.sh[l]) != 0)) f |= 1u << l;
    return f;
}

// Per wave tile and level: the nodes that start in the tile ([level][tile]).
template <int ROUNDS>
__global__ __launch_bounds__(BUILD_BLOCK) void k_link_count(const uint64_t* keys, int64_t m, LevelShifts ls,
                                                            uint32_t* tile_cnt, uint32_t n_tiles) {
    const uint32_t tile = blockIdx.x * (BUILD_BLOCK / 64) + (threadIdx.x >> 6);
    if (tile >= n_tiles) return;
    uint32_t c[PCRL_MAX_LEVELS] = {0u, 0u, 0u, 0u};
    constexpr int B = ROUNDS < LINK_BATCH ? ROUNDS : LINK_BATCH;
    const int64_t first = (int64_t)tile * (64 * ROUNDS);
    uint64_t last = first > 0 ? keys[first - 1] : 0ull;
    for (int r0 = 0; r0 < ROUNDS; r0 += B) {
        uint64_t k[B];
        link_load<B>(keys, m, first + 64 * r0, k);
#pragma unroll
        for (int r = 0; r < B; ++r) {
            const int64_t e = first + 64 * (r0 + r) + lane_id();
            const uint64_t prev = link_prev<B>(k, r, last);
            const uint32_t f = e < m ? link_flags(k[r], prev, e, ls) : 0u;
#pragma unroll
            for (int l = 0; l < PCRL_MAX_LEVELS; ++l) c[l] += (f >> l) & 1u;
        }
        last = __shfl((unsigned long long)k[B - 1], 63, 64);
    }
#pragma unroll
    for (int l = 0; l < PCRL_MAX_LEVELS; ++l) {
        const uint32_t t = (uint32_t)wave_sum_u64(c[l]);
        if (l < ls.nlev && lane_id() == 0) tile_cnt[(size_t)l * n_tiles + tile] = t;
    }
}

// For every entry that opens a node: register the node with its parent (its
// bit in the parent brick's mask, the parent's first child), the level-0 map
// and the leaf's first entry and key.  tile_off[l][t] is the exclusive scan
// of the tiles' node counts, so the node of level l holding entry e is the
// number of level-l nodes opened up to and including e, minus one.
template <int ROUNDS>
__global__ __launch_bounds__(BUILD_BLOCK) void k_link(const uint64_t* keys, int64_t m, LevelShifts ls, SceneView v,
                                                      const uint32_t* tile_off, uint32_t n_tiles, HierOut h,
                                                      int id_bits) {
    const uint32_t tile = blockIdx.x * (BUILD_BLOCK / 64) + (threadIdx.x >> 6);
    if (tile >= n_tiles) return;
    const int L = ls.nlev;
    uint32_t carry[PCRL_MAX_LEVELS] = {0u, 0u, 0u, 0u};
    for (int l = 0; l < L; ++l) carry[l] = tile_off[(size_t)l * n_tiles + tile];
    constexpr int B = ROUNDS < LINK_BATCH ? ROUNDS : LINK_BATCH;
    const int64_t first = (int64_t)tile * (64 * ROUNDS);
    uint64_t last = first > 0 ? keys[first - 1] : 0ull, kr[B] = {};
#pragma unroll
    for (int r0 = 0; r0 < ROUNDS; ++r0) {
        const int r = r0 % B;
        if (r == 0) {
            if (r0 > 0) last = __shfl((unsigned long long)kr[B - 1], 63, 64);
            link_load<B>(keys, m, first + 64 * r0, kr);
        }
        const int64_t e = first + 64 * r0 + lane_id();
        const bool in = e < m;
        const uint64_t k = kr[r], prev = link_prev<B>(kr, r, last);
        const uint32_t f = in ? link_flags(k, prev, e, ls) : 0u;
        // the levels' flags in 8-bit fields of one word (at most 64 per field): one wave scan
        uint32_t fp = 0;
#pragma unroll
        for (int l = 0; l < PCRL_MAX_LEVELS; ++l) fp |= ((f >> l) & 1u) << (8 * l);
        const uint32_t incl = wave_incl_scan(fp);
        const uint32_t sum = __shfl(incl, 63, 64);
        uint32_t node[PCRL_MAX_LEVELS];
#pragma unroll
        for (int l = 0; l < PCRL_MAX_LEVELS; ++l) {
            node[l] = carry[l] + ((incl >> (8 * l)) & 0xFFu) - 1u;
            carry[l] += (sum >> (8 * l)) & 0xFFu;
        }
        if (!in) continue;
#pragma unroll
        for (int l = 0; l < PCRL_MAX_LEVELS; ++l) {
            if (!((f >> l) & 1u)) continue;
            if (l == 0) {
                const uint64_t top = k >> ls.sh[0];
                if (h.map0) h.map0[h.unmap0 ? (uint64_t)h.unmap0[top] : top] = (int32_t)node[0];
            }
            if (l == h.F) {
                // the node's cell of the top grid: its level-0 cell, then the local cells down to level F
                const uint64_t top = k >> ls.sh[0];
                const uint32_t c0 = (uint32_t)(h.unmap0 ? (uint64_t)h.unmap0[top] : top);
                uint32_t x = c0 % (uint32_t)v.dim0[0], y = c0 / (uint32_t)v.dim0[0], z = y / (uint32_t)v.dim0[1];
                y -= z * (uint32_t)v.dim0[1];
#pragma unroll
                for (int i = 1; i < PCRL_MAX_LEVELS; ++i) {
                    if (i > h.F) break;
                    const uint32_t r = (uint32_t)v.ratio[i - 1];
                    const uint32_t loc = (uint32_t)((k >> ls.sh[i]) & ((uint64_t(1) << v.lbits[i]) - 1));
                    x = x * r + loc % r;
                    y = y * r + (loc / r) % r;
                    z = z * r + loc / (r * r);
                }
                const size_t row = (size_t)y + (size_t)v.tdim[1] * z;
                const size_t cell = row * (size_t)v.tdim[0] + x;
                h.top[cell].x = node[l];
                if (h.tcell) h.tcell[node[l]] = (uint32_t)cell;
                atomicOr((unsigned long long*)&h.occ[row * (size_t)h.words + (x >> 6)], 1ull << (x & 63u));
            }
            if (l == L - 1) {
                const uint64_t top = k >> ls.sh[0];
                const uint64_t cell0 = h.unmap0 ? (uint64_t)h.unmap0[top] : top;
                const uint64_t kk = k >> id_bits;
                h.leaf[node[l]].x = (uint32_t)e;
                // the leaf's key with level 0 as the linear cell index
                h.leaf_key[node[l]] = (cell0 << h.g_sh0) | (kk & ((uint64_t(1) << h.g_sh0) - 1));
            }
            if (l > 0) {
                const uint32_t parent = node[l - 1];
                const uint32_t local = (uint32_t)((k >> ls.sh[l]) & ((uint64_t(1) << v.lbits[l]) - 1));
                atomicOr((unsigned long long*)&h.mask[l - 1][(size_t)parent * v.nw[l - 1] + (local >> 6)],
                         (unsigned long long)(uint64_t(1) << (local & 63)));
                // the first child of a parent is the entry that opens the parent too
                if ((f >> (l - 1)) & 1u) h.first_child[l - 1][parent] = node[l];
            }
        }
    }
}

__global__ void k_brick_base(const uint64_t* mask, const uint32_t* first_child, int64_t n_nodes, int nw,
                             uint32_t* base) {
    int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n_nodes) return;
    uint32_t run = first_child[p];
    for (int w = 0; w < nw; ++w) {
        base[(size_t)p * nw + w] = run;
        run += (uint32_t)__popcll(mask[(size_t)p * nw + w]);
    }
}

void launch_brick_base(const uint64_t* mask, const uint32_t* first_child, int64_t n_nodes, int nw, uint32_t* base,
                       hipStream_t s) {
    hipLaunchKernelGGL(k_brick_base, dim3(blocks_for(n_nodes)), dim3(BUILD_BLOCK), 0, s, mask, first_child, n_nodes, nw,
                       base);
}

__global__ void k_leaf_counts(uint2* leaf, int64_t n_leaves, int64_t m) {
    int64_t l = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (l >= n_leaves) return;
    const uint32_t end = (l + 1 < n_leaves) ? leaf[l + 1].x : (uint32_t)m;
    leaf[l].y = end - leaf[l].x;
}

// ---------------------------------------------------------------------------
// traversal structures (trace_core.h)
// ---------------------------------------------------------------------------

// Skip codes of the empty top cells.  A ray moves ahead only, so what counts
// at a cell is, per direction octant, the largest empty box of s^3 cells that
// starts at the cell and extends along the octant's signs, s in TOP_SIZES.
// The test is separable (a box is free when no cell of it is occupied), and
// runs on rows of occupancy bits, 64 cells per word:
//   k_top_rows  per (x sign, y sign, size): the cells whose s x s square of
//               rows holds an occupied cell (x by shifts, y over s rows);
//   k_top_codes the same along z per octant, then one 4-bit code s - 1 per
//               octant and cell.
// Cells outside the grid count as empty (a ray that reaches them has left).
// Both work on the rows of y0 <= y < y0 + ny of every slab: a large grid is
// done in turns, so that the planes (224 B a word) stay small.
// Bound by the loads of the rows (each word read 16 times from the caches) and
// the 8 B written per cell.  8 M cells (a 20M-point street's 1 m cells): 31 us
// and 96 us; the isotropic radii of every leaf cell and the bricks' boxes that
// they replace took 1.1 ms.  Small grids by the latency of the loads, which are
// batched: 360 k cells 13 and 20 us (16 and 24 one after another).
constexpr int TOP_NS = 7;
__device__ constexpr int TOP_SIZES[TOP_NS] = {2, 3, 4, 6, 8, 12, 16};

__global__ __launch_bounds__(BUILD_BLOCK) void k_top_rows(const uint64_t* occ, int words, int dy, int dz, int y0, int ny,
                                                          uint64_t* plane) {
    const int64_t n = (int64_t)words * ny * dz;
    const int64_t i = (int64_t)blockIdx.x * BUILD_BLOCK + threadIdx.x;
    const int q = blockIdx.y;  // bit 0: towards -x, bit 1: towards -y
    if (i >= n) return;
    const int64_t r = i / words;
    const int w = (int)(i - r * words), z = (int)(r / ny), y = y0 + (int)(r - (int64_t)z * ny);
    const int64_t row0 = ((int64_t)z * dy + y) * words;  // first word of the row
    uint64_t acc[TOP_NS] = {0, 0, 0, 0, 0, 0, 0};
    const bool nx = q & 1, my = q & 2;
    // eight rows are loaded before any is used
    for (int j0 = 0; j0 < TOP_SIZES[TOP_NS - 1]; j0 += 8) {
        uint64_t cur[8], nb[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int yy = my ? y - (j0 + j) : y + (j0 + j);
            const bool in = yy >= 0 && yy < dy;
            const uint64_t* row = occ + row0 + (int64_t)(in ? yy - y : 0) * words;
            const int wn = nx ? w - 1 : w + 1;
            cur[j] = in ? row[w] : 0ull;
            nb[j] = in && wn >= 0 && wn < words ? row[wn] : 0ull;
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (!(cur[j] | nb[j])) continue;
            uint64_t d = cur[j];
            int k = 1;
#pragma unroll
            for (int s = 0; s < TOP_NS; ++s) {
                for (; k < TOP_SIZES[s]; ++k)
                    d |= nx ? (cur[j] << k) | (nb[j] >> (64 - k)) : (cur[j] >> k) | (nb[j] << (64 - k));
                if (j0 + j < TOP_SIZES[s]) acc[s] |= d;
            }
        }
    }
#pragma unroll
    for (int s = 0; s < TOP_NS; ++s) plane[((int64_t)q * TOP_NS + s) * n + i] = acc[s];
}

constexpr int TOP_WORDS = BUILD_BLOCK / 8;  // words per block: one thread per (word, octant)

__global__ __launch_bounds__(BUILD_BLOCK) void k_top_codes(const uint64_t* occ, const uint64_t* plane, int words,
                                                           int dx, int dy, int dz, int y0, int ny, uint2* top) {
    __shared__ uint64_t bits[TOP_WORDS][8][4];
    const int64_t slab = (int64_t)words * ny, n = slab * dz;
    const int64_t i0 = (int64_t)blockIdx.x * TOP_WORDS;
    {
        const int o = threadIdx.x / TOP_WORDS, wl = threadIdx.x % TOP_WORDS;
        const int64_t i = i0 + wl;
        uint64_t e[TOP_NS] = {0, 0, 0, 0, 0, 0, 0};  // cells with a free box of the size
        if (i < n) {
            const int z = (int)(i / slab);
            const bool nz = o & 4;
            uint64_t above = ~0ull;
#pragma unroll
            for (int s = 0; s < TOP_NS; ++s) {
                if (!above) break;
                const uint64_t* pl = plane + ((int64_t)(o & 3) * TOP_NS + s) * n + i;
                uint64_t occd = 0;
#pragma unroll
                for (int k = 0; k < TOP_SIZES[s]; ++k) {
                    const int zz = nz ? z - k : z + k;
                    if (zz >= 0 && zz < dz) occd |= pl[(int64_t)(zz - z) * slab];
                }
                above = e[s] = ~occd;
            }
        }
        // code s - 1 of the largest free size in bit planes (the sizes' sets are nested)
        bits[wl][o][0] = (e[0] & ~e[1]) | e[2];
        bits[wl][o][1] = (e[1] & ~e[3]) | e[4];
        bits[wl][o][2] = (e[3] & ~e[5]) | e[6];
        bits[wl][o][3] = e[5];
    }
    __syncthreads();
    const int lane = (int)lane_id();
    for (int wl = threadIdx.x >> 6; wl < TOP_WORDS; wl += BUILD_BLOCK / 64) {
        const int64_t i = i0 + wl;
        if (i >= n) break;
        const int64_t r = i / words, z = r / ny, row = z * dy + y0 + (r - z * ny);
        const int w = (int)(i - r * words), x = w * 64 + lane;
        if (x >= dx || ((occ[row * words + w] >> lane) & 1ull)) continue;
        uint32_t code = 0;
#pragma unroll
        for (int o = 0; o < 8; ++o)
#pragma unroll
            for (int b = 0; b < 4; ++b) code |= (uint32_t)((bits[wl][o][b] >> lane) & 1ull) << (4 * o + b);
        top[row * dx + x] = make_uint2(0xFFFFFFFFu, code);
    }
}

// One wave per leaves' parent: the occupancy of its blocks of 4 x 4 x 4
// leaves from the parent's linear mask, the box of its occupied leaves, and
// the leaves' entry ranges in block order (the leaves themselves stay in key
// order, so a block's leaves are not consecutive there).  lds: nblk^3 masks
// and first ranges.  Bound by the leaf keys and ranges read and written once
// (24 B per leaf).
struct BlockArgs {
    const uint64_t* mask;
    const uint32_t* first;      // first leaf of every parent
    const uint64_t* leaf_key;
    uint2* leaf;                // .x given, .y (the count) set here
    int64_t n_parents, n_leaves, m;
    int32_t nw, r, nblk, lbits;
    uint4* blk;
    uint2* rng;
    const uint32_t* tcell;      // top cell of every parent, or null: the box goes to pbox
    uint2* top;
    uint32_t* pbox;
};

__device__ __forceinline__ void brick_blocks(const BlockArgs& a, int64_t P, uint64_t* bmask) {
    const int B = a.nblk, B3 = B * B * B, r = a.r;
    uint32_t* bfirst = reinterpret_cast<uint32_t*>(bmask + B3);
    const int lane = (int)lane_id();
    const uint64_t* mask = a.mask + (size_t)P * a.nw;
    const uint32_t first = a.first[P];
    const uint32_t end = P + 1 < a.n_parents ? a.first[P + 1] : (uint32_t)a.n_leaves;
    uint32_t run = first;
    const int sh = r > 32 ? 1 : 0;
    uint32_t ox = 0, oy = 0, oz = 0;
    for (int b0 = 0; b0 < B3; b0 += 64) {
        const int b = b0 + lane;
        uint64_t m = 0;
        if (b < B3) {
            const int bx = 4 * (b % B), by = 4 * ((b / B) % B), bz = 4 * (b / (B * B));
            const int wx = min(4, r - bx);
            for (int z = 0; z < 4 && bz + z < r; ++z)
                for (int y = 0; y < 4 && by + y < r; ++y) {
                    const int p = bx + r * (by + y + r * (bz + z));
                    uint64_t f = mask[p >> 6] >> (p & 63);
                    if ((p & 63) + wx > 64) f |= mask[(p >> 6) + 1] << (64 - (p & 63));
                    const uint32_t nib = (uint32_t)f & ((1u << wx) - 1u);
                    if (nib) {
                        m |= (uint64_t)nib << (4 * (y + 4 * z));
                        // in units of one leaf, or of two beyond ratio 32 (bits 0-31)
                        ox |= sh ? ((nib & 3u) ? 1u << (bx >> 1) : 0u) | ((nib & 12u) ? 2u << (bx >> 1) : 0u)
                                 : nib << bx;
                        oy |= 1u << ((by + y) >> sh);
                        oz |= 1u << ((bz + z) >> sh);
                    }
                }
        }
        const uint32_t c = (uint32_t)__popcll(m);
        const uint32_t incl = wave_incl_scan(c);
        if (b < B3) {
            const uint32_t f = run + incl - c;
            a.blk[(size_t)P * B3 + b] = make_uint4((uint32_t)m, (uint32_t)(m >> 32), f, 0u);
            bmask[b] = m;
            bfirst[b] = f;
        }
        run += __shfl(incl, 63, 64);
    }
    for (int off = 32; off > 0; off >>= 1) {
        ox |= __shfl_xor(ox, off, 64);
        oy |= __shfl_xor(oy, off, 64);
        oz |= __shfl_xor(oz, off, 64);
    }
    if (lane == 0) {
        const uint32_t box = (uint32_t)(__ffs(ox) - 1) | ((uint32_t)(__ffs(oy) - 1) << 5) |
                             ((uint32_t)(__ffs(oz) - 1) << 10) | ((uint32_t)(31 - __clz(ox)) << 15) |
                             ((uint32_t)(31 - __clz(oy)) << 20) | ((uint32_t)(31 - __clz(oz)) << 25);
        if (a.tcell) a.top[a.tcell[P]].y = box;
        else a.pbox[P] = box;
    }
    __syncthreads();
    for (uint32_t g = first + lane; g < end; g += 64) {
        const uint32_t loc = (uint32_t)(a.leaf_key[g] & ((uint64_t(1) << a.lbits) - 1));
        const int x = (int)(loc % (uint32_t)r), y = (int)((loc / (uint32_t)r) % (uint32_t)r),
                  z = (int)(loc / (uint32_t)(r * r));
        const int b = ((z >> 2) * B + (y >> 2)) * B + (x >> 2);
        const int bit = (x & 3) | ((y & 3) << 2) | ((z & 3) << 4);
        const uint32_t e0 = a.leaf[g].x;
        const uint32_t e1 = g + 1 < (uint32_t)a.n_leaves ? a.leaf[g + 1].x : (uint32_t)a.m;
        a.leaf[g].y = e1 - e0;
        a.rng[bfirst[b] + (uint32_t)__popcll(bmask[b] & ((uint64_t(1) << bit) - 1))] = make_uint2(e0, e1 - e0);
    }
}

__global__ __launch_bounds__(64) void k_brick_blocks(BlockArgs a) {
    extern __shared__ uint64_t bmask[];  // [nblk^3] masks, then [nblk^3] first ranges (32 bits)
    for (int64_t P = blockIdx.x; P < a.n_parents; P += gridDim.x) {
        brick_blocks(a, P, bmask);
        __syncthreads();
    }
}

__global__ void k_split_leaf(const uint2* r, int64_t n, uint32_t* b, uint32_t* c) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint2 x = r[i];
    if (b) b[i] = x.x;
    if (c) c[i] = x.y;
}

// With packed items (`packed` non-null) the point index is taken from their
// low id_bits, else from ids (the sort's values).  The block's entries pass
// through LDS, so that a wave stores 1 KB in a row.
__global__ __launch_bounds__(BUILD_BLOCK) void k_gather_surfels(uint32_t* ids, const uint64_t* packed, int id_bits, int64_t m,
                                                                const float* xyz, const float4* un, const uint32_t* label,
                                                                const uint32_t* gid, float4* surf) {
    __shared__ float4 out[2 * BUILD_BLOCK];
    const int64_t first = (int64_t)blockIdx.x * BUILD_BLOCK, e = first + threadIdx.x;
    if (e < m) {
        const uint32_t i = packed ? (uint32_t)(packed[e] & ((uint64_t(1) << id_bits) - 1)) : ids[e];
        out[2 * threadIdx.x] = make_float4(xyz[3 * (size_t)i], xyz[3 * (size_t)i + 1], xyz[3 * (size_t)i + 2],
                                           __uint_as_float(gid ? gid[i] : i));
        const float4 nn = un[i];
        out[2 * threadIdx.x + 1] = make_float4(nn.x, nn.y, nn.z, __uint_as_float(label[i]));
    }
    __syncthreads();
    const uint32_t n = 2u * (uint32_t)min((int64_t)BUILD_BLOCK, m - first);
    for (uint32_t h = threadIdx.x; h < n; h += BUILD_BLOCK) surf[2 * first + h] = out[h];
}

// Entry -> point table of a scene from its surfels.
__global__ void k_entry_points(const float4* surf, int64_t m, uint32_t* out) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < m) out[e] = __float_as_uint(surf[2 * e].w);
}

// ---------------------------------------------------------------------------
// host orchestration
// ---------------------------------------------------------------------------

static int validate_params(const PcrlVoxelParams* p, int32_t ratio[PCRL_MAX_LEVELS]) {
    if (!p) { set_error("build_voxels: params is NULL"); return PCRL_EINVAL; }
    if (p->n_levels < 1 || p->n_levels > PCRL_MAX_LEVELS) {
        set_error("build_voxels: n_levels must be in [1, %d], got %d", PCRL_MAX_LEVELS, p->n_levels);
        return PCRL_EINVAL;
    }
    if (p->flags & ~PCRL_VOXEL_COMPACT) {
        set_error("build_voxels: unknown flags 0x%x", (unsigned)p->flags);
        return PCRL_EINVAL;
    }
    if (!(p->surfel_radius > 0.f) || !std::isfinite(p->surfel_radius)) {
        set_error("build_voxels: surfel_radius must be positive and finite");
        return PCRL_EINVAL;
    }
    for (int i = 0; i < p->n_levels; ++i)
        if (!(p->level_size[i] > 0.f) || !std::isfinite(p->level_size[i])) {
            set_error("build_voxels: level_size[%d] must be positive and finite", i);
            return PCRL_EINVAL;
        }
    for (int i = 0; i + 1 < p->n_levels; ++i) {
        const double q = (double)p->level_size[i] / (double)p->level_size[i + 1];
        const double r = std::round(q);
        if (r < 1.0 || std::fabs(q - r) > 1e-4 * q || r > 64.0) {
            set_error("build_voxels: level_size[%d] = %g is not an integer multiple (1..64) of level_size[%d] = %g", i,
                      p->level_size[i], i + 1, p->level_size[i + 1]);
            return PCRL_EINVAL;
        }
        ratio[i] = (int32_t)r;
    }
    ratio[p->n_levels - 1] = 1;
    return PCRL_OK;
}

// Level of the dense top grid: the leaves' parents (the traversal then finds
// a leaf's brick with one load) while their grid has at most this many cells
// (8 bytes each), else the finest coarser level that has, or level 0.
constexpr int64_t TOP_MAX_CELLS = (int64_t)64 << 20;
// Words of occupancy whose skip codes are made at a time (0.94 GB of planes).
constexpr int64_t TOP_PLANE_WORDS = (int64_t)4 << 20;

// An overlay is built anew for every frame: its own top grid has at most this
// many cells, or so many a point when they are more, so that few points cost
// little in a large scene.  Frame and launch (300 k or 1 M rays) in a 20M-point
// street, 8 M cells: of 1.4 k points 0.42 + 1.55 ms and 64.5 MB with the grid of
// its 1 m cells, 0.35 + 1.50 ms and 0.6 MB with that of its 8 m cells; of 50 k
// points 0.50 + 2.19 ms and 81.5 MB, 0.41 + 2.15 ms and 17.6 MB.  100 k points
// in a grid of 2.1 M cells of 1 m (launches of 65 k to 1 M rays): 1.37 ms a
// launch with that grid, 1.40 with the coarser one that 16 a point would take.
constexpr int64_t OVERLAY_TOP_CELLS = (int64_t)1 << 18, OVERLAY_CELLS_PER_POINT = 32;

static int64_t top_cells(const SceneView& v) { return (int64_t)v.tdim[0] * v.tdim[1] * v.tdim[2]; }

// The top grid (of at most `most` cells where a level has so few), the brick
// levels below it and the blocks' layout of a frame.
static void set_top(SceneView& v, int64_t most) {
    const int P = v.nlev - 2;  // the leaves' parents
    int F = std::max(P, 0);
    auto dims = [&](int l) {
        for (int a = 0; a < 3; ++a) v.tdim[a] = v.dim[a] / v.span[l];
        return top_cells(v);
    };
    while (dims(F) > most && F > 0) --F;
    // depth counts at most two brick levels: with four voxel levels a top grid on level 0 leaves two above the parents
    v.depth = P < 0 ? -1 : P - F;
    const float span = (float)v.span[F];
    v.tspan = span;
    v.tinv = 1.0f / span;
    v.thalf = 0.5f / span;
    const int r = P < 0 ? 1 : v.ratio[P];
    v.rf = (float)r;
    v.r1 = (float)(r - 1);
    v.pinv = 1.0f / v.rf;
    v.phalf = 0.5f / v.rf;
    v.bunit = r <= 32 ? 1.f : 2.f;
    v.nblk = (r + 3) / 4;
    v.nblk3 = v.nblk * v.nblk * v.nblk;
    for (int a = 0; a < 3; ++a) {
        v.dimf[a] = (float)v.dim[a];
        v.dim1[a] = (float)(v.dim[a] - 1);
        v.tdim1[a] = (float)(v.tdim[a] - 1);
    }
    v.stop_pad = 1e-3f * v.h;
    for (int i = 0; i < v.depth; ++i) {
        const float s = (float)v.span[F + 1 + i];
        v.minv[i] = 1.0f / s;
        v.mhalf[i] = 0.5f / s;
        v.mspan_f[i] = s;
        v.mratio[i] = (float)v.ratio[F + i];
        v.mnw[i] = v.nw[F + i];
    }
}

// Grid frame of a new scene from its parameters and point AABB.
static int make_frame(const PcrlVoxelParams* params, const int32_t ratio[PCRL_MAX_LEVELS], const IngestOut& io,
                      SceneView& v) {
    const int L = params->n_levels;
    v.nlev = L;
    v.span[L - 1] = 1;
    for (int i = L - 2; i >= 0; --i) v.span[i] = v.span[i + 1] * ratio[i];
    if (v.span[0] > (1 << 18)) {
        set_error("build_voxels: at most 2^18 leaves per coarse cell edge (got %d)", v.span[0]);
        return PCRL_EINVAL;
    }
    for (int i = 0; i < L; ++i) v.mspan[i] = (((uint64_t)1 << 40) + (uint64_t)v.span[i] - 1) / (uint64_t)v.span[i];
    for (int i = 0; i < PCRL_MAX_LEVELS; ++i) v.ratio[i] = ratio[i];
    const float h = params->level_size[L - 1];
    v.h = h;
    v.inv_h = 1.0f / h;
    const float r_s = params->surfel_radius;
    v.r_s = r_s;
    v.rs2 = r_s * r_s;
    float amax = 0.f;
    for (int a = 0; a < 3; ++a) amax = std::max(amax, std::max(std::fabs(io.lo[a]), std::fabs(io.hi[a])));
    v.pad = 1e-3f * h + 4e-6f * amax;
    const double cell0 = (double)h * v.span[0];
    for (int a = 0; a < 3; ++a) {
        const double lo = (double)io.lo[a] - r_s - v.pad - h;
        const double hi = (double)io.hi[a] + r_s + v.pad + h;
        int64_t d0 = (int64_t)std::ceil((hi - lo) / cell0);
        if (d0 < 1) d0 = 1;
        if (d0 * v.span[0] >= (int64_t)1 << 22) {
            set_error("build_voxels: leaf grid too large along axis %d (%lld leaves, max 2^22)", a,
                      (long long)(d0 * v.span[0]));
            return PCRL_EINVAL;
        }
        v.dim0[a] = (int32_t)d0;
        v.dim[a] = (int32_t)(d0 * v.span[0]);
        v.org[a] = (float)lo;
        v.hi[a] = (float)((double)v.org[a] + (double)v.dim[a] * h);
    }
    const uint64_t cells0 = (uint64_t)v.dim0[0] * v.dim0[1] * v.dim0[2];
    v.lbits[0] = bits_for(cells0 - 1);
    int key_bits = v.lbits[0];
    for (int i = 1; i < L; ++i) {
        const uint64_t r3 = (uint64_t)ratio[i - 1] * ratio[i - 1] * ratio[i - 1];
        v.lbits[i] = bits_for(r3 - 1);
        key_bits += v.lbits[i];
        v.nw[i - 1] = (int32_t)((r3 + 63) / 64);
    }
    if (key_bits > 64) {
        set_error("build_voxels: hierarchical key needs %d bits (max 64); use coarser levels", key_bits);
        return PCRL_EINVAL;
    }
    v.key_bits = key_bits;
    set_top(v, TOP_MAX_CELLS);
    const double diag = std::sqrt((double)(io.hi[0] - io.lo[0]) * (io.hi[0] - io.lo[0]) +
                                  (double)(io.hi[1] - io.lo[1]) * (io.hi[1] - io.lo[1]) +
                                  (double)(io.hi[2] - io.lo[2]) * (io.hi[2] - io.lo[2]));
    v.t_eps = params->t_eps > 0.f ? params->t_eps : (float)std::max(1e-5 * diag, 1e-6);
    return PCRL_OK;
}

// What a hierarchy build produces besides its view.
struct HierBuild {
    int64_t n_entries = 0;
    int64_t n_leaves = 0;
    int64_t n_nodes[PCRL_MAX_LEVELS] = {0, 0, 0, 0};
    int64_t bytes = 0;
    uint64_t* leaf_key = nullptr;
    uint32_t* entry_point = nullptr;
    uint2* leaf_range = nullptr;
    uint32_t* first_child[PCRL_MAX_LEVELS - 1] = {};
};

// Voxelise n ingested points into the frame already set in v (level-0 map,
// bricks, leaves, surfels).  gid: global point ids (null: 0..n-1);
// base: with the level-0 map (the implicit surface's, which overlays have not).
static int build_hierarchy(const float* xyz, const float4* unit_nrm, const uint32_t* label, const uint32_t* gid,
                           int64_t n, hipStream_t s, bool base, SceneView& v, DevBufs& B, DevBufs& T,
                           HierBuild& hb) {
    const int L = v.nlev;
    int rc = PCRL_OK;
    LevelShifts ls{};
    ls.nlev = L;
    {
        int acc = 0;
        for (int l = L - 1; l >= 0; --l) {
            ls.sh[l] = acc;
            acc += v.lbits[l];
        }
    }
    const uint64_t cells0 = (uint64_t)v.dim0[0] * v.dim0[1] * v.dim0[2];
    int32_t* map0 = nullptr;
    if (base) {
        if ((rc = B.alloc(&map0, (size_t)cells0))) return rc;
        if ((rc = fill_u32((uint32_t*)map0, 0xFFFFFFFFu, (int64_t)cells0, s))) return rc;
    }
    v.map0 = map0;
    for (int l = 0; l < PCRL_MAX_LEVELS; ++l) v.nn[l] = 0;
    hb.bytes = base ? (int64_t)cells0 * 4 : 0;
    const int64_t cells = top_cells(v);
    uint2* top = nullptr;
    if ((rc = B.alloc(&top, (size_t)cells))) return rc;
    v.top = top;
    hb.bytes += cells * 8;
    if (n == 0) return fill_u32((uint32_t*)top, 0xFFFFFFFFu, 2 * cells, s);  // all empty: the largest skips

    // dilated key counts and their total
    KeyParams kp{};
    kp.v = v;
    kp.r_s = v.r_s;
    kp.pad = v.pad;
    uint32_t *cnt = nullptr, *tot = nullptr, *rank0 = nullptr;
    uint8_t* occ0 = nullptr;
    if ((rc = T.alloc(&cnt, (size_t)n)) || (rc = T.alloc(&tot, 2)) || (rc = T.alloc(&rank0, (size_t)cells0)) ||
        (rc = T.alloc(&occ0, (size_t)((cells0 + 3) & ~3ull))) ||
        (rc = fill_u32((uint32_t*)occ0, 0u, (int64_t)((cells0 + 3) / 4), s)))
        return rc;
    kp.occ0 = occ0;
    hipLaunchKernelGGL(k_key_count, dim3(blocks_for(n)), dim3(BUILD_BLOCK), 0, s, kp, xyz, unit_nrm, n, cnt);
    // the key's level-0 part: the rank of the cell among the marked ones
    hipLaunchKernelGGL(k_occ0_widen, dim3(blocks_for((int64_t)cells0)), dim3(BUILD_BLOCK), 0, s, occ0,
                       (int64_t)cells0, rank0);
    if ((rc = scan_u32(rank0, rank0, (int64_t)cells0, tot + 1, s))) return rc;
    // a disk meets at most (ceil(2 (r_s + pad) / leaf) + 1)^3 leaves: when n times
    // that could reach 2^32, the counts are also summed in 64 bits
    const double span = std::ceil(2.0 * ((double)v.r_s + (double)v.pad) / (double)v.h) + 1.0;
    const bool may_wrap = (double)n * span * span * span >= 4294967280.0;
    unsigned long long* tot64 = nullptr;
    if (may_wrap) {
        if ((rc = T.alloc(&tot64, 1)) || (rc = fill_u64((uint64_t*)tot64, 0ull, 1, s))) return rc;
        hipLaunchKernelGGL(k_count_total, dim3(std::min<unsigned>(blocks_for(n), 4096u)), dim3(BUILD_BLOCK), 0, s, cnt,
                           n, tot64);
    }
    if ((rc = scan_u32(cnt, cnt, n, tot, s))) return rc;
    unsigned long long host_tot = 0;
    uint32_t host_tot2[2] = {0u, 0u};
    const bool copied = read_back(host_tot2, tot, 8, s) == PCRL_OK &&
                        (!may_wrap || read_back(&host_tot, tot64, 8, s) == PCRL_OK);
    const uint32_t host_tot32 = host_tot2[0], n_marked0 = host_tot2[1];
    if (!copied) {
        set_error("build_voxels: key count failed: %s", hipGetErrorString(hipGetLastError()));
        return PCRL_EHIP;
    }
    if (!may_wrap) host_tot = host_tot32;
    // entries are indexed with 32 bits throughout (ranges, sort values, surfel ids)
    if (host_tot > 0xFFFFFFF0ull) {
        set_error("build_voxels: %llu (leaf, point) entries exceed the 32-bit entry index; use a larger leaf size "
                  "or fewer points", host_tot);
        return PCRL_EINVAL;
    }
    const int64_t m = (int64_t)host_tot;
    hb.n_entries = m;

    // the key's level 0 numbered by rank among the marked cells when that
    // takes fewer bits than the linear cell index (fewer radix passes)
    const int lbits0 = bits_for(n_marked0 > 1 ? n_marked0 - 1 : 1);
    const bool ranked0 = lbits0 < v.lbits[0];
    const int kbits = ranked0 ? v.key_bits - v.lbits[0] + lbits0 : v.key_bits;
    uint32_t* unmap0 = nullptr;
    if (ranked0) {
        if ((rc = T.alloc(&unmap0, n_marked0))) return rc;
        hipLaunchKernelGGL(k_occ0_unmap, dim3(blocks_for((int64_t)cells0)), dim3(BUILD_BLOCK), 0, s, occ0, rank0,
                           (int64_t)cells0, unmap0);
        kp.c0 = rank0;
    }
    kp.occ0 = nullptr;

    // emit and sort (key, local point index): the point index packed below the
    // key in one 64-bit item when both fit (the stable sort on the key bits
    // then moves one 8-byte item per entry), else 64-bit keys and 32-bit ids
    int id_bits = 1;
    while (id_bits < 32 && ((uint64_t)(n > 0 ? n - 1 : 0) >> id_bits)) ++id_bits;
    const bool packed = kbits + id_bits <= 64;
    kp.id_bits = packed ? id_bits : 0;
    const int g_sh0 = ls.sh[0];
    uint64_t* keys = nullptr;
    uint32_t* ids = nullptr;  // entry -> point: packed items carry it; else the sort's values
    if (!packed && (rc = B.alloc(&ids, (size_t)m))) return rc;
    if (packed) {
        if ((rc = T.alloc(&keys, (size_t)m))) return rc;
        hipLaunchKernelGGL(k_key_emit<uint64_t>, dim3(blocks_for(n, 64)), dim3(64), 0, s, kp, xyz, unit_nrm, n, cnt,
                           keys, (uint32_t*)nullptr);
        if ((rc = radix_sort_u64_bits(keys, nullptr, m, id_bits, kbits, s))) return rc;
        for (int l = 0; l < L; ++l) ls.sh[l] += id_bits;
    } else {
        if ((rc = T.alloc(&keys, (size_t)m))) return rc;
        hipLaunchKernelGGL(k_key_emit<uint64_t>, dim3(blocks_for(n, 64)), dim3(64), 0, s, kp, xyz, unit_nrm, n, cnt,
                           keys, ids);
        if ((rc = radix_sort_u64(keys, ids, m, kbits, s))) return rc;
    }
    hb.entry_point = ids;

    // per-level node boundaries: node starts counted per tile, the tiles' counts scanned
    const bool few = m <= LINK_FEW;
    const int64_t link_tile = 64 * (few ? LINK_ROUNDS_FEW : LINK_ROUNDS);
    const int64_t n_tiles64 = (m + link_tile - 1) / link_tile;
    const uint32_t n_tiles = (uint32_t)n_tiles64;
    uint32_t *tiles = nullptr, *ltot = nullptr;
    if ((rc = T.alloc(&tiles, (size_t)L * n_tiles)) || (rc = T.alloc(&ltot, PCRL_MAX_LEVELS))) return rc;
    const unsigned link_blocks = (unsigned)((n_tiles64 + BUILD_BLOCK / 64 - 1) / (BUILD_BLOCK / 64));
    if (few)
        hipLaunchKernelGGL(k_link_count<LINK_ROUNDS_FEW>, dim3(link_blocks), dim3(BUILD_BLOCK), 0, s, keys, m, ls, tiles,
                           n_tiles);
    else
        hipLaunchKernelGGL(k_link_count<LINK_ROUNDS>, dim3(link_blocks), dim3(BUILD_BLOCK), 0, s, keys, m, ls, tiles, n_tiles);
    for (int l = 0; l < L; ++l)
        if ((rc = scan_u32(tiles + (size_t)l * n_tiles, tiles + (size_t)l * n_tiles, n_tiles, ltot + l, s))) return rc;
    uint32_t host_nodes[PCRL_MAX_LEVELS] = {0, 0, 0, 0};
    if (read_back(host_nodes, ltot, 4 * L, s) != PCRL_OK) {
        set_error("build_voxels: level scan failed: %s", hipGetErrorString(hipGetLastError()));
        return PCRL_EHIP;
    }
    for (int l = 0; l < L; ++l) {
        hb.n_nodes[l] = host_nodes[l];
        v.nn[l] = host_nodes[l];
    }
    const int64_t n_leaves = host_nodes[L - 1];
    hb.n_leaves = n_leaves;

    HierOut ho{};
    ho.unmap0 = unmap0;
    ho.g_sh0 = g_sh0;
    ho.map0 = map0;
    for (int l = 0; l + 1 < L; ++l) {
        const size_t words = (size_t)host_nodes[l] * v.nw[l];
        uint64_t* mk = nullptr;
        uint32_t* fc = nullptr;
        if ((rc = B.alloc(&mk, words)) || (rc = B.alloc(&fc, host_nodes[l]))) return rc;
        if ((rc = fill_u64(mk, 0ull, (int64_t)words, s))) return rc;
        ho.mask[l] = mk;
        ho.first_child[l] = fc;
        hb.first_child[l] = fc;
        v.mask[l] = mk;
        hb.bytes += (int64_t)words * 8 + (int64_t)host_nodes[l] * 4;
    }
    uint2* leaf = nullptr;
    uint64_t* lkey = nullptr;
    if ((rc = B.alloc(&leaf, (size_t)n_leaves)) || (rc = B.alloc(&lkey, (size_t)n_leaves))) return rc;
    ho.leaf = leaf;
    ho.leaf_key = lkey;
    const int P = L - 2;
    const int F = P < 0 ? 0 : P - v.depth;
    const int words = (v.tdim[0] + 63) / 64;
    const int64_t occ_words = (int64_t)words * v.tdim[1] * v.tdim[2];
    uint64_t* occ = nullptr;
    uint32_t* tcell = nullptr;
    if ((rc = T.alloc(&occ, (size_t)occ_words)) || (rc = fill_u64(occ, 0ull, occ_words, s))) return rc;
    if (v.depth == 0 && (rc = T.alloc(&tcell, (size_t)host_nodes[P]))) return rc;
    ho.F = F;
    ho.words = words;
    ho.top = top;
    ho.occ = occ;
    ho.tcell = tcell;
    if (few)
        hipLaunchKernelGGL(k_link<LINK_ROUNDS_FEW>, dim3(link_blocks), dim3(BUILD_BLOCK), 0, s, keys, m, ls, v, tiles, n_tiles,
                           ho, packed ? id_bits : 0);
    else
        hipLaunchKernelGGL(k_link<LINK_ROUNDS>, dim3(link_blocks), dim3(BUILD_BLOCK), 0, s, keys, m, ls, v, tiles, n_tiles, ho,
                           packed ? id_bits : 0);
    // the brick levels between the top grid and the leaves' parents
    for (int i = 0; i < v.depth; ++i) {
        uint32_t* bs = nullptr;
        if ((rc = B.alloc(&bs, (size_t)host_nodes[F + i] * v.nw[F + i]))) return rc;
        launch_brick_base(ho.mask[F + i], ho.first_child[F + i], host_nodes[F + i], v.nw[F + i], bs, s);
        v.mmask[i] = ho.mask[F + i];
        v.mbase[i] = bs;
        hb.bytes += (int64_t)host_nodes[F + i] * v.nw[F + i] * 4;
    }
    {
        const int64_t per_row = (int64_t)words * v.tdim[2];
        const int rows = (int)std::min<int64_t>(v.tdim[1], std::max<int64_t>(1, TOP_PLANE_WORDS / per_row));
        uint64_t* plane = nullptr;
        if ((rc = T.alloc(&plane, (size_t)(4 * TOP_NS * per_row * rows)))) return rc;
        for (int y0 = 0; y0 < v.tdim[1]; y0 += rows) {
            const int ny = std::min(rows, v.tdim[1] - y0);
            hipLaunchKernelGGL(k_top_rows, dim3(blocks_for(per_row * ny), 4), dim3(BUILD_BLOCK), 0, s, (const uint64_t*)occ,
                               words, v.tdim[1], v.tdim[2], y0, ny, plane);
            hipLaunchKernelGGL(k_top_codes, dim3(blocks_for(per_row * ny, TOP_WORDS)), dim3(BUILD_BLOCK), 0, s,
                               (const uint64_t*)occ, (const uint64_t*)plane, words, v.tdim[0], v.tdim[1], v.tdim[2], y0, ny,
                               top);
        }
    }
    v.leaf = leaf;
    hb.leaf_range = leaf;
    hb.leaf_key = lkey;
    if (P < 0) {
        hipLaunchKernelGGL(k_leaf_counts, dim3(blocks_for(n_leaves)), dim3(BUILD_BLOCK), 0, s, leaf, n_leaves, m);
        v.rng = leaf;
    } else {
        uint4* blk = nullptr;
        uint2* rng = nullptr;
        uint32_t* pbox = nullptr;
        const size_t nb = (size_t)host_nodes[P] * (size_t)v.nblk3;
        if ((rc = B.alloc(&blk, nb)) || (rc = B.alloc(&rng, (size_t)n_leaves)) ||
            (v.depth > 0 && (rc = B.alloc(&pbox, (size_t)host_nodes[P]))))
            return rc;
        BlockArgs ba{};
        ba.mask = ho.mask[P];
        ba.first = ho.first_child[P];
        ba.leaf_key = lkey;
        ba.leaf = leaf;
        ba.n_parents = host_nodes[P];
        ba.n_leaves = n_leaves;
        ba.m = m;
        ba.nw = v.nw[P];
        ba.r = v.ratio[P];
        ba.nblk = v.nblk;
        ba.lbits = v.lbits[L - 1];
        ba.blk = blk;
        ba.rng = rng;
        ba.tcell = tcell;
        ba.top = top;
        ba.pbox = pbox;
        hipLaunchKernelGGL(k_brick_blocks, dim3((unsigned)std::min<int64_t>(host_nodes[P], WAVES_MAX)), dim3(64),
                           (size_t)v.nblk3 * 12, s, ba);
        v.blk = blk;
        v.rng = rng;
        v.pbox = pbox;
        hb.bytes += (int64_t)nb * 16 + n_leaves * 8 + (pbox ? (int64_t)host_nodes[P] * 4 : 0);
    }

    // surfels in leaf order
    float4* surf = nullptr;
    if ((rc = B.alloc(&surf, 2 * (size_t)m))) return rc;
    hipLaunchKernelGGL(k_gather_surfels, dim3(blocks_for(m)), dim3(BUILD_BLOCK), 0, s, ids,
                       packed ? (const uint64_t*)keys : (const uint64_t*)nullptr, packed ? id_bits : 0, m, xyz,
                       unit_nrm, label, gid, surf);
    v.surf = surf;
    if (hipGetLastError() != hipSuccess) {
        set_error("build_voxels: kernel launch failed");
        return PCRL_EHIP;
    }
    hb.bytes += m * ((ids ? 4 : 0) + 32) + n_leaves * 16;
    return PCRL_OK;
}

// Validate and normalise n points (one synchronisation).  unit_nrm is
// allocated in T.
static int ingest(const float* xyz, const float* nrm, const uint32_t* label, int64_t n, hipStream_t s, DevBufs& T,
                  float4** unit_nrm, IngestOut& io, const char* fn) {
    for (int a = 0; a < 3; ++a) { io.lo[a] = 0.f; io.hi[a] = 0.f; }
    io.max_label = 0;
    io.bad = 0;
    *unit_nrm = nullptr;
    if (n == 0) return PCRL_OK;
    int rc;
    if ((rc = T.alloc(unit_nrm, (size_t)n))) return rc;
    const unsigned nb = std::min<unsigned>(blocks_for(n), (unsigned)device_cus() * 4);
    IngestOut *partial = nullptr, *res = nullptr;
    if ((rc = T.alloc(&partial, nb)) || (rc = T.alloc(&res, 1))) return rc;
    hipLaunchKernelGGL(k_ingest, dim3(nb), dim3(BUILD_BLOCK), 0, s, xyz, nrm, label, n, *unit_nrm, partial);
    hipLaunchKernelGGL(k_ingest_final, dim3(1), dim3(BUILD_BLOCK), 0, s, partial, (int)nb, res);
    if (hipGetLastError() != hipSuccess || read_back(&io, res, sizeof io, s) != PCRL_OK) {
        set_error("%s: ingest failed: %s", fn, hipGetErrorString(hipGetLastError()));
        return PCRL_EHIP;
    }
    if (io.bad & 1u) { set_error("%s: non-finite point coordinate", fn); return PCRL_EINVAL; }
    if (io.bad & 2u) { set_error("%s: zero or non-finite normal", fn); return PCRL_EINVAL; }
    return PCRL_OK;
}

static int build_impl(const float* xyz, const float* nrm, const uint32_t* label, int64_t n,
                      const PcrlVoxelParams* params, hipStream_t s, PcrlScene* S) {
    int32_t ratio[PCRL_MAX_LEVELS] = {1, 1, 1, 1};
    PCRL_TRY(validate_params(params, ratio));
    if (n < 0 || (n > 0 && (!xyz || !nrm || !label))) {
        set_error("build_voxels: invalid point arrays (n = %lld)", (long long)n);
        return PCRL_EINVAL;
    }
    if (n > (int64_t)0x7FFFFFFF) {
        set_error("build_voxels: at most 2^31-1 points are supported");
        return PCRL_EINVAL;
    }
    (void)hipGetDevice(&S->device);
    S->bufs.stream = s;
    DevBufs T;
    T.stream = s;
    auto fail = [&](int code) { T.release(); return code; };
    float4* unit_nrm = nullptr;
    IngestOut io{};
    int rc;
    if ((rc = ingest(xyz, nrm, label, n, s, T, &unit_nrm, io, "build_voxels"))) return fail(rc);
    SceneView& v = S->view;
    if ((rc = make_frame(params, ratio, io, v))) return fail(rc);
    HierBuild hb;
    S->compact = (params->flags & PCRL_VOXEL_COMPACT) != 0;
    if ((rc = build_hierarchy(xyz, unit_nrm, label, nullptr, n, s, true, v, S->bufs, T, hb))) return fail(rc);
    S->max_label = io.max_label;
    S->leaf_key = hb.leaf_key;
    S->entry_point = hb.entry_point;
    S->leaf_range = hb.leaf_range;
    for (int l = 0; l + 1 < PCRL_MAX_LEVELS; ++l) S->first_child[l] = hb.first_child[l];
    PcrlSceneInfo& info = S->info;
    info.n_points = n;
    info.n_entries = hb.n_entries;
    info.n_leaves = hb.n_leaves;
    for (int l = 0; l < PCRL_MAX_LEVELS; ++l) info.n_nodes[l] = hb.n_nodes[l];
    info.max_label = (int32_t)io.max_label;
    info.n_levels = params->n_levels;
    for (int a = 0; a < 3; ++a) {
        info.dims[a] = v.dim[a];
        info.dims0[a] = v.dim0[a];
        info.origin[a] = v.org[a];
        info.aabb[a] = io.lo[a];
        info.aabb[3 + a] = io.hi[a];
    }
    info.leaf_size = v.h;
    info.surfel_radius = v.r_s;
    info.t_eps = v.t_eps;
    info.key_bits = v.key_bits;
    info.device_bytes = hb.bytes;
    info.n_dynamic = 0;
    info.epoch = 0;
    T.release();
    return PCRL_OK;
}

// Overlay of dynamic points on the frame of `base`.
static int overlay_impl(PcrlScene* S, const uint32_t* gid, const float* xyz, const float* nrm, const uint32_t* label,
                        int64_t n, hipStream_t s) {
    auto ov = std::make_shared<Overlay>();
    ov->bufs.stream = s;
    DevBufs T;
    T.stream = s;
    auto fail = [&](int code) { T.release(); return code; };
    float4* unit_nrm = nullptr;
    IngestOut io{};
    int rc;
    if ((rc = ingest(xyz, nrm, label, n, s, T, &unit_nrm, io, "update_points"))) return fail(rc);
    const SceneView& bv = S->view;
    // every dynamic disk, dilated as in disk_leaf_box, must lie inside the base grid (no leaf clamped)
    for (int a = 0; a < 3; ++a) {
        const float m = bv.r_s + 2.f * bv.pad;
        if (n > 0 && (io.lo[a] - m <= bv.org[a] || io.hi[a] + m >= bv.hi[a])) {
            set_error("update_points: dynamic points leave the scene grid along axis %d ([%g, %g] vs grid [%g, %g])", a,
                      io.lo[a], io.hi[a], bv.org[a], bv.hi[a]);
            return fail(PCRL_EINVAL);
        }
    }
    SceneView v = bv;  // same frame: origin, levels, padding, t_eps
    // never a finer top grid than the base's (with_depths)
    set_top(v, std::min(top_cells(bv), std::max(OVERLAY_TOP_CELLS, OVERLAY_CELLS_PER_POINT * n)));
    v.map0 = nullptr;
    for (int l = 0; l + 1 < PCRL_MAX_LEVELS; ++l) v.mask[l] = nullptr;
    for (int i = 0; i < 2; ++i) {
        v.mmask[i] = nullptr;
        v.mbase[i] = nullptr;
    }
    v.top = v.rng = nullptr;
    v.blk = nullptr;
    v.pbox = nullptr;
    v.leaf = nullptr;
    v.surf = nullptr;
    HierBuild hb;
    if ((rc = build_hierarchy(xyz, unit_nrm, label, gid, n, s, false, v, ov->bufs, T, hb))) return fail(rc);
    ov->view = v;
    ov->n_points = n;
    ov->n_entries = hb.n_entries;
    ov->max_label = io.max_label;
    ov->bytes = hb.bytes;
    T.release();
    ov->epoch = S->info.epoch + 1;
    S->info.epoch = ov->epoch;
    S->info.n_dynamic = n;
    S->overlay = n > 0 ? ov : nullptr;
    return PCRL_OK;
}

}  // namespace pcrl

using namespace pcrl;

extern "C" int build_voxels(const float* xyz, const float* normal, const uint32_t* label, int64_t n_points,
                            const PcrlVoxelParams* params, pcrl_stream_t stream, PcrlScene** out) {
    clear_error();
    if (!out) {
        set_error("build_voxels: out is NULL");
        return PCRL_EINVAL;
    }
    *out = nullptr;
    PcrlScene* S = new (std::nothrow) PcrlScene();
    if (!S) {
        set_error("build_voxels: host allocation failed");
        return PCRL_ENOMEM;
    }
    int rc = build_impl(xyz, normal, label, n_points, params, (hipStream_t)stream, S);
    if (rc != PCRL_OK) {
        S->bufs.release();
        delete S;
        return rc;
    }
    *out = S;
    return PCRL_OK;
}

extern "C" int update_points(PcrlScene* scene, const uint32_t* ids, const float* xyz, const float* normal,
                             const uint32_t* label, int64_t n, pcrl_stream_t stream) {
    clear_error();
    if (!scene || n < 0 || (n > 0 && (!ids || !xyz || !normal || !label)) || n > (int64_t)0x7FFFFFFF) {
        set_error("update_points: invalid arguments");
        return PCRL_EINVAL;
    }
    return overlay_impl(scene, ids, xyz, normal, label, n, (hipStream_t)stream);
}

extern "C" int scene_info(const PcrlScene* scene, PcrlSceneInfo* out) {
    clear_error();
    if (!scene || !out) {
        set_error("scene_info: NULL argument");
        return PCRL_EINVAL;
    }
    *out = scene->info;
    out->device_bytes += scene->index_bytes;
    if (scene->overlay) out->device_bytes += scene->overlay->bytes;
    return PCRL_OK;
}

extern "C" int scene_leaf_table(const PcrlScene* scene, uint64_t* leaf_key, uint32_t* leaf_begin,
                                uint32_t* leaf_count, uint32_t* entry_point, pcrl_stream_t stream) {
    clear_error();
    if (!scene) {
        set_error("scene_leaf_table: scene is NULL");
        return PCRL_EINVAL;
    }
    hipStream_t s = (hipStream_t)stream;
    const int64_t nl = scene->info.n_leaves;
    const int64_t m = scene->info.n_entries;
    if (leaf_key && nl)
        PCRL_TRY_HIP(hipMemcpyAsync(leaf_key, scene->leaf_key, (size_t)nl * 8, hipMemcpyDeviceToDevice, s));
    if ((leaf_begin || leaf_count) && nl) {
        hipLaunchKernelGGL(k_split_leaf, dim3(blocks_for(nl)), dim3(BUILD_BLOCK), 0, s, scene->leaf_range, nl,
                           leaf_begin, leaf_count);
        PCRL_TRY_HIP(hipGetLastError());
    }
    if (entry_point && m) {
        if (scene->entry_point) {
            PCRL_TRY_HIP(hipMemcpyAsync(entry_point, scene->entry_point, (size_t)m * 4, hipMemcpyDeviceToDevice, s));
        } else {
            // the point id rides in the surfel (x, y, z, id)
            hipLaunchKernelGGL(k_entry_points, dim3(blocks_for(m)), dim3(BUILD_BLOCK), 0, s, scene->view.surf, m,
                               entry_point);
            PCRL_TRY_HIP(hipGetLastError());
        }
    }
    PCRL_TRY_HIP(hipStreamSynchronize(s));
    return PCRL_OK;
}

extern "C" int release_scene(PcrlScene* scene) {
    clear_error();
    if (!scene) return PCRL_OK;
    // launches on any stream may still read the scene (their release does not
    // wait for them), and the build stream may no longer exist: finish all
    // device work, then free on the null stream
    (void)hipDeviceSynchronize();
    scene->overlay.reset();
    scene->bufs.stream = nullptr;
    scene->bufs.release();
    delete scene;
    return PCRL_OK;
}
