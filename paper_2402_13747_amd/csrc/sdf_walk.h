// sdf_walk.h -- the per-lane leaf walk of the implicit-surface kernels
// (sdf.hip): hierarchical DDA in leaf coordinates over the level-0 map, the
// occupancy bricks and their skip structures, one leaf at a time in ray order.
// The structures it reads beside the scene's own (child bases, boxes, skip
// radii, dense cell table) are built with the scene's own-point index.
#pragma once

#include "internal.h"

namespace pcrl {

// Level-indexed constants for a per-lane level index.  The values are
// selected arithmetically after loading all NL of them: a select between
// loads of argument fields would become a pointer select into the argument
// struct and keep the struct in scratch memory.
template <int NL>
__device__ __forceinline__ int span_at(const SceneView& v, int lvl) {
    int s = 0;
#pragma unroll
    for (int i = 0; i < NL; ++i) s += v.span[i] * (int)(lvl == i);
    return s;
}

template <int NL>
__device__ __forceinline__ uint64_t mspan_at(const SceneView& v, int lvl) {
    uint64_t m = 0;
#pragma unroll
    for (int i = 0; i < NL; ++i) m += v.mspan[i] * (uint64_t)(lvl == i);
    return m;
}

// Box word that no child lies outside of (lo 0, hi 31 on every axis): the
// value used where a brick has no box.
constexpr uint32_t NO_BOX = (31u << 15) | (31u << 20) | (31u << 25);

// Descend from level 0 to level TO (< nlev) for leaf cell c.  Returns the
// level at which the path is empty, or TO + 1 when the level-TO node exists
// (its index in `node`).  Quotients c / span[i] use the precomputed magics.
// `box` receives the occupied-children box of the brick that holds the
// empty cell (empty at level i >= 1: the level-(i-1) brick), or of the
// level-TO node's own brick when the path exists (TO < nlev - 1); NO_BOX
// where there is none.  The box of a brick is loaded with its mask word.
template <int TO>
__device__ __forceinline__ int descend(const SceneView& v, const int c[3], uint32_t& node, int& skip0,
                                       uint32_t& box) {
    int p[3] = {span_div(c[0], v.mspan[0]), span_div(c[1], v.mspan[0]), span_div(c[2], v.mspan[0])};
    const size_t i0 = (size_t)p[0] + (size_t)v.dim0[0] * ((size_t)p[1] + (size_t)v.dim0[1] * p[2]);
    // the level-0 node and the cell's skip radius are loaded together
    const int32_t n0 = v.map0[i0];
    const int d0 = v.dist0 ? (int)v.dist0[i0] : 1;
    box = NO_BOX;
    if (n0 < 0 || (uint32_t)n0 >= v.nn[0]) {
        skip0 = d0;
        return 0;
    }
    uint32_t n = (uint32_t)n0;
#pragma unroll
    for (int i = 1; i <= TO; ++i) {
        const int q[3] = {span_div(c[0], v.mspan[i]), span_div(c[1], v.mspan[i]), span_div(c[2], v.mspan[i])};
        const int r = v.ratio[i - 1];
        const int loc = (q[0] - r * p[0]) + r * ((q[1] - r * p[1]) + r * (q[2] - r * p[2]));
        const size_t wi = (size_t)n * v.nw[i - 1] + (loc >> 6);
        const uint64_t w = v.mask[i - 1][wi];
        const uint32_t bx = v.baabb[i - 1] ? v.baabb[i - 1][n] : NO_BOX;
        const uint64_t bit = uint64_t(1) << (loc & 63);
        if (!(w & bit)) {
            box = bx;
            return i;
        }
        n = v.base[i - 1][wi] + (uint32_t)__popcll(w & (bit - 1));
        if (n >= v.nn[i]) return i;
        p[0] = q[0];
        p[1] = q[1];
        p[2] = q[2];
    }
    node = n;
    if (v.baabb[TO]) box = v.baabb[TO][n];
    return TO + 1;
}

// DDA state of one lane's segment.
struct Seg {
    float inv[3];   // 1 / d (0 on axes the ray does not move along)
    int c[3];       // current leaf cell
    int cq[3];      // parent cell of the cached descent
    int cres;       // cached descent result
    int cskip0;     // cached skip radius of an empty level-0 cell (cres == 0)
    uint32_t cnode; // cached parent node
    uint32_t cbox;  // cached box word: of the parent node's brick (cres > P), or of the brick holding
                    // the empty cell (0 < cres <= P)
    int it;         // DDA steps taken
    int oct_shift;  // 4 x the ray's direction octant (bit a: component a negative)
};

__device__ __forceinline__ int dir_step(float x) { return x > 0.f ? 1 : (x < 0.f ? -1 : 0); }

// Start a segment from o along d: clip to the grid and find the first cell.
// Returns false when the ray misses the grid.
__device__ __forceinline__ bool seg_begin(const SceneView& v, const float o[3], const float d[3], Seg& S) {
    float t0 = 0.f, t1 = INFINITY;
    // slab test; both faces are read on every path (a choice between two
    // argument fields would be turned into a pointer select into the argument
    // struct, which then stays in scratch memory)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float lo_a = v.org[a], hi_a = v.hi[a];
        if (d[a] != 0.f) {
            S.inv[a] = 1.0f / d[a];
            const float ta = (lo_a - o[a]) * S.inv[a], tb = (hi_a - o[a]) * S.inv[a];
            t0 = fmaxf(t0, fminf(ta, tb));
            t1 = fminf(t1, fmaxf(ta, tb));
        } else {
            S.inv[a] = 0.f;
            if (o[a] < lo_a || o[a] > hi_a) t1 = -1.f;
        }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int ci = (int)floorf((o[a] + t0 * d[a] - v.org[a]) * v.inv_h);
        S.c[a] = min(max(ci, 0), v.dim[a] - 1);
        S.cq[a] = -1;
    }
    S.cres = 0;
    S.cskip0 = 1;
    S.cbox = NO_BOX;
    S.oct_shift = 4 * ((d[0] < 0.f ? 1 : 0) | (d[1] < 0.f ? 2 : 0) | (d[2] < 0.f ? 4 : 0));
    S.cnode = 0;
    S.it = 0;
    return t0 <= t1;
}

// Whether local child coordinates (x, y, z) of a brick lie outside its box word.
__device__ __forceinline__ bool box_outside(uint32_t box, int x, int y, int z) {
    return x < (int)(box & 31u) || y < (int)((box >> 5) & 31u) || z < (int)((box >> 10) & 31u) ||
           x > (int)((box >> 15) & 31u) || y > (int)((box >> 20) & 31u) || z > (int)((box >> 25) & 31u);
}

// What the DDA found at the current cell: an occupied leaf (lvl == NL, its
// node and entry range) or an empty cell of level lvl with the empty region
// around it that the ray may skip.
struct DdaCell {
    uint32_t node;
    uint2 range;    // entries of an occupied leaf
    int skip;       // > 1: an empty cube of 2 skip - 1 units centred on the unit holding c
    int oct;        // > 1: an empty box of oct leaves from c along the ray's octant; -1: an empty cell
                    // of level lvl whose brick's occupied-children box is `node` (a box word)
    int unit;       // edge of a skip unit in leaves (1, or a level-0 cell)
    int lvl;        // level of the empty cell containing c, or NL for an occupied leaf
};

__device__ __forceinline__ void dda_cell_reset(DdaCell& k) {
    k.node = 0;
    k.range = make_uint2(0u, 0u);
    k.skip = 1;
    k.oct = 1;
    k.unit = 1;
    k.lvl = 0;
}

// Look the lane's current cell S.c up top-down through a hierarchy of NL
// levels (NL == v.nlev).  Per lane; no cross-lane operations.
template <int NL>
__device__ __forceinline__ void dda_locate(const SceneView& v, Seg& S, DdaCell& k) {
    constexpr int L = NL;
    constexpr int P = L - 2;  // level of the leaves' parents (-1: single-level grid)
    const int* c = S.c;
    if constexpr (P < 0) {
        const size_t i0 = (size_t)c[0] + (size_t)v.dim0[0] * ((size_t)c[1] + (size_t)v.dim0[1] * c[2]);
        const int32_t n0 = v.map0[i0];
        const int d0 = v.dist0 ? (int)v.dist0[i0] : 1;
        k.lvl = (n0 < 0 || (uint32_t)n0 >= v.nn[0]) ? 0 : L;
        k.node = (uint32_t)n0;
        if (k.lvl == 0) k.skip = max(1, d0);
        if (k.lvl == L) {
            k.range = v.leaf[k.node];
        }
    } else {
        // the descent from level 0 runs only when the parent cell changes
        const int q[3] = {span_div(c[0], v.mspan[P]), span_div(c[1], v.mspan[P]), span_div(c[2], v.mspan[P])};
        if (q[0] != S.cq[0] || q[1] != S.cq[1] || q[2] != S.cq[2]) {
            S.cq[0] = q[0];
            S.cq[1] = q[1];
            S.cq[2] = q[2];
            S.cres = descend<P>(v, c, S.cnode, S.cskip0, S.cbox);
        }
        if (S.cres <= P) {
            k.lvl = S.cres;
            if (k.lvl == 0) {
                // empty level-0 cell: the cube of radius cskip0 - 1 level-0 cells around it is empty
                k.skip = max(1, S.cskip0);
                k.unit = v.span[0];
            } else if (S.cbox != NO_BOX) {
                // empty cell of a brick: the rest of the brick outside its box may be empty too
                k.oct = -1;
                k.node = S.cbox;
            }
        } else if (S.cbox != NO_BOX && !v.cells &&
                   box_outside(S.cbox, c[0] - v.ratio[P] * q[0], c[1] - v.ratio[P] * q[1],
                               c[2] - v.ratio[P] * q[2])) {
            // a leaf outside its parent brick's occupied box: empty, no lookup
            k.lvl = L - 1;
            k.oct = -1;
            k.node = S.cbox;
        } else if (v.cells) {
            // one load: the leaf's entry range, or its skip radius
            const int r = v.ratio[P];
            const int loc = (c[0] - r * q[0]) + r * ((c[1] - r * q[1]) + r * (c[2] - r * q[2]));
            const uint2 cl = v.cells[(size_t)S.cnode * (size_t)(r * r * r) + loc];
            if (cl.y) {
                k.lvl = L;
                k.range = cl;
                k.node = cl.x;
            } else {
                // empty leaf: the box of oct cells from it along the ray's octant is empty
                k.lvl = L - 1;
                k.oct = (int)((cl.x >> S.oct_shift) & 15u);
            }
        } else {
            const int r = v.ratio[P];
            const int loc = (c[0] - r * q[0]) + r * ((c[1] - r * q[1]) + r * (c[2] - r * q[2]));
            const size_t wi = (size_t)S.cnode * v.nw[P] + (loc >> 6);
            // the mask word, the word's child base and the leaf's skip radius are
            // loaded together (one memory round trip); only one of the last two is used
            const uint64_t w = v.mask[P][wi];
            const uint32_t wbase = v.base[P][wi];
            const int ld = v.ldist ? (int)v.ldist[(size_t)S.cnode * (size_t)(r * r * r) + loc] : 1;
            const uint64_t bit = uint64_t(1) << (loc & 63);
            k.lvl = L - 1;
            if (w & bit) {
                k.node = wbase + (uint32_t)__popcll(w & (bit - 1));
                if (k.node < v.nn[L - 1]) {
                    k.lvl = L;
                    k.range = v.leaf[k.node];
                }
            } else {
                // empty leaf: the whole cube of radius skip - 1 around it is empty
                k.skip = max(1, ld);
            }
        }
    }
}

// Move the lane past the cell (or empty region) `k` describes: S.c becomes
// the next cell along the ray, and `te` the distance at which the ray enters
// it.  Clears `walking` when the next cell starts beyond t_stop or the ray
// leaves the grid.  Per lane; no cross-lane operations.
template <int NL>
__device__ __forceinline__ void dda_advance(const SceneView& v, bool& walking, const float o[3], const float d[3],
                                            Seg& S, const DdaCell& k, bool at_leaf, float t_stop, float& te) {
    int* c = S.c;
    const int Sz = at_leaf ? 1 : span_at<NL>(v, k.lvl);
    // An empty cell of a brick with an occupied-children box: when the cell is
    // outside the box along some axes, each such axis a bounds an empty slab
    // of the brick (the brick cut at the box's face on a); the ray crosses the
    // slab that it leaves last in one step.
    // The slab along a ends at the box's near face when the ray moves towards
    // the box, else at the brick's face; the ray leaves the slab at
    // min(that face, T) with T its exit from the whole brick.
    int slab = -1, bs = 0;
    bool below = false;
    if (NL > 1 && k.oct < 0) {
        const int us = span_at<NL>(v, k.lvl);
        bs = span_at<NL>(v, k.lvl - 1);
        const uint64_t um = mspan_at<NL>(v, k.lvl), bm = mspan_at<NL>(v, k.lvl - 1);
        const uint32_t box = k.node;
        float T = INFINITY;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int blo = span_div(c[a], bm) * bs;
            if (d[a] != 0.f) T = fminf(T, ((float)(d[a] > 0.f ? blo + bs : blo) * v.h + v.org[a] - o[a]) * S.inv[a]);
        }
        float best = -INFINITY;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int blo = span_div(c[a], bm) * bs;
            const int lc = span_div(c[a] - blo, um);
            const int alo = (int)((box >> (5 * a)) & 31u), ahi = (int)((box >> (15 + 5 * a)) & 31u);
            float t_a = T;
            if (d[a] > 0.f && lc < alo) t_a = fminf(T, ((float)(blo + alo * us) * v.h + v.org[a] - o[a]) * S.inv[a]);
            if (d[a] < 0.f && lc > ahi)
                t_a = fminf(T, ((float)(blo + (ahi + 1) * us) * v.h + v.org[a] - o[a]) * S.inv[a]);
            if ((lc < alo || lc > ahi) && t_a > best) {
                best = t_a;
                slab = a;
                below = lc < alo;
            }
        }
    }
    // exit of the current cell (size Sz leaves)
    int lo[3], hi[3];
    te = INFINITY;
    int axis = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (slab >= 0) {
            // the brick's range, cut at the box's face along the slab axis
            lo[a] = span_div(c[a], mspan_at<NL>(v, k.lvl - 1)) * bs;
            hi[a] = lo[a] + bs;
            if (a == slab) {
                const int us = span_at<NL>(v, k.lvl);
                const int alo = (int)((k.node >> (5 * a)) & 31u), ahi = (int)((k.node >> (15 + 5 * a)) & 31u);
                if (below)
                    hi[a] = lo[a] + alo * us;
                else
                    lo[a] = lo[a] + (ahi + 1) * us;
            }
        } else if (k.oct > 1) {
            // the octant box (inside its brick)
            lo[a] = d[a] < 0.f ? c[a] - (k.oct - 1) : c[a];
            hi[a] = d[a] < 0.f ? c[a] + 1 : c[a] + k.oct;
        } else if (k.skip > 1) {
            // the skip cube, clipped to the grid (beyond it the ray leaves)
            const int uc = (k.unit == 1) ? c[a] : span_div(c[a], v.mspan[0]);
            lo[a] = max((uc - (k.skip - 1)) * k.unit, 0);
            hi[a] = min((uc + k.skip) * k.unit, v.dim[a]);
        } else {
            lo[a] = (Sz == 1) ? c[a] : span_div(c[a], mspan_at<NL>(v, k.lvl)) * Sz;
            hi[a] = lo[a] + Sz;
        }
        float ta = INFINITY;
        if (d[a] > 0.f)
            ta = ((float)hi[a] * v.h + v.org[a] - o[a]) * S.inv[a];
        else if (d[a] < 0.f)
            ta = ((float)lo[a] * v.h + v.org[a] - o[a]) * S.inv[a];
        if (ta < te) {
            te = ta;
            axis = a;
        }
    }
    // next cell along the exit axis (selects, no dynamic indexing of private arrays)
    int nc = 0, dim_ax = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a)
        if (a == axis) {
            nc = d[a] > 0.f ? hi[a] : lo[a] - 1;
            dim_ax = v.dim[a];
        }
    const int max_iter = v.dim[0] + v.dim[1] + v.dim[2] + 8;
    // no later cell can hold a nearer hit; or the ray leaves the grid
    if (te > t_stop || nc < 0 || nc >= dim_ax || ++S.it >= max_iter) {
        walking = false;
    } else {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            if (a == axis) {
                c[a] = nc;
                continue;
            }
            const int sg = dir_step(d[a]);
            if (sg == 0) continue;
            int j = (int)floorf((o[a] + te * d[a] - v.org[a]) * v.inv_h);
            j = min(max(j, lo[a]), hi[a] - 1);
            j = sg > 0 ? max(j, c[a]) : min(j, c[a]);
            c[a] = j;
        }
    }
}

// ---------------------------------------------------------------------------
// the walk's structures
// ---------------------------------------------------------------------------

constexpr int WALK_BLOCK = 256;

// Box of the occupied children of every brick, in the brick's local child
// coordinates (x + r (y + r z) order of the mask bits): lo x, y, z in bits
// 0-14 and hi x, y, z in bits 15-29, 5 bits each (r <= 32).  Every child
// outside the box is empty, so a ray in such a child crosses the brick's
// empty rest up to the box or the brick's exit in one step.
__global__ void k_brick_aabb(const uint64_t* mask, int64_t n_nodes, int nw, int r, uint32_t* aabb) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n_nodes) return;
    int lo0 = 31, lo1 = 31, lo2 = 31, hi0 = 0, hi1 = 0, hi2 = 0;
    for (int w = 0; w < nw; ++w) {
        uint64_t m = mask[(size_t)p * nw + w];
        while (m) {
            const int loc = 64 * w + __ffsll((long long)m) - 1;
            m &= m - 1;
            const int x = loc % r, y = (loc / r) % r, z = loc / (r * r);
            lo0 = min(lo0, x); lo1 = min(lo1, y); lo2 = min(lo2, z);
            hi0 = max(hi0, x); hi1 = max(hi1, y); hi2 = max(hi2, z);
        }
    }
    aabb[p] = (uint32_t)lo0 | ((uint32_t)lo1 << 5) | ((uint32_t)lo2 << 10) | ((uint32_t)hi0 << 15) |
              ((uint32_t)hi1 << 20) | ((uint32_t)hi2 << 25);
}

// Empty-space skip radius of every leaf cell of an occupied parent brick
// (r^3 cells, r <= 16): R = 0 for an occupied leaf; otherwise the largest k
// such that the cube of cells within Chebyshev distance k - 1 is empty and
// inside the brick.  This is the per-voxel march distance of Section 2.2.4
// (the longest per-axis distance to the closest voxel with content), limited
// to the brick.  The cells within Chebyshev distance k of an occupied cell
// are the occupancy dilated k times by the 3 x 3 x 3 cube, and the dilation
// is separable: with the brick held as r^2 rows of r bits (row y + r z, bit
// x), one step ORs each row with its shifts along x, then with its y and z
// neighbour rows.  A cell first reached at step k is at distance k; the
// border limits every radius to at most (r - 1) / 2 + 1, so that many steps
// suffice.  One wave per brick (rows and distances in the wave's LDS).
// RC > 0: the ratio is the compile-time constant RC (index arithmetic by
// constants); RC = 0: the runtime r.
constexpr int BDIST_RMAX = 16;

__device__ __forceinline__ void walk_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int RC>
__global__ __launch_bounds__(WALK_BLOCK) void k_brick_dist(const uint64_t* mask, int nw, int r_rt, int64_t n_bricks,
                                                            uint8_t* dist) {
    __shared__ uint32_t rows_s[WALK_BLOCK / 64][2][BDIST_RMAX * BDIST_RMAX];
    __shared__ uint8_t d_s[WALK_BLOCK / 64][BDIST_RMAX * BDIST_RMAX * BDIST_RMAX];
    const int r = RC > 0 ? RC : r_rt;
    const int n2 = r * r, n3 = n2 * r;
    const int w = threadIdx.x >> 6;
    const int lane = (int)lane_id();
    uint32_t* cur = rows_s[w][0];
    uint32_t* tmp = rows_s[w][1];
    uint8_t* D = d_s[w];
    const uint32_t full = (1u << r) - 1u;
    // whole waves go on or end: no block-wide barrier in here
    for (int64_t P = (int64_t)blockIdx.x * (WALK_BLOCK / 64) + w; P < n_bricks; P += (int64_t)gridDim.x * (WALK_BLOCK / 64)) {
        // row j holds bits [r j, r j + r) of the brick's mask
        for (int j = lane; j < n2; j += 64) {
            const int b0 = r * j;
            const uint64_t* m = mask + (size_t)P * nw + (b0 >> 6);
            uint64_t bits = m[0] >> (b0 & 63);
            if ((b0 & 63) + r > 64) bits |= m[1] << (64 - (b0 & 63));
            cur[j] = (uint32_t)bits & full;
        }
        walk_wave_sync();
        for (int c = lane; c < n3; c += 64) D[c] = ((cur[c / r] >> (c % r)) & 1u) ? 0 : 255;
        const int K = (r - 1) / 2 + 1;
        for (int k = 1; k <= K; ++k) {
            // along x, then y
            for (int j = lane; j < n2; j += 64) {
                const int y = j % r;
                const uint32_t a = cur[j];
                uint32_t t = a | (a << 1) | (a >> 1);
                if (y > 0) {
                    const uint32_t b = cur[j - 1];
                    t |= b | (b << 1) | (b >> 1);
                }
                if (y < r - 1) {
                    const uint32_t b = cur[j + 1];
                    t |= b | (b << 1) | (b >> 1);
                }
                tmp[j] = t & full;
            }
            walk_wave_sync();
            // along z; the cells reached now are at distance k
            for (int j = lane; j < n2; j += 64) {
                const int z = j / r;
                uint32_t t = tmp[j];
                if (z > 0) t |= tmp[j - r];
                if (z < r - 1) t |= tmp[j + r];
                uint32_t nb = t & ~cur[j];
                while (nb) {
                    const int x = __ffs(nb) - 1;
                    nb &= nb - 1u;
                    D[x + r * j] = (uint8_t)k;
                }
                cur[j] = t;
            }
            walk_wave_sync();
        }
        for (int c = lane; c < n3; c += 64) {
            const int x = c % r, y = (c / r) % r, z = c / n2;
            const int db = min(min(min(x, r - 1 - x), min(y, r - 1 - y)), min(z, r - 1 - z));
            dist[P * n3 + c] = (uint8_t)min((int)D[c], db + 1);
        }
        walk_wave_sync();
    }
}

// Empty-space skip radii of the level-0 grid: for every cell the Chebyshev
// distance (in cells, at most DIST0_CAP + 1) to the nearest occupied cell, so
// the cube of radius d - 1 around an empty cell holds no occupied cell.  The
// same march distance as inside the bricks, one level up.  Separable: one
// pass per axis of out(c) = min over |t| <= DIST0_CAP of max(|t|, in(c + t e)),
// starting from 0 (occupied) / 255 (empty).  A window that misses the
// nearest occupied cell only lowers the result (conservative).
constexpr int DIST0_CAP = 15;

// Largest dense cell table built: the table pays off while it stays resident
// in the 256 MB last-level (MALL) cache; a larger one (3.3 GB for a 20M-point
// street canyon) turns every step into an HBM round trip.  Beyond it the walk
// reads the bricks' masks.
constexpr int64_t CELL_TABLE_MAX_BYTES = (int64_t)256 << 20;

__global__ void k_dist0_pass(const int32_t* map0, const uint8_t* in, uint8_t* out, int dx, int dy, int dz, int axis) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t n = (int64_t)dx * dy * dz;
    if (c >= n) return;
    const int x = (int)(c % dx), y = (int)((c / dx) % dy), z = (int)(c / ((int64_t)dx * dy));
    const int pos = axis == 0 ? x : (axis == 1 ? y : z);
    const int len = axis == 0 ? dx : (axis == 1 ? dy : dz);
    const int64_t stride = axis == 0 ? 1 : (axis == 1 ? dx : (int64_t)dx * dy);
    int m = 255;
    const int t0 = max(-DIST0_CAP, -pos), t1 = min(DIST0_CAP, len - 1 - pos);
    for (int t = t0; t <= t1; ++t) {
        const int64_t q = c + t * stride;
        const int a = map0 ? (map0[q] >= 0 ? 0 : 255) : (int)in[q];
        m = min(m, max(abs(t), a));
    }
    out[c] = (uint8_t)min(m, DIST0_CAP + 1);
}

// Dense cell table of the leaves' parent bricks: one 8-byte load per DDA
// step gives an occupied leaf's entry range, or, for an empty leaf, its skip
// radii per direction octant.  Radius s of octant (sx, sy, sz) (bit a set:
// the ray's component a is negative) means the box of s x s x s cells that
// starts at the cell and extends along the octant's signs is empty and inside
// the brick; a ray whose direction lies in that octant crosses the box in one
// step.  s is the octant-restricted Chebyshev distance to the nearest
// occupied cell, capped by the brick's far faces and by 15 (4 bits per
// octant, 8 octants in the first word).
// Computed on bit rows (the r <= 16 cells of a brick row along x in one
// 16-bit word), per octant: E_1 = empty cells; E_{s+1}(c) = AND of E_s over the
// 8 cells c + delta, delta in {0, 1}^3 along the octant's signs (a box of s + 1
// is the union of 8 boxes of s), cells outside the brick counting as not
// empty.  The radius of a cell is the number of s <= 15 with E_s(c), kept as a
// 4-bit counter in bit planes.
constexpr int OCT_ITEMS = 8;  // (octant, row) items per thread: 8 * r^2 <= OCT_ITEMS * WALK_BLOCK for r <= 16

__global__ __launch_bounds__(WALK_BLOCK) void k_brick_cells(const uint64_t* mask, const uint32_t* base,
                                                            const uint2* leaf, int nw, int r, uint2* cells) {
    extern __shared__ uint16_t rows[];  // [2][8][r^2]: E_s and E_{s+1} per octant and row; then the radii
    __shared__ uint64_t wmask[64];      // the brick's occupancy words (nw <= 64 for r <= 16)
    const int r2 = r * r, n3 = r2 * r;
    const int items = 8 * r2;
    const uint32_t full = (1u << r) - 1u;
    const size_t P = blockIdx.x;
    uint16_t* Ecur = rows;
    uint16_t* Enext = rows + items;
    for (int k = threadIdx.x; k < nw; k += WALK_BLOCK) wmask[k] = mask[P * nw + k];
    __syncthreads();
    // E_1: empty cells of every row, the same for all octants
    for (int row = threadIdx.x; row < r2; row += WALK_BLOCK) {
        uint32_t e = 0;
        for (int x = 0; x < r; ++x) {
            const int c = x + r * row;
            if (!((wmask[c >> 6] >> (c & 63)) & 1ull)) e |= 1u << x;
        }
        for (int o = 0; o < 8; ++o) Ecur[o * r2 + row] = (uint16_t)e;
    }
    __syncthreads();
    uint16_t plane[OCT_ITEMS][4];
    for (int k = 0; k < OCT_ITEMS; ++k)
        for (int b = 0; b < 4; ++b) plane[k][b] = 0;
    for (int sz = 1; sz <= 15; ++sz) {
        int any = 0;  // some E_{s+1} is not empty
        for (int k = 0; k < OCT_ITEMS; ++k) {
            const int it = threadIdx.x + k * WALK_BLOCK;
            if (it >= items) break;
            const int o = it / r2, row = it % r2;
            const uint32_t e = Ecur[it];
            // count this s (4-bit ripple add of the bits of E_s)
            uint32_t carry = e;
            for (int b = 0; b < 4; ++b) {
                const uint32_t pb = plane[k][b];
                plane[k][b] = (uint16_t)(pb ^ carry);
                carry &= pb;
            }
            if (sz == 15) continue;
            const int y = row % r, z = row / r;
            const int sy = (o & 2) ? -1 : 1, szn = (o & 4) ? -1 : 1;
            const bool negx = (o & 1) != 0;
            const uint16_t* Eo = Ecur + (size_t)o * r2;
            auto get = [&](int yy, int zz) -> uint32_t {
                if (yy < 0 || yy >= r || zz < 0 || zz >= r) return 0u;
                const uint32_t v = Eo[yy + r * zz];
                const uint32_t sh = negx ? ((v << 1) & full) : (v >> 1);  // the neighbour along x
                return v & sh;
            };
            const uint16_t en = (uint16_t)(get(y, z) & get(y + sy, z) & get(y, z + szn) & get(y + sy, z + szn));
            Enext[it] = en;
            any |= en;
        }
        // once every E_{s+1} is empty, no later size counts anything
        if (!__syncthreads_or(any)) break;
        uint16_t* t = Ecur;
        Ecur = Enext;
        Enext = t;
    }
    // radii packed per cell (octant o in bits 4o..4o+3), written with the occupied leaves' ranges
    __syncthreads();
    uint32_t* packed = reinterpret_cast<uint32_t*>(rows + 2 * items);  // [n3]
    for (int c = threadIdx.x; c < n3; c += WALK_BLOCK) packed[c] = 0u;
    __syncthreads();
    for (int k = 0; k < OCT_ITEMS; ++k) {
        const int it = threadIdx.x + k * WALK_BLOCK;
        if (it >= items) break;
        const int o = it / r2, row = it % r2;
        for (int x = 0; x < r; ++x) {
            const uint32_t n = ((plane[k][0] >> x) & 1u) | (((plane[k][1] >> x) & 1u) << 1) |
                               (((plane[k][2] >> x) & 1u) << 2) | (((plane[k][3] >> x) & 1u) << 3);
            if (n) atomicOr(&packed[x + r * row], n << (4 * o));
        }
    }
    __syncthreads();
    for (int c = threadIdx.x; c < n3; c += WALK_BLOCK) {
        const size_t i = P * (size_t)n3 + c;
        const uint64_t w = wmask[c >> 6];
        const uint64_t bit = uint64_t(1) << (c & 63);
        if (w & bit)
            cells[i] = leaf[base[P * nw + (c >> 6)] + (uint32_t)__popcll(w & (bit - 1))];
        else
            cells[i] = make_uint2(packed[c], 0u);
    }
}

}  // namespace pcrl
