// sdf.hip -- ray intersection with the implicit surface of Eq. 1 (paper,
// Section 2.2.1 "Intersections"): the signed distance
//   f(x) = (x - p(x)) . n(x),
// p and n the weighted averages of the positions and normals of the points
// within h of x (weights (1 - |x - q|^2 / h^2)^4; n normalised), is marched
// along the ray: for every occupied leaf the ray crosses, a line segment one
// leaf diagonal long is centred on the projection onto the ray of the centre
// of the box around the leaf's own points (points whose centre lies in the
// leaf); from its near end the march moves by |f(s_i)| and stops at a sample
// with |f| <= eps, or between two samples of opposite sign (at the zero of
// the linear interpolation), or at the segment's far end, or after max_steps
// evaluations.  Where no point lies within h, f is undefined: the march moves
// by h / 2 and compares no sign across that sample.  The ray's intersection is
// the nearest over the leaves; its normal is n at the final sample.
//
// Lane = ray.  The leaves come from a hierarchical DDA (sdf_walk.h), walked per
// lane; the walk stops once the next cell starts more than 1.5 leaf diagonals
// beyond the nearest intersection found (no later leaf's segment starts before
// that).  Every lane walks to its next sample, then the wave evaluates f for
// all of them.  The neighbours of x are the points of the 27 leaves around x's
// leaf (h is at most 0.98 leaf edges); each point is listed once, in the leaf
// that holds its centre, so the leaves of a row along x lie next to each other
// and a sample reads at most 9 such runs (18 across bricks).
#include "sdf_walk.h"
#include "trace_core.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace pcrl {

constexpr int SDF_BLOCK = 64;  // one wave per block: the lanes finish unevenly, small blocks refill the CUs sooner
constexpr int64_t SDF_ORDER_MIN = 65536;  // rays from which a call sorts them into a coherent order

struct SdfArgs {
    SceneView v;           // the scene with its leaf-walk structures
    const float* o;        // [n][3]
    const float* d;        // [n][3]
    const float* tr;       // [n][2] (t_lo, t_hi), or null for (0, inf)
    const uint32_t* order; // null, or lane -> ray (a coherent order of the rays)
    const uint32_t* oscan; // [n_entries + 1] own entries before each entry of the hierarchy
    const float4* own;     // own entries (each point once, in the leaf of its centre, leaf order): pairs of
                           // (position, id bits) and (unit normal, label bits)
    const float4* lbox;    // [n_points] at the first own entry of a leaf: centre of the box around its own points
    const uint32_t* first; // [n_leaves + 1] own entries before each leaf
    const uint32_t* cells; // own entries before each cell: [parents][r^3 + 1], or [cells + 1] without parents
    uint32_t n;
    int32_t max_steps;
    float h2;              // h^2
    float rh2;             // 1 / h2
    float hl2;             // (h / leaf edge + 1e-3)^2: leaves farther than this from x hold no neighbour
    float half_h;          // step over an undefined sample
    float eps;
    float half_diam;       // half the segment length (half a leaf diagonal)
    float reach;           // 1.5 leaf diagonals and a rounding margin
    int32_t empty;         // the scene holds no point
    float* t;              // [n]
    float* pt;             // [n][3]
    float* nrm;            // [n][3]
    int32_t* cell;         // [n][3] or null
    unsigned long long* stats;  // null, or [2]: evaluations of f, entries read
    // rays left to the tail kernel (one wave each)
    uint32_t budget;       // samples of one segment after which a lane leaves its ray to it
    uint32_t tail_cap;     // most of them; further rays stay with their lanes
    uint32_t leaves;       // leaves handed out at first (then four times as many, up to 64)
    uint32_t* tail;        // their ray ids
    uint32_t* tail_cnt;    // [0] their number, [1] the next to be taken
    float4* tail_ray;      // launches: per ray (o, L), (d, t_lo)
    uint32_t* tail_b;      // launches: its segment
};

// a . b with the fused form written out (results must not depend on the
// compiler's choice).
__device__ __forceinline__ float dot3(float ax, float ay, float az, float bx, float by, float bz) {
    return fmaf(az, bz, fmaf(ax, bx, ay * by));
}

// The kernel's arguments (its first parameter is, or starts with, a SdfArgs),
// read again where they are needed: holding all of them through the march
// spilled 150 scalar registers.
typedef const SdfArgs __attribute__((address_space(4)))* SdfArgsPtr;
__device__ __forceinline__ const SdfArgs& reread_sdf() {
    uint32_t zero;
    asm volatile("s_mov_b32 %0, 0" : "=s"(zero));  // unknown to the compiler: the loads stay behind it
    const char __attribute__((address_space(4)))* p =
        (const char __attribute__((address_space(4)))*)__builtin_amdgcn_kernarg_segment_ptr() + zero;
    return *(const SdfArgs*)(SdfArgsPtr)p;
}

constexpr int SDF_RUNS = 18;  // (y, z) rows x the two bricks a row may cross
typedef uint2 SdfRuns[SDF_RUNS][64];

// Own entries before the position p of brick `node` (p < r^3): those of the
// leaves before it.
__device__ __forceinline__ uint32_t own_before(const SdfArgs& a, int P, uint32_t node, uint32_t p) {
    const size_t w = (size_t)node * a.v.nw[P] + (p >> 6);
    return a.first[a.v.base[P][w] + (uint32_t)__popcll(a.v.mask[P][w] & ((uint64_t(1) << (p & 63u)) - 1ull))];
}

// The runs of own entries of the up to 27 leaves around x that may hold a
// point within h, in the order of the leaves (x fastest, then y, z): run s of
// this lane in runs[s][lane] for every bit s of the result, [first, end).
// NL voxel levels; FAST: bricks from the dense top grid and per-cell prefixes
// (one load each); else by descent and the bricks' masks (scenes whose
// prefixes would be too large).  The leaves' parents hold at least two leaves
// an axis (build_walk), so three cells next to each other lie in at most two.
template <int NL, bool FAST>
__device__ __forceinline__ uint32_t sdf_runs(const float x[3], SdfRuns& runs, uint32_t& reads) {
    constexpr int P = NL - 2;
    const SdfArgs& a = reread_sdf();
    const SceneView& v = a.v;
    const uint32_t lane = lane_id();
    int lc[3], ql[3], qh[3];   // x's cell; parents of the cells below and above it per axis
    float g[3][3];             // squared distance (leaf edges) from x to the cells below, at and above
    bool in[3][3];
    const int r = P < 0 ? 1 : v.ratio[P < 0 ? 0 : P];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float u = (x[k] - v.org[k]) * v.inv_h;
        const float f = floorf(u), fr = u - f;
        lc[k] = (int)f;
        g[k][0] = fr * fr;
        g[k][1] = 0.f;
        g[k][2] = (1.f - fr) * (1.f - fr);
#pragma unroll
        for (int d = 0; d < 3; ++d) in[k][d] = lc[k] + d - 1 >= 0 && lc[k] + d - 1 < v.dim[k];
        if (P >= 0) {
            ql[k] = (int)floorf(fmaf(f - 1.f, v.pinv, v.phalf));
            qh[k] = (int)floorf(fmaf(f + 1.f, v.pinv, v.phalf));
        }
    }
    uint32_t found = 0;
    // per (z, y): the cells along x within reach
    auto reach = [&](int dz, int dy, int& x0, int& x1) -> bool {
        const float gyz = g[2][dz] + g[1][dy];
        const bool c = in[0][1] && gyz < a.hl2;
        const bool lo = in[0][0] && gyz + g[0][0] < a.hl2, hi = in[0][2] && gyz + g[0][2] < a.hl2;
        x0 = lo ? -1 : (c ? 0 : 1);
        x1 = hi ? 1 : (c ? 0 : -1);
        return in[2][dz] && in[1][dy] && (lo || c || hi);
    };
    if constexpr (P < 0) {
        uint2 e[9];
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            int x0, x1;
            e[q] = make_uint2(0u, 0u);
            if (!reach(q / 3, q % 3, x0, x1)) continue;
            const size_t p = (size_t)(lc[0] + x0) +
                             (size_t)v.dim[0] * ((size_t)(lc[1] + q % 3 - 1) + (size_t)v.dim[1] * (lc[2] + q / 3 - 1));
            e[q] = make_uint2(a.cells[p], a.cells[p + (x1 - x0 + 1)]);
        }
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            if (e[q].x < e[q].y) {
                runs[2 * q][lane] = e[q];
                found |= 1u << (2 * q);
                reads += e[q].y - e[q].x;
            }
        }
    } else {
        // the up to eight bricks around x
        int32_t node[2][2][2];
#pragma unroll
        for (int iz = 0; iz < 2; ++iz)
#pragma unroll
            for (int iy = 0; iy < 2; ++iy)
#pragma unroll
                for (int ix = 0; ix < 2; ++ix) {
                    const int q[3] = {ix ? qh[0] : ql[0], iy ? qh[1] : ql[1], iz ? qh[2] : ql[2]};
                    int32_t n = -1;
                    if (FAST) {
                        if (q[0] >= 0 && q[1] >= 0 && q[2] >= 0 && q[0] < v.tdim[0] && q[1] < v.tdim[1] &&
                            q[2] < v.tdim[2])
                            n = (int32_t)v.top[(size_t)q[0] + (size_t)v.tdim[0] * (q[1] + v.tdim[1] * q[2])].x;
                    } else {
                        const int c[3] = {q[0] * r, q[1] * r, q[2] * r};
                        uint32_t m = 0, box;
                        int skip;
                        if (q[0] >= 0 && q[1] >= 0 && q[2] >= 0 && c[0] < v.dim[0] && c[1] < v.dim[1] &&
                            c[2] < v.dim[2] && descend<P>(v, c, m, skip, box) == P + 1)
                            n = (int32_t)m;
                    }
                    node[iz][iy][ix] = n;
                }
        // runs of the rows' parts in the lower and (where a row crosses into it) the upper brick along x
        const int bx = qh[0] * r - lc[0];  // the first cell (relative to x's) of the upper brick
        const bool two = qh[0] != ql[0];
        auto part_runs = [&](auto part_c, int32_t n00, int32_t n01, int32_t n10, int32_t n11) {
            constexpr int part = decltype(part_c)::value;
            uint2 e[9];
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                const int dz = q / 3, dy = q % 3;
                int x0, x1;
                e[q] = make_uint2(0u, 0u);
                if (!reach(dz, dy, x0, x1)) continue;
                const int cz = lc[2] + dz - 1, cy = lc[1] + dy - 1;
                const bool hz = cz >= qh[2] * r, hy = cy >= qh[1] * r;
                const int32_t ny = hy ? n01 : n00, nz = hy ? n11 : n10, n = hz ? nz : ny;
                if (two) {
                    if (part == 0) x1 = min(x1, bx - 1);
                    else x0 = max(x0, bx);
                } else if (part == 1) {
                    continue;
                }
                if (n < 0 || x0 > x1) continue;
                const int lz = cz - (hz ? qh[2] : ql[2]) * r, ly = cy - (hy ? qh[1] : ql[1]) * r;
                const int lx = lc[0] + x0 - (part ? qh[0] : ql[0]) * r;
                const uint32_t p = (uint32_t)(lx + r * (ly + r * lz));
                const uint32_t len = (uint32_t)(x1 - x0 + 1);
                if (FAST) {
                    const uint32_t* c = a.cells + (uint64_t)(uint32_t)n * (uint32_t)(r * r * r + 1) + p;
                    e[q] = make_uint2(c[0], c[len]);
                } else {
                    const uint32_t l = p + len - 1;
                    const size_t w = (size_t)n * v.nw[P] + (l >> 6);
                    const uint32_t last = v.base[P][w] + (uint32_t)__popcll(v.mask[P][w] & (~0ull >> (63u - (l & 63u))));
                    e[q] = make_uint2(own_before(a, P, (uint32_t)n, p), a.first[last]);
                }
            }
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                if (e[q].x < e[q].y) {
                    runs[2 * q + part][lane] = e[q];
                    found |= 1u << (2 * q + part);
                    reads += e[q].y - e[q].x;
                }
            }
        };
        part_runs(std::integral_constant<int, 0>{}, node[0][0][0], node[0][1][0], node[1][0][0], node[1][1][0]);
        if (__ballot(two))
            part_runs(std::integral_constant<int, 1>{}, node[0][0][1], node[0][1][1], node[1][0][1], node[1][1][1]);
    }
    return found;
}

// f(x) of Eq. 1 and the unit normal n(x); false where f is undefined.  The
// offset p(x) - x is accumulated relative to x.  Four points (32 bytes each)
// are loaded before any is used.
template <int NL, bool FAST>
__device__ __forceinline__ bool sdf_eval(const float x[3], SdfRuns& runs, float& f, float n[3], uint32_t& reads) {
    const uint32_t lane = lane_id();
    uint32_t todo = sdf_runs<NL, FAST>(x, runs, reads);
    const SdfArgs& a = reread_sdf();
    float sw = 0.f, sp[3] = {0.f, 0.f, 0.f}, sn[3] = {0.f, 0.f, 0.f};
    uint32_t e = 0, end = 0;
    for (;;) {
        if (e >= end) {
            if (!todo) break;
            const uint2 run = runs[__ffs((int)todo) - 1][lane];
            todo &= todo - 1u;
            e = run.x;
            end = run.y;
        }
        float4 Q[4], N[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float4* r = a.own + 2 * (size_t)min(e + k, end - 1u);
            Q[k] = r[0];
            N[k] = r[1];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float ex = Q[k].x - x[0], ey = Q[k].y - x[1], ez = Q[k].z - x[2];
            const float d2 = dot3(ex, ey, ez, ex, ey, ez);
            if (e + k < end && d2 < a.h2) {
                // d2 / h2, correctly rounded (rh2 is the correctly rounded reciprocal)
                const float q = d2 * a.rh2;
                const float u = 1.0f - fmaf(fmaf(-q, a.h2, d2), a.rh2, q);
                const float u2 = u * u, w = u2 * u2;
                sw = fmaf(u2, u2, sw);
                sp[0] = fmaf(ex, w, sp[0]);
                sp[1] = fmaf(ey, w, sp[1]);
                sp[2] = fmaf(ez, w, sp[2]);
                sn[0] = fmaf(w, N[k].x, sn[0]);
                sn[1] = fmaf(w, N[k].y, sn[1]);
                sn[2] = fmaf(w, N[k].z, sn[2]);
            }
        }
        e += 4;
    }
    const float ln = sqrtf(dot3(sn[0], sn[1], sn[2], sn[0], sn[1], sn[2]));
    if (!(sw > 0.f) || !(ln > 0.f)) return false;
    const float inv = 1.0f / ln;
    n[0] = sn[0] * inv;
    n[1] = sn[1] * inv;
    n[2] = sn[2] * inv;
    f = -dot3(sp[0], sp[1], sp[2], n[0], n[1], n[2]) / sw;
    return true;
}

// 1 for each entry of the hierarchy listed in the leaf that holds its point's
// centre (the cell taken in FP32 as everywhere else), else 0.
template <int TD>
__global__ void k_own_flags(SceneView v, uint32_t m, uint32_t* flag) {
    const uint32_t e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= m) return;
    const float4 P = v.surf[2 * (size_t)e];
    const int x = (int)floorf((P.x - v.org[0]) * v.inv_h), y = (int)floorf((P.y - v.org[1]) * v.inv_h),
              z = (int)floorf((P.z - v.org[2]) * v.inv_h);
    uint2 r = make_uint2(0u, 0u);
    if (x >= 0 && y >= 0 && z >= 0 && x < v.dim[0] && y < v.dim[1] && z < v.dim[2]) r = leaf_range<TD>(v, x, y, z);
    flag[e] = r.x <= e && e - r.x < r.y ? 1u : 0u;
}

// Copy the own entries to their compacted slots.
__global__ void k_own_scatter(const float4* surf, const uint32_t* scan, uint32_t m, uint32_t cap,
                              float4* own) {
    const uint32_t e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= m) return;
    const uint32_t j = scan[e];
    if (scan[e + 1] == j || j >= cap) return;
    own[2 * (size_t)j] = surf[2 * (size_t)e];
    own[2 * (size_t)j + 1] = surf[2 * (size_t)e + 1];
}

// Own entries before each leaf, and the centre of the box around each leaf's
// own points (at its first own entry).
__global__ void k_own_leaves(const uint2* leaf, uint32_t n, const uint32_t* scan, const float4* own, uint32_t* first,
                             float4* lbox, uint32_t* single, const uint64_t* leaf_key, int key_shift) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint2 r = leaf[i];
    const uint32_t e0 = scan[r.x], e1 = scan[r.x + r.y];
    first[i] = e0;
    if (i == n - 1) first[n] = e1;
    if (single) single[leaf_key[i] >> key_shift] = e1 - e0;
    if (!(e0 < e1)) return;
    float lo0 = INFINITY, lo1 = INFINITY, lo2 = INFINITY, hi0 = -INFINITY, hi1 = -INFINITY, hi2 = -INFINITY;
    for (uint32_t e = e0; e < e1; ++e) {
        const float4 q = own[2 * (size_t)e];
        lo0 = fminf(lo0, q.x);
        lo1 = fminf(lo1, q.y);
        lo2 = fminf(lo2, q.z);
        hi0 = fmaxf(hi0, q.x);
        hi1 = fmaxf(hi1, q.y);
        hi2 = fmaxf(hi2, q.z);
    }
    lbox[e0] = make_float4(0.5f * (lo0 + hi0), 0.5f * (lo1 + hi1), 0.5f * (lo2 + hi2), 0.f);
}

// Own entries before each cell of every leaves' parent ([n3 + 1] per parent).
__global__ void k_own_cells(const uint64_t* mask, const uint32_t* base, const uint32_t* first, int nw, uint32_t n3,
                            uint64_t n, uint32_t* cells) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint64_t P = i / (n3 + 1);
    const uint32_t p = (uint32_t)(i - P * (n3 + 1));
    // the end of a brick is counted from its last cell
    const uint32_t c = min(p, n3 - 1);
    const size_t w = (size_t)P * nw + (c >> 6);
    const uint64_t below = p < n3 ? (uint64_t(1) << (c & 63u)) - 1ull : ~0ull >> (63u - (c & 63u));
    cells[i] = first[base[w] + (uint32_t)__popcll(mask[w] & below)];
}

// 8 bits spread to the even bits of 16.
__device__ __forceinline__ uint32_t spread_bits8(uint32_t x) {
    x &= 0xFFu;
    x = (x | (x << 4)) & 0x0F0Fu;
    x = (x | (x << 2)) & 0x3333u;
    x = (x | (x << 1)) & 0x5555u;
    return x;
}

// Coherence key of a ray: Morton code of its origin on a 16^3 grid over the
// scene (12 bits) above the Morton code of its direction's cell on a 256 x 256
// octahedral grid (16 bits).  Sorting by it puts rays that start close
// together in close directions into the same waves, which then march the same
// leaves (shared cache lines, similar step counts).  The octahedral map only
// needs the direction's signs and ratios, so d need not be normalised.
__device__ __forceinline__ uint64_t coherence_key(const float o[3], const float d[3], float3 lo, float3 scale) {
    float u = 0.f, w = 0.f;
    octahedral(d[0], d[1], d[2], u, w);
    const uint32_t dk = spread_bits8(cell_of(u, 256)) | (spread_bits8(cell_of(w, 256)) << 1);
    const uint32_t cx = (uint32_t)fminf(fmaxf((o[0] - lo.x) * scale.x, 0.f), 15.f);
    const uint32_t cy = (uint32_t)fminf(fmaxf((o[1] - lo.y) * scale.y, 0.f), 15.f);
    const uint32_t cz = (uint32_t)fminf(fmaxf((o[2] - lo.z) * scale.z, 0.f), 15.f);
    const uint32_t m = spread_bits4x3(cx) | (spread_bits4x3(cy) << 1) | (spread_bits4x3(cz) << 2);
    return ((uint64_t)m << 16) | dk;
}

__global__ void k_sdf_keys(const float* o, const float* d, uint32_t n, float3 lo, float3 scale, uint64_t* keys,
                           uint32_t* idx) {
    const uint32_t j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    const size_t j3 = 3 * (size_t)j;
    const float oj[3] = {o[j3], o[j3 + 1], o[j3 + 2]};
    const float dj[3] = {d[j3], d[j3 + 1], d[j3 + 2]};
    keys[j] = coherence_key(oj, dj, lo, scale);
    idx[j] = j;
}

// Id and label of the point nearest to x among those within h (smallest
// distance, then smallest id); false if none.
template <int NL, bool FAST>
__device__ __forceinline__ bool nearest_own(const float x[3], SdfRuns& runs, uint32_t& id, uint32_t& label) {
    const uint32_t lane = lane_id();
    uint32_t reads = 0;
    uint32_t todo = sdf_runs<NL, FAST>(x, runs, reads);
    const SdfArgs& a = reread_sdf();
    float bd = a.h2;
    uint32_t best = 0;
    bool found = false;
    while (todo) {
        const uint2 run = runs[__ffs((int)todo) - 1][lane];
        todo &= todo - 1u;
        for (uint32_t e = run.x; e < run.y; ++e) {
            const float4 Q = a.own[2 * (size_t)e];
            const float ex = Q.x - x[0], ey = Q.y - x[1], ez = Q.z - x[2];
            const float d2 = dot3(ex, ey, ez, ex, ey, ez);
            const uint32_t pid = __float_as_uint(Q.w);
            if (d2 < bd || (d2 == bd && found && pid < id)) {
                bd = d2;
                id = pid;
                best = e;
                found = true;
            }
        }
    }
    if (found) label = __float_as_uint(a.own[2 * (size_t)best + 1].w);
    return found;
}

// One lane's march: the leaf walk, the march of the current leaf, and the
// nearest intersection so far.
struct SdfMarch {
    Seg S;
    float t_in;           // where the ray enters the current cell
    float best, bn[3];
    int bc[3];
    // the current leaf's march
    float t, tb, fp, tp;
    int s;
    bool in_leaf, shared, prev, stop;
    // Every leaf whose segment starts at or before t_lo marches from t_lo: the
    // same samples, cut at different far ends.  One shared march serves them
    // all: a leaf whose far end it has already passed, or after it found an
    // intersection or stopped (step limit, nothing nearer possible), adds
    // nothing; a leaf reaching further resumes it.  Exact: the nearest over
    // these leaves is unchanged.
    float c_t, c_fp, c_tp, c_tb;
    int c_s;
    bool c_prev, c_done;
};

// Start the march of the ray (o, d) from t_lo; false when it meets no cell.
__device__ __forceinline__ bool march_begin(SdfMarch& M, const float o[3], const float d[3], float t_lo, float t_hi) {
    const SdfArgs& a = reread_sdf();
    const SceneView& v = a.v;
    M.best = INFINITY;
    M.bn[0] = M.bn[1] = M.bn[2] = 0.f;
    M.bc[0] = M.bc[1] = M.bc[2] = -1;
    M.in_leaf = false;
    M.c_t = t_lo;
    M.c_fp = M.c_tp = 0.f;
    M.c_tb = -INFINITY;
    M.c_s = 0;
    M.c_prev = M.c_done = false;
    M.t_in = 0.f;
    if (a.empty || !(t_lo <= t_hi) || !seg_begin(v, o, d, M.S)) return false;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        float tf = -INFINITY;
        if (d[ax] > 0.f) tf = (fmaf((float)M.S.c[ax], v.h, v.org[ax]) - o[ax]) * M.S.inv[ax];
        else if (d[ax] < 0.f) tf = (fmaf((float)(M.S.c[ax] + 1), v.h, v.org[ax]) - o[ax]) * M.S.inv[ax];
        M.t_in = fmaxf(M.t_in, tf);
    }
    return true;
}

// Move a lane on to its next sample (at M.t) or to the end of its walk
// (`walking` false): one step of the leaf walk or one turn of the leaf's
// march.  Returns true when a sample is to be evaluated.
template <int NL>
__device__ __forceinline__ bool march_next(const SdfArgs& a, SdfMarch& M, bool& walking, const float o[3],
                                           const float d[3], float t_lo, float t_hi, uint32_t& reads) {
    const SceneView& v = a.v;
    DdaCell k;
    dda_cell_reset(k);
    bool at_leaf = true;
    if (!M.in_leaf) {
        dda_locate<NL>(v, M.S, k);
        at_leaf = k.lvl == NL;
        if (at_leaf && M.t_in <= t_hi) {
            const uint32_t o0 = a.oscan[k.range.x], o1 = a.oscan[k.range.x + k.range.y];
            if (o0 < o1) {
                reads += o1 - o0;
                const float4 c = a.lbox[o0];
                const float tc = dot3(c.x - o[0], c.y - o[1], c.z - o[2], d[0], d[1], d[2]);
                M.in_leaf = true;
                M.stop = false;
                M.shared = tc - a.half_diam <= t_lo;
                M.t = fmaxf(tc - a.half_diam, t_lo);
                M.tb = fminf(tc + a.half_diam, t_hi);
                M.fp = M.tp = 0.f;
                M.prev = false;
                M.s = 0;
                if (M.shared) {
                    const bool old = M.c_done || M.tb <= M.c_tb;  // nothing new from this leaf
                    M.s = old ? a.max_steps : M.c_s;
                    M.t = M.c_t;
                    M.fp = M.c_fp;
                    M.tp = M.c_tp;
                    M.prev = M.c_prev;
                }
            }
        }
    }
    if (M.in_leaf) {
        if (!M.stop && M.s < a.max_steps && M.t <= M.tb) {
            // every later result of this leaf lies at or beyond t
            if (!(M.t >= M.best && !(M.prev && M.tp < M.best))) return true;
            M.stop = true;
        }
        if (M.shared && !M.c_done && M.tb > M.c_tb) {
            M.c_t = M.t;
            M.c_fp = M.fp;
            M.c_tp = M.tp;
            M.c_prev = M.prev;
            M.c_s = M.s;
            M.c_tb = M.tb;
            M.c_done = M.stop || M.s >= a.max_steps;
        }
        M.in_leaf = false;
    }
    float te;
    dda_advance<NL>(v, walking, o, d, M.S, k, at_leaf, fminf(M.best + a.reach, t_hi), te);
    M.t_in = te;
    return false;
}

// Evaluate f at the lane's sample and move its march on.
template <int NL, bool FAST>
__device__ __forceinline__ void march_sample(SdfMarch& M, SdfRuns& runs, const float o[3], const float d[3],
                                             uint32_t& reads) {
    const float t = M.t;
    const float x[3] = {fmaf(t, d[0], o[0]), fmaf(t, d[1], o[1]), fmaf(t, d[2], o[2])};
    float f, n[3];
    const bool defined = sdf_eval<NL, FAST>(x, runs, f, n, reads);
    const SdfArgs& a = reread_sdf();
    if (!defined) {
        M.prev = false;
        M.t = t + a.half_h;
        ++M.s;
        return;
    }
    float th = t;
    bool found = fabsf(f) <= a.eps;
    if (!found && M.prev && ((f < 0.f) != (M.fp < 0.f))) {
        th = M.tp + (t - M.tp) * M.fp / (M.fp - f);
        found = true;
    }
    if (found) {
        if (th < M.best) {
            M.best = th;
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                M.bn[ax] = n[ax];
                M.bc[ax] = M.S.c[ax];
            }
        }
        M.stop = true;
        return;
    }
    M.prev = true;
    M.fp = f;
    M.tp = t;
    M.t = t + fabsf(f);
    ++M.s;
}

// This lane's slot in the tail list (one atomic per wave).
__device__ __forceinline__ uint32_t tail_slot(uint32_t* cnt) {
    const uint64_t m = __ballot(1);
    const int leader = __ffsll((long long)m) - 1;
    uint32_t first = 0;
    if ((int)lane_id() == leader) first = atomicAdd(cnt, (uint32_t)__popcll(m));
    return __shfl(first, leader, 64) + (uint32_t)__popcll(m & lanemask_lt());
}

__device__ __forceinline__ void sdf_write(const SdfArgs& a, uint32_t i, const float o[3], const float d[3], float best,
                                          const float bn[3], const int bc[3]) {
    const size_t i3 = 3 * (size_t)i;
    a.t[i] = best;
    const bool hit = bc[0] >= 0;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        a.pt[i3 + ax] = hit ? fmaf(best, d[ax], o[ax]) : NAN;
        a.nrm[i3 + ax] = bn[ax];
        if (a.cell) a.cell[i3 + ax] = bc[ax];
    }
}

template <int NL, bool FAST>
__global__ __launch_bounds__(SDF_BLOCK) void k_sdf(SdfArgs a) {
    __shared__ SdfRuns runs;
    const uint32_t lane_ray = blockIdx.x * SDF_BLOCK + threadIdx.x;
    bool in = lane_ray < a.n;
    const uint32_t i = !in ? 0u : a.order ? a.order[lane_ray] : lane_ray;
    const size_t i3 = 3 * (size_t)i, i2 = 2 * (size_t)i;  // n may exceed 2^32 / 3
    const float o[3] = {a.o[i3], a.o[i3 + 1], a.o[i3 + 2]};
    float d[3] = {a.d[i3], a.d[i3 + 1], a.d[i3 + 2]};
    const float t_lo = a.tr ? a.tr[i2] : 0.f;
    const float t_hi = a.tr ? a.tr[i2 + 1] : INFINITY;
    const float len = sqrtf(dot3(d[0], d[1], d[2], d[0], d[1], d[2]));
    const bool ok = in && len > 0.f && isfinite(len) && isfinite(o[0]) && isfinite(o[1]) && isfinite(o[2]);
    uint32_t evals = 0, reads = 0;
    SdfMarch M;
    M.best = INFINITY;
    M.bn[0] = M.bn[1] = M.bn[2] = 0.f;
    M.bc[0] = M.bc[1] = M.bc[2] = -1;
    bool walking = false;
    if (ok) {
        const float il = 1.0f / len;
        d[0] *= il;
        d[1] *= il;
        d[2] *= il;
        walking = march_begin(M, o, d, t_lo, t_hi);
    }
    for (;;) {
        bool want = false;
        {
            const SdfArgs& w = reread_sdf();
            while (walking && !want) want = march_next<NL>(w, M, walking, o, d, t_lo, t_hi, reads);
        }
        if (!__ballot(want)) break;
        if (want) {
            if (evals++ == a.budget) {
                const uint32_t slot = tail_slot(a.tail_cnt);
                if (slot < a.tail_cap) {
                    a.tail[slot] = i;
                    in = walking = false;
                    continue;
                }
            }
            march_sample<NL, FAST>(M, runs, o, d, reads);
        }
    }
    if (!in) return;
    sdf_write(a, i, o, d, M.best, M.bn, M.bc);
    if (a.stats) {
        atomicAdd(&a.stats[0], (unsigned long long)evals);
        atomicAdd(&a.stats[1], (unsigned long long)reads);
    }
}

// A launch whose intersections are those of the implicit surface (launch_rays
// with PCRL_LAUNCH_SDF): one lane per ray runs all its segments.
struct SdfLaunchArgs {
    SdfArgs s;
    const float* tx;
    const float* rx;
    const float* dirs;
    const uint32_t* order;  // null, or lane -> global ray id
    int32_t n_rx;
    int32_t K;
    uint32_t n_rays;
    uint32_t n_total;
    float sig_c;            // rho(u) = sig_c * u
    float4* hist;
    uint4* rec;
    uint32_t rec_cap;
    uint32_t* counters;
    int32_t* hit_id;
    float* hit_t;
};

// Add 1 to counters[b] for each lane active here: one atomic per wave and
// different b (the lanes stand at different segments).
__device__ __forceinline__ void wave_count(uint32_t* counters, int b) {
    for (bool left = true; left;) {
        const int first = __builtin_amdgcn_readfirstlane(b);
        const uint64_t same = __ballot(b == first);  // of the lanes left
        if (b != first) continue;
        if ((int)lane_id() == __ffsll((long long)same) - 1) atomicAdd(&counters[first], (uint32_t)__popcll(same));
        left = false;
    }
}

__device__ __forceinline__ void launch_ray(const SdfLaunchArgs& A, uint32_t g, float o[3], float d[3]) {
    const uint32_t ti = g / A.n_rays, j = g - ti * A.n_rays;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        o[k] = A.tx[3 * ti + k];
        d[k] = A.dirs[3 * (size_t)j + k];
    }
    const float il = 1.0f / sqrtf(dot3(d[0], d[1], d[2], d[0], d[1], d[2]));
    d[0] *= il;
    d[1] *= il;
    d[2] *= il;
}

// End of segment b of ray g at its first intersection (t = best, normal n):
// hit log, receptions, history, and the reflected ray (o, d, L, t_lo).  False
// when the ray ends.  Only lanes with `write` store.
template <int NL, bool FAST>
__device__ __forceinline__ bool segment_end(const SdfLaunchArgs& A, SdfRuns& runs, uint32_t g, int b, float o[3],
                                            float d[3], float& L, float& t_lo, float best, const float n[3], bool hit,
                                            bool write = true) {
    float t = best;
    const float q[3] = {fmaf(t, d[0], o[0]), fmaf(t, d[1], o[1]), fmaf(t, d[2], o[2])};
    uint32_t pid = 0, lab = 0;
    if (hit) hit = nearest_own<NL, FAST>(q, runs, pid, lab);
    if (!hit) t = INFINITY;
    if (A.hit_id && write) {
        const size_t idx = (size_t)g * (A.K + 1) + b;
        A.hit_id[idx] = hit ? (int32_t)pid : -1;
        A.hit_t[idx] = hit ? t : NAN;
    }
    for (int r = 0; r < A.n_rx; ++r) {
        const float vx = A.rx[3 * r] - o[0], vy = A.rx[3 * r + 1] - o[1], vz = A.rx[3 * r + 2] - o[2];
        const float sp = dot3(vx, vy, vz, d[0], d[1], d[2]);
        if (!(sp > 0.f && sp <= t)) continue;
        const float cx = fmaf(-d[0], sp, vx), cy = fmaf(-d[1], sp, vy), cz = fmaf(-d[2], sp, vz);
        const float rho = A.sig_c * (L + sp);
        if (!(dot3(cx, cy, cz, cx, cy, cz) <= rho * rho) || !write) continue;
        const uint32_t slot = atomicAdd(&A.counters[PCRL_CNT_REC(A.K)], 1u);
        if (slot < A.rec_cap) {
            const float lp = L + sqrtf(dot3(vx, vy, vz, vx, vy, vz));
            A.rec[slot] = make_uint4(g, (uint32_t)r | ((uint32_t)b << 16), __float_as_uint(lp),
                                     __float_as_uint(L + sp));
        }
    }
    if (!hit || b >= A.K) return false;
    if (write) A.hist[(size_t)b * A.n_total + g] = make_float4(q[0], q[1], q[2], __uint_as_float(lab));
    L += t;
    const float dn = fmaf(d[2], n[2], fmaf(d[1], n[1], d[0] * n[0])), dn2 = 2.f * dn;
    const float ex = fmaf(-n[0], dn2, d[0]), ey = fmaf(-n[1], dn2, d[1]), ez = fmaf(-n[2], dn2, d[2]);
    const float inv = 1.0f / sqrtf(dot3(ex, ey, ez, ex, ey, ez));
    d[0] = ex * inv;
    d[1] = ey * inv;
    d[2] = ez * inv;
    o[0] = q[0];
    o[1] = q[1];
    o[2] = q[2];
    t_lo = 4.f * A.s.eps / fmaxf(fabsf(dn), 0.05f);
    return true;
}

// Every segment of a ray, as the launcher's bounce kernels do with surfels:
// the segment from o along d ends at the implicit surface's first
// intersection (from t_lo: 0 from the TX, after a reflection 4 eps / |d.n|
// so that the march starts outside the |f| <= eps band it left); the RX
// spheres are tested on [0, t]; at the intersection the ray reflects about
// n(x) and records the label of the nearest point.  A lane goes on to its
// next segment at once, so the wave ends with its longest ray, not with the
// longest of every segment.
template <int NL, bool FAST>
__global__ __launch_bounds__(SDF_BLOCK) void k_sdf_launch(SdfLaunchArgs A) {
    __shared__ SdfRuns runs;
    const uint32_t lane_ray = blockIdx.x * SDF_BLOCK + threadIdx.x;
    bool alive = lane_ray < A.n_total;
    const uint32_t g = !alive ? 0u : A.order ? A.order[lane_ray] : lane_ray;
    const SdfArgs& a = A.s;
    float o[3], d[3];
    launch_ray(A, g, o, d);
    float L = 0.f, t_lo = 0.f;
    uint32_t evals = 0, reads = 0;
    int b = 0;
    SdfMarch M;
    bool walking = false;
    if (alive) {
        wave_count(A.counters, 0);
        walking = march_begin(M, o, d, 0.f, INFINITY);
    }
    for (;;) {
        bool want = false;
        const SdfArgs& w = reread_sdf();
        while (alive && !want) {
            if (walking) {
                want = march_next<NL>(w, M, walking, o, d, t_lo, INFINITY, reads);
                continue;
            }
            if (!segment_end<NL, FAST>(A, runs, g, b, o, d, L, t_lo, M.best, M.bn, M.bc[0] >= 0)) {
                alive = false;
                break;
            }
            evals = 0;
            ++b;
            wave_count(A.counters, b);
            walking = march_begin(M, o, d, t_lo, INFINITY);
        }
        if (!__ballot(want)) break;
        if (want) {
            if (evals++ == a.budget) {
                const uint32_t slot = tail_slot(a.tail_cnt);
                if (slot < a.tail_cap) {
                    a.tail[slot] = g;
                    a.tail_ray[2 * (size_t)slot] = make_float4(o[0], o[1], o[2], L);
                    a.tail_ray[2 * (size_t)slot + 1] = make_float4(d[0], d[1], d[2], t_lo);
                    a.tail_b[slot] = (uint32_t)b;
                    alive = false;
                    continue;
                }
            }
            march_sample<NL, FAST>(M, runs, o, d, reads);
        }
    }
}

// First intersection of one ray found by a whole wave (every lane holds the
// same ray): the walk hands its leaves out to the lanes, `leaves` of them, then
// four times as many, up to 64 at a time, and every lane marches its own.  The nearest over the leaves is the same as
// marching them one after another, the earliest leaf of the walk among equals:
// a march is only ever cut where no nearer result can follow.  Leaves of the
// shared march from t_lo continue each other's samples, so every lane marches
// those alike.
// The walk waits in LDS (`keep`) meanwhile: it is the same in every lane, and
// registers are what the marches lack.
template <int NL, bool FAST>
__device__ __forceinline__ void wave_first_hit(SdfRuns& runs, SdfMarch& keep, const float o[3], const float d[3], float t_lo, float t_hi,
                                               float& best, float bn[3], int bc[3]) {
    const uint32_t lane = lane_id();
    uint32_t reads = 0;  // not counted here
    SdfMarch M;
    bool walking = march_begin(M, o, d, t_lo, t_hi);
    for (uint32_t most = reread_sdf().leaves; walking; most = min(64u, most * 4u)) {
        // hand out leaves
        uint32_t n = 0;
        float jt = 0.f, jtb = -INFINITY;
        int jc[3] = {-1, -1, -1};
        {
            const SdfArgs& a = reread_sdf();
            const SceneView& v = a.v;
            while (walking && n < most) {
                DdaCell k;
                dda_cell_reset(k);
                dda_locate<NL>(v, M.S, k);
                const bool at_leaf = k.lvl == NL;
                if (at_leaf && M.t_in <= t_hi) {
                    const uint32_t o0 = a.oscan[k.range.x], o1 = a.oscan[k.range.x + k.range.y];
                    if (o0 < o1) {
                        const float4 c = a.lbox[o0];
                        const float tc = dot3(c.x - o[0], c.y - o[1], c.z - o[2], d[0], d[1], d[2]);
                        if (tc - a.half_diam <= t_lo) {
                            // a leaf of the shared march: after the leaves handed out before it
                            if (n) break;
                            M.in_leaf = M.shared = true;
                            M.stop = false;
                            M.tb = fminf(tc + a.half_diam, t_hi);
                            M.s = M.c_done || M.tb <= M.c_tb ? a.max_steps : M.c_s;
                            M.t = M.c_t;
                            M.fp = M.c_fp;
                            M.tp = M.c_tp;
                            M.prev = M.c_prev;
                            break;
                        }
                        if (lane == n) {
                            jt = fmaxf(tc - a.half_diam, t_lo);
                            jtb = fminf(tc + a.half_diam, t_hi);
                            jc[0] = M.S.c[0];
                            jc[1] = M.S.c[1];
                            jc[2] = M.S.c[2];
                        }
                        ++n;
                    }
                }
                float te;
                dda_advance<NL>(v, walking, o, d, M.S, k, at_leaf, fminf(M.best + a.reach, t_hi), te);
                M.t_in = te;
            }
        }
        if (M.in_leaf) {
            bool at_sample = true;
            while (at_sample) {
                at_sample = march_next<NL>(reread_sdf(), M, walking, o, d, t_lo, t_hi, reads);
                if (!at_sample) break;  // the leaf is done and the walk one step further
                march_sample<NL, FAST>(M, runs, o, d, reads);
            }
            continue;
        }
        // march the lane's leaf
        const float best0 = M.best;
        keep = M;
        __syncthreads();
        float fp = 0.f, tp = 0.f, th = INFINITY, nn[3] = {0.f, 0.f, 0.f};
        bool prev = false, go = lane < n;
        int s = 0;
        for (;;) {
            const SdfArgs& a = reread_sdf();
            go = go && s < a.max_steps && jt <= jtb && !(jt >= best0 && !(prev && tp < best0));
            if (!__ballot(go)) break;
            if (!go) continue;
            const float x[3] = {fmaf(jt, d[0], o[0]), fmaf(jt, d[1], o[1]), fmaf(jt, d[2], o[2])};
            float f, nv[3];
            ++s;
            if (!sdf_eval<NL, FAST>(x, runs, f, nv, reads)) {
                prev = false;
                jt += reread_sdf().half_h;
                continue;
            }
            bool found = fabsf(f) <= reread_sdf().eps;
            float h = jt;
            if (!found && prev && ((f < 0.f) != (fp < 0.f))) {
                h = tp + (jt - tp) * fp / (fp - f);
                found = true;
            }
            if (found) {
                th = h;
                nn[0] = nv[0];
                nn[1] = nv[1];
                nn[2] = nv[2];
                go = false;
            }
            prev = true;
            fp = f;
            tp = jt;
            jt += fabsf(f);
        }
        __syncthreads();
        M = keep;
        float m = th;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) m = fminf(m, __shfl_xor(m, off, 64));
        if (m < M.best) {
            const int src = __ffsll((long long)__ballot(th == m)) - 1;
            M.best = m;
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                M.bn[ax] = __shfl(nn[ax], src, 64);
                M.bc[ax] = __shfl(jc[ax], src, 64);
            }
        }
    }
    best = M.best;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        bn[ax] = M.bn[ax];
        bc[ax] = M.bc[ax];
    }
}

// The next item of the tail list for this wave, or false when none is left.
__device__ __forceinline__ bool tail_next(const SdfArgs& a, uint32_t& item) {
    uint32_t q = 0;
    if (lane_id() == 0) q = atomicAdd(&a.tail_cnt[1], 1u);
    item = (uint32_t)__builtin_amdgcn_readfirstlane((int)q);
    return item < min(a.tail_cnt[0], a.tail_cap);
}

// The rays left over by k_sdf, or all rays (no list), one wave each.
template <int NL, bool FAST>
__global__ __launch_bounds__(SDF_BLOCK) void k_sdf_tail(SdfArgs a) {
    __shared__ SdfRuns runs;
    __shared__ SdfMarch keep;
    uint32_t item = blockIdx.x;
    for (; a.tail ? tail_next(a, item) : item < a.n; item += gridDim.x) {
        const uint32_t i = a.tail ? a.tail[item] : item;
        const size_t i3 = 3 * (size_t)i, i2 = 2 * (size_t)i;
        const float o[3] = {a.o[i3], a.o[i3 + 1], a.o[i3 + 2]};
        float d[3] = {a.d[i3], a.d[i3 + 1], a.d[i3 + 2]};
        const float t_lo = a.tr ? a.tr[i2] : 0.f;
        const float t_hi = a.tr ? a.tr[i2 + 1] : INFINITY;
        const float len = sqrtf(dot3(d[0], d[1], d[2], d[0], d[1], d[2]));
        const bool ok = len > 0.f && isfinite(len) && isfinite(o[0]) && isfinite(o[1]) && isfinite(o[2]);
        float best = INFINITY, bn[3] = {0.f, 0.f, 0.f};
        int bc[3] = {-1, -1, -1};
        if (ok) {
            const float il = 1.0f / len;
            d[0] *= il;
            d[1] *= il;
            d[2] *= il;
            wave_first_hit<NL, FAST>(runs, keep, o, d, t_lo, t_hi, best, bn, bc);
        }
        if (lane_id() == 0) sdf_write(a, i, o, d, best, bn, bc);
    }
}

// The rays left over by k_sdf_launch, one wave each from the segment they had
// reached.
template <int NL, bool FAST>
__global__ __launch_bounds__(SDF_BLOCK) void k_sdf_launch_tail(SdfLaunchArgs A) {
    __shared__ SdfRuns runs;
    __shared__ SdfMarch keep;
    __shared__ float path;      // L, the ray and its segment, in LDS between the segments' ends
    __shared__ uint32_t at[2];
    const SdfArgs& a = A.s;
    uint32_t item;
    while (tail_next(a, item)) {
        float o[3], d[3], t_lo;
        const float4 O = a.tail_ray[2 * (size_t)item], D = a.tail_ray[2 * (size_t)item + 1];
        o[0] = O.x;
        o[1] = O.y;
        o[2] = O.z;
        d[0] = D.x;
        d[1] = D.y;
        d[2] = D.z;
        t_lo = D.w;
        path = O.w;
        at[0] = a.tail[item];
        at[1] = a.tail_b[item];
        __syncthreads();
        for (;;) {
            float best, bn[3];
            int bc[3];
            wave_first_hit<NL, FAST>(runs, keep, o, d, t_lo, INFINITY, best, bn, bc);
            // every lane ends the segment alike; lane 0 writes
            const uint32_t b = at[1];
            float L = path;
            if (!segment_end<NL, FAST>(A, runs, at[0], (int)b, o, d, L, t_lo, best, bn, bc[0] >= 0, lane_id() == 0)) break;
            __syncthreads();
            path = L;
            at[1] = b + 1u;
            __syncthreads();
            if (lane_id() == 0) atomicAdd(&A.counters[b + 1u], 1u);
        }
        __syncthreads();
    }
}

// Coherence key of global ray g of a launch (its TX and launch direction).
__global__ void k_sdf_launch_keys(const float* tx, const float* dirs, uint32_t n_rays, uint32_t n_total, float3 lo,
                                  float3 scale, uint64_t* keys, uint32_t* idx) {
    const uint32_t g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n_total) return;
    const uint32_t ti = g / n_rays, j = g - ti * n_rays;
    const float o[3] = {tx[3 * ti], tx[3 * ti + 1], tx[3 * ti + 2]};
    const float d[3] = {dirs[3 * (size_t)j], dirs[3 * (size_t)j + 1], dirs[3 * (size_t)j + 2]};
    keys[g] = coherence_key(o, d, lo, scale);
    idx[g] = g;
}

// Samples of one segment after which a lane leaves its ray to the tail kernel
// (bundles of at most SDF_TAIL_ALL rays are its from the start), and room for
// at least so many rays (a sixteenth of larger bundles; the rest stay with
// their lanes).  A lane marches a ray's samples one after another at about
// 20 us each, so a kernel lasts as long as its longest ray: of 500 k rays in a
// 1M-point room the median takes 15 samples, 0.7 % more than 100 and the
// longest, along a wall, 1,122.  A wave on one ray marches 64 of its leaves at
// once, but also leaves behind the first hit.  The 500 k rays take 23.1 ms
// without the tail and 31.5, 11.6, 9.7 and 12.8 ms with a budget of 24, 48, 96
// and 192 (k_sdf 7.0, k_sdf_tail 2.1 ms at 96); a launch of 150 k rays with
// two reflections (400 k points) 36.3, then 44.3, 24.7, 21.5 and 24.1 ms.
// Up to SDF_SOON rays a wave hands four leaves out at first: most of a few rays
// end at one of them.  One ray, mean of 64: 160 us against 208 with 64 leaves
// (294 marched on a lane) in the room, 128 against 151 (218) in a street, 266
// against 341 (237) there with bricks of 40^3 leaves, whose walk is long; in more
// rays, and among the stragglers, the longest one counts, which loses a tenth
// by it.
constexpr uint32_t SDF_BUDGET = 96, SDF_TAIL_ALL = 4096, SDF_TAIL_MIN = 65536, SDF_SOON = 8;

// Waves of the tail kernel: four per SIMD stay resident.
static unsigned tail_waves(uint32_t n) { return std::min<unsigned>(std::max(n, 1u), (unsigned)device_cus() * 16); }

template <int NL, bool FAST>
static void launch_sdf_fast(const SdfArgs& a, hipStream_t s) {
    const unsigned grid = (a.n + SDF_BLOCK - 1) / SDF_BLOCK;
    if (a.tail) hipLaunchKernelGGL((k_sdf<NL, FAST>), dim3(grid), dim3(SDF_BLOCK), 0, s, a);
    hipLaunchKernelGGL((k_sdf_tail<NL, FAST>), dim3(tail_waves(a.n)), dim3(SDF_BLOCK), 0, s, a);
}

template <int NL>
static void launch_sdf_nl(const SdfArgs& a, hipStream_t s) {
    if (NL == 1 || a.cells || a.empty) launch_sdf_fast<NL, true>(a, s);
    else launch_sdf_fast<NL, NL == 1>(a, s);
}

// The tail list of n rays (in T), empty; launches keep their rays' state too.
static int tail_alloc(SdfArgs& a, uint32_t n, bool launch, DevBufs& T, hipStream_t s) {
    // counted runs march every ray on its lane: the counts are those of the serial march
    a.budget = a.stats ? ~0u : n <= SDF_TAIL_ALL ? 0u : SDF_BUDGET;
    a.leaves = n <= SDF_SOON && !launch ? 4u : 64u;
    if (a.budget == 0u && !launch) return PCRL_OK;  // no list: all rays
    a.tail_cap = std::min(n, std::max(n / 16, SDF_TAIL_MIN));
    n = std::max(a.tail_cap, 1u);
    PCRL_TRY(T.alloc(&a.tail_cnt, 2));
    PCRL_TRY(fill_u32(a.tail_cnt, 0u, 2, s));
    PCRL_TRY(T.alloc(&a.tail, (size_t)n));
    if (!launch) return PCRL_OK;
    PCRL_TRY(T.alloc(&a.tail_ray, 2 * (size_t)n));
    return T.alloc(&a.tail_b, (size_t)n);
}

// Largest table of own entries before each cell (4 bytes per leaf cell of
// every leaves' parent); beyond it, in compact scenes, where the parents have
// no dense top grid and where the table finds no memory, a sample's runs are
// found through the bricks' masks (two more dependent loads each).
constexpr int64_t OWN_CELLS_MAX_BYTES = (int64_t)4 << 30;

// The scene's arrays for the kernels (the index is built).
static void own_args(const PcrlScene* S, SdfArgs& a) {
    a.v = S->walk;
    a.oscan = S->own_scan;
    a.own = S->own;
    a.lbox = S->own_box;
    a.first = S->own_first;
    a.cells = S->own_cells;
}

template <int TD>
static void launch_own_flags(const SceneView& v, uint32_t m, uint32_t* flag, hipStream_t s) {
    hipLaunchKernelGGL((k_own_flags<TD>), dim3((unsigned)(((uint64_t)m + 255) / 256)), dim3(256), 0, s, v, m, flag);
}

// The structures of the leaf walk for scene S in its view v, owned by B: child
// bases and boxes of every brick, the leaves' skip radii (a dense cell table
// where it fits, else isotropic radii) and those of the level-0 grid.  A last
// level that divides nothing (ratio 1) is left out: the nodes above it are the
// leaves, one by one in the same order.
static int build_walk(const PcrlScene* S, hipStream_t s, DevBufs& B, SceneView& v) {
    v = S->view;
    while (v.nlev > 1 && v.ratio[v.nlev - 2] == 1) --v.nlev;
    const int L = v.nlev;
    if (L >= 2) {
        v.pinv = 1.0f / (float)v.ratio[L - 2];
        v.phalf = 0.5f / (float)v.ratio[L - 2];
    }
    int rc;
    auto blocks = [](int64_t n, int block) { return dim3((unsigned)std::max<int64_t>(1, (n + block - 1) / block)); };
    for (int l = 0; l + 1 < L; ++l) {
        const int64_t nodes = v.nn[l];
        uint32_t *bs = nullptr, *ab = nullptr;
        if ((rc = B.alloc(&bs, (size_t)nodes * v.nw[l]))) return rc;
        launch_brick_base(v.mask[l], S->first_child[l], nodes, v.nw[l], bs, s);
        v.base[l] = bs;
        if (v.ratio[l] > 32 || nodes == 0) continue;
        if ((rc = B.alloc(&ab, (size_t)nodes))) return rc;
        hipLaunchKernelGGL(k_brick_aabb, blocks(nodes, WALK_BLOCK), dim3(WALK_BLOCK), 0, s, v.mask[l], nodes, v.nw[l],
                           v.ratio[l], ab);
        v.baabb[l] = ab;
    }
    if (L >= 2 && v.nn[L - 2] > 0) {
        const int r = v.ratio[L - 2];
        const int64_t r3 = (int64_t)r * r * r, nb = v.nn[L - 2], n_cells = nb * r3;
        if (!S->compact && r <= 16 && n_cells * 8 <= CELL_TABLE_MAX_BYTES) {
            uint2* cells = nullptr;
            if ((rc = B.alloc(&cells, (size_t)n_cells))) return rc;
            const size_t lds = (size_t)2 * 8 * r * r * 2 + (size_t)r3 * 4;
            hipLaunchKernelGGL(k_brick_cells, dim3((unsigned)nb), dim3(WALK_BLOCK), lds, s, v.mask[L - 2],
                               v.base[L - 2], v.leaf, v.nw[L - 2], r, cells);
            v.cells = cells;
        } else if (r >= 3 && r <= 16) {
            uint8_t* ld = nullptr;
            if ((rc = B.alloc(&ld, (size_t)n_cells))) return rc;
            const dim3 g = blocks(std::min(nb, WAVES_MAX), WALK_BLOCK / 64);
            if (r == 10)
                hipLaunchKernelGGL(k_brick_dist<10>, g, dim3(WALK_BLOCK), 0, s, v.mask[L - 2], v.nw[L - 2], r, nb, ld);
            else if (r == 8)
                hipLaunchKernelGGL(k_brick_dist<8>, g, dim3(WALK_BLOCK), 0, s, v.mask[L - 2], v.nw[L - 2], r, nb, ld);
            else
                hipLaunchKernelGGL(k_brick_dist<0>, g, dim3(WALK_BLOCK), 0, s, v.mask[L - 2], v.nw[L - 2], r, nb, ld);
            v.ldist = ld;
        }
    }
    const int64_t cells0 = (int64_t)v.dim0[0] * v.dim0[1] * v.dim0[2];
    uint8_t *d0 = nullptr, *tmp = nullptr;
    if ((rc = B.alloc(&d0, (size_t)cells0)) || (rc = dalloc((void**)&tmp, (size_t)cells0, s))) return rc;
    const dim3 g0 = blocks(cells0, WALK_BLOCK);
    hipLaunchKernelGGL(k_dist0_pass, g0, dim3(WALK_BLOCK), 0, s, v.map0, (const uint8_t*)nullptr, d0, v.dim0[0],
                       v.dim0[1], v.dim0[2], 0);
    hipLaunchKernelGGL(k_dist0_pass, g0, dim3(WALK_BLOCK), 0, s, (const int32_t*)nullptr, (const uint8_t*)d0, tmp,
                       v.dim0[0], v.dim0[1], v.dim0[2], 1);
    hipLaunchKernelGGL(k_dist0_pass, g0, dim3(WALK_BLOCK), 0, s, (const int32_t*)nullptr, (const uint8_t*)tmp, d0,
                       v.dim0[0], v.dim0[1], v.dim0[2], 2);
    v.dist0 = d0;
    dfree(tmp, s);
    return hipGetLastError() == hipSuccess ? PCRL_OK : PCRL_EHIP;
}

// Every point once, in the leaf that holds its centre (under the scene's
// lock; the caller waits for the stream).
static int own_points(PcrlScene* S, hipStream_t s) {
    if (S->own_scan) return PCRL_OK;
    const SceneView& v = S->view;
    const int64_t m = S->info.n_entries, np = S->info.n_points;
    DevBufs B;  // handed to the scene when complete
    B.stream = s;
    uint32_t* scan = nullptr;
    float4* own = nullptr;
    int rc = B.alloc(&scan, (size_t)m + 1);
    if (!rc) rc = B.alloc(&own, 2 * (size_t)(np > 0 ? np : 1));
    if (!rc) {
        switch (v.depth) {
        case -1: launch_own_flags<-1>(v, (uint32_t)m, scan, s); break;
        case 0: launch_own_flags<0>(v, (uint32_t)m, scan, s); break;
        case 1: launch_own_flags<1>(v, (uint32_t)m, scan, s); break;
        default: launch_own_flags<2>(v, (uint32_t)m, scan, s); break;
        }
        rc = hipGetLastError() == hipSuccess ? scan_u32(scan, scan, m, scan + m, s) : PCRL_EHIP;
    }
    if (!rc) {
        hipLaunchKernelGGL(k_own_scatter, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, s, v.surf, scan,
                           (uint32_t)m, (uint32_t)np, own);
        if (hipGetLastError() != hipSuccess) rc = PCRL_EHIP;
    }
    if (rc) {
        B.release();
        if (rc == PCRL_EHIP) set_error("building the scene's own-point index failed");
        return rc;
    }
    S->bufs.ptrs.insert(S->bufs.ptrs.end(), B.ptrs.begin(), B.ptrs.end());
    S->index_bytes += B.bytes;
    S->own = own;
    S->own_scan = scan;
    return PCRL_OK;
}

int scene_own_index(PcrlScene* S, hipStream_t s) {
    std::lock_guard<std::mutex> lock(S->own_mu);
    if (S->own_scan) return PCRL_OK;
    PCRL_TRY(own_points(S, s));
    PCRL_TRY_HIP(hipStreamSynchronize(s));
    return PCRL_OK;
}

// The implicit surface's index of the scene (the own points, their leaves'
// boxes and prefixes, and the leaf walk), built on the first call (under the
// scene's lock) and kept with the scene.  The build waits for its stream, so
// calls on any stream find the index complete.
static int sdf_index(PcrlScene* S, hipStream_t s) {
    std::lock_guard<std::mutex> lock(S->own_mu);
    if (S->own_first) return PCRL_OK;
    PCRL_TRY(own_points(S, s));
    DevBufs B;  // handed to the scene when complete
    B.stream = s;
    SceneView v{};
    int rc = build_walk(S, s, B, v);
    if (rc) {
        (void)hipStreamSynchronize(s);  // the own points stay
        B.release();
        if (rc == PCRL_EHIP) set_error("sdf_intersect: building the leaf walk failed");
        return rc;
    }
    const uint32_t n_leaves = v.nn[v.nlev - 1];
    const int P = v.nlev - 2;
    const uint32_t n3 = P < 0 ? 0u : (uint32_t)v.ratio[P] * v.ratio[P] * v.ratio[P];
    const int64_t n_cells = P < 0 ? (int64_t)v.dim[0] * v.dim[1] * v.dim[2] + 1 : (int64_t)v.nn[P] * (n3 + 1);
    const int F = std::max(S->view.nlev - 2 - v.depth, 0);  // level of the top grid
    const bool table = P < 0 || (F == P && !S->compact && n_cells * 4 <= OWN_CELLS_MAX_BYTES);
    int key_shift = 0;  // key bits of the levels left out
    for (int l = v.nlev; l < S->view.nlev; ++l) key_shift += v.lbits[l];
    uint32_t *first = nullptr, *cells = nullptr;
    float4* box = nullptr;
    const int64_t np = S->info.n_points;
    rc = B.alloc(&box, (size_t)(np > 0 ? np : 1));
    if (!rc) rc = B.alloc(&first, (size_t)n_leaves + 1);
    if (!rc && table) {
        rc = B.alloc(&cells, (size_t)n_cells);
        if (rc == PCRL_ENOMEM && P >= 0) {
            clear_error();
            cells = nullptr;
            rc = PCRL_OK;
        }
    }
    if (!rc && P < 0) rc = fill_u32(cells, 0u, n_cells, s);
    if (!rc) {
        hipLaunchKernelGGL(k_own_leaves, dim3((n_leaves + 255) / 256), dim3(256), 0, s, v.leaf, n_leaves,
                           (const uint32_t*)S->own_scan, (const float4*)S->own, first, box,
                           P < 0 ? cells : (uint32_t*)nullptr, (const uint64_t*)S->leaf_key, key_shift);
        if (P < 0)
            rc = scan_u32(cells, cells, n_cells, nullptr, s);
        else if (cells)
            hipLaunchKernelGGL(k_own_cells, dim3((unsigned)((n_cells + 255) / 256)), dim3(256), 0, s, v.mask[P],
                               v.base[P], (const uint32_t*)first, v.nw[P], n3, (uint64_t)n_cells, cells);
        if (!rc) rc = hipGetLastError() == hipSuccess && hipStreamSynchronize(s) == hipSuccess ? PCRL_OK : PCRL_EHIP;
    }
    if (rc) {
        (void)hipStreamSynchronize(s);
        B.release();
        if (rc == PCRL_EHIP) set_error("sdf_intersect: building the own-point index failed");
        return rc;
    }
    S->bufs.ptrs.insert(S->bufs.ptrs.end(), B.ptrs.begin(), B.ptrs.end());
    S->index_bytes += B.bytes;
    S->walk = v;
    S->own_box = box;
    S->own_cells = cells;
    S->own_first = first;
    return PCRL_OK;
}

// Defaults of the implicit surface for a scene (h, eps, max_steps as
// sdf_intersect's when its parameters are not given).
static void sdf_defaults(const PcrlScene* scene, SdfArgs& a) {
    const float leaf = scene->view.h;
    const float h = 0.95f * leaf;
    a.max_steps = 64;
    a.h2 = h * h;
    a.rh2 = 1.0f / a.h2;
    a.hl2 = (h / leaf + 1e-3f) * (h / leaf + 1e-3f);
    a.half_h = 0.5f * h;
    a.eps = 1e-3f * leaf;
    const float diag = sqrtf(3.0f) * leaf;
    a.half_diam = 0.5f * diag;
    a.reach = 1.5f * diag * (1.0f + 1e-5f) + 1e-3f * leaf;
    a.empty = scene->info.n_points == 0;
}

template <int NL, bool FAST>
static void launch_sdf_launch_fast(const SdfLaunchArgs& A, hipStream_t s) {
    const unsigned grid = (A.n_total + SDF_BLOCK - 1) / SDF_BLOCK;
    hipLaunchKernelGGL((k_sdf_launch<NL, FAST>), dim3(grid), dim3(SDF_BLOCK), 0, s, A);
    hipLaunchKernelGGL((k_sdf_launch_tail<NL, FAST>), dim3(tail_waves(A.n_total)), dim3(SDF_BLOCK), 0, s, A);
}

template <int NL>
static void launch_sdf_launch_nl(const SdfLaunchArgs& A, hipStream_t s) {
    if (NL == 1 || A.s.cells || A.s.empty) launch_sdf_launch_fast<NL, true>(A, s);
    else launch_sdf_launch_fast<NL, NL == 1>(A, s);
}

int sdf_launch_run(PcrlLaunch* L, const TraceArgs& t) {
    const PcrlScene* scene = L->scene;
    hipStream_t s = L->stream;
    if (L->stats || t.has_ov) {
        set_error("launch_rays: PCRL_LAUNCH_SDF takes no PCRL_LAUNCH_STATS and no scene with dynamic points");
        return PCRL_EINVAL;
    }
    SdfLaunchArgs A{};
    sdf_defaults(scene, A.s);
    if (!A.s.empty) {
        PCRL_TRY(sdf_index(const_cast<PcrlScene*>(scene), s));
        own_args(scene, A.s);
    }
    A.tx = t.tx;
    A.rx = t.rx;
    A.dirs = t.dirs;
    A.n_rx = t.n_rx;
    A.K = t.K;
    A.n_rays = t.n_rays;
    A.n_total = t.n_total;
    A.sig_c = t.sig_c;
    A.hist = t.hist;
    A.rec = t.rec;
    A.rec_cap = t.rec_cap;
    A.counters = t.counters;
    A.hit_id = t.hit_id;
    A.hit_t = t.hit_t;
    if ((L->flags & PCRL_LAUNCH_COHERENT) && !A.s.empty) {
        uint64_t* keys = nullptr;
        uint32_t* idx = nullptr;
        int rc = L->bufs.alloc(&keys, (size_t)A.n_total);
        if (!rc) rc = L->bufs.alloc(&idx, (size_t)A.n_total);
        if (rc) return rc;
        const SceneView& v = scene->view;
        const float3 lo = make_float3(v.org[0], v.org[1], v.org[2]);
        const float3 sc = make_float3(16.f / (v.hi[0] - v.org[0]), 16.f / (v.hi[1] - v.org[1]),
                                      16.f / (v.hi[2] - v.org[2]));
        hipLaunchKernelGGL(k_sdf_launch_keys, dim3((A.n_total + 255) / 256), dim3(256), 0, s, A.tx, A.dirs, A.n_rays,
                           A.n_total, lo, sc, keys, idx);
        PCRL_TRY_HIP(hipGetLastError());
        PCRL_TRY(radix_sort_u64_bits(keys, idx, (int64_t)A.n_total, 0, 28, s));
        A.order = idx;
    }
    PCRL_TRY(tail_alloc(A.s, A.n_total, true, L->bufs, s));
    const bool timing = !L->events.empty();
    if (timing) PCRL_TRY_HIP(hipEventRecord(L->events[0], s));
    switch (A.s.empty ? 1 : A.s.v.nlev) {
    case 1: launch_sdf_launch_nl<1>(A, s); break;
    case 2: launch_sdf_launch_nl<2>(A, s); break;
    case 3: launch_sdf_launch_nl<3>(A, s); break;
    default: launch_sdf_launch_nl<4>(A, s); break;
    }
    PCRL_TRY_HIP(hipGetLastError());
    if (timing) {
        // one kernel runs every segment: its time is reported as bounce 0's
        for (size_t e = 1; e < L->events.size(); ++e) PCRL_TRY_HIP(hipEventRecord(L->events[e], s));
    }
    return PCRL_OK;
}

}  // namespace pcrl

using namespace pcrl;

extern "C" int sdf_intersect(const PcrlScene* scene, const float* o, const float* d, const float* t_range,
                             int64_t n_rays, const PcrlSdfParams* params, float* t, float* point, float* normal,
                             int32_t* leaf_cell, pcrl_stream_t stream) {
    clear_error();
    if (!scene || n_rays < 0 || n_rays >= ((int64_t)1 << 31)) {
        set_error("sdf_intersect: invalid scene or ray count (0 <= n_rays < 2^31)");
        return PCRL_EINVAL;
    }
    if (n_rays > 0 && (!o || !d || !t || !point || !normal)) {
        set_error("sdf_intersect: a ray or output array is NULL");
        return PCRL_EINVAL;
    }
    if (scene->overlay && scene->overlay->n_entries > 0) {
        set_error("sdf_intersect: the scene has dynamic points (update_points); the implicit surface is defined "
                  "over the static points only");
        return PCRL_EINVAL;
    }
    PcrlSdfParams P{};
    if (params) P = *params;
    const float leaf = scene->view.h;
    const float h = P.h > 0.f ? P.h : 0.95f * leaf;
    const float eps = P.eps > 0.f ? P.eps : 1e-3f * leaf;
    const int32_t max_steps = P.max_steps > 0 ? P.max_steps : 64;
    if (!(h <= 0.98f * leaf) || !std::isfinite(eps) || max_steps > (1 << 20) || P.flags != 0) {
        set_error("sdf_intersect: need 0 < h <= 0.98 leaf edges (h %g, leaf %g), a finite eps, max_steps <= 2^20 "
                  "and flags 0", (double)h, (double)leaf);
        return PCRL_EINVAL;
    }
    if (n_rays == 0) return PCRL_OK;
    SdfArgs a{};
    a.o = o;
    a.d = d;
    a.tr = t_range;
    a.n = (uint32_t)n_rays;
    a.max_steps = max_steps;
    a.h2 = h * h;
    a.rh2 = 1.0f / a.h2;
    a.hl2 = (h / leaf + 1e-3f) * (h / leaf + 1e-3f);
    a.half_h = 0.5f * h;
    a.eps = eps;
    const float diag = sqrtf(3.0f) * leaf;
    a.half_diam = 0.5f * diag;
    a.reach = 1.5f * diag * (1.0f + 1e-5f) + 1e-3f * leaf;
    a.empty = scene->info.n_points == 0;
    a.t = t;
    a.pt = point;
    a.nrm = normal;
    a.cell = leaf_cell;
    a.stats = (unsigned long long*)P.stats;
    hipStream_t s = (hipStream_t)stream;
    if (!a.empty) {
        // the index is a cache of the scene's data: building it does not change the scene
        const int rc = sdf_index(const_cast<PcrlScene*>(scene), s);
        if (rc) return rc;
        own_args(scene, a);
    }
    DevBufs T;
    T.stream = s;
    // large batches run in a coherent order (the outputs keep the callers')
    if (n_rays >= SDF_ORDER_MIN && !a.empty) {
        uint64_t* keys = nullptr;
        uint32_t* idx = nullptr;
        int rc = T.alloc(&keys, (size_t)n_rays);
        if (!rc) rc = T.alloc(&idx, (size_t)n_rays);
        if (rc) {
            T.release();
            return rc;
        }
        const SceneView& v = scene->view;
        const float3 lo = make_float3(v.org[0], v.org[1], v.org[2]);
        const float3 sc = make_float3(16.f / (v.hi[0] - v.org[0]), 16.f / (v.hi[1] - v.org[1]),
                                      16.f / (v.hi[2] - v.org[2]));
        hipLaunchKernelGGL(k_sdf_keys, dim3((unsigned)((n_rays + 255) / 256)), dim3(256), 0, s, o, d,
                           (uint32_t)n_rays, lo, sc, keys, idx);
        rc = hipGetLastError() == hipSuccess ? radix_sort_u64_bits(keys, idx, n_rays, 0, 28, s) : PCRL_EHIP;
        if (rc) {
            T.release();
            set_error("sdf_intersect: ordering the rays failed");
            return rc;
        }
        a.order = idx;
    }
    if (const int rc = tail_alloc(a, (uint32_t)n_rays, false, T, s)) {
        T.release();
        return rc;
    }
    switch (a.empty ? 1 : a.v.nlev) {
    case 1: launch_sdf_nl<1>(a, s); break;
    case 2: launch_sdf_nl<2>(a, s); break;
    case 3: launch_sdf_nl<3>(a, s); break;
    default: launch_sdf_nl<4>(a, s); break;
    }
    const bool ok = hipGetLastError() == hipSuccess;
    T.release();  // stream-ordered: the buffers stay valid for the kernel
    if (!ok) {
        set_error("sdf_intersect: kernel launch failed");
        return PCRL_EHIP;
    }
    return PCRL_OK;
}
