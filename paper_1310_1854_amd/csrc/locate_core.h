// locate_core.h -- the cell-location function C(r) (Sect. 2.3) on the device,
// shared by the trace and the serving start passes: the paper's block lists
// and the bucket-grid ring search, per lane or for a point a whole wave
// shares.
#pragma once

#include "vrt_internal.h"

namespace vrt {

// C(r) through the paper's block lists (Sect. 2.3, steps 2-4), for a point
// inside the closed box: the block holding the point, then the nearest site
// among the cells listed for that block (equal distances: the lowest user
// index). The cell holding the point is listed there, so this is the
// nearest site of all. Returns the internal index (-1 for an empty list,
// which a point inside the box cannot meet) and the user index in *uid.
struct LocView {
    double lo[3], hi[3], inv_h[3];
    int32_t dims[3];
    const int32_t *start;   // null: the grid has no block lists
    const int32_t *cells;
    const Site *sites;
};

inline LocView loc_view(const Grid &g)
{
    LocView L;
    for (int a = 0; a < 3; ++a) {
        L.lo[a] = g.box[a];
        L.hi[a] = g.box[a + 3];
        L.inv_h[a] = g.loc_inv_h[a];
        L.dims[a] = g.loc_dims[a];
    }
    L.start = g.loc_start;
    L.cells = g.loc_cells;
    L.sites = g.sites;
    return L;
}

// STOP_AT_SITE: the search ends at a site the point coincides with (no
// other is as near), and takes the list four entries per round, their
// indices and sites loaded together (the minimum does not depend on the
// order the entries are seen in); the one-at-a-time loop of the other
// instance holds fewer registers in the kernels that inline it.
template <bool STOP_AT_SITE = false>
__device__ __forceinline__ int32_t nearest_in_blocks(const LocView &L, const double q[3], int32_t *uid)
{
    int b[3];
    for (int a = 0; a < 3; ++a) b[a] = bucket_coord(q[a], L.lo[a], L.inv_h[a], L.dims[a]);
    const int64_t k = ((int64_t)b[0] * L.dims[1] + b[1]) * L.dims[2] + b[2];
    double best = __builtin_huge_val();
    int32_t best_u = -1, best_m = -1;
    auto visit = [&](int32_t m, const Site &p) {
        const double dx = q[0] - p.x, dy = q[1] - p.y, dz = q[2] - p.z;
        const double d2 = dx * dx + dy * dy + dz * dz;
        const int32_t u = (int32_t)p.uid;
        if (d2 < best || (d2 == best && u < best_u)) {
            best = d2;
            best_u = u;
            best_m = m;
        }
        return dx == 0.0 && dy == 0.0 && dz == 0.0;
    };
    const int s0 = L.start[k], s1 = L.start[k + 1];
    if constexpr (STOP_AT_SITE) {
#ifndef VRT_LOC_BATCH
#define VRT_LOC_BATCH 4
#endif
        constexpr int kBatch = VRT_LOC_BATCH;
        for (int s = s0; s < s1; s += kBatch) {
            int32_t m[kBatch];
            Site p[kBatch];
#pragma unroll
            for (int j = 0; j < kBatch; ++j) m[j] = (s + j < s1) ? L.cells[s + j] : -1;
#pragma unroll
            for (int j = 0; j < kBatch; ++j)
                if (m[j] >= 0) p[j] = L.sites[m[j]];
            bool at_site = false;
#pragma unroll
            for (int j = 0; j < kBatch; ++j)
                if (m[j] >= 0) at_site |= visit(m[j], p[j]);
            if (at_site) break;
        }
    } else {
        for (int s = s0; s < s1; ++s) {
            const int32_t m = L.cells[s];
            visit(m, L.sites[m]);
        }
    }
    *uid = best_u;
    return best_m;
}

// The same search by W lanes for one point that they share (a whole wave, or
// an aligned group of 16): the lanes take the list in turn, then the best
// (distance, user index) is reduced across them. Returns the internal index
// on every lane.
template <int W = 64>
__device__ __forceinline__ int32_t nearest_in_blocks_wave(const LocView &L, const double q[3])
{
    int b[3];
    for (int a = 0; a < 3; ++a) b[a] = bucket_coord(q[a], L.lo[a], L.inv_h[a], L.dims[a]);
    const int64_t k = ((int64_t)b[0] * L.dims[1] + b[1]) * L.dims[2] + b[2];
    double best = __builtin_huge_val();
    int32_t best_u = 0x7fffffff, best_m = -1;
    for (int s = L.start[k] + (int)(threadIdx.x & (W - 1)); s < L.start[k + 1]; s += W) {
        const int32_t m = L.cells[s];
        const Site p = L.sites[m];
        const double dx = q[0] - p.x, dy = q[1] - p.y, dz = q[2] - p.z;
        const double d2 = dx * dx + dy * dy + dz * dz;
        const int32_t u = (int32_t)p.uid;
        if (d2 < best || (d2 == best && u < best_u)) {
            best = d2;
            best_u = u;
            best_m = m;
        }
    }
    for (int off = W / 2; off > 0; off >>= 1) {
        const double ob = __shfl_xor(best, off, 64);
        const int32_t ou = __shfl_xor(best_u, off, 64);
        const int32_t om = __shfl_xor(best_m, off, 64);
        if (ob < best || (ob == best && ou < best_u)) {
            best = ob;
            best_u = ou;
            best_m = om;
        }
    }
    return best_m;
}

// nearest_site for a point that W lanes share: the sites of each bucket are
// split over them, and after each shell the lanes agree
// on the lexicographic minimum of (squared distance, user index). The
// shells visited, the distances and the minimum are those of nearest_site.
template <int W = 64>
__device__ inline int32_t nearest_site_wave(const BucketGridView &g, const double q[3], int32_t *uid_out)
{
    const int lane = threadIdx.x & (W - 1);
    int b[3];
    for (int a = 0; a < 3; ++a) b[a] = bucket_coord(q[a], g.lo[a], g.inv_h[a], g.dims[a]);
    double best = 1e308 * 10.0;
    int32_t best_i = -1;
    int32_t best_u = 0x7fffffff;
    for (int r = 0;; ++r) {
        for_shell(g, b, r, [&](int bk) {
            const int s0 = g.start[bk], s1 = g.start[bk + 1];
            for (int s = s0 + lane; s < s1; s += W) {
                const Site p = g.items[s];
                const double dx = q[0] - p.x, dy = q[1] - p.y, dz = q[2] - p.z;
                const double d = dx * dx + dy * dy + dz * dz;
                const int32_t idx = (int32_t)(p.uid & 0xffffffff);
                const int32_t uid = (int32_t)(p.uid >> 32);
                if (d < best || (d == best && uid < best_u)) {
                    best = d;
                    best_i = idx;
                    best_u = uid;
                }
            }
        });
        for (int off = W / 2; off > 0; off >>= 1) {
            const double ob = __shfl_xor(best, off, 64);
            const int32_t ou = __shfl_xor(best_u, off, 64);
            const int32_t oi = __shfl_xor(best_i, off, 64);
            if (ob < best || (ob == best && ou < best_u)) {
                best = ob;
                best_u = ou;
                best_i = oi;
            }
        }
        const double lb = shell_bound(g, q, b, r);
        if (lb < 0.0) break;
        const double lb2 = lb * lb * (1.0 - 1e-12);
        if (best < lb2) break;
    }
    if (uid_out) *uid_out = best_u;
    return best_i;
}

// The nearest site by a walk along the neighbour table.
struct WalkView {
    const Slot *blk64;      // FP64 cell blocks
    const int32_t *blk64_off;
    const int32_t *seed;
    int32_t levels;
    double lo[3], hi[3], scale;
    double sure;            // 2e-11 of the box diagonal
};

inline WalkView walk_view(const Grid &g)
{
    WalkView V;
    V.blk64 = g.blk64;
    V.blk64_off = g.blk64_off;
    V.seed = g.seed;
    V.levels = g.seed_levels;
    double d2 = 0.0;
    for (int a = 0; a < 3; ++a) {
        V.lo[a] = g.box[a];
        V.hi[a] = g.box[a + 3];
        d2 += (g.box[a + 3] - g.box[a]) * (g.box[a + 3] - g.box[a]);
    }
    V.scale = g.key_scale;
    V.sure = 2e-11 * sqrt(d2);
    return V;
}

// C(r) by a walk: from a site near q (the first one of the smallest occupied
// octree cube around it) to whichever neighbour is nearest to q, until none
// is nearer than the cell's own site. That site is the nearest of all when q
// lies inside the cell by a margin that covers the rounding of the distances
// and of the table: for every neighbour, d_j^2 - d_m^2 -- twice |n_j| times
// the distance of q from the bisector -- exceeds |n_j| (2e-9 d_m + 2e-11 of
// the box diagonal), and |n_j| exceeds 1e-5 d_m. (A ball around q of more
// than the table's own tolerance then lies in the cell, so no other site's
// bisector comes nearer, and none of them is so close to the cell's site
// that the computed distances could not tell them apart: the neighbours'
// bisectors leave a ball of 5e-6 d_m around it.) So is a site that q coincides
// with. Returns -1 when the margin is not there (on or next to a boundary, as
// lattice points are): the caller then searches the ball around q that the last
// site lies on, r2 being its squared distance. The user index goes to *uid.
__device__ __forceinline__ int32_t walk_to_site(const WalkView &V, const double q[3], int32_t *uid, double &r2)
{
    const uint32_t key = hilbert_key(key_coord(q[0], V.lo[0], V.scale), key_coord(q[1], V.lo[1], V.scale),
                                     key_coord(q[2], V.lo[2], V.scale));
    int32_t m = -1;
    for (int l = V.levels; m < 0 && l > 0; --l) m = V.seed[seed_base(l) + (key >> (30 - 3 * l))];
    int32_t b = V.blk64_off[m < 0 ? 0 : m];
    for (int step = 0; step < 128; ++step) {
        const Slot *B = V.blk64 + b;
        const double2 s0 = *reinterpret_cast<const double2 *>(B);
        const double2 s1 = *reinterpret_cast<const double2 *>(B + 1);
        const int4 s2 = *reinterpret_cast<const int4 *>(B + 2);
        const int n = s2.z;
        const double ex = q[0] - s0.x, ey = q[1] - s0.y, ez = q[2] - s1.x;
        const double d2m = ex * ex + ey * ey + ez * ez;
        r2 = d2m;
        if (d2m == 0.0) {
            *uid = s2.x;
            return s2.y;
        }
        const double c = 2e-9 * sqrt(d2m) + V.sure, c2 = c * c;
        double best = d2m;
        int w = -1;
        bool sure = true;
#pragma unroll
        for (int a = 0; a < 3; ++a) sure &= (q[a] - V.lo[a] > c) & (V.hi[a] - q[a] > c);
        const double2 *rec = reinterpret_cast<const double2 *>(B + kHdrSlots);
        for (int e0 = 0; e0 < n; e0 += 4) {   // 4 sites are 6 aligned 16-byte loads; past the row end masked
            double p[12];
#pragma unroll
            for (int u = 0; u < 6; ++u) {
                const double2 x = rec[3 * e0 / 2 + u];
                p[2 * u] = x.x;
                p[2 * u + 1] = x.y;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const double dx = q[0] - p[3 * u], dy = q[1] - p[3 * u + 1], dz = q[2] - p[3 * u + 2];
                const double d2 = dx * dx + dy * dy + dz * dz;
                const double nx = p[3 * u] - s0.x, ny = p[3 * u + 1] - s0.y, nz = p[3 * u + 2] - s1.x;
                const double n2 = nx * nx + ny * ny + nz * nz;
                const bool in = e0 + u < n;
                const double gap = d2 - d2m;
                sure &= !in | ((gap > 0.0) & (gap * gap > n2 * c2) & (n2 > 1e-10 * d2m));
                const bool t = in & (d2 < best);
                best = t ? d2 : best;
                w = t ? e0 + u : w;
            }
        }
        if (w < 0) {
            *uid = s2.x;
            return sure ? s2.y : -1;
        }
        b = reinterpret_cast<const int32_t *>(reinterpret_cast<const double *>(rec) + 3 * n)[w];
    }
    return -1;
}

// The start cell of the ray on each lane, whose path starts at q (ok: the
// ray has a path; else -1): through the block lists when the grid has them
// (a point they cannot place falls back to the ring search), else the ring
// search; one cooperative search when all 64 lanes of the wave share the
// point (a point source), else one per lane. Every lane of the wave must
// call it. STOP_AT_SITE: a search ends at a site the point coincides with
// (rays that start at sites), which costs the calling kernel registers.
template <bool STOP_AT_SITE = true>
__device__ __forceinline__ int32_t start_cell(const BucketGridView &grid, const LocView &L, const double q[3], bool ok)
{
    const double q0 = __shfl(q[0], 0, 64), q1 = __shfl(q[1], 0, 64), q2 = __shfl(q[2], 0, 64);
    const bool same = ok && q[0] == q0 && q[1] == q1 && q[2] == q2;
    const bool shared = __ballot(true) == ~0ull && __ballot(same) == ~0ull;
    int32_t m = -1, uid;
    if (L.start) {
        if (shared) m = nearest_in_blocks_wave(L, q);
        else if (ok) m = nearest_in_blocks<STOP_AT_SITE>(L, q, &uid);
        if (ok && m < 0) m = nearest_site<STOP_AT_SITE>(grid, q, nullptr);   // empty list: not in the box
    } else if (shared) {
        m = nearest_site_wave(grid, q, nullptr);
    } else if (ok) {
        m = nearest_site<STOP_AT_SITE>(grid, q, nullptr);
    }
    return ok ? m : -1;
}

}  // namespace vrt
