// build.hip -- vor_build_grid: the setup phase of the straight-path method
// (Sect. 2.2, setup items 1-3) on the GPU.
//
//  1. validate the sites and give each a 30-bit Hilbert key;
//  2. radix-sort the sites into Hilbert order (internal order);
//  3. bucket the sites into a uniform grid (stable radix sort by bucket);
//  4. per site, clip the box by the bisector half-spaces of nearby sites --
//     its neighbours in Hilbert order first, then every other site nearer
//     than twice the cell's largest vertex radius, found through a tree of
//     bounding boxes over that order; the planes left bounding the cell are
//     its neighbours (Sect. 2.1);
//  5. make the lists symmetric, order each row nearest neighbour first, and
//     lay out the trace records (FP64 sites and FP32 offsets per neighbour,
//     CSR by cell).
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <vector>

#include "../../include/voronoi_rt_diag.h"
#include "clip_wave.h"

using namespace vrt;

namespace {

__global__ void k_validate_keys(const double *__restrict__ sites, int64_t M, BoxArg box, double scale,
                                uint32_t *__restrict__ keys, int32_t *__restrict__ vals, int *__restrict__ err)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= M) return;
    uint32_t c[3];
    bool ok = true;
    for (int a = 0; a < 3; ++a) {
        double x = sites[3 * i + a];
        if (!(x >= box.lo[a] && x <= box.hi[a])) ok = false;   // also rejects NaN
        c[a] = ok ? key_coord(x, box.lo[a], scale) : 0u;
    }
    if (!ok) atomicOr(err, ERR_OUTSIDE);
    keys[i] = hilbert_key(c[0], c[1], c[2]);
    vals[i] = (int32_t)i;
}

// The sites in Hilbert order, and the boxes of their runs of kLeaf (level 0
// of the box tree; the grid covers whole runs).
__global__ void __launch_bounds__(256) k_gather_sites(const double *__restrict__ sites,
                                                      const int32_t *__restrict__ order, int64_t M,
                                                      Site *__restrict__ out, int32_t *__restrict__ perm,
                                                      int32_t *__restrict__ inv_perm, Box6 *__restrict__ leaf)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    Box6 b;
    for (int a = 0; a < 3; ++a) {
        b.lo[a] = __builtin_huge_val();
        b.hi[a] = -__builtin_huge_val();
    }
    if (i < M) {
        const int32_t u = order[i];
        Site s;
        s.x = b.lo[0] = b.hi[0] = sites[3 * (int64_t)u];
        s.y = b.lo[1] = b.hi[1] = sites[3 * (int64_t)u + 1];
        s.z = b.lo[2] = b.hi[2] = sites[3 * (int64_t)u + 2];
        s.uid = u;
        out[i] = s;
        perm[i] = u;
        inv_perm[u] = (int32_t)i;
    }
    for (int a = 0; a < 3; ++a)
        for (int off = kLeaf / 2; off > 0; off >>= 1) {
            b.lo[a] = fmin(b.lo[a], __shfl_xor(b.lo[a], off, 64));
            b.hi[a] = fmax(b.hi[a], __shfl_xor(b.hi[a], off, 64));
        }
    if (i < M && i % kLeaf == 0) leaf[i / kLeaf] = b;
}

// The seed table from the sorted Hilbert keys: the first site of every
// octree cube that has one.
__global__ void k_seeds(const uint32_t *__restrict__ keys, int64_t M, int levels, int32_t *__restrict__ seed)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= M) return;
    const uint32_t key = keys[i], before = i > 0 ? keys[i - 1] : 0u;
    for (int l = levels; l > 0; --l) {
        const int sh = 30 - 3 * l;
        if (i > 0 && key >> sh == before >> sh) break;   // not the first there, nor in the cubes around it
        seed[seed_base(l) + (key >> sh)] = (int32_t)i;
    }
}

// A level of the box tree: box k covers the 64 boxes [64 k, 64 k + 64) below
// (one wave each).
__global__ void __launch_bounds__(64) k_box_level(const Box6 *__restrict__ below, int64_t n, Box6 *__restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * 64 + threadIdx.x;
    Box6 b;
    for (int a = 0; a < 3; ++a) {
        b.lo[a] = __builtin_huge_val();
        b.hi[a] = -__builtin_huge_val();
    }
    if (i < n) b = below[i];
    for (int a = 0; a < 3; ++a) {
        b.lo[a] = wave_min_f64(b.lo[a]);
        b.hi[a] = wave_max_f64(b.hi[a]);
    }
    if (threadIdx.x == 0) out[blockIdx.x] = b;
}

struct GridArg {
    double lo[3];
    double inv_h[3];
    int32_t dims[3];
};

__global__ void k_bucket_keys(const Site *__restrict__ sites, int64_t M, GridArg g, uint32_t *__restrict__ keys,
                              int32_t *__restrict__ vals, int32_t *__restrict__ counts)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= M) return;
    Site s = sites[i];
    int bx = bucket_coord(s.x, g.lo[0], g.inv_h[0], g.dims[0]);
    int by = bucket_coord(s.y, g.lo[1], g.inv_h[1], g.dims[1]);
    int bz = bucket_coord(s.z, g.lo[2], g.inv_h[2], g.dims[2]);
    uint32_t b = (uint32_t)((bz * g.dims[1] + by) * g.dims[0] + bx);
    keys[i] = b;
    vals[i] = (int32_t)i;
    atomicAdd(&counts[b], 1);
}

__global__ void k_bucket_fill(const Site *__restrict__ sites, const int32_t *__restrict__ order, int64_t M,
                              Site *__restrict__ out)
{
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= M) return;
    int32_t i = order[k];
    Site s = sites[i];
    s.uid = (s.uid << 32) | (int64_t)(uint32_t)i;
    out[k] = s;
}

struct ClipArgs {
    const Site *sites;        // internal order
    BoxTree tree;
    BoxArg box;
    int64_t M;
    int32_t *nbr;             // [M * kMaxNbr] first-pass lists
    int32_t *cnt;             // [M]
    uint8_t *walls;           // [M]
    int32_t *retry;           // [M] sites whose cell needs the large capacity
    int32_t *n_retry;
    int32_t *touched;         // [M] sites whose cell goes to the strict order; null: every one
    int32_t *n_touched;
    int32_t *open;            // [M] sites whose cell came out of the strict order as no polyhedron
    int32_t *n_open;
    int *err;
    double *volume;           // [M] cell volumes
    double *bbox;             // [6 M] cell bounding boxes, or null
};

// The result of the clipped cell i (n faces, or -ERR_*), by one lane.
__device__ __forceinline__ void clip_result(const ClipArgs &A, int64_t i, int n, uint32_t walls, double vol)
{
    A.volume[i] = vol;
    if (n == -ERR_CAPACITY) {
        A.retry[atomicAdd(A.n_retry, 1)] = (int32_t)i;
        n = 0;
    } else if (n == -ERR_TOUCH) {
        A.touched[atomicAdd(A.n_touched, 1)] = (int32_t)i;
        n = 0;
    } else if (n == -ERR_OPEN) {
        A.open[atomicAdd(A.n_open, 1)] = (int32_t)i;
        n = 0;
    } else if (n < 0) {
        atomicOr(A.err, -n);
        n = 0;
    }
    A.cnt[i] = n;
    A.walls[i] = (uint8_t)walls;
}

// First pass: one wave per site with a small cell; cells that run out of
// vertices are queued for the large capacity, cells in which a cut passes
// through a vertex (lattices), or which degenerate (no vertex is left, a new
// one is not finite, or they bound no polyhedron), for the strict order. The
// grid is a multiple of kXcds blocks: block b runs on XCD b mod kXcds, and each
// XCD takes one contiguous part of the Hilbert order, so that its L2 holds the
// sites around it.
constexpr int kXcds = 8;
__global__ void __launch_bounds__(64) k_clip(ClipArgs A)
{
    __shared__ WaveCellSmall cell;
    const int64_t i = (int64_t)(blockIdx.x % kXcds) * (gridDim.x / kXcds) + blockIdx.x / kXcds;
    if (i >= A.M) return;
    uint32_t walls = 0;
    double vol = 0.0;
    int n = wclip_site<WaveCellSmall, false>(cell, A.sites, A.M, A.tree, A.box, i, A.nbr + i * kMaxNbr, kMaxNbr, walls,
                                             vol, A.bbox ? A.bbox + 6 * i : nullptr, kCutTol, false);
    if (n == -ERR_DEGENERATE || n == -ERR_OPEN) n = -ERR_TOUCH;
    if (threadIdx.x == 0) clip_result(A, i, n, walls, vol);
}

// The queued cells again, in the strict order; up to 64 sites, every cell (the
// loose order's head start would be all of them). (All of a lattice's are: the
// build of 10^6 sites on a cubic one takes 14.4 ms, on a body-centred one of
// 4x10^5 11.9 ms; with every cell taken nearest first from the start, by rings
// of buckets, 27.6 and 13.4 ms.)
__global__ void __launch_bounds__(64) k_clip_strict(ClipArgs A)
{
    __shared__ WaveCellSmall cell;
    const int64_t i = A.touched ? A.touched[blockIdx.x] : (int)blockIdx.x;
    uint32_t walls = 0;
    double vol = 0.0;
    int n = wclip_site<WaveCellSmall, true>(cell, A.sites, A.M, A.tree, A.box, i, A.nbr + i * kMaxNbr, kMaxNbr, walls, vol,
                                            A.bbox ? A.bbox + 6 * i : nullptr, kCutTol, false);
    if (n == -ERR_DEGENERATE) n = -ERR_OPEN;
    if (threadIdx.x == 0) clip_result(A, i, n, walls, vol);
}

// Those that came out as no polyhedron, with other tolerances (in a kernel of
// its own: the loop costs two of five waves per SIMD).
__global__ void __launch_bounds__(64) k_clip_open(ClipArgs A)
{
    __shared__ WaveCellSmall cell;
    const int64_t i = A.open[blockIdx.x];
    uint32_t walls = 0;
    double vol = 0.0;
    const int n = strict_site(cell, A.sites, A.M, A.tree, A.box, i, A.nbr + i * kMaxNbr, kMaxNbr, walls, vol,
                              A.bbox ? A.bbox + 6 * i : nullptr, 1);
    if (threadIdx.x == 0) clip_result(A, i, n, walls, vol);
}

// The queued sites with large cells (up to 255 planes).
__global__ void __launch_bounds__(64) k_clip_big(ClipArgs A, int32_t *__restrict__ big_nbr, int32_t *__restrict__ slot)
{
    __shared__ WaveCellBig cell;
    const int k = blockIdx.x;
    const int64_t i = A.retry[k];
    uint32_t wm = 0;
    double vol = 0.0;
    int n = strict_site(cell, A.sites, A.M, A.tree, A.box, i, big_nbr + (int64_t)k * kMaxNbrBig, kMaxNbrBig, wm, vol,
                        A.bbox ? A.bbox + 6 * i : nullptr, 0);
    if (threadIdx.x == 0) {
        A.volume[i] = vol;
        slot[i] = k;
        if (n < 0) {
            atomicOr(A.err, -n);
            n = 0;
        }
        A.cnt[i] = n;
        A.walls[i] = (uint8_t)wm;
    }
}

// The paper's locate structure (Sect. 2.3): a regular grid of blocks over
// the box; block k lists every cell whose bounding box overlaps it. The box
// of cell i is widened by 1e-9 of its extent (plus 1e-12 of the domain's)
// on each side, so that rounding in its vertices cannot drop a block the
// cell reaches. Blocks are numbered (x * ny + y) * nz + z.
struct LocArgs {
    const double *bbox;   // [6 M] internal order
    int64_t M;
    double lo[3], inv_h[3], ext[3];
    int32_t dims[3];
};

__device__ __forceinline__ void loc_range(const LocArgs &A, int64_t i, int b0[3], int b1[3])
{
    for (int a = 0; a < 3; ++a) {
        const double lo = A.bbox[6 * i + a], hi = A.bbox[6 * i + a + 3];
        const double m = 1e-9 * (hi - lo) + 1e-12 * A.ext[a];
        b0[a] = bucket_coord(lo - m, A.lo[a], A.inv_h[a], A.dims[a]);
        b1[a] = bucket_coord(hi + m, A.lo[a], A.inv_h[a], A.dims[a]);
    }
}

// One cell per 16 lanes, which share out the blocks of its box, z fastest
// (one cell per lane leaves the wave waiting for its largest box: sparse cells
// next to a dense disc have boxes of thousands of blocks).
constexpr int kRowLanes = 16;
constexpr int kExportLds = 256;   // entries of a row held in LDS to order it
template <class F>
__device__ __forceinline__ int64_t loc_each(const LocArgs &A, int64_t i, F &&f)
{
    int b0[3], b1[3];
    loc_range(A, i, b0, b1);
    const uint32_t nz = (uint32_t)(b1[2] - b0[2] + 1), ny = (uint32_t)(b1[1] - b0[1] + 1);
    const int64_t n = (int64_t)(b1[0] - b0[0] + 1) * ny * nz;
    for (int64_t q = threadIdx.x & (kRowLanes - 1); q < n; q += kRowLanes) {
        const uint32_t u = (uint32_t)(q / nz), z = (uint32_t)(q - (int64_t)u * nz);
        const uint32_t x = u / ny, y = u - x * ny;
        f(((int64_t)(b0[0] + (int)x) * A.dims[1] + b0[1] + (int)y) * A.dims[2] + b0[2] + (int)z);
    }
    return n;
}

__global__ void __launch_bounds__(256) k_loc_count(LocArgs A, int32_t *__restrict__ cnt,
                                                   unsigned long long *__restrict__ total)
{
    __shared__ unsigned long long sum;
    if (threadIdx.x == 0) sum = 0;
    __syncthreads();
    for (int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) / kRowLanes; i < A.M; i += (int64_t)gridDim.x * (256 / kRowLanes)) {
        const int64_t n = loc_each(A, i, [&](int64_t k) { atomicAdd(&cnt[k], 1); });
        if ((threadIdx.x & (kRowLanes - 1)) == 0) atomicAdd(&sum, (unsigned long long)n);
    }
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(total, sum);
}

__global__ void __launch_bounds__(256) k_loc_fill(LocArgs A, const int32_t *__restrict__ start,
                                                  int32_t *__restrict__ cursor, int32_t *__restrict__ cells)
{
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) / kRowLanes;
    if (i < A.M) loc_each(A, i, [&](int64_t k) { cells[start[k] + atomicAdd(&cursor[k], 1)] = (int32_t)i; });
}

// The rows as the clipping left them, each ascending: in the first pass's
// table or, for sites redone with the large capacity (slot[i] >= 0), in
// big_nbr at that slot; or, with col set, complete in CSR at offs[i].x.
struct RowTable {
    const int32_t *nbr;
    const int32_t *cnt;
    const int32_t *slot;
    const int32_t *big_nbr;
    const int32_t *col;
    const int4 *offs;
    __device__ const int32_t *row(int64_t i) const
    {
        if (col) return col + offs[i].x;
        const int k = slot[i];
        return k < 0 ? nbr + i * kMaxNbr : big_nbr + (int64_t)k * kMaxNbrBig;
    }
};

__device__ __forceinline__ bool row_has(const int32_t *__restrict__ row, int n, int32_t x)
{
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (row[mid] < x) lo = mid + 1;
        else hi = mid;
    }
    return lo < n && row[lo] == x;
}

// For every entry i -> j whose reverse is missing (hardly ever: a face at the
// clipping's tolerance), count an extra entry for row j. kRowLanes lanes per
// row.
__global__ void __launch_bounds__(256) k_symm_count(RowTable T, int64_t M, int32_t *__restrict__ extra,
                                                    int32_t *__restrict__ n_missing)
{
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) / kRowLanes;
    if (i >= M) return;
    const int32_t *row = T.row(i);
    const int n = T.cnt[i];
    for (int e = threadIdx.x & (kRowLanes - 1); e < n; e += kRowLanes) {
        const int32_t j = row[e];
        if (!row_has(T.row(j), T.cnt[j], (int32_t)i)) {
            atomicAdd(&extra[j], 1);
            atomicAdd(n_missing, 1);
        }
    }
}

__device__ __forceinline__ int wave_max_int(int v)
{
    for (int off = 32; off > 0; off >>= 1) v = max(v, __shfl_xor(v, off, 64));
    return v;
}

// What each row takes: entries, slots of its FP64 block (the header, then 28
// bytes per neighbour), slots of its compact block (12 bytes per neighbour;
// blocks start on any slot: starting them on 64- or 128-byte lines was
// measured slower), entries of the export (with walls); and the longest row.
__global__ void __launch_bounds__(256) k_row_sizes(const int32_t *__restrict__ cnt, const int32_t *__restrict__ extra,
                                                   const uint8_t *__restrict__ walls, int64_t M,
                                                   int4 *__restrict__ sizes, int *__restrict__ max_row)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int n = 0;
    if (i < M) {
        n = cnt[i] + extra[i];
        sizes[i] = make_int4(n, kHdrSlots + (7 * n + 3) / 4, kHdrSlots + (3 * n + 3) / 4, n + __popc((unsigned)walls[i]));
    }
    const int m = wave_max_int(n);
    if ((threadIdx.x & 63) == 0 && m > __hip_atomic_load(max_row, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMax(max_row, m);
}

// Rows with entries missing: each row to the front of its place in CSR
// (cursor = its length), the missing reverses after it, then sorted.
__global__ void k_copy_rows(RowTable T, int64_t M, int32_t *__restrict__ col, int32_t *__restrict__ cursor)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= M) return;
    const int32_t *row = T.row(i);
    const int n = T.cnt[i], o = T.offs[i].x;
    for (int e = 0; e < n; ++e) col[o + e] = row[e];
    cursor[i] = n;
}

__global__ void k_symm_fill(RowTable T, int64_t M, int32_t *__restrict__ col, int32_t *__restrict__ cursor)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= M) return;
    const int32_t *row = T.row(i);
    for (int e = 0; e < T.cnt[i]; ++e) {
        const int32_t j = row[e];
        if (!row_has(T.row(j), T.cnt[j], (int32_t)i)) col[T.offs[j].x + atomicAdd(&cursor[j], 1)] = (int32_t)i;
    }
}

__global__ void k_row_sort(int32_t *__restrict__ col, const int4 *__restrict__ offs, int64_t M)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= M) return;
    int32_t *row = col + offs[i].x;
    const int n = offs[i + 1].x - offs[i].x;
    for (int a = 1; a < n; ++a) {
        int32_t x = row[a];
        int k = a - 1;
        while (k >= 0 && row[k] > x) {
            row[k + 1] = row[k];
            --k;
        }
        row[k + 1] = x;
    }
}

// The cell blocks, the FP64 records and the FP64 blocks, kRowLanes lanes per
// row, so that a row's records leave as whole lines. Block i starts at
// offs[i].z (compact) or block_of(row, i), its FP64 block at offs[i].y; each
// header records the start of the cell's FP64 row. FP32 blocks hold the
// offsets p_j - p_m rounded to FP32; compact blocks hold them as 21-bit
// integers against the cell's scale 2^(E - 19), E the smallest exponent with
// every offset component below 2^E (so |q| <= 2^19), but at least e_min, so
// that the box in the cell's units stays far inside the FP32 range; rounding
// to the nearest integer leaves each component within half a unit of the
// scale. FP64 blocks hold the neighbour sites. The neighbours' block offsets
// follow the records. Every row lists its neighbours nearest first (equal
// distances: the lower index), so that an exit search can stop where the
// rest are too far away to matter.
struct FillArgs {
    const Site *sites;
    RowTable rows_in;
    int64_t M;
    int2 *rows;
    Rec64 *r64;
    Slot *blk, *blk64;
    int32_t *blk_off, *blk64_off;   // blk_off null: FP32 blocks
    int e_min;
};
__global__ void __launch_bounds__(256) k_fill_rows(FillArgs A)
{
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) / kRowLanes;
    const int li = threadIdx.x & (kRowLanes - 1);
    if (i >= A.M) return;
    const int4 o = A.rows_in.offs[i];
    const int32_t *row = A.rows_in.row(i);
    const int n = A.rows_in.offs[i + 1].x - o.x;
    const Site si = A.sites[i];
    const bool compact = A.blk_off != nullptr;
    const int32_t bo = compact ? o.z : block_of(make_int2(o.x, n), (int32_t)i);
    // squared distances, for the order (rows too long for the LDS: read again)
    __shared__ double s_d2[256 / kRowLanes][kExportLds];
    double *d2s = s_d2[threadIdx.x / kRowLanes];
    const bool held = n <= kExportLds;
    auto dist2 = [&](int e) {
        const Site sj = A.sites[row[e]];
        const double dx = sj.x - si.x, dy = sj.y - si.y, dz = sj.z - si.z;
        return dx * dx + dy * dy + dz * dz;
    };
    if (held)
        for (int e = li; e < n; e += kRowLanes) d2s[e] = dist2(e);
    lds_order();
    auto place = [&](int e) {   // entries before e (the row comes in ascending order of index)
        const double d = held ? d2s[e] : dist2(e);
        int r = 0;
        for (int k = 0; k < n; ++k) {
            const double dk = held ? d2s[k] : dist2(k);
            r += (dk < d) | ((dk == d) & (k < e)) ? 1 : 0;
        }
        return r;
    };
    int E = 0;
    if (compact) {
        double mc = 0.0;
        for (int e = li; e < n; e += kRowLanes) {
            const Site sj = A.sites[row[e]];
            mc = fmax(mc, fmax(fabs(sj.x - si.x), fmax(fabs(sj.y - si.y), fabs(sj.z - si.z))));
        }
        group_exchange<kRowLanes>([&](auto x) { mc = fmax(mc, x.f64(mc)); });
        E = mc > 0.0 ? ilogb(mc) + 1 : A.e_min;
        E = E < A.e_min ? A.e_min : (E > 127 ? 127 : E);
    }
    if (li == 0) {
        A.rows[i] = make_int2(o.x, n);
        A.blk64_off[i] = o.y;
        if (compact) A.blk_off[i] = o.z;
        if (i == A.M - 1) {   // the ends
            A.blk64_off[A.M] = A.rows_in.offs[A.M].y;
            if (compact) A.blk_off[A.M] = A.rows_in.offs[A.M].z;
        }
        BlockHdr h;
        h.x = si.x;
        h.y = si.y;
        h.z = si.z;
        h.uid = (int32_t)si.uid;
        h.j = (int32_t)i;
        h.row = o.x;
        h.rho = 0.0;
        h.len = n;
        *reinterpret_cast<BlockHdr *>(A.blk64 + o.y) = h;
        h.len = n | (compact ? (E + kScaleBias) << 24 : 0);
        *reinterpret_cast<BlockHdr *>(A.blk + bo) = h;
    }
    float *rec = reinterpret_cast<float *>(A.blk + bo + kHdrSlots);    // FP32: n records of 3 floats
    uint2 *crec = reinterpret_cast<uint2 *>(A.blk + bo + kHdrSlots);   // compact: n records of 8 bytes
    int32_t *nb = compact ? reinterpret_cast<int32_t *>(crec + n) : reinterpret_cast<int32_t *>(rec + 3 * n);
    double *rec64 = reinterpret_cast<double *>(A.blk64 + o.y + kHdrSlots);
    int32_t *nb64 = reinterpret_cast<int32_t *>(rec64 + 3 * n);
    const double sc = ldexp(1.0, kQShift - E);
    for (int f = li; f < n; f += kRowLanes) {
        const int32_t j = row[f];
        const Site sj = A.sites[j];
        const int4 oj = A.rows_in.offs[j];
        const int e = place(f);
        Rec64 a;
        a.x = sj.x;
        a.y = sj.y;
        a.z = sj.z;
        a.j = j;
        a.uid = (int32_t)sj.uid;
        A.r64[o.x + e] = a;
        rec64[3 * e] = sj.x;
        rec64[3 * e + 1] = sj.y;
        rec64[3 * e + 2] = sj.z;
        nb64[e] = oj.y;
        if (compact) {
            const uint64_t m21 = (1ull << kQBits) - 1;
            const uint64_t qx = (uint64_t)(int64_t)rint((sj.x - si.x) * sc) & m21;
            const uint64_t qy = (uint64_t)(int64_t)rint((sj.y - si.y) * sc) & m21;
            const uint64_t qz = (uint64_t)(int64_t)rint((sj.z - si.z) * sc) & m21;
            const uint64_t v = qx | (qy << kQBits) | (qz << (2 * kQBits));
            crec[e] = make_uint2((uint32_t)v, (uint32_t)(v >> 32));
            nb[e] = oj.z;
        } else {
            rec[3 * e] = (float)(sj.x - si.x);
            rec[3 * e + 1] = (float)(sj.y - si.y);
            rec[3 * e + 2] = (float)(sj.z - si.z);
            nb[e] = block_of(make_int2(oj.x, 0), j);
        }
    }
}

__global__ void k_export_counts(const int32_t *__restrict__ inv_perm, const int2 *__restrict__ rows,
                                const uint8_t *__restrict__ walls, int64_t M, int32_t *__restrict__ cnt)
{
    int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= M) return;
    int32_t i = inv_perm[u];
    cnt[u] = rows[i].y + __popc((unsigned)walls[i]);
}

// Rows of user indices, ascending, then walls: kRowLanes lanes per row, an
// entry's place being the number of smaller ones in its row (rows too long
// for their part of the LDS are sorted by their first lane).
__global__ void __launch_bounds__(256) k_export_fill(const int32_t *__restrict__ inv_perm, const int2 *__restrict__ rows,
                                                     const Rec64 *__restrict__ r64, const uint8_t *__restrict__ walls,
                                                     int64_t M, const int64_t *__restrict__ row_ptr,
                                                     int32_t *__restrict__ col)
{
    __shared__ int32_t ids[256 / kRowLanes][kExportLds];
    const int64_t u = ((int64_t)blockIdx.x * 256 + threadIdx.x) / kRowLanes;
    const int li = threadIdx.x & (kRowLanes - 1);
    int32_t *id = ids[threadIdx.x / kRowLanes];
    int2 rw = make_int2(0, 0);
    int32_t i = 0;
    if (u < M) {
        i = inv_perm[u];
        rw = rows[i];
        if (rw.y <= kExportLds)
            for (int e = li; e < rw.y; e += kRowLanes) id[e] = r64[rw.x + e].uid;
    }
    __syncthreads();
    if (u >= M) return;
    int32_t *out = col + row_ptr[u];
    if (rw.y <= kExportLds) {
        for (int e = li; e < rw.y; e += kRowLanes) {
            const int32_t x = id[e];
            int r = 0;
            for (int k = 0; k < rw.y; ++k) r += id[k] < x ? 1 : 0;
            out[r] = x;
        }
    } else if (li == 0) {
        for (int e = 0; e < rw.y; ++e) {
            const int32_t x = r64[rw.x + e].uid;
            int k = e - 1;
            while (k >= 0 && out[k] > x) {
                out[k + 1] = out[k];
                --k;
            }
            out[k + 1] = x;
        }
    }
    if (li == 0) {
        int n = rw.y;
        for (int w = 0; w < 6; ++w)
            if ((walls[i] >> w) & 1) out[n++] = -(w + 1);
    }
}

// Device memory of a grid: from the caller's allocator when one is given
// (e.g. a framework's caching allocator), else hipMalloc.
struct DevBlock {
    void *p;
    size_t bytes;
};

struct DevAlloc {
    vor_allocator a{};
    bool custom = false;
    void *stream = nullptr;
    void *get(size_t bytes) const
    {
        if (custom) return a.alloc(bytes, a.ctx, stream);
        void *p = nullptr;
        return hipMalloc(&p, bytes) == hipSuccess ? p : nullptr;
    }
    void put(const DevBlock &b) const
    {
        if (!b.p) return;
        if (custom) a.free(b.p, b.bytes, a.ctx, stream);
        else (void)hipFree(b.p);
    }
};

// Several arrays in one allocation, each on a 256-byte boundary: an
// allocation and its release cost tens to hundreds of microseconds each, so
// a build makes four or five of them instead of one per array.
struct Batch {
    struct Part {
        void *p;   // the pointer to set
        size_t off;
    };
    std::vector<Part> parts;
    size_t bytes = 0;
    template <typename T>
    void add(T *&p, size_t n)
    {
        p = nullptr;
        parts.push_back(Part{&p, bytes});
        bytes += (n * sizeof(T) + 255) & ~(size_t)255;
    }
    bool alloc(std::vector<DevBlock> &track, const DevAlloc &A)
    {
        if (bytes == 0) return true;
        char *base = (char *)A.get(bytes);
        if (!base) return false;
        track.push_back(DevBlock{base, bytes});
        for (const Part &q : parts) {
            char *at = base + q.off;
            std::memcpy(q.p, &at, sizeof(at));
        }
        return true;
    }
};

unsigned blocks_for(int64_t n, int threads) { return (unsigned)((n + threads - 1) / threads); }

}  // namespace

// Cell blocks of more than this many bytes in the FP32 layout do not stay in
// the last-level cache; the automatic layout makes them compact.
constexpr int64_t kCompactAutoBytes = 512ll << 20;

// The smallest scale exponent of a compact block: 2^40 below the box
// diagonal, so that points of the box in a cell's units stay below 2^60
// (their squares inside the FP32 range); and at least -126.
static int compact_min_exp(const double box[6])
{
    double d2 = 0.0;
    for (int a = 0; a < 3; ++a) d2 += (box[a + 3] - box[a]) * (box[a + 3] - box[a]);
    const int e = d2 > 0.0 ? ilogb(sqrt(d2)) - 40 : -126;
    return e < -126 ? -126 : (e > 127 ? 127 : e);
}

struct vor_grid {
    vrt::Grid g;
    DevAlloc alloc;                 // where its arrays came from
    std::vector<DevBlock> owned;    // ... and the arrays, returned by vor_grid_free
};

extern "C" vor_status vor_build_grid(const double *sites, int64_t M, const double *box, const vor_build_opts *opts,
                                     const vor_allocator *allocator, void *stream, vor_grid **out)
{
    if (out) *out = nullptr;
    if (!sites || !box || !out || M < 1 || M >= 0x7fffffffLL) return VOR_EINVAL;
    if (allocator && (!allocator->alloc || !allocator->free)) return VOR_EINVAL;
    for (int a = 0; a < 3; ++a)
        if (!std::isfinite(box[a]) || !std::isfinite(box[a + 3]) || !(box[a] < box[a + 3])) return VOR_EINVAL;
    double occ = (opts && opts->bucket_occupancy > 0) ? opts->bucket_occupancy : 2.0;
    const bool want_loc = opts && opts->block_lists;
    const double locc = (opts && opts->block_occupancy > 0) ? opts->block_occupancy : 0.25;
    if (opts && (opts->block_lists < 0 || opts->block_lists > 1 || !(opts->block_occupancy >= 0))) return VOR_EINVAL;
    const int layout = opts ? opts->record_layout : VOR_RECORDS_AUTO;
    if (layout < VOR_RECORDS_AUTO || layout > VOR_RECORDS_COMPACT) return VOR_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    auto t0 = std::chrono::steady_clock::now();

    vor_grid *G = new (std::nothrow) vor_grid;
    if (!G) return VOR_ENOMEM;
    Grid &g = G->g;
    G->alloc.custom = allocator != nullptr;
    if (allocator) G->alloc.a = *allocator;
    G->alloc.stream = stream;
    const DevAlloc &A = G->alloc;
    (void)hipGetDevice(&g.device);
    if (hipDeviceGetAttribute(&g.cus, hipDeviceAttributeMultiprocessorCount, g.device) != hipSuccess || g.cus < 1) {
        delete G;
        return VOR_EDEVICE;
    }
    g.M = M;
    for (int a = 0; a < 6; ++a) g.box[a] = box[a];

    vor_status rc = VOR_OK;
    std::vector<DevBlock> tmp, &keep = G->owned;
    BoxArg ba;
    for (int a = 0; a < 3; ++a) {
        ba.lo[a] = box[a];
        ba.hi[a] = box[a + 3];
    }
    double ext = std::max(box[3] - box[0], std::max(box[4] - box[1], box[5] - box[2]));
    double hscale = (double)(1 << kHilbertBits) / ext;

    // bucket grid dimensions: about `occ` sites per bucket, cube-like buckets
    double vol = (box[3] - box[0]) * (box[4] - box[1]) * (box[5] - box[2]);
    double hb = std::cbrt(vol * occ / (double)M);
    int64_t B = 1;
    for (int a = 0; a < 3; ++a) {
        double e = box[a + 3] - box[a];
        int n = (int)std::ceil(e / hb);
        n = std::max(1, std::min(n, 1024));
        g.dims[a] = n;
        g.h[a] = e / n;
        g.inv_h[a] = n / e;
        B *= n;
    }
    // block-list dimensions: about M / locc blocks, cube-like
    LocArgs la;
    int64_t K = 1;
    if (want_loc) {
        const double hl = std::cbrt(vol * locc / (double)M);
        for (int a = 0; a < 3; ++a) {
            const double e = box[a + 3] - box[a];
            const int n = std::max(1, std::min((int)std::ceil(e / hl), 1024));
            g.loc_dims[a] = la.dims[a] = n;
            g.loc_inv_h[a] = la.inv_h[a] = n / e;
            la.lo[a] = box[a];
            la.ext[a] = e;
            K *= n;
        }
        if (K >= 0x7fffffffLL) {
            delete G;
            return VOR_ECAPACITY;
        }
    }
    const int64_t hist_len = vrt_radix_hist_len(M);
    g.seed_levels = seed_levels_of(M);
    g.key_scale = hscale;
    const int64_t n_seed = seed_base(g.seed_levels + 1);
    Batch kept, temps;
    kept.add(g.sites, M);
    kept.add(g.perm, M);
    kept.add(g.inv_perm, M);
    kept.add(g.wall_mask, M);
    kept.add(g.volume, M);
    kept.add(g.rho_int, M);
    kept.add(g.bucket_sites, M);
    kept.add(g.bucket_start, B + 1);
    kept.add(g.seed, n_seed);
    kept.add(g.rows, M);
    kept.add(g.blk64_off, M + 1);
    if (want_loc) {
        kept.add(g.bbox, (size_t)M * 6);
        kept.add(g.loc_start, K + 1);
    }
    uint32_t *keys, *keys2;
    int32_t *vals, *vals2, *hist, *bcount, *nbr0, *cnt0, *retry, *slot, *extra, *lcnt = nullptr;
    int *err;   // error flags, -, sites to retry, touched, longest row, missing entries, open
    int4 *sizes, *offs;
    unsigned long long *ltot = nullptr;
    BoxTree tree;   // boxes over runs of kLeaf sites, then over 64 boxes each
    Box6 *boxes[3];
    temps.add(keys, M);
    temps.add(vals, M);
    temps.add(keys2, M);
    temps.add(vals2, M);
    temps.add(hist, 2 * hist_len + 1);
    temps.add(err, 8);
    temps.add(bcount, B);
    temps.add(nbr0, (size_t)M * kMaxNbr);
    temps.add(cnt0, M);
    temps.add(retry, M);
    temps.add(slot, M);
    temps.add(extra, M);
    temps.add(sizes, M);
    temps.add(offs, M + 1);
    for (int v = 0; v < 3; ++v) {
        const int64_t per = v == 0 ? kLeaf : 64, below = v == 0 ? M : tree.n[v - 1];
        tree.n[v] = (below + per - 1) / per;
        temps.add(boxes[v], tree.n[v]);
    }
    if (want_loc) {
        temps.add(lcnt, K);
        temps.add(ltot, 1);
    }

    auto fail = [&](vor_status s) {
        (void)hipStreamSynchronize(st);
        for (const DevBlock &b : tmp) A.put(b);
        for (const DevBlock &b : keep) A.put(b);
        delete G;
        return s;
    };
    if (!kept.alloc(keep, A) || !temps.alloc(tmp, A)) return fail(VOR_ENOMEM);
    for (int v = 0; v < 3; ++v) tree.level[v] = boxes[v];
    if (hipMemsetAsync(err, 0, 8 * sizeof(int), st) != hipSuccess) return fail(VOR_EDEVICE);

    const int T = 256;
    hipLaunchKernelGGL(k_validate_keys, dim3(blocks_for(M, T)), dim3(T), 0, st, sites, M, ba, hscale, keys, vals, err);
    int herr = 0;
    if (hipMemcpyAsync(&herr, err, sizeof(int), hipMemcpyDeviceToHost, st) != hipSuccess ||
        hipStreamSynchronize(st) != hipSuccess)
        return fail(VOR_EDEVICE);
    if (herr & ERR_OUTSIDE) return fail(VOR_EOUTSIDE);

    rc = vrt_radix_sort_pairs(keys, vals, keys2, vals2, M, 3 * kHilbertBits, hist, hist_len, st);
    if (rc != VOR_OK) return fail(rc);
    hipLaunchKernelGGL(k_gather_sites, dim3(blocks_for(M, T)), dim3(T), 0, st, sites, vals, M, g.sites, g.perm,
                       g.inv_perm, boxes[0]);
    for (int v = 1; v < 3; ++v)
        hipLaunchKernelGGL(k_box_level, dim3((unsigned)tree.n[v]), dim3(64), 0, st, boxes[v - 1], tree.n[v - 1],
                           boxes[v]);

    if (hipMemsetAsync(g.seed, 0xff, sizeof(int32_t) * n_seed, st) != hipSuccess) return fail(VOR_EDEVICE);
    hipLaunchKernelGGL(k_seeds, dim3(blocks_for(M, T)), dim3(T), 0, st, keys, M, g.seed_levels, g.seed);

    // bucket the Hilbert-ordered sites (stable: within a bucket, Hilbert order)
    GridArg ga;
    for (int a = 0; a < 3; ++a) {
        ga.lo[a] = box[a];
        ga.inv_h[a] = g.inv_h[a];
        ga.dims[a] = g.dims[a];
    }
    if (hipMemsetAsync(bcount, 0, sizeof(int32_t) * B, st) != hipSuccess) return fail(VOR_EDEVICE);
    hipLaunchKernelGGL(k_bucket_keys, dim3(blocks_for(M, T)), dim3(T), 0, st, g.sites, M, ga, keys, vals, bcount);
    int bbits = 1;
    while ((1ll << bbits) < B) ++bbits;
    rc = vrt_radix_sort_pairs(keys, vals, keys2, vals2, M, bbits, hist, hist_len, st);
    if (rc != VOR_OK) return fail(rc);
    rc = vrt_scan_i32_to_i32(bcount, B, g.bucket_start, st);
    if (rc != VOR_OK) return fail(rc);
    hipLaunchKernelGGL(k_bucket_fill, dim3(blocks_for(M, T)), dim3(T), 0, st, g.sites, vals, M, g.bucket_sites);

    // clip every cell: small cells first, the overflowing ones again with large cells
    ClipArgs ca;
    ca.sites = g.sites;
    ca.tree = tree;
    ca.box = ba;
    ca.M = M;
    ca.nbr = nbr0;
    ca.cnt = cnt0;
    ca.walls = g.wall_mask;
    ca.retry = retry;
    ca.n_retry = err + 2;
    ca.touched = extra;   // filled again for the rows
    ca.n_touched = err + 3;
    ca.open = vals2;      // (the sorts are done)
    ca.n_open = err + 6;
    ca.err = err;
    ca.volume = g.volume;
    ca.bbox = g.bbox;
    if (hipMemsetAsync(slot, 0xff, sizeof(int32_t) * M, st) != hipSuccess) return fail(VOR_EDEVICE);
    if (M <= 64) {
        ca.touched = nullptr;
        hipLaunchKernelGGL(k_clip_strict, dim3((unsigned)M), dim3(64), 0, st, ca);
    } else {
        hipLaunchKernelGGL(k_clip, dim3((unsigned)(kXcds * ((M + kXcds - 1) / kXcds))), dim3(64), 0, st, ca);
    }
    if (hipGetLastError() != hipSuccess) return fail(VOR_EDEVICE);
    int hflags[7] = {0, 0, 0, 0, 0, 0, 0};
    auto clipped = [&]() {   // the counts so far, or why the build has failed
        if (hipMemcpyAsync(hflags, err, sizeof(hflags), hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess || hipGetLastError() != hipSuccess)
            return VOR_EDEVICE;
        if (hflags[0] & ERR_DUP) return VOR_EDUP;
        return hflags[0] & (ERR_CAPACITY | ERR_DEGENERATE) ? VOR_ECAPACITY : VOR_OK;
    };
    if ((rc = clipped()) != VOR_OK) return fail(rc);
    if (hflags[3] > 0) {
        hipLaunchKernelGGL(k_clip_strict, dim3((unsigned)hflags[3]), dim3(64), 0, st, ca);
        if ((rc = clipped()) != VOR_OK) return fail(rc);
    }
    if (hflags[6] > 0) {
        hipLaunchKernelGGL(k_clip_open, dim3((unsigned)hflags[6]), dim3(64), 0, st, ca);
        if ((rc = clipped()) != VOR_OK) return fail(rc);
    }
    const int n_retry = hflags[2];
    int32_t *big_nbr = nullptr;
    if (n_retry > 0) {
        Batch more;
        more.add(big_nbr, (size_t)n_retry * kMaxNbrBig);
        if (!more.alloc(tmp, A)) return fail(VOR_ENOMEM);
        hipLaunchKernelGGL(k_clip_big, dim3((unsigned)n_retry), dim3(64), 0, st, ca, big_nbr, slot);
        if ((rc = clipped()) != VOR_OK) return fail(rc);
    }
    g.n_big = n_retry;

    // symmetric rows: which reverse entries are missing, what every row takes, where it goes
    RowTable rt{nbr0, cnt0, slot, big_nbr, nullptr, offs};
    if (hipMemsetAsync(extra, 0, sizeof(int32_t) * M, st) != hipSuccess) return fail(VOR_EDEVICE);
    hipLaunchKernelGGL(k_symm_count, dim3(blocks_for(M * kRowLanes, T)), dim3(T), 0, st, rt, M, extra, err + 5);
    hipLaunchKernelGGL(k_row_sizes, dim3(blocks_for(M, T)), dim3(T), 0, st, cnt0, extra, g.wall_mask, M, sizes, err + 4);
    rc = vrt_scan_int4(sizes, M, offs, st);
    if (rc != VOR_OK) return fail(rc);
    int4 ends;
    int rflags[2] = {0, 0};
    if (hipMemcpyAsync(&ends, offs + M, sizeof(ends), hipMemcpyDeviceToHost, st) != hipSuccess ||
        hipMemcpyAsync(rflags, err + 4, sizeof(rflags), hipMemcpyDeviceToHost, st) != hipSuccess ||
        hipStreamSynchronize(st) != hipSuccess || hipGetLastError() != hipSuccess)
        return fail(VOR_EDEVICE);
    g.nnz = ends.x;
    g.nnz_walls = ends.w;
    g.max_row = rflags[0];
    if (rflags[1] > 0) {   // complete and sort them in CSR
        Batch more;
        int32_t *col;
        more.add(col, ends.x);
        if (!more.alloc(tmp, A)) return fail(VOR_ENOMEM);
        hipLaunchKernelGGL(k_copy_rows, dim3(blocks_for(M, T)), dim3(T), 0, st, rt, M, col, extra);
        hipLaunchKernelGGL(k_symm_fill, dim3(blocks_for(M, T)), dim3(T), 0, st, rt, M, col, extra);
        hipLaunchKernelGGL(k_row_sort, dim3(blocks_for(M, T)), dim3(T), 0, st, col, offs, M);
        rt.col = col;
    }

    // cell blocks are addressed by 32-bit slot offsets; FP32 blocks take
    // kHdrSlots + n slots, compact ones kHdrSlots + ceil(3n / 4), FP64 ones at
    // most 4 + 7n / 4
    int64_t nslots = g.nnz + (int64_t)kHdrSlots * M;
    if (nslots + kRecPad > 0x7fffffffLL) return fail(VOR_ECAPACITY);   // compact blocks take no more slots
    if ((int64_t)4 * M + 2 * g.nnz + kRecPad > 0x7fffffffLL) return fail(VOR_ECAPACITY);
    g.compact = layout == VOR_RECORDS_COMPACT || (layout == VOR_RECORDS_AUTO && nslots * 16 > kCompactAutoBytes);
    Batch records;
    if (g.compact) {   // blocks not at rows[j].x + 3j: their starts are kept
        records.add(g.blk_off, M + 1);
        nslots = ends.z;
    }
    g.nslots = nslots;
    g.nslots64 = ends.y;
    records.add(g.rec64, g.nnz + kRecPad);
    records.add(g.blk, nslots + kRecPad);
    records.add(g.blk64, g.nslots64 + kRecPad);
    if (!records.alloc(keep, A)) return fail(VOR_ENOMEM);
    if (hipMemsetAsync(g.rec64 + g.nnz, 0, sizeof(Rec64) * kRecPad, st) != hipSuccess ||
        hipMemsetAsync(g.blk + nslots, 0, sizeof(Slot) * kRecPad, st) != hipSuccess ||
        hipMemsetAsync(g.blk64 + g.nslots64, 0, sizeof(Slot) * kRecPad, st) != hipSuccess)
        return fail(VOR_EDEVICE);
    const FillArgs fa{g.sites, rt, M, g.rows, g.rec64, g.blk, g.blk64, g.blk_off, g.blk64_off, compact_min_exp(g.box)};
    hipLaunchKernelGGL(k_fill_rows, dim3(blocks_for(M * kRowLanes, T)), dim3(T), 0, st, fa);

    if (want_loc) {
        la.bbox = g.bbox;
        la.M = M;
        if (hipMemsetAsync(lcnt, 0, sizeof(int32_t) * K, st) != hipSuccess ||
            hipMemsetAsync(ltot, 0, sizeof(unsigned long long), st) != hipSuccess)
            return fail(VOR_EDEVICE);
        // (few blocks: their atomics on the total take turns)
        hipLaunchKernelGGL(k_loc_count, dim3(std::min(blocks_for(M * kRowLanes, T), 4096u)), dim3(T), 0, st, la, lcnt, ltot);
        unsigned long long entries = 0;
        if (hipMemcpyAsync(&entries, ltot, sizeof(entries), hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess || hipGetLastError() != hipSuccess)
            return fail(VOR_EDEVICE);
        if (entries >= 0x7fffffffULL) return fail(VOR_ECAPACITY);
        rc = vrt_scan_i32_to_i32(lcnt, K, g.loc_start, st);
        if (rc != VOR_OK) return fail(rc);
        Batch lists;
        lists.add(g.loc_cells, std::max<unsigned long long>(entries, 1));
        if (!lists.alloc(keep, A)) return fail(VOR_ENOMEM);
        if (hipMemsetAsync(lcnt, 0, sizeof(int32_t) * K, st) != hipSuccess) return fail(VOR_EDEVICE);
        hipLaunchKernelGGL(k_loc_fill, dim3(blocks_for(M * kRowLanes, T)), dim3(T), 0, st, la, g.loc_start, lcnt, g.loc_cells);
        if (hipStreamSynchronize(st) != hipSuccess || hipGetLastError() != hipSuccess) return fail(VOR_EDEVICE);
        g.loc_entries = (int64_t)entries;
    }

    if (hipStreamSynchronize(st) != hipSuccess) return fail(VOR_EDEVICE);
    for (const DevBlock &b : tmp) A.put(b);
    tmp.clear();
    g.device_bytes = (int64_t)M * (sizeof(Site) * 2 + 4 * 2 + 1 + sizeof(int2) + 2 * sizeof(double)) + (B + 1) * 4 +
                     (g.nnz + kRecPad) * (int64_t)sizeof(Rec64) + (nslots + kRecPad) * (int64_t)sizeof(Slot) +
                     (g.blk_off ? (M + 1) * 4 : 0) + (g.nslots64 + kRecPad) * (int64_t)sizeof(Slot) + (M + 1) * 4 +
                     n_seed * 4;
    if (want_loc)
        g.device_bytes += (int64_t)M * 6 * (int64_t)sizeof(double) +
                          ((int64_t)g.loc_dims[0] * g.loc_dims[1] * g.loc_dims[2] + 1 + g.loc_entries) * 4;
    g.build_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    *out = G;
    return VOR_OK;
}

extern "C" void vor_grid_free(vor_grid *G)
{
    if (!G) return;
    (void)hipDeviceSynchronize();
    for (const DevBlock &b : G->owned) G->alloc.put(b);
    delete G;
}

extern "C" vor_status vor_grid_get_info(const vor_grid *G, vor_grid_info *info)
{
    if (!G || !info) return VOR_EINVAL;
    const Grid &g = G->g;
    info->n_sites = g.M;
    info->nnz = g.nnz;
    info->nnz_with_walls = g.nnz_walls;
    info->max_row = g.max_row;
    for (int a = 0; a < 3; ++a) info->dims[a] = g.dims[a];
    for (int a = 0; a < 6; ++a) info->box[a] = g.box[a];
    info->build_ms = g.build_ms;
    info->device_bytes = g.device_bytes;
    for (int a = 0; a < 3; ++a) info->block_dims[a] = g.loc_dims[a];
    info->block_entries = g.loc_entries;
    info->record_layout = g.compact ? VOR_RECORDS_COMPACT : VOR_RECORDS_FP32;
    return VOR_OK;
}

extern "C" vor_status vor_grid_neighbors(const vor_grid *G, int64_t *row_ptr, int32_t *col, void *stream)
{
    if (!G || !row_ptr || (!col && G->g.nnz_walls > 0)) return VOR_EINVAL;
    const Grid &g = G->g;
    hipStream_t st = (hipStream_t)stream;
    // per-row counts are staged in col, which holds at least M entries
    // (every clipped cell has at least one face)
    if (g.nnz_walls < g.M) return VOR_EINVAL;
    const int T = 256;
    hipLaunchKernelGGL(k_export_counts, dim3(blocks_for(g.M, T)), dim3(T), 0, st, g.inv_perm, g.rows, g.wall_mask,
                       g.M, col);
    vor_status rc = vrt_scan_i32_to_i64(col, g.M, row_ptr, st);
    if (rc != VOR_OK) return rc;
    hipLaunchKernelGGL(k_export_fill, dim3(blocks_for(g.M * kRowLanes, T)), dim3(T), 0, st, g.inv_perm, g.rows, g.rec64,
                       g.wall_mask, g.M, row_ptr, col);
    return hipGetLastError() == hipSuccess ? VOR_OK : VOR_EDEVICE;
}

extern "C" vor_status vor_grid_truncate_row(vor_grid *G, int64_t site, int32_t keep)
{
    if (!G || site < 0 || site >= G->g.M || keep < 0) return VOR_EINVAL;
    Grid &g = G->g;
    int32_t i = 0;
    int2 rw;
    if (hipMemcpy(&i, g.inv_perm + site, sizeof(i), hipMemcpyDeviceToHost) != hipSuccess ||
        hipMemcpy(&rw, g.rows + i, sizeof(rw), hipMemcpyDeviceToHost) != hipSuccess)
        return VOR_EDEVICE;
    if (keep >= rw.y) return VOR_OK;
    g.rows_cut = 1;   // no more walks along the table
    const int n = rw.y;
    std::vector<Rec64> rec(n);
    if (hipMemcpy(rec.data(), g.rec64 + rw.x, sizeof(Rec64) * n, hipMemcpyDeviceToHost) != hipSuccess) return VOR_EDEVICE;
    // the places of the keep lowest internal indices; they stay nearest first
    std::vector<int> at(n);
    for (int e = 0; e < n; ++e) at[e] = e;
    std::sort(at.begin(), at.end(), [&](int x, int y) { return rec[x].j < rec[y].j; });
    at.resize(keep);
    std::sort(at.begin(), at.end());
    // the kept entries of a row of n, then their block offsets, to the front
    auto shorten = [&](void *row, size_t bytes, size_t offsets) {
        const size_t entry = bytes + offsets;
        std::vector<char> all(entry * n), kept(entry * keep);
        if (hipMemcpy(all.data(), row, all.size(), hipMemcpyDeviceToHost) != hipSuccess) return false;
        for (int e = 0; e < keep; ++e) {
            std::memcpy(&kept[bytes * e], &all[bytes * at[e]], bytes);
            std::memcpy(kept.data() + bytes * keep + offsets * e, all.data() + bytes * n + offsets * at[e], offsets);
        }
        return kept.empty() || hipMemcpy(row, kept.data(), kept.size(), hipMemcpyHostToDevice) == hipSuccess;
    };
    int32_t bo = block_of(rw, i), bo64 = 0, len = 0;
    if ((g.blk_off && hipMemcpy(&bo, g.blk_off + i, sizeof(bo), hipMemcpyDeviceToHost) != hipSuccess) ||
        hipMemcpy(&bo64, g.blk64_off + i, sizeof(bo64), hipMemcpyDeviceToHost) != hipSuccess)
        return VOR_EDEVICE;
    BlockHdr *h = reinterpret_cast<BlockHdr *>(g.blk + bo), *h64 = reinterpret_cast<BlockHdr *>(g.blk64 + bo64);
    if (!shorten(g.rec64 + rw.x, sizeof(Rec64), 0) ||
        !shorten(g.blk + bo + kHdrSlots, g.compact ? 8 : 12, sizeof(int32_t)) ||
        !shorten(g.blk64 + bo64 + kHdrSlots, 24, sizeof(int32_t)) ||
        hipMemcpy(&len, &h->len, sizeof(len), hipMemcpyDeviceToHost) != hipSuccess)
        return VOR_EDEVICE;
    len = (len & ~kLenMask) | keep;   // the scale exponent stays
    rw.y = keep;
    if (hipMemcpy(g.rows + i, &rw, sizeof(rw), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(&h->len, &len, sizeof(len), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(&h64->len, &keep, sizeof(keep), hipMemcpyHostToDevice) != hipSuccess)
        return VOR_EDEVICE;
    return VOR_OK;
}

__global__ void k_export_bboxes(const int32_t *__restrict__ perm, const double *__restrict__ bb, int64_t M,
                                double *__restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= M) return;
    const int64_t u = perm[i];
    for (int a = 0; a < 6; ++a) out[6 * u + a] = bb[6 * i + a];
}

extern "C" vor_status vor_grid_bboxes(const vor_grid *G, double *bbox, void *stream)
{
    if (!G || !bbox || !G->g.bbox) return VOR_EINVAL;
    const Grid &g = G->g;
    const int T = 256;
    hipLaunchKernelGGL(k_export_bboxes, dim3(blocks_for(g.M, T)), dim3(T), 0, (hipStream_t)stream, g.perm, g.bbox,
                       g.M, bbox);
    return hipGetLastError() == hipSuccess ? VOR_OK : VOR_EDEVICE;
}

__global__ void k_bind_density(Slot *__restrict__ blk, Slot *__restrict__ blk64, const int2 *__restrict__ rows,
                               const int32_t *__restrict__ blk_off, const int32_t *__restrict__ blk64_off,
                               const int32_t *__restrict__ perm, int64_t M, const double *__restrict__ density,
                               double *__restrict__ rho_int)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= M) return;
    const double r = density ? density[perm[i]] : 0.0;
    const int32_t bo = blk_off ? blk_off[i] : block_of(rows[i], (int32_t)i);
    reinterpret_cast<BlockHdr *>(blk + bo)->rho = r;
    reinterpret_cast<BlockHdr *>(blk64 + blk64_off[i])->rho = r;
    rho_int[i] = r;
}

extern "C" vor_status vor_grid_bind_density(vor_grid *G, const double *density, void *stream)
{
    if (!G) return VOR_EINVAL;
    Grid &g = G->g;
    const int T = 256;
    hipLaunchKernelGGL(k_bind_density, dim3(blocks_for(g.M, T)), dim3(T), 0, (hipStream_t)stream, g.blk, g.blk64,
                       g.rows, g.blk_off, g.blk64_off, g.perm, g.M, density, g.rho_int);
    if (hipGetLastError() != hipSuccess) return VOR_EDEVICE;
    g.rho_bound = density ? 1 : 0;
    return VOR_OK;
}

__global__ void k_export_volumes(const int32_t *__restrict__ perm, const double *__restrict__ vol, int64_t M,
                                 double *__restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < M) out[perm[i]] = vol[i];
}

extern "C" vor_status vor_grid_volumes(const vor_grid *G, double *volume, void *stream)
{
    if (!G || !volume) return VOR_EINVAL;
    const Grid &g = G->g;
    const int T = 256;
    hipLaunchKernelGGL(k_export_volumes, dim3(blocks_for(g.M, T)), dim3(T), 0, (hipStream_t)stream, g.perm, g.volume,
                       g.M, volume);
    return hipGetLastError() == hipSuccess ? VOR_OK : VOR_EDEVICE;
}

// accessor for the other translation units
const vrt::Grid &vrt_grid_of(const vor_grid *G) { return G->g; }
