// clip_wave.h -- the neighbour-table builder's cell clipping, one 64-lane
// wave per site with the cell's vertices held in registers.
//
// A site's Voronoi cell is the box cut by the bisector half-space of every
// other site (Sect. 2.1); only sites closer than twice the cell's largest
// vertex distance can cut it. The cell is stored as the dual of its
// boundary: each vertex is a triangle of three plane slots, oriented so that
// the normals' triple product is positive; each polyhedron edge then appears
// once in each direction. Vertex q * 64 + l lives in lane l. Coordinates are
// relative to the site: a site at offset n gives the plane n.x <= |n|^2/2.
// The faces left at the end are the site's neighbours.
//
// Candidates. The sites are in Hilbert order, so the 64 sites around the
// cell's own in that order are mostly near ones, whatever the density: they
// are taken first, nearest first, and shrink the cell to about its final
// size. The rest come from a tree of bounding boxes over runs of 16, 1024
// and 65536 consecutive sites: the wave tests 64 boxes at a time against
// the sphere of twice the largest vertex distance (and, where many boxes
// pass, against the balls around the vertices in which a site must lie to
// cut one off), then reads four runs of 16 sites per load. A batch of 64
// candidates is tested against every vertex at once, one candidate per lane
// and the vertices broadcast, so only those that cut the cell as it stands
// are cut in turn.
//
// Cuts. Every lane classifies its vertices against the plane (cut off when
// beyond it by more than a relative tolerance, so planes that merely touch
// an edge or a vertex leave no sliver face -- provided that they come after
// the planes they meet there, so a cell in which a cut passes through a
// vertex is clipped again strictly nearest first, as lattices need). The
// vertices kept stay where they are. The rim of the cut (edges of removed
// vertices whose twin edge is kept) comes from a table of the vertex that
// holds each directed edge, one LDS read per edge; the new vertices go to free
// lanes and write their edges there. (Small cells only; a table for 255 planes
// would fill the LDS, so large cells compare the removed vertices pairwise.)
//
// Where the vertices of many planes fall together (sites on a sphere or a
// circle: every bisector goes through its centre), their rounding may exceed
// the tolerance; the vertices a cut removes are then no connected part of the
// boundary, its rim is no single cycle, and what is left is no polyhedron. The
// edges, which no longer come in pairs, and Euler's relation (V = 2 F - 4 for
// a simple polyhedron) show that at the end, and the cell is clipped again
// with another tolerance: see strict_site.
//
// What bounds it: vector issue (98% busy), with 4 waves per SIMD to hide the
// LDS round trips. About 22 cuts of some 220 instructions per cell are more
// than half of it, the walk through the boxes a quarter. On a flared disc of
// 10^6 sites this takes 17.3 ms for the small cells and 3.4 ms for the 213
// large ones (the latency of the largest, 99 faces); rings of a uniform
// bucket grid with the cell in LDS, as before, took 137 and 38 ms. The tests
// against every vertex read them in FP32 from LDS, four ahead; broadcast from
// the lanes' FP64 registers they took 3.4 ms more.
#pragma once

#include <type_traits>

#include "lanes.h"
#include "vrt_internal.h"

namespace vrt {

constexpr int kHilbertBits = 10;   // per axis

enum : int { ERR_OUTSIDE = 1, ERR_DUP = 2, ERR_CAPACITY = 4, ERR_DEGENERATE = 8, ERR_TOUCH = 16, ERR_OPEN = 32 };

struct BoxArg {
    double lo[3], hi[3];
};

// Bounding box of a run of sites; the tree of them over the Hilbert order:
// level 0 over runs of kLeaf sites, each level above over 64 boxes.
struct Box6 {
    double lo[3], hi[3];
};
constexpr int kLeaf = 16;
struct BoxTree {
    const Box6 *level[3];
    int64_t n[3];
};

struct __align__(16) Plane {
    double x, y, z, d;
};

// LDS of a cell with up to K * 64 vertices and P planes (<= 255, packed in 8
// bits). A simple polyhedron of V vertices has V / 2 + 2 faces.
template <int K, int P>
struct WaveCell {
    static constexpr int kPerLane = K;
    static constexpr int kPlanes = P;
    static constexpr bool kTable = K == 1 && P == 64;
    static constexpr int kMaxFaces = K * 32 + 2 < P ? K * 32 + 2 : P;
    Plane pl[P];
    int32_t id[P];          // internal site index, or -(w+1) for box wall w
    uint16_t rim[P];        // rim edges of the current cut
    static constexpr int kWait = kTable ? 64 : 1024;   // candidates that may wait between loads of 64
    using Key = std::conditional_t<kTable, uint32_t, uint64_t>;
    int32_t buf[kWait + 64];                  // candidates waiting; the list of faces at the end
    Key key[kWait + 64];                      // the bits of their squared distances (small cells: the high words)
    int32_t chunk[kTable ? 1 : 64];           // large cells: those taken together
    uint8_t twin[kTable ? P * P : 1];         // [a * P + b]: the vertex with the directed edge a -> b
    float4 ball[K * 64];    // every vertex in FP32 and scaled, with the squared radius of its (widened) ball;
                            // where there is none, a ball that meets nothing (0, 0, 0, -1)
    float4 met[kTable ? 1 : 3 * K * 64];      // large cells: the balls that the boxes at each level meet
    uint32_t list[kTable ? 1 : K * 64];       // large cells: removed vertices; all vertices at the end
    double v[kTable ? 1 : 3 * K * 64];        // large cells: the vertices at the end
};

using WaveCellSmall = WaveCell<1, 64>;
using WaveCellBig = WaveCell<8, 255>;
// Rows of the first pass: WaveCellSmall::kMaxFaces, in whole 16-byte units.
constexpr int kMaxNbr = 36;
constexpr int kMaxNbrBig = 250;
static_assert(kMaxNbr >= WaveCellSmall::kMaxFaces && kMaxNbr % 4 == 0, "a first-pass row holds every face");

// The vertices of the cell in this lane.
template <int K>
struct LaneVerts {
    double x[K], y[K], z[K];
    uint32_t tri[K];
    uint64_t valid[K];      // wave-uniform: lanes whose vertex q is one of the cell's
    double r2;              // wave-uniform: bound on the largest squared vertex distance (at most 2^-20 above it)
    double sr;              // its square root
    double sc;              // wave-uniform: a power of two that scales the box to about 1, for FP32
    int np;                 // wave-uniform: plane slots in use
    double tol;             // wave-uniform: relative tolerance of the cuts
};

__device__ __forceinline__ uint32_t wpack3(int a, int b, int c)
{
    return (uint32_t)a | ((uint32_t)b << 8) | ((uint32_t)c << 16);
}

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

__device__ __forceinline__ uint64_t lanemask_lt()
{
    int l = lane_id();
    return l == 0 ? 0ull : ((~0ull) >> (64 - l));
}

// Orders this wave's LDS accesses (they complete in order; the compiler must
// keep them so). Each block is one wave.
__device__ __forceinline__ void lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ uint64_t wave_or_u64(uint64_t v)
{
    for (int off = 32; off > 0; off >>= 1) v |= (uint64_t)__shfl_xor((unsigned long long)v, off, 64);
    return v;
}

// Positive doubles compare as their bits do, and nearly so as their high words.
__device__ __forceinline__ uint32_t high_word(double v) { return (uint32_t)((uint64_t)__double_as_longlong(v) >> 32); }
__device__ __forceinline__ uint32_t low_word(double v) { return (uint32_t)(uint64_t)__double_as_longlong(v); }
template <class Key>
__device__ __forceinline__ Key key_of(double v)
{
    return sizeof(Key) == 4 ? (Key)high_word(v) : (Key)(uint64_t)__double_as_longlong(v);
}
__device__ __forceinline__ uint32_t wave_min_key(uint32_t v) { return wave_min_u32(v); }
__device__ __forceinline__ uint32_t wave_max_key(uint32_t v) { return wave_max_u32(v); }
__device__ __forceinline__ uint64_t wave_min_key(uint64_t v)
{
    const uint32_t h = wave_min_u32((uint32_t)(v >> 32));
    return (uint64_t)h << 32 | wave_min_u32((uint32_t)(v >> 32) == h ? (uint32_t)v : 0xffffffffu);
}
__device__ __forceinline__ uint64_t wave_max_key(uint64_t v)
{
    const uint32_t h = wave_max_u32((uint32_t)(v >> 32));
    return (uint64_t)h << 32 | wave_max_u32((uint32_t)(v >> 32) == h ? (uint32_t)v : 0u);
}

// Vertex of planes a, b, p by Cramer's rule.
__device__ __forceinline__ bool wvertex(const Plane &a, const Plane &b, const Plane &p, double &x, double &y, double &z)
{
    double bxpx = b.y * p.z - b.z * p.y;
    double bxpy = b.z * p.x - b.x * p.z;
    double bxpz = b.x * p.y - b.y * p.x;
    double pxax = p.y * a.z - p.z * a.y;
    double pxay = p.z * a.x - p.x * a.z;
    double pxaz = p.x * a.y - p.y * a.x;
    double axbx = a.y * b.z - a.z * b.y;
    double axby = a.z * b.x - a.x * b.z;
    double axbz = a.x * b.y - a.y * b.x;
    double det = a.x * bxpx + a.y * bxpy + a.z * bxpz;
    double inv = 1.0 / det;
    x = (a.d * bxpx + b.d * pxax + p.d * axbx) * inv;
    y = (a.d * bxpy + b.d * pxay + p.d * axby) * inv;
    z = (a.d * bxpz + b.d * pxaz + p.d * axbz) * inv;
    return isfinite(x) && isfinite(y) && isfinite(z);
}

// The bound r2 from the vertices: positive doubles compare as their high
// words do, so one 32-bit reduction gives the largest to 2^-20, rounded up.
template <int K>
__device__ __forceinline__ void update_r2(LaneVerts<K> &R)
{
    const int l = lane_id();
    uint32_t h = 0;
#pragma unroll
    for (int q = 0; q < K; ++q)
        if ((R.valid[q] >> l) & 1ull)
            h = max(h, high_word(R.x[q] * R.x[q] + R.y[q] * R.y[q] + R.z[q] * R.z[q]));
    h = min(wave_max_u32(h), 0x7fefffffu);
    R.r2 = __longlong_as_double((long long)(((uint64_t)h << 32) | 0xffffffffull));
    R.sr = __builtin_amdgcn_sqrt(R.r2);   // the scale of a tolerance: the hardware's accuracy will do
}

// Vertex l (of lane l, q = 0 ..) now belongs to the cell: its edges.
template <class C>
__device__ __forceinline__ void own_edges(C &c, uint32_t t, int vert)
{
    if constexpr (C::kTable) {
        const int a = t & 255, b = (t >> 8) & 255, d = (t >> 16) & 255;
        c.twin[a * C::kPlanes + b] = (uint8_t)vert;
        c.twin[b * C::kPlanes + d] = (uint8_t)vert;
        c.twin[d * C::kPlanes + a] = (uint8_t)vert;
    }
}

// Vertex `vert` in FP32: see ball_meets and cuts_now.
template <class C>
__device__ __forceinline__ void set_ball(C &c, const LaneVerts<C::kPerLane> &R, int vert, double x, double y, double z)
{
    const float fx = (float)(x * R.sc), fy = (float)(y * R.sc), fz = (float)(z * R.sc);
    c.ball[vert] = make_float4(fx, fy, fz, fmaf(fx, fx, fmaf(fy, fy, fz * fz)) * 1.00002f);
}

template <class C>
__device__ __forceinline__ void no_ball(C &c, int vert)
{
    c.ball[vert] = make_float4(0.0f, 0.0f, 0.0f, -1.0f);
}

// One past the last vertex in use.
template <int K>
__device__ __forceinline__ int verts_end(const LaneVerts<K> &R)
{
    int n = 0;
#pragma unroll
    for (int q = 0; q < K; ++q)
        if (R.valid[q]) n = q * 64 + 64 - __clzll((long long)R.valid[q]);
    return n;
}

// The box as the initial cell (6 wall planes, 8 corner vertices).
template <class C>
__device__ __forceinline__ void wcell_init(C &c, LaneVerts<C::kPerLane> &R, const double p[3], const BoxArg &box)
{
    const int l = lane_id();
    if (l < 6) {
        const int a = l >> 1;
        const double s = (l & 1) ? 1.0 : -1.0;
        const double pa = a == 0 ? p[0] : a == 1 ? p[1] : p[2];
        const double lo = a == 0 ? box.lo[0] : a == 1 ? box.lo[1] : box.lo[2];
        const double hi = a == 0 ? box.hi[0] : a == 1 ? box.hi[1] : box.hi[2];
        Plane w;
        w.x = (a == 0) ? s : 0.0;
        w.y = (a == 1) ? s : 0.0;
        w.z = (a == 2) ? s : 0.0;
        w.d = (l & 1) ? (hi - pa) : (pa - lo);
        c.pl[l] = w;
        c.id[l] = -(l + 1);
    }
#pragma unroll
    for (int q = 0; q < C::kPerLane; ++q) {
        R.x[q] = R.y[q] = R.z[q] = 0.0;
        R.tri[q] = 0;
        R.valid[q] = 0;
        no_ball(c, q * 64 + l);
    }
    R.valid[0] = 0xff;
    lds_order();
    {
        double ext = 0.0;
        for (int a = 0; a < 3; ++a) ext = fmax(ext, box.hi[a] - box.lo[a]);
        R.sc = ldexp(1.0, -min(max(ilogb(ext), -1000), 1000));
    }
    if (l < 8) {
        const int sx = l & 1, sy = (l >> 1) & 1, sz = (l >> 2) & 1;
        const int X = sx, Y = 2 + sy, Z = 4 + sz;
        const int sign = (sx ? 1 : -1) * (sy ? 1 : -1) * (sz ? 1 : -1);
        R.tri[0] = sign > 0 ? wpack3(X, Y, Z) : wpack3(X, Z, Y);
        R.x[0] = sx ? (box.hi[0] - p[0]) : -(p[0] - box.lo[0]);
        R.y[0] = sy ? (box.hi[1] - p[1]) : -(p[1] - box.lo[1]);
        R.z[0] = sz ? (box.hi[2] - p[2]) : -(p[2] - box.lo[2]);
        own_edges(c, R.tri[0], l);
        set_ball(c, R, l, R.x[0], R.y[0], R.z[0]);
    }
    R.np = 6;
    update_r2(R);
    lds_order();
}

// Cut the cell by {v : n.v <= d} (plane id `id`, all wave-uniform). Returns
// 1, 0 when the plane cuts nothing off, or an -ERR_* code: unless STRICT
// ERR_TOUCH when the cut passes through a vertex, to within its tolerance.
template <bool STRICT, class C>
__device__ __forceinline__ int wcell_cut(C &c, LaneVerts<C::kPerLane> &R, double nx, double ny, double nz, double d,
                                         int32_t id)
{
    constexpr int K = C::kPerLane, P = C::kPlanes;
    const int l = lane_id();
    const uint64_t lt = lanemask_lt();
    // relative tolerance: the scale of the terms of n.v - d (d = |n|^2 / 2)
    const double tol = R.tol * (__builtin_amdgcn_sqrt(2.0 * d) * R.sr + d);
    uint64_t off[K], any = 0, kept = 0, on = 0;
#pragma unroll
    for (int q = 0; q < K; ++q) {
        const double over = nx * R.x[q] + ny * R.y[q] + nz * R.z[q] - d;
        off[q] = __ballot(over > tol) & R.valid[q];
        on |= __ballot(fabs(over) <= tol) & R.valid[q];
        any |= off[q];
        kept |= R.valid[q] & ~off[q];
    }
    if (any == 0) return 0;
    if (!STRICT && on != 0) return -ERR_TOUCH;
    if (kept == 0) return -ERR_DEGENERATE;   // the site itself is always strictly inside
    // plane slot of the new face: a fresh one, or one no kept vertex uses
    int Pn = R.np;
    if (Pn >= P) {
        constexpr int W = (P + 63) / 64;
        uint64_t used[W];
        for (int w = 0; w < W; ++w) used[w] = 0;
#pragma unroll
        for (int q = 0; q < K; ++q)
            if (((R.valid[q] & ~off[q]) >> l) & 1ull) {
                const int v0 = R.tri[q] & 255, v1 = (R.tri[q] >> 8) & 255, v2 = (R.tri[q] >> 16) & 255;
#pragma unroll
                for (int w = 0; w < W; ++w)
                    used[w] |= ((v0 >> 6) == w ? 1ull << (v0 & 63) : 0ull) | ((v1 >> 6) == w ? 1ull << (v1 & 63) : 0ull) |
                               ((v2 >> 6) == w ? 1ull << (v2 & 63) : 0ull);
            }
        Pn = -1;
        for (int w = 0; w < W && Pn < 0; ++w) {
            uint64_t freem = ~wave_or_u64(used[w]);
            if (w == W - 1 && (P & 63)) freem &= (1ull << (P & 63)) - 1;
            if (freem) Pn = w * 64 + __ffsll((long long)freem) - 1;
        }
        Pn = __builtin_amdgcn_readfirstlane(Pn);
        if (Pn < 0) return -ERR_CAPACITY;
    }
    // rim edges: (a -> b) of a removed vertex whose reverse (b -> a) is not
    // an edge of another removed vertex
    int nrim = 0;
    if constexpr (C::kTable) {
        const bool rem = (off[0] >> l) & 1ull;
        const uint32_t t = R.tri[0];
        const int v[3] = {(int)(t & 255), (int)((t >> 8) & 255), (int)((t >> 16) & 255)};
        int tw[3] = {0, 0, 0};
        if (rem) {
#pragma unroll
            for (int k = 0; k < 3; ++k) tw[k] = c.twin[v[(k + 1) % 3] * P + v[k]];
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const bool edge = rem && !((off[0] >> (tw[k] & 63)) & 1ull);
            const uint64_t bal = __ballot(edge);
            const int pos = nrim + __popcll(bal & lt);
            if (edge && pos < P) c.rim[pos] = (uint16_t)(v[k] | (v[(k + 1) % 3] << 8));
            nrim += __popcll(bal);
        }
    } else {
        int nrem = 0;
        lds_order();
#pragma unroll
        for (int q = 0; q < K; ++q) {
            if ((off[q] >> l) & 1ull) c.list[nrem + __popcll(off[q] & lt)] = R.tri[q];
            nrem += __popcll(off[q]);
        }
        lds_order();
        for (int r0 = 0; r0 < nrem; r0 += 64) {
            const int r = r0 + l;
            const bool act = r < nrem;
            const uint32_t t = act ? c.list[r] : 0u;
            const int v[3] = {(int)(t & 255), (int)((t >> 8) & 255), (int)((t >> 16) & 255)};
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const int a = v[k], b = v[(k + 1) % 3];
                bool edge = act;
                for (int s = 0; s < nrem; ++s) {
                    const uint32_t u = c.list[s];
                    const int w0 = u & 255, w1 = (u >> 8) & 255, w2 = (u >> 16) & 255;
                    if ((w0 == b && w1 == a) || (w1 == b && w2 == a) || (w2 == b && w0 == a)) edge = false;
                }
                const uint64_t bal = __ballot(edge);
                const int pos = nrim + __popcll(bal & lt);
                if (edge && pos < P) c.rim[pos] = (uint16_t)(a | (b << 8));
                nrim += __popcll(bal);
            }
        }
    }
    if (nrim > P) return -ERR_CAPACITY;
    const Plane pn = {nx, ny, nz, d};
    if (l == 0) {
        c.pl[Pn] = pn;
        c.id[Pn] = id;
    }
    lds_order();
    if (Pn == R.np) R.np++;
    // one new vertex per rim edge, in the lanes without a vertex
    int base = 0;
    bool bad = false;
#pragma unroll
    for (int q = 0; q < K; ++q) {
        const uint64_t keep = R.valid[q] & ~off[q];
        const int r = base + __popcll(~keep & lt);
        const bool take = !((keep >> l) & 1ull) && r < nrim;
        if (take) {
            const uint32_t e = c.rim[r];
            const int a = e & 255, b = e >> 8;
            bad = bad || !wvertex(c.pl[a], c.pl[b], pn, R.x[q], R.y[q], R.z[q]);
            R.tri[q] = wpack3(a, b, Pn);
            own_edges(c, R.tri[q], q * 64 + l);
            set_ball(c, R, q * 64 + l, R.x[q], R.y[q], R.z[q]);
        } else if ((off[q] >> l) & 1ull) {
            no_ball(c, q * 64 + l);
        }
        R.valid[q] = keep | __ballot(take);
        base += 64 - __popcll(keep);
        if (K > 1 && base >= nrim) {   // the slots above keep what they hold
#pragma unroll
            for (int q2 = 0; q2 < K; ++q2)
                if (q2 > q) {
                    if ((off[q2] >> l) & 1ull) no_ball(c, q2 * 64 + l);
                    R.valid[q2] &= ~off[q2];
                }
            break;
        }
    }
    if (base < nrim) return -ERR_CAPACITY;
    if (__ballot(bad)) return -ERR_DEGENERATE;
    lds_order();
    update_r2(R);
    return 1;
}

// Which of the 64 candidates (one per lane: offset n, d = |n|^2 / 2) may cut
// the cell as it stands: whether the largest n.v over the vertices exceeds d.
// In FP32, with more than its rounding in hand, so that none is passed over
// which the cut itself would take; what falls out of its range passes.
template <class C>
__device__ __forceinline__ bool cuts_now(const C &c, const LaneVerts<C::kPerLane> &R, double nx, double ny, double nz,
                                         double d)
{
    const float fx = (float)(nx * R.sc), fy = (float)(ny * R.sc), fz = (float)(nz * R.sc);
    const float fd = (float)(d * R.sc * R.sc), fr = (float)(R.sr * R.sc);
    const float thr = fd * 0.999999f - 1e-6f * (fabsf(fx) + fabsf(fy) + fabsf(fz)) * fr;
    float m = -__builtin_huge_valf();
    const int end = verts_end(R);
#pragma unroll 4
    for (int k = 0; k < end; ++k) {   // no vertex there: 0, which decides nothing (thr > 0, or all pass)
        const float4 v = c.ball[k];
        m = fmaxf(m, fmaf(fx, v.x, fmaf(fy, v.y, fz * v.z)));
    }
    return !(m < thr);
}

// Takes a batch of candidates, one per lane (site offset n, squared distance
// d2, site j, act: there is one), nearest first (unless STRICT by the high
// words alone; the strict order is exact, because the sites of a far cluster
// share a high word and their planes are nearly parallel). cull: test them all
// against the cell beforehand; after a candidate that cut nothing the rest are
// tested again, if the cell has changed. Returns 0 or an -ERR_* code.
constexpr int kCullMin = 6;   // fewer candidates are as well cut by one by one
template <bool STRICT, class C>
__device__ __forceinline__ int wcell_take(C &c, LaneVerts<C::kPerLane> &R, double nx, double ny, double nz, double d2,
                                          int32_t j, bool act, bool cull)
{
    const uint32_t key = high_word(d2);
    bool tested = false;   // against the cell as it stands
    for (;;) {
        act = act && d2 < 4.0 * R.r2;
        uint64_t am = __ballot(act);
        if (am == 0) return 0;
        if (cull && !tested && __popcll(am) >= kCullMin) {
            const bool cuts = cuts_now(c, R, nx, ny, nz, 0.5 * d2);
            act = act && cuts;
            am = __ballot(act);
            if (am == 0) return 0;
            tested = true;
        }
        const uint32_t k = wave_min_u32(act ? key : 0xffffffffu);
        uint64_t first = __ballot(act && key == k);
        if (STRICT && (first & (first - 1))) {
            const uint32_t lo = wave_min_u32(act && key == k ? low_word(d2) : 0xffffffffu);
            first = __ballot(act && key == k && low_word(d2) == lo);
        }
        const int w = __ffsll((long long)first) - 1;
        const double dd = 0.5 * lane_f64(d2, w);
        const int rc = wcell_cut<STRICT>(c, R, lane_f64(nx, w), lane_f64(ny, w), lane_f64(nz, w), dd,
                                         (int32_t)lane_u32((uint32_t)j, w));
        if (rc < 0) return rc;
        act = act && lane_id() != w;
        tested = tested && rc == 0;
        cull = rc == 0;
    }
}

// Squared distance from p to a box (0 inside; infinite for an empty one).
// Rounding keeps it at most the computed squared distance of a site in it.
__device__ __forceinline__ double box_dist2(const Box6 &b, const double p[3])
{
    double s = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double e = fmax(fmax(b.lo[a] - p[a], p[a] - b.hi[a]), 0.0);
        s += e * e;
    }
    return s;
}

// Whether a site in a box may cut a vertex v off: it would lie in the ball
// around the vertex that the cell's own site lies on. In FP32 relative to
// that site: the box is widened by twice the rounding of its coordinates
// (slack: that of the FP64 ones) and the ball by more than the rounding of
// the vertex and of the test; what overflows passes.
struct BoxF {
    float lx, ly, lz, hx, hy, hz;
};
__device__ __forceinline__ BoxF box_f32(const Box6 &b, const double p[3], double slack, double sc)
{
    auto lo = [&](int a) { const float f = (float)((b.lo[a] - p[a] - slack) * sc); return f - 2.4e-7f * fabsf(f); };
    auto hi = [&](int a) { const float f = (float)((b.hi[a] - p[a] + slack) * sc); return f + 2.4e-7f * fabsf(f); };
    return BoxF{lo(0), lo(1), lo(2), hi(0), hi(1), hi(2)};
}
__device__ __forceinline__ bool ball_meets(const BoxF &b, const float4 &v)
{
    const float ex = fmaxf(fmaxf(b.lx - v.x, v.x - b.hx), 0.0f);
    const float ey = fmaxf(fmaxf(b.ly - v.y, v.y - b.hy), 0.0f);
    const float ez = fmaxf(fmaxf(b.lz - v.z, v.z - b.hz), 0.0f);
    return !(fmaf(ex, ex, fmaf(ey, ey, ez * ez)) > v.w);
}

// The cell's balls, one after another, at the first level of met (large cells).
template <class C>
__device__ __forceinline__ int list_balls(C &c, const LaneVerts<C::kPerLane> &R)
{
    int n = 0;
    if constexpr (!C::kTable) {
        lds_order();
#pragma unroll
        for (int q = 0; q < C::kPerLane; ++q) {
            if ((R.valid[q] >> lane_id()) & 1ull)
                c.met[n + __popcll(R.valid[q] & lanemask_lt())] = c.ball[q * 64 + lane_id()];
            n += __popcll(R.valid[q]);
        }
        lds_order();
    }
    return n;
}

// Of the n balls listed for level `at` of met, those that a box
// (wave-uniform) meets, listed for the next level. Returns their number.
template <class C>
__device__ __forceinline__ int balls_met(C &c, int at, int n, const BoxF &b)
{
    constexpr int kList = C::kPerLane * 64;
    int m = 0;
    lds_order();
    for (int e = 0; e < n; e += 64) {
        const int k = e + lane_id();
        const float4 v = c.met[at * kList + (k < n ? k : 0)];
        const bool in = k < n && ball_meets(b, v);
        const uint64_t bal = __ballot(in);
        if (in) c.met[(at + 1) * kList + m + __popcll(bal & lanemask_lt())] = v;
        m += __popcll(bal);
    }
    lds_order();
    return m;
}

// 64 boxes of a level, one per lane, and which of them hold candidates at a
// squared distance in [from, to): within the sphere of twice the largest
// vertex distance and, where many are, in the ball of one of the vertices
// (large cells: of the n listed for level `at`, which the boxes above meet).
// Boxes in the sphere from which the ball test pays: 6 / 10 / 12 / 16 / never
// measured 23.3 / 23.1 / 23.1 / 23.2 / 28.1 ms for the whole build of a
// 10^6-site flared disc, 36.4 / 35.8 / 35.7 / 35.7 / 36.0 ms for a clumpy medium
// of 2x10^6.
constexpr int kBallMin = 12;
template <class C>
__device__ __forceinline__ uint64_t boxes_hit(const C &c, const LaneVerts<C::kPerLane> &R, int at, int n_balls,
                                              const Box6 *boxes, int64_t n, int64_t first, const double p[3],
                                              double from, double to, double slack, Box6 &b)
{
    const int64_t i = first + lane_id();
    for (int a = 0; a < 3; ++a) {
        b.lo[a] = __builtin_huge_val();
        b.hi[a] = -__builtin_huge_val();
    }
    if (i < n) b = boxes[i];
    bool in = box_dist2(b, p) < fmin(to, 4.0 * R.r2);
    if (from > 0.0) {
        double far = 0.0;   // the farthest corner
        for (int a = 0; a < 3; ++a) {
            const double e = fmax(b.hi[a] - p[a], p[a] - b.lo[a]);
            far += e * e;
        }
        in = in && far >= from;
    }
    uint64_t hit = __ballot(in);
    if (__popcll(hit) >= kBallMin) {
        const BoxF f = box_f32(b, p, slack, R.sc);
        bool may = false;
        if constexpr (C::kTable) {
            const int end = verts_end(R);
#pragma unroll 4
            for (int k = 0; k < end; ++k) may |= ball_meets(f, c.ball[k]);
        } else {
#pragma unroll 4
            for (int k = 0; k < n_balls; ++k) may |= ball_meets(f, c.met[at * C::kPerLane * 64 + k]);
        }
        hit &= __ballot(may);
    }
    return hit;
}

__device__ __forceinline__ Box6 lane_box(const Box6 &b, int l)
{
    Box6 o;
    for (int a = 0; a < 3; ++a) {
        o.lo[a] = lane_f64(b.lo[a], l);
        o.hi[a] = lane_f64(b.hi[a], l);
    }
    return o;
}

// The smallest double whose key is above k.
__device__ __forceinline__ double above(uint32_t k) { return __longlong_as_double((long long)((uint64_t)(k + 1u) << 32)); }
__device__ __forceinline__ double above(uint64_t k) { return __longlong_as_double((long long)(k + 1u)); }

// How many of the n waiting candidates have a key in [k0, k1].
template <class C>
__device__ __forceinline__ int count_waiting(const C &c, int n, typename C::Key k0, typename C::Key k1)
{
    int m = 0;
    for (int e = 0; e < n; e += 64) {
        const int at = e + lane_id();
        const typename C::Key k = c.key[at < n ? at : 0];
        m += __popcll(__ballot(at < n && k >= k0 && k <= k1));
    }
    return m;
}

// The nearest of the n waiting candidates with keys of k0 or more: the key up
// to which there are at most `most` of them (and, unless equal keys prevent
// it, at least three quarters of that), their number in m. With more than
// `most` at the smallest key, that key and their number.
template <class C>
__device__ __forceinline__ typename C::Key nearest_waiting(const C &c, int n, typename C::Key k0, int most, int &m)
{
    using Key = typename C::Key;
    Key lo = ~(Key)0, hi = 0;
    for (int e = 0; e < n; e += 64) {
        const int at = e + lane_id();
        const Key k = c.key[at < n ? at : 0];
        if (at < n && k >= k0) {
            lo = min(lo, k);
            hi = max(hi, k);
        }
    }
    lo = wave_min_key(lo);
    hi = wave_max_key(hi);
    m = count_waiting(c, n, k0, hi);
    if (m <= most) return hi;
    m = count_waiting(c, n, k0, lo);
    while (hi - lo > 1 && 4 * m < 3 * most) {   // count(lo) <= most < count(hi)
        const Key mid = lo + (hi - lo) / 2;
        const int k = count_waiting(c, n, k0, mid);
        if (k > most) {
            hi = mid;
        } else {
            lo = mid;
            m = k;
        }
    }
    return lo;
}

// Drops the waiting candidates with keys above k1. Returns how many stay.
template <class C>
__device__ __forceinline__ int drop_waiting(C &c, int n, typename C::Key k1)
{
    const uint64_t lt = lanemask_lt();
    int kept = 0;
    for (int e = 0; e < n; e += 64) {   // in place: nothing moves up
        const int at = e + lane_id();
        const typename C::Key k = at < n ? c.key[at] : 0;
        const int32_t j = at < n ? c.buf[at] : 0;
        const bool stay = at < n && k <= k1;
        const uint64_t bal = __ballot(stay);
        lds_order();
        if (stay) {
            c.key[kept + __popcll(bal & lt)] = k;
            c.buf[kept + __popcll(bal & lt)] = j;
        }
        kept += __popcll(bal);
        lds_order();
    }
    return kept;
}

// Whether x -> y is an edge of the vertex of planes w.
__device__ __forceinline__ bool has_edge(uint32_t w, int x, int y)
{
    const int a = w & 255, b = (w >> 8) & 255, c = (w >> 16) & 255;
    return ((a == x) & (b == y)) | ((b == x) & (c == y)) | ((c == x) & (a == y));
}

// Volume of the clipped cell, by the whole wave. The cell is the union of
// the cones from the site (the origin here) to its faces, so
// V = sum over faces x of (h_x / 3) * area_x, with h_x = d_x / |n_x| the
// distance of plane x from the site. Around face x the vertices come in a
// cyclic order: from vertex t = (x, y, z) (oriented) the next is the vertex
// holding the reversed edge (y, x), the other end of the polyhedron edge
// between faces x and y; so 2 area_x = |sum over the face's vertices of
// n_x / |n_x| . (v_t x v_next)|, with one orientation for every face.
// closed: every edge (x, y) is one vertex's, and its reverse one vertex's.
template <class C>
__device__ __forceinline__ double wcell_volume(C &c, const LaneVerts<C::kPerLane> &R, bool &closed)
{
    constexpr int K = C::kPerLane, P = C::kPlanes;
    const int l = lane_id();
    double acc = 0.0;
    bool apart = false;
    int nt = 0;
    if constexpr (!C::kTable) {   // all vertices in LDS
        for (int q = 0; q < K; ++q) {
            if ((R.valid[q] >> l) & 1ull) {
                const int t = nt + __popcll(R.valid[q] & lanemask_lt());
                c.list[t] = R.tri[q];
                c.v[3 * t] = R.x[q];
                c.v[3 * t + 1] = R.y[q];
                c.v[3 * t + 2] = R.z[q];
            }
            nt += __popcll(R.valid[q]);
        }
        lds_order();
    }
    auto cone = [&](int x, double tx, double ty, double tz, double ux, double uy, double uz) {
        const double cx = ty * uz - tz * uy;
        const double cy = tz * ux - tx * uz;
        const double cz = tx * uy - ty * ux;
        const Plane f = c.pl[x];
        const double nn = f.x * f.x + f.y * f.y + f.z * f.z;
        acc += f.d / nn * (f.x * cx + f.y * cy + f.z * cz);
    };
    if constexpr (C::kTable) {
        const bool have = (R.valid[0] >> l) & 1ull;
        const uint32_t u = R.tri[0];
        const int corner[3] = {(int)(u & 255), (int)((u >> 8) & 255), (int)((u >> 16) & 255)};
#pragma unroll
        for (int e = 0; e < 3; ++e) {
            const int x = corner[e], y = corner[(e + 1) % 3];
            const int t2 = have ? c.twin[y * P + x] & 63 : l;
            const uint32_t w = __shfl(u, t2, 64);   // (of a vertex no longer there: what it was)
            const bool there = (R.valid[0] >> t2) & 1ull;
            apart |= have & (!there | !has_edge(w, y, x) | (c.twin[x * P + y] != l));
            const double ux = __shfl(R.x[0], t2, 64), uy = __shfl(R.y[0], t2, 64), uz = __shfl(R.z[0], t2, 64);
            if (have) cone(x, R.x[0], R.y[0], R.z[0], ux, uy, uz);
        }
    } else {
        for (int t = l; t < nt; t += 64) {
            const uint32_t u = c.list[t];
            const int corner[3] = {(int)(u & 255), (int)((u >> 8) & 255), (int)((u >> 16) & 255)};
            for (int e = 0; e < 3; ++e) {
                const int x = corner[e], y = corner[(e + 1) % 3];
                int t2 = -1;
                for (int s = 0; s < nt; ++s) {
                    const uint32_t w = c.list[s];
                    apart |= has_edge(w, x, y) & (s != t);
                    if (has_edge(w, y, x)) {
                        apart |= t2 >= 0;
                        t2 = t2 < 0 ? s : t2;
                    }
                }
                apart |= t2 < 0;
                if (t2 < 0) continue;
                cone(x, c.v[3 * t], c.v[3 * t + 1], c.v[3 * t + 2], c.v[3 * t2], c.v[3 * t2 + 1], c.v[3 * t2 + 2]);
            }
        }
    }
    closed = __ballot(apart) == 0;
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    return fabs(acc) / 6.0;
}

// Bounding box of the clipped cell from its vertices (Sect. 2.3: the cell
// is convex), absolute coordinates {xmin, ymin, zmin, xmax, ymax, zmax}.
template <int K>
__device__ __forceinline__ void wcell_bbox(const LaneVerts<K> &R, const double p[3], double *__restrict__ bb)
{
    const int l = lane_id();
    double lo[3] = {__builtin_huge_val(), __builtin_huge_val(), __builtin_huge_val()};
    double hi[3] = {-__builtin_huge_val(), -__builtin_huge_val(), -__builtin_huge_val()};
#pragma unroll
    for (int q = 0; q < K; ++q)
        if ((R.valid[q] >> l) & 1ull) {
            const double v[3] = {R.x[q], R.y[q], R.z[q]};
            for (int a = 0; a < 3; ++a) {
                lo[a] = fmin(lo[a], v[a]);
                hi[a] = fmax(hi[a], v[a]);
            }
        }
    for (int a = 0; a < 3; ++a) {
        const double b0 = p[a] + wave_min_f64(lo[a]), b1 = p[a] + wave_max_f64(hi[a]);
        if (l == 0) {
            bb[a] = b0;
            bb[a + 3] = b1;
        }
    }
}

// Clip site i's cell. Writes the neighbour indices, ascending, to nbr
// (capacity max_nbr) and the bounding box to bbox (unless null); the wall
// mask and the volume go to the caller's variables. Returns the count or
// -ERR_*. All lanes of the wave call it with the same i. STRICT takes every
// site nearest first, without the Hilbert neighbourhood's head start;
// otherwise the order is loose, and a cell in which a cut passes through a
// vertex is refused with ERR_TOUCH. tol is the relative
// tolerance of the cuts; a cell that is no closed polyhedron at the end is
// refused with ERR_OPEN unless `open` lets it pass.
template <class C, bool STRICT>
__device__ __forceinline__ int wclip_site(C &c, const Site *__restrict__ sites, int64_t M, const BoxTree &tree,
                                          const BoxArg &box, int64_t i, int32_t *nbr, int max_nbr, uint32_t &walls,
                                          double &volume, double *bbox, double tol, bool open)
{
    constexpr int K = C::kPerLane, P = C::kPlanes;
    const int l = lane_id();
    const uint64_t lt = lanemask_lt();
    const Site si = sites[i];
    const double p[3] = {si.x, si.y, si.z};
    double slack = 0.0;   // rounding of box coordinates
    for (int a = 0; a < 3; ++a) slack = fmax(slack, 1e-15 * fmax(fabs(box.lo[a]), fabs(box.hi[a])));
    LaneVerts<K> R;
    R.tol = tol;
    wcell_init(c, R, p, box);
    // the nearer half of the neighbourhood in Hilbert order (of up to 64 sites: everything)
    const int64_t w0 = max((int64_t)0, min(i - 32, M - 64));
    uint32_t near;   // those up to this high word of the squared distance are taken here
    {
        const int64_t j = w0 + l;
        const bool act = j < M && j != i;
        const Site o = sites[act ? j : i];
        const double dx = o.x - p[0], dy = o.y - p[1], dz = o.z - p[2];
        const double d2 = dx * dx + dy * dy + dz * dz;
        if (__ballot(act && d2 == 0.0)) return -ERR_DUP;
        const uint32_t key = high_word(d2);
        uint32_t k0 = wave_min_u32(act ? key : 0xffffffffu);
        near = wave_max_u32(act ? key : 0u);
        for (int it = 0; M > 64 && it < 10 && k0 < near; ++it) {
            const uint32_t mid = k0 + (near - k0) / 2;
            if (__popcll(__ballot(act && key <= mid)) >= 32) near = mid;
            else k0 = mid + 1;
        }
        if (!STRICT || M <= 64) {
            const int rc = wcell_take<STRICT>(c, R, dx, dy, dz, d2, (int32_t)j, act && key <= near, false);
            if (rc < 0) return rc;
        }
    }
    // Everything else in reach, through the tree of boxes, in shells of
    // squared distance [from, to), cut back whenever more than C::kWait sites
    // wait, so that the sites are taken nearest first (a cell still open on one
    // side would otherwise grow hundreds of faces against far sites).
    double from = 0.0, to = 4.0 * above(near);
    while (M > 64) {
        int nbuf = 0;
        bool crowded = false;   // the shell was cut back
        const int n_all = list_balls(c, R);
        // The balls a box's sites may lie in, for the boxes below it (few of a
        // large cell's; small cells go through all of theirs). A cut during the
        // pass leaves the lists good: what cuts the smaller cell cuts the larger.
        auto below = [&](int at, int n, const Box6 &boxes, int lane, int &met) {
            met = n;
            if (C::kTable) return true;
            met = balls_met(c, at, n, box_f32(lane_box(boxes, lane), p, slack, R.sc));
            return met > 0;
        };
        auto take = [&](const int32_t *list, int n) {   // up to 64 candidates
            lds_order();
            const bool act = l < n;
            const int32_t j = act ? list[l] : (int32_t)i;
            const Site o = sites[j];
            const double dx = o.x - p[0], dy = o.y - p[1], dz = o.z - p[2];
            const double d2 = dx * dx + dy * dy + dz * dz;
            return wcell_take<STRICT>(c, R, dx, dy, dz, d2, j, act, true);
        };
        auto take_waiting = [&]() {   // all of them, nearest first
            int rc = 0;
            if constexpr (C::kTable) {
                rc = take(c.buf, min(nbuf, 64));
                if (rc >= 0 && nbuf > 64) rc = take(c.buf + 64, nbuf - 64);
            } else {
                typename C::Key k0 = 0;
                for (int left = nbuf; left > 0 && rc >= 0;) {
                    int m;
                    const typename C::Key k1 = nearest_waiting(c, nbuf, k0, 64, m);
                    for (int first = 0; first < m && rc >= 0; first += 64) {   // several rounds of equal keys only
                        int at = 0;
                        lds_order();
                        for (int e = 0; e < nbuf; e += 64) {
                            const typename C::Key k = c.key[e + l < nbuf ? e + l : 0];
                            const bool in = e + l < nbuf && k >= k0 && k <= k1;
                            const uint64_t bal = __ballot(in);
                            const int to_ = at + __popcll(bal & lt) - first;
                            if (in && to_ >= 0 && to_ < 64) c.chunk[to_] = c.buf[e + l];
                            at += __popcll(bal);
                        }
                        rc = take(c.chunk, min(64, m - first));
                    }
                    left -= m;
                    k0 = k1 + 1;
                }
            }
            nbuf = 0;
            return rc;
        };
        for (int64_t g2 = 0; g2 < tree.n[2]; g2 += 64) {
            Box6 b2;
            for (uint64_t h2 = boxes_hit(c, R, 0, n_all, tree.level[2], tree.n[2], g2, p, from, to, slack, b2);
                 h2; h2 &= h2 - 1) {
                const int c2 = __ffsll((long long)h2) - 1;
                const int64_t g1 = (g2 + c2) * 64;
                int n2;
                Box6 b1;
                if (!below(0, n_all, b2, c2, n2)) continue;
                for (uint64_t h1 = boxes_hit(c, R, 1, n2, tree.level[1], tree.n[1], g1, p, from, to, slack, b1); h1;
                     h1 &= h1 - 1) {
                    const int c1 = __ffsll((long long)h1) - 1;
                    const int64_t g0 = (g1 + c1) * 64;
                    int n1;
                    Box6 b0;
                    if (!below(1, n2, b1, c1, n1)) continue;
                    uint64_t h0 = boxes_hit(c, R, 2, n1, tree.level[0], tree.n[0], g0, p, from, to, slack, b0);
                    while (h0) {   // four runs of kLeaf sites per load
                        int leaf[4];
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            leaf[k] = h0 ? __ffsll((long long)h0) - 1 : -1;
                            h0 &= h0 - 1;   // 0 stays 0
                        }
                        const int grp = l >> 4;
                        const int lf = grp == 0 ? leaf[0] : grp == 1 ? leaf[1] : grp == 2 ? leaf[2] : leaf[3];
                        const int64_t j = (g0 + lf) * kLeaf + (l & 15);
                        const bool in = lf >= 0 && j < M && j != i;
                        const Site o = sites[in ? j : i];
                        const double dx = o.x - p[0], dy = o.y - p[1], dz = o.z - p[2];
                        const double d2 = dx * dx + dy * dy + dz * dz;
                        if (__ballot(in && d2 == 0.0)) return -ERR_DUP;
                        const uint32_t key = high_word(d2);
                        bool want = in && d2 >= from && d2 < fmin(to, 4.0 * R.r2) &&
                                    (STRICT || key > near || j < w0 || j >= w0 + 64);
                        uint64_t wm = __ballot(want);
                        if (nbuf + __popcll(wm) > C::kWait) {   // crowded: only those that cut the cell as it stands
                            const bool cuts = cuts_now(c, R, dx, dy, dz, 0.5 * d2);
                            want = want && cuts;
                            wm = __ballot(want);
                        }
                        if (want) {
                            const int at = nbuf + __popcll(wm & lt);
                            c.buf[at] = (int32_t)j;
                            c.key[at] = key_of<typename C::Key>(d2);
                        }
                        nbuf += __popcll(wm);
                        lds_order();
                        if (nbuf > C::kWait) {
                            int m;
                            const typename C::Key k1 = nearest_waiting(c, nbuf, (typename C::Key)0, C::kWait, m);
                            if (m <= C::kWait) {
                                nbuf = drop_waiting(c, nbuf, k1);
                                to = above(k1);
                                crowded = true;
                            } else if (STRICT && C::kTable) {   // too many with one high word: their order is lost
                                return -ERR_CAPACITY;
                            } else {   // too many at one distance: take all that wait now
                                const int rc = take_waiting();
                                if (rc < 0) return rc;
                            }
                        }
                    }
                }
            }
        }
        if (nbuf > 0) {
            const int rc = take_waiting();
            if (rc < 0) return rc;
        }
        if (!(to < 4.0 * R.r2)) break;   // no farther site can cut
        // the next shell: four times as far, or as wide as this one if that had to be cut back
        const double next = to + (crowded ? 1.0 : 3.0) * (to - from);
        from = to;
        to = next;
    }
    // faces: plane slots some vertex still uses
    constexpr int W = (P + 63) / 64;
    uint64_t face[W];
    int faces = 0, verts = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) face[w] = 0;
#pragma unroll
    for (int q = 0; q < K; ++q) {
        verts += __popcll(R.valid[q]);
        if ((R.valid[q] >> l) & 1ull) {
            const uint32_t u = R.tri[q];
            const int v0 = u & 255, v1 = (u >> 8) & 255, v2 = (u >> 16) & 255;
#pragma unroll
            for (int w = 0; w < W; ++w)
                face[w] |= ((v0 >> 6) == w ? 1ull << (v0 & 63) : 0ull) | ((v1 >> 6) == w ? 1ull << (v1 & 63) : 0ull) |
                           ((v2 >> 6) == w ? 1ull << (v2 & 63) : 0ull);
        }
    }
#pragma unroll
    for (int w = 0; w < W; ++w) {
        face[w] = wave_or_u64(face[w]);
        faces += __popcll(face[w]);
    }
    bool closed;
    volume = wcell_volume(c, R, closed);
    if (!open && (!closed || verts != 2 * faces - 4)) return -ERR_OPEN;
    if (bbox) wcell_bbox(R, p, bbox);
    int nn = 0;
    walls = 0;
    lds_order();
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const int s = w * 64 + l;
        const bool is = (face[w] >> l) & 1ull;
        const int32_t id = is ? c.id[s] : 0;
        const uint64_t bal = __ballot(is && id >= 0);
        if (is && id >= 0) c.buf[nn + __popcll(bal & lt)] = id;
        nn += __popcll(bal);
        for (int k = 0; k < 6; ++k)
            if (__ballot(is && id == -(k + 1))) walls |= 1u << k;
    }
    if (nn > max_nbr) return -ERR_CAPACITY;
    lds_order();
    for (int s = l; s < nn; s += 64) {   // in ascending order: a face's place is the number of smaller indices
        const int32_t id = c.buf[s];
        int r = 0;
        for (int k = 0; k < nn; ++k) r += c.buf[k] < id ? 1 : 0;
        nbr[r] = id;
    }
    return nn;
}

// Clip site i's cell with the planes strictly nearest first (wclip_site's
// results). A cell that degenerates or is no polyhedron with one tolerance is
// taken again with the next, the wider ones first (a smaller one first took two
// to four tries each where 1e-11 nearly always does); where none of them helps,
// as it comes out with the one of all cells. Of the cells of 1000 sites on a
// sphere 4 need another tolerance, of 3000 on a circle 70.
constexpr double kCutTol = 1e-12;
constexpr int kCutTols = 7;
template <class C>
__device__ __forceinline__ int strict_site(C &c, const Site *__restrict__ sites, int64_t M, const BoxTree &tree,
                                           const BoxArg &box, int64_t i, int32_t *nbr, int max_nbr, uint32_t &walls,
                                           double &volume, double *bbox, int first)
{
    for (int t = first;; ++t) {
        const bool last = t == kCutTols - 1;
        const double tol = t == 1 ? 1e-11 : t == 2 ? 1e-10 : t == 3 ? 1e-9 : t == 4 ? 1e-13 : t == 5 ? 1e-14 : kCutTol;
        const int n = wclip_site<C, true>(c, sites, M, tree, box, i, nbr, max_nbr, walls, volume, bbox, tol, last);
        if (last || (n != -ERR_DEGENERATE && n != -ERR_OPEN)) return n;
        lds_order();
    }
}

}  // namespace vrt
