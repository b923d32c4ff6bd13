// group_core.h -- the straight-path loop (Sect. 2.2, Eqs. 1-5) with one ray
// per group of W lanes instead of one per lane, for launches too small to
// fill the device.
//
// A lane that walks alone meets five to seven dependent memory round trips
// per step (a row of records in batches, the winner's block offset, its
// header), and a small launch has nothing to hide them behind. Here the
// lanes of a group hold the records of the cell, one each and two ahead of
// knowing the row's length, so a cell arrives in one round trip with its
// header; the neighbours' block offsets, in the same lines, follow while the
// exit search runs; the search is one plane per lane, then an exchange
// across the group. Everything else of a step is done by every lane of the
// group alike. (Holding the block as plain slots as well, so that the offsets
// need no second load, costs 50 registers and was slower throughout.)
//
// The arithmetic, the tie rules and the certificate of the mixed mode are
// those of trace_core.h, so the paths are the same bit for bit.
#pragma once

#include "lanes.h"
#include "locate_core.h"
#include "trace_core.h"

namespace vrt {

constexpr int kGroupRounds = 2;   // records a lane loads ahead

// The cell a group's ray is in.
template <int MODE>
struct GroupCell {
    double pm[3];
    double rho;           // its bound density (0 if none)
    int32_t uid, j;
    int32_t n, row;       // records, start of its row in rec64
    int32_t b;            // offset of its block
    int32_t qe;           // compact blocks: scale exponent
    float f[kGroupRounds][3];        // this lane's records: FP32,
    uint2 q[kGroupRounds];           // compact,
    double d[kGroupRounds][3];       // or FP64
};

template <int MODE>
__device__ __forceinline__ const Slot *group_blocks(const GridRef &G)
{
    return MODE == VOR_MODE_FP64 ? G.blk64 : G.blk;
}

template <int MODE>
constexpr int record_bytes()
{
    return MODE == VOR_MODE_FP64 ? 24 : MODE == kModeCompact ? 8 : 12;
}

struct __attribute__((packed, aligned(4))) Rec12 {
    float x, y, z;
};
struct __attribute__((packed, aligned(8))) Rec24 {
    double x, y, z;
};

// Loads the block at offset b: its header, and this lane's first records
// (record lane + W * r in round r). They are asked for before the row's
// length is known; where that would be past the end of the blocks, the first
// one instead (kRecPad slots of padding: it can always be read).
template <int MODE, int W>
__device__ __forceinline__ void load_cell(const GridRef &G, int32_t b, GroupCell<MODE> &C)
{
    const Slot *B = group_blocks<MODE>(G) + b;
    const int32_t slots = (MODE == VOR_MODE_FP64 ? G.blk64_slots : G.blk_slots) - b;
    const int li = threadIdx.x & (W - 1);
    const char *rec = reinterpret_cast<const char *>(B + kHdrSlots);
    const double2 s0 = *reinterpret_cast<const double2 *>(B);
    const double2 s1 = *reinterpret_cast<const double2 *>(B + 1);
    const int4 s2 = *reinterpret_cast<const int4 *>(B + 2);
#pragma unroll
    for (int r = 0; r < kGroupRounds; ++r) {
        constexpr int bytes = record_bytes<MODE>();
        int i = li + W * r;
        i = kHdrSlots + (bytes * (i + 1) + 15) / 16 <= slots ? i : 0;
        if (MODE == VOR_MODE_FP64) {
            const Rec24 x = *reinterpret_cast<const Rec24 *>(rec + bytes * i);
            C.d[r][0] = x.x;
            C.d[r][1] = x.y;
            C.d[r][2] = x.z;
        } else if (MODE == kModeCompact) {
            C.q[r] = *reinterpret_cast<const uint2 *>(rec + bytes * i);
        } else {
            const Rec12 x = *reinterpret_cast<const Rec12 *>(rec + bytes * i);
            C.f[r][0] = x.x;
            C.f[r][1] = x.y;
            C.f[r][2] = x.z;
        }
    }
    C.b = b;
    C.pm[0] = s0.x;
    C.pm[1] = s0.y;
    C.pm[2] = s1.x;
    C.rho = s1.y;
    C.uid = s2.x;
    C.j = s2.y;
    C.n = s2.z & kLenMask;
    C.row = s2.w;
    C.qe = MODE == kModeCompact ? scale_exp(s2.z) : 0;
}

// The block of cell m (internal index).
template <int MODE>
__device__ __forceinline__ int32_t cell_block(const GridRef &G, int32_t m)
{
    if (MODE == VOR_MODE_FP64) return G.blk64_off[m];
    return G.blk_off ? G.blk_off[m] : block_of(G.rows[m], m);
}

// FP64 exit search: site(r, i) gives record i of the row (round r of the
// lane's own, or later), key(i) a number that grows with the neighbour's
// internal index. The winner's place in the row, or -1 when the chord end
// comes first; the crossing in best. exit_fp64's rules: the smallest crossing
// below L, then the larger n.k, then the lower index.
template <int W, class F, class K>
__device__ __forceinline__ int group_exit_fp64(F &&site, K &&key, int n, const double pm[3], const double r0[3],
                                               const double k[3], double L, double &best)
{
    const int li = threadIdx.x & (W - 1);
    constexpr int32_t kNone = 0x7fffffff;
    double bs = __builtin_huge_val();
    int32_t bi = kNone;
    bool twice = false;   // this lane has its least crossing more than once
    // (& and | throughout: short-circuits would become branches)
    auto take = [&](int i, const Rec24 &q) {
        double den;
        const double s = cross_fp64(q.x, q.y, q.z, pm, r0, k, den);
        const bool ok = (i < n) & (den > 0.0) & (s < L);
        const bool t = ok & ((bi == kNone) | (s < bs));
        twice = t ? false : twice | (ok & (s == bs));
        bs = t ? s : bs;
        bi = t ? i : bi;
    };
#pragma unroll
    for (int r = 0; r < kGroupRounds; ++r) take(li + W * r, site(r, li + W * r));
    for (int i = li + W * kGroupRounds; i < n; i += W) take(i, site(kGroupRounds, i));
    double least = bs;   // a lane without a candidate has +inf, which no crossing below L equals
    group_exchange<W>([&](auto x) { least = fmin(least, x.f64(least)); });
    const bool own = (bi != kNone) & (bs == least);
    const uint32_t owners = group_bits<W>(__ballot(own));
    const bool tied = ((owners & (owners - 1u)) != 0u) | (group_bits<W>(__ballot(own & twice)) != 0u);
    if (__ballot(tied)) {   // some group has equal crossings: all of them again, with the other rules
        double bden = -1.0;
        int32_t bk = kNone;
        bi = kNone;
        for (int i = li, r = 0; i < n; i += W, ++r) {
            double den;
            const Rec24 q = site(kGroupRounds, i);
            const double s = cross_fp64(q.x, q.y, q.z, pm, r0, k, den);
            if (!(den > 0.0) || s != least) continue;
            const int32_t ki = key(i);
            if (den > bden || (den == bden && ki < bk)) {
                bden = den;
                bk = ki;
                bi = i;
            }
        }
        group_exchange<W>([&](auto x) {
            const double od = x.f64(bden);
            const int32_t ok = x.i32(bk), oi = x.i32(bi);
            const bool t = (od > bden) | ((od == bden) & (ok < bk));
            bden = t ? od : bden;
            bk = t ? ok : bk;
            bi = t ? oi : bi;
        });
    } else {
        bi = own ? bi : 0;
        group_exchange<W>([&](auto x) { bi |= x.i32(bi); });
    }
    best = owners ? least : L;
    return owners ? bi : -1;
}

// Mixed-precision exit search (exit_mixed and exit_mixed_compact): the
// winner's place in the row or -1 (the chord end) when the FP32 ranking is
// certain; redo when it is not.
template <int MODE, int W>
__device__ __forceinline__ int group_exit_mixed(const GridRef &G, const GroupCell<MODE> &C, const double r0[3],
                                                const double k[3], double L, double s_c, bool &redo)
{
    const int li = threadIdx.x & (W - 1);
    const float inf = __builtin_huge_valf();
    Query32 Q;
    Query32q Qq;
    float tw, ew;
    if (MODE == kModeCompact) {
        const double qs = ldexp(1.0, kQShift - C.qe);
        const float e_abs_s = (float)((double)G.eps_abs * qs);
        Qq = query32q(C.pm, r0, k, s_c, G.eps_mix, e_abs_s, qs);
        tw = (float)((L - s_c) * qs);
        ew = 2.0f * 5.9604645e-8f * fabsf(tw) + e_abs_s;
    } else {
        Q = query32(C.pm, r0, k, s_c, G.eps_mix, G.eps_abs);
        wall32(L, s_c, G.eps_abs, tw, ew);
    }
    // the wall is lane 0's
    float t1 = li == 0 ? tw : inf, err1 = li == 0 ? ew : 0.0f;
    int32_t w1 = li == 0 ? -1 : 0x7fffffff;
    float lo_a = li == 0 ? tw - ew : inf, lo_b = inf;
    bool graze = false;
    auto rank = [&](int i, float nx, float ny, float nz) {
        float t, err;
        bool pos, maybe;
        if (MODE == kModeCompact) plane_bound32q(nx, ny, nz, Qq, t, err, pos, maybe);
        else plane_bound32(nx, ny, nz, Q, t, err, pos, maybe);
        const bool in = i < C.n;
        pos = pos & in;
        graze |= maybe & in & !pos;
        const float lo = pos ? t - err : inf;
        const bool w = pos & (t < t1);
        t1 = w ? t : t1;
        err1 = w ? err : err1;
        w1 = w ? i : w1;
        lo_b = __builtin_amdgcn_fmed3f(lo_a, lo_b, lo);
        lo_a = fminf(lo_a, lo);
    };
    auto decode = [&](int i, uint2 v) {
        const int32_t ix = __builtin_amdgcn_sbfe((int32_t)v.x, 0, kQBits);
        const int32_t iy = __builtin_amdgcn_sbfe((int32_t)__builtin_amdgcn_alignbit(v.y, v.x, kQBits), 0, kQBits);
        const int32_t iz = __builtin_amdgcn_sbfe((int32_t)v.y, 2 * kQBits - 32, kQBits);
        rank(i, (float)ix, (float)iy, (float)iz);
    };
    const char *rec = reinterpret_cast<const char *>(G.blk + C.b + kHdrSlots);
#pragma unroll
    for (int r = 0; r < kGroupRounds; ++r) {
        if (MODE == kModeCompact) decode(li + W * r, C.q[r]);
        else rank(li + W * r, C.f[r][0], C.f[r][1], C.f[r][2]);
    }
    for (int i = li + W * kGroupRounds; i < C.n; i += W) {
        if (MODE == kModeCompact) {
            decode(i, *reinterpret_cast<const uint2 *>(rec + 8 * i));
        } else {
            const Rec12 x = *reinterpret_cast<const Rec12 *>(rec + 12 * i);
            rank(i, x.x, x.y, x.z);
        }
    }
    float least = t1;
    group_exchange<W>([&](auto x) {
        least = fminf(least, x.f32(least));
        lo_b = fminf(fmaxf(lo_a, x.f32(lo_a)), fminf(lo_b, x.f32(lo_b)));   // the two smallest of both halves
        lo_a = fminf(lo_a, x.f32(lo_a));
    });
    // The winner's bound and place, from the lane that has it. Two lanes with
    // the same estimate mix theirs, to a bound no smaller than either (bits
    // of positive floats): their intervals meet, so the step is redone.
    const bool own = t1 == least;
    uint32_t eb = own ? __float_as_uint(err1) : 0u, wb = own ? (uint32_t)(w1 + 1) : 0u;
    group_exchange<W>([&](auto x) {
        eb |= x.u32(eb);
        wb |= x.u32(wb);
    });
    err1 = __uint_as_float(eb);
    const float lo1 = least - err1;
    const float lo_other = (lo1 == lo_a) ? lo_b : lo_a;
    redo = (group_bits<W>(__ballot(graze)) != 0u) | !(least + err1 < lo_other);
    return (int)wb - 1;
}

// Segments a group holds back: lane i has the i-th since the last write.
struct GroupHeld {
    int32_t cell;
    double len;
    int32_t n, room;      // how many, and how many the run they are written in can take
    int64_t slot;         // where the first goes, -1 nowhere
    bool spill;
};

template <bool LP>
__device__ __forceinline__ void group_write(const SegOut &O, GroupHeld &H, int li)
{
    if (H.slot >= 0 && li < H.n) {
        slot_cells<LP>(O, H.spill)[H.slot + li] = H.cell;
        slot_lens<LP>(O, H.spill)[H.slot + li] = H.len;
    }
    H.n = 0;
}

// The ray's next spill chunk, taken by the group's first lane.
template <bool LP>
__device__ __forceinline__ void group_chunk(const SegOut &O, RayState &R, int li, int W)
{
    int32_t c = -2;
    if (li == 0) {
        unsigned long long *head = LP ? O.pool->head : O.chunk_head;
        int32_t *next = LP ? O.pool->next : O.spill_next;
        int64_t *first = LP ? O.pool->first : O.spill_first;
        const int64_t c0 = LP ? O.pool->base_chunk : 0;
        const int64_t at = (int64_t)atomicAdd(head, 1ull);
        if (at < (LP ? O.pool->chunks : O.spill_chunks)) {
            next[at] = -1;
            if (R.chunk < 0) first[R.ray] = at;
            else next[R.chunk - c0] = (int32_t)at;
            c = (int32_t)(c0 + at);
        }
    }
    R.chunk = __shfl(c, (threadIdx.x & 63) & ~(W - 1), 64);
}

// Segment number idx of the ray.
template <int W, bool LP>
__device__ __forceinline__ void group_segment(const SegOut &O, RayState &R, GroupHeld &H, int li, int64_t idx,
                                              int32_t cell, double len)
{
    if (H.n == 0) {   // a new run: to the end of the window or spill chunk, W at most
        const int64_t past = idx - R.cap;
        if (past >= 0 && (LP || O.spill_cell) && past % kSpillChunk == 0 && R.chunk != -2) group_chunk<LP>(O, R, li, W);
        H.slot = segment_slot<LP>(O, R, idx, H.spill);
        const int64_t left = past < 0 ? -past : kSpillChunk - past % kSpillChunk;
        H.room = left < W ? (int32_t)left : W;
    }
    H.cell = li == H.n ? cell : H.cell;
    H.len = li == H.n ? len : H.len;
    if (++H.n == H.room) group_write<LP>(O, H, li);
}

// Tallies of a block's groups, added up in LDS: the cells that several of its
// rays meet (those around a point source, or a small grid's) take one atomic
// per block instead of one per ray on the caller's arrays, where updates of
// one line take turns (12 ns each). A cell finds its slot by its index; where
// another cell has it, the deposit goes to the caller's arrays directly. 32768
// rays from one point in a cube of 1000 sites, FP64: 578 us with an atomic per
// deposit, 226 with these, 248 with one ray per lane. (The look-up costs paths
// that few others meet 5%: a ray does without after kMisses taken slots, and
// launches of less than kMinRays altogether.)
struct GroupTally {
    static constexpr int kCells = 64;
    static constexpr int kMisses = 4;
    static constexpr int64_t kMinRays = 1024;
    int32_t cell[kCells];   // -1: free
    double len[kCells], abs[kCells];
};

// Threads 0 .. kCells - 1 of the block clear it; a barrier must follow.
__device__ __forceinline__ void tally_clear(GroupTally &T)
{
    if (threadIdx.x < GroupTally::kCells) {
        T.cell[threadIdx.x] = -1;
        T.len[threadIdx.x] = 0.0;
        T.abs[threadIdx.x] = 0.0;
    }
}

// deposit() through the block's tallies (T, null for none), by one lane of the
// group. misses: the slots that the ray has found taken.
__device__ __forceinline__ void group_deposit(const Extras &X, RayState &R, GroupTally *T, int &misses, double l, double kr)
{
    if (!T || misses >= GroupTally::kMisses) {
        deposit<false>(X, R, l, kr);
        return;
    }
    deposit<true>(X, R, l, kr);
    const uint32_t u = (uint32_t)R.dep_uid;
    const int at = (u * 2654435761u) >> 26;
    const int32_t was = atomicCAS(&T->cell[at], -1, R.dep_uid);
    if (was == -1 || was == R.dep_uid) {
        if (X.tally_len) atomicAdd(&T->len[at], R.dep_len);
        if (X.tally_abs) atomicAdd(&T->abs[at], R.dep_abs);
    } else {
        ++misses;
        if (X.tally_len) atomicAdd(&X.tally_len[R.dep_uid], R.dep_len);
        if (X.tally_abs) atomicAdd(&X.tally_abs[R.dep_uid], R.dep_abs);
    }
    R.dep_uid = -1;
}

// The block's tallies to the caller's arrays, by the wave that ends last.
__device__ __forceinline__ void tally_flush(const Extras &X, const GroupTally &T)
{
    const int i = threadIdx.x & 63;
    const int32_t c = __hip_atomic_load(&T.cell[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (c < 0) return;
    if (X.tally_len) atomicAdd(&X.tally_len[c], T.len[i]);
    if (X.tally_abs) atomicAdd(&X.tally_abs[c], T.abs[i]);
}

// Walks the ray whose set-up R holds (r0, k, L, s_c, window, status) from
// cell m to its end; R and S are then those of a ray whose segments are all
// written. Every lane of the group calls it with the same values.
template <int MODE, bool SEGS, bool EXT, bool LP, int W>
__device__ __forceinline__ void group_walk(const GridRef &G, const RayIn &I, const SegOut &O, const Extras &X,
                                           RayState &R, RayStats &S, int32_t m, GroupTally *T)
{
    const int li = threadIdx.x & (W - 1);
    GroupCell<MODE> C;
    GroupHeld H;
    H.n = 0;
    load_cell<MODE, W>(G, cell_block<MODE>(G, m), C);
    R.uid = C.uid;
    if (EXT) ray_extras_begin(X, R.ray, R);
    const bool has_rho = I.grid_rho || I.density;
    const bool tallies = EXT && (X.tally_len || X.tally_abs);
    int misses = 0;
    for (;;) {
        if (!(R.L > 0.0)) break;
        if (S.steps > G.max_steps) {
            R.st = RAY_STEPLIMIT;
            break;
        }
        ++S.steps;
        S.recs += C.n;
        // the neighbours' block offsets, under way during the search
        const int32_t *off = reinterpret_cast<const int32_t *>(
            reinterpret_cast<const char *>(group_blocks<MODE>(G) + C.b + kHdrSlots) + record_bytes<MODE>() * C.n);
        int32_t nb[kGroupRounds];
#pragma unroll
        for (int r = 0; r < kGroupRounds; ++r) nb[r] = off[li + W * r < C.n ? li + W * r : 0];   // (past the row: not used)
        double rho = 0.0;
        if (I.grid_rho) rho = C.rho;
        else if (I.density) rho = I.density[C.uid];
        double best = R.L;
        int w;
        if (MODE == VOR_MODE_FP64) {
            const Rec24 *rec = reinterpret_cast<const Rec24 *>(G.blk64 + C.b + kHdrSlots);
            w = group_exit_fp64<W>(
                [&](int r, int i) {
                    if (r >= kGroupRounds) return rec[i];
                    return Rec24{C.d[r][0], C.d[r][1], C.d[r][2]};
                },
                [&](int i) { return off[i]; }, C.n, C.pm, R.r0, R.k, R.L, best);
        } else {
            bool redo;
            w = group_exit_mixed<MODE, W>(G, C, R.r0, R.k, R.L, R.s_c, redo);
            if (redo) {
                ++S.nredo;
                const Rec64 *rec = G.rec64 + C.row;   // in the order of the block's records
                w = group_exit_fp64<W>(
                    [&](int, int i) {
                        const Rec64 q = rec[i < C.n ? i : 0];
                        return Rec24{q.x, q.y, q.z};
                    },
                    [&](int i) { return rec[i].j; }, C.n, C.pm, R.r0, R.k, R.L, best);
            }
        }
        GroupCell<MODE> N;
        if (w >= 0) {
            int32_t j1 = 0;
            if (w < W * kGroupRounds) {
#pragma unroll
                for (int r = 0; r < kGroupRounds; ++r) j1 |= w == li + W * r ? nb[r] : 0;
                group_exchange<W>([&](auto x) { j1 |= x.i32(j1); });
            } else {
                j1 = off[w];
            }
            load_cell<MODE, W>(G, j1, N);
            double den;
            if (MODE != VOR_MODE_FP64) best = cross_fp64(N.pm[0], N.pm[1], N.pm[2], C.pm, R.r0, R.k, den);
        }
        const double len = best - R.s_c;
        if (len > 0.0) {
            if (EXT) {
                const double kr = has_rho ? I.kappa * rho : 0.0;
                if (X.tau_stop) {
                    const double tn = R.tau + kr * len;
                    if (kr > 0.0 && tn >= R.tstop) {   // the package interacts in this cell
                        const double lp = (R.tstop - R.tau) / kr;
                        if (SEGS) group_segment<W, LP>(O, R, H, li, S.cnt, C.uid, lp);
                        if (li == 0 && tallies) group_deposit(X, R, T, misses, lp, kr);
                        R.tau = R.tau + kr * lp;
                        ++S.cnt;
                        R.stop_uid = C.uid;
                        R.stop_s = R.s_c + lp;
                        break;
                    }
                }
                if (li == 0 && tallies) group_deposit(X, R, T, misses, len, kr);
            }
            if (has_rho) R.tau += I.kappa * rho * len;
            if (SEGS) group_segment<W, LP>(O, R, H, li, S.cnt, C.uid, len);
            ++S.cnt;
            R.s_c = best;
        } else if (len < -1e-9 * R.L) {   // the no-exit fallback (see ray_step_end)
            R.s_c += G.eps_fb;
            ++S.nfb;
            if (R.s_c >= R.L) break;
            double r[3];
            for (int a = 0; a < 3; ++a) r[a] = R.r0[a] + R.s_c * R.k[a];
            load_cell<MODE, W>(G, cell_block<MODE>(G, nearest_site_wave<W>(G.grid, r, nullptr)), C);
            R.uid = C.uid;
            continue;
        }
        if (w < 0) break;
        C = N;
        R.uid = C.uid;
    }
    if (SEGS) group_write<LP>(O, H, li);
}

}  // namespace vrt
