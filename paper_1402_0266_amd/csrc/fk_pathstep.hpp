// fk_pathstep.hpp -- per-lane Euler-Maruyama path state and step, shared
// by the plain and the control-variate path kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fk.h"
#include "fk_accum.hpp"
#include "fk_device.hpp"
#include "fk_internal.hpp"

namespace fk {

// Lane path state.
struct Lane {
    float xh, xl, yh, yl;  // position as hi + lo pairs
    int32_t k;             // steps taken
    int32_t K;             // steps allowed
    uint32_t path, nid, ctr3;
    uint32_t out;          // output row of the path's node
    float px, py;          // start point (score shift for identity data)
    float horizon, dt, dt_last, cbm, cbm_last;
    float ox, oy;          // frozen / static centre offset
    float rev0, drev, cos_d, sin_d;  // orbit angle at path start, step, rotation
    float s_hi, s_lo;      // exponential time-stepping: elapsed time as a hi + lo pair
    DensityRegs dens;
};

// Index of the lane's path in the optional per-path outputs [n_out][n_paths].
__device__ __forceinline__ uint64_t path_rec(const Lane &L, uint32_t n_paths) {
    return (uint64_t)L.out * n_paths + L.path;
}

// Adds an increment to a (hi, lo) pair and renormalises so that hi is the
// FP32 rounding of hi + lo.
__device__ __forceinline__ void comp_add(float &hi, float &lo, float inc) {
    const float t = lo + inc;
    const float s = hi + t;
    lo = (hi - s) + t;
    hi = s;
}

// Outside the closed unit square: x, y, 1 - x or 1 - y negative.  hi is the
// rounded position; (1 - hi) is exact near 1, so the tests against 1 see the
// lo part too.  The minimum drops NaN: a position that is not a number (a
// grid density's drift, or an analytic one's beyond FP32's range) is outside
// only where its other coordinate is.  (The sign bits take cheaper
// instructions, but a NaN has a sign bit too.)  Written out: fminf, fmaxf or
// four comparisons here made the compiler order the loops around it differently
// (16 levels of up to 200 to 1100 steps 2% slower).
__device__ __forceinline__ bool outside(float xh, float xl, float yh, float yl) {
    const float x1 = (1.f - xh) - xl, y1 = (1.f - yh) - yl;
    float m;
    asm("v_min3_f32 %0, %1, %2, %3" : "=v"(m) : "v"(xh), "v"(yh), "v"(x1));
    asm("v_min_f32 %0, %0, %1" : "+v"(m) : "v"(y1));
    return m < 0.f;
}

// One Euler-Maruyama step of length D (cb = -4 ln2 D) of the position with
// centre offset (ox, oy); the step's Brownian part sqrt(2 D) z in (dwx, dwy).
// m: kUnitMask, in a vector register.
template <int KIND>
__device__ __forceinline__ void em_move(float &xh, float &xl, float &yh, float &yl, const DensityRegs &dens,
                                        uint32_t ra, uint32_t rb, float ox, float oy, float D, float cb, uint32_t m,
                                        float &dwx, float &dwy) {
    brownian_increment(ra, rb, cb, m, dwx, dwy);
    float bx, by;
    drift<KIND>(dens, ox, oy, xh, yh, bx, by);
    comp_add(xh, xl, fmaf(bx, D, dwx));
    comp_add(yh, yl, fmaf(by, D, dwy));
}

// Distances of the lane's position to the sides 0 (x = 0), 1 (x = 1),
// 2 (y = 0) and 3 (y = 1).
struct SideDist {
    float d[4];
};
__device__ __forceinline__ SideDist side_dist(float xh, float xl, float yh, float yl) {
    return SideDist{{xh + xl, (1.f - xh) - xl, yh + yl, (1.f - yh) - yl}};
}
__device__ __forceinline__ SideDist side_dist(const Lane &L) { return side_dist(L.xh, L.xl, L.yh, L.yl); }

// Brownian-bridge exit test of a step of length D (iD = 1/D) between two
// points inside, at the distances a and b from the sides.  The diffusion
// sqrt(2) W pinned at both ends crosses a side at distances d0, d1 with
// probability exp(-d0 d1 / D); the four sides combine as independent events.
// A side whose exponent d0 d1 / D exceeds 17 counts as 0 (below the
// uniforms' resolution 2^-24; a zero-length step on a side, 0/0, too).
// Returns the crossing probability and the side most likely crossed (-1:
// none within reach, and the caller needs no uniform).
__device__ __forceinline__ float bridge_prob(const SideDist &a, const SideDist &b, float iD, int &side) {
    float p = 0.f, pmax = 0.f;
    side = -1;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float e = a.d[i] * b.d[i] * iD;
        if (e <= 17.f) {
            const float ps = hw_exp2(-1.44269504f * e);
            p = (p + ps) - p * ps;  // 1 - (1 - p)(1 - ps)
            if (ps > pmax) {
                pmax = ps;
                side = i;
            }
        }
    }
    return p;
}

// The bridge test's uniform ((r >> 8) + 1) 2^-24: on u < p the path has left
// within the step and is moved onto the side it most likely crossed.
__device__ __forceinline__ float bridge_uniform(uint32_t r) { return fmaf((float)(r >> 8), 0x1p-24f, 0x1p-24f); }

// The lane's end point projected onto a side (-1: left as it is), by selects,
// so that the position stays in registers.
__device__ __forceinline__ void move_to_side(Lane &L, int side) {
    const bool mx = side == 0 || side == 1, my = side >= 2;
    const float to = (side & 1) ? 1.f : 0.f;
    L.xh = mx ? to : L.xh;
    L.xl = mx ? 0.f : L.xl;
    L.yh = my ? to : L.yh;
    L.yl = my ? 0.f : L.yl;
}

// Bilinear interpolation in a nodal grid; off the grid, the nearest cell's
// bilinear function continued (linear extrapolation).
__device__ __forceinline__ float grid_bilinear(const double *g, int n, float x, float y) {
    const float fx = x * (float)n, fy = y * (float)n;
    int i = (int)floorf(fx), j = (int)floorf(fy);
    i = min(max(i, 0), n - 1);
    j = min(max(j, 0), n - 1);
    const float ax = fx - (float)i, ay = fy - (float)j;
    const double *r0 = g + (int64_t)j * (n + 1);
    const double *r1 = r0 + (n + 1);
    const float v00 = (float)r0[i], v01 = (float)r0[i + 1];
    const float v10 = (float)r1[i], v11 = (float)r1[i + 1];
    return (1.f - ay) * ((1.f - ax) * v00 + ax * v01) + ay * ((1.f - ax) * v10 + ax * v11);
}

// Gradient of the bilinear interpolant of a nodal grid at (x, y) (the cell
// grid_bilinear uses); differences taken in FP64.
__device__ __forceinline__ void grid_gradient(const double *g, int n, float x, float y, float &gx, float &gy) {
    const float fx = x * (float)n, fy = y * (float)n;
    int i = (int)floorf(fx), j = (int)floorf(fy);
    i = min(max(i, 0), n - 1);
    j = min(max(j, 0), n - 1);
    const float ax = fx - (float)i, ay = fy - (float)j;
    const double *r0 = g + (int64_t)j * (n + 1);
    const double *r1 = r0 + (n + 1);
    const float d0x = (float)(r0[i + 1] - r0[i]), d1x = (float)(r1[i + 1] - r1[i]);
    const float d0y = (float)(r1[i] - r0[i]), d1y = (float)(r1[i + 1] - r0[i + 1]);
    gx = (float)n * fmaf(ay, d1x - d0x, d0x);
    gy = (float)n * fmaf(ax, d1y - d0y, d0y);
}

// The same gradient of component comp from the per-cell table (fk_cv.hip,
// grad_table_kernel).
__device__ __forceinline__ void table_gradient(const float4 *tab, int n, int comp, float x, float y, float &gx,
                                               float &gy) {
    const float fx = x * (float)n, fy = y * (float)n;
    int i = (int)floorf(fx), j = (int)floorf(fy);
    i = min(max(i, 0), n - 1);
    j = min(max(j, 0), n - 1);
    const float ax = fx - (float)i, ay = fy - (float)j;
    const float4 t = tab[2 * ((int64_t)j * n + i) + comp];
    gx = (float)n * fmaf(ay, t.y, t.x);
    gy = (float)n * fmaf(ax, t.w, t.z);
}

// Work chunks of a wavefront in the control-variate kernels (wave-uniform).
// A wavefront's first chunk is its own index in the grid, so a launch starts
// without every wavefront contending for the one counter at once; later
// chunks come from the counter, past the first grid-full.  Which wavefront
// runs which chunk does not change any result: paths draw their numbers by
// their own counters.  (The plain path kernel keeps its first grab on the
// counter: the same change there costs ~3% in its hot loop's code.)
__device__ __forceinline__ uint32_t first_chunk() { return blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); }
__device__ __forceinline__ uint32_t next_chunk(const PathArgs &a) {
    uint32_t c = 0;
    if ((threadIdx.x & 63u) == 0) c = atomicAdd(a.queue, 1u);
    return __builtin_amdgcn_readfirstlane(c) + gridDim.x * (blockDim.x >> 6);
}
// The launch's work-chunk count (set by the node-table kernels or the host).
__device__ __forceinline__ uint32_t launch_chunks(const PathArgs &a) {
    return __builtin_amdgcn_readfirstlane(a.queue[kCtrTotal]);
}

// Node slot and path chunk of work chunk c (c < total).  Node by node, or
// (tile_shift > 0) with the chunks of 2^tile_shift consecutive slots
// interleaved; a last, partial tile runs node by node.  Only the division by
// cpn of the node-by-node order is needed: the tile is a power of two, so the
// rest is masks and shifts.  The order only changes the schedule: every path
// draws from its own counters and every sum is exact.
__device__ __forceinline__ void chunk_slot(const PathArgs &a, uint32_t total, uint32_t c, uint32_t &slot,
                                           uint32_t &pc) {
    const uint32_t q = c / a.cpn;
    slot = q;
    pc = c - q * a.cpn;
    const uint32_t sh = a.tile_shift;
    if (sh == 0u) return;
    const uint32_t m = (1u << sh) - 1u;
    if ((uint64_t)((q | m) + 1u) * a.cpn > total) return;   // in the partial last tile
    const uint32_t r = (q & m) * a.cpn + pc;                 // rank of the chunk within its tile
    slot = (q & ~m) | (r & m);
    pc = r >> sh;
}

// The cursor (node slot, path range) of chunk c; false past the last chunk.
__device__ __forceinline__ bool chunk_cursor(const PathArgs &a, uint32_t total, uint32_t c, uint32_t &slot,
                                             uint32_t &next, uint32_t &end) {
    if (c >= total) return false;
    uint32_t pc;
    chunk_slot(a, total, c, slot, pc);
    next = pc * a.chunk;
    end = min(next + a.chunk, a.n_paths);
    return true;
}

// chunk_cursor, and on success the chunk's accumulation slot: its tag
// (wave-uniform; every lane calls this).
template <int NV>
__device__ __forceinline__ bool grab_chunk(const PathArgs &a, uint32_t total, uint32_t c, uint32_t &slot,
                                           uint32_t &next, uint32_t &end, AccSlot<NV> *slots, NodeAcc *const *accs,
                                           uint32_t &tag, uint32_t &grabs, uint32_t lane) {
    if (!chunk_cursor(a, total, c, slot, next, end)) return false;
    tag = slot_open<NV>(slots, accs, grabs++, (uint32_t)a.nodes[slot].out, end - next, lane);
    return true;
}

// The level constants of a lane (horizon, step sizes, density parameters,
// Philox counter word 3), loaded with every path: a wavefront may hold paths
// of several levels in a batched launch.  (Held once per launch in scalar
// registers instead, they cost the hot loop more than they save: a VALU
// instruction reads one scalar operand, and the extra scalar pressure
// spills.)
template <int KIND, int TMODE>
__device__ __forceinline__ void lane_level(Lane &L, const LevelDev &lv) {
    L.K = lv.K;
    L.ctr3 = lv.ctr3;
    L.horizon = lv.horizon;
    L.dt = lv.dt;
    L.dt_last = lv.dt_last;
    L.cbm = lv.cbm;
    L.cbm_last = lv.cbm_last;
    L.rev0 = lv.rev0;
    L.drev = lv.drev;
    L.cos_d = lv.cos_d;
    L.sin_d = lv.sin_d;
    L.dens.amp = lv.amp;
    L.dens.nscale = lv.nscale;
    L.dens.a2s = lv.a2s;
    L.dens.cx = lv.cx;
    L.dens.cy = lv.cy;
    L.dens.orbit_r = lv.orbit_r;
    L.dens.omega_rev = lv.omega_rev;
    if constexpr (KIND == KIND_GRID) {
        L.dens.gb = lv.gb;
        L.dens.gn = lv.gn;
        L.dens.fn = lv.fn;
    }
    L.ox = 0.f;
    L.oy = 0.f;
    if constexpr (moving_kind(KIND) && TMODE == TIME_FROZEN) {
        orbit(L.dens, lv.t_freeze, L.ox, L.oy);
    }
}

// Loads path `path` of node `nd` into a lane, with its level's constants.
template <int KIND, int TMODE>
__device__ __forceinline__ void lane_start(Lane &L, const NodeDev &nd, const LevelDev *levels, uint32_t path) {
    L.path = path;
    L.xh = nd.x;
    L.yh = nd.y;
    L.xl = nd.xlo;
    L.yl = nd.ylo;
    L.px = nd.x;
    L.py = nd.y;
    L.k = 0;
    L.nid = nd.nid;
    L.out = (uint32_t)nd.out;
    lane_level<KIND, TMODE>(L, levels[nd.level]);
}

// ---------------------------------------------------------------------------
// Steps with a branch after each: what the refilling kernels take where paths
// end after a few of them (the wavefront then scores and refills at nearly
// every pair, and what a branch-free pair saves goes into sorting out its
// ends; 12 to 25 registers fewer keep more wavefronts resident).
// ---------------------------------------------------------------------------

// One step; its Brownian part is added to (dbx, dby).  True if the path left.
template <int KIND, bool UNIFORM>
__device__ __forceinline__ bool one_step(Lane &L, uint32_t ra, uint32_t rb, float ox, float oy, float &dbx,
                                         float &dby) {
    float D = L.dt, cb = L.cbm;
    if constexpr (!UNIFORM) {
        const bool last = (L.k == L.K - 1);
        D = last ? L.dt_last : D;
        cb = last ? L.cbm_last : cb;
    }
    float wx, wy;
    em_move<KIND>(L.xh, L.xl, L.yh, L.yl, L.dens, ra, rb, ox, oy, D, cb, kUnitMask, wx, wy);
    L.k += 1;
    const bool out = outside(L.xh, L.xl, L.yh, L.yl);
    dbx += wx;
    dby += wy;
    return out;
}

// The two steps of one Philox call r, the second one if the path is still
// inside and under way.  True if it left.
template <int KIND, int TMODE, bool UNIFORM>
__device__ __forceinline__ bool two_steps(Lane &L, const PhiloxOut &r, float &dbx, float &dby) {
    constexpr bool kMovingBackward = moving_kind(KIND) && TMODE == TIME_BACKWARD;
    float ox = L.ox, oy = L.oy, cr = 0.f, sr = 0.f;
    if constexpr (kMovingBackward) {
        // orbit angle at PDE time t_init + t - k dt, in revolutions
        const float rev = fmaf(-(float)L.k, L.drev, L.rev0);
        cr = hw_cos_rev(rev);
        sr = hw_sin_rev(rev);
        ox = L.dens.orbit_r * cr;
        oy = L.dens.orbit_r * sr;
    }
    if (one_step<KIND, UNIFORM>(L, r.r0, r.r1, ox, oy, dbx, dby)) return true;
    if (L.k >= L.K) return false;
    if constexpr (kMovingBackward) {
        // one step later it is smaller by omega dt: rotate (cos, sin)
        ox = L.dens.orbit_r * fmaf(cr, L.cos_d, sr * L.sin_d);
        oy = L.dens.orbit_r * fmaf(sr, L.cos_d, -cr * L.sin_d);
    }
    return one_step<KIND, UNIFORM>(L, r.r2, r.r3, ox, oy, dbx, dby);
}

// ---------------------------------------------------------------------------
// Steps in pairs (the two steps of one Philox call) without a branch between
// them: both are taken, and the rare path that ends in the pair is sorted out
// afterwards (pair_end).
// ---------------------------------------------------------------------------
struct PairLane {
    PhiloxLane pp;            // the path's fixed Philox products
    uint32_t bridge_ck;       // pp.ck of the bridge test's stream
    SideDist dist;            // the bridge test's distances at the lane's position
    float iD, iD_last;        // the bridge test's 1 / D
    float drev2;              // 2 drev
    int32_t half, half_end;   // pairs taken; the number of them by which the path has ended
};

// The pair's first point, its Brownian parts, and the bridge test's outcomes.
struct Pair {
    float xh, xl, yh, yl;
    float w1x, w1y, w2x, w2y;
    int side1, side2;
};

// half_end past this (as a float's bits, 0.5) would read as a float >= 1:
// there every pair is looked at.
constexpr int32_t kHalfMax = 0x3f000000;

// A lane without a path: a point that stays at (0.5, 0.5).  L.k is kept.
template <bool BRIDGE>
__device__ __forceinline__ void pair_idle(Lane &L, PairLane &P) {
    L.xh = L.yh = 0.5f;
    L.xl = L.yl = 0.f;
    L.dt = L.cbm = 0.f;
    L.K = 0x7fffffff;
    P.half = 0;
    P.half_end = kHalfMax;
    if constexpr (BRIDGE) {
        P.dist = side_dist(L);
        P.iD = 1e30f;
    }
}

// After lane_start.
template <bool BRIDGE>
__device__ __forceinline__ void pair_start(Lane &L, PairLane &P, uint32_t key0, uint32_t key1) {
    P.pp = philox_lane(L.path, L.nid, L.ctr3, key0, key1);
    P.half = 0;
    P.half_end = min((L.K - 1) >> 1, kHalfMax);
    P.drev2 = 2.f * L.drev;
    if (L.K <= 0) {      // scored where it starts: keeps its low parts in values it has no use for
        L.horizon = L.xl;
        L.dt_last = L.yl;
    }
    if constexpr (BRIDGE) {
        P.bridge_ck = (L.ctr3 | 4u) ^ key1;
        P.dist = side_dist(L);
        P.iD = 1.f / L.dt;
        P.iD_last = 1.f / L.dt_last;
    }
}

// Takes a pair of steps; true where the path may have ended in it.
template <int KIND, int TMODE, bool UNIFORM, bool BRIDGE>
__device__ __forceinline__ bool pair_step(Lane &L, PairLane &P, const PhiloxKeys &keys, uint32_t mask, Pair &p) {
    const PhiloxOut r = philox4x32_10_lane((uint32_t)P.half, P.pp, keys);
    float ox = L.ox, oy = L.oy, ox2 = ox, oy2 = oy;
    if constexpr (moving_kind(KIND) && TMODE == TIME_BACKWARD) {
        // Orbit angle at PDE time t_init + t - k dt (k = 2 half), in
        // revolutions; one step later it is smaller by omega dt: rotate
        // (cos, sin) instead of re-evaluating them.
        const float rev = fmaf(-(float)P.half, P.drev2, L.rev0);
        const float cr = hw_cos_rev(rev), sr = hw_sin_rev(rev);
        ox = L.dens.orbit_r * cr;
        oy = L.dens.orbit_r * sr;
        ox2 = L.dens.orbit_r * fmaf(cr, L.cos_d, sr * L.sin_d);
        oy2 = L.dens.orbit_r * fmaf(sr, L.cos_d, -cr * L.sin_d);
    }
    float D1 = L.dt, D2 = L.dt, cb1 = L.cbm, cb2 = L.cbm, iD1 = P.iD, iD2 = P.iD;
    if constexpr (!UNIFORM) {
        // the last step K - 1 is the pair's first (K odd) or second one
        const bool l1 = 2 * P.half == L.K - 1, l2 = 2 * P.half == L.K - 2;
        D1 = l1 ? L.dt_last : D1;
        cb1 = l1 ? L.cbm_last : cb1;
        iD1 = l1 ? P.iD_last : iD1;
        D2 = l2 ? L.dt_last : D2;
        cb2 = l2 ? L.cbm_last : cb2;
        iD2 = l2 ? P.iD_last : iD2;
    }
    p.xh = L.xh;
    p.xl = L.xl;
    p.yh = L.yh;
    p.yl = L.yl;
    em_move<KIND>(p.xh, p.xl, p.yh, p.yl, L.dens, r.r0, r.r1, ox, oy, D1, cb1, mask, p.w1x, p.w1y);
    L.xh = p.xh;
    L.xl = p.xl;
    L.yh = p.yh;
    L.yl = p.yl;
    em_move<KIND>(L.xh, L.xl, L.yh, L.yl, L.dens, r.r2, r.r3, ox2, oy2, D2, cb2, mask, p.w2x, p.w2y);
    P.half += 1;
    // As unsigned numbers, the bit patterns of the floats in [0, 1) lie below
    // that of 1, all others (1 itself among them, hence "may") from there on,
    // and half_end - half once it is negative.
    uint32_t m = max(max(__float_as_uint(p.xh), __float_as_uint(p.yh)), __float_as_uint(L.xh));
    m = max(max(m, __float_as_uint(L.yh)), (uint32_t)(P.half_end - P.half));
    bool ends = m >= 0x3f800000u;
    p.side1 = p.side2 = -1;
    if constexpr (BRIDGE) {
        // The bridge tests of both steps; their uniforms are words 0 and 1 of
        // Philox(k/2, path, node, ctr3 | 4).
        const PhiloxOut u =
            philox4x32_10_lane((uint32_t)P.half - 1u, PhiloxLane{P.bridge_ck, P.pp.bk, P.pp.hk, P.pp.lk}, keys);
        const SideDist d1 = side_dist(p.xh, p.xl, p.yh, p.yl), d2 = side_dist(L);
        const float p1 = bridge_prob(P.dist, d1, iD1, p.side1), p2 = bridge_prob(d1, d2, iD2, p.side2);
        p.side1 = bridge_uniform(u.r0) < p1 ? p.side1 : -1;
        p.side2 = bridge_uniform(u.r1) < p2 ? p.side2 : -1;
        ends |= (p.side1 & p.side2) >= 0;
        P.dist = d2;
    }
    return ends;
}

// How a path ends in the pair just taken: not (0), with its first step (1) or
// with its second one (2).
__device__ __forceinline__ int pair_ends(const Lane &L, const PairLane &P, const Pair &p) {
    const int32_t k0 = 2 * P.half - 2;
    if (outside(p.xh, p.xl, p.yh, p.yl) || p.side1 >= 0 || k0 + 1 >= L.K) return 1;
    return outside(L.xh, L.xl, L.yh, L.yl) || p.side2 >= 0 || k0 + 2 >= L.K ? 2 : 0;
}

// The end state of a path that ended with step `with` of the pair: its
// position, its steps in L.k; true if it left the square.
template <bool BRIDGE>
__device__ __forceinline__ bool pair_end(Lane &L, const PairLane &P, const Pair &p, int with) {
    const bool first = with == 1;
    if (first) {
        L.xh = p.xh;
        L.xl = p.xl;
        L.yh = p.yh;
        L.yl = p.yl;
    }
    const bool cross = outside(L.xh, L.xl, L.yh, L.yl);
    const int side = first ? p.side1 : p.side2;
    const bool out = L.K > 0 && (cross || side >= 0);
    if (L.K <= 0) {
        L.xh = L.px;
        L.xl = L.horizon;
        L.yh = L.py;
        L.yl = L.dt_last;
    }
    if constexpr (BRIDGE) move_to_side(L, cross || !out ? -1 : side);
    L.k = out ? 2 * P.half - (first ? 1 : 0) : L.K;
    return out;
}

// Score of a finished path (eq. (7b)): boundary data at the exit point if
// it left the square (out), else the initial data at its end point.  With
// a.shift the identity scores are stored relative to the start point.
// FK_SCORE_EXTEND scores an exit with the grid initial data extrapolated
// bilinearly to the exit point (grid_bilinear extrapolates off the grid);
// FK_SCORE_PROJECT, FK_SCORE_BRIDGE and FK_SCORE_EXPONENTIAL score it at
// the point clamped onto the square (boundary data FK_DATA_GRID: the grid's
// edge there).
__device__ __forceinline__ void score_path(const PathArgs &a, const Lane &L, bool out, float &sx, float &sy) {
    const int kind = out ? (a.score_mode == FK_SCORE_EXTEND ? FK_DATA_GRID : a.bdry_kind) : a.init_kind;
    float x = L.xh, y = L.yh;
    float lx = L.xl, ly = L.yl;
    if (out && (a.score_mode == FK_SCORE_PROJECT || a.score_mode == FK_SCORE_BRIDGE ||
                a.score_mode == FK_SCORE_EXPONENTIAL)) {
        if (x < 0.f || x > 1.f) { x = fminf(fmaxf(x, 0.f), 1.f); lx = 0.f; }
        if (y < 0.f || y > 1.f) { y = fminf(fmaxf(y, 0.f), 1.f); ly = 0.f; }
    }
    // zero data (FK_DATA_ZERO); formed here, ahead of the branches: as a last
    // branch's constants they were lost in some variants' code
    asm("v_mov_b32 %0, 0" : "=v"(sx));
    asm("v_mov_b32 %0, 0" : "=v"(sy));
    if (kind == FK_DATA_IDENTITY) {
        const float bx0 = a.shift ? L.px : 0.f, by0 = a.shift ? L.py : 0.f;
        sx = (x - bx0) + lx;
        sy = (y - by0) + ly;
    } else if (kind == FK_DATA_SIN) {
        float v = sin_mode(x, y);
        if (out) {
            // elapsed time since the initial data: t - s_kappa
            float s = (L.k >= L.K) ? L.horizon : (float)L.k * L.dt;
            if (a.score_mode == FK_SCORE_EXPONENTIAL) s = L.s_hi + L.s_lo;
            v *= hw_exp2(-2.f * 9.8696044f * 1.44269504f * (L.horizon - s));
        }
        sx = v;
        sy = v;
    } else if (kind == FK_DATA_GRID) {
        sx = grid_bilinear(a.grid_xi, a.grid_n, x, y);
        // one grid at a time: keeps the scoring's registers below the path
        // loop's (this runs once per path)
        __builtin_amdgcn_sched_barrier(0);
        sy = grid_bilinear(a.grid_eta, a.grid_n, x, y);
    }
}

}  // namespace fk
