// fk_paths.hip -- the Monte-Carlo hot path: a persistent path kernel (one
// path per lane, lanes refilled from a device work queue as their paths
// end) and the FP64 estimator reduction.
//
// Method (Sect. 3, eqs. (5)-(7); Sect. 4): for an interface node P, a path
// X_0 = P, X_{k+1} = X_k + b(tau_k, X_k) D_k + sqrt(2 D_k) z_k takes
// Euler-Maruyama steps of dX = -(grad w / w) ds + sqrt(2) dW with a boundary
// test after every step.  A path that leaves the square scores the boundary
// data at its exit point; a path alive after K steps scores the initial data.
// The node value is the mean of the scores over its paths.
//
// MI355X mapping:
//  * The path loop is bound by VALU issue (per pair of steps: 18 64-bit
//    multiplies and 20 bit operations of one Philox call, 10-14 hardware
//    transcendentals, ~60 FP32 ops) and touches no memory, so every lane keeps
//    its whole path state in registers.
//  * Exit times vary by two orders of magnitude between nodes and
//    geometrically within a node; lanes therefore refill individually: a
//    wavefront grabs `chunk` consecutive paths of one node from a global
//    atomic queue and hands them to whichever lanes are idle, so a lane never
//    waits for the rest of its wavefront.  Nodes are queued in decreasing
//    expected cost so the launch ends on short paths.
//  * Each finished path adds its score to its node's sums inside the kernel
//    (fixed-point integer sums: per wavefront in LDS per work chunk, then
//    per node in HBM), so results do not depend on the launch schedule and
//    no per-path record is written unless the caller asks for the scores;
//    a small kernel turns the sums into means and standard errors.
//  * Positions are FP32 pairs (hi, lo): each increment is added to lo and the
//    pair renormalised, which keeps the position to ~2^-48 over 10^4 steps
//    (plain FP32 accumulation drifts by ~1e-6 and flips exit decisions).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <utility>

#include "fk_accum.hpp"
#include "fk_device.hpp"
#include "fk_internal.hpp"
#include "fk_pathstep.hpp"

namespace fk {

__global__ void zero_u32_kernel(uint32_t *p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

hipError_t launch_zero_u32(uint32_t *p, int n_words, hipStream_t s) {
    const int blocks = (n_words + 255) / 256;
    hipLaunchKernelGGL(zero_u32_kernel, dim3(blocks), dim3(256), 0, s, p, n_words);
    return hipGetLastError();
}

__global__ void counters_init_kernel(uint32_t *c, uint32_t total_chunks) {
    const int i = threadIdx.x;
    if (i < 64) c[i] = (i == kCtrTotal) ? total_chunks : 0u;
}

hipError_t launch_counters_init(uint32_t *counters, uint32_t total_chunks, hipStream_t s) {
    hipLaunchKernelGGL(counters_init_kernel, dim3(1), dim3(64), 0, s, counters, total_chunks);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Node tables from device coordinates.  Nodes are queued in decreasing
// expected cost -- a proxy of the mean exit time, capped by the horizon --
// bucketed into kCostBuckets classes (the order within a class is that of
// the atomics: it only changes the schedule, never a result, since every
// path draws its numbers by its own counters).
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool node_wanted(const TableArgs &t, int64_t i, double &x, double &y, bool &ok) {
    x = t.pts[2 * i];
    y = t.pts[2 * i + 1];
    ok = (x >= 0.0 && x <= 1.0 && y >= 0.0 && y <= 1.0);   // false for NaN
    return !t.mask || t.mask[i];
}

__device__ __forceinline__ int cost_bucket(const TableArgs &t, double x, double y) {
    if (!t.sort) return 0;
    const double ax = x * (1.0 - x), ay = y * (1.0 - y);
    double c = 0.0;
    if (ax > 0.0 && ay > 0.0) c = fmin((double)t.horizon, 1.0 / (2.0 / ax + 2.0 / ay));
    const double f = t.horizon > 0.f ? c / (double)t.horizon : 0.0;     // in [0, 1]
    return min(kCostBuckets - 1, max(0, (int)((1.0 - f) * kCostBuckets)));
}

// Adds, for every lane with `take`, one to hist[b] -- one atomic per
// distinct b in the wavefront (a mesh step's nodes mostly share a bucket,
// and one atomic per node on one address serialises) -- and returns the
// lane's slot: the old count plus its rank among the wavefront's lanes with
// the same b.  Every lane of the wavefront calls it.
__device__ __forceinline__ uint32_t wave_bucket_add(uint32_t *hist, bool take, int b) {
    const int lane = (int)(threadIdx.x & 63u);
    uint64_t left = ballot(take);
    uint32_t slot = 0;
    while (left != 0ull) {
        const int leader = __builtin_ctzll(left);
        const int lb = __shfl(b, leader, 64);
        const bool mine = take && b == lb;
        const uint64_t grp = ballot(mine);
        uint32_t base = 0;
        if (lane == leader) base = atomicAdd(&hist[lb], (uint32_t)__popcll(grp));
        base = (uint32_t)__shfl((int)base, leader, 64);
        if (mine) slot = base + __builtin_amdgcn_mbcnt_hi((uint32_t)(grp >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)grp, 0u));
        left &= ~grp;
    }
    return slot;
}

__global__ void table_count_kernel(const TableArgs t) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) *t.levels_out = t.level;
    bool take = false;
    int bucket = 0;
    if (i < t.n) {
        double x, y;
        bool ok;
        const bool want = node_wanted(t, i, x, y, ok);
        OutDev o{};
        o.shift_x = t.shift ? (double)(float)x : 0.0;
        o.shift_y = t.shift ? (double)(float)y : 0.0;
        o.K = t.level.K;
        t.outs_out[i] = o;
        if (t.outs_zero_out) {
            o.shift_x = o.shift_y = 0.0;
            t.outs_zero_out[i] = o;
        }
        if (want && !ok) {
            // not a node of the square: no paths, NaN results
            t.acc[i].bad = 1u;
            if (t.acc2) t.acc2[i].bad = 1u;
        }
        take = want && ok;
        if (take) bucket = cost_bucket(t, x, y);
    }
    wave_bucket_add(t.counters + kCtrHist, take, bucket);
}

__global__ void table_scan_kernel(uint32_t *c, uint32_t cpn) {
    if (threadIdx.x != 0) return;
    uint32_t run = 0;
    for (int b = 0; b < kCostBuckets; ++b) {
        const uint32_t k = c[kCtrHist + b];
        c[kCtrHist + b] = run;
        run += k;
    }
    c[kCtrActive] = run;
    c[kCtrTotal] = run * cpn;
}

__global__ void table_scatter_kernel(const TableArgs t) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double x = 0.0, y = 0.0;
    bool ok = false, take = false;
    int bucket = 0;
    if (i < t.n) {
        take = node_wanted(t, i, x, y, ok) && ok;
        if (take) bucket = cost_bucket(t, x, y);
    }
    const uint32_t slot = wave_bucket_add(t.counters + kCtrHist, take, bucket);
    if (!take) return;
    NodeDev nd{};
    // the start point as an FP32 (hi, lo) pair holding the FP64 node to ~2^-48
    nd.x = (float)x + 0.f;   // + 0: no -0, whose sign bit the path kernels would look at
    nd.y = (float)y + 0.f;
    nd.xlo = (float)(x - (double)nd.x);
    nd.ylo = (float)(y - (double)nd.y);
    nd.nid = (uint32_t)i;
    nd.level = 0;
    nd.out = (uint64_t)i;
    t.nodes_out[slot] = nd;
}

hipError_t launch_tables(const TableArgs &t, hipStream_t s) {
    const unsigned blocks = (unsigned)std::max<int64_t>(1, (t.n + 255) / 256);
    hipLaunchKernelGGL(table_count_kernel, dim3(blocks), dim3(256), 0, s, t);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(table_scan_kernel, dim3(1), dim3(64), 0, s, t.counters, t.cpn);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(table_scatter_kernel, dim3(blocks), dim3(256), 0, s, t);
    return hipGetLastError();
}

// Node tables of the short-horizon kernel (fk_short.hip): the sums cleared,
// the nodes in the caller's order (their paths all cost about the same), or
// with a mask the wanted ones packed.  A node outside the square keeps its
// place, marked by a NaN low part: without a mask a node's slot is its index,
// so nothing is counted.
__global__ void short_table_kernel(const TableArgs t, unsigned long long *total_steps) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) {
        *t.levels_out = t.level;
        if (total_steps) *total_steps = 0ull;
        if (!t.mask) t.counters[kCtrActive] = (uint32_t)t.n;
    }
    bool take = false, ok = false;
    double x = 0.0, y = 0.0;
    if (i < t.n) {
        take = node_wanted(t, i, x, y, ok);
        OutDev o{};
        o.shift_x = t.shift ? (double)(float)x : 0.0;
        o.shift_y = t.shift ? (double)(float)y : 0.0;
        o.K = t.level.K;
        t.outs_out[i] = o;
        if (t.outs_zero_out) {
            o.shift_x = o.shift_y = 0.0;
            t.outs_zero_out[i] = o;
        }
        NodeAcc z{};
        z.bad = take && !ok ? 1u : 0u;
        t.acc[i] = z;
        if (t.acc2) t.acc2[i] = z;
    }
    uint32_t slot = (uint32_t)i;
    if (t.mask) slot = wave_bucket_add(t.counters + kCtrActive, take, 0);
    if (!take) return;
    NodeDev nd{};
    nd.x = ok ? (float)x + 0.f : 0.5f;   // + 0: no -0, whose sign bit the kernel would look at
    nd.y = ok ? (float)y + 0.f : 0.5f;
    nd.xlo = ok ? (float)(x - (double)nd.x) : __builtin_nanf("");
    nd.ylo = ok ? (float)(y - (double)nd.y) : 0.f;
    nd.nid = (uint32_t)i;
    nd.level = 0;
    nd.out = (uint64_t)i;
    t.nodes_out[slot] = nd;
}

hipError_t launch_short_tables(const TableArgs &t, unsigned long long *total_steps, hipStream_t s) {
    hipError_t e;
    if (t.mask && (e = launch_counters_init(t.counters, 0u, s)) != hipSuccess) return e;
    const unsigned blocks = (unsigned)std::max<int64_t>(1, (t.n + 255) / 256);
    hipLaunchKernelGGL(short_table_kernel, dim3(blocks), dim3(256), 0, s, t, total_steps);
    return hipGetLastError();
}

// BRIDGE: the Brownian-bridge crossing test after every step that stays
// inside (score mode FK_SCORE_BRIDGE).  FEW_STEPS (horizons of 33 to 64 steps
// over which paths leave): steps with a branch after each (two_steps), on seven
// wavefronts per SIMD, and a wavefront's first chunk is its index in the grid,
// later ones come from the counter past the first grid-full, so a launch of
// short paths does not open with every wavefront contending for the counter.
// Long horizons keep the counter for every grab (the other form costs their
// hot loop ~3% in code).  Ring and moving bump, 1521 nodes x 4096 paths, 64
// steps over t = 0.1: 736 and 605 us, in branch-free pairs 785 and 628 us; a
// path ends every second pair or so of a wavefront there.  (With 100 paths a
// node 79 against 71 us: pairs would be faster where the chip is part-empty.)
//
// The inner loop of the others takes step pairs without a branch until some
// lane's path may have ended: both steps are taken at once, and one unsigned
// maximum over the four new coordinates and the pair count finds the
// wavefronts that have to look closer.  The two forms share the scoring below
// as it stands: in a function or lambda of its own it changes the order of the
// pair loop's instructions, and 73920 paths per node take 628 ms, not 598.  Idle lanes hold a point that stays at (0.5, 0.5).  Scores,
// refill and queue stand outside the inner loop: kept in one loop they cost
// it ~20 register moves a pair.  Five to six wavefronts per SIMD (78 - 96
// registers, 15 of them Philox round keys): with the keys in scalar registers
// eight fit, and run 2% slower; forced to 72 or 64 registers the kernel
// spills.  Measured (moving bump, 1521 nodes x 4096 paths x <= 10^4 steps):
// 35.5 ms, 117 VALU instructions and ~410 issue cycles a pair, against
// 41.1 ms of the form with a branch after each step; with the bridge test
// (125 nodes x 16384 paths to their exits) 4.6 ms against 6.9, of which the
// one Philox call for the uniforms of both steps and a position that stays
// in registers are the larger part.  A wavefront alone on its SIMD takes 1050
// cycles a pair, 2.2 ms for 10^4 steps; while the wavefronts thin out after
// the queue has run empty ~5 ms pass at six per SIMD and half that at three
// (the default there: long_blocks, fk_api.hip).
template <int KIND, int TMODE, bool UNIFORM, bool BRIDGE, bool FEW_STEPS = false>
__global__ void __launch_bounds__(256, 5) fk_path_kernel(const PathArgs a) {
    const uint32_t lane = threadIdx.x & 63u;
    __shared__ AccSlot<2> slot_tab[4][kAccSlots];
    AccSlot<2> *slots = slot_tab[threadIdx.x >> 6];
    NodeAcc *const accs[1] = {a.acc};
    slots_init<2>(slots, lane);
    // Wavefront-uniform queue cursor: current node slot and path range, and
    // the grab number of the chunk (its accumulation slot).
    uint32_t q_slot = 0, q_next = 0, q_end = 0, q_tag = 0, grabs = 0;
    bool q_done = false;
    const uint32_t total_chunks = launch_chunks(a);
    if constexpr (FEW_STEPS) {
        q_done = !chunk_cursor(a, total_chunks, first_chunk(), q_slot, q_next, q_end);
        if (!q_done) {
            q_tag = slot_open<2>(slots, accs, grabs++, (uint32_t)a.nodes[q_slot].out, q_end - q_next, lane);
        }
    }
    const uint32_t key0 = a.key0, key1 = a.key1;
    const PhiloxKeys keys = philox_keys(key0, key1);
    const uint32_t mask = in_vgpr(kUnitMask);

    Lane L;
    PairLane P{};
    PhiloxPath pp{};          // the lane's path's fixed Philox products
    uint32_t my_tag = 0;      // accumulation tag of the lane's path's chunk
    uint32_t my_steps = 0;
    uint64_t act = 0;         // the lanes with a path
    if constexpr (!FEW_STEPS) {
        lane_level<KIND, TMODE>(L, a.levels[0]);
        pair_idle<BRIDGE>(L, P);
    }

    for (;;) {
        // ---- refill idle lanes -------------------------------------------
        while (~act != 0ull && !q_done) {
            if (q_next >= q_end) {
                if constexpr (FEW_STEPS) {
                    // a grid no larger than the chunk count hands out no more
                    // chunks: finish without touching the counter
                    if (gridDim.x * (blockDim.x >> 6) >= total_chunks) {
                        q_done = true;
                        break;
                    }
                }
                uint32_t c = 0;
                if (lane == 0) c = atomicAdd(a.queue, 1u);
                c = __builtin_amdgcn_readfirstlane(c);
                if constexpr (FEW_STEPS) c += gridDim.x * (blockDim.x >> 6);
                if (c >= total_chunks) {
                    q_done = true;
                    break;
                }
                uint32_t pc;
                chunk_slot(a, total_chunks, c, q_slot, pc);
                q_next = pc * a.chunk;
                q_end = min(q_next + a.chunk, a.n_paths);
                q_tag = slot_open<2>(slots, accs, grabs++, (uint32_t)a.nodes[q_slot].out, q_end - q_next, lane);
                continue;
            }
            const uint64_t need = ~act;
            const uint32_t avail = q_end - q_next;
            const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(need >> 32),
                                                            __builtin_amdgcn_mbcnt_lo((uint32_t)need, 0u));
            const bool take = __builtin_amdgcn_inverse_ballot_w64(need) && rank < avail;
            if (take) {
                lane_start<KIND, TMODE>(L, a.nodes[q_slot], a.levels, q_next + rank);
                if constexpr (FEW_STEPS) pp = philox_path(L.path, L.nid, key0);
                else pair_start<BRIDGE>(L, P, key0, key1);
                my_tag = q_tag;
            }
            act |= ballot(take);
            q_next += min((uint32_t)__popcll(need), avail);
        }
        if (act == 0ull) break;

        // ---- two steps, or step pairs until a path ends -------------------------
        Pair p;
        uint64_t fin;             // the lanes whose path has ended
        int with = 0;
        bool out = false;
        if constexpr (FEW_STEPS) {
            bool end = false;
            if (__builtin_amdgcn_inverse_ballot_w64(act)) {
                float dbx = 0.f, dby = 0.f;
                if (L.k < L.K) {
                    const PhiloxOut r = philox4x32_10_path((uint32_t)L.k >> 1, L.ctr3, pp, key0, key1);
                    out = two_steps<KIND, TMODE, UNIFORM>(L, r, dbx, dby);
                }
                end = out || L.k >= L.K;
            }
            fin = ballot(end);
        } else {
            do {
                fin = ballot(pair_step<KIND, TMODE, UNIFORM, BRIDGE>(L, P, keys, mask, p)) & act;
            } while (fin == 0ull);
            with = pair_ends(L, P, p);
            fin &= ballot(with != 0);
        }

        // ---- score (eq. (7b)) and the node's sums ------------------------------
        bool closed = false;      // the lane's path closed its chunk's slot
        if (__builtin_amdgcn_inverse_ballot_w64(fin)) {
            if constexpr (!FEW_STEPS) out = pair_end<BRIDGE>(L, P, p, with);
            float v[2];
            score_path(a, L, out, v[0], v[1]);
            closed = acc_path<2>(slots, accs, my_tag, L.out, v, (uint32_t)L.k);
            my_steps += (uint32_t)L.k;      // the path's steps, counted once at its end
            if (a.scores) a.scores[path_rec(L, a.n_paths)] = make_float2(v[0], v[1]);
            if (a.exit_step) a.exit_step[path_rec(L, a.n_paths)] = out ? L.k : -1;
            if constexpr (!FEW_STEPS) pair_idle<BRIDGE>(L, P);
        }
        act &= ~fin;
        if (ballot(closed) != 0ull) slots_collect<2>(slots, accs, lane);
    }

    // ---- the last closed chunks' sums ----------------------------------------
    slots_collect<2>(slots, accs, lane);
    // ---- step count: wavefront sum, one atomic per wavefront --------------
    unsigned long long st = my_steps;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) st += __shfl_xor(st, off, 64);
    // a null count: the caller did not ask for it (every kernel skips it)
    if (lane == 0 && st != 0ull && a.total_steps) atomicAdd(a.total_steps, st);
}

// Exponential time-stepping (FK_SCORE_EXPONENTIAL): the same persistent
// queue and in-kernel estimator as fk_path_kernel; each step has its own
// length D = -dt ln u (u from word 2 + (k & 1) of Philox(k/2, path, node,
// ctr3 | 4)), cut at the horizon, then the Euler-Maruyama step of length D
// and the bridge test for D with that Philox call's word k & 1.  The elapsed
// time is kept as a hi + lo pair; the orbit angle of a moving density at
// PDE time t_init + t - s follows it.  A path ends when it exits or when
// the cut step has been taken (L.K is set to the step count then).
template <int KIND, int TMODE>
__global__ void __launch_bounds__(256) fk_expo_path_kernel(const PathArgs a) {
    constexpr bool kMovingBackward = moving_kind(KIND) && TMODE == TIME_BACKWARD;
    const uint32_t lane = threadIdx.x & 63u;
    __shared__ AccSlot<2> slot_tab[4][kAccSlots];
    AccSlot<2> *slots = slot_tab[threadIdx.x >> 6];
    NodeAcc *const accs[1] = {a.acc};
    slots_init<2>(slots, lane);
    uint32_t q_slot = 0, q_next = 0, q_end = 0, q_tag = 0, grabs = 0;
    bool q_done = false;
    const uint32_t total_chunks = launch_chunks(a);
    const uint32_t key0 = a.key0, key1 = a.key1;
    Lane L;
    bool active = false;
    uint32_t my_tag = 0, my_steps = 0;
    bool closed = false;
    for (;;) {
        if (ballot(closed) != 0ull) {
            slots_collect<2>(slots, accs, lane);
            closed = false;
        }
        uint64_t need = ballot(!active);
        while (need != 0ull && !q_done) {
            if (q_next >= q_end) {
                uint32_t c = 0;
                if (lane == 0) c = atomicAdd(a.queue, 1u);
                c = __builtin_amdgcn_readfirstlane(c);
                if (!grab_chunk<2>(a, total_chunks, c, q_slot, q_next, q_end, slots, accs, q_tag, grabs, lane)) {
                    q_done = true;
                    break;
                }
                continue;
            }
            const uint32_t avail = q_end - q_next;
            const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(need >> 32),
                                                            __builtin_amdgcn_mbcnt_lo((uint32_t)need, 0u));
            if (!active && rank < avail) {
                lane_start<KIND, TMODE>(L, a.nodes[q_slot], a.levels, q_next + rank);
                L.K = L.K > 0 ? 0x7fffffff : 0;      // open-ended; 0 for a zero horizon
                L.s_hi = 0.f;
                L.s_lo = 0.f;
                my_tag = q_tag;
                active = true;
            }
            q_next += min((uint32_t)__popcll(need), avail);
            need = ballot(!active);
        }
        if (ballot(active) == 0ull) break;

        if (active) {
            bool out = false;
            if (L.k < L.K) {
                const PhiloxOut r = philox4x32_10((uint32_t)L.k >> 1, L.path, L.nid, L.ctr3, key0, key1);
                const PhiloxOut q = philox4x32_10((uint32_t)L.k >> 1, L.path, L.nid, L.ctr3 | 4u, key0, key1);
                const bool odd = (L.k & 1) != 0;
                const float u = fmaf((float)((odd ? q.r3 : q.r2) >> 8), 0x1p-24f, 0x1p-24f);
                float D = -0.69314718f * L.dt * hw_log2(u);
                const float rem = (L.horizon - L.s_hi) - L.s_lo;
                const bool last = D >= rem;
                D = last ? rem : D;
                float ox = L.ox, oy = L.oy;
                if constexpr (kMovingBackward) {
                    const float rev = fmaf(-L.s_hi, L.dens.omega_rev, L.rev0);
                    ox = L.dens.orbit_r * hw_cos_rev(rev);
                    oy = L.dens.orbit_r * hw_sin_rev(rev);
                }
                float dwx, dwy;
                brownian_increment(odd ? r.r2 : r.r0, odd ? r.r3 : r.r1, -2.77258872f * D, dwx, dwy);
                float bx, by;
                drift<KIND>(L.dens, ox, oy, L.xh, L.yh, bx, by);
                const SideDist d0 = side_dist(L);
                comp_add(L.xh, L.xl, fmaf(bx, D, dwx));
                comp_add(L.yh, L.yl, fmaf(by, D, dwy));
                if (last) {
                    L.s_hi = L.horizon;
                    L.s_lo = 0.f;
                } else {
                    comp_add(L.s_hi, L.s_lo, D);
                }
                L.k += 1;
                my_steps += 1;
                const float lo = fminf(L.xh, L.yh);
                const float hi = fmaxf((L.xh - 1.f) + L.xl, (L.yh - 1.f) + L.yl);
                out = (lo < 0.f) | (hi > 0.f);
                if (!out) {
                    int side;
                    const float p = bridge_prob(d0, side_dist(L), 1.f / D, side);
                    out = side >= 0 && bridge_uniform(odd ? q.r1 : q.r0) < p;
                    if (out) move_to_side(L, side);
                }
                if (last) L.K = L.k;
            }
            if (out || L.k >= L.K) {
                float v[2];
                score_path(a, L, out, v[0], v[1]);
                closed = acc_path<2>(slots, accs, my_tag, L.out, v, (uint32_t)L.k);
                if (a.scores) a.scores[path_rec(L, a.n_paths)] = make_float2(v[0], v[1]);
                if (a.exit_step) a.exit_step[path_rec(L, a.n_paths)] = out ? L.k : -1;
                active = false;
            }
        }
    }
    slots_collect<2>(slots, accs, lane);
    unsigned long long st = my_steps;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) st += __shfl_xor(st, off, 64);
    if (lane == 0 && st != 0ull && a.total_steps) atomicAdd(a.total_steps, st);
}

namespace {
template <int KIND, int TMODE, bool UNIFORM, bool BRIDGE, bool FEW_STEPS>
hipError_t launch_one(const PathArgs &a, int grid, int block, hipStream_t s) {
    hipLaunchKernelGGL((fk_path_kernel<KIND, TMODE, UNIFORM, BRIDGE, FEW_STEPS>), dim3(grid), dim3(block), 0, s, a);
    return hipGetLastError();
}

template <int KIND, int TMODE, bool UNIFORM, bool BRIDGE, bool FEW_STEPS>
int max_blocks(int block) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fk_path_kernel<KIND, TMODE, UNIFORM, BRIDGE, FEW_STEPS>, block,
                                                     0) != hipSuccess)
        return 0;
    return nb;
}

// Calls F<KIND, TMODE, UNIFORM, BRIDGE, FEW_STEPS>::run(args...) for the runtime
// values; the few-steps form only without the bridge test.
template <template <int, int, bool, bool, bool> class F, typename... Args>
auto dispatch(int kind, int time_mode, bool uniform, bool bridge, bool few_steps, Args &&...args) {
    const bool frozen = (time_mode == TIME_FROZEN);
#define FK_CASE(K, T)                                                                          \
    if (bridge)                                                                                \
        return uniform ? F<K, T, true, true, false>::run(std::forward<Args>(args)...)         \
                       : F<K, T, false, true, false>::run(std::forward<Args>(args)...);       \
    if (few_steps)                                                                             \
        return uniform ? F<K, T, true, false, true>::run(std::forward<Args>(args)...)         \
                       : F<K, T, false, false, true>::run(std::forward<Args>(args)...);       \
    return uniform ? F<K, T, true, false, false>::run(std::forward<Args>(args)...)            \
                   : F<K, T, false, false, false>::run(std::forward<Args>(args)...)
    switch (kind) {
    case KIND_CONST: FK_CASE(KIND_CONST, TIME_BACKWARD);
    case KIND_BUMP: FK_CASE(KIND_BUMP, TIME_BACKWARD);
    case KIND_RIDGE: FK_CASE(KIND_RIDGE, TIME_BACKWARD);
    case KIND_GRID: FK_CASE(KIND_GRID, TIME_BACKWARD);
    case KIND_MOVING:
        if (frozen) { FK_CASE(KIND_MOVING, TIME_FROZEN); }
        FK_CASE(KIND_MOVING, TIME_BACKWARD);
    case KIND_RING:
        if (frozen) { FK_CASE(KIND_RING, TIME_FROZEN); }
        FK_CASE(KIND_RING, TIME_BACKWARD);
    default:
        if (frozen) { FK_CASE(KIND_TWO, TIME_FROZEN); }
        FK_CASE(KIND_TWO, TIME_BACKWARD);
    }
#undef FK_CASE
}

template <int K, int T, bool U, bool B, bool F>
struct LaunchF {
    static hipError_t run(const PathArgs &a, int grid, int block, hipStream_t s) {
        return launch_one<K, T, U, B, F>(a, grid, block, s);
    }
};
template <int K, int T, bool U, bool B, bool F>
struct OccF {
    static int run(int block) { return max_blocks<K, T, U, B, F>(block); }
};

bool kind_known(int kind) {
    return kind == KIND_CONST || kind == KIND_BUMP || kind == KIND_RIDGE || kind == KIND_MOVING || kind == KIND_TWO ||
           kind == KIND_RING || kind == KIND_GRID;
}
}  // namespace

hipError_t launch_paths(int kind, int time_mode, bool uniform, bool few_steps, const PathArgs &a, int grid,
                        int block, hipStream_t s) {
    if (!kind_known(kind)) return hipErrorInvalidValue;
    return dispatch<LaunchF>(kind, time_mode, uniform, a.score_mode == FK_SCORE_BRIDGE, few_steps, a, grid,
                             block, s);
}

int path_kernel_max_blocks_per_cu(int kind, int time_mode, bool uniform, bool bridge, bool few_steps,
                                  int block) {
    if (!kind_known(kind)) return 0;
    return dispatch<OccF>(kind, time_mode, uniform, bridge, few_steps, block);
}

namespace {
template <int K, int T, bool U, bool B, bool F>
struct ExpoLaunchF {
    static hipError_t run(const PathArgs &a, int grid, int block, hipStream_t s) {
        hipLaunchKernelGGL((fk_expo_path_kernel<K, T>), dim3(grid), dim3(block), 0, s, a);
        return hipGetLastError();
    }
};
template <int K, int T, bool U, bool B, bool F>
struct ExpoOccF {
    static int run(int block) {
        int nb = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fk_expo_path_kernel<K, T>, block, 0) != hipSuccess)
            return 0;
        return nb;
    }
};
}  // namespace

// The kind / time-mode dispatch of the fixed-step kernels, with one
// instantiation per pair (uniform, bridge and first-chunk flags unused).
hipError_t launch_expo_paths(int kind, int time_mode, const PathArgs &a, int grid, int block, hipStream_t s) {
    if (!kind_known(kind)) return hipErrorInvalidValue;
    return dispatch<ExpoLaunchF>(kind, time_mode, false, false, false, a, grid, block, s);
}

int expo_kernel_max_blocks_per_cu(int kind, int time_mode, int block) {
    if (!kind_known(kind)) return 0;
    return dispatch<ExpoOccF>(kind, time_mode, false, false, false, block);
}

// ---------------------------------------------------------------------------
// Estimator (Sect. 4: expectations replaced by arithmetic means): the node
// sums of the path kernel -> mean, sample variance (N - 1), standard error,
// in FP64; one thread per output node.
// ---------------------------------------------------------------------------
size_t acc_bytes(int64_t n_out) { return sizeof(NodeAcc) * (size_t)(n_out > 0 ? n_out : 0); }

__global__ void __launch_bounds__(256) fk_finalize_kernel(const FinalArgs f) {
    const int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (o < f.n_out && (!f.mask || f.mask[o])) {
        const NodeAcc &A = f.acc[o];
        const double N = (double)f.n_paths;
        double mean[2], se[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const double s1 = split_to_double(A.sum[2 * c]) * (1.0 / kQ1);
            const double s2 = split_to_double(A.sum[2 * c + 1]) * (1.0 / kQ2);
            const double m = s1 / N;
            const double var = fmax((s2 - s1 * m) / (N - 1.0), 0.0);
            mean[c] = m;
            se[c] = sqrt(var / N);
        }
        const bool bad = A.bad != 0u;
        const double nan = __builtin_nan("");
        f.xi[o] = bad ? nan : f.outs[o].shift_x + mean[0];
        f.eta[o] = bad ? nan : f.outs[o].shift_y + mean[1];
        f.se_xi[o] = bad ? nan : se[0];
        f.se_eta[o] = bad ? nan : se[1];
        if (f.steps) f.steps[o] = (int64_t)A.steps;
    }
    if (!f.total_steps) return;   // the launch's argument
    // the launch's step count, one atomic per wavefront of nodes (the sums of
    // nodes that were not solved are zero)
    unsigned long long st = o < f.n_out ? f.acc[o].steps : 0ull;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) st += __shfl_xor(st, off, 64);
    if ((threadIdx.x & 63u) == 0 && st != 0ull) atomicAdd(f.total_steps, st);
}

hipError_t launch_finalize(const FinalArgs &f, hipStream_t s) {
    if (f.n_out == 0) return hipSuccess;
    const unsigned blocks = (unsigned)((f.n_out + 255) / 256);
    hipLaunchKernelGGL(fk_finalize_kernel, dim3(blocks), dim3(256), 0, s, f);
    return hipGetLastError();
}

}  // namespace fk
