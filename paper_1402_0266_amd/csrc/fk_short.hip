// fk_short.hip -- the path kernel of a mesh step's short horizons: every
// lane of a wavefront runs a path of the same node, and all of them take
// their steps together.
//
// Over a mesh step (a few tens of sub-steps over a short time) nearly every
// path takes all its steps, so lanes need no refill: a wavefront takes
// `chunk` paths of one node, 64 at a time, and a lane whose path leaves the
// square waits for the rest of its 64.  What that buys over the refilling
// kernel (fk_paths.hip):
//  * the node, the step number and with them the density's centre, the step
//    length and rounds 1 to 3 of Philox (but for three products and four
//    XORs) are the wavefront's, formed by the scalar unit or once per node;
//  * a path is scored into its lane's own registers (the same exact
//    fixed-point integers as fk_accum.hpp), and a chunk's sums are reduced
//    once, instead of eight 64-bit LDS atomics per path;
//  * wavefronts take chunks in a fixed stride (all chunks cost about the
//    same), so there is no queue and no counter to clear.
//
// The kernel is bound by VALU issue, so the loop's constants and the round
// keys are kept in vector registers (in_vgpr, fk_device.hpp).
//
// While every path of a wavefront is inside, steps run in pairs without a
// branch (as pair_step, fk_pathstep.hpp); after the first exit, and for the
// pair with the last step, lane by lane under a mask.
//
// Past 32 steps, and with more paths than fit at once (lockstep_refill), a node
// so near a side that most of its paths leave early (short_leaves) has its
// lanes take other paths instead (short_refill): 1521 nodes within 0.02 of a
// side x 4096 paths x 64 steps over 0.05: 680 us in lockstep, 391 in the
// refilling kernel, 242 here.  That takes 5 registers more, and a wavefront per
// SIMD with some densities, so it is a form of its own.
//
// Measured (two bumps frozen, 10689 nodes x 16384 paths x 20 steps): 5.8 ms
// (6.1 with the masked loop alone) against the refilling kernel's 9.7 ms when
// it tested after each step; the ring's 77 nodes x 10^4 paths: 36 us for the
// whole solve against 106 us.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <utility>

#include "fk_accum.hpp"
#include "fk_device.hpp"
#include "fk_internal.hpp"
#include "fk_pathstep.hpp"

namespace fk {

// The same value, formed where it stands: keeps the branch around it (two
// selects per step otherwise).
__device__ __forceinline__ float last_step(float v) {
    asm volatile("" : "+v"(v));
    return v;
}
// A scalar in a vector register, formed where it stands (the step counter
// itself stays a scalar).
__device__ __forceinline__ int32_t step_number(int32_t k) {
    int32_t v;
    asm volatile("v_mov_b32 %0, %1" : "=v"(v) : "s"(k));
    return v;
}

// Philox4x32-10 with every counter word but the path (word 1) wave-uniform.
// After three rounds the uniform words have met the path's word everywhere;
// until then they are scalar work.
struct PhiloxWave {
    uint32_t k0[6], k1[6];   // keys of rounds 5 .. 10
    uint32_t k0r4;           // round 4's first key
};

__device__ __forceinline__ PhiloxWave philox_wave(uint32_t key0, uint32_t key1) {
    PhiloxWave W;
#pragma unroll
    for (int r = 0; r < 6; ++r) {
        W.k0[r] = in_vgpr(key0 + (uint32_t)(r + 4) * kW0);
        W.k1[r] = in_vgpr(key1 + (uint32_t)(r + 4) * kW1);
    }
    W.k0r4 = in_vgpr(key0 + 3u * kW0);
    return W;
}

// philox4x32_10(c0, path, nid, c3, key0, key1) for wave-uniform c0, c3, and
// P = philox_path(path, nid, key0): bitwise the same four words.  nlo: the
// low half of M1 nid (P.b, as a scalar).
__device__ __forceinline__ PhiloxOut philox4x32_10_wave(uint32_t c0, uint32_t c3, uint32_t nlo, const PhiloxPath &P,
                                                        const PhiloxWave &W, uint32_t key0, uint32_t key1) {
    // scalar: round 1's second output pair, round 2's first, round 3's products
    const uint64_t p0 = (uint64_t)kM0 * c0;
    const uint32_t x2 = (uint32_t)(p0 >> 32) ^ c3 ^ key1, x3 = (uint32_t)p0;
    const uint64_t q1 = (uint64_t)kM1 * x2;
    const uint32_t y0 = (uint32_t)(q1 >> 32) ^ nlo ^ (key0 + kW0), y1 = (uint32_t)q1;
    const uint64_t r0 = (uint64_t)kM0 * y0;
    // round 2's third word, the first that depends on the path
    const uint32_t y2 = P.h0 ^ (x3 ^ (key1 + kW1));
    // round 3
    const uint64_t r1 = (uint64_t)kM1 * y2;
    uint32_t v0 = (uint32_t)(r1 >> 32) ^ (y1 ^ (key0 + 2u * kW0)), v1 = (uint32_t)r1;
    uint32_t v2 = P.l0 ^ ((uint32_t)(r0 >> 32) ^ (key1 + 2u * kW1)), v3;
    // round 4 (its fourth word is still scalar)
    {
        const uint64_t a = (uint64_t)kM0 * v0, b = (uint64_t)kM1 * v2;
        const uint32_t n0 = xor3((uint32_t)(b >> 32), v1, W.k0r4);
        const uint32_t n2 = (uint32_t)(a >> 32) ^ ((uint32_t)r0 ^ (key1 + 3u * kW1));
        v1 = (uint32_t)b;
        v3 = (uint32_t)a;
        v0 = n0;
        v2 = n2;
    }
#pragma unroll
    for (int r = 0; r < 6; ++r) {
        const uint64_t a = (uint64_t)kM0 * v0, b = (uint64_t)kM1 * v2;
        const uint32_t n0 = xor3((uint32_t)(b >> 32), v1, W.k0[r]);
        const uint32_t n2 = xor3((uint32_t)(a >> 32), v3, W.k1[r]);
        v1 = (uint32_t)b;
        v3 = (uint32_t)a;
        v0 = n0;
        v2 = n2;
    }
    return PhiloxOut{v0, v1, v2, v3};
}

template <int CTRL>
__device__ __forceinline__ unsigned long long dpp_u64(unsigned long long v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)v, CTRL, 0xf, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(v >> 32), CTRL, 0xf, 0xf, false);
    return ((unsigned long long)hi << 32) | lo;
}

// Sum of a 64-bit integer over the wavefront, wave-uniform: within each row
// of 16 lanes by DPP, then the four rows.
__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v) {
    v += dpp_u64<0xB1>(v);    // quad_perm [1, 0, 3, 2]
    v += dpp_u64<0x4E>(v);    // quad_perm [2, 3, 0, 1]
    v += dpp_u64<0x141>(v);   // row_half_mirror
    v += dpp_u64<0x140>(v);   // row_mirror
    unsigned long long s = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, 16 * r);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), 16 * r);
        s += ((unsigned long long)hi << 32) | lo;
    }
    return s;
}

// What a path's control needs: nothing (the plain estimate), the mesh's
// gradient (as fk_mgg_path_kernel, fk_cv.hip) from memory, or the same from
// the node's tile of the mesh in LDS.  CTL_REFILL: nothing, and nodes near a
// side by short_refill.
enum { CTL_NONE = 0, CTL_MESH = 1, CTL_TILE = 2, CTL_REFILL = 3 };

// The launch's constants of a wavefront.
struct ShortWave {
    Lane L;
    int32_t K;
    uint32_t ctr3, key0, key1;
    float dt, cbm, dt_last, cbm_last, rev0, drev, cos_d, sin_d;
    uint32_t mask;
    PhiloxWave W;
};

template <int KIND, int TMODE>
__device__ __forceinline__ ShortWave short_wave(const PathArgs &a) {
    ShortWave S;
    const LevelDev &lv = a.levels[0];
    lane_level<KIND, TMODE>(S.L, lv);
    S.K = lv.K;
    S.ctr3 = lv.ctr3;
    S.key0 = a.key0;
    S.key1 = a.key1;
    S.dt = in_vgpr(S.L.dt);
    S.cbm = in_vgpr(S.L.cbm);
    S.dt_last = in_vgpr(S.L.dt_last);
    S.cbm_last = in_vgpr(S.L.cbm_last);
    S.rev0 = in_vgpr(S.L.rev0);
    S.drev = in_vgpr(S.L.drev);
    S.cos_d = in_vgpr(S.L.cos_d);
    S.sin_d = in_vgpr(S.L.sin_d);
    S.mask = in_vgpr(kUnitMask);
    S.L.dens.amp = in_vgpr(S.L.dens.amp);
    S.L.dens.nscale = in_vgpr(S.L.dens.nscale);
    S.L.dens.a2s = in_vgpr(S.L.dens.a2s);
    S.L.dens.cx = in_vgpr(S.L.dens.cx);
    S.L.dens.cy = in_vgpr(S.L.dens.cy);
    S.L.dens.orbit_r = in_vgpr(S.L.dens.orbit_r);
    if constexpr (KIND == KIND_GRID) S.L.dens.fn = in_vgpr(S.L.dens.fn);
    S.W = philox_wave(S.key0, S.key1);
    return S;
}

// A tile of the mesh around a node: per grid node the FP32 differences the
// gradient is formed from, to the next node in x (xi, eta) and in y (xi, eta).
constexpr int kTile = 100;
struct MeshTile {
    float4 d[kTile * kTile];
};

__device__ __forceinline__ void load_tile(MeshTile &T, const double *gxi, const double *geta, int n, int i0, int j0) {
    for (int e = threadIdx.x; e < kTile * kTile; e += blockDim.x) {
        const int tj = e / kTile, i = min(i0 + e - kTile * tj, n), j = min(j0 + tj, n);
        const int64_t at = (int64_t)j * (n + 1) + i;
        const int64_t ax = i < n ? at + 1 : at, ay = j < n ? at + (n + 1) : at;
        T.d[e] = make_float4((float)(gxi[ax] - gxi[at]), (float)(geta[ax] - geta[at]), (float)(gxi[ay] - gxi[at]),
                             (float)(geta[ay] - geta[at]));
    }
}

// The gradient of both components at (x, y), bitwise table_gradient's.
template <int CTL>
__device__ __forceinline__ void mesh_gradient(const PathArgs &a, const MggArgs &c, const MeshTile *tile, int i0, int j0,
                                              float x, float y, float (&g)[4]) {
    const int n = a.grid_n;
    if constexpr (CTL == CTL_TILE) {
        const float fx = x * (float)n, fy = y * (float)n;
        int i = (int)floorf(fx), j = (int)floorf(fy);
        i = min(max(i, 0), n - 1);
        j = min(max(j, 0), n - 1);
        const uint32_t ti = (uint32_t)(i - i0), tj = (uint32_t)(j - j0);
        if (max(ti, tj) < (uint32_t)(kTile - 1)) {
            const float ax = fx - (float)i, ay = fy - (float)j;
            const float4 *at = tile->d + (tj * kTile + ti);
            const float4 d = at[0];
            const float2 h = *reinterpret_cast<const float2 *>(at + kTile);
            const float2 v = reinterpret_cast<const float2 *>(at + 1)[1];
            g[0] = (float)n * fmaf(ay, h.x - d.x, d.x);
            g[1] = (float)n * fmaf(ax, v.x - d.z, d.z);
            g[2] = (float)n * fmaf(ay, h.y - d.y, d.y);
            g[3] = (float)n * fmaf(ax, v.y - d.w, d.w);
            return;
        }
    }
    if (c.gtab) {
        table_gradient(c.gtab, n, 0, x, y, g[0], g[1]);
        table_gradient(c.gtab, n, 1, x, y, g[2], g[3]);
    } else {
        grid_gradient(a.grid_xi, n, x, y, g[0], g[1]);
        grid_gradient(a.grid_eta, n, x, y, g[2], g[3]);
    }
}

// The score (eq. (7b)) of an ended path of node nd, at its end point after
// k_end steps, less the control (mx, my); its moments are added to q.
template <int CTL>
__device__ __forceinline__ void short_score(const PathArgs &a, const MggArgs &c, const ShortWave &S, const NodeDev &nd,
                                            uint32_t out_row, uint32_t path, float xh, float xl, float yh, float yl,
                                            int32_t k_end, bool out, float mx, float my, unsigned long long (&q)[4],
                                            uint32_t &steps) {
    constexpr bool MESH = CTL != CTL_NONE;
    const uint64_t rec = (uint64_t)out_row * a.n_paths + path;
    NodeAcc *const accs[1] = {MESH ? c.acc_cv : a.acc};
    Lane E = S.L;
    E.xh = xh;
    E.xl = xl;
    E.yh = yh;
    E.yl = yl;
    E.px = nd.x;
    E.py = nd.y;
    E.k = k_end;
    E.K = S.K;
    float v[2];
    score_path(a, E, out, v[0], v[1]);
    if constexpr (MESH) {
        const float sx0 = a.shift ? nd.x : 0.f, sy0 = a.shift ? nd.y : 0.f;
        v[0] = (v[0] + sx0) - mx;
        v[1] = (v[1] + sy0) - my;
        if (c.cv_scores) c.cv_scores[rec] = make_float2(v[0], v[1]);
    } else {
        if (a.scores) a.scores[rec] = make_float2(v[0], v[1]);
    }
    if (a.exit_step) a.exit_step[rec] = out ? k_end : -1;
    steps += (uint32_t)k_end;
    // (a comparison per value: false for NaN, which a maximum would drop)
    if (fabsf(v[0]) < kLdsBound && fabsf(v[1]) < kLdsBound) {
        q[0] += (unsigned long long)q1_small(v[0]);
        q[1] += (unsigned long long)q2_small(v[0]);
        q[2] += (unsigned long long)q1_small(v[1]);
        q[3] += (unsigned long long)q2_small(v[1]);
    } else {
        acc_direct<2>(accs, out_row, v, fabsf(v[0]) < kGlobalBound && fabsf(v[1]) < kGlobalBound);
    }
}

// Paths next .. end - 1 of node nd without a control, each lane on to another
// one when its own has ended, step by step.
template <int KIND, int TMODE>
__device__ __forceinline__ void short_refill(const PathArgs &a, const ShortWave &S, const NodeDev &nd, uint32_t out_row,
                                             uint32_t nid, uint32_t next, uint32_t end, unsigned long long (&q)[4],
                                             uint32_t &steps) {
    Lane L = S.L;
    L.K = S.K;
    PhiloxPath pp{};
    uint64_t act = 0;
    for (;;) {
        const uint64_t need = ~act;
        if (need != 0ull && next < end) {
            const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(need >> 32),
                                                            __builtin_amdgcn_mbcnt_lo((uint32_t)need, 0u));
            const bool take = __builtin_amdgcn_inverse_ballot_w64(need) && rank < end - next;
            if (take) {
                L.path = next + rank;
                L.xh = nd.x;
                L.xl = nd.xlo;
                L.yh = nd.y;
                L.yl = nd.ylo;
                L.k = 0;
                pp = philox_path(L.path, nid, S.key0);
            }
            act |= ballot(take);
            next += min((uint32_t)__popcll(need), end - next);
        }
        if (act == 0ull) break;
        bool done = false;
        if (__builtin_amdgcn_inverse_ballot_w64(act)) {
            float dbx = 0.f, dby = 0.f;
            const PhiloxOut r = philox4x32_10_path((uint32_t)L.k >> 1, S.ctr3, pp, S.key0, S.key1);
            const bool out = two_steps<KIND, TMODE, false>(L, r, dbx, dby);
            done = out || L.k >= S.K;
            if (done)
                short_score<CTL_NONE>(a, MggArgs{}, S, nd, out_row, L.path, L.xh, L.xl, L.yh, L.yl, L.k, out, 0.f, 0.f, q,
                                      steps);
        }
        act &= ~ballot(done);
    }
}

// Whether most of a node's paths leave early: it lies within 0.56 sqrt(t) of a
// side, where a path takes half of its steps on average (the integral of
// erf(d / (2 sqrt(s))) over s).
__device__ __forceinline__ bool short_leaves(const ShortWave &S, const NodeDev &nd) {
    const float d = fminf(fminf(nd.x, 1.f - nd.x), fminf(nd.y, 1.f - nd.y));
    return d * d < 0.31f * S.L.horizon;
}

// One path per lane of the wavefront (has: the lane holds one), of node nd;
// its moments are added to q, its steps to `steps`.
template <int KIND, int TMODE, int CTL>
__device__ __forceinline__ void short_paths(const PathArgs &a, const MggArgs &c, const ShortWave &S, const NodeDev &nd,
                                            uint32_t out_row, uint32_t nid, float4 ofs, const MeshTile *tile, int i0,
                                            int j0, uint32_t path, bool has, unsigned long long (&q)[4],
                                            uint32_t &steps) {
    constexpr bool kMovingBackward = moving_kind(KIND) && TMODE == TIME_BACKWARD;
    constexpr bool MESH = CTL != CTL_NONE;
    const int32_t K = S.K;
    const uint32_t nlo = kM1 * nid;
    const PhiloxPath pp = philox_path(path, nid, S.key0);
    float xh = nd.x, xl = nd.xlo, yh = nd.y, yl = nd.ylo;
    float g[4] = {0.f, 0.f, 0.f, 0.f}, dbx = 0.f, dby = 0.f, mx = 0.f, my = 0.f;
    uint32_t blk_left = 0;   // pairs of steps to the next block boundary
    bool alive = has;
    int32_t k_end = K;       // steps the lane's path takes

    auto new_block = [&]() {
        mx = fmaf(g[0], dbx, fmaf(g[1], dby, mx));
        my = fmaf(g[2], dbx, fmaf(g[3], dby, my));
        dbx = dby = 0.f;
        mesh_gradient<CTL>(a, c, tile, i0, j0, xh, yh, g);
        if (c.gofs) {
            g[0] += ofs.x;
            g[1] += ofs.y;
            g[2] += ofs.z;
            g[3] += ofs.w;
        }
    };
    // the density's centre offset at step k and at k + 1
    auto centre = [&](int32_t k, float &ox, float &oy, float &ox2, float &oy2) {
        ox = ox2 = S.L.ox;
        oy = oy2 = S.L.oy;
        if constexpr (kMovingBackward) {
            const float rev = fmaf(-(float)k, S.drev, S.rev0);
            const float cr = hw_cos_rev(rev), sr = hw_sin_rev(rev);
            ox = S.L.dens.orbit_r * cr;
            oy = S.L.dens.orbit_r * sr;
            ox2 = S.L.dens.orbit_r * fmaf(cr, S.cos_d, sr * S.sin_d);
            oy2 = S.L.dens.orbit_r * fmaf(sr, S.cos_d, -cr * S.sin_d);
        }
    };

    // ---- while every path is inside: pairs of steps without a branch -------
    // (the loop is the wavefront's: k is a scalar)
    const uint64_t held = ballot(has);
    int32_t k = 0;
    for (; k + 2 < K; k += 2) {
        const PhiloxOut r = philox4x32_10_wave((uint32_t)k >> 1, S.ctr3, nlo, pp, S.W, S.key0, S.key1);
        if constexpr (MESH) {
            if (blk_left == 0) {
                blk_left = c.stride_iters;
                new_block();
            }
            --blk_left;
        }
        float ox, oy, ox2, oy2, w1x, w1y, w2x, w2y;
        centre(k, ox, oy, ox2, oy2);
        float x1h = xh, x1l = xl, y1h = yh, y1l = yl;
        em_move<KIND>(x1h, x1l, y1h, y1l, S.L.dens, r.r0, r.r1, ox, oy, S.dt, S.cbm, S.mask, w1x, w1y);
        xh = x1h;
        xl = x1l;
        yh = y1h;
        yl = y1l;
        em_move<KIND>(xh, xl, yh, yl, S.L.dens, r.r2, r.r3, ox2, oy2, S.dt, S.cbm, S.mask, w2x, w2y);
        const float d1x = dbx + w1x, d1y = dby + w1y;
        if constexpr (MESH) {
            dbx = d1x + w2x;
            dby = d1y + w2y;
        }
        // as in pair_step: not all four coordinates in [0, 1)
        uint32_t m = max(max(__float_as_uint(x1h), __float_as_uint(y1h)), __float_as_uint(xh));
        m = max(m, __float_as_uint(yh));
        if ((ballot(m >= 0x3f800000u) & held) != 0ull) {
            const bool o1 = outside(x1h, x1l, y1h, y1l), o2 = outside(xh, xl, yh, yl);
            if ((ballot(o1 || o2) & held) != 0ull) {
                if (has && o1) {
                    xh = x1h;
                    xl = x1l;
                    yh = y1h;
                    yl = y1l;
                    if constexpr (MESH) {
                        dbx = d1x;
                        dby = d1y;
                    }
                }
                if (has && (o1 || o2)) {
                    alive = false;
                    k_end = step_number(k + 1) + (o1 ? 0 : 1);
                }
                k += 2;
                break;
            }
        }
    }
    // ---- the last pair, and paths that wait for the others -----------------
    float D = S.dt, cb = S.cbm;
    for (; k < K && ballot(alive) != 0ull; k += 2) {
        const PhiloxOut r = philox4x32_10_wave((uint32_t)k >> 1, S.ctr3, nlo, pp, S.W, S.key0, S.key1);
        if constexpr (MESH) {
            if (blk_left == 0) {
                blk_left = c.stride_iters;
                if (alive) new_block();
            }
            --blk_left;
        }
        float ox, oy, ox2, oy2;
        centre(k, ox, oy, ox2, oy2);
        if (k == K - 1) {
            D = last_step(S.dt_last);
            cb = last_step(S.cbm_last);
        }
        float wx, wy;
        if (alive) {
            em_move<KIND>(xh, xl, yh, yl, S.L.dens, r.r0, r.r1, ox, oy, D, cb, S.mask, wx, wy);
            if constexpr (MESH) {
                dbx += wx;
                dby += wy;
            }
            if (outside(xh, xl, yh, yl)) {
                alive = false;
                k_end = step_number(k + 1);
            }
        }
        if (k + 1 >= K) break;
        if (k + 1 == K - 1) {
            D = last_step(S.dt_last);
            cb = last_step(S.cbm_last);
        }
        if (alive) {
            em_move<KIND>(xh, xl, yh, yl, S.L.dens, r.r2, r.r3, ox2, oy2, D, cb, S.mask, wx, wy);
            if constexpr (MESH) {
                dbx += wx;
                dby += wy;
            }
            if (outside(xh, xl, yh, yl)) {
                alive = false;
                k_end = step_number(k + 2);
            }
        }
    }
    if (!has) return;
    mx = fmaf(g[0], dbx, fmaf(g[1], dby, mx));
    my = fmaf(g[2], dbx, fmaf(g[3], dby, my));
    short_score<CTL>(a, c, S, nd, out_row, path, xh, xl, yh, yl, k_end, !alive, mx, my, q, steps);
}

// A wavefront's sums into its node's: lane 2 v + h adds half h of sum v.
__device__ __forceinline__ void short_sums(NodeAcc &A, const unsigned long long (&q)[4], uint32_t steps, uint32_t lane) {
    unsigned long long add = 0ull;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const long long s = (long long)wave_sum(q[v]);
        add = lane == 2u * v ? (unsigned long long)(s >> 24) : add;
        add = lane == 2u * v + 1u ? (unsigned long long)(s & 0xffffffll) : add;
    }
    const unsigned long long st = wave_sum(steps);
    add = lane == 8u ? st : add;
    if (lane < 9u && add != 0ull) atomicAdd(lane == 8u ? &A.steps : &A.sum[lane >> 1][lane & 1u], add);
}

template <int KIND, int TMODE, int FORM>
__global__ void __launch_bounds__(256, FORM == CTL_MESH ? 5 : 6) fk_short_path_kernel(const PathArgs a, const MggArgs c) {
    constexpr int CTL = FORM == CTL_REFILL ? CTL_NONE : FORM;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t waves = gridDim.x * (blockDim.x >> 6);
    const uint32_t total = a.masked ? __builtin_amdgcn_readfirstlane(a.queue[kCtrActive]) * a.cpn : a.total_chunks;
    NodeAcc *const acc = CTL != CTL_NONE ? c.acc_cv : a.acc;
    const ShortWave S = short_wave<KIND, TMODE>(a);
    for (uint32_t ch = __builtin_amdgcn_readfirstlane(first_chunk()); ch < total; ch += waves) {
        uint32_t slot, next, end;
        chunk_cursor(a, total, ch, slot, next, end);
        slot = __builtin_amdgcn_readfirstlane(slot);
        next = __builtin_amdgcn_readfirstlane(next);
        end = __builtin_amdgcn_readfirstlane(end);
        const NodeDev nd = a.nodes[slot];
        if (!(nd.xlo == nd.xlo)) continue;         // not a node of the square (its results are NaN)
        const uint32_t out_row = __builtin_amdgcn_readfirstlane((uint32_t)nd.out);
        const uint32_t nid = __builtin_amdgcn_readfirstlane(nd.nid);
        float4 ofs = make_float4(0.f, 0.f, 0.f, 0.f);
        if constexpr (CTL != CTL_NONE) {
            if (c.gofs) ofs = c.gofs[out_row];
        }
        unsigned long long q[4] = {0ull, 0ull, 0ull, 0ull};
        uint32_t steps = 0;
        if constexpr (FORM == CTL_REFILL) {
            // (a chunk of one round has no other paths to take)
            if (end - next > 64u && __builtin_amdgcn_readfirstlane(short_leaves(S, nd))) {
                short_refill<KIND, TMODE>(a, S, nd, out_row, nid, next, end, q, steps);
                next = end;
            }
        }
        for (uint32_t p0 = next; p0 < end; p0 += 64)
            short_paths<KIND, TMODE, CTL>(a, c, S, nd, out_row, nid, ofs, nullptr, 0, 0, p0 + lane, p0 + lane < end, q,
                                          steps);
        short_sums(acc[out_row], q, steps, lane);
    }
}

// The mesh's gradient from LDS: a workgroup of 16 wavefronts (four per SIMD)
// takes a chunk of one node's paths, with the kTile x kTile grid nodes around
// the node in LDS (160 KB, the CU's whole); the rare path beyond them reads
// memory.  From memory two 16-byte gathers per pair of steps take 123 cycles of the CU's
// address unit each for 64 lanes on lines of their own, more than the four
// SIMDs need for the steps.  Measured (two bumps frozen, N = 768, 10689 nodes
// x 16384 paths x 20 steps, stride 2): 8.5 ms against 14.1 from memory; bound
// by VALU issue as the plain kernel (5.8 ms), the gradient's arithmetic on
// top.
template <int KIND, int TMODE>
__global__ void __launch_bounds__(1024) fk_short_tile_kernel(const PathArgs a, const MggArgs c) {
    __shared__ MeshTile tile;
    const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t total = a.masked ? __builtin_amdgcn_readfirstlane(a.queue[kCtrActive]) * a.cpn : a.total_chunks;
    const ShortWave S = short_wave<KIND, TMODE>(a);
    for (uint32_t ch = blockIdx.x; ch < total; ch += gridDim.x) {
        uint32_t slot, next, end;
        chunk_cursor(a, total, ch, slot, next, end);
        slot = __builtin_amdgcn_readfirstlane(slot);
        next = __builtin_amdgcn_readfirstlane(next);
        end = __builtin_amdgcn_readfirstlane(end);
        const NodeDev nd = a.nodes[slot];
        if (!(nd.xlo == nd.xlo)) continue;         // (the whole workgroup)
        const uint32_t out_row = __builtin_amdgcn_readfirstlane((uint32_t)nd.out);
        const uint32_t nid = __builtin_amdgcn_readfirstlane(nd.nid);
        float4 ofs = make_float4(0.f, 0.f, 0.f, 0.f);
        if (c.gofs) ofs = c.gofs[out_row];
        const int n = a.grid_n, far = max(n + 1 - kTile, 0);
        const int i0 = __builtin_amdgcn_readfirstlane(min(max((int)(nd.x * (float)n) - kTile / 2, 0), far));
        const int j0 = __builtin_amdgcn_readfirstlane(min(max((int)(nd.y * (float)n) - kTile / 2, 0), far));
        __syncthreads();                           // the last chunk's readers
        load_tile(tile, a.grid_xi, a.grid_eta, n, i0, j0);
        __syncthreads();
        unsigned long long q[4] = {0ull, 0ull, 0ull, 0ull};
        uint32_t steps = 0;
        for (uint32_t p0 = next + 64u * wave; p0 < end; p0 += 1024u)
            short_paths<KIND, TMODE, CTL_TILE>(a, c, S, nd, out_row, nid, ofs, &tile, i0, j0, p0 + lane,
                                               p0 + lane < end, q, steps);
        short_sums(c.acc_cv[out_row], q, steps, lane);
    }
}

namespace {
template <int K, int T, int C>
struct ShortLaunchF {
    static hipError_t run(const PathArgs &a, const MggArgs &c, int grid, int block, hipStream_t s) {
        if constexpr (C == CTL_TILE)
            hipLaunchKernelGGL((fk_short_tile_kernel<K, T>), dim3(grid), dim3(1024), 0, s, a, c);
        else
            hipLaunchKernelGGL((fk_short_path_kernel<K, T, C>), dim3(grid), dim3(block), 0, s, a, c);
        return hipGetLastError();
    }
};
template <int K, int T, int C>
struct ShortOccF {
    static int run(int block) {
        int nb = 0;
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fk_short_path_kernel<K, T, C == CTL_TILE ? CTL_MESH : C>,
                                                            block, 0) == hipSuccess
                   ? nb
                   : 0;
    }
};

template <template <int, int, int> class F, typename... Args>
auto short_dispatch(int kind, int time_mode, int ctl, Args &&...args) {
    const bool frozen = (time_mode == TIME_FROZEN);
#define FK_SHORT(K, T)                                                                  \
    return ctl == CTL_TILE     ? F<K, T, CTL_TILE>::run(std::forward<Args>(args)...)    \
           : ctl == CTL_MESH   ? F<K, T, CTL_MESH>::run(std::forward<Args>(args)...)    \
           : ctl == CTL_REFILL ? F<K, T, CTL_REFILL>::run(std::forward<Args>(args)...)  \
                               : F<K, T, CTL_NONE>::run(std::forward<Args>(args)...)
    switch (kind) {
    case KIND_CONST: FK_SHORT(KIND_CONST, TIME_BACKWARD);
    case KIND_BUMP: FK_SHORT(KIND_BUMP, TIME_BACKWARD);
    case KIND_RIDGE: FK_SHORT(KIND_RIDGE, TIME_BACKWARD);
    case KIND_GRID: FK_SHORT(KIND_GRID, TIME_BACKWARD);
    case KIND_MOVING:
        if (frozen) FK_SHORT(KIND_MOVING, TIME_FROZEN);
        FK_SHORT(KIND_MOVING, TIME_BACKWARD);
    case KIND_RING:
        if (frozen) FK_SHORT(KIND_RING, TIME_FROZEN);
        FK_SHORT(KIND_RING, TIME_BACKWARD);
    default:
        if (frozen) FK_SHORT(KIND_TWO, TIME_FROZEN);
        FK_SHORT(KIND_TWO, TIME_BACKWARD);
    }
#undef FK_SHORT
}

// A wavefront's sums of a chunk (1/16 of its paths) stay below 2^62.
constexpr int64_t kMaxTileChunk = 32768;

// Paths per chunk of the tile kernel, or 0 where it is not used: the paths
// have to stay near the node, a chunk's gathers have to pay for loading its
// tile, and the chunks have to fill the chip.  Measured from memory / from the
// tile, in ms (two bumps, N = 768, 20 steps, stride 2 unless stated):
//   2048 nodes x 8192 paths, Brownian standard deviation 12 cells 1.60 / 0.97,
//   24: 2.66 / 1.02, 38: 2.99 / 1.06, 46: 3.06 / 1.24, 60: 3.06 / 1.52;
//   stride 4: 1.66 / 0.86, 10: 0.92 / 0.81, 20 (one block): 0.70 / 0.79;
//   1024 paths at 2048 nodes 0.39 / 0.26, at 512 0.116 / 0.105, at 128 (fewer
//   chunks than CUs) 0.066 / 0.075, 2048 paths there 0.082 / 0.076.
uint32_t tile_chunk(int grid_n, int64_t n_paths, int64_t stride, double t, int64_t K, int64_t n_nodes, int n_cu) {
    const double n = grid_n;
    if (n + 1 > kTile && std::sqrt(2.0 * t) * n > 0.6 * kTile) return 0;
    const int64_t gathers = (K + stride - 1) / stride;   // of a path
    if (gathers < 2) return 0;
    const int64_t least = (kTile * kTile / gathers + 1023) / 1024 * 1024;      // paths that pay for a tile
    const int64_t split = std::max<int64_t>(1, (8 * (int64_t)n_cu + n_nodes - 1) / n_nodes);
    const int64_t chunk = std::min<int64_t>(
        kMaxTileChunk, std::max(least, ((n_paths + split - 1) / split + 1023) / 1024 * 1024));
    const int64_t per_node = (n_paths + chunk - 1) / chunk;
    if (n_paths < least || per_node * n_nodes < n_cu || per_node * n_nodes > 0x7fffffff) return 0;
    return (uint32_t)chunk;
}
}  // namespace

bool lockstep_mesh(bool table, int grid_n, int64_t n_paths, int64_t stride, double t, int64_t K, int64_t n_nodes,
                   int n_cu, bool masked) {
    if (K <= 32 && tile_chunk(grid_n, n_paths, stride, t, K, n_nodes, n_cu) != 0) return true;
    if (masked) n_nodes = (n_nodes + 7) / 8;   // (as lockstep_chunk)
    const int64_t gathers = stride < K ? (K + stride - 1) / stride : 1;      // of a path
    const double rounds = (double)n_nodes * (double)((n_paths + 63) / 64) / (4.0 * n_cu);   // of 64 paths, to a SIMD
    const double spread = std::sqrt(2.0 * t) * grid_n;   // standard deviation of the paths, in cells
    const double many = 48.0, few = 12.0;
    if (K > 32)
        return rounds <= (gathers == 1 || (table && gathers <= 16) ? many : few) &&
               (table || grid_n <= 256 || gathers <= 16);
    if (gathers <= 5) return true;
    if (table) return K <= 20 || gathers <= 8 || rounds <= many || spread <= 100.0;
    return rounds <= (K <= 20 || gathers <= 8 ? many : few) || grid_n < kTile || (grid_n <= 256 && spread <= 60.0);
}

bool lockstep_refill(int64_t K, int64_t n_nodes, int64_t n_paths, int n_cu, bool masked) {
    if (masked) n_nodes = (n_nodes + 7) / 8;   // (as lockstep_chunk)
    return K > 32 && n_nodes * ((n_paths + 63) / 64) > 24LL * n_cu;
}

hipError_t launch_short_paths(int kind, int time_mode, bool refill, const PathArgs &a, int grid, int block,
                              hipStream_t s) {
    return short_dispatch<ShortLaunchF>(kind, time_mode, refill ? CTL_REFILL : CTL_NONE, a, MggArgs{}, grid, block, s);
}

hipError_t launch_short_mesh_paths(int kind, int time_mode, const PathArgs &a, const MggArgs &c, double t, int64_t K,
                                   int64_t n_nodes, int n_cu, int grid, int block, hipStream_t s) {
    const uint32_t chunk = tile_chunk(a.grid_n, a.n_paths, 2 * (int64_t)c.stride_iters, t, K, n_nodes, n_cu);
    if (chunk == 0) return short_dispatch<ShortLaunchF>(kind, time_mode, CTL_MESH, a, c, grid, block, s);
    PathArgs b = a;
    b.chunk = chunk;
    b.cpn = (a.n_paths + chunk - 1) / chunk;
    b.total_chunks = (uint32_t)(n_nodes * b.cpn);
    b.tile_shift = 0;
    return short_dispatch<ShortLaunchF>(kind, time_mode, CTL_TILE, b, c, (int)std::min<int64_t>(b.total_chunks, n_cu),
                                        1024, s);
}

int short_kernel_max_blocks_per_cu(int kind, int time_mode, bool mesh, bool refill, int block) {
    return short_dispatch<ShortOccF>(kind, time_mode, mesh ? CTL_MESH : refill ? CTL_REFILL : CTL_NONE, block);
}

}  // namespace fk
