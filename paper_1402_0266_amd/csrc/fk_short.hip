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
// Measured (two bumps frozen, 10689 nodes x 16384 paths x 20 steps): 6.1 ms
// against the refilling kernel's 9.7 ms, 70 VALU instructions per step of a
// wavefront at one per 3.8 cycles and SIMD (the rates above give 3.6 for this
// mix); the ring's 77 nodes x 10^4 paths: 37 us for the whole solve against
// 106 us.
#include <hip/hip_runtime.h>
#include <stdint.h>

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

// MESH: the martingale form with the mesh's gradient as control (as
// fk_mgg_path_kernel, fk_cv.hip), else the plain estimate.
template <int KIND, int TMODE, bool MESH>
__global__ void __launch_bounds__(256, MESH ? 5 : 6) fk_short_path_kernel(const PathArgs a, const MggArgs c) {
    constexpr bool kMovingBackward = moving_kind(KIND) && TMODE == TIME_BACKWARD;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t waves = gridDim.x * (blockDim.x >> 6);
    const uint32_t total = a.masked ? __builtin_amdgcn_readfirstlane(a.queue[kCtrActive]) * a.cpn : a.total_chunks;
    const uint32_t key0 = a.key0, key1 = a.key1;
    NodeAcc *const acc = MESH ? c.acc_cv : a.acc;
    NodeAcc *const accs[1] = {acc};

    const LevelDev &lv = a.levels[0];
    Lane L;
    lane_level<KIND, TMODE>(L, lv);
    const int32_t K = lv.K;
    const uint32_t ctr3 = lv.ctr3;
    const float dt = in_vgpr(L.dt), cbm = in_vgpr(L.cbm);
    const float dt_last = in_vgpr(L.dt_last), cbm_last = in_vgpr(L.cbm_last);
    const uint32_t fmask = in_vgpr(kUnitMask);
    const float rev0 = in_vgpr(L.rev0), drev = in_vgpr(L.drev), cos_d = in_vgpr(L.cos_d), sin_d = in_vgpr(L.sin_d);
    L.dens.amp = in_vgpr(L.dens.amp);
    L.dens.nscale = in_vgpr(L.dens.nscale);
    L.dens.a2s = in_vgpr(L.dens.a2s);
    L.dens.cx = in_vgpr(L.dens.cx);
    L.dens.cy = in_vgpr(L.dens.cy);
    L.dens.orbit_r = in_vgpr(L.dens.orbit_r);
    if constexpr (KIND == KIND_GRID) L.dens.fn = in_vgpr(L.dens.fn);
    const PhiloxWave W = philox_wave(key0, key1);

    for (uint32_t ch = __builtin_amdgcn_readfirstlane(first_chunk()); ch < total; ch += waves) {
        uint32_t slot, next, end;
        chunk_cursor(a, total, ch, slot, next, end);
        slot = __builtin_amdgcn_readfirstlane(slot);
        next = __builtin_amdgcn_readfirstlane(next);
        end = __builtin_amdgcn_readfirstlane(end);
        const NodeDev nd = a.nodes[slot];
        if (!(nd.xlo == nd.xlo)) continue;         // not a node of the square (its results are NaN)
        const uint32_t out_row = __builtin_amdgcn_readfirstlane((uint32_t)nd.out);
        const uint32_t nid = __builtin_amdgcn_readfirstlane(nd.nid), nlo = kM1 * nid;
        const uint64_t rec0 = (uint64_t)out_row * a.n_paths;
        float4 ofs = make_float4(0.f, 0.f, 0.f, 0.f);
        if constexpr (MESH) {
            if (c.gofs) ofs = c.gofs[out_row];
        }
        unsigned long long q[4] = {0ull, 0ull, 0ull, 0ull};
        uint32_t steps = 0;
        for (uint32_t p0 = next; p0 < end; p0 += 64) {
            const uint32_t path = p0 + lane;
            const bool has = path < end;
            const PhiloxPath pp = philox_path(path, nid, key0);
            float xh = nd.x, xl = nd.xlo, yh = nd.y, yl = nd.ylo;
            float D = dt, cb = cbm;
            float gxx = 0.f, gxy = 0.f, gyx = 0.f, gyy = 0.f, dbx = 0.f, dby = 0.f, mx = 0.f, my = 0.f;
            uint32_t blk_left = 0;   // iterations (2 steps each) to the next block boundary
            bool alive = has;
            int32_t k_end = K;       // steps the lane's path takes
            // The loop is the wavefront's (k is a scalar): it ends at K, or
            // with the last path that is still inside.
            for (int32_t k = 0; k < K && ballot(alive) != 0ull; k += 2) {
                const PhiloxOut r = philox4x32_10_wave((uint32_t)k >> 1, ctr3, nlo, pp, W, key0, key1);
                if constexpr (MESH) {
                    if (blk_left == 0) {
                        blk_left = c.stride_iters;
                        if (alive) {
                            mx = fmaf(gxx, dbx, fmaf(gxy, dby, mx));
                            my = fmaf(gyx, dbx, fmaf(gyy, dby, my));
                            dbx = dby = 0.f;
                            if (c.gtab) {
                                table_gradient(c.gtab, a.grid_n, 0, xh, yh, gxx, gxy);
                                table_gradient(c.gtab, a.grid_n, 1, xh, yh, gyx, gyy);
                            } else {
                                grid_gradient(a.grid_xi, a.grid_n, xh, yh, gxx, gxy);
                                grid_gradient(a.grid_eta, a.grid_n, xh, yh, gyx, gyy);
                            }
                            if (c.gofs) {
                                gxx += ofs.x;
                                gxy += ofs.y;
                                gyx += ofs.z;
                                gyy += ofs.w;
                            }
                        }
                    }
                    --blk_left;
                }
                float ox = L.ox, oy = L.oy, cr = 0.f, sr = 0.f;
                if constexpr (kMovingBackward) {
                    const float rev = fmaf(-(float)k, drev, rev0);
                    cr = hw_cos_rev(rev);
                    sr = hw_sin_rev(rev);
                    ox = L.dens.orbit_r * cr;
                    oy = L.dens.orbit_r * sr;
                }
                if (k == K - 1) {
                    D = last_step(dt_last);
                    cb = last_step(cbm_last);
                }
                float wx, wy;
                if (alive) {
                    const bool out = em_update<KIND>(xh, xl, yh, yl, L.dens, r.r0, r.r1, ox, oy, D, cb, fmask, wx, wy) < 0;
                    if constexpr (MESH) {
                        dbx += wx;
                        dby += wy;
                    }
                    if (out) {
                        alive = false;
                        k_end = step_number(k + 1);
                    }
                }
                if (k + 1 >= K) break;
                if constexpr (kMovingBackward) {
                    const float c2 = fmaf(cr, cos_d, sr * sin_d);
                    const float s2 = fmaf(sr, cos_d, -cr * sin_d);
                    ox = L.dens.orbit_r * c2;
                    oy = L.dens.orbit_r * s2;
                }
                if (k + 1 == K - 1) {
                    D = last_step(dt_last);
                    cb = last_step(cbm_last);
                }
                if (alive) {
                    const bool out = em_update<KIND>(xh, xl, yh, yl, L.dens, r.r2, r.r3, ox, oy, D, cb, fmask, wx, wy) < 0;
                    if constexpr (MESH) {
                        dbx += wx;
                        dby += wy;
                    }
                    if (out) {
                        alive = false;
                        k_end = step_number(k + 2);
                    }
                }
            }
            if (has) {
                const bool out = !alive;
                // ---- score (eq. (7b)) ---------------------------------------
                Lane E = L;
                E.xh = xh;
                E.xl = xl;
                E.yh = yh;
                E.yl = yl;
                E.px = nd.x;
                E.py = nd.y;
                E.k = k_end;
                E.K = K;
                float v[2];
                score_path(a, E, out, v[0], v[1]);
                if constexpr (MESH) {
                    mx = fmaf(gxx, dbx, fmaf(gxy, dby, mx));
                    my = fmaf(gyx, dbx, fmaf(gyy, dby, my));
                    const float sx0 = a.shift ? nd.x : 0.f, sy0 = a.shift ? nd.y : 0.f;
                    v[0] = (v[0] + sx0) - mx;
                    v[1] = (v[1] + sy0) - my;
                    if (c.cv_scores) c.cv_scores[rec0 + path] = make_float2(v[0], v[1]);
                } else {
                    if (a.scores) a.scores[rec0 + path] = make_float2(v[0], v[1]);
                }
                if (a.exit_step) a.exit_step[rec0 + path] = out ? k_end : -1;
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
        }
        // ---- the chunk's sums into its node's: lane 2 v + h adds half h of sum v ----
        unsigned long long add = 0ull;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const long long s = (long long)wave_sum(q[v]);
            add = lane == 2u * v ? (unsigned long long)(s >> 24) : add;
            add = lane == 2u * v + 1u ? (unsigned long long)(s & 0xffffffll) : add;
        }
        const unsigned long long st = wave_sum(steps);
        add = lane == 8u ? st : add;
        if (lane < 9u && add != 0ull) {
            NodeAcc &A = acc[out_row];
            unsigned long long *at = lane == 8u ? &A.steps : &A.sum[lane >> 1][lane & 1u];
            atomicAdd(at, add);
        }
    }
}

namespace {
template <int K, int T, bool M>
struct ShortLaunchF {
    static hipError_t run(const PathArgs &a, const MggArgs &c, int grid, int block, hipStream_t s) {
        hipLaunchKernelGGL((fk_short_path_kernel<K, T, M>), dim3(grid), dim3(block), 0, s, a, c);
        return hipGetLastError();
    }
};
template <int K, int T, bool M>
struct ShortOccF {
    static int run(int block) {
        int nb = 0;
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fk_short_path_kernel<K, T, M>, block, 0) == hipSuccess
                   ? nb
                   : 0;
    }
};

template <template <int, int, bool> class F, typename... Args>
auto short_dispatch(int kind, int time_mode, bool mesh, Args &&...args) {
    const bool frozen = (time_mode == TIME_FROZEN);
#define FK_SHORT(K, T) \
    return mesh ? F<K, T, true>::run(std::forward<Args>(args)...) : F<K, T, false>::run(std::forward<Args>(args)...)
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
}  // namespace

hipError_t launch_short_paths(int kind, int time_mode, const PathArgs &a, const MggArgs *mesh, int grid, int block,
                              hipStream_t s) {
    return short_dispatch<ShortLaunchF>(kind, time_mode, mesh != nullptr, a, mesh ? *mesh : MggArgs{}, grid, block, s);
}

int short_kernel_max_blocks_per_cu(int kind, int time_mode, bool mesh, int block) {
    return short_dispatch<ShortOccF>(kind, time_mode, mesh, block);
}

}  // namespace fk
