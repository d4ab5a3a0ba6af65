// fk_dissect.hip -- the sub-domain systems of Sect. 4 by nested dissection
// (George 1973) in its multifrontal form.
//
// A sub-domain's grid of unknowns is a box.  A box is split by a grid line
// across its longer side, both halves likewise, down to leaves of a few
// (nd_leaf) unknowns.  With 5-point rows, a box's unknowns couple to the rest of
// the grid only through the unknowns on the lines around it (no corners), so
// going up the tree each box eliminates its separator (a leaf: all it has)
// from a dense front over
//
//     [separator | lines around the box],
//
// which is the sum of its children's Schur complements and of the matrix
// entries of the separator's rows and columns, and hands the Schur complement
// over the lines around it to its parent.  The elimination is Gauss-Jordan
// without pivoting (the Schur complements of a diagonally dominant matrix are
// diagonally dominant), so what a box keeps is x_sep = y - W x_around: going
// down the tree is one matrix-vector product per box, no triangular solves.
//
// Why: a banded elimination of a q x q grid is a chain of q^2 dependent
// pivots (half as many from both ends) and q^4 multiply-adds.  The tree's
// chain is its separators one after the other, about 3 q pivots, with many
// boxes at work at every level, and about 10 q^3 multiply-adds.
//
// A front is held in registers by a grid of LN x LN lanes (8, 16 or 32),
// lane (rg, cg) with the entries of rows rg + LN t and columns cg + LN u.  Two
// pivots are taken per barrier: their rows and columns go through LDS (one
// 16-byte read per register row and column), and every lane applies both to
// its tile.
//
// Measured, 8 x 8 sub-domains of 95 x 95 unknowns: 0.66 ms against 3.98 ms for
// the banded LU from both ends (4512 dependent pivots, 128 workgroups).  The
// fronts of the ten levels take 66, 52, 45, 50 us (one wavefront each, bound
// by instructions -- about 1000 a front -- and by 1.1 GB of Schur complements
// and kept rows), 50, 70, 73, 51, 47 and 40 us (bound by the chain of pivots,
// 0.8 us a pair); the way down 18 and 86 us.  2 x 2 sub-domains of 19 x 19
// with their edge data: 56 us against 192 us.
#include "fk_dissect.hpp"

#include <algorithm>

namespace fk {

// Most unknowns of a leaf: few with many sub-domains (the work counts: 12
// against 30 took 240 us off the lowest levels of 64 x 95 x 95), more with few
// (the levels count: 20 against 12 took one of six off 4 x 19 x 19).
constexpr int nd_leaf(int64_t blocks) { return blocks >= 32 ? 12 : 20; }

// Box [x0, x1) x [y0, y1) of a sub-domain's unknowns (empty if a side is not
// positive).
struct NdBox {
    int x0, x1, y0, y1;
};

// The separating line of a box: column or row `at`.
__host__ __device__ inline bool nd_split(const NdBox &b, int &at) {
    const int w = b.x1 - b.x0, h = b.y1 - b.y0;
    const bool vertical = w >= h;
    at = vertical ? b.x0 + w / 2 : b.y0 + h / 2;
    return vertical;
}

__host__ __device__ inline NdBox nd_child(const NdBox &b, bool vertical, int at, int which) {
    NdBox c = b;
    if (vertical) {
        if (which) c.x0 = at + 1;
        else c.x1 = at;
    } else {
        if (which) c.y0 = at + 1;
        else c.y1 = at;
    }
    return c;
}

__host__ __device__ inline bool nd_empty(const NdBox &b) { return b.x1 <= b.x0 || b.y1 <= b.y0; }

// Box number idx of depth l: its path from the root is idx's bits, high first.
__device__ __forceinline__ NdBox nd_box(int qx, int qy, int l, int idx) {
    NdBox b{0, qx, 0, qy};
    for (int d = l - 1; d >= 0; --d) {
        int at;
        const bool v = nd_split(b, at);
        b = nd_child(b, v, at, (idx >> d) & 1);
    }
    return b;
}

// The lines around a box, in the order left, right, below, above: where each
// starts in the list of boundary unknowns, and their number in all.
struct NdRim {
    int r, d, u, n;   // starts of right, below, above (left starts at 0); total
};
__host__ __device__ inline NdRim nd_rim(const NdBox &b, int qx, int qy) {
    const int w = b.x1 - b.x0, h = b.y1 - b.y0;
    NdRim m;
    m.r = b.x0 > 0 ? h : 0;
    m.d = m.r + (b.x1 < qx ? h : 0);
    m.u = m.d + (b.y0 > 0 ? w : 0);
    m.n = m.u + (b.y1 < qy ? w : 0);
    return m;
}
// Unknown j of the rim, as x | y << 16.
__device__ __forceinline__ int nd_rim_node(const NdBox &b, const NdRim &m, int j) {
    if (j < m.r) return (b.x0 - 1) | ((b.y0 + j) << 16);
    if (j < m.d) return b.x1 | ((b.y0 + j - m.r) << 16);
    if (j < m.u) return (b.x0 + j - m.d) | ((b.y0 - 1) << 16);
    return (b.x0 + j - m.u) | (b.y1 << 16);
}
// The place of unknown (x, y) in a box's rim, or -1.
__device__ __forceinline__ int nd_rim_place(const NdBox &b, const NdRim &m, int x, int y) {
    const bool iny = y >= b.y0 && y < b.y1, inx = x >= b.x0 && x < b.x1;
    if (iny && x == b.x0 - 1) return y - b.y0;
    if (iny && x == b.x1) return m.r + y - b.y0;
    if (inx && y == b.y0 - 1) return m.d + x - b.x0;
    if (inx && y == b.y1) return m.u + x - b.x0;
    return -1;
}

// Pivots of a box: its separator, or all of a leaf.
__host__ __device__ inline int nd_pivots(const NdBox &b, bool leaf) {
    if (nd_empty(b)) return 0;
    const int w = b.x1 - b.x0, h = b.y1 - b.y0;
    return leaf ? w * h : (w >= h ? h : w);
}
__device__ __forceinline__ int nd_pivot_node(const NdBox &b, bool leaf, bool vertical, int at, int i) {
    if (leaf) {
        const int w = b.x1 - b.x0;
        return (b.x0 + i % w) | ((b.y0 + i / w) << 16);
    }
    return vertical ? (at | ((b.y0 + i) << 16)) : ((b.x0 + i) | (at << 16));
}

constexpr int kNoNode = -1;

// Wavefronts per SIMD a front kernel is compiled for: its tile takes 2 T^2
// registers, the pivot rows and columns 8 T.
constexpr int nd_waves(int lanes, int T) {
    if (lanes == 32) return 4;
    const int regs = 2 * T * T + 8 * T + 40;
    return regs <= 64 ? 8 : regs <= 100 ? 5 : regs <= 128 ? 4 : regs <= 168 ? 3 : regs <= 256 ? 2 : 1;
}

// 1 / x by the hardware reciprocal and two Newton steps (an ulp or two).
__device__ __forceinline__ double nd_rcp(double x) {
    double y = __builtin_amdgcn_rcp(x);
    double e = fma(-x, y, 1.0);
    y = fma(y, e, y);
    e = fma(-x, y, 1.0);
    return fma(y, e, y);
}

// Grid index of unknown (x, y) of sub-domain sd.
__device__ __forceinline__ int64_t nd_grid(const NdArgs &a, int sd, int node) {
    const int gi = (sd % a.px) * a.mx + 1 + (node & 0xffff), gj = (sd / a.px) * a.my + 1 + (node >> 16);
    return (int64_t)gj * (a.N + 1) + gi;
}

// The Schur complement of box idx of level l (unused beyond the leaves).
__device__ __forceinline__ double *nd_schur(const NdArgs &a, const NdTree &t, int l, int sd, int idx) {
    if (l > t.depth) return nullptr;
    return a.buf + t.s_off + (((int64_t)sd << t.depth) + ((int64_t)idx << (t.depth - l))) * t.s_leaf;
}

// A double at a byte offset from a wave-uniform base.
__device__ __forceinline__ double nd_at(const double *base, uint32_t off) {
    return *reinterpret_cast<const double *>(reinterpret_cast<const char *>(base) + off);
}

// One front per workgroup: box blockIdx.x of level l, on LN x LN lanes.
template <int LN, int T>
__global__ void __launch_bounds__(LN * LN) __attribute__((amdgpu_waves_per_eu(1, nd_waves(LN, T))))
nd_front_kernel(const NdArgs a, const NdTree t, const int l) {
    constexpr int W = LN * T;
    __shared__ int pos[W];                    // the front's unknowns, x | y << 16 (kNoNode: padding)
    __shared__ int cmap[2][W];                // their places in the children's rims, or -1
    __shared__ double2 colb[2][W];            // [buffer][row]: the two pivot columns
    __shared__ double2 rowb[2][W + 2];        // [buffer][column]: the two pivot rows, then the right-hand sides
    const int per = 1 << l, sd = blockIdx.x >> l, idx = blockIdx.x & (per - 1);
    const bool leaf = l == t.depth;
    const NdBox box = nd_box(t.qx, t.qy, l, idx);
    if (nd_empty(box)) return;
    const NdLevel lv = t.lv[l];
    int at;
    const bool vertical = nd_split(box, at);
    const int s = nd_pivots(box, leaf), s2 = (s + 1) & ~1;   // an odd count gets an identity row
    const NdRim rim = nd_rim(box, t.qx, t.qy);
    const int f = s2 + rim.n;
    const NdBox c0 = nd_child(box, vertical, at, 0), c1 = nd_child(box, vertical, at, 1);
    const NdRim m0 = nd_rim(c0, t.qx, t.qy), m1 = nd_rim(c1, t.qx, t.qy);
    const int tid = threadIdx.x, rg = tid / LN, cg = tid % LN;
    if (tid < W) {
        int p = kNoNode;
        if (tid < s) p = nd_pivot_node(box, leaf, vertical, at, tid);
        else if (tid >= s2 && tid < f) p = nd_rim_node(box, rim, tid - s2);
        pos[tid] = p;
        const int x = p & 0xffff, y = p >> 16;
        const bool has = !leaf && p != kNoNode;
        cmap[0][tid] = has && !nd_empty(c0) ? nd_rim_place(c0, m0, x, y) : -1;
        cmap[1][tid] = has && !nd_empty(c1) ? nd_rim_place(c1, m1, x, y) : -1;
    }
    __syncthreads();
    // ---- assembly ----------------------------------------------------------
    const int64_t n = (int64_t)t.qx * t.qy;
    const double2 *cf = a.cf + sd * n;
    const double2 *rh = a.rh + sd * n;
    const bool rhs = cg < 2;
    double A[T][T], B[T];
    int pj[T];
#pragma unroll
    for (int u = 0; u < T; ++u) pj[u] = pos[cg + LN * u];
    // the matrix entries of the pivots' rows and columns
#pragma unroll
    for (int r = 0; r < T; ++r) {
        const int i = rg + LN * r, p = pos[i];
        const bool real = p != kNoNode;
        const int node = real ? (p >> 16) * t.qx + (p & 0xffff) : 0;
        const double2 cr = cf[node], fr = rh[node];
#pragma unroll
        for (int u = 0; u < T; ++u) {
            double v = 0.0;
            if (LN * r < s2 || LN * u < s2) {     // wave-uniform
                const int j = cg + LN * u, d = pj[u] - p;   // east 1, west -1, north 1 << 16, south -(1 << 16)
                const bool ew = d == 1 || d == -1, ns = d == (1 << 16) || d == -(1 << 16);
                const double k = ns ? cr.y : cr.x;
                const double e = -a.c - (d > 0 ? k : -k);
                v = (ew || ns) && real && pj[u] != kNoNode && (i < s2 || j < s2) ? e : 0.0;
            }
            if (r == u && rg == cg) v = i >= f || !real ? 1.0 : i < s2 ? a.diag : 0.0;
            A[r][u] = v;
        }
        B[r] = real && i < s2 ? (cg == 0 ? fr.x : fr.y) : 0.0;
    }
    // the children's Schur complements: every load is issued, whether or not
    // its value counts (the addresses stay inside the children's places)
    if (!leaf) {
        const uint32_t ld = (uint32_t)t.lv[l + 1].lds;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            if (nd_empty(c ? c1 : c0)) continue;
            const double *S = nd_schur(a, t, l + 1, sd, 2 * idx + c);
            int qc[T];
#pragma unroll
            for (int u = 0; u < T; ++u) qc[u] = cmap[c][cg + LN * u];
#pragma unroll
            for (int r = 0; r < T; ++r) {
                const int qr = cmap[c][rg + LN * r];
                const uint32_t row = 8u * ld * (uint32_t)max(qr, 0);
                double v[T];
#pragma unroll
                for (int u = 0; u < T; ++u) v[u] = nd_at(S, row + 8u * (uint32_t)max(qc[u], 0));
                const double vb = nd_at(S, row + 8u * (ld - 2u + (uint32_t)(cg & 1)));
#pragma unroll
                for (int u = 0; u < T; ++u) A[r][u] += (qr | qc[u]) >= 0 ? v[u] : 0.0;
                B[r] += qr >= 0 ? vb : 0.0;
            }
        }
    }
    // ---- Gauss-Jordan, two pivots k, k + 1 per barrier ----------------------
    int buf = 0;
#pragma unroll
    for (int t0 = 0; t0 < T; ++t0) {
        for (int g = 0; g < LN; g += 2) {
            const int k = LN * t0 + g;
            if (k >= s2) break;
            double *cb = reinterpret_cast<double *>(colb[buf]), *rb = reinterpret_cast<double *>(rowb[buf]);
            if (cg == g || cg == g + 1) {
#pragma unroll
                for (int r = 0; r < T; ++r) cb[2 * (LN * r + rg) + (cg - g)] = A[r][t0];
            }
            if (rg == g || rg == g + 1) {
#pragma unroll
                for (int u = t0; u < T; ++u) rb[2 * (LN * u + cg) + (rg - g)] = A[t0][u];
                if (rhs) rb[2 * (W + cg) + (rg - g)] = B[t0];
            }
            __syncthreads();
            const double2 d0 = colb[buf][k], d1 = colb[buf][k + 1];   // (a_kk, a_k,k+1), (a_k+1,k, a_k+1,k+1)
            const double inv0 = nd_rcp(d0.x), w01 = d0.y * inv0;
            const double inv1 = nd_rcp(fma(-d1.x, w01, d1.y));
            double r0[T], r1[T], l0[T], l1[T];
            // row k scaled; row k + 1 after step k, scaled
#pragma unroll
            for (int u = t0; u < T; ++u) {
                const double2 v = rowb[buf][LN * u + cg];
                r0[u] = v.x * inv0;
                r1[u] = fma(-d1.x, r0[u], v.y) * inv1;
            }
            double b0 = 0.0, b1 = 0.0;
            if (rhs) {
                const double2 v = rowb[buf][W + cg];
                b0 = v.x * inv0;
                b1 = fma(-d1.x, b0, v.y) * inv1;
            }
#pragma unroll
            for (int r = 0; r < T; ++r) {
                const double2 v = colb[buf][LN * r + rg];
                l0[r] = v.x;
                l1[r] = fma(-v.x, w01, v.y);
            }
            if (rg == g || rg == g + 1) {
                // the pivot rows themselves become the scaled rows; row k also
                // loses its entry in column k + 1
                const bool first = rg == g;
#pragma unroll
                for (int u = t0; u < T; ++u) A[t0][u] = first ? r0[u] : r1[u];
                B[t0] = first ? b0 : b1;
                l0[t0] = 0.0;
                l1[t0] = first ? w01 : 0.0;
            }
#pragma unroll
            for (int r = 0; r < T; ++r) {
#pragma unroll
                for (int u = t0; u < T; ++u) A[r][u] = fma(-l1[r], r1[u], fma(-l0[r], r0[u], A[r][u]));
                B[r] = fma(-l1[r], b1, fma(-l0[r], b0, B[r]));
            }
            buf ^= 1;
        }
    }
    // ---- results -------------------------------------------------------------
    if (l == 0) {
        // the root has no lines around it: its unknowns are solved
#pragma unroll
        for (int r = 0; r < T; ++r) {
            const int i = rg + LN * r;
            if (rhs && i < s) (cg == 0 ? a.xi_out : a.eta_out)[nd_grid(a, sd, pos[i])] = B[r];
        }
        return;
    }
    double *Wk = a.buf + lv.w_off + ((int64_t)sd * per + idx) * lv.s * lv.ldw;
    double *Sk = nd_schur(a, t, l, sd, idx);   // over the children's: they have been read
#pragma unroll
    for (int r = 0; r < T; ++r) {
        const int i = rg + LN * r;
        if (i >= f) continue;
        double *row = i < s2 ? Wk + (int64_t)i * lv.ldw : Sk + (int64_t)(i - s2) * lv.lds;
#pragma unroll
        for (int u = 0; u < T; ++u) {
            const int j = cg + LN * u - s2;
            if (j >= 0 && j < rim.n) row[j] = A[r][u];
        }
        if (rhs) row[(i < s2 ? lv.ldw : lv.lds) - 2 + cg] = B[r];
    }
}

template <int CTRL>
__device__ __forceinline__ double nd_dpp(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)b, CTRL, 0xf, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(b >> 32), CTRL, 0xf, 0xf, false);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
// Sum over each row of 16 lanes, in every lane of the row.
__device__ __forceinline__ double nd_sum16(double v) {
    v += nd_dpp<0xB1>(v);    // quad_perm [1, 0, 3, 2]
    v += nd_dpp<0x4E>(v);    // quad_perm [2, 3, 0, 1]
    v += nd_dpp<0x141>(v);   // row_half_mirror
    v += nd_dpp<0x140>(v);   // row_mirror
    return v;
}

// x_sep = y - W x_around for the boxes of levels l0 .. l1 below box
// blockIdx.x of level l0, level by level (one workgroup); the values around
// a box are read from the output grids, where the levels above wrote them.
// 16 lanes take a row, so a wavefront has four in hand: NC columns a lane.
template <int NC>
__device__ __forceinline__ void nd_down_box(const NdArgs &a, const NdTree &t, int l, int sd, int idx, int part, int parts) {
    const int lane = threadIdx.x & 63, li = lane & 15;
    const bool leaf = l == t.depth;
    const NdLevel &lv = t.lv[l];
    const NdBox box = nd_box(t.qx, t.qy, l, idx);
    if (nd_empty(box)) return;
    int at;
    const bool vertical = nd_split(box, at);
    const int s = nd_pivots(box, leaf);
    const NdRim rim = nd_rim(box, t.qx, t.qy);
    double x[NC], y[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int j = li + 16 * c;
        const int64_t g = nd_grid(a, sd, nd_rim_node(box, rim, j < rim.n ? j : 0));
        const bool in = j < rim.n;
        x[c] = in ? a.xi_out[g] : 0.0;
        y[c] = in ? a.eta_out[g] : 0.0;
    }
    const double *Wk = a.buf + lv.w_off + ((int64_t)sd * (1 << l) + idx) * lv.s * lv.ldw;
    for (int i0 = 4 * part; i0 < s; i0 += 4 * parts) {
        const int i = i0 + (lane >> 4), ic = min(i, s - 1);
        const double *row = Wk + (int64_t)ic * lv.ldw;
        double sx = 0.0, sy = 0.0, w[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) w[c] = row[min(li + 16 * c, lv.ldw - 1)];   // past the rim x is 0
        const double yv = row[lv.ldw - 2 + (li & 1)];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const double v = li + 16 * c < rim.n ? w[c] : 0.0;
            sx = fma(v, x[c], sx);
            sy = fma(v, y[c], sy);
        }
        sx = nd_sum16(sx);
        sy = nd_sum16(sy);
        if (i < s && li < 2) {
            const int64_t g = nd_grid(a, sd, nd_pivot_node(box, leaf, vertical, at, i));
            (li == 0 ? a.xi_out : a.eta_out)[g] = yv - (li == 0 ? sx : sy);
        }
    }
}

__global__ void __launch_bounds__(512) nd_down_kernel(const NdArgs a, const NdTree t, const int l0, const int l1) {
    const int sd = blockIdx.x >> l0, top = blockIdx.x & ((1 << l0) - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
    for (int l = l0; l <= l1; ++l) {
        const int nbox = 1 << (l - l0), b = t.lv[l].b;
        // several wavefronts share a box where there are more wavefronts than boxes
        const int share = nbox < waves ? waves / nbox : 1;
        for (int q = wave / share; q < nbox; q += waves / share) {
            const int idx = (top << (l - l0)) + q;
            if (b <= 16) nd_down_box<1>(a, t, l, sd, idx, wave % share, share);
            else if (b <= 32) nd_down_box<2>(a, t, l, sd, idx, wave % share, share);
            else if (b <= 64) nd_down_box<4>(a, t, l, sd, idx, wave % share, share);
            else if (b <= 96) nd_down_box<6>(a, t, l, sd, idx, wave % share, share);
            else nd_down_box<12>(a, t, l, sd, idx, wave % share, share);
        }
        __syncthreads();
    }
}

// Work-items of a launch: 2^32 and more are refused.
constexpr int64_t kMaxItems = ((int64_t)1 << 32) - 1;
// The way down: the levels from 1 to 3 (all of them, of at most five) by one
// workgroup of 512 for each box of level 1, those from kDownCut on by one for
// each box of that level.
constexpr int kDownCut = 4, kDownOne = 5;

bool nd_tree(int qx, int qy, int64_t blocks, NdTree *t) {
    // unknowns are packed as x | y << 16 in an int; nd_assemble_kernel
    // (fk_subdomain.hip) takes a work-item for each
    if (qx > 32767 || qy > 32767 || blocks > kMaxItems || (int64_t)qx * qy * blocks > kMaxItems - 255) return false;
    // the distinct boxes of a level: sizes and which sides have lines around them
    struct Kind {
        int w, h;
        bool side[4];   // left, right, below, above
    };
    Kind cur[64], nxt[64];
    int n = 1;
    cur[0] = Kind{qx, qy, {false, false, false, false}};
    t->qx = qx;
    t->qy = qy;
    int64_t w_off = 0, s_size[kNdMaxLevels];   // s_size: doubles of a box's Schur complement
    for (int l = 0;; ++l) {
        if (l >= kNdMaxLevels || l > 16) return false;
        int most = 0;
        for (int i = 0; i < n; ++i) most = std::max(most, cur[i].w * cur[i].h);
        const bool leaf = most <= nd_leaf(blocks);
        int s = 0, b = 0, f = 0;
        for (int i = 0; i < n; ++i) {
            const Kind &k = cur[i];
            const int p = leaf ? k.w * k.h : std::min(k.w, k.h), p2 = (p + 1) & ~1;
            const int r = (k.side[0] + k.side[1]) * k.h + (k.side[2] + k.side[3]) * k.w;
            if (p2 + r > kNdMaxFront) return false;
            s = std::max(s, p2);
            b = std::max(b, r);
            f = std::max(f, p2 + r);
        }
        NdLevel &lv = t->lv[l];
        lv.s = s;
        lv.b = b;
        lv.f = f;
        lv.ldw = b + 2;
        lv.lds = b + 2;
        const int64_t boxes = blocks << l;
        const int lanes = nd_lanes(boxes, f);
        if (boxes * lanes * lanes > kMaxItems) return false;
        lv.w_off = w_off;
        w_off += l > 0 ? boxes * s * lv.ldw : 0;
        s_size[l] = (int64_t)b * lv.lds;
        if (leaf) {
            t->depth = l;
            break;
        }
        int m = 0;
        for (int i = 0; i < n; ++i) {
            const bool v = cur[i].w >= cur[i].h;
            for (int c = 0; c < 2; ++c) {
                Kind k = cur[i];
                int &len = v ? k.w : k.h;
                len = c ? len - len / 2 - 1 : len / 2;
                k.side[v ? (c ? 0 : 1) : (c ? 2 : 3)] = true;
                if (len <= 0) continue;
                bool seen = false;
                for (int j = 0; j < m && !seen; ++j)
                    seen = nxt[j].w == k.w && nxt[j].h == k.h && std::equal(k.side, k.side + 4, nxt[j].side);
                if (seen) continue;
                if (m == 64) return false;
                nxt[m++] = k;
            }
        }
        n = m;
        std::copy(nxt, nxt + m, cur);
    }
    if (t->depth > 0 && (blocks << (t->depth <= kDownOne ? 1 : kDownCut)) * 512 > kMaxItems) return false;
    // a box's Schur complement takes the place of its children's
    t->s_off = w_off;
    t->s_leaf = 0;
    for (int l = 0; l <= t->depth; ++l) {
        const int64_t leaves = (int64_t)1 << (t->depth - l);
        t->s_leaf = std::max(t->s_leaf, (s_size[l] + leaves - 1) / leaves);
    }
    t->doubles = w_off + (blocks << t->depth) * t->s_leaf;
    return true;
}

static hipError_t nd_launch(int ln, int T, const NdTree &t, const NdArgs &a, unsigned fronts, int l, hipStream_t s) {
#define FK_ND(LN, n)                                                                                  \
    case 16 * LN + n:                                                                                 \
        hipLaunchKernelGGL((nd_front_kernel<LN, n>), dim3(fronts), dim3(LN * LN), 0, s, a, t, l);     \
        break;
    switch (16 * ln + T) {
        FK_ND(8, 1) FK_ND(8, 2) FK_ND(8, 3) FK_ND(8, 4) FK_ND(8, 5) FK_ND(8, 6) FK_ND(8, 7) FK_ND(8, 8)
        FK_ND(16, 1) FK_ND(16, 2) FK_ND(16, 3) FK_ND(16, 4) FK_ND(16, 5) FK_ND(16, 6) FK_ND(16, 7) FK_ND(16, 8) FK_ND(16, 9)
        FK_ND(32, 5) FK_ND(32, 6)   // (1024 lanes only past 144)
    default: return hipErrorInvalidValue;
    }
#undef FK_ND
    return hipGetLastError();
}

hipError_t nd_solve(const NdTree &t, const NdArgs &a, int blocks, hipStream_t s) {
    hipError_t e;
    for (int l = t.depth; l >= 0; --l) {
        const int f = t.lv[l].f;
        const int64_t fronts = (int64_t)blocks << l;
        const int ln = nd_lanes(fronts, f);
        if ((e = nd_launch(ln, (f + ln - 1) / ln, t, a, (unsigned)fronts, l, s)) != hipSuccess) return e;
    }
    if (t.depth > 0) {
        const int mid = t.depth <= kDownOne ? t.depth : kDownCut - 1;
        hipLaunchKernelGGL(nd_down_kernel, dim3((unsigned)blocks << 1), dim3(512), 0, s, a, t, 1, mid);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if (mid < t.depth) {
            hipLaunchKernelGGL(nd_down_kernel, dim3((unsigned)blocks << kDownCut), dim3(512), 0, s, a, t, kDownCut,
                               t.depth);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

}  // namespace fk
