// fk_dissect.hpp -- nested dissection of the sub-domain systems
// (fk_dissect.hip): the tree's sizes, and the launch.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fk {

constexpr int kNdMaxLevels = 20;
constexpr int kNdMaxFront = 192;   // 32 x 32 lanes of 6 x 6 register tiles

// One level of the tree: the boxes of depth l.
struct NdLevel {
    int s, b;            // most pivots (even) and boundary unknowns of a box (not always the same box)
    int f;               // most of both together: the largest front
    int ldw, lds;        // row strides of the kept rows and of the Schur complements
    int64_t w_off;       // kept rows (W, y) of the level, in doubles
};

struct NdTree {
    int depth;           // leaves are the boxes of this depth
    int qx, qy;          // unknowns a side of a sub-domain
    NdLevel lv[kNdMaxLevels];
    int64_t s_off;       // Schur complements: those of a box lie in the place of its leaves',
    int64_t s_leaf;      // this many doubles for each leaf of the full tree
    int64_t doubles;     // buffer for all sub-domains
};

struct NdArgs {
    const double2 *cf;   // [blocks][qy][qx] (cx, cy): east -c - cx, west -c + cx, north -c - cy, south -c + cy
    const double2 *rh;   // right-hand sides (xi, eta)
    double *buf;
    double *xi_out, *eta_out;
    double c, diag;
    int N, px, mx, my;   // grid cells a side; sub-domains in a row; cells of a sub-domain
};

// Lanes a side of a front's workgroup.  Many small fronts: a wavefront each
// (the work per lane outweighs the pivots' fixed cost); else 256 lanes, which
// take a pair of pivots sooner than 1024 do (every wavefront repeats the
// pivots' reciprocals; 95 pivots: 40 us against 43, 47 in a front of 142: 47
// against 49) as long as the tile fits their registers.
inline int nd_lanes(int64_t fronts, int f) { return fronts > 256 && f <= 64 ? 8 : f <= 144 ? 16 : 32; }

// The tree of a qx x qy grid of unknowns in each of `blocks` sub-domains;
// false where a front would be larger than kNdMaxFront, a launch would have
// 2^32 work-items, or a side has 32768 unknowns.
bool nd_tree(int qx, int qy, int64_t blocks, NdTree *t);
// Factorises and solves every sub-domain (Dirichlet data in the output grids,
// cf and rh assembled): interior values of xi_out, eta_out.
hipError_t nd_solve(const NdTree &t, const NdArgs &a, int blocks, hipStream_t s);

}  // namespace fk
