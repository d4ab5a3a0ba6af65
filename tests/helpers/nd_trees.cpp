// Checks the nested-dissection trees the library accepts, box by box.
//
// Reads lines "qx qy blocks"; for each prints "qx qy blocks accepted ok depth
// front": ok is 1 if on every level each box's own front (even pivots + lines
// around it) is within what the level is launched for, the level's workgroup
// is one that is compiled, every launch has fewer than 2^32 threads, and the
// unknowns' packing x | y << 16 holds.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <set>
#include <tuple>

#include "fk_dissect.hpp"

using namespace fk;

// Width, height, and whether there is a line to the left, right, below, above.
typedef std::tuple<int, int, int, int, int, int> Box;

static bool compiled(int lanes, int tile) {
    return lanes == 8 ? tile >= 1 && tile <= 8 : lanes == 16 ? tile >= 1 && tile <= 9 : lanes == 32 && tile >= 5 && tile <= 6;
}

static bool check(const NdTree &t, int64_t qx, int64_t qy, int64_t blocks) {
    const int64_t limit = (int64_t)1 << 32;
    bool ok = qx < 32768 && qy < 32768 && blocks * qx * qy < limit - 256;
    ok = ok && (t.depth == 0 || (blocks << (t.depth <= 5 ? 1 : 4)) * 512 < limit);
    std::set<Box> boxes{Box{(int)qx, (int)qy, 0, 0, 0, 0}};
    for (int l = 0; l <= t.depth; ++l) {
        const NdLevel &lv = t.lv[l];
        const int64_t fronts = blocks << l;
        const int lanes = nd_lanes(fronts, lv.f);
        ok = ok && compiled(lanes, (lv.f + lanes - 1) / lanes) && fronts * lanes * lanes < limit;
        std::set<Box> next;
        for (const Box &k : boxes) {
            const auto [w, h, left, right, below, above] = k;
            const int pivots = l == t.depth ? w * h : std::min(w, h), even = (pivots + 1) & ~1;
            const int rim = (left + right) * h + (below + above) * w;
            ok = ok && even <= lv.s && rim <= lv.b && even + rim <= lv.f && lv.f <= kNdMaxFront;
            // across the longer side, at a tie the width
            if (w >= h) {
                if (w / 2 > 0) next.insert(Box{w / 2, h, left, 1, below, above});
                if (w - w / 2 - 1 > 0) next.insert(Box{w - w / 2 - 1, h, 1, right, below, above});
            } else {
                if (h / 2 > 0) next.insert(Box{w, h / 2, left, right, below, 1});
                if (h - h / 2 - 1 > 0) next.insert(Box{w, h - h / 2 - 1, left, right, 1, above});
            }
        }
        boxes = next;
    }
    return ok;
}

int main() {
    long long qx, qy, blocks;
    while (std::scanf("%lld %lld %lld", &qx, &qy, &blocks) == 3) {
        NdTree t{};
        const bool accepted = nd_tree((int)qx, (int)qy, blocks, &t);
        int front = 0;
        for (int l = 0; accepted && l <= t.depth; ++l) front = std::max(front, t.lv[l].f);
        std::printf("%lld %lld %lld %d %d %d %d\n", qx, qy, blocks, accepted, accepted ? check(t, qx, qy, blocks) : 1,
                    accepted ? t.depth : -1, front);
    }
}
