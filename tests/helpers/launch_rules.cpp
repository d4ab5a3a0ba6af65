// Prints what the library's launch rules answer.  Reads lines
//   levels K n [K n ...]        -> steps of Tables (one step size, n nodes a level)
//   blocks steps longest per_lane block -> long_blocks
//   lockstep K t mode            -> lockstep_paths
//   mesh table grid_n paths stride t K nodes -> lockstep_mesh on 256 CUs
//   network nodes paths masked heavy -> network_chunk on 256 CUs
//   mgg K t u bridge            -> mgg_form where four and six workgroups fit: 10 pairs + blocks
#include <hip/hip_runtime.h>

#include <cstdio>
#include <iostream>
#include <sstream>
#include <string>
#include <vector>

#include "fk_internal.hpp"

using namespace fk;

static int64_t table_steps(const std::vector<int64_t> &v) {
    const double dt = 1e-5;
    std::vector<LevelSpec> lv;
    int64_t total = 0;
    for (size_t i = 0; i + 1 < v.size(); i += 2) {
        LevelSpec s{};
        s.w.kind = FK_DENSITY_CONST;
        s.t = (double)v[i] * dt;
        s.node_offset = total;
        s.n_nodes = v[i + 1];
        s.level_id = (uint32_t)(i / 2);
        total += v[i + 1];
        lv.push_back(s);
    }
    const std::vector<double> pts((size_t)(2 * total), 0.5);
    fk_data d{};
    Tables T;
    if (build_tables(lv.data(), (int)lv.size(), pts.data(), total, &d, dt, T) != FK_OK) return -1;
    return T.steps;
}

int main() {
    std::string line, what;
    while (std::getline(std::cin, line)) {
        std::istringstream in(line);
        in >> what;
        std::vector<double> v;
        for (double x; in >> x;) v.push_back(x);
        long long r = -1;
        if (what == "levels") r = table_steps(std::vector<int64_t>(v.begin(), v.end()));
        if (what == "blocks") r = long_blocks((int64_t)v.at(0), (int64_t)v.at(1), v.at(2), (int)v.at(3));
        if (what == "lockstep") r = lockstep_paths((int64_t)v.at(0), v.at(1), (int)v.at(2));
        if (what == "mesh")
            r = lockstep_mesh(v.at(0) != 0.0, (int)v.at(1), (int64_t)v.at(2), (int64_t)v.at(3), v.at(4),
                              (int64_t)v.at(5), (int64_t)v.at(6), 256, false);
        if (what == "network")
            r = network_chunk((int64_t)v.at(0), (int64_t)v.at(1), 256, v.at(2) != 0.0, v.at(3) != 0.0);
        if (what == "mgg") {
            const MggForm f = mgg_form((int64_t)v.at(0), v.at(1), v.at(2), v.at(3) != 0.0, 4, 6);
            r = 10 * f.pairs + f.blocks;
        }
        std::printf("%lld\n", r);
    }
}
