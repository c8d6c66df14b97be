// Whether a plan carries the fused execution of the arithmetic that a
// contraction of it takes by default, also where the search lowered its count
// bound.
//   exec_check FORMULA_FILE ORDER THREADS ROUNDS
#include <cstdio>
#include <cstdlib>
#include <fstream>
#include <vector>

#include "fuse.hpp"
#include "internal.hpp"

using namespace tn;

int main(int argc, char** argv) {
    if (argc < 5) return 2;
    std::ifstream in(argv[1]);
    int n, m;
    in >> n >> m;
    std::vector<int32_t> ptr{0}, lits;
    std::vector<uint8_t> kinds;
    for (int c = 0; c < m; ++c) {
        int kind, len, v;
        in >> kind >> len;
        kinds.push_back(uint8_t(kind));
        for (int k = 0; k < len; ++k) {
            in >> v;
            lits.push_back(v);
        }
        ptr.push_back(int32_t(lits.size()));
    }
    tn_formula f{n, m, ptr.data(), lits.data(), kinds.data()};
    Network net;
    Plan plan;
    if (build_network(&f, net) != TN_OK) return 1;
    if (make_order(net, std::atoi(argv[2]), 1, nullptr, plan, std::atoi(argv[3]), std::atoi(argv[4])) != TN_OK) return 1;
    const int mode = default_residue_mode(plan.count_bits);
    const int es = mode == RM_WIDE ? 4 : mode == RM_SMALL || counts_by_residues(plan) ? 1 : 8;
    std::printf("bits %d of %d, entries of %d bytes%s\n", plan.count_bits, net.count_bits, es,
                default_residue_mode(net.count_bits) != mode ? ", lowered" : "");
    if (!plan_exec(plan, es)) {
        std::printf("BAD no execution\n");
        return 1;
    }
    std::printf("ok\n");
    return 0;
}
