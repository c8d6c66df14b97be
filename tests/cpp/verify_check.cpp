// verify_exec accepts a plan's fused execution and refuses it with a program's
// result, a reader's offset or an LDS place moved.
//   verify_check FORMULA_FILE ORDER ES
#include <cstdio>
#include <cstdlib>
#include <fstream>
#include <vector>

#include "fuse.hpp"
#include "internal.hpp"

using namespace tn;

static int bad = 0;
static void expect(const char* what, tn_status got, tn_status want) {
    if (got != want) {
        std::printf("BAD %s: %d\n", what, int(got));
        bad = 1;
    }
}

int main(int argc, char** argv) {
    if (argc < 4) return 2;
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
    if (build_network(&f, net) != TN_OK || make_order(net, std::atoi(argv[2]), 1, nullptr, plan, 1, 0) != TN_OK) return 1;
    const int es = std::atoi(argv[3]);
    Exec ex;
    build_exec(plan, es, ex);
    expect("as built", verify_exec(plan, ex, es), TN_OK);
    size_t a = ex.progs.size(), b = a;
    for (size_t i = 0; i < ex.progs.size(); ++i)
        if (!ex.progs[i].final) (a == ex.progs.size() ? a : b) = i;
    std::printf("%zu programs, %zu steps\n", ex.progs.size(), ex.steps.size());
    if (a < ex.progs.size()) {
        Exec x = ex;
        x.progs[a].root_off += 64;
        expect("a result written elsewhere", verify_exec(plan, x, es), TN_EINVAL);
        x = ex;
        x.progs[a].root_off = x.arena_elems;
        for (Step& st : x.steps) {
            if (st.a == x.prog_out[a]) st.offA = x.arena_elems;
            if (st.b == x.prog_out[a]) st.offB = x.arena_elems;
        }
        expect("a result beyond the arena", verify_exec(plan, x, es), TN_EINVAL);
    }
    if (b < ex.progs.size()) {
        // both the write and the read of b's result moved onto a's
        Exec x = ex;
        x.progs[b].root_off = x.progs[a].root_off;
        for (Step& st : x.steps) {
            if (st.a == x.prog_out[b]) st.offA = x.progs[a].root_off;
            if (st.b == x.prog_out[b]) st.offB = x.progs[a].root_off;
        }
        expect("two results in one place", verify_exec(plan, x, es), TN_EINVAL);
        x = ex;
        std::swap(x.prog_out[a], x.prog_out[b]);
        expect("results exchanged", verify_exec(plan, x, es), TN_EINVAL);
    }
    for (size_t i = 0; i < ex.progs.size(); ++i) {
        Exec x = ex;
        x.progs[i].lds_elems = 15;
        expect("LDS too small", verify_exec(plan, x, es), TN_EINVAL);
        x = ex;
        x.progs[i].prog_bytes = uint32_t(kMaxProgramLds);
        expect("LDS too large", verify_exec(plan, x, es), TN_EINVAL);
    }
    for (size_t k = 0; k < ex.psteps.size(); k += 7) {
        Exec x = ex;
        x.psteps[k].offA = 1u << 20;
        expect("an operand out of LDS", verify_exec(plan, x, es), TN_EINVAL);
        x = ex;
        x.psteps[k].offB = 0xfffffff0u;
        expect("an operand out of LDS", verify_exec(plan, x, es), TN_EINVAL);
    }
    if (!bad) std::printf("ok\n");
    return bad;
}
