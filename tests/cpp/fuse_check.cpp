// Runs a plan's fused execution (fuse.hpp) on the host, reading the blob as
// the kernel does, and checks every LDS and arena access: entries are read
// only after they were written and before their place is reused, offsets stay
// within the announced sizes. The scalar (modulo 2^64) is compared with the
// plan run step by step.
//   fuse_check FORMULA_FILE ORDER ES WIDE
// FORMULA_FILE: n_vars n_clauses, then per clause: kind length literals...
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <fstream>
#include <string>
#include <vector>

#include "fuse.hpp"
#include "internal.hpp"

using namespace tn;

static uint64_t pext(uint64_t x, uint64_t m) {
    uint64_t r = 0;
    for (int k = 0; m; m &= m - 1, ++k) r |= ((x >> __builtin_ctzll(m)) & 1) << k;
    return r;
}
static void die(const char* what) {
    std::printf("BAD %s\n", what);
    std::exit(1);
}

struct Mem {
    std::vector<uint64_t> v;
    std::vector<uint8_t> set;
    explicit Mem(size_t n) : v(n, 0), set(n, 0) {}
    uint64_t get(uint64_t i) const {
        if (i >= v.size()) die("read out of range");
        if (!set[i]) die("read before write");
        return v[i];
    }
    void put(uint64_t i, uint64_t x) {
        if (i >= v.size()) die("write out of range");
        v[i] = x;
        set[i] = 1;
    }
};

static uint64_t run_steps(const Network& net, const Plan& plan, const Exec& ex, Mem& arena, bool have, uint64_t res) {
    Mem init(size_t(ex.init_elems));
    std::vector<uint64_t> e;
    for (size_t k = 0; k < ex.init_ids.size(); ++k) {
        init_entries(net.t[size_t(ex.init_ids[k])], plan.layout[size_t(ex.init_ids[k])], e);
        for (size_t x = 0; x < e.size(); ++x) init.put(uint64_t(ex.init_off[k]) + x, e[x]);
    }
    if (have) return res;
    for (const Step& st : ex.steps) {
        const Mem &A = st.initA ? init : arena, &B = st.initB ? init : arena;
        const uint64_t cm = (uint64_t(1) << st.rC) - 1;
        std::vector<uint64_t> out(size_t(cm + 1));
        for (uint64_t c = 0; c <= cm; ++c) {
            const uint64_t xa = pext(c, st.maskA) << st.s, xb = pext(c, cm & ~st.maskA) << st.s;
            uint64_t acc = 0;
            for (uint64_t z = 0; z < (uint64_t(1) << st.s); ++z)
                acc += A.get(uint64_t(st.offA) + xa + z) * B.get(uint64_t(st.offB) + xb + z);
            out[size_t(c)] = acc;
        }
        // the kernels write C while A and B are still read: they must not overlap
        auto apart = [&](bool in, int64_t off, int r) {
            if (!in && off < st.offC + (int64_t(1) << st.rC) && st.offC < off + (int64_t(1) << r)) die("C over an operand");
        };
        apart(st.initA, st.offA, st.rA);
        apart(st.initB, st.offB, st.rB);
        for (uint64_t c = 0; c <= cm; ++c) arena.put(uint64_t(st.offC) + c, out[size_t(c)]);
        // operands die here
        if (!st.initA) std::fill_n(arena.set.begin() + st.offA, size_t(1) << st.rA, 0);
        if (!st.initB) std::fill_n(arena.set.begin() + st.offB, size_t(1) << st.rB, 0);
    }
    return arena.get(uint64_t(ex.steps.back().offC));
}

static uint64_t run_exec(const Network& net, const Plan& plan, const Exec& ex, bool wide, int es) {
    const int64_t nb = ex.progs.empty() ? 0 : blob_bytes(ex, wide);
    std::vector<uint8_t> blob(size_t(nb), 0);
    Mem arena(size_t(ex.arena_elems));
    bool final = false;
    uint64_t res = 0;
    if (nb) fill_blob(net, plan, ex, wide, blob.data());
    for (size_t i = 0; i < ex.progs.size(); ++i) {
        FuseProg pg;
        std::memcpy(&pg, blob.data() + i * sizeof pg, sizeof pg);
        if (pg.prog % 16 || pg.prog + pg.prog_bytes > ex.prog_end || lds_of(pg, es) > ex.lds_bytes) die("program bytes");
        if (int64_t(ex.prog_end) + int64_t(pg.init + pg.n_init) * (wide ? 4 : 1) > nb) die("initial entries");
        Mem lds(pg.lds_elems);
        const uint8_t* e0 = blob.data() + ex.prog_end;
        for (uint32_t k = 0; k < pg.n_init; ++k)
            lds.put(k, wide ? reinterpret_cast<const uint32_t*>(e0)[pg.init + k] : e0[pg.init + k]);
        const FuseStep* steps = reinterpret_cast<const FuseStep*>(blob.data() + pg.prog);
        const uint32_t* items = reinterpret_cast<const uint32_t*>(steps + pg.n_steps);
        const uint32_t* levels = items + pg.n_items;
        if (levels[0] != 0 || levels[pg.n_levels] != pg.n_items) die("levels");
        uint64_t outputs = 0;
        for (uint32_t L = 0; L < pg.n_levels; ++L) {
            // every read of a level before any of its writes: a write must not
            // land on an entry read by the same level
            std::vector<std::pair<uint64_t, uint64_t>> writes;
            std::vector<uint8_t> read(lds.v.size(), 0);
            for (uint32_t t = levels[L]; t < levels[L + 1]; ++t) {
                if ((items[t] & 0xffff) >= pg.n_steps) die("item's step");
                const FuseStep& st = steps[items[t] & 0xffff];
                const uint32_t s = st.sr & 0xff, rC = (st.sr >> 8) & 0x7f, cm = (1u << rC) - 1;
                for (uint32_t l = 0; l < 64; ++l) {
                    const uint32_t c = (items[t] >> 16) * 64 + l;
                    if (c > cm) break;
                    const uint64_t a = st.offA + (pext(c, st.maskA) << s), b = st.offB + (pext(c, cm & ~st.maskA) << s);
                    if (st.offA % 16 || st.offB % 16) die("alignment");
                    uint64_t acc = 0;
                    for (uint64_t z = 0; z < (uint64_t(1) << s); ++z) {
                        acc += lds.get(a + z) * lds.get(b + z);
                        read[a + z] = read[b + z] = 1;
                    }
                    if (!(st.sr & kFuseRoot)) {
                        writes.push_back({st.offC + c, acc});
                    } else if (pg.final) {
                        final = true;
                        res = acc;
                    } else {
                        arena.put(uint64_t(pg.root_off) + c, acc);
                    }
                    ++outputs;
                }
            }
            std::vector<uint8_t> seen(lds.v.size(), 0);
            for (auto& wv : writes) {
                if (wv.first >= lds.v.size() || read[wv.first] || seen[wv.first]) die("LDS write");
                seen[wv.first] = 1;
                lds.put(wv.first, wv.second);
            }
        }
        uint64_t want = 0;
        for (uint32_t k = 0; k < pg.n_steps; ++k) want += uint64_t(1) << ((steps[k].sr >> 8) & 0x7f);
        if (want != outputs) die("outputs of a program");
    }
    if (final != ex.steps.empty()) die("final program");
    return run_steps(net, plan, ex, arena, final, res);
}

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
    if (build_network(&f, net) != TN_OK) die("build");
    Plan plan;
    if (make_order(net, std::atoi(argv[2]), 1, nullptr, plan, 1, 0) != TN_OK) die("order");
    const int es = std::atoi(argv[3]);
    Exec ex, plain;
    build_exec(plan, es, ex);
    plain_exec(plan, plain);
    if (ex.progs.empty()) die("no programs");
    const uint64_t a = run_exec(net, plan, ex, std::atoi(argv[4]) != 0, es),
                   b = run_exec(net, plan, plain, false, es);
    size_t fused = 0;
    for (auto& p : ex.progs) fused += p.n_steps;
    if (fused + ex.steps.size() != plan.steps.size()) die("steps lost");
    std::printf("fused %zu of %zu in %zu programs, lds %u, arena %lld against %lld, blob %lld\n", fused,
                plan.steps.size(), ex.progs.size(), ex.lds_bytes, (long long)ex.arena_elems,
                (long long)plain.arena_elems, (long long)blob_bytes(ex, false));
    std::printf("%llu\n", (unsigned long long)a);
    if (a != b) die("value");
    std::printf("ok\n");
    return 0;
}
