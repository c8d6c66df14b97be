// Host side of the fused small steps (fuse.hpp): which steps are fused, and
// the programs' layout.
#include "fuse.hpp"

#include <algorithm>
#include <cmath>
#include <cstring>

#include "arena.hpp"

namespace tn {

namespace {

struct Limits {
    int rank;        // largest tensor rank of a fused step
    int64_t work;    // largest work of a program (work_of)
    int64_t elems;   // largest LDS use of its tensors (entries)
};

// A work-group does about 30 multiply-adds per clock on bytes and 4 on 64-bit
// words, so these programs end within a few launch times; a program's tensors
// are held to 96 KB of LDS (most programs take less than 12), and with its text,
// which a long chain of tiny steps makes the larger part, to what a work-group
// may ask for. Measured with half and twice the work:
// vertex cover n = 60 82 / 53 / 53 us (2^15, 2^17, 2^18), hard-core n = 100 534 /
// 489 / 498 us (2^16 and rank 12, 2^17, 2^18), vertex cover n = 120 95 / 93 / 93
// us (2^16, 2^17, 2^18).
Limits limits_of(int es) {
    if (es == 1) return {13, int64_t(1) << 17, int64_t(96) << 10};
    if (es == 4) return {13, int64_t(1) << 17, int64_t(24) << 10};
    return {12, int64_t(1) << 17, int64_t(12) << 10};
}

// Work of a step for one work-group, in multiply-adds: every output costs
// about eight more (index gathers, reduction, store).
int64_t work_of(const Step& st) {
    return (int64_t(1) << (st.rA + st.rB - st.s)) + (int64_t(8) << st.rC);
}

// Items of a step (64 outputs each) and bytes of a program's text.
int64_t items_of(int rank) { return int64_t(1) << std::max(rank - 6, 0); }
int64_t text_bytes(int64_t steps, int64_t items, int64_t levels) {
    return (steps * int64_t(sizeof(FuseStep)) + (items + levels + 1) * 4 + 15) / 16 * 16;
}

int64_t lds_size(int rank) { return std::max<int64_t>(16, int64_t(1) << rank); }

// Tensors of a class lie at multiples of its unit, in a part of the arena of
// their own: the matrix-core kernels read rows in lines of 128 bytes, and write
// tiles of powers of two. At offsets of any multiple of 64 entries the largest
// 1-in-3 plan (n = 300, 11 planes) took 103.7 ms, with tensors of 2^20 entries
// and more at multiples of that 98.5 ms. Sizes are powers of two, so the first
// fit keeps the multiples.
constexpr int kClasses = 3;
constexpr int64_t kUnit[kClasses] = {256, int64_t(1) << 12, int64_t(1) << 20};
int class_of(int rank) {
    int c = 0;
    while (c + 1 < kClasses && (int64_t(1) << rank) >= kUnit[c + 1]) ++c;
    return c;
}

int64_t align_up(int64_t x, int64_t a) { return (x + a - 1) / a * a; }

}  // namespace

void plain_exec(const Plan& plan, Exec& ex) {
    ex = Exec{};
    ex.steps = plan.steps;
    ex.init_ids.resize(size_t(plan.n_init));
    for (int32_t i = 0; i < plan.n_init; ++i) ex.init_ids[size_t(i)] = i;
    ex.init_off = plan.init_off;
    ex.init_elems = plan.init_elems;
    ex.arena_elems = plan.arena_elems;
}

void build_exec(const Plan& plan, int es, Exec& ex) {
    ex = Exec{};
    const Limits lim = limits_of(es);
    const int32_t n_init = plan.n_init, n_steps = int32_t(plan.steps.size());
    const int32_t n_ids = n_init + n_steps;
    // fused[k]: step k and everything below it fits one program
    std::vector<uint8_t> fused(size_t(n_steps), 0), inner(size_t(n_steps), 0);
    std::vector<int64_t> work(size_t(n_steps), 0);
    // steps and items of step k and all below, and entries that are in LDS
    // together at the end of the first level (its inputs, and its outputs other
    // than k's): what a program takes at least (it has its root's levels). The
    // layout below decides; without this a long formula laid out thousands of
    // programs that could not fit, one step smaller each time (3000 unit clauses,
    // bytes: 0.4 s).
    struct Size {
        int64_t steps, items, first;
    };
    std::vector<Size> size(size_t(n_steps), Size{});
    for (int32_t k = 0; k < n_steps; ++k) {
        const Step& st = plan.steps[size_t(k)];
        if (std::max({st.rA, st.rB, st.rC}) > lim.rank) continue;
        int64_t w = work_of(st);
        Size z{1, items_of(st.rC), 0};
        bool ok = true;
        for (int32_t id : {st.a, st.b}) {
            if (id < n_init) {
                z.first += lds_size(plan.rank[size_t(id)]);
                continue;
            }
            const size_t c = size_t(id - n_init);
            ok = ok && fused[c];
            w += work[c];
            const Step& below = plan.steps[c];
            z = {z.steps + size[c].steps, z.items + size[c].items,
                 z.first + size[c].first + (below.level == 1 ? lds_size(below.rC) : 0)};
        }
        if (!ok || w > lim.work) continue;
        if (z.first > lim.elems ||
            align_up(z.first * es, 16) + text_bytes(z.steps, z.items, st.level) > kMaxProgramLds)
            continue;
        fused[size_t(k)] = 1;
        work[size_t(k)] = w;
        size[size_t(k)] = z;
        for (int32_t id : {st.a, st.b})
            if (id >= n_init) inner[size_t(id - n_init)] = 1;
    }
    // programs: depth-first lists of the steps below each root, roots last
    // to first so that a root whose program does not fit LDS can hand its
    // children on as roots
    std::vector<int64_t> loff(size_t(n_ids), -1);
    std::vector<int32_t> mine, stack, by_level, inits, count;
    std::vector<uint8_t> in_prog(size_t(n_steps), 0);
    Arena lds;
    std::vector<int32_t> root_step;
    for (int32_t r = n_steps - 1; r >= 0; --r) {
        if (!fused[size_t(r)] || inner[size_t(r)] || in_prog[size_t(r)]) continue;
        mine.clear();
        inits.clear();
        stack.assign(1, r);
        while (!stack.empty()) {
            const int32_t k = stack.back();
            stack.pop_back();
            mine.push_back(k);
            const Step& st = plan.steps[size_t(k)];
            for (int32_t id : {st.a, st.b}) {
                if (id < n_init)
                    inits.push_back(id);
                else
                    stack.push_back(id - n_init);
            }
        }
        // LDS: every initial tensor from the start, then level by level,
        // outputs of a level before the release of its inputs
        std::sort(mine.begin(), mine.end(), [&](int32_t x, int32_t y) {
            const int32_t lx = plan.steps[size_t(x)].level, ly = plan.steps[size_t(y)].level;
            return lx != ly ? lx < ly : x < y;
        });
        lds = Arena{};
        int64_t n_entries = 0;
        for (int32_t id : inits) {
            loff[size_t(id)] = lds.alloc(lds_size(plan.rank[size_t(id)]));
            n_entries = std::max(n_entries, loff[size_t(id)] + lds_size(plan.rank[size_t(id)]));
        }
        size_t at = 0;
        while (at < mine.size()) {
            size_t end = at;
            const int32_t L = plan.steps[size_t(mine[at])].level;
            for (; end < mine.size() && plan.steps[size_t(mine[end])].level == L; ++end) {
                const Step& st = plan.steps[size_t(mine[end])];
                if (mine[end] != r) loff[size_t(st.out)] = lds.alloc(lds_size(st.rC));
            }
            for (; at < end; ++at) {
                const Step& st = plan.steps[size_t(mine[at])];
                lds.release(loff[size_t(st.a)], lds_size(st.rA));
                lds.release(loff[size_t(st.b)], lds_size(st.rB));
            }
        }
        int64_t n_items = 0, n_levels = 0;
        for (size_t j = 0; j < mine.size(); ++j) {
            const Step& st = plan.steps[size_t(mine[j])];
            n_items += items_of(st.rC);
            n_levels += j == 0 || st.level != plan.steps[size_t(mine[j - 1])].level;
        }
        const int64_t text = text_bytes(int64_t(mine.size()), n_items, n_levels);
        if (lds.high > lim.elems || align_up(lds.high * es, 16) + text > kMaxProgramLds) {
            const Step& st = plan.steps[size_t(r)];
            fused[size_t(r)] = 0;
            for (int32_t id : {st.a, st.b})
                if (id >= n_init) inner[size_t(id - n_init)] = 0;
            continue;
        }
        // levels of a program are the plan's, renumbered without gaps
        FuseProg pg{};
        pg.n_steps = uint32_t(mine.size());
        const size_t item0 = ex.pitems.size(), level0 = ex.plevels.size();
        int32_t last_level = -1;
        for (size_t j = 0; j < mine.size(); ++j) {
            const int32_t k = mine[j];
            const Step& st = plan.steps[size_t(k)];
            in_prog[size_t(k)] = 1;
            if (st.level != last_level) {
                ex.plevels.push_back(uint32_t(ex.pitems.size() - item0));
                last_level = st.level;
            }
            FuseStep fs{};
            fs.offA = uint32_t(loff[size_t(st.a)]);
            fs.offB = uint32_t(loff[size_t(st.b)]);
            fs.offC = k == r ? 0 : uint32_t(loff[size_t(st.out)]);
            fs.maskA = uint16_t(st.maskA);
            fs.sr = uint16_t(uint32_t(st.s) | (uint32_t(st.rC) << 8) | (k == r ? kFuseRoot : 0));
            ex.psteps.push_back(fs);
            const uint32_t chunks = uint32_t(items_of(st.rC));
            for (uint32_t c = 0; c < chunks; ++c) ex.pitems.push_back(uint32_t(j) | (c << 16));
            ex.prog_entries += std::ldexp(1.0, st.rA) + std::ldexp(1.0, st.rB) + std::ldexp(1.0, st.rC);
            ex.prog_macs += std::ldexp(1.0, st.rA + st.rB - st.s);
        }
        ex.plevels.push_back(uint32_t(ex.pitems.size() - item0));
        pg.n_items = uint32_t(ex.pitems.size() - item0);
        pg.n_levels = uint32_t(ex.plevels.size() - level0 - 1);
        pg.n_init = uint32_t(n_entries);
        pg.final = plan.steps[size_t(r)].out == plan.root ? 1u : 0u;
        pg.prog_bytes = uint32_t(text);
        ex.pinit_first.push_back(int32_t(ex.pinit.size()));
        for (int32_t id : inits) {
            ex.pinit.push_back(id);
            ex.pinit_off.push_back(uint32_t(loff[size_t(id)]));
        }
        pg.lds_elems = uint32_t(lds.high);
        ex.lds_bytes = std::max(ex.lds_bytes, lds_of(pg, es));
        ex.progs.push_back(pg);
        ex.prog_out.push_back(plan.steps[size_t(r)].out);
        root_step.push_back(r);
    }
    ex.pinit_first.push_back(int32_t(ex.pinit.size()));
    // blob: headers, programs, initial entries
    int64_t off = int64_t(ex.progs.size()) * int64_t(sizeof(FuseProg));
    for (FuseProg& pg : ex.progs) {
        pg.prog = uint32_t(off);
        off += pg.prog_bytes;
    }
    ex.prog_end = uint32_t(off);
    for (FuseProg& pg : ex.progs) {
        pg.init = ex.n_entries;
        ex.n_entries += uint32_t(align_up(pg.n_init, 16));
    }
    // arena: the programs' results live from the start, then the other
    // steps in plan order; a part per size class
    Arena part[kClasses];
    std::vector<int64_t> goff(size_t(n_ids), -1);
    const auto take = [&](int rank) {
        const int c = class_of(rank);
        return part[c].alloc(align_up(int64_t(1) << rank, kUnit[c]));
    };
    const auto drop = [&](int64_t off, int rank) {
        const int c = class_of(rank);
        part[c].release(off, align_up(int64_t(1) << rank, kUnit[c]));
    };
    for (size_t i = 0; i < ex.progs.size(); ++i) {
        const Step& st = plan.steps[size_t(root_step[i])];
        if (ex.progs[i].final) continue;
        goff[size_t(st.out)] = take(st.rC);
        ex.progs[i].root_off = goff[size_t(st.out)];
        ex.progs[i].root_rank = st.rC;
    }
    std::vector<int64_t> ioff(size_t(n_init), -1);
    for (int32_t k = 0; k < n_steps; ++k) {
        if (in_prog[size_t(k)]) continue;
        Step st = plan.steps[size_t(k)];
        st.offC = goff[size_t(st.out)] = take(st.rC);
        for (int side = 0; side < 2; ++side) {
            const int32_t id = side ? st.b : st.a;
            const int rank = side ? st.rB : st.rA;
            int64_t& o = side ? st.offB : st.offA;
            if (id < n_init) {
                if (ioff[size_t(id)] < 0) {
                    ioff[size_t(id)] = ex.init_elems;
                    ex.init_ids.push_back(id);
                    ex.init_off.push_back(ex.init_elems);
                    ex.init_elems += align_up(int64_t(1) << rank, kAlignElems);
                }
                o = ioff[size_t(id)];
            } else {
                o = goff[size_t(id)];
                drop(o, rank);
            }
        }
        ex.steps.push_back(st);
    }
    // parts one after the other
    int64_t base[kClasses], end = 0;
    for (int c = 0; c < kClasses; ++c) {
        base[c] = part[c].high > 0 ? align_up(end, kUnit[c]) : end;
        end = base[c] + part[c].high;
    }
    for (FuseProg& pg : ex.progs)
        if (!pg.final) pg.root_off += base[class_of(pg.root_rank)];
    for (Step& st : ex.steps) {
        if (!st.initA) st.offA += base[class_of(st.rA)];
        if (!st.initB) st.offB += base[class_of(st.rB)];
        st.offC += base[class_of(st.rC)];
    }
    // planes keep the largest class's multiples
    int64_t unit = kUnit[0];
    for (int c = 0; c < kClasses; ++c)
        if (part[c].high > 0) unit = kUnit[c];
    ex.arena_elems = std::max<int64_t>(align_up(end, unit), kAlignElems);
}

int64_t blob_bytes(const Exec& ex, bool wide) {
    return align_up(int64_t(ex.prog_end) + int64_t(ex.n_entries) * (wide ? 4 : 1), 256);
}

void fill_blob(const Network& net, const Plan& plan, const Exec& ex, bool wide, uint8_t* blob) {
    size_t step = 0, item = 0, level = 0;
    std::memcpy(blob, ex.progs.data(), ex.progs.size() * sizeof(FuseProg));
    std::vector<uint64_t> v;
    for (size_t i = 0; i < ex.progs.size(); ++i) {
        const FuseProg& pg = ex.progs[i];
        uint8_t* p = blob + pg.prog;
        std::memcpy(p, ex.psteps.data() + step, pg.n_steps * sizeof(FuseStep));
        p += pg.n_steps * sizeof(FuseStep);
        std::memcpy(p, ex.pitems.data() + item, pg.n_items * 4);
        p += pg.n_items * 4;
        std::memcpy(p, ex.plevels.data() + level, (pg.n_levels + 1) * 4);
        step += pg.n_steps;
        item += pg.n_items;
        level += pg.n_levels + 1;
        for (int32_t j = ex.pinit_first[i]; j < ex.pinit_first[i + 1]; ++j) {
            const int32_t id = ex.pinit[size_t(j)];
            init_entries(net.t[size_t(id)], plan.layout[size_t(id)], v);
            const size_t at = size_t(pg.init) + ex.pinit_off[size_t(j)];
            if (wide)
                for (size_t x = 0; x < v.size(); ++x)
                    reinterpret_cast<uint32_t*>(blob + ex.prog_end)[at + x] = uint32_t(v[x]);
            else
                for (size_t x = 0; x < v.size(); ++x) blob[ex.prog_end + at + x] = uint8_t(v[x]);
        }
    }
}

const Exec* plan_exec(const Plan& plan, int es) {
    return plan.exec && plan.exec_es == es ? plan.exec.get() : nullptr;
}

}  // namespace tn
