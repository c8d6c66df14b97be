// Batched counting of many formulas of uneven size.
//
// Host worker threads build and order the networks while the calling thread
// packs ready instances into sub-batches that fit the workspace. A sub-batch
// first runs the programs of every instance and residue plane (fuse.hpp, all
// their small steps) in a launch per element kind and LDS class; what is left
// of an instance is a chain of larger steps, and the chains, independent of
// each other, go to a few streams side by side: one chain's launches
// (529 matrix-core launches of 19 us for 256 mixed instances) leave most of
// the GPU idle. A final gather collects every instance's scalar per plane for
// one device-to-host copy, followed by CRT per instance.
//
// Measured, 256 mixed instances of 30 to 120 variables (greedy order): 55 ms
// with a wave kernel per level of small steps (34 MB of tile descriptors built and
// copied per call) and one stream, 23 ms now, of which 20 are the host threads'
// building and ordering.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <condition_variable>
#include <cstring>
#include <mutex>
#include <new>
#include <thread>
#include <vector>

#include "internal.hpp"
#include "kernels.hpp"
#include "launch.hpp"
#include "profile.hpp"
#include "streams.hpp"

namespace tn {

namespace {

struct GItem {
    const void* src;
    uint64_t* dst;
    int64_t el;  // element kind
};

// int8 residues are returned sign-extended (centred)
__global__ __launch_bounds__(256) void k_gather(const GItem* g, int64_t n) {
    const int64_t j = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (j >= n) return;
    const void* src = g[j].src;
    *g[j].dst = g[j].el == EL_U64  ? *static_cast<const uint64_t*>(src)
                : g[j].el == EL_I8 ? uint64_t(int64_t(*static_cast<const int8_t*>(src)))
                                   : *static_cast<const uint32_t*>(src);
}

struct Inst {
    Network net;
    Plan plan;
    Exec own;                 // when the plan holds no execution for its arithmetic
    const Exec* ex = nullptr;
    tn_status st = TN_OK;
    Resolved R;
    int P = 0;                // residue planes (1 for 64-bit)
    int64_t es = 4;
    int64_t blob = 0, init = 0, arena = 0;  // bytes (arena: one plane)
    int64_t arena_off = 0, blob_off = 0, init_off = 0, result = 0;  // in the sub-batch
    std::vector<uint32_t> res;
    uint64_t u64v = 0;
    int el() const { return R.u64 ? EL_U64 : R.i8 ? EL_I8 : EL_U32; }
};

int worker_count(int n) {
    unsigned hw = std::thread::hardware_concurrency();
    int w = int(hw ? hw : 4);
    w = std::min(w, 16);
    return std::max(1, std::min(w, n));
}

// milliseconds without a newly ordered instance after which the pending
// sub-batch is contracted
constexpr int kIdleFlushMs = 2;
// Instances after which the pending sub-batch is contracted while the worker
// threads go on ordering: enough programs to fill the GPU many times over.
constexpr size_t kFlush = 64;
// Chains of larger steps run side by side on this many streams (a process has
// four hardware queues).
constexpr int kChains = 4;
// LDS classes of the programs: work-groups of 512 threads, four, two or one
// of which fit a CU's 160 KB.
constexpr uint32_t kLdsClass[3] = {40u << 10, 80u << 10, uint32_t(kMaxProgramLds)};

int64_t align_up(int64_t x, int64_t a) { return (x + a - 1) / a * a; }
// where an instance's planes start in the workspace (large tensors are laid
// out at multiples of 2^20 entries of an arena)
int64_t arena_align(const Inst& I) { return I.arena >= (int64_t(1) << 20) ? int64_t(1) << 20 : 256; }

struct SubBatch {
    std::vector<int32_t> ids;
    int64_t bytes = 0;
};

int64_t bytes_of(const Inst& I) {
    const int64_t per_plane = int64_t(sizeof(FusePlane) + sizeof(GItem)) + 8;
    return I.P * I.arena + arena_align(I) + I.blob + I.init +
           I.P * (per_plane + int64_t(I.ex->progs.size()) * int64_t(sizeof(uint2))) + 2048;
}

// Workspace a call keeps for the scratch of its chains; one chain at a time
// when the workspace is small.
int chains_of(const tn_contract_opts* o) {
    const int64_t one = int64_t(kMaxGroup) * kScratchPerPrime;
    return (o->flags & TN_FLAG_TIMING) || int64_t(o->workspace_bytes) < 16 * kChains * one ? 1 : kChains;
}

// Runs one sub-batch: every instance in it has a plan and fits the layout.
tn_status run_sub(std::vector<Inst>& ins, const SubBatch& sb, const tn_contract_opts* o, int chains) {
    hipStream_t stream = static_cast<hipStream_t>(o->stream);
    char* base = static_cast<char*>(o->workspace);
    // layout: [arenas][scratch of every chain][image][results]; the image is
    // one upload: [initial tensors][blobs][planes][work lists][gather list]
    int64_t off = 0, img = 0, results = 0;
    size_t n_planes = 0;
    std::vector<uint2> work[3][3];  // element kind, LDS class
    uint32_t lds_max[3][3] = {};
    for (int32_t i : sb.ids) {
        Inst& I = ins[size_t(i)];
        I.arena_off = off = align_up(off, arena_align(I));
        off += I.P * I.arena;
        I.init_off = img;
        I.blob_off = img + I.init;
        img += I.init + I.blob;
        I.result = results;
        for (int q = 0; q < I.P; ++q)
            for (size_t p = 0; p < I.ex->progs.size(); ++p) {
                const uint32_t l = lds_of(I.ex->progs[p], int(I.es));
                const int c = l <= kLdsClass[0] ? 0 : l <= kLdsClass[1] ? 1 : 2;
                work[I.el()][c].push_back(uint2{uint32_t(n_planes) + uint32_t(q), uint32_t(p)});
                lds_max[I.el()][c] = std::max(lds_max[I.el()][c], l);
            }
        n_planes += size_t(I.P);
        results += I.P;
    }
    const int64_t scratch_bytes = int64_t(kMaxGroup) * kScratchPerPrime;
    const int64_t scratch_off = off = align_up(off, 256);
    off += chains * scratch_bytes;
    const int64_t img_off = off;
    const int64_t planes_off = img = align_up(img, 256);
    img = align_up(img + int64_t(n_planes * sizeof(FusePlane)), 256);
    int64_t work_off[3][3];
    for (int e = 0; e < 3; ++e)
        for (int c = 0; c < 3; ++c) {
            work_off[e][c] = img;
            img += int64_t(work[e][c].size() * sizeof(uint2));
        }
    const int64_t gather_off = img = align_up(img, 256);
    const int64_t result_off = img_off + align_up(img + results * int64_t(sizeof(GItem)), 256);
    if (result_off + results * 8 > int64_t(o->workspace_bytes)) return TN_ETOOBIG;
    uint64_t* d_res = reinterpret_cast<uint64_t*>(base + result_off);

    std::vector<uint8_t> host(size_t(gather_off + results * int64_t(sizeof(GItem))), 0);
    std::vector<GItem> gathers;
    size_t plane = 0;
    for (int32_t i : sb.ids) {
        Inst& I = ins[size_t(i)];
        fill_init(I.net, I.plan, I.ex->init_ids, I.ex->init_off, I.el(), host.data() + I.init_off);
        if (I.blob) fill_blob(I.net, I.plan, *I.ex, false, host.data() + I.blob_off);
        for (int q = 0; q < I.P; ++q, ++plane) {
            FusePlane pl{};
            char* arena = base + I.arena_off + q * I.arena;
            pl.blob = reinterpret_cast<const uint8_t*>(base + img_off + I.blob_off);
            pl.arena = arena;
            pl.res = d_res + I.result + q;
            pl.prog_end = I.ex->prog_end;
            if (!I.R.u64) {
                pl.p = I.R.primes[size_t(q)];
                pl.r2 = uint32_t((uint64_t(1) << 32) % pl.p);
                pl.r16 = uint32_t(65536u % pl.p);
                pl.pinv = 1.0f / float(pl.p);
            }
            std::memcpy(host.data() + planes_off + plane * sizeof pl, &pl, sizeof pl);
            if (!I.ex->steps.empty())
                gathers.push_back({arena + I.ex->steps.back().offC * I.es, pl.res, int64_t(I.el())});
        }
    }
    for (int e = 0; e < 3; ++e)
        for (int c = 0; c < 3; ++c)
            if (!work[e][c].empty())
                std::memcpy(host.data() + work_off[e][c], work[e][c].data(), work[e][c].size() * sizeof(uint2));
    if (!gathers.empty()) std::memcpy(host.data() + gather_off, gathers.data(), gathers.size() * sizeof(GItem));
    std::vector<uint64_t> out(static_cast<size_t>(results), 0);
    // chains, heaviest first, each to the stream with the least so far
    struct Chain {
        int32_t id;
        double us;
        std::vector<uint8_t> dig;
    };
    std::vector<Chain> list;
    for (int32_t i : sb.ids) {
        const Inst& I = ins[size_t(i)];
        if (I.ex->steps.empty()) continue;
        Chain c{i, 0, {}};
        const int mode = I.R.u64 ? RM_U64 : I.R.i8 ? RM_SMALL : RM_WIDE;
        std::vector<KernelClass> cls(I.ex->steps.size());
        for (size_t k = 0; k < cls.size(); ++k) {
            const Step& st = I.ex->steps[k];
            cls[k] = choose_class(st, I.el(), o->flags);
            c.us += 5.0 + I.P * step_cost_model(st.rA, st.rB, st.s, st.rC, mode);
        }
        c.dig = digit_plan(I.ex->steps, I.plan.rank.size(), cls, I.el());
        list.push_back(std::move(c));
    }
    std::sort(list.begin(), list.end(), [](const Chain& x, const Chain& y) {
        return x.us != y.us ? x.us > y.us : x.id < y.id;
    });

    Profiler& prof = profiler();
    // the side streams are drained by their owner before anything above goes
    // away, and the caller's by its guard where a failure or an exception ends
    // the call first
    DrainGuard guard(stream);
    SideStreams side(std::min<int>(chains, int(list.size())) - 1);
    auto fail = [&]() {
        for (size_t k = 0; k < side.size(); ++k) (void)hipStreamSynchronize(side[k].stream);
        (void)hipStreamSynchronize(stream);
        prof.collect();
        return TN_EHIP;
    };
    hipError_t err =
        hipMemcpyAsync(base + img_off, host.data(), host.size(), hipMemcpyHostToDevice, stream);
    for (int e = 0; e < 3 && err == hipSuccess; ++e)
        for (int c = 0; c < 3 && err == hipSuccess; ++c) {
            const int64_t n = int64_t(work[e][c].size());
            if (n == 0) continue;
            prof.cur_rA = prof.cur_rB = prof.cur_s = prof.cur_rC = 0;
            prof.cur_G = int32_t(n);  // programs in the launch
            prof.before(stream);
            err = launch_fused_many(e, reinterpret_cast<const FusePlane*>(base + img_off + planes_off),
                                    base + img_off + work_off[e][c], n, lds_max[e][c], stream);
            prof.after_raw(stream, KC_BATCH, 0, 0);
        }
    if (prof.on) {
        // the programs' work, booked with their first launch
        for (int32_t i : sb.ids) {
            const Inst& I = ins[size_t(i)];
            prof.acc[KC_BATCH].bytes += double(I.es) * I.P * I.ex->prog_entries;
            prof.acc[KC_BATCH].macs += I.P * I.ex->prog_macs;
        }
    }
    if (err != hipSuccess) return fail();
    // fork: the side streams wait for the programs
    const size_t n_streams = 1 + side.size();
    for (size_t k = 0; k < side.size() && err == hipSuccess; ++k) {
        err = hipEventRecord(side[k].event, stream);
        if (err == hipSuccess) err = hipStreamWaitEvent(side[k].stream, side[k].event, 0);
    }
    std::vector<double> load(n_streams, 0.0);
    for (size_t k = 0; k < list.size() && err == hipSuccess; ++k) {
        Inst& I = ins[size_t(list[k].id)];
        const size_t t = size_t(std::min_element(load.begin(), load.end()) - load.begin());
        load[t] += list[k].us;
        hipStream_t s = t == 0 ? stream : side[t - 1].stream;
        char* scratch = base + scratch_off + int64_t(t) * scratch_bytes;
        for (int g0 = 0; g0 < I.P && err == hipSuccess; g0 += kMaxGroup) {
            const int gn = std::min(kMaxGroup, I.P - g0);
            for (size_t j = 0; j < I.ex->steps.size() && err == hipSuccess; ++j) {
                KernelClass kc = KC_GENERIC;
                err = launch_step(I.ex->steps[j], I.el(), o->flags, I.R.u64 ? nullptr : I.R.primes.data() + g0, gn,
                                  base + img_off + I.init_off, base + I.arena_off + g0 * I.arena, I.arena / I.es,
                                  scratch, s, &kc, -1, list[k].dig[j]);
            }
        }
    }
    // join
    for (size_t k = 0; k < side.size() && err == hipSuccess; ++k) {
        err = hipEventRecord(side[k].event, side[k].stream);
        if (err == hipSuccess) err = hipStreamWaitEvent(stream, side[k].event, 0);
    }
    if (err == hipSuccess && !gathers.empty()) {
        const int64_t n = int64_t(gathers.size());
        hipLaunchKernelGGL(k_gather, dim3(uint32_t((n + 255) / 256)), dim3(256), 0, stream,
                           reinterpret_cast<const GItem*>(base + img_off + gather_off), n);
        err = hipGetLastError();
    }
    if (err == hipSuccess && !out.empty())
        err = hipMemcpyAsync(out.data(), d_res, out.size() * 8, hipMemcpyDeviceToHost, stream);
    if (err != hipSuccess) return fail();
    if (hipStreamSynchronize(stream) != hipSuccess) return fail();
    guard.drained();
    prof.collect();
    for (int32_t i : sb.ids) {
        Inst& I = ins[size_t(i)];
        for (int q = 0; q < I.P; ++q) {
            const uint64_t v = out[size_t(I.result + q)];
            if (I.R.u64) {
                I.u64v = v;
            } else if (I.R.i8) {
                const int64_t m = I.R.primes[size_t(q)], c = int64_t(v);
                I.res[size_t(q)] = uint32_t(c < 0 ? c + m : c);
            } else {
                I.res[size_t(q)] = uint32_t(v);
            }
        }
    }
    return TN_OK;
}

}  // namespace

}  // namespace tn

using namespace tn;

extern "C" tn_status tn_count_batch(const tn_formula* fs, int32_t n, tn_order_kind kind, uint64_t seed,
                                    const tn_contract_opts* opts, uint32_t* limbs, size_t cap_per,
                                    size_t* n_limbs, tn_plan_stats* stats) {
    if (n < 0 || (n > 0 && (!fs || !opts || !n_limbs || !opts->workspace))) return TN_EINVAL;
    if (n == 0) return TN_OK;
    std::vector<Inst> ins;
    try {
        ins.resize(size_t(n));
    } catch (const std::bad_alloc&) {
        return TN_ENOMEM;
    }
    profiler().start(opts->flags & TN_FLAG_TIMING);
    std::mutex mu;
    std::condition_variable cv;
    std::atomic<int32_t> next{0};
    std::vector<int32_t> done;  // instances in the order their plans were finished
    done.reserve(size_t(n));
    auto work = [&]() {
        for (;;) {
            const int32_t i = next.fetch_add(1);
            if (i >= n) return;
            Inst& s = ins[size_t(i)];
            s.st = build_network(&fs[i], s.net);
            if (s.st == TN_OK) s.st = make_order(s.net, kind, seed + uint64_t(i), nullptr, s.plan);
            {
                std::lock_guard<std::mutex> lk(mu);
                done.push_back(i);
            }
            cv.notify_all();
        }
    };
    std::vector<std::thread> pool;
    const int W = worker_count(n);
    for (int w = 0; w < W; ++w) pool.emplace_back(work);

    const int chains = chains_of(opts);
    const int64_t cap = int64_t(opts->workspace_bytes) - int64_t(chains) * kMaxGroup * kScratchPerPrime - (1 << 20);
    tn_status first_err = TN_OK;
    auto note = [&](tn_status s) {
        if (s != TN_OK && first_err == TN_OK) first_err = s;
    };
    SubBatch sb;
    auto flush = [&]() {
        if (sb.ids.empty()) return;
        tn_status s;
        try {
            s = run_sub(ins, sb, opts, chains);
        } catch (const std::bad_alloc&) {
            s = TN_ENOMEM;
        }
        for (int32_t i : sb.ids) {
            if (s != TN_OK) ins[i].st = s;
        }
        note(s);
        sb = SubBatch{};
    };
    // resolves an ordered instance and adds it to the pending sub-batch
    auto take = [&](int32_t i, Inst& I) {
        if (I.st != TN_OK) return;
        I.st = resolve(I.plan, opts, I.R);
        if (I.st != TN_OK) return;
        const Resolved asked = I.R;
        if (Resolved rr; residue_route(I.net, I.plan, I.R, opts, rr)) I.R = rr;
        I.P = I.R.u64 ? 1 : I.R.k;
        I.es = I.R.es();
        I.res.assign(size_t(I.R.u64 ? 0 : I.R.k), 0);
        if (I.plan.n_init == 0 || I.plan.steps.empty()) {
            // empty network or a single scalar tensor: no device work
            std::vector<uint64_t> one(1, 1);
            if (I.plan.n_init != 0) init_entries(I.net.t[size_t(I.plan.root)], {}, one);
            const uint64_t v = one[0];
            I.u64v = v;
            for (int q = 0; q < int(I.res.size()); ++q) I.res[size_t(q)] = uint32_t(v % I.R.primes[size_t(q)]);
            return;
        }
        if (opts->flags & TN_FLAG_GENERIC_ONLY) {
            plain_exec(I.plan, I.own);
            I.ex = &I.own;
        } else if (!(I.ex = plan_exec(I.plan, int(I.es)))) {
            build_exec(I.plan, int(I.es), I.own);
            I.ex = &I.own;
        }
        I.init = align256(I.ex->init_elems * I.es);
        I.blob = I.ex->progs.empty() ? 0 : blob_bytes(*I.ex, false);
        I.arena = align256(I.ex->arena_elems * I.es);
        const int64_t need = bytes_of(I);
        if (need > cap) {
            // too large to share the workspace: run alone, primes grouped as memory allows
            // (and 64-bit counts by the route that suits the planes that fit)
            flush();
            std::vector<uint32_t> res;
            uint64_t v = 0;
            I.R = asked;
            I.st = run_plan(I.net, I.plan, opts, I.R, res, &v);
            I.res = res;
            I.u64v = v;
            return;
        }
        if (sb.bytes + need > cap) flush();
        sb.ids.push_back(i);
        sb.bytes += need;
        if (sb.ids.size() >= kFlush) flush();
    };
    // Instances are contracted in the order their plans become ready (order
    // searches differ in length). When no new plan arrives for a while, the
    // pending sub-batch goes to the device rather than leaving it idle.
    size_t taken = 0;
    for (int32_t got = 0; got < n; ++got) {
        int32_t i;
        {
            std::unique_lock<std::mutex> lk(mu);
            auto more = [&] { return taken < done.size(); };
            if (!sb.ids.empty() && !cv.wait_for(lk, std::chrono::milliseconds(kIdleFlushMs), more)) {
                lk.unlock();
                flush();
                lk.lock();
            }
            cv.wait(lk, more);
            i = done[taken++];
        }
        Inst& I = ins[size_t(i)];
        try {
            take(i, I);
        } catch (const std::bad_alloc&) {
            I.st = TN_ENOMEM;
        }
    }
    flush();
    for (auto& t : pool) t.join();

    for (int32_t i = 0; i < n; ++i) {
        Inst& I = ins[size_t(i)];
        if (stats) stats[i] = I.plan.stats;
        if (I.st != TN_OK) {
            n_limbs[i] = 0;
            note(I.st);
            continue;
        }
        std::vector<uint32_t> L;
        if (I.R.u64) {
            L = {uint32_t(I.u64v), uint32_t(I.u64v >> 32)};
            while (L.size() > 1 && L.back() == 0) L.pop_back();
        } else {
            crt_limbs(I.res.data(), I.R.primes.data(), I.R.k, L);
        }
        n_limbs[i] = L.size();
        if (limbs && L.size() <= cap_per)
            std::copy(L.begin(), L.end(), limbs + size_t(i) * cap_per);
        else
            note(TN_EBUFSIZE);
    }
    return first_err;
}
