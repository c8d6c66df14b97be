// Host entry points with every one of their allocations failing in turn: a
// status comes back and no exception crosses the C interface.
#include <cstdio>
#include <cstdlib>
#include <new>
#include <vector>

#include "tn.h"

static long left = -1;  // allocations until one fails; < 0: none does

void* operator new(std::size_t n) {
    if (left == 0) throw std::bad_alloc();
    if (left > 0) --left;
    if (void* p = std::malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void* operator new(std::size_t n, const std::nothrow_t&) noexcept {
    if (left == 0) return nullptr;
    if (left > 0) --left;
    return std::malloc(n ? n : 1);
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

template <class F>
static void each(const char* what, F f) {
    long n = 0;
    for (;; ++n) {
        left = n;
        tn_status st;
        try {
            st = f();
        } catch (...) {
            left = -1;
            std::printf("BAD %s: an exception at allocation %ld\n", what, n);
            std::exit(1);
        }
        left = -1;
        if (st == TN_OK) break;
        if (st != TN_ENOMEM) {
            std::printf("BAD %s: status %d at allocation %ld\n", what, int(st), n);
            std::exit(1);
        }
    }
    std::printf("%s: %ld allocations\n", what, n);
}

int main() {
    // vertex cover of a 2 x 8 grid
    std::vector<int32_t> ptr{0}, lits;
    std::vector<uint8_t> kinds;
    const auto edge = [&](int a, int b) {
        lits.push_back(a);
        lits.push_back(b);
        ptr.push_back(int32_t(lits.size()));
        kinds.push_back(TN_CLAUSE_OR);
    };
    for (int i = 1; i <= 8; ++i) edge(i, i + 8);
    for (int i = 1; i < 8; ++i) edge(i, i + 1), edge(i + 8, i + 9);
    tn_formula f{16, int32_t(kinds.size()), ptr.data(), lits.data(), kinds.data()};
    tn_network* net = nullptr;
    tn_plan* plan = nullptr;
    if (tn_build(&f, &net) != TN_OK || tn_order(net, TN_ORDER_GREEDY, 0, nullptr, &plan, nullptr) != TN_OK) return 1;
    std::size_t bytes = 0;
    tn_contract_opts o{};
    each("tn_plan_verify", [&] { return tn_plan_verify(plan); });
    each("tn_workspace_bytes", [&] { return tn_workspace_bytes(net, plan, &o, &bytes); });
    o.arith = TN_ARITH_RNS;
    each("tn_workspace_bytes (primes)", [&] {
        o.flags = TN_FLAG_WIDE_RNS;
        return tn_workspace_bytes(net, plan, &o, &bytes);
    });
    std::printf("ok\n");
    return 0;
}
