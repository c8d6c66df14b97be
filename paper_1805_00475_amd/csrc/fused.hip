// Small steps fused: one work-group per program (a maximal subtree of small
// steps, fuse.cpp) and residue plane, every intermediate in LDS.
//
// Run one launch per step, such steps cost a launch each (3 us on an idle
// queue, whatever the step's size), and 94-100 % of a plan's steps are of this
// kind: vertex cover n = 120 has 299 steps of which 292 fit programs. A program
// runs its steps level by level: the items of a level (64 outputs of one step)
// are dealt to the work-group's waves, then one barrier. What bounds a program
// is its depth: about 10 levels of a barrier, a step's index gathers and its
// sum, each a few LDS latencies; so programs are kept to the work at which a
// step's sums would take longer than its own launch. Measured, one count with
// its plan in hand, the narrow and generic kernels of its larger steps
// included: vertex cover n = 60 (149 steps, 64-bit counts) 620 -> 50 us, n = 120
// (9 planes) 1161 -> 97 us, hard-core n = 100 (349 steps, 66 primes) 7.0 -> 0.34 ms;
// the launch itself takes 11-27 us. Measured and not used: a wave's next item
// and step read ahead (n = 120: 22.6 -> 22.4 us of the launch), row offsets formed by an
// unrolled pass over the bits instead of a loop over each mask (26.1).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "fuse.hpp"
#include "kernels.hpp"
#include "launch.hpp"

namespace tn {

namespace {

constexpr int kFuseThreads = 512;

struct FuseArgs {
    const uint8_t* blob;
    void* arena;
    int64_t stride;      // entries between the planes' arenas
    uint64_t* res;
    uint32_t prog_end;   // blob offset of the initial entries
    uint32_t p[kMaxGroup], r2[kMaxGroup], r16[kMaxGroup];
    float pinv[kMaxGroup];
};

// Bits of x at the set bits of a wave-uniform mask, gathered.
__device__ __forceinline__ uint32_t pext16(uint32_t x, uint32_t mask) {
    uint32_t r = 0, k = 0;
    while (mask) {
        const uint32_t pos = uint32_t(__builtin_ctz(mask));
        r |= ((x >> pos) & 1u) << k;
        ++k;
        mask &= mask - 1;
    }
    return r;
}

typedef int v4i __attribute__((ext_vector_type(4)));

// Sum of n products of consecutive entries: n is 1, 2 or a multiple of 4,
// rows of at least 16 bytes start 16-byte aligned.
__device__ __forceinline__ int32_t dot_lds(const int8_t* a, const int8_t* b, int n) {
    int32_t acc = 0;
    if (n >= 16) {
        const v4i *va = reinterpret_cast<const v4i*>(a), *vb = reinterpret_cast<const v4i*>(b);
        for (int z = 0; z < n / 16; ++z) {
            const v4i x = va[z], y = vb[z];
            acc = __builtin_amdgcn_sdot4(x[0], y[0], acc, false);
            acc = __builtin_amdgcn_sdot4(x[1], y[1], acc, false);
            acc = __builtin_amdgcn_sdot4(x[2], y[2], acc, false);
            acc = __builtin_amdgcn_sdot4(x[3], y[3], acc, false);
        }
    } else if (n >= 4) {
        const int *va = reinterpret_cast<const int*>(a), *vb = reinterpret_cast<const int*>(b);
        for (int z = 0; z < n / 4; ++z) acc = __builtin_amdgcn_sdot4(va[z], vb[z], acc, false);
    } else {
        acc = int32_t(a[0]) * b[0];
        if (n == 2) acc += int32_t(a[1]) * b[1];
    }
    return acc;
}

// Residues below 2^16: every product is below 2^32, so 2^32 of them fit the
// 64-bit sum unreduced.
__device__ __forceinline__ uint64_t dot_lds(const uint32_t* a, const uint32_t* b, int n) {
    uint64_t acc = 0;
    if (n >= 4) {
        for (int z = 0; z < n; z += 4) {
            const uint4 x = *reinterpret_cast<const uint4*>(a + z), y = *reinterpret_cast<const uint4*>(b + z);
            acc += uint64_t(x.x) * y.x;
            acc += uint64_t(x.y) * y.y;
            acc += uint64_t(x.z) * y.z;
            acc += uint64_t(x.w) * y.w;
        }
    } else {
        acc = uint64_t(a[0]) * b[0];
        if (n == 2) acc += uint64_t(a[1]) * b[1];
    }
    return acc;
}

__device__ __forceinline__ uint64_t dot_lds(const uint64_t* a, const uint64_t* b, int n) {
    uint64_t acc = 0;
    if (n >= 2) {
        for (int z = 0; z < n; z += 2) {
            const ulonglong2 x = *reinterpret_cast<const ulonglong2*>(a + z),
                             y = *reinterpret_cast<const ulonglong2*>(b + z);
            acc += x.x * y.x;
            acc += x.y * y.y;
        }
    } else {
        acc = a[0] * b[0];
    }
    return acc;
}

// Program ``prog`` of a blob in one residue plane (arena: the plane's; res: the
// plane's result). WIDE: the initial entries are 32-bit words to be reduced
// modulo the plane's modulus (else bytes, valid residues in every plane).
template <int E, bool WIDE>
__device__ __forceinline__ void run_program(uint8_t* lds, const uint8_t* blob, uint32_t prog, uint32_t prog_end,
                                            typename ElemT<E>::T* arena, uint64_t* res, const ModSmall& ms) {
    using T = typename ElemT<E>::T;
    T* const mem = reinterpret_cast<T*>(lds);
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const FuseProg pg = reinterpret_cast<const FuseProg*>(blob)[prog];
    const uint32_t p = uint32_t(ms.m);
    const ModP mp{p, ms.r32};
    uint8_t* const lprog = lds + (pg.lds_elems * uint32_t(sizeof(T)) + 15) / 16 * 16;
    // the program and the initial tensors into LDS
    {
        const uint4* src = reinterpret_cast<const uint4*>(blob + pg.prog);
        uint4* dst = reinterpret_cast<uint4*>(lprog);
        for (uint32_t i = uint32_t(tid); i < pg.prog_bytes / 16; i += kFuseThreads) dst[i] = src[i];
        const uint8_t* e0 = blob + prog_end;
        for (uint32_t i = uint32_t(tid); i < pg.n_init; i += kFuseThreads) {
            if constexpr (WIDE) {
                const uint32_t v = reinterpret_cast<const uint32_t*>(e0)[pg.init + i];
                if constexpr (E == EL_U64) {
                    mem[i] = v;
                } else if constexpr (E == EL_U32) {
                    mem[i] = v % p;
                } else {
                    const int32_t r = int32_t(v % p);
                    mem[i] = T(r > int32_t(p >> 1) ? r - int32_t(p) : r);
                }
            } else {
                mem[i] = T(e0[pg.init + i]);
            }
        }
    }
    __syncthreads();
    const uint4* steps = reinterpret_cast<const uint4*>(lprog);
    const uint32_t* items = reinterpret_cast<const uint32_t*>(lprog + pg.n_steps * 16);
    const uint32_t* levels = items + pg.n_items;
    uint32_t i0 = 0;
    for (uint32_t L = 0; L < pg.n_levels; ++L) {
        const uint32_t i1 = uint32_t(__builtin_amdgcn_readfirstlane(int(levels[L + 1])));
        for (uint32_t i = i0 + uint32_t(w); i < i1; i += kFuseThreads / 64) {
            const uint32_t word = uint32_t(__builtin_amdgcn_readfirstlane(int(items[i])));
            const uint4 d = steps[word & 0xffffu];
            const uint32_t offA = uint32_t(__builtin_amdgcn_readfirstlane(int(d.x)));
            const uint32_t offB = uint32_t(__builtin_amdgcn_readfirstlane(int(d.y)));
            const uint32_t offC = uint32_t(__builtin_amdgcn_readfirstlane(int(d.z)));
            const uint32_t mw = uint32_t(__builtin_amdgcn_readfirstlane(int(d.w)));
            const uint32_t maskA = mw & 0xffffu, s = (mw >> 16) & 0xffu, rC = (mw >> 24) & 0x7fu;
            const uint32_t maskB = ((1u << rC) - 1) & ~maskA;
            // fewer than 64 outputs: the spare lanes take parts of K
            const uint32_t lo = rC < 6 ? rC : 6;
            const uint32_t sp = min(6 - lo, s > 4 ? s - 4 : 0u);
            const uint32_t c = (word >> 16) * 64 + (uint32_t(lane) & ((1u << lo) - 1));
            const uint32_t part = uint32_t(lane) >> lo;
            const int len = 1 << (s - sp);
            const uint32_t z0 = part << (s - sp);
            const bool live = part < (1u << sp);
            const T* ra = mem + offA + (pext16(c, maskA) << s) + z0;
            const T* rb = mem + offB + (pext16(c, maskB) << s) + z0;
            T out;
            if constexpr (E == EL_I8) {
                int32_t acc = live ? dot_lds(ra, rb, len) : 0;
                for (uint32_t o = lo; o < lo + sp; ++o) acc += __shfl_xor(acc, 1 << o);
                out = T(ms.center32(acc));
            } else {
                uint64_t acc = live ? dot_lds(ra, rb, len) : 0;
                for (uint32_t o = lo; o < lo + sp; ++o) acc += __shfl_xor(acc, 1 << o);
                if constexpr (E == EL_U64)
                    out = acc;
                else
                    out = mp.finish(acc);
            }
            if (part == 0) {
                if (!(mw & (kFuseRoot << 16)))
                    mem[offC + c] = out;
                else if (pg.final)
                    *res = uint64_t(int64_t(out));
                else
                    arena[pg.root_off + c] = out;
            }
        }
        i0 = i1;
        __syncthreads();
    }
}

// One plan: programs over blockIdx.x, residue planes over blockIdx.y.
template <int E, bool WIDE>
__global__ __launch_bounds__(kFuseThreads) void k_fused(FuseArgs a) {
    extern __shared__ __align__(16) uint8_t lds[];
    const int g = blockIdx.y;
    const ModSmall ms{int32_t(a.p[g]), a.r2[g], a.r16[g], a.pinv[g]};
    run_program<E, WIDE>(lds, a.blob, blockIdx.x, a.prog_end,
                         static_cast<typename ElemT<E>::T*>(a.arena) + g * a.stride, a.res + g, ms);
}

// Many plans: one (plane, program) pair per work-group.
template <int E>
__global__ __launch_bounds__(kFuseThreads) void k_fused_many(const FusePlane* planes, const uint2* work) {
    extern __shared__ __align__(16) uint8_t lds[];
    const uint2 wk = work[blockIdx.x];
    const FusePlane pl = planes[wk.x];
    const ModSmall ms{int32_t(pl.p), pl.r2, pl.r16, pl.pinv};
    run_program<E, false>(lds, pl.blob, wk.y, pl.prog_end, static_cast<typename ElemT<E>::T*>(pl.arena), pl.res, ms);
}

template <int E>
__global__ __launch_bounds__(64) void k_result(const void* arena, int64_t stride, int64_t off, uint64_t* res, int G) {
    using T = typename ElemT<E>::T;
    const int g = threadIdx.x;
    if (g < G) res[g] = uint64_t(int64_t((static_cast<const T*>(arena) + g * stride)[off]));
}

__global__ __launch_bounds__(256) void k_upload(const uint4* src, uint4* dst, int64_t n16) {
    for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < n16; i += int64_t(gridDim.x) * 256) dst[i] = src[i];
}

template <int E>
hipError_t launch_el(const FuseArgs& a, bool wide, dim3 grid, uint32_t lds, hipStream_t stream) {
    if (wide)
        hipLaunchKernelGGL((k_fused<E, true>), grid, dim3(kFuseThreads), lds, stream, a);
    else
        hipLaunchKernelGGL((k_fused<E, false>), grid, dim3(kFuseThreads), lds, stream, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_fused(const Exec& ex, int el, const uint32_t* primes, int G, const void* d_blob, bool wide,
                        char* arena_base, int64_t arena_elems, uint64_t* res, hipStream_t stream) {
    FuseArgs a{};
    a.blob = static_cast<const uint8_t*>(d_blob);
    a.arena = arena_base;
    a.stride = arena_elems;
    a.res = res;
    a.prog_end = ex.prog_end;
    StepArgs m{};
    fill_moduli(m, primes, G);
    std::copy(m.p, m.p + G, a.p);
    std::copy(m.r2, m.r2 + G, a.r2);
    std::copy(m.r16, m.r16 + G, a.r16);
    std::copy(m.pinv, m.pinv + G, a.pinv);
    const uint32_t lds = ex.lds_bytes;
    const dim3 grid(uint32_t(ex.progs.size()), uint32_t(G), 1);
    return el == EL_U64  ? launch_el<EL_U64>(a, wide, grid, lds, stream)
           : el == EL_I8 ? launch_el<EL_I8>(a, wide, grid, lds, stream)
                         : launch_el<EL_U32>(a, wide, grid, lds, stream);
}

hipError_t launch_fused_many(int el, const FusePlane* planes, const void* work, int64_t n, uint32_t lds,
                             hipStream_t stream) {
    const dim3 grid(static_cast<uint32_t>(n));
    const uint2* w = static_cast<const uint2*>(work);
    if (el == EL_U64)
        hipLaunchKernelGGL(k_fused_many<EL_U64>, grid, dim3(kFuseThreads), lds, stream, planes, w);
    else if (el == EL_I8)
        hipLaunchKernelGGL(k_fused_many<EL_I8>, grid, dim3(kFuseThreads), lds, stream, planes, w);
    else
        hipLaunchKernelGGL(k_fused_many<EL_U32>, grid, dim3(kFuseThreads), lds, stream, planes, w);
    return hipGetLastError();
}

hipError_t launch_gather(int el, int G, const char* arena_base, int64_t arena_elems, int64_t off, uint64_t* res,
                         hipStream_t stream) {
    if (el == EL_U64)
        hipLaunchKernelGGL(k_result<EL_U64>, dim3(1), dim3(64), 0, stream, arena_base, arena_elems, off, res, G);
    else if (el == EL_I8)
        hipLaunchKernelGGL(k_result<EL_I8>, dim3(1), dim3(64), 0, stream, arena_base, arena_elems, off, res, G);
    else
        hipLaunchKernelGGL(k_result<EL_U32>, dim3(1), dim3(64), 0, stream, arena_base, arena_elems, off, res, G);
    return hipGetLastError();
}

hipError_t launch_upload(const void* src, void* dst, int64_t n16, hipStream_t stream) {
    hipLaunchKernelGGL(k_upload, dim3(uint32_t(std::min<int64_t>((n16 + 255) / 256, 256))), dim3(256), 0, stream,
                       static_cast<const uint4*>(src), static_cast<uint4*>(dst), n16);
    return hipGetLastError();
}

}  // namespace tn
