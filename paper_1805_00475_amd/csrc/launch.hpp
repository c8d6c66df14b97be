// Step launcher and initial-tensor helpers shared by the single-instance
// and the batched contraction paths.
#pragma once

#include <hip/hip_runtime.h>

#include <vector>

#include "fuse.hpp"
#include "internal.hpp"
#include "kernels.hpp"
#include "profile.hpp"

namespace tn {

// scratch per prime: partial sums of the split-K dot kernels (1024 blocks x
// 64 outputs x 8 B) and of split-K matrix-core steps (up to 2^20 residues)
constexpr int kDotBlocks = 1024;
constexpr int64_t kScratchPerPrime = int64_t(1) << 22;

int64_t align256(int64_t b);

// Chooses and launches the kernel(s) of one step for G residue planes (or
// the single 64-bit plane). Operands that are initial tensors live in the
// init region (shared by all planes); the others in the plane's arena.
// force >= 0 selects a kernel class (test hook). dig: bit 0 / bit 1 = operand
// A / B of the plan's step is already held as digit planes (see mfma.hip),
// bit 2 = write the output as digit planes (only the matrix-core kernel
// does; the caller sets it only where choose_class says so for this step
// and for the output's consumer).
hipError_t launch_step(const Step& st, int el, int flags, const uint32_t* primes, int G, char* init_base,
                       char* arena_base, int64_t arena_elems, char* scratch, hipStream_t stream, KernelClass* kc,
                       int force = -1, unsigned dig = 0, int64_t init_stride = 0);

// The kernel class launch_step picks for a step (no launch, force < 0).
KernelClass choose_class(const Step& st, int el, int flags);

// Digit-plane hand-over between matrix-core steps: for every step, the dig
// bits of launch_step, given the class each step runs with. A tensor is
// written as digit planes when its producer and its consumer both run the
// matrix-core kernel, which then skips the digit pass on it.
std::vector<uint8_t> digit_plan(const std::vector<Step>& steps, size_t n_ids, const std::vector<KernelClass>& cls,
                                int el);

// Bytes per entry of an element kind (EL_U32, EL_U64, EL_I8 of kernels.hpp).
int elem_size(int el);
// Moduli and their reduction constants of G residue planes.
void fill_moduli(StepArgs& a, const uint32_t* primes, int G);

// Runs an Exec's programs (blob at d_blob, in device memory) for G residue
// planes: roots go to the arena, the network's scalar, when it is one of the
// roots, to res[plane] (int8 residues sign-extended).
hipError_t launch_fused(const Exec& ex, int el, const uint32_t* primes, int G, const void* d_blob, bool wide,
                        char* arena_base, int64_t arena_elems, uint64_t* res, hipStream_t stream);
// One residue plane of one of many plans, in device memory.
struct FusePlane {
    const uint8_t* blob;
    void* arena;
    uint64_t* res;
    uint32_t prog_end, p, r2, r16;
    float pinv;
    uint32_t pad;
};
// Programs of many plans of one element kind: n work-groups, work[i] = (index
// into planes, program), all in device memory; lds: what the largest needs.
hipError_t launch_fused_many(int el, const FusePlane* planes, const void* work, int64_t n, uint32_t lds,
                             hipStream_t stream);
// res[g] = entry off of plane g
hipError_t launch_gather(int el, int G, const char* arena_base, int64_t arena_elems, int64_t off, uint64_t* res,
                         hipStream_t stream);
// dst = src, n16 blocks of 16 bytes (src may be pinned host memory)
hipError_t launch_upload(const void* src, void* dst, int64_t n16, hipStream_t stream);

// The streaming kernel with 2^nb B rows per thread (autotuner launches).
hipError_t launch_stream_step(const StepArgs& a, int el, int G, int nb, hipStream_t st);

// Writes the initial tensors ids at the entry offsets off, in plan layout
// (reduced modulo *mod when given).
void fill_init(const Network& net, const Plan& plan, const std::vector<int32_t>& ids,
               const std::vector<int64_t>& off, int el, uint8_t* host, const uint32_t* mod = nullptr);

}  // namespace tn
