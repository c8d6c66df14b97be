// Narrow dense steps on the matrix cores for residues modulo 16-bit primes
// (u32 words): C[xA, j] = sum_z A[z | xA] B[z | j] with few B rows (2^fB <= 64)
// and a shared dimension of at least 64 entries.
//
// Such a step is bound by reading its operands once. The wave-per-output
// kernel (k_rowdot) reads A once per B row: rank 21 x 22, K = 2^16, 6 planes took
// 785 us for 150 MB. Here a wave takes a block of A rows, every B row and a
// range of K, reads its rows straight into registers (four lanes 64 consecutive
// bytes of a row per instruction, 256 per chunk), splits every residue into two centred
// base-256 digits there and runs the four digit products on
// v_mfma_i32_16x16x64_i8, whose sums stay exact for 2^15 entries (as in
// mfma.hip). Partial residues of the K ranges go to scratch and are added by a
// second kernel. 61 us for the step above (2.5 TB/s), and a step of 2^5 outputs over
// K = 2^10 in 16 planes 12 us (split-K dot: 33 us).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "kernels.hpp"
#include "mfma.hpp"
#include "profile.hpp"

namespace tn {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

constexpr int kRange = 1 << 15;   // entries summed exactly in int32
constexpr int kWavesPerGroup = 4;

// The digits of a lane's 16 residues: word k holds those of its k-th load (A and B
// lanes hold the same entries of K, in whatever order). A residue
// r is centred, c = r - p where r > p / 2 (|c| <= 32639); its digits are c's low
// byte, signed, and (c + 128) >> 8, the second byte of c + 128.
struct Digits {
    v4i d0, d1;
};
__device__ __forceinline__ Digits digits_of(const v4u (&r)[4], uint32_t p) {
    const int32_t half = int32_t(p >> 1);
    Digits out;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        uint32_t c[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) c[e] = r[k][e] - (uint32_t((half - int32_t(r[k][e])) >> 31) & p);
        const uint32_t lo0 = __builtin_amdgcn_perm(c[1], c[0], 0x0c0c0400u);
        const uint32_t lo1 = __builtin_amdgcn_perm(c[3], c[2], 0x0c0c0400u);
        out.d0[k] = int32_t(__builtin_amdgcn_perm(lo1, lo0, 0x05040100u));
#pragma unroll
        for (int e = 0; e < 4; ++e) c[e] += 128u;
        const uint32_t hi0 = __builtin_amdgcn_perm(c[1], c[0], 0x0c0c0501u);
        const uint32_t hi1 = __builtin_amdgcn_perm(c[3], c[2], 0x0c0c0501u);
        out.d1[k] = int32_t(__builtin_amdgcn_perm(hi1, hi0, 0x05040100u));
    }
    return out;
}

// X = T0 + 2^8 T1 + 2^16 T2 (|T_t| <= 2^30, an integer below 2^47) modulo p in
// double precision, where every step is exact (inv_p: the double nearest 1 / p).
__device__ __forceinline__ uint32_t combine(int32_t t0, int32_t t1, int32_t t2, uint32_t p, double inv_p) {
    const double x = fma(double(t2), 65536.0, fma(double(t1), 256.0, double(t0)));
    const double q = floor(x * inv_p);
    int32_t r = int32_t(fma(-q, double(p), x));
    r += r < 0 ? int32_t(p) : 0;
    r -= r >= int32_t(p) ? int32_t(p) : 0;
    return uint32_t(r);
}

// RB x CB blocks of 16 x 16 outputs per wave. Wave (tile, range): A rows
// 16 RB tile.., K entries `len` of range; rows beyond the operands' read the
// last row and are not stored. part: partial residues [range][xA][j] when there
// are several ranges.
template <int RB, int CB>
__global__ __launch_bounds__(64 * kWavesPerGroup) void k_narrow32(StepArgs a, uint32_t tiles, uint32_t ranges,
                                                                  uint32_t* part, int64_t part_stride) {
    const int g = blockIdx.z;
    const uint32_t* A = static_cast<const uint32_t*>(a.A) + g * a.strideA;
    const uint32_t* B = static_cast<const uint32_t*>(a.B) + g * a.strideB;
    uint32_t* C = static_cast<uint32_t*>(a.C) + g * a.strideC;
    const uint32_t p = a.p[g];
    const double inv_p = 1.0 / double(p);
    const int lane = threadIdx.x & 63, fr = lane & 15, q = lane >> 4;
    const uint32_t wave =
        blockIdx.x * kWavesPerGroup + uint32_t(__builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)));
    const uint32_t tile = wave % tiles, range = wave / tiles;
    if (range >= ranges) return;
    const uint64_t K = uint64_t(1) << a.s, len = K / ranges;
    const uint64_t rowsA = uint64_t(1) << a.fA;
    const int nB = 1 << a.fB;
    const uint64_t row0 = uint64_t(tile) * (16 * RB);
    const uint64_t kofs = uint64_t(range) * len + uint64_t(4 * q);
    const uint32_t* pa[RB];
    const uint32_t* pb[CB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) pa[rb] = A + min(row0 + uint64_t(16 * rb + fr), rowsA - 1) * K + kofs;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) pb[cb] = B + uint64_t(min(16 * cb + fr, nB - 1)) * K + kofs;
    v4i acc[3][RB][CB];
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) acc[t][rb][cb] = v4i{0, 0, 0, 0};
    v4u ra[RB][4], rbuf[CB][4];
    const auto load = [&](uint64_t z) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int k = 0; k < 4; ++k) ra[rb][k] = *reinterpret_cast<const v4u*>(pa[rb] + z + 16 * k);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int k = 0; k < 4; ++k) rbuf[cb][k] = *reinterpret_cast<const v4u*>(pb[cb] + z + 16 * k);
    };
    load(0);
    for (uint64_t z = 0; z < len; z += 64) {
        Digits da[RB], db[CB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) da[rb] = digits_of(ra[rb], p);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) db[cb] = digits_of(rbuf[cb], p);
        // the next chunk is requested before this one's products
        if (z + 64 < len) load(z + 64);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                acc[0][rb][cb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(da[rb].d0, db[cb].d0, acc[0][rb][cb], 0, 0, 0);
                acc[1][rb][cb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(da[rb].d0, db[cb].d1, acc[1][rb][cb], 0, 0, 0);
                acc[1][rb][cb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(da[rb].d1, db[cb].d0, acc[1][rb][cb], 0, 0, 0);
                acc[2][rb][cb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(da[rb].d1, db[cb].d1, acc[2][rb][cb], 0, 0, 0);
            }
        if (((z + 64) & (kRange - 1)) == 0 && z + 64 < len) {
            // T0 takes the residue (below 2^16), the others restart: the next
            // range keeps every sum below 2^30 + 2^16
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        acc[0][rb][cb][v] = int32_t(
                            combine(acc[0][rb][cb][v], acc[1][rb][cb][v], acc[2][rb][cb][v], p, inv_p));
                        acc[1][rb][cb][v] = acc[2][rb][cb][v] = 0;
                    }
        }
    }
    // lane holds A rows row0 + 16 rb + 4 q + v, B row 16 cb + fr
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const uint64_t xa = row0 + uint64_t(16 * rb + 4 * q + v);
            if (xa >= rowsA) continue;
            const uint64_t cA = ranges > 1 ? 0 : pdep64(xa, a.maskA);
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                const int j = 16 * cb + fr;
                if (j >= nB) continue;
                const uint32_t r = combine(acc[0][rb][cb][v], acc[1][rb][cb][v], acc[2][rb][cb][v], p, inv_p);
                if (ranges > 1)
                    part[g * part_stride + ((int64_t(range) << (a.fA + a.fB)) + (int64_t(xa) << a.fB)) + j] = r;
                else
                    C[cA | pdep64(uint64_t(j), a.maskB)] = r;
            }
        }
}

// adds the ranges' partial residues: a group of 4 waves per 64 outputs, each
// wave a quarter of the ranges
__global__ __launch_bounds__(256) void k_narrow32_reduce(StepArgs a, const uint32_t* part, int64_t part_stride,
                                                         uint32_t ranges) {
    __shared__ uint32_t red[4][64];
    const int g = blockIdx.z;
    uint32_t* C = static_cast<uint32_t*>(a.C) + g * a.strideC;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint64_t n = uint64_t(1) << (a.fA + a.fB);
    const uint64_t e = uint64_t(blockIdx.x) * 64 + lane;
    const uint32_t* p0 = part + g * part_stride + e;
    uint32_t sum = 0;  // at most 2^12 residues below 2^16
    if (e < n) {
#pragma unroll 4
        for (uint32_t k = uint32_t(w); k < ranges; k += 4) sum += p0[uint64_t(k) * n];
    }
    red[w][lane] = sum;
    __syncthreads();
    if (w != 0 || e >= n) return;
    const uint32_t r = (red[0][lane] + red[1][lane] + red[2][lane] + red[3][lane]) % a.p[g];
    const uint64_t xa = e >> a.fB, j = e & ((uint64_t(1) << a.fB) - 1);
    C[pdep64(xa, a.maskA) | pdep64(j, a.maskB)] = r;
}

template <int RB, int CB>
hipError_t launch_cb(const StepArgs& a, int G, hipStream_t stream, char* scratch, int64_t scratch_per_plane) {
    const uint64_t tiles = ((uint64_t(1) << a.fA) + 16 * RB - 1) / (16 * RB);
    const uint64_t outs = uint64_t(1) << (a.fA + a.fB), K = uint64_t(1) << a.s;
    // K in ranges until there are about 4096 waves, each with at least two
    // chunks, the partial residues fitting the scratch area
    uint64_t ranges = 1;
    while (tiles * uint64_t(G) * ranges < 4096 && K / (2 * ranges) >= 128 && ranges < 4096 &&
           outs * ranges * 2 * 4 <= uint64_t(scratch_per_plane))
        ranges *= 2;
    uint32_t* part = reinterpret_cast<uint32_t*>(scratch);
    const dim3 grid(uint32_t((tiles * ranges + kWavesPerGroup - 1) / kWavesPerGroup), 1, uint32_t(G));
    hipLaunchKernelGGL((k_narrow32<RB, CB>), grid, dim3(64 * kWavesPerGroup), 0, stream, a, uint32_t(tiles),
                       uint32_t(ranges), part, scratch_per_plane / 4);
    if (ranges > 1)
        hipLaunchKernelGGL(k_narrow32_reduce, dim3(uint32_t((outs + 63) / 64), 1, uint32_t(G)), dim3(256), 0, stream, a,
                           part, scratch_per_plane / 4, uint32_t(ranges));
    return hipGetLastError();
}

}  // namespace

bool narrow32_eligible(const StepArgs& a) {
    // the shapes the tiled kernel does not take: B side of at most 64 rows
    // (with 64, fewer than 128 A rows); A row tiles in 32 bits. Up to four outputs over
    // K >= 2^10 stay the split-K dot's: it sums them by whole lines of both operands,
    // while a tile here would be at least three quarters padding.
    return a.s >= 6 && a.s <= 32 && a.fA >= a.fB && a.fA <= 32 && (a.fB <= 5 || (a.fB == 6 && a.fA < 7)) &&
           !(a.fA + a.fB <= 2 && a.s >= 10);
}

hipError_t launch_narrow32(const StepArgs& a, int G, hipStream_t stream, Profiler* prof, double step_bytes,
                           double step_macs, char* scratch, int64_t scratch_per_plane) {
    if (!narrow32_eligible(a)) return hipErrorInvalidValue;
    prof->before(stream);
    const hipError_t e = a.fB <= 4   ? launch_cb<4, 1>(a, G, stream, scratch, scratch_per_plane)
                         : a.fB == 5 ? launch_cb<4, 2>(a, G, stream, scratch, scratch_per_plane)
                                     : launch_cb<2, 4>(a, G, stream, scratch, scratch_per_plane);
    prof->after_raw(stream, KC_NARROW, step_bytes, step_macs);
    return e;
}

}  // namespace tn
