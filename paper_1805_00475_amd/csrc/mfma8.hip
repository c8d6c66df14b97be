// Dense contraction steps on the matrix cores for residues modulo small
// moduli (m <= 255), stored as centred int8 values (|r| <= 127).
//
// A step C = A B^T (rows of A and B contiguous along the shared bonds, Sec.
// 2.1 / Eq. 5 in the plan's layout) is an int8 matrix product: every
// product of two residues is at most 127^2 < 2^14 in magnitude, so
// v_mfma_i32_16x16x64_i8 sums 2^16 of them exactly in int32 (< 2^30); wider
// K is reduced to a centred residue every 2^16 entries. The epilogue reduces
// each sum modulo m (ModSmall) and stores the int8 residue, which the next
// step reads as it is: no digit pass and one product per multiply-add.
//
// Work-group tile WM (xA) x WN (xB) with waves of 16 RA x 16 CB outputs:
// 8 waves (two per SIMD) on 256 x 256 tiles when both free sides have 8
// bits, else 256 x 128 or 128 x 128; 4 waves on 256 x 64 or 128 x 64 tiles
// when B's free side has 6 bits (those steps stream A at the memory rate).
//
// K goes in stages of 128 entries: 128-byte LDS rows, whole lines of memory,
// filled straight from it (global_load_lds_dwordx4, 8 rows per wave
// instruction). A stage is two steps of 64 entries; while a step's products
// run, the wave reads the next step's fragments, and one barrier per stage,
// before its second step, makes the next stage visible and frees this one's
// buffers. A has three buffers and B two: B's stage k+2 and A's stage k+3 are
// requested at that barrier, two and four steps before they are read (A's
// rows are the ones that come from beyond the L2 most often). At a tile's
// last step (every fragment in registers) the next tile's first two stages
// are requested; A's third buffer takes the outputs on their way to memory.
//
// With 64-byte stages (four buffers of 32 KiB, the same bytes in flight) the
// loads bound the kernel: a line left the L1 before its second half was
// asked for, and one CU took in 19 bytes per clock. 256 x 256 tiles, K = 2^13:
// 2013 us, 1418 with the loads left out, 1814 now.
//
// LDS rows: 8 slots of 16 bytes, slot c of row r stored at slot c ^ (r % 8).
// A 16-byte read is served eight lanes at a time, and eight lanes free of
// bank conflicts cover 128 distinct bytes modulo 128: a fragment read has
// eight consecutive lanes on eight consecutive rows at one logical slot, which
// the XOR sends to eight distinct slots. (K = 64: 64-byte rows, slot c at
// c ^ ((r / 2) % 4), rows of one parity lying 128 bytes apart.)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "kernels.hpp"
#include "mfma.hpp"
#include "mfma_common.hpp"
#include "profile.hpp"
#include "tune.hpp"

namespace tn {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int k8Flush = (1 << 16) / 128;   // stages per exact int32 range
constexpr int k8MaxRowBytesLog = 25;       // 127 rows of a stage within 32-bit load offsets

// Output addressing of the epilogue, by the host. A lane holds, per 16 x 16
// block, four outputs: A indices v = 0..3 (A's two lowest bits) at one B
// index. mode 0: those are C's two lowest bits, so the four are consecutive
// bytes; mode 1: C's two lowest bits are A's lowest and B's lowest (either
// order), so a lane and its neighbour (B indices differing in the lowest bit)
// swap halves and each holds 4 consecutive bytes, the even lane those of v < 2
// and the odd lane those of v >= 2; sel are the byte selectors of that swap
// (even, odd lane); mode 2 (both are B's): single bytes, at the C offset bits
// dA, dV, dB of the tile-local A indices 16 rb and v and of the B indices
// 16 cb.
//
// In modes 0 and 1 (other tiles are launched with the operands exchanged where
// that gives mode 0) a wave's words go through its part of LDS, a piece of at
// most 4 KiB at a time, and leave in C's order: consecutive lanes store
// consecutive 16 bytes wherever C is consecutive (at least 32 bytes, as the
// wave's tile takes the five lowest bits of either side). A word's place is
// the XOR of a part per lane bit (sLane), per A block (sRb) and per B block
// (sCb): the C-ordered index of the piece's bits, with the low four bits of
// the 16-byte chunk index XORed by a map M of the higher ones chosen so that
// a wave's 64 words fall into 64 banks. Chunk t 64 + lane is read at
// 16 lane ^ rM.. ^ rT[t] and stored at C offset bits cLane.. | cT[t].
struct Mfma8Extra {
    uint64_t hiA, hiB;  // masks of the tile indices: maskA, maskB less the tile's own bits
    uint64_t dA[8], dV[4], dB[4];
    uint32_t sel[2];
    int32_t mode;
    uint32_t sLane[6], sRb[8], sCb[4], rM[2], rT[4];
    uint64_t cLane[6], cT[4], cPiece;
};

// How an exact sum x reaches the reduction: RED_BIAS: the accumulator started
// at the bits of 1.5 2^23, so that as a float it is 1.5 2^23 + x (K <= 256,
// |x| <= 256 127^2 < 2^22), RED_PLAIN: as it is (K <= 512, |x| < 2^23), RED_FOLD:
// folded at 2^16 first (|x| < 2^30).
enum Reduce { RED_BIAS, RED_PLAIN, RED_FOLD };
constexpr float kBias = 12582912.0f;          // 1.5 2^23
constexpr int32_t kBiasBits = 0x4b400000;

// Centred residue of an exact int32 sum modulo m <= 255, returned as the low
// byte of a word. With RED_FOLD, x = h 2^16 + l becomes y = h (2^16 mod m) + l
// = x + h ((2^16 mod m) - 2^16) (one 24-bit multiply-add, modulo 2^32),
// |y| < 2^15 (m - 1) + 2^16; else y = x. Either way |y| < 2^23 is exact in
// single precision (RED_BIAS: one subtraction, at half the conversion's
// cycles). One fma adds y fl(1/m) to 1.5 2^23 and rounds the exact sum once:
// with |y fl(1/m)| < 2^22 the result lies where floats are spaced 1 apart, so
// its low 24 bits, read as a signed 24-bit integer, are 2^22 + q, q the nearest
// integer to y fl(1/m) (ties to even). One 24-bit multiply-add gives
// y - m (2^22 + q) = r - 2^22 m with r = y - q m, whose low byte is r's since
// 256 divides 2^22 m (and the bias). |r| <= 127 for every m in 2..255 (checked
// over every reachable y), so that byte is r in two's complement.
template <int RED>
__device__ __forceinline__ uint32_t res8(int32_t x, int32_t r16, int32_t negm, float inv) {
    const int32_t y = RED == RED_FOLD ? __mul24(x >> 16, r16 - 65536) + x : x;
    const float f = RED == RED_BIAS ? __int_as_float(x) - kBias : float(y);
    const float u = __builtin_fmaf(f, inv, kBias);
    return uint32_t(__mul24(int32_t(__float_as_uint(u)), negm) + y);
}

// The low bytes of four words, packed (word 0 in byte 0).
__device__ __forceinline__ uint32_t pack4(uint32_t t0, uint32_t t1, uint32_t t2, uint32_t t3) {
    const uint32_t lo = __builtin_amdgcn_perm(t1, t0, 0x0c0c0400u), hi = __builtin_amdgcn_perm(t3, t2, 0x0c0c0400u);
    return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}

// The lane's word of block (rb, cb) (see Mfma8Extra): four reduced outputs
// packed; with PAIR, half exchanged with the neighbour lane.
template <int RA, int CB, int RED, bool PAIR>
__device__ __forceinline__ uint32_t out_word(const v4i (&acc)[RA][CB], int rb, int cb, const ModSmall& ms,
                                             uint32_t sel) {
    const int32_t negm = -int32_t(ms.m);
    const int32_t r16 = int32_t(ms.r16);
    const uint32_t x =
        pack4(res8<RED>(acc[rb][cb][0], r16, negm, ms.inv), res8<RED>(acc[rb][cb][1], r16, negm, ms.inv),
              res8<RED>(acc[rb][cb][2], r16, negm, ms.inv), res8<RED>(acc[rb][cb][3], r16, negm, ms.inv));
    if constexpr (!PAIR) return x;
    // the neighbour lane's word (quad permutation 1, 0, 3, 2)
    const uint32_t y = uint32_t(__builtin_amdgcn_mov_dpp(int(x), 0xb1, 0xf, 0xf, false));
    return __builtin_amdgcn_perm(x, y, sel);
}

// Bytes of LDS a wave's output piece takes, and pieces of its tile.
template <int RA, int CB>
struct Piece {
    static constexpr int N = RA * CB * 256 > 4096 ? 2 : 1;
    static constexpr int RAP = RA / N;  // A blocks of a piece
    static constexpr int BYTES = RAP * CB * 256;
    static constexpr int NT = BYTES / 1024;  // chunks per lane
};

// Stores a wave's outputs of one tile (modes 0 and 1): base is the C offset of
// the tile and the wave (uniform), st the wave's LDS piece. LDS accesses of a
// wave are served in order, so its pieces need no barrier. (Lane parts are
// formed here, per tile: kept in registers through the K loop they would only
// add pressure.)
template <int RA, int CB, int RED, bool PAIR>
__device__ __forceinline__ void store_staged(const v4i (&acc)[RA][CB], int8_t* C, uint64_t base, const Mfma8Extra& ex,
                                             const ModSmall& ms, int lane, uint8_t* st) {
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    using Pc = Piece<RA, CB>;
    __asm__ volatile("" : "+v"(lane));
    // (a select: indexing the argument array per lane would load it from
    // memory, and that load's wait would also wait for every load and store
    // in flight)
    const uint32_t sel = (lane & 1) ? ex.sel[1] : ex.sel[0];
    uint32_t wl = 0, rl = 16u * uint32_t(lane);
    uint64_t cl = 0;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const bool on = (lane >> k) & 1;
        wl ^= on ? ex.sLane[k] : 0u;
        cl |= on ? ex.cLane[k] : 0ull;
    }
    rl ^= (lane & 16) ? ex.rM[0] : 0u;
    rl ^= (lane & 32) ? ex.rM[1] : 0u;
    int8_t* const out = C + (base | cl);
#pragma unroll
    for (int h = 0; h < Pc::N; ++h) {
#pragma unroll
        for (int rb = 0; rb < Pc::RAP; ++rb) {
            // (through an empty asm statement: all RAP x CB table
            // combinations in scalar registers would spill)
            uint32_t row = wl ^ ex.sRb[rb];
            __asm__ volatile("" : "+v"(row));
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
                *reinterpret_cast<uint32_t*>(st + (row ^ ex.sCb[cb])) =
                    out_word<RA, CB, RED, PAIR>(acc, h * Pc::RAP + rb, cb, ms, sel);
        }
        u4 v[Pc::NT];
#pragma unroll
        for (int t = 0; t < Pc::NT; ++t) v[t] = *reinterpret_cast<const u4*>(st + (rl ^ ex.rT[t]));
#pragma unroll
        for (int t = 0; t < Pc::NT; ++t) *reinterpret_cast<u4*>(out + ((h ? ex.cPiece : 0ull) | ex.cT[t])) = v[t];
    }
}

// Store a wave's outputs of one tile: lane (fr, q) holds acc[rb][cb][v] for
// A index 16 rb + 4 q + v and B index 16 cb + fr (plus the wave's offsets wr,
// wc, whose C offset is part of base).
template <int RA, int CB, int RED>
__device__ __forceinline__ void store_tile8(const v4i (&acc)[RA][CB], int8_t* C, uint64_t base, const StepArgs& a,
                                            const Mfma8Extra& ex, const ModSmall& ms, int lane, uint8_t* st) {
    if (ex.mode == 0) {
        store_staged<RA, CB, RED, false>(acc, C, base, ex, ms, lane, st);
    } else if (ex.mode == 1) {
        store_staged<RA, CB, RED, true>(acc, C, base, ex, ms, lane, st);
    } else {
        const int32_t negm = -int32_t(ms.m);
        const int32_t r16 = int32_t(ms.r16);
        const uint64_t lo = base | pdep64(uint64_t(4 * (lane >> 4)), a.maskA) | pdep64(uint64_t(lane & 15), a.maskB);
        // (row offsets pass through an empty asm statement so that the
        // compiler does not precompute all table combinations in scalar
        // registers, which would spill)
#pragma unroll
        for (int rb = 0; rb < RA; ++rb) {
            uint64_t row = lo | ex.dA[rb];
            __asm__ volatile("" : "+v"(row));
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    C[row | ex.dV[v] | ex.dB[cb]] = int8_t(res8<RED>(acc[rb][cb][v], r16, negm, ms.inv));
        }
    }
}

constexpr int lg2(int x) { return x <= 1 ? 0 : 1 + lg2(x / 2); }

// Tile shape: WM x WN outputs, NW waves, each on 16 RA x 16 CB outputs.
template <int WM_, int WN_, int NW_, int RA_, int CB_>
struct Cfg {
    static constexpr int WM = WM_, WN = WN_, NW = NW_, RA = RA_, CB = CB_;
    static constexpr int THREADS = 64 * NW;
    static constexpr int WAVES_A = WM / (16 * RA);
    static constexpr int LGM = lg2(WM), LGN = lg2(WN);
    static_assert(WAVES_A * (WN / (16 * CB)) == NW, "waves cover the tile");
};
using Cfg256x256 = Cfg<256, 256, 8, 8, 4>;
using Cfg256x128 = Cfg<256, 128, 8, 8, 2>;
using Cfg128x128 = Cfg<128, 128, 8, 4, 2>;
using Cfg256x64 = Cfg<256, 64, 4, 4, 4>;
using Cfg128x64 = Cfg<128, 64, 4, 2, 4>;
// few rows on one side (K <= 32), or 256 of the other held in registers
using Cfg512x16 = Cfg<512, 16, 4, 8, 1>;
using Cfg512x32 = Cfg<512, 32, 4, 8, 2>;
using Cfg64x256 = Cfg<64, 256, 4, 4, 4>;
using Cfg32x256 = Cfg<32, 256, 4, 2, 4>;
using Cfg16x256 = Cfg<16, 256, 4, 1, 4>;

// One step on int8 residues: the tiles of WM x WN outputs of all residue planes
// are dealt round-robin to a grid that fills the GPU once, K split over
// blockIdx.y into `splits` ranges (partial residues to `part` when splits > 1).
// NST: stages of 128 entries per tile and block row: 1, 2, or 4 for any power
// of two >= 4; 0: K = 64.
//
// Loads and stores share one completion counter and complete in order. The
// next tile's first stages are requested before the epilogue's stores (STORES
// per lane), so the waits of its first stage leave that many operations
// outstanding on top; waiting for the stores themselves to reach memory would
// hold every tile up.
template <class G, int NST, int RED>
__global__ __launch_bounds__(G::THREADS, 1) void k_mfma8(StepArgs a, Mfma8Extra ex, int planes, int splits,
                                                         int8_t* part, int64_t part_stride) {
    constexpr int RA = G::RA, CB = G::CB;
    using Pc = Piece<RA, CB>;
    constexpr int STORES = Pc::N * Pc::NT;
    constexpr int ROW = NST ? 128 : 64;               // LDS row bytes
    constexpr int RPI = 1024 / ROW;                   // rows per load instruction
    constexpr int LA = G::WM / (RPI * G::NW), LB = G::WN / (RPI * G::NW);  // loads per wave and stage
    static_assert(LA * RPI * G::NW == G::WM && LB * RPI * G::NW == G::WN, "whole load instructions");
    constexpr int BUFA = G::WM * ROW, BUFB = G::WN * ROW;
    // A's buffers (the last one takes the outputs) and B's
    constexpr int NA = NST >= 2 ? 3 : 2, NB = NST >= 2 ? 2 : 1;
    constexpr int OUTB = G::NW * Pc::BYTES;           // output pieces of the waves
    constexpr int LASTA = OUTB > BUFA ? OUTB : BUFA;
    // (one array for everything: with two, the compiler waits for every load
    // into LDS in flight before each fragment read)
    __shared__ __align__(1024) uint8_t lds[NB * BUFB + (NA - 1) * BUFA + LASTA];
    uint8_t* const ldsA = lds + NB * BUFB;

    const int8_t* const A = static_cast<const int8_t*>(a.A);
    const int8_t* const B = static_cast<const int8_t*>(a.B);
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = (w % G::WAVES_A) * 16 * RA, wc = (w / G::WAVES_A) * 16 * CB;
    const uint64_t rowBytes = uint64_t(1) << a.s;
    const int nst = NST >= 4 ? (1 << (a.s - 7)) / splits : NST;  // stages per tile and block row
    const uint64_t k0 = uint64_t(blockIdx.y) * uint64_t(nst) * 128;
    const int lgA = a.fA - G::LGM, lgB = a.fB - G::LGN;
    const uint32_t T = 1u << (lgA + lgB);
    const uint64_t total = uint64_t(T) * uint64_t(planes);
    if (blockIdx.x >= total) return;
    // outputs leave through the staged stores, STORES per lane and tile
    const bool staged = splits == 1 && ex.mode != 2;

    const int fr = lane & 15, q = lane >> 4;
    const uint64_t waveC = pdep64(uint64_t(wr), a.maskA) | pdep64(uint64_t(wc), a.maskB);
    uint8_t* const wstage = ldsA + (NA - 1) * BUFA + w * Pc::BYTES;
    // loads: lane l of wave w, instruction i fills physical slot l % 8 (4) of
    // stage row r = RPI (NW i + w) + l / 8 (4), i.e. logical slot
    // (l % 8) ^ (r % 8) ((l % 4) ^ ((r / 2) % 4)): 16 bytes of the row
    const uint32_t voff =
        NST ? uint32_t(8 * w + (lane >> 3)) * uint32_t(rowBytes) + 16u * uint32_t((lane & 7) ^ (lane >> 3))
            : uint32_t(16 * w + (lane >> 2)) * uint32_t(rowBytes) + 16u * uint32_t((lane & 3) ^ ((lane >> 3) & 3));
    // fragment reads: row wr + fr of A's buffer, wc + fr of B's, at logical
    // slot q of the stage's first step (its second: physical slot ^ 4)
    const int sw = NST ? 16 * (q ^ (fr & 7)) : 16 * (q ^ ((fr >> 1) & 3));
    const uint32_t rdA = uint32_t((wr + fr) * ROW + sw), rdB = uint32_t((wc + fr) * ROW + sw);

    // The per-lane offsets pass through empty asm statements where they are
    // used, so that addresses are formed there from uniform bases (kept in
    // scalar registers) instead of being kept per lane across the loop.
    auto fetch = [&](const int8_t* t, int stage, uint8_t* dst, auto n) {
        uint32_t vo = voff;
        __asm__ volatile("" : "+v"(vo));
        const int8_t* base = t + (k0 + uint64_t(stage) * 128);
#pragma unroll
        for (int i = 0; i < decltype(n)::value; ++i)
            __builtin_amdgcn_global_load_lds(base + uint64_t(RPI * G::NW * i) * rowBytes + vo,
                                             (lds_ptr_t)(dst + w * 1024 + i * (G::NW * 1024)), 16, 0, 0);
    };
    using nA = std::integral_constant<int, LA>;
    using nB = std::integral_constant<int, LB>;
    v4i fa[RA], b0[CB], b1[CB];
    auto lane_at = [&](uint32_t o, int flip) {
        __asm__ volatile("" : "+v"(o));
        return o ^ uint32_t(flip);
    };
    auto read_b = [&](const uint8_t* p, v4i(&b)[CB]) {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) b[cb] = *reinterpret_cast<const v4i*>(p + cb * 16 * ROW);
    };

    // tile L of plane g = L / T: its coordinates and first rows
    const auto locate = [&](uint64_t L, uint32_t& g, uint32_t& ta, uint32_t& tb, const int8_t*& pA, const int8_t*& pB) {
        g = uint32_t(L >> (lgA + lgB));
        tile_coords_lg(uint32_t(L) & (T - 1), lgA, lgB, ta, tb);
        pA = A + g * a.strideA + uint64_t(ta) * G::WM * rowBytes;
        pB = B + g * a.strideB + uint64_t(tb) * G::WN * rowBytes;
    };
    // a tile's first stage, and its second
    const auto fetch_first = [&](const int8_t* pA, const int8_t* pB) {
        fetch(pA, 0, ldsA, nA());
        fetch(pB, 0, lds, nB());
        if constexpr (NST >= 2) {
            fetch(pA, 1, ldsA + BUFA, nA());
            fetch(pB, 1, lds + BUFB, nB());
        }
    };
    uint64_t L = blockIdx.x;
    uint32_t g, ta, tb;
    const int8_t *tA, *tB;
    locate(L, g, ta, tb, tA, tB);
    fetch_first(tA, tB);
    // (the first tile follows no stores)
    __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0(0));

    for (;;) {
        v4i acc[RA][CB];
        // stage 0 has landed and is visible to all waves. A fragments: one set,
        // each refilled with the next step's as soon as its last product of
        // the step is issued; B fragments: two sets
        if (staged)
            chunk_barrier<(NST >= 2 ? LA + LB : 0) + STORES>();
        else
            chunk_barrier<0>();
        {
            const uint8_t* pa = ldsA + lane_at(rdA, 0);
#pragma unroll
            for (int rb = 0; rb < RA; ++rb) fa[rb] = *reinterpret_cast<const v4i*>(pa + rb * 16 * ROW);
            read_b(lds + lane_at(rdB, 0), b0);
        }

        const uint64_t next = L + gridDim.x;
        const bool more = next < total;
        uint32_t ng = 0, nta = 0, ntb = 0;
        const int8_t *nxA = A, *nxB = B;
        if (more) locate(next, ng, nta, ntb, nxA, nxB);
        // The products of one step from fa and bc (START: the tile's first, onto
        // the bias or zero); meanwhile, with READ, the next step's fragments
        // from pa and pb into fa and bn.
        auto products = [&](v4i(&bc)[CB], v4i(&bn)[CB], const uint8_t* pa, const uint8_t* pb, auto read, auto start) {
            constexpr bool READ = decltype(read)::value, START = decltype(start)::value;
            constexpr int32_t Z = RED == RED_BIAS ? kBiasBits : 0;
            if constexpr (READ) {
                // (the compiler would otherwise wait at the MFMAs for the
                // fragment reads below, to order them after loads in flight)
                __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0(63));
                read_b(pb, bn);
            }
#pragma unroll
            for (int rb = 0; rb < RA; ++rb) {
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
                    acc[rb][cb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(
                        fa[rb], bc[cb], START ? v4i{Z, Z, Z, Z} : acc[rb][cb], 0, 0, 0);
                if constexpr (READ) fa[rb] = *reinterpret_cast<const v4i*>(pa + rb * 16 * ROW);
            }
        };
        using yes = std::true_type;
        using no = std::false_type;
        // first step of a stage in A buffer sa, B buffer sb
        auto first = [&](int sa, int sb, auto start) {
            products(b0, b1, ldsA + sa * BUFA + lane_at(rdA, 64), lds + sb * BUFB + lane_at(rdB, 64), yes(), start);
        };
        // its second step; the next stage is in A buffer na, B buffer nb
        auto second = [&](int na, int nb) {
            products(b1, b0, ldsA + na * BUFA + lane_at(rdA, 0), lds + nb * BUFB + lane_at(rdB, 0), yes(), no());
        };
        // the tile's last step: every fragment is in registers, so the
        // buffers take the next tile's first stages
        auto last = [&](v4i(&bc)[CB], v4i(&bn)[CB], auto start) {
            chunk_barrier<63>();
            if (more) fetch_first(nxA, nxB);
            products(bc, bn, nullptr, nullptr, no(), start);
        };
        const ModSmall ms{int32_t(a.p[g]), a.r2[g], a.r16[g], a.pinv[g]};
        // the tile's C offset, formed while the first products run
        uint64_t baseC = 0;
        const auto place = [&]() { baseC = (pdep_from(ta, ex.hiA) | pdep_from(tb, ex.hiB)) | waveC; };
        if constexpr (NST == 0) {
            last(b0, b1, yes());
            place();
        } else if constexpr (NST == 1) {
            first(0, 0, yes());
            place();
            last(b1, b0, no());
        } else if constexpr (NST == 2) {
            first(0, 0, yes());
            place();
            chunk_barrier<STORES>();  // stage 1 has landed (younger: the last tile's stores)
            second(1, 1);
            first(1, 1, no());
            last(b1, b0, no());
        } else {
            first(0, 0, yes());
            place();
            chunk_barrier<STORES>();
            fetch(tA, 2, ldsA + 2 * BUFA, nA());
            fetch(tB, 2, lds, nB());
            fetch(tA, 3, ldsA, nA());
            second(1, 1);
            // Stage st, in A buffer sa: the barrier waits for stage st + 1
            // (younger: A's stage st + 2). The sums stay exact in int32 for
            // k8Flush stages; after each full range they are reduced to
            // centred residues (the last range ends in the epilogue).
            int st = 1, sa = 1, range = k8Flush;
            while (st + 3 < nst) {
                const int end = std::min(nst - 3, range);
                for (; st < end; ++st) {
                    const int na = sa == 2 ? 0 : sa + 1, sb = st & 1;
                    first(sa, sb, no());
                    chunk_barrier<LA>();
                    fetch(tB, st + 2, lds + sb * BUFB, nB());
                    fetch(tA, st + 3, ldsA + sa * BUFA, nA());
                    second(na, sb ^ 1);
                    sa = na;
                }
                range += k8Flush;
                if (st + 3 < nst) {
#pragma unroll
                    for (int i = 0; i < RA; ++i)
#pragma unroll
                        for (int j = 0; j < CB; ++j)
#pragma unroll
                            for (int v = 0; v < 4; ++v) acc[i][j][v] = ms.center32(acc[i][j][v]);
                }
            }
            // the last three stages (st = nst - 3 is odd)
            int na = sa == 2 ? 0 : sa + 1;
            first(sa, 1, no());
            chunk_barrier<LA>();
            fetch(tB, nst - 1, lds + BUFB, nB());
            second(na, 0);
            sa = na;
            na = sa == 2 ? 0 : sa + 1;
            first(sa, 0, no());
            chunk_barrier<0>();
            second(na, 1);
            first(na, 1, no());
            last(b1, b0, no());
        }

        // epilogue: lane holds A index wr + 16 rb + 4 q + v, B index
        // wc + 16 cb + fr of each 16x16 block
        const int32_t negm = -int32_t(ms.m);
        const int32_t r16 = int32_t(ms.r16);
        auto packed = [&](int rb, int cb) {
            return pack4(res8<RED>(acc[rb][cb][0], r16, negm, ms.inv), res8<RED>(acc[rb][cb][1], r16, negm, ms.inv),
                         res8<RED>(acc[rb][cb][2], r16, negm, ms.inv), res8<RED>(acc[rb][cb][3], r16, negm, ms.inv));
        };
        if (splits > 1) {
            // partial residues of this K range, tile-local order (j, i): the
            // lane's four A indices are consecutive bytes
            int8_t* pt =
                part + g * part_stride + (uint64_t(blockIdx.y) * T + (uint32_t(L) & (T - 1))) * (G::WM * G::WN);
            uint32_t lo = uint32_t((wc + fr) * G::WM + wr + 4 * q);
            __asm__ volatile("" : "+v"(lo));
#pragma unroll
            for (int rb = 0; rb < RA; ++rb)
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
                    *reinterpret_cast<uint32_t*>(pt + lo + uint32_t(16 * cb * G::WM + 16 * rb)) = packed(rb, cb);
        } else {
            store_tile8<RA, CB, RED>(acc, static_cast<int8_t*>(a.C) + g * a.strideC, baseC, a, ex, ms, lane, wstage);
        }
        if (!more) break;
        L = next;
        g = ng;
        ta = nta;
        tb = ntb;
        tA = nxA;
        tB = nxB;
    }
}

// K = 64 CH = 128, 256 or 512 with 256 or more rows on both sides: one side's rows stay
// in registers, the other's stream past. With K this short a tile of k_mfma8
// spends most of its time outside its products, in an epilogue that no
// products run beside (two waves per SIMD, both in the same phase) and in two
// or three barriers: 256 x 256 tiles over K = 256 took 8.7 us, 2.7 of them products.
// Here a work-group of four waves holds 256 resident rows, 64 per wave, as
// fragments (16 CH registers per lane) and walks 2^lgL tiles of 64 streamed rows,
// double-buffered whole in LDS (16 KiB each at K = 256) and shared by its waves.
// Two such work-groups fit a CU (80 KiB each at K = 512; three at K = 128) and run
// freely, so that one's epilogue lies beside another's products. Bound by
// writing C: K = 2^8, rank 26 x 18, 10 planes, 1486 -> 890 us (3.8 TB/s), 31 x 17, 2 planes,
// 4460 -> 3550, 23 x 19, 10 planes, 328 -> 267; K = 2^7: 24 x 17, 8 planes, 403 -> 295 us
// (4.1 TB/s); K = 2^9: 26 x 19, 8 planes, 769 -> 545. Tiles of 128 streamed rows (255
// registers) and three work-groups at K = 256 (168) spilled fragments: 1313 us for
// the first. A third buffer gave nothing.
//
// RES_A: A's rows are resident (256 x 64 tiles), else B's (64 x 256). Items are
// (plane, run of streamed tiles, resident tile); with `spread` the resident
// tiles of one run go to one XCD's work-groups.
constexpr uint32_t kCUs = 256;
// work-groups per CU: 253 registers at K = 512, 193 at K = 256, 157 at K = 128
template <int CH>
constexpr int kRowsPerCU = CH >= 4 ? 2 : 3;
template <class G, bool RES_A, int CH, int RED, bool PAIR>
__global__ __launch_bounds__(G::THREADS, kRowsPerCU<CH>) void k_mfma8_rows(StepArgs a, Mfma8Extra ex,
                                                                            uint32_t items, int lgL, int spread) {
    constexpr int RA = G::RA, CB = G::CB;
    using Pc = Piece<RA, CB>;
    constexpr int STORES = Pc::N * Pc::NT;
    constexpr int ROW = 64 * CH, SLOTS = 4 * CH;  // LDS row bytes, slots of 16 bytes
    constexpr int SW = CH == 8 ? 8 : SLOTS;
    constexpr int NS = 4, NR = 4;                 // streamed and resident blocks of a wave
    static_assert(G::NW == 4 && (RES_A ? CB : RA) == NS && (RES_A ? RA : CB) == NR, "one wave: 64 resident rows");
    constexpr int BUF = 64 * ROW, LD = BUF / 4096;  // loads per wave and tile
    __shared__ __align__(1024) uint8_t lds[2 * BUF + 4 * Pc::BYTES];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fr = lane & 15, q = lane >> 4;
    const int lgS = (RES_A ? a.fB : a.fA) - 6, lgR = (RES_A ? a.fA : a.fB) - 8, lgSeg = lgS - lgL;
    const uint64_t hiS = RES_A ? ex.hiB : ex.hiA, hiR = RES_A ? ex.hiA : ex.hiB;
    const uint64_t oneS = hiS & (~hiS + 1);
    const uint64_t waveC = pdep64(uint64_t(64 * w), RES_A ? a.maskA : a.maskB);
    uint8_t* const wstage = lds + 2 * BUF + w * Pc::BYTES;
    // lane l of wave w, instruction i fills physical slot l % SLOTS of row
    // r = (64 / SLOTS) (4 i + w) + l / SLOTS: logical slot (l % SLOTS) ^ (r % SW) (the
    // work-group's instruction covers a multiple of SW rows: i does not matter)
    constexpr int RPI = 64 / SLOTS;
    const int lr = RPI * w + lane / SLOTS;
    const uint32_t voff = uint32_t(lr * ROW + 16 * ((lane % SLOTS) ^ (lr % SW)));
    // fragment of chunk c: row fr at logical slot 4 c + q, i.e. rd ^ 64 c
    const uint32_t rd = uint32_t(fr * ROW + 16 * (q ^ (fr % SW)));
    constexpr int32_t Z = RED == RED_BIAS ? kBiasBits : 0;
    const uint32_t tiles = 1u << lgL;

    for (uint32_t it = blockIdx.x; it < items; it += gridDim.x) {
        const uint32_t j = spread ? it >> 3 : it;
        const uint32_t r = j & ((1u << lgR) - 1);
        const uint32_t sg = spread ? ((j >> lgR) << 3) | (it & 7) : j >> lgR;
        const uint32_t g = sg >> lgSeg, s0 = (sg & ((1u << lgSeg) - 1)) << lgL;
        const int8_t* const pS = (RES_A ? static_cast<const int8_t*>(a.B) + g * a.strideB
                                        : static_cast<const int8_t*>(a.A) + g * a.strideA) +
                                 uint64_t(s0) * BUF;
        const int8_t* const pR = (RES_A ? static_cast<const int8_t*>(a.A) + g * a.strideA
                                        : static_cast<const int8_t*>(a.B) + g * a.strideB) +
                                 (uint64_t(r) * 256 + uint64_t(64 * w)) * ROW;
        int8_t* const C = static_cast<int8_t*>(a.C) + g * a.strideC;
        const ModSmall ms{int32_t(a.p[g]), a.r2[g], a.r16[g], a.pinv[g]};
        const auto fetch = [&](uint32_t t) {
            uint32_t vo = voff;
            __asm__ volatile("" : "+v"(vo));
            const int8_t* base = pS + uint64_t(t < tiles ? t : tiles - 1) * BUF;
            uint8_t* dst = lds + (t & 1) * BUF + w * 1024;
#pragma unroll
            for (int i = 0; i < LD; ++i)
                __builtin_amdgcn_global_load_lds(base + i * 4096 + vo, (lds_ptr_t)(dst + i * 4096), 16, 0, 0);
        };
        // every wave has read its last fragments of the item before, and the
        // loads behind that run's end have landed
        chunk_barrier<STORES>();
        fetch(0);
        fetch(1);
        v4i res[CH][NR];
        uint32_t ro = uint32_t(fr * ROW + 16 * q);
        __asm__ volatile("" : "+v"(ro));
#pragma unroll
        for (int c = 0; c < CH; ++c)
#pragma unroll
            for (int b = 0; b < NR; ++b) res[c][b] = *reinterpret_cast<const v4i*>(pR + (16 * b * ROW + 64 * c) + ro);
        __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0(0));
        uint64_t depS = pdep_from(s0, hiS);
        const uint64_t baseR = pdep_from(r, hiR) | waveC;
        for (uint32_t t = 0; t < tiles; ++t) {
            // tile t has landed; younger: the stores of tile t - 2, the loads of
            // tile t + 1, the stores of tile t - 1 (fewer operations only behind
            // the drain above, which covers tiles 0 and 1)
            chunk_barrier<LD + 2 * STORES>();
            v4i acc[RA][CB], fs[NS];
            uint32_t at = rd + (t & 1) * uint32_t(BUF);
            __asm__ volatile("" : "+v"(at));
#pragma unroll
            for (int b = 0; b < NS; ++b) fs[b] = *reinterpret_cast<const v4i*>(lds + at + b * 16 * ROW);
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                if (c + 1 < CH)
                    __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0(63));  // as in k_mfma8
                else {
                    // every fragment is in registers: the buffer takes tile
                    // t + 2 (the last tile again behind the run's end, where
                    // the count of operations has to stay the same)
                    chunk_barrier<63>();
                    fetch(t + 2);
                }
                uint32_t nx = rd;
                __asm__ volatile("" : "+v"(nx));
                nx = (nx ^ uint32_t(64 * (c + 1))) + (t & 1) * uint32_t(BUF);
#pragma unroll
                for (int b = 0; b < NS; ++b) {
#pragma unroll
                    for (int x = 0; x < NR; ++x) {
                        v4i& d = acc[RES_A ? x : b][RES_A ? b : x];
                        const v4i z = c == 0 ? v4i{Z, Z, Z, Z} : d;
                        d = RES_A ? __builtin_amdgcn_mfma_i32_16x16x64_i8(res[c][x], fs[b], z, 0, 0, 0)
                                  : __builtin_amdgcn_mfma_i32_16x16x64_i8(fs[b], res[c][x], z, 0, 0, 0);
                    }
                    if (c + 1 < CH) fs[b] = *reinterpret_cast<const v4i*>(lds + nx + b * 16 * ROW);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            store_staged<RA, CB, RED, PAIR>(acc, C, depS | baseR, ex, ms, lane, wstage);
            depS = ((depS | ~hiS) + oneS) & hiS;
        }
    }
}

// split-K: sum the partial residues of every K range and scatter into C; a
// thread takes 16 consecutive A indices, whose C offsets differ by the same
// 16 deposits everywhere (one output and two bit deposits per thread made
// this kernel 5 times as long as the products: 144 us for 16 planes of rank
// 20 against 24).
template <class G>
__global__ __launch_bounds__(256) void k_mfma8_reduce(StepArgs a, const int8_t* part, int64_t part_stride,
                                                      int splits) {
    const int g = blockIdx.z;
    const ModSmall ms{int32_t(a.p[g]), a.r2[g], a.r16[g], a.pinv[g]};
    int8_t* C = static_cast<int8_t*>(a.C) + g * a.strideC;
    const int lgA = a.fA - G::LGM, lgB = a.fB - G::LGN;
    const uint64_t T = uint64_t(1) << (lgA + lgB);
    const uint64_t n = T * (G::WM * G::WN / 16);
    const int8_t* pg = part + g * part_stride;
    uint64_t off[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) off[v] = pdep64(uint64_t(v), a.maskA);
    for (uint64_t e = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < n; e += uint64_t(gridDim.x) * blockDim.x) {
        const uint64_t tile = e / (G::WM * G::WN / 16), loc = 16 * (e % (G::WM * G::WN / 16));  // loc = j WM + i
        int32_t sum[16] = {};  // at most 1024 residues of magnitude 127
        for (int y = 0; y < splits; ++y) {
            const v4i x = *reinterpret_cast<const v4i*>(pg + (uint64_t(y) * T + tile) * (G::WM * G::WN) + loc);
#pragma unroll
            for (int v = 0; v < 16; ++v) sum[v] += int32_t(int8_t(x[v / 4] >> (8 * (v % 4))));
        }
        uint32_t ta, tb;
        tile_coords_lg(uint32_t(tile), lgA, lgB, ta, tb);
        const uint64_t j = loc / G::WM, i = loc % G::WM;
        int8_t* const out = C + (pdep64(uint64_t(ta) * G::WM + i, a.maskA) | pdep64(uint64_t(tb) * G::WN + j, a.maskB));
#pragma unroll
        for (int v = 0; v < 16; ++v) out[off[v]] = int8_t(ms.center32(sum[v]));
    }
}

// Short shared dimension, K = 2^S <= 32: no staging. Each lane reads its
// fragments straight from A's and B's rows (K consecutive bytes, the tile's
// rows consecutive in memory, so a wave's fragment load covers 16 whole rows)
// -- 8 bytes at K offset 8 q, zero where 8 q >= K -- and one
// v_mfma_i32_16x16x32_i8 per 16x16 block gives the exact sums (at most
// 32 127^2 < 2^21). Such steps are bound by writing C. The next tile's
// fragments are requested as soon as a tile's products are issued. (Loads and
// stores share one completion counter, so the wait for them also covers the
// stores before; two or four tiles per wait were no faster on the largest
// 1-in-3 configuration.)
template <class G, int S>
__global__ __launch_bounds__(G::THREADS) void k_mfma8_short(StepArgs a, Mfma8Extra ex) {
    constexpr int RA = G::RA, CB = G::CB, K = 1 << S;
    __shared__ __align__(1024) uint8_t stage[G::NW * Piece<RA, CB>::BYTES];
    const int g = blockIdx.z;
    const int8_t* A = static_cast<const int8_t*>(a.A) + g * a.strideA;
    const int8_t* B = static_cast<const int8_t*>(a.B) + g * a.strideB;
    int8_t* C = static_cast<int8_t*>(a.C) + g * a.strideC;
    const ModSmall ms{int32_t(a.p[g]), a.r2[g], a.r16[g], a.pinv[g]};
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = (w % G::WAVES_A) * 16 * RA, wc = (w / G::WAVES_A) * 16 * CB;
    const int lgA = a.fA - G::LGM, lgB = a.fB - G::LGN;
    const uint32_t T = 1u << (lgA + lgB);
    const int fr = lane & 15, q = lane >> 4;
    const uint64_t waveC = pdep64(uint64_t(wr), a.maskA) | pdep64(uint64_t(wc), a.maskB);
    uint8_t* const wstage = stage + w * Piece<RA, CB>::BYTES;
    // lane's fragment offset within a tile's rows: row wr + fr (A) or
    // wc + fr (B), K offset 8 q
    const uint32_t offA = uint32_t((wr + fr) * K + 8 * q), offB = uint32_t((wc + fr) * K + 8 * q);
    typedef long frag_t;
    auto load = [&](const int8_t* p) -> frag_t {
        if constexpr (S >= 3) {
            if (8 * q >= K) return 0;
            return *reinterpret_cast<const frag_t*>(p);
        } else {
            if (q != 0) return 0;
            if constexpr (S == 2) return frag_t(*reinterpret_cast<const uint32_t*>(p));
            if constexpr (S == 1) return frag_t(*reinterpret_cast<const uint16_t*>(p));
            return frag_t(*reinterpret_cast<const uint8_t*>(p));
        }
    };
    frag_t fa[RA], fb[CB];
    auto fetch = [&](uint32_t tile) {
        uint32_t ta, tb;
        tile_coords_lg(tile, lgA, lgB, ta, tb);
        const int8_t* pA = A + uint64_t(ta) * G::WM * K + offA;
        const int8_t* pB = B + uint64_t(tb) * G::WN * K + offB;
#pragma unroll
        for (int rb = 0; rb < RA; ++rb) fa[rb] = load(pA + 16 * K * rb);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) fb[cb] = load(pB + 16 * K * cb);
    };
    uint32_t tile = blockIdx.x;
    if (tile >= T) return;
    fetch(tile);
    for (;;) {
        v4i acc[RA][CB];
#pragma unroll
        for (int rb = 0; rb < RA; ++rb)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
                acc[rb][cb] = __builtin_amdgcn_mfma_i32_16x16x32_i8(
                    fa[rb], fb[cb], v4i{kBiasBits, kBiasBits, kBiasBits, kBiasBits}, 0, 0, 0);
        const uint32_t next = tile + gridDim.x;
        if (next < T) fetch(next);
        uint32_t ta, tb;
        tile_coords_lg(tile, lgA, lgB, ta, tb);
        const uint64_t baseC = (pdep_from(ta, ex.hiA) | pdep_from(tb, ex.hiB)) | waveC;
        store_tile8<RA, CB, RED_BIAS>(acc, C, baseC, a, ex, ms, lane, wstage);
        if (next >= T) break;
        tile = next;
    }
}

uint64_t pdep_host(uint64_t x, uint64_t m) {
    uint64_t r = 0;
    for (; m; m &= m - 1, x >>= 1)
        if (x & 1) r |= m & (~m + 1);
    return r;
}

template <class Gm>
Mfma8Extra extra_of(const StepArgs& a) {
    using Pc = Piece<Gm::RA, Gm::CB>;
    constexpr int nA = 4 + lg2(Pc::RAP), nB = 4 + lg2(Gm::CB), n = nA + nB;
    static_assert(n >= 10 && n <= 12, "piece of 1 to 4 KiB");
    Mfma8Extra ex{};
    ex.hiA = a.maskA & ~pdep_host(Gm::WM - 1, a.maskA);
    ex.hiB = a.maskB & ~pdep_host(Gm::WN - 1, a.maskB);
    for (int rb = 0; rb < 8; ++rb) ex.dA[rb] = pdep_host(uint64_t(16 * rb), a.maskA);
    for (int v = 0; v < 4; ++v) ex.dV[v] = pdep_host(uint64_t(v), a.maskA);
    for (int cb = 0; cb < 4; ++cb) ex.dB[cb] = pdep_host(uint64_t(16 * cb), a.maskB);
    // v_perm selectors: bytes 0..3 of the neighbour's word are 0..3, the
    // lane's own are 4..7
    if ((a.maskA & 3) == 3) {
        ex.mode = 0;
        ex.sel[0] = ex.sel[1] = 0x07060504u;
    } else if ((a.maskB & 1) && (a.maskA & 2)) {  // C bit 0 from B, bit 1 from A
        ex.mode = 1;
        ex.sel[0] = 0x01050004u;  // own v0, neighbour v0, own v1, neighbour v1
        ex.sel[1] = 0x07030602u;  // neighbour v2, own v2, neighbour v3, own v3
    } else if ((a.maskA & 1) && (a.maskB & 2)) {  // C bit 0 from A, bit 1 from B
        ex.mode = 1;
        ex.sel[0] = 0x01000504u;  // own v0, own v1, neighbour v0, neighbour v1
        ex.sel[1] = 0x07060302u;  // neighbour v2, neighbour v3, own v2, own v3
    } else {
        ex.mode = 2;
        return ex;
    }
    // the piece's bits in C's order: C bit of A index bit i / B index bit j,
    // and its rank among them
    uint64_t posA[nA], posB[nB], all = 0;
    for (int i = 0; i < nA; ++i) all |= posA[i] = pdep_host(uint64_t(1) << i, a.maskA);
    for (int j = 0; j < nB; ++j) all |= posB[j] = pdep_host(uint64_t(1) << j, a.maskB);
    const auto rank_of = [&](uint64_t pos) { return __builtin_popcountll(all & (pos - 1)); };
    // lane bits: B index bits 0..3 and A index bits 2, 3; in mode 1 lane bit
    // 0 stands for A index bit 1
    int lr[6];
    for (int k = 0; k < 4; ++k) lr[k] = rank_of(posB[k]);
    lr[4] = rank_of(posA[2]);
    lr[5] = rank_of(posA[3]);
    if (ex.mode == 1) lr[0] = rank_of(posA[1]);
    // M: chunk index bit c >= 4 (index bit c + 4) is XORed into the low four
    // bits as M[c - 4]; a lane bit up there takes a low bit that no other lane
    // bit has
    uint32_t M[4] = {0, 0, 0, 0}, used = 0;
    for (int k = 0; k < 6; ++k)
        if (lr[k] >= 4 && lr[k] < 8) used |= 1u << (lr[k] - 4);
    for (int k = 0; k < 6; ++k)
        if (lr[k] >= 8) {
            const uint32_t low = ~used & 15u, bit = low & (~low + 1);
            M[lr[k] - 8] = bit;
            used |= bit;
        }
    // byte place of an index bit
    const auto place = [&](int rank) -> uint32_t {
        uint32_t x = 1u << rank;
        if (rank >= 8) x ^= M[rank - 8] << 4;
        return x;
    };
    for (int k = 0; k < 6; ++k) ex.sLane[k] = place(lr[k]);
    for (int rb = 0; rb < Pc::RAP; ++rb)
        for (int i = 4; i < nA; ++i)
            if ((rb >> (i - 4)) & 1) ex.sRb[rb] ^= place(rank_of(posA[i]));
    for (int cb = 0; cb < Gm::CB; ++cb)
        for (int j = 4; j < nB; ++j)
            if ((cb >> (j - 4)) & 1) ex.sCb[cb] ^= place(rank_of(posB[j]));
    ex.rM[0] = M[0] << 4;
    ex.rM[1] = M[1] << 4;
    const auto pos_of = [&](int rank) { return pdep_host(uint64_t(1) << rank, all); };
    for (int k = 0; k < 6; ++k) ex.cLane[k] = pos_of(4 + k);
    for (int t = 0; t < Pc::NT; ++t)
        for (int k = 0; k < 2; ++k)
            if ((t >> k) & 1) {
                ex.rT[t] ^= place(10 + k);
                ex.cT[t] |= pos_of(10 + k);
            }
    ex.cPiece = pdep_host(uint64_t(16 * Pc::RAP), a.maskA);
    return ex;
}

// A grid that fills the GPU once: the work-groups walk the tiles of every
// plane, so that only their first tile waits for its first stages unhidden
// (launched per plane with 1024 work-groups, a group had 4 to 32 tiles).
template <class Gm, int NST, int RED>
void launch_nst(const StepArgs& a, const Mfma8Extra& ex, int G, uint64_t T, int splits, int8_t* part,
               int64_t scratch_per_plane, hipStream_t stream) {
    static const int per_cu = [] {
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, (const void*)k_mfma8<Gm, NST, RED>, Gm::THREADS, 0) !=
            hipSuccess)
            n = 1;
        return std::max(n, 1);
    }();
    const dim3 grid(uint32_t(std::min<uint64_t>(T * uint64_t(G), uint64_t(kCUs) * uint64_t(per_cu))), uint32_t(splits),
                    1);
    hipLaunchKernelGGL((k_mfma8<Gm, NST, RED>), grid, dim3(Gm::THREADS), 0, stream, a, ex, G, splits, part,
                       scratch_per_plane);
}

template <class Gm>
hipError_t launch_cfg(const StepArgs& a, int G, hipStream_t stream, char* scratch, int64_t scratch_per_plane) {
    const Mfma8Extra ex = extra_of<Gm>(a);
    const uint64_t T = (uint64_t(1) << (a.fA - Gm::LGM)) * (uint64_t(1) << (a.fB - Gm::LGN));
    // too few output tiles to fill the GPU (one work-group of the larger tiles
    // per CU, two of the others): split K over block rows (powers of two, as
    // many partial tiles per plane as the scratch area holds, at least 8 steps
    // each so that reading operands outweighs writing the partial tile)
    const int nk = 1 << (a.s - 6);
    const uint64_t fill = kCUs * (Gm::WM * Gm::WN > 128 * 128 ? 1 : 2);
    const uint64_t cap_tiles = uint64_t(scratch_per_plane) / uint64_t(Gm::WM * Gm::WN);
    int splits = 1;
    while (T * G * splits * 2 <= fill && splits * 16 <= nk && T * splits * 2 <= cap_tiles) splits *= 2;
    int8_t* part = reinterpret_cast<int8_t*>(scratch);
    const int per = nk / splits;  // steps of 64 entries
    // (the bias takes four registers that the largest tile does not have)
    constexpr int RED = Gm::RA * Gm::CB == 32 ? RED_PLAIN : RED_BIAS;
    if (per > 8)
        launch_nst<Gm, 4, RED_FOLD>(a, ex, G, T, splits, part, scratch_per_plane, stream);
    else if (per == 8)
        launch_nst<Gm, 4, RED_PLAIN>(a, ex, G, T, splits, part, scratch_per_plane, stream);
    else if (per == 4)
        launch_nst<Gm, 2, RED>(a, ex, G, T, splits, part, scratch_per_plane, stream);
    else if (per == 2)
        launch_nst<Gm, 1, RED>(a, ex, G, T, splits, part, scratch_per_plane, stream);
    else
        launch_nst<Gm, 0, RED>(a, ex, G, T, splits, part, scratch_per_plane, stream);
    if (splits > 1) {
        const uint64_t n = T * uint64_t(Gm::WM * Gm::WN / 16);
        dim3 gr(uint32_t(std::min<uint64_t>((n + 255) / 256, 4096)), 1, G);
        hipLaunchKernelGGL((k_mfma8_reduce<Gm>), gr, dim3(256), 0, stream, a, part, scratch_per_plane, splits);
    }
    return hipGetLastError();
}

template <class Gm, int S>
hipError_t launch_short(const StepArgs& a, int G, hipStream_t stream) {
    const uint64_t T = (uint64_t(1) << (a.fA - Gm::LGM)) * (uint64_t(1) << (a.fB - Gm::LGN));
    // A work-group walks up to eight tiles, so that all but the first tile's
    // loads run beside products and stores, as long as 2048 work-groups remain
    // (rank 16 x 16 over K = 16, 8 planes: one tile each 57 us, four 44; rank 21 x 14
    // over K = 32 126, 91). Where there are more the old bound of 2048 a plane
    // holds: rank 17 x 15 over K = 4 631 us, 650 with 2048 in all.
    const uint64_t walk = std::max<uint64_t>({T / 8, 2048u / uint64_t(G), 1});
    dim3 grid(uint32_t(std::min<uint64_t>({T, walk, 2048})), 1, G);
    hipLaunchKernelGGL((k_mfma8_short<Gm, S>), grid, dim3(Gm::THREADS), 0, stream, a, extra_of<Gm>(a));
    return hipGetLastError();
}

template <class Gm>
hipError_t launch_short_s(const StepArgs& a, int G, hipStream_t stream) {
    switch (a.s) {
        case 0: return launch_short<Gm, 0>(a, G, stream);
        case 1: return launch_short<Gm, 1>(a, G, stream);
        case 2: return launch_short<Gm, 2>(a, G, stream);
        case 3: return launch_short<Gm, 3>(a, G, stream);
        case 4: return launch_short<Gm, 4>(a, G, stream);
        default: return launch_short<Gm, 5>(a, G, stream);
    }
}

// Work-groups that hold rows in registers run in pairs on every CU; a run is
// as long as leaves four of them for each.
template <class Gm, bool RES_A, int CH, int RED>
hipError_t launch_rows(const StepArgs& a, int G, hipStream_t stream) {
    const int lgS = (RES_A ? a.fB : a.fA) - 6, lgR = (RES_A ? a.fA : a.fB) - 8;
    int lgL = std::min(lgS, 6);
    while (lgL > 2 && (uint64_t(G) << (lgS - lgL + lgR)) < 4 * kRowsPerCU<CH> * kCUs) --lgL;
    const uint32_t runs = uint32_t(G) << (lgS - lgL), items = runs << lgR;
    const Mfma8Extra ex = extra_of<Gm>(a);
    const dim3 grid(std::min<uint32_t>(items, kRowsPerCU<CH> * kCUs)), block(Gm::THREADS);
    const int spread = runs % 8 == 0;
    if (ex.mode == 0)
        hipLaunchKernelGGL((k_mfma8_rows<Gm, RES_A, CH, RED, false>), grid, block, 0, stream, a, ex, items, lgL,
                           spread);
    else
        hipLaunchKernelGGL((k_mfma8_rows<Gm, RES_A, CH, RED, true>), grid, block, 0, stream, a, ex, items, lgL, spread);
    return hipGetLastError();
}

// A as B and B as A.
void exchange(StepArgs& a) {
    std::swap(a.A, a.B);
    std::swap(a.strideA, a.strideB);
    std::swap(a.maskA, a.maskB);
    std::swap(a.fA, a.fB);
}

}  // namespace

bool mfma8_eligible(const StepArgs& a) {
    // at least one 128 x 64 tile, K of at least one 64-entry chunk, a
    // stage's rows within 32-bit load offsets and the tile count in 32 bits
    // (K below 64: the unstaged kernel, 128 x 128 or 128 x 64 tiles)
    return a.s >= 0 && a.s <= k8MaxRowBytesLog && a.fA >= 7 && a.fB >= 6 && a.fA + a.fB <= 45;
}

int mfma8_rule_cfg(const StepArgs& a) {
    if (a.fB >= 8) return MFMA8_256x256;
    if (a.fB == 7) return a.fA >= 8 ? MFMA8_256x128 : MFMA8_128x128;
    return a.fA >= 8 ? MFMA8_256x64 : MFMA8_128x64;
}

hipError_t launch_mfma8_cfg(const StepArgs& a0, int G, hipStream_t stream, char* scratch, int64_t scratch_per_plane,
                            int cfg) {
    if (!mfma8_eligible(a0) || (cfg != MFMA8_RULE && !mfma8_cfg_fits(cfg, a0.fA, a0.fB))) return hipErrorInvalidValue;
    StepArgs a = a0;
    // C's two lowest bits are B's: with the operands exchanged they are A's
    // and outputs leave as words instead of bytes (tiles of 128 x 128 or more
    // take either side as A)
    if ((a.maskB & 3) == 3 && a.fB >= 7) {
        exchange(a);
        if (cfg == MFMA8_RULE && a.s >= 6) cfg = a.fA >= 8 && a.fB >= 8 ? MFMA8_256x256 : MFMA8_128x128;
        if (cfg == MFMA8_256x128 || cfg == MFMA8_256x64) cfg = MFMA8_128x128;
    }
    // (a B side of 6 bits exchanges where K is short: tiles of 64 x 256)
    if (a.s < 6 && a.fB == 6 && a.fA >= 8 && (a.maskB & 3) == 3) {
        exchange(a);
        return launch_short_s<Cfg64x256>(a, G, stream);
    }
    if (a.s < 6)
        return a.fB >= 7 ? launch_short_s<Cfg128x128>(a, G, stream) : launch_short_s<Cfg128x64>(a, G, stream);
    if (cfg == MFMA8_RULE) cfg = mfma8_rule_cfg(a);
    switch (cfg) {
        case MFMA8_256x256: return launch_cfg<Cfg256x256>(a, G, stream, scratch, scratch_per_plane);
        case MFMA8_256x128: return launch_cfg<Cfg256x128>(a, G, stream, scratch, scratch_per_plane);
        case MFMA8_128x128: return launch_cfg<Cfg128x128>(a, G, stream, scratch, scratch_per_plane);
        case MFMA8_256x64: return launch_cfg<Cfg256x64>(a, G, stream, scratch, scratch_per_plane);
        default: return launch_cfg<Cfg128x64>(a, G, stream, scratch, scratch_per_plane);
    }
}

// From 2048 tiles of 64 x 256 on; below, a work-group has too few tiles per resident
// fragment load (K = 256: 9 planes of 2^20 outputs 14.1 us against 13.3 in k_mfma8, 2^22
// 27.5 against 28.2, 2^24 68 against 70; K = 128: 2^22 21.5 against 23.4, 2^24 48 against
// 54). At K = 512 from 16384 on (9 planes of 2^24 113 against 103, 8 of 2^25 172 against 186, of
// 2^27 547 against 715).
bool rows8_eligible(const StepArgs& a, int G) {
    const int hi = std::max(a.fA, a.fB), lo = std::min(a.fA, a.fB);
    return a.s >= 7 && a.s <= 9 && lo >= 8 && hi + lo <= 45 &&
           (uint64_t(G) << (hi - 6 + lo - 8)) >= (a.s == 9 ? 16384 : 2048);
}

hipError_t launch_rows8(const StepArgs& a0, int G, hipStream_t stream) {
    StepArgs a = a0;
    if (a.fB > a.fA) exchange(a);
    // the larger side streams; C's two lowest bits are A's or one of each
    if ((a.maskB & 3) == 3) {
        exchange(a);
        return a.s == 9   ? launch_rows<Cfg256x64, true, 8, RED_PLAIN>(a, G, stream)
               : a.s == 8 ? launch_rows<Cfg256x64, true, 4, RED_BIAS>(a, G, stream)
                          : launch_rows<Cfg256x64, true, 2, RED_BIAS>(a, G, stream);
    }
    return a.s == 9   ? launch_rows<Cfg64x256, false, 8, RED_PLAIN>(a, G, stream)
           : a.s == 8 ? launch_rows<Cfg64x256, false, 4, RED_BIAS>(a, G, stream)
                      : launch_rows<Cfg64x256, false, 2, RED_BIAS>(a, G, stream);
}

// K of at most 32 entries and a B side of 16 or 32 rows: bound by reading A and
// writing C, which the streaming kernel did a byte per lane (2^21 x 2^4 outputs
// over K = 32: 80 us a plane, over K = 16: 78 us; here 22 and 20). At least
// one tile of 512 rows; fewer B rows would leave most of a block's columns
// empty.
bool short8_eligible(const StepArgs& a) {
    return a.s >= 0 && a.s <= 5 && (a.fB == 4 || a.fB == 5) && a.fA >= 9 && a.fA + a.fB <= 45;
}

hipError_t launch_short8(const StepArgs& a0, int G, hipStream_t stream, Profiler* prof, double step_bytes,
                         double step_macs) {
    if (!short8_eligible(a0)) return hipErrorInvalidValue;
    StepArgs a = a0;
    const bool ex = (a.maskB & 3) == 3;  // as in launch_mfma8_cfg
    if (ex) exchange(a);
    prof->before(stream);
    const hipError_t e = a0.fB == 4 ? (ex ? launch_short_s<Cfg16x256>(a, G, stream)
                                          : launch_short_s<Cfg512x16>(a, G, stream))
                                    : (ex ? launch_short_s<Cfg32x256>(a, G, stream)
                                          : launch_short_s<Cfg512x32>(a, G, stream));
    prof->after_raw(stream, KC_NARROW, step_bytes, step_macs);
    return e;
}

hipError_t launch_mfma8(const StepArgs& a, int G, hipStream_t stream, Profiler* prof, double step_bytes,
                        double step_macs, char* scratch, int64_t scratch_per_plane) {
    if (!mfma8_eligible(a)) return hipErrorInvalidValue;
    prof->before(stream);
    // the autotuner's measured tile shape for the nearest tuned shape, else the rule
    const int cfg = a.s >= 6 ? tuned_choice(TK_MFMA8, EL_I8, a.fA, a.fB, a.s) : MFMA8_RULE;
    const hipError_t e = rows8_eligible(a, G) ? launch_rows8(a, G, stream)
                                              : launch_mfma8_cfg(a, G, stream, scratch, scratch_per_plane, cfg);
    prof->after_raw(stream, KC_MFMA, step_bytes, step_macs);
    return e;
}

}  // namespace tn
