// Training and inference kernels of the order-scoring perceptron (fp32):
//   h1 = relu(W1 x + b1), h2 = relu(W2 h1 + b2), y = w3 . h2 + b3
// over rows x of pair features. The loss is listwise: the rows of a group
// are the candidate pairs of one state of a teacher's order, some of them
// marked as merges the teacher makes next; per group
//   L = log sum_all exp(y) - log sum_pos exp(y),
// averaged over groups. Gradients go through the three layers by hand. Adam
// updates the packed parameters in place. Every buffer belongs to the caller.
//
// The 128 x 128 products (h1 W2^T, dZ2 W2, dZ2^T h1) run on the matrix cores in
// fp32 (v_mfma_f32_16x16x4: fp32 products and sums, lane l holding row or
// column l % 16 at K index l / 16 of a step), 16 x 16 blocks per wave, with the
// weights of a wave's 32 columns kept in registers over all of its rows. What
// is left bounds a training step: six launches, each little more than its
// latency at 13 k rows (the longest: k_back1 24, k_forward 17, k_back2 15 us).
// Measured (MI355X, 13.4 k rows, 64 groups): forward + backward + Adam 717 us with
// one-output-per-thread products and atomic sums of every weight gradient, 62 us
// now; forward of 201 rows 37.8 us in three launches, 7.3 us in one.
#include <hip/hip_runtime.h>

#include <cmath>

#include "internal.hpp"
#include "learned.hpp"

namespace tn {

namespace {

constexpr int F = kFeatures, H = kHidden;

typedef float v4f __attribute__((ext_vector_type(4)));
// four floats at any 4-byte aligned address
typedef float v4u __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kThreads = 256;  // 4 waves, 32 of the 128 columns each
constexpr int kPad = H + 4;    // LDS row of a 128-wide tile read four floats at a time
constexpr int kRec = H * H + 2 * H + 1;  // gradients of W2, b2, w3, b3, packed as in the parameters
static_assert(kOffB2 == kOffW2 + H * H && kOffW3 == kOffB2 + H && kOffB3 == kOffW3 + H, "packing");

// Place of unit u in a tile's row: the four units that a lane takes in one
// 16-byte read, 16 kb + 4 j + l / 16 for j = 0..3, lie side by side.
__device__ __forceinline__ constexpr int place(int u) { return (u & ~15) | ((u & 3) << 2) | ((u >> 2) & 3); }

// The lane halves' (quarters') places of a and b exchanged: upper 32 lanes of a
// with lower 32 of b (odd 16-lane rows of a with even ones of b).
__device__ __forceinline__ void swap32(float& a, float& b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap16(float& a, float& b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}
// Float j of lane row q (lane / 16) becomes float q of lane row j.
__device__ __forceinline__ v4f transpose4(v4f x) {
    float a = x[0], b = x[1], c = x[2], d = x[3];
    swap32(a, c);
    swap32(b, d);
    swap16(a, b);
    swap16(c, d);
    return v4f{a, b, c, d};
}
// Sum over the wave, in every lane: v + v at lane ^ 32, then ^ 16, 8, 4, 2, 1 (what is
// left repeats every 16, 8, 4 lanes, so that a rotation stands for the exchange).
template <int CTRL>
__device__ __forceinline__ float add_dpp(float v) {
    return v + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float wave_sum(float v) {
    float o = v;
    swap32(v, o);
    v += o;
    o = v;
    swap16(v, o);
    v += o;
    return add_dpp<0xb1>(add_dpp<0x4e>(add_dpp<0x124>(add_dpp<0x128>(v))));
}

// acc[rb][cb] += rows of a tile (LDS, kPad floats each, units at their places)
// times the wave's fragments w[cb][kb]: lane l's float j holds unit
// 16 kb + 4 j + l / 16, so that every sum takes the units in ascending order, as a
// loop over them would: a pre-activation within rounding of zero has one sign
// in every kernel that forms it, and the backward pass drops or keeps a whole
// gradient by that sign.
template <int RT>
__device__ __forceinline__ void mul_tile(const float (&tile)[16 * RT][kPad], const v4f (&w)[2][8], int lane,
                                         v4f (&acc)[RT][2]) {
    const int fr = lane & 15, q = lane >> 4;
#pragma unroll
    for (int kb = 0; kb < 8; ++kb)
#pragma unroll
        for (int rb = 0; rb < RT; ++rb) {
            const v4f a = *reinterpret_cast<const v4f*>(&tile[16 * rb + fr][16 * kb + 4 * q]);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int cb = 0; cb < 2; ++cb)
                    acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], w[cb][kb][j], acc[rb][cb], 0, 0, 0);
        }
}

// The layers of LAYERS (bit l - 1: layer l) for 16 RT rows per tile: all three, or
// one, which takes the other layer's rows from memory.
template <int RT, int LAYERS>
__global__ __launch_bounds__(kThreads) void k_forward(const float* P, const float* X, int64_t n, float* H1, float* H2,
                                                      float* y) {
    __shared__ __align__(16) float t1[16 * RT][kPad];
    __shared__ float t2[16 * RT][kPad];
    __shared__ float sx[16 * RT][F];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, fr = lane & 15, q = lane >> 4;
    const int j = t & (H - 1);
    float w1[F];
#pragma unroll
    for (int k = 0; k < F; ++k) w1[k] = P[kOffW1 + j * F + k];
    const float b1 = P[kOffB1 + j];
    v4f wf[2][8];
    float b2[2];
    if constexpr (LAYERS & 2) {
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            const int col = 32 * w + 16 * cb + fr;
#pragma unroll
            for (int kb = 0; kb < 8; ++kb)
                wf[cb][kb] = transpose4(*reinterpret_cast<const v4u*>(P + kOffW2 + col * H + 16 * kb + 4 * q));
            b2[cb] = P[kOffB2 + col];
        }
    }
    const float w3[2] = {P[kOffW3 + lane], P[kOffW3 + lane + 64]}, b3 = P[kOffB3];
    const int64_t tiles = (n + 16 * RT - 1) / (16 * RT);
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int64_t base = tile * (16 * RT);
        __syncthreads();
        if constexpr (LAYERS & 1) {
            for (int e = t; e < 16 * RT * F; e += kThreads)
                sx[e / F][e % F] = base + e / F < n ? X[base * F + e] : 0.0f;
            __syncthreads();
        }
#pragma unroll 4
        for (int r = t >> 7; r < 16 * RT; r += 2) {
            const int64_t i = base + r;
            float h = 0.0f;
            if (i < n) {
                if constexpr (LAYERS & 1) {
                    float a = b1;
#pragma unroll
                    for (int k = 0; k < F; ++k) a += w1[k] * sx[r][k];
                    h = a > 0.0f ? a : 0.0f;
                    H1[i * H + j] = h;
                } else if constexpr (LAYERS & 2) {
                    h = H1[i * H + j];
                } else {
                    t2[r][j] = H2[i * H + j];
                }
            }
            if constexpr (LAYERS & 2) t1[r][place(j)] = h;
        }
        __syncthreads();
        if constexpr (LAYERS & 2) {
            v4f acc[RT][2];
#pragma unroll
            for (int rb = 0; rb < RT; ++rb)
#pragma unroll
                for (int cb = 0; cb < 2; ++cb) acc[rb][cb] = v4f{b2[cb], b2[cb], b2[cb], b2[cb]};
            mul_tile<RT>(t1, wf, lane, acc);
#pragma unroll
            for (int rb = 0; rb < RT; ++rb)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int r = 16 * rb + 4 * q + v;
                    const int64_t i = base + r;
#pragma unroll
                    for (int cb = 0; cb < 2; ++cb) {
                        const float a = acc[rb][cb][v];
                        const float h = a > 0.0f ? a : 0.0f;
                        if (i < n) H2[i * H + 32 * w + 16 * cb + fr] = h;
                        t2[r][32 * w + 16 * cb + fr] = h;
                    }
                }
            __syncthreads();
        }
        if constexpr (LAYERS & 4) {
            // a wavefront per row, 4 RT of them side by side
            float s3 = 0.0f;
#pragma unroll
            for (int r = 0; r < 4 * RT; ++r) {
                const float a = wave_sum(w3[0] * t2[4 * r + w][lane] + w3[1] * t2[4 * r + w][lane + 64]);
                s3 = lane == r ? a : s3;
            }
            const int64_t i = base + 4 * lane + w;
            if (lane < 4 * RT && i < n) y[i] = s3 + b3;
        }
    }
}

// what atomics add to starts at zero
__global__ __launch_bounds__(256) void k_zero(float* grad, int n, float* loss) {
    for (int i = threadIdx.x; i < n; i += 256) grad[i] = 0.0f;
    if (threadIdx.x == 0) *loss = 0.0f;
}

// listwise loss per group: dy = (softmax_all - softmax_pos) / G; the group's loss
// to loss_of[g], or added to *loss without such a place
__global__ __launch_bounds__(256) void k_loss(const float* y, const uint8_t* lab, const int32_t* groups, int32_t G,
                                              float* dy, float* loss, float* loss_of) {
    __shared__ float red[3][4];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    for (int32_t g = blockIdx.x; g < G; g += gridDim.x) {
        const int64_t b = groups[g], e = groups[g + 1];
        float mx = -INFINITY;
        for (int64_t i = b + threadIdx.x; i < e; i += blockDim.x) mx = fmaxf(mx, y[i]);
        for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
        if (lane == 0) red[0][wv] = mx;
        __syncthreads();
        mx = fmaxf(fmaxf(red[0][0], red[0][1]), fmaxf(red[0][2], red[0][3]));
        float sa = 0.0f, sp = 0.0f;
        for (int64_t i = b + threadIdx.x; i < e; i += blockDim.x) {
            const float ex = expf(y[i] - mx);
            sa += ex;
            if (lab[i]) sp += ex;
        }
        for (int o = 32; o > 0; o >>= 1) {
            sa += __shfl_xor(sa, o);
            sp += __shfl_xor(sp, o);
        }
        __syncthreads();
        if (lane == 0) {
            red[1][wv] = sa;
            red[2][wv] = sp;
        }
        __syncthreads();
        sa = red[1][0] + red[1][1] + red[1][2] + red[1][3];
        sp = red[2][0] + red[2][1] + red[2][2] + red[2][3];
        const float inv_g = 1.0f / float(G);
        for (int64_t i = b + threadIdx.x; i < e; i += blockDim.x) {
            const float ex = expf(y[i] - mx);
            const float d = ex / sa - (lab[i] && sp > 0.0f ? ex / sp : 0.0f);
            dy[i] = sp > 0.0f ? d * inv_g : 0.0f;
        }
        if (threadIdx.x == 0) {
            const float l = sp > 0.0f ? (logf(sa) - logf(sp)) * inv_g : 0.0f;
            if (loss_of)
                loss_of[g] = l;
            else if (sp > 0.0f)
                atomicAdd(loss, l);
        }
        __syncthreads();
    }
}

// Backward through layer 3 and the gradients of W2, b2, w3, b3 over a range
// of rows (blockIdx.y): dZ2[i][j] = dy[i] w3[j] [h2 > 0] for the 16 columns j
// of strip blockIdx.x, and G[j][k] = sum_i dZ2[i][j] h1[i][k] (rows are the K
// of the matrix product) into the range's record of ``part`` (kRec floats).
// Partial records and a second kernel instead of float atomics: every range's
// 16 k sums would meet the others' at the memory side.
__global__ __launch_bounds__(kThreads) void k_back2(const float* P, const float* H1, const float* H2, const float* dy,
                                                    int64_t n, int64_t rows, float* dZ2, float* part) {
    constexpr int R = 32;             // rows per step
    constexpr int kRow = H + 16;      // four rows of 16 floats cover the banks
    __shared__ __align__(16) float si[R][kRow];
    __shared__ float sd[R][16];
    __shared__ float red[3][16][17];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, fr = lane & 15, q = lane >> 4;
    const int j0 = 16 * int(blockIdx.x);
    const int64_t i0 = rows * blockIdx.y, i1 = i0 + rows < n ? i0 + rows : n;
    const int c = t & 15, r0 = t >> 4;
    const float w3 = P[kOffW3 + j0 + c];
    float gw = 0.0f, gd = 0.0f, gb = 0.0f;
    v4f acc[2] = {v4f{0, 0, 0, 0}, v4f{0, 0, 0, 0}};
    // the next step's rows are requested before the current one's products
    v4f h1v[R * (H / 4) / kThreads];
    float h2v[R / 16], dyv[R / 16];
    const auto request = [&](int64_t base) {
#pragma unroll
        for (int u = 0; u < R / 16; ++u) {
            const int64_t i = base + r0 + 16 * u;
            h2v[u] = i < i1 ? H2[i * H + j0 + c] : 0.0f;
            dyv[u] = i < i1 ? dy[i] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < R * (H / 4) / kThreads; ++u) {
            const int64_t i = base + (t + kThreads * u) / (H / 4);
            h1v[u] = v4f{0, 0, 0, 0};
            if (i < i1) h1v[u] = *reinterpret_cast<const v4u*>(H1 + i * H + 4 * (t % (H / 4)));
        }
    };
    request(i0);
    for (int64_t base = i0; base < i1; base += R) {
        __syncthreads();
#pragma unroll
        for (int u = 0; u < R / 16; ++u) {
            const int64_t i = base + r0 + 16 * u;
            const float h = h2v[u], d = dyv[u];
            const float dz = h > 0.0f ? d * w3 : 0.0f;
            if (i < i1) dZ2[i * H + j0 + c] = dz;
            gw += d * h;
            gd += d;
            gb += dz;
            sd[r0 + 16 * u][c] = dz;
        }
#pragma unroll
        for (int u = 0; u < R * (H / 4) / kThreads; ++u)
            *reinterpret_cast<v4f*>(&si[(t + kThreads * u) / (H / 4)][4 * (t % (H / 4))]) = h1v[u];
        request(base + R);
        __syncthreads();
#pragma unroll
        for (int ib = 0; ib < R / 4; ++ib) {
            const float a = sd[4 * ib + q][fr];
#pragma unroll
            for (int cb = 0; cb < 2; ++cb)
                acc[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, si[4 * ib + q][32 * w + 16 * cb + fr], acc[cb], 0, 0, 0);
        }
    }
    float* out = part + blockIdx.y * kRec;
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int v = 0; v < 4; ++v) out[(j0 + 4 * q + v) * H + 32 * w + 16 * cb + fr] = acc[cb][v];
    red[0][r0][c] = gb;
    red[1][r0][c] = gw;
    red[2][r0][c] = gd;
    __syncthreads();
    if (t < 48) {
        const int which = t >> 4;
        float s = 0.0f;
        for (int r = 0; r < 16; ++r) s += red[which][r][c];
        if (which < 2)
            out[H * H + which * H + j0 + c] = s;
        else if (t == 32 && blockIdx.x == 0)
            out[H * H + 2 * H] = s;
    }
}

// Sum of the ranges' records (64 entries per work-group, every wave a quarter
// of the ranges) into out; the last work-group sums the groups' losses, left
// at loss_of, and then clears that place: the gradients of W1 and b1.
__global__ __launch_bounds__(256) void k_sum_records(const float* part, int ranges, float* out, float* loss_of,
                                                     int n_groups, float* loss) {
    __shared__ float red[4][64];
    const int lane = int(threadIdx.x) & 63, w = int(threadIdx.x) >> 6;
    if (blockIdx.x + 1 == gridDim.x) {
        if (n_groups == 0) return;
        float s = 0.0f;
        for (int g = int(threadIdx.x); g < n_groups; g += 256) s += loss_of[g];
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
        if (lane == 0) red[w][0] = s;
        __syncthreads();
        for (int g = int(threadIdx.x); g < kOffW2; g += 256) loss_of[g] = 0.0f;
        if (threadIdx.x == 0) *loss = (red[0][0] + red[1][0]) + (red[2][0] + red[3][0]);
        return;
    }
    if (ranges < 2) return;
    const int e = int(blockIdx.x) * 64 + lane;
    float s = 0.0f;
    if (e < kRec) {
#pragma unroll 8
        for (int r = w; r < ranges; r += 4) s += part[int64_t(r) * kRec + e];
    }
    red[w][lane] = s;
    __syncthreads();
    if (w == 0 && e < kRec) out[e] = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
}

// Backward through layer 2, dZ1 = dZ2 W2 masked by h1 > 0, and the gradients
// of W1 and b1 (summed over the work-group's rows, then by atomics)
template <int RT>
__global__ __launch_bounds__(kThreads) void k_back1(const float* P, const float* X, const float* H1, const float* dZ2,
                                                    int64_t n, float* dZ1, float* grad) {
    __shared__ __align__(16) float t2[16 * RT][kPad];
    __shared__ float sx[16 * RT][F];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, fr = lane & 15, q = lane >> 4;
    v4f wf[2][8];
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int kb = 0; kb < 8; ++kb)
#pragma unroll
            for (int jj = 0; jj < 4; ++jj)
                wf[cb][kb][jj] = P[kOffW2 + (16 * kb + 4 * jj + q) * H + 32 * w + 16 * cb + fr];
    // thread t sums unit k = t % 128: features 0..4 and the bias, or 5..9
    const int k = t & (H - 1), half = t >> 7;
    float g[F / 2], gb = 0.0f;
#pragma unroll
    for (int f = 0; f < F / 2; ++f) g[f] = 0.0f;
    const int64_t tiles = (n + 16 * RT - 1) / (16 * RT);
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int64_t base = tile * (16 * RT);
        __syncthreads();
#pragma unroll
        for (int u = 0; u < RT * 2; ++u) {
            // two rows per wave: lane row q holds the 16-byte pieces q of the
            // rows' groups of 16 units
            const int r = 8 * u + 2 * w + (fr >> 3), c = 16 * (fr & 7) + 4 * q;
            v4f d = {0, 0, 0, 0};
            if (base + r < n) d = *reinterpret_cast<const v4u*>(dZ2 + (base + r) * H + c);
            *reinterpret_cast<v4f*>(&t2[r][c]) = transpose4(d);
        }
        for (int e = t; e < 16 * RT * F; e += kThreads) sx[e / F][e % F] = base + e / F < n ? X[base * F + e] : 0.0f;
        __syncthreads();
        v4f acc[RT][2];
#pragma unroll
        for (int rb = 0; rb < RT; ++rb)
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) acc[rb][cb] = v4f{0, 0, 0, 0};
        mul_tile<RT>(t2, wf, lane, acc);
        __syncthreads();  // every wave has read the tile: it takes dZ1
#pragma unroll
        for (int rb = 0; rb < RT; ++rb)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = 16 * rb + 4 * q + v;
                const int64_t i = base + r;
#pragma unroll
                for (int cb = 0; cb < 2; ++cb) {
                    const int col = 32 * w + 16 * cb + fr;
                    float d = 0.0f;
                    if (i < n) {
                        d = H1[i * H + col] > 0.0f ? acc[rb][cb][v] : 0.0f;
                        dZ1[i * H + col] = d;
                    }
                    t2[r][col] = d;
                }
            }
        __syncthreads();
#pragma unroll 4
        for (int r = 0; r < 16 * RT; ++r) {
            const float d = t2[r][k];
#pragma unroll
            for (int f = 0; f < F / 2; ++f) g[f] += d * sx[r][half * (F / 2) + f];
            gb += d;
        }
    }
    // through LDS, so that a wave's atomics go to consecutive addresses (one
    // gradient per lane at stride F took 75 us for the kernel at 13.4 k rows,
    // mostly these)
    __syncthreads();
    float* sg = &t2[0][0];
    static_assert(kOffW2 <= 16 * kPad, "fits the smallest tile");
#pragma unroll
    for (int f = 0; f < F / 2; ++f) sg[kOffW1 + k * F + half * (F / 2) + f] = g[f];
    if (half == 0) sg[kOffB1 + k] = gb;
    __syncthreads();
    for (int e = t; e < kOffW2; e += kThreads) atomicAdd(&grad[e], sg[e]);
}

__global__ __launch_bounds__(256) void k_adam(float* P, const float* g, float* m, float* v, int64_t n, float lr,
                                              float b1, float b2, float eps, float c1, float c2) {
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x) {
        const float gi = g[i];
        const float mi = b1 * m[i] + (1.0f - b1) * gi;
        const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        P[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    }
}

constexpr int64_t kManyRows = 4096;

uint32_t blocks_for(int64_t work, int64_t per, uint32_t cap) {
    return uint32_t(std::max<int64_t>(1, std::min<int64_t>((work + per - 1) / per, cap)));
}

}  // namespace

}  // namespace tn

using namespace tn;

extern "C" {

tn_status tn_mlp_forward(const float* P, const float* X, int64_t n, float* H1, float* H2, float* y, void* stream_) {
    if (!P || n < 0 || (n > 0 && (!X || !H1 || !H2 || !y))) return TN_EINVAL;
    if (n == 0) return TN_OK;
    hipStream_t s = static_cast<hipStream_t>(stream_);
    const auto meet = [](const float* p, int64_t np, const float* q, int64_t nq) { return p < q + nq && q < p + np; };
    const dim3 g1(blocks_for(n, 16, 1024)), g2(blocks_for(n, 32, 1024)), block(kThreads);
    if (meet(H2, n * H, X, n * F) || meet(y, n, X, n * F) || meet(y, n, H1, n * H)) {
        // an output lies where an earlier layer's rows are still to be read:
        // layer by layer
        hipLaunchKernelGGL((k_forward<1, 1>), g1, block, 0, s, P, X, n, H1, H2, y);
        hipLaunchKernelGGL((k_forward<1, 2>), g1, block, 0, s, P, X, n, H1, H2, y);
        hipLaunchKernelGGL((k_forward<1, 4>), g1, block, 0, s, P, X, n, H1, H2, y);
    } else if (n >= kManyRows) {
        // 32-row tiles once they fill the GPU, 16-row tiles below
        hipLaunchKernelGGL((k_forward<2, 7>), g2, block, 0, s, P, X, n, H1, H2, y);
    } else {
        hipLaunchKernelGGL((k_forward<1, 7>), g1, block, 0, s, P, X, n, H1, H2, y);
    }
    return hipGetLastError() == hipSuccess ? TN_OK : TN_EHIP;
}

tn_status tn_mlp_backward(const float* P, const float* X, const float* H1, const float* H2, const float* y,
                          const uint8_t* labels, const int32_t* groups, int32_t n_groups, int64_t n, float* grad,
                          float* dZ2, float* dZ1, float* dy, float* loss, void* stream_) {
    if (!P || !grad || !loss || n < 0 || n_groups < 0) return TN_EINVAL;
    if (n > 0 && (!X || !H1 || !H2 || !y || !labels || !groups || !dZ2 || !dZ1 || !dy)) return TN_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream_);
    if (n == 0 || n_groups == 0) {
        hipLaunchKernelGGL(k_zero, dim3(1), dim3(256), 0, s, grad, kParams, loss);
        return hipGetLastError() == hipSuccess ? TN_OK : TN_EHIP;
    }
    // the groups' losses go where the gradients of W1 and b1 come later; more
    // groups than that add up by atomics
    float* loss_of = n_groups <= kOffW2 ? grad : nullptr;
    if (!loss_of) hipLaunchKernelGGL(k_zero, dim3(1), dim3(256), 0, s, grad, kOffW2, loss);
    hipLaunchKernelGGL(k_loss, dim3(uint32_t(std::min<int32_t>(n_groups, 65535))), dim3(256), 0, s, y, labels, groups,
                       n_groups, dy, loss, loss_of);
    // ranges of rows whose partial gradients fit dZ1 (written after them); one
    // range writes the gradient itself, also where a caller lets dZ1 share
    // memory with a buffer that is still read
    const auto meets = [&](const float* p, int64_t len) { return p < dZ1 + n * H && dZ1 < p + len; };
    const bool shared = meets(H1, n * H) || meets(H2, n * H) || meets(dZ2, n * H) || meets(dy, n) || meets(X, n * F);
    const int64_t ranges = shared ? 1 : std::max<int64_t>(1, std::min<int64_t>({n / 128, n * H / kRec, 64}));
    const int64_t rows = (n + ranges - 1) / ranges;
    float* part = ranges > 1 ? dZ1 : grad + kOffW2;
    hipLaunchKernelGGL(k_back2, dim3(H / 16, uint32_t(ranges)), dim3(kThreads), 0, s, P, H1, H2, dy, n, rows, dZ2,
                       part);
    if (ranges > 1 || loss_of)
        hipLaunchKernelGGL(k_sum_records, dim3((kRec + 63) / 64 + 1), dim3(256), 0, s, part, int(ranges),
                           grad + kOffW2, grad, loss_of ? n_groups : 0, loss);
    if (n >= kManyRows)
        hipLaunchKernelGGL(k_back1<2>, dim3(blocks_for(n, 32, 256)), dim3(kThreads), 0, s, P, X, H1, dZ2, n, dZ1, grad);
    else
        hipLaunchKernelGGL(k_back1<1>, dim3(blocks_for(n, 16, 256)), dim3(kThreads), 0, s, P, X, H1, dZ2, n, dZ1, grad);
    return hipGetLastError() == hipSuccess ? TN_OK : TN_EHIP;
}

tn_status tn_mlp_adam(float* P, const float* grad, float* m, float* v, int32_t step, float lr, float beta1,
                      float beta2, float eps, void* stream_) {
    if (!P || !grad || !m || !v || step < 1) return TN_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream_);
    const float c1 = 1.0f - std::pow(beta1, float(step)), c2 = 1.0f - std::pow(beta2, float(step));
    hipLaunchKernelGGL(k_adam, dim3(blocks_for(kParams, 256, 1024)), dim3(256), 0, s, P, grad, m, v, int64_t(kParams),
                       lr, beta1, beta2, eps, c1, c2);
    return hipGetLastError() == hipSuccess ? TN_OK : TN_EHIP;
}

}  // extern "C"
