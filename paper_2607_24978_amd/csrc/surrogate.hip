// Learned surrogate kernels for gfx950: periodic 3x3x3 convolutions as
// implicit GEMMs on BF16 MFMA (v_mfma_f32_16x16x32_bf16, FP32 accumulate),
// their input and weight gradients, GELU, MSE, Adam, and the packing of
// lattice states into network inputs.
//
// Activations are channels-last BF16, act[site][C] with C = 8 or 32 and
// site = (x*N + y)*N + z.  Weights for a convolution are BF16
// w[o][co][ci] (o = 27 stencil offsets, (dx+1)*9 + (dy+1)*3 + (dz+1); a 28th
// all-zero offset pads the 8-channel case), so that one MFMA operand
// fragment -- 8 consecutive input channels -- is one 16-byte load.
//
// MFMA 16x16x32 lane layout (gfx950): lane l holds A[m = l%16][k = 8g..8g+7]
// and B[k = 8g..8g+7][n = l%16] with g = l/16, and gets
// D[m = 4g + r][n = l%16], r = 0..3.  Here A = weights (m = output channel),
// B = inputs (n = site), so each lane ends with 4 consecutive output
// channels of one site.
#include "surrogate.h"
#include "static_for.h"
#include "xcd_order.h"

#include <hip/hip_runtime.h>
#include <algorithm>
#include <cmath>
#include <cstdint>

#pragma clang fp contract(off)

namespace cl {
namespace sg {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// staging registers: a plain vector type, which (unlike uint4) is promoted to VGPRs
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t f2bf(float f) {
    // round to nearest, ties to even (finite values)
    uint32_t u = __builtin_bit_cast(uint32_t, f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return static_cast<uint16_t>(u >> 16);
}

__device__ __forceinline__ float bf2f(uint16_t h) { return __builtin_bit_cast(float, static_cast<uint32_t>(h) << 16); }

// Two FP32 values to packed BF16 (round to nearest even) with the hardware
// conversion; the same rounding as f2bf.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t cvt2(float lo, float hi) {
    const bf16x2 v = {static_cast<__bf16>(lo), static_cast<__bf16>(hi)};
    return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ uint2 cvt4(const float* f) { return make_uint2(cvt2(f[0], f[1]), cvt2(f[2], f[3])); }

// Two words of 4 packed BF16 values to FP32
__device__ __forceinline__ void unpack4(uint2 u, float* f) {
    f[0] = __builtin_bit_cast(float, u.x << 16);
    f[1] = __builtin_bit_cast(float, u.x & 0xFFFF0000u);
    f[2] = __builtin_bit_cast(float, u.y << 16);
    f[3] = __builtin_bit_cast(float, u.y & 0xFFFF0000u);
}

__device__ __forceinline__ bf16x8 load8(const uint16_t* p) {
    const uint4 v = *reinterpret_cast<const uint4*>(p);
    return __builtin_bit_cast(bf16x8, v);
}

__device__ __forceinline__ bf16x8 zero8() { return __builtin_bit_cast(bf16x8, make_uint4(0, 0, 0, 0)); }

// GELU(z) = z Phi(z) and GELU'(z) = Phi(z) + z phi(z) (Phi, phi: standard
// normal distribution and density).  The epilogues evaluate them for every
// output, so Phi goes through erfc(x), x = |z|/sqrt 2, in the Chebyshev-fitted
// form t exp(-x^2 + P(t)), t = 1/(1 + x/2), of Press et al. (Numerical Recipes,
// erfcc; relative error below 1.2e-7 for all x >= 0, so also in the negative
// tail where Phi is small), with the hardware reciprocal and exp2: one rcp, two
// exp2 and ten FMAs instead of the library's branchy erff and expf.
constexpr float kErfc[10] = {0.17087277f,  -0.82215223f, 1.48851587f, -1.13520398f, 0.27886807f,
                             -0.18628806f, 0.09678418f,  0.37409196f, 1.00002368f,  -1.26551223f};
constexpr float kLog2e = 1.4426950408889634f;
__device__ __forceinline__ float phi_cdf(float z, float* dens) {
    const float x = fabsf(z) * 0.70710678118654752f;
    const float t = __builtin_amdgcn_rcpf(fmaf(0.5f, x, 1.0f));
    float p = kErfc[0];
#pragma unroll
    for (int i = 1; i < 10; ++i) p = fmaf(p, t, kErfc[i]);
    const float mx2 = -x * x;
    const float half_erfc = 0.5f * t * __builtin_amdgcn_exp2f((mx2 + p) * kLog2e);
    if (dens) *dens = 0.39894228040143268f * __builtin_amdgcn_exp2f(mx2 * kLog2e);
    return z >= 0.f ? 1.0f - half_erfc : half_erfc;
}

__device__ __forceinline__ float gelu(float z) { return z * phi_cdf(z, nullptr); }

__device__ __forceinline__ float gelu_grad(float z) {
    float d;
    const float c = phi_cdf(z, &d);
    return c + z * d;
}

// ---------------------------------------------------------------- forward
// What the tiled convolutions make of their FP32 sums plus bias v: z_out = v
// (kEpiZ), a_out = GELU(v) (kEpiGelu), that and zh_out = v (kEpiGeluKeep, when
// the backward pass follows), or a_out = v GELU'(gz) (kEpiGeluGrad).
enum ConvEpilogue { kEpiZ, kEpiGelu, kEpiGeluKeep, kEpiGeluGrad };

// Four outputs of one lane: a_out of the modes that write one.
template <int MODE>
__device__ __forceinline__ uint2 epilogue4(const float* v, uint2 gz) {
    float h[4], zv[4];
    if constexpr (MODE == kEpiGeluGrad) unpack4(gz, zv);
#pragma unroll
    for (int q = 0; q < 4; ++q) h[q] = MODE == kEpiGeluGrad ? v[q] * gelu_grad(zv[q]) : gelu(v[q]);
    return cvt4(h);
}

// One stage of the epilogue of four outputs of a lane, in kEpiStages pieces so
// that the march below can put a piece between its matrix products.  The
// arithmetic is that of gelu and gelu_grad, operation for operation.
struct EpiState {
    float x[4], t[4], p[4], d[4];
};
constexpr int kEpiStages = 11;

template <int MODE, int S>
__device__ __forceinline__ void epi_stage(EpiState& e, const f32x4 v, uint2 gz, uint2& out) {
    float z[4] = {v[0], v[1], v[2], v[3]};
    if constexpr (MODE == kEpiGeluGrad) unpack4(gz, z);
    if constexpr (MODE == kEpiZ) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if constexpr (S == 0) {
            e.x[q] = fabsf(z[q]) * 0.70710678118654752f;
            e.t[q] = fmaf(0.5f, e.x[q], 1.0f);
        } else if constexpr (S == 1) {
            e.t[q] = __builtin_amdgcn_rcpf(e.t[q]);
            e.p[q] = kErfc[0];
        } else if constexpr (S <= 5) {
            e.p[q] = fmaf(e.p[q], e.t[q], kErfc[2 * S - 3]);
            e.p[q] = fmaf(e.p[q], e.t[q], kErfc[2 * S - 2]);
        } else if constexpr (S == 6) {
            e.p[q] = fmaf(e.p[q], e.t[q], kErfc[9]);
            e.x[q] = -e.x[q] * e.x[q];
            if constexpr (MODE == kEpiGeluGrad) e.d[q] = e.x[q] * kLog2e;
        } else if constexpr (S == 7) {
            e.p[q] = (e.x[q] + e.p[q]) * kLog2e;
            if constexpr (MODE == kEpiGeluGrad) e.d[q] = __builtin_amdgcn_exp2f(e.d[q]);
        } else if constexpr (S == 8) {
            e.p[q] = __builtin_amdgcn_exp2f(e.p[q]);
        } else if constexpr (S == 9) {
            e.p[q] = 0.5f * e.t[q] * e.p[q];
            if constexpr (MODE == kEpiGeluGrad) e.d[q] = z[q] * (0.39894228040143268f * e.d[q]);
        } else {
            const float c = z[q] >= 0.f ? 1.0f - e.p[q] : e.p[q];
            e.p[q] = MODE == kEpiGeluGrad ? v[q] * (c + e.d[q]) : z[q] * c;
        }
    }
    if constexpr (S == kEpiStages - 1) out = cvt4(e.p);
}

// Forward for 32 input channels and NB 16-wide output blocks (the hidden
// layers, the last layer, and the input gradient through the hidden layers).
//
// A workgroup of eight waves owns a column of RY y-rows x 16 z-sites and
// marches along x, four output planes a step.  The planes with their halo
// ((RY+2) x 18 sites x 32 channels, 11.5 KB) live in a ring of ten in LDS: six
// are read in a step while the four of the next come from memory through
// registers, one barrier a step.  Two waves share each output plane: with two
// output blocks each takes one of them, with one block each takes half the
// rows (RW rows).  A wave keeps all 27 weight fragments of its block in
// registers for the whole march, and every input fragment it reads from LDS
// feeds the three output rows it is a neighbour of; chunks of a site are
// rotated by zi/4 in LDS.  The epilogue of a step (GELU: about 20 vector
// operations and two transcendental ones per output, as long as the matrix
// products themselves) is cut into pieces that go between the products of the
// next step, so that the two units work at the same time within a wave.
//
// Bound: the matrix cores at the rate they sustain here.  32 -> 32 channels on
// 128^3 with GELU: 130 us, 900 TFLOP/s of the 1160 TFLOP/s a large library
// product reaches; without the epilogue and memory traffic the same loop takes
// 73 us, without the products 65 us.  A kernel that staged one 4 x 8 x 16
// tile, multiplied, then ran its epilogue took 171 us, with four waves per SIMD
// instead of two still 165 us: its phases did not overlap.  32 -> 8 (NB = 1):
// 79 us before, 57 us now.
template <int RY, int NB, int MODE>
__global__ __launch_bounds__(512, 2) void conv32_march(ConvArgs a, int L) {
    static_assert(NB == 2 || MODE == kEpiZ, "only an epilogue that computes nothing has lanes without an output");
    constexpr int ZR = 18, YR = RY + 2, RING = 10;
    constexpr int PLANE = YR * ZR * 32;
    constexpr int RW = NB == 2 ? RY : RY / 2;
    __shared__ __align__(16) uint16_t tin[RING * PLANE + 8];  // and one chunk for the writes of threads without one
    const uint16_t* __restrict__ in = reinterpret_cast<const uint16_t*>(a.in);
    const int N = a.N;
    const int nzt = N / 16, nyt = N / RY;
    int t = xcd_order(blockIdx.x, gridDim.x);
    const int z0 = (t % nzt) * 16;
    t /= nzt;
    const int y0 = (t % nyt) * RY;
    int x0 = (t / nyt) * (4 * L);
    const int steps = min(L, (N - x0) / 4);
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) & 3);
    const int half = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
    const int n = lane & 15, g = lane >> 4;
    const int bs = NB == 2 ? half : 0;       // output block of this wave
    const int r0 = NB == 2 ? 0 : half * RW;  // its first row in the tile
    const uint16_t* __restrict__ wg = reinterpret_cast<const uint16_t*>(a.w) + (16 * bs + n) * 32 + 8 * g;
    bf16x8 wa[27];
#pragma unroll
    for (int j = 0; j < 27; ++j) wa[j] = load8(wg + j * NB * 16 * 32);

    // staging: a thread keeps its 16-byte chunk of the z row and walks the
    // (plane, row) pairs, ROWS at a time
    constexpr int RC = ZR * 4, ROWS = 512 / RC;
    const int rr = threadIdx.x / RC, ch = threadIdx.x % RC;
    const int zc = ch >> 2;
    int zz = z0 - 1 + zc;
    zz = zz < 0 ? zz + N : (zz >= N ? zz - N : zz);
    const uint32_t zoff = static_cast<uint32_t>(zz * 64 + (ch & 3) * 16);
    const int zslot = (zc * 4 + (((ch & 3) + (zc >> 2)) & 3)) * 8;
    auto wrap = [N](int i) { return i < 0 ? i + N : (i >= N ? i - N : i); };
    {
        constexpr int NROW = 6 * YR, ITER = (NROW + ROWS - 1) / ROWS;
        u32x4 v[ITER];
#pragma unroll
        for (int k = 0; k < ITER; ++k) {
            // past the last row a thread re-reads it (in bounds) and stores nothing
            const int row = min(rr + k * ROWS, NROW - 1), pi = row / YR, yi = row - pi * YR;
            v[k] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(in) +
                                                   static_cast<size_t>(wrap(x0 - 1 + pi) * N + wrap(y0 - 1 + yi)) * (N * 64) + zoff);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < ITER; ++k) {
            const int row = rr + k * ROWS;
            if (rr < ROWS && row < NROW) *reinterpret_cast<u32x4*>(tin + row * (ZR * 32) + zslot) = v[k];
        }
    }
    constexpr int NROW = 4 * YR, ITER = (NROW + ROWS - 1) / ROWS;
    uint32_t loff[ITER];  // byte offset of a thread's chunks from the first of the four planes
#pragma unroll
    for (int k = 0; k < ITER; ++k) {
        const int row = min(rr + k * ROWS, NROW - 1), pi = row / YR, yi = row - pi * YR;
        loff[k] = static_cast<uint32_t>(pi * N + wrap(y0 - 1 + yi)) * static_cast<uint32_t>(N * 64) + zoff;
    }
    const int c0 = 16 * bs + 4 * g;
    const bool on = c0 < a.cout;  // not a channel that only pads the block
    float bias[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) bias[q] = a.bias && on ? a.bias[c0 + q] : 0.f;
    uint32_t roff[3];  // of a lane's fragment in an LDS row, for each dz
#pragma unroll
    for (int dz = 0; dz < 3; ++dz) {
        const int zi = n + dz;
        roff[dz] = (zi * 4 + ((g + (zi >> 2)) & 3)) * 8 + r0 * ZR * 32;
    }
    f32x4 acc[RW], old[RW];
    uint2 zg[RW];
    int slot0 = 0;  // ring slot of plane x0 - 1
    // weights and bias are here: else every step's waits, which have to hold for
    // the first step too, would wait for that step's own loads and stores
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    // Stores of row r of plane xo.  No branch on a run-time value around what the
    // epilogue computes: the compiler would move all of its pieces into it.
    auto finish = [&](auto R, uint2 o, int xo) {
        constexpr int r = decltype(R)::value;
        const size_t site = static_cast<size_t>((xo * N + y0 + r0 + r) * N + z0);
        if constexpr (MODE == kEpiZ) {
            if (on) *reinterpret_cast<f32x4*>(a.z_out + (site * a.z_stride + 16 * bs) + (n * a.z_stride + 4 * g)) = old[r];
        } else {
            if constexpr (MODE == kEpiGeluKeep) {
                const float u[4] = {old[r][0], old[r][1], old[r][2], old[r][3]};
                *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(a.zh_out) + (site * a.zh_stride + 16 * bs) +
                                          (n * a.zh_stride + 4 * g)) = cvt4(u);
            }
            *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(a.a_out) + (site * a.a_stride + 16 * bs) +
                                      (n * a.a_stride + 4 * g)) = o;
        }
    };
    EpiState es;
    uint2 eo;
    // piece `i` of the epilogue of the previous step's rows
    auto piece = [&](auto I, int xo) {
        constexpr int i = decltype(I)::value;
        if constexpr (i >= 0 && i < RW * kEpiStages) {
            constexpr int r = i / kEpiStages, s = i % kEpiStages;
            epi_stage<MODE, s>(es, old[r], zg[r], eo);
            if constexpr (s == kEpiStages - 1) finish(std::integral_constant<int, r>{}, eo, xo);
        }
    };
    auto products = [&](auto WithOld, int xo) {
        constexpr int G = 9 * (RW + 2);  // (dx, yi, dz) groups, one input fragment each
        constexpr int AHEAD = 2;
        bf16x8 xb[AHEAD + 1];
        const uint16_t* pl[3];
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) {
            int sl = slot0 + w + dx;
            sl = sl >= RING ? sl - RING : sl;
            pl[dx] = tin + sl * PLANE;
        }
        auto fetch = [&](auto GI) {
            constexpr int gi = decltype(GI)::value;
            if constexpr (gi < G) {
                constexpr int dx = gi / (3 * (RW + 2)), yi = (gi / 3) % (RW + 2), dz = gi % 3;
                xb[gi % (AHEAD + 1)] = load8(pl[dx] + roff[dz] + yi * ZR * 32);
            }
        };
#pragma unroll
        for (int r = 0; r < RW; ++r) acc[r] = f32x4{0.f, 0.f, 0.f, 0.f};
        static_for<AHEAD>([&](auto GI) { fetch(GI); });
        static_for<G>([&](auto GI) {
            constexpr int gi = decltype(GI)::value;
            constexpr int dx = gi / (3 * (RW + 2)), yi = (gi / 3) % (RW + 2), dz = gi % 3;
            fetch(std::integral_constant<int, gi + AHEAD>{});
#pragma unroll
            for (int dy = 0; dy < 3; ++dy) {
                const int r = yi - dy;  // output row fed by input row yi at this dy
                if (r < 0 || r >= RW) continue;
                acc[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[dx * 9 + dy * 3 + dz], xb[gi % (AHEAD + 1)], acc[r], 0, 0, 0);
            }
            if constexpr (decltype(WithOld)::value) {
                constexpr int first = G - RW * kEpiStages;
                piece(std::integral_constant<int, gi - (first > 0 ? first : 0)>{}, xo);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // one step: its products, with the epilogue of the step before; the planes the
    // next step adds to the ring are in flight meanwhile.  The first step has its
    // own copy so that the waits of the others know how many stores follow a load.
    const size_t box = static_cast<size_t>(N) * N * (N * 64);
    auto step = [&](auto WithOld, bool more) {
        u32x4 v[ITER];
        if (more) {
            const char* base = reinterpret_cast<const char*>(in) + static_cast<size_t>(x0 + 5) * N * (N * 64);
            const size_t back = x0 + 8 == N ? box : 0;  // only the last plane can be a periodic image
#pragma unroll
            for (int k = 0; k < ITER; ++k) {
                const bool last = (ROWS - 1 + k * ROWS) / YR >= 3 && rr + k * ROWS >= 3 * YR;
                v[k] = *reinterpret_cast<const u32x4*>((last ? base - back : base) + loff[k]);
            }
        }
        products(WithOld, x0 - 4 + w);
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int q = 0; q < 4; ++q) old[r][q] = acc[r][q] + bias[q];
        if constexpr (MODE == kEpiGeluGrad) {
#pragma unroll
            for (int r = 0; r < RW; ++r)
                zg[r] = *reinterpret_cast<const uint2*>(reinterpret_cast<const uint16_t*>(a.gz) +
                                                        (static_cast<size_t>(((x0 + w) * N + y0 + r0 + r) * N + z0) * a.gz_stride + 16 * bs) +
                                                        (n * a.gz_stride + 4 * g));
        }
        if (more) {
#pragma unroll
            for (int k = 0; k < ITER; ++k) {
                const int row = rr + k * ROWS, pi = row / YR;
                int sl = slot0 + 6 + pi;
                sl = sl >= RING ? sl - RING : sl;
                // every thread writes: a branch around it would make the next loads wait for this step's stores
                const int at = sl * PLANE + (row - pi * YR) * (ZR * 32) + zslot;
                *reinterpret_cast<u32x4*>(tin + (rr < ROWS && row < NROW ? at : RING * PLANE)) = v[k];
            }
            slot0 = slot0 + 4 >= RING ? slot0 + 4 - RING : slot0 + 4;
            __syncthreads();
        }
    };
    step(std::false_type{}, steps > 1);
    for (int s = 1; s < steps; ++s) {
        x0 += 4;
        step(std::true_type{}, s + 1 < steps);
    }
    static_for<RW * kEpiStages>([&](auto I) { piece(I, x0 + w); });
}

// Forward for 8 input channels and 32 outputs (the first layer, and
// the input gradient through the last one), one 4 x 8 x 16 tile a workgroup:
// one K = 32 step packs the 8 channels of 4 stencil offsets, lane group g
// taking offset 4s + g, so the weights of a wave's output block (7 steps) stay
// in registers.  Two waves share a plane, one per output block, and go through
// it row by row: 70 registers a wave, so twelve and more waves per CU hide the
// tile's loads and the epilogue, which bounds this kernel (57 of 85 us for 128^3
// with GELU; four waves a tile with both blocks and all rows at once: 103 us).
template <int RY, int MODE>
__global__ __launch_bounds__(512, 4) void conv8_fwd_tiled(ConvArgs a) {
    static_assert(MODE != kEpiZ, "no layer of 8 inputs ends in plain sums");
    constexpr int ZR = 18, YR = RY + 2, PL = 6, KS = 7;
    __shared__ __align__(16) uint16_t tin[PL * YR * ZR * 8];
    const uint16_t* __restrict__ in = reinterpret_cast<const uint16_t*>(a.in);
    const uint16_t* __restrict__ wg = reinterpret_cast<const uint16_t*>(a.w);
    const int N = a.N;
    const int nzt = N / 16, nyt = N / RY;
    int t = xcd_order(blockIdx.x, gridDim.x);
    const int tz = t % nzt;
    t /= nzt;
    const int ty = t % nyt;
    const int tx = t / nyt;
    const int x0 = tx * 4, y0 = ty * RY, z0 = tz * 16;
    constexpr int SITES = PL * YR * ZR;
    constexpr int ITER = (SITES + 511) / 512;
    const int lane = threadIdx.x & 63, w = (threadIdx.x >> 6) & 3;
    const int n = lane & 15, g = lane >> 4;
    const int bs = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);  // output block of this wave
    // the weights (they do not depend on the tile) and all loads of the tile
    // first, then all LDS stores (past the last site a thread re-reads it, in
    // bounds, and stores nothing)
    bf16x8 wa[KS];
    int off[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const int o = 4 * s + g;  // 27 is the all-zero padding offset
        wa[s] = load8(wg + static_cast<size_t>(o * 32 + 16 * bs + n) * 8);
        const int dx = o / 9, dy = (o / 3) % 3, dz = o % 3;
        off[s] = o < 27 ? (((w + dx) * YR + dy) * ZR + n + dz) * 8 : -1;
    }
    u32x4 v[ITER];
#pragma unroll
    for (int k = 0; k < ITER; ++k) {
        const int i = min(static_cast<int>(threadIdx.x) + k * 512, SITES - 1);
        const int zi = i % ZR, yi = (i / ZR) % YR, pi = i / (ZR * YR);
        int xx = x0 - 1 + pi, yy = y0 - 1 + yi, zz = z0 - 1 + zi;
        xx = xx < 0 ? xx + N : (xx >= N ? xx - N : xx);
        yy = yy < 0 ? yy + N : (yy >= N ? yy - N : yy);
        zz = zz < 0 ? zz + N : (zz >= N ? zz - N : zz);
        v[k] = *reinterpret_cast<const u32x4*>(in + static_cast<size_t>((xx * N + yy) * N + zz) * 8);
    }
    // pre-activations for the input gradient's epilogue, in flight with the tile
    const int x = x0 + w, c0 = 16 * bs + 4 * g;
    const size_t site0 = static_cast<size_t>((x * N + y0) * N + z0 + n);
    uint2 zg[RY];
    if constexpr (MODE == kEpiGeluGrad) {
#pragma unroll
        for (int r = 0; r < RY; ++r)
            zg[r] = *reinterpret_cast<const uint2*>(reinterpret_cast<const uint16_t*>(a.gz) + (site0 + r * N) * a.gz_stride + c0);
    }
    float bias[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) bias[q] = a.bias ? a.bias[c0 + q] : 0.f;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < ITER; ++k) {
        const int i = static_cast<int>(threadIdx.x) + k * 512;
        if (i < SITES) *reinterpret_cast<u32x4*>(tin + static_cast<size_t>(i) * 8) = v[k];
    }
    __syncthreads();
    // row by row: the stores of a row leave while the next row's products run
#pragma unroll
    for (int r = 0; r < RY; ++r) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const bf16x8 xb = off[s] >= 0 ? load8(tin + off[s] + r * ZR * 8) : zero8();
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[s], xb, acc, 0, 0, 0);
        }
        float u[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) u[q] = acc[q] + bias[q];
        const size_t site = site0 + r * N;
        if constexpr (MODE == kEpiGeluKeep)
            *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(a.zh_out) + site * a.zh_stride + c0) = cvt4(u);
        *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(a.a_out) + site * a.a_stride + c0) = epilogue4<MODE>(u, zg[r]);
    }
}

// ---------------------------------------------------------------- weight gradient
// dW[o][co][ci] = sum_n dz[n][co] x[n + o][ci],  db[co] = sum_n dz[n][co],
// as MFMA products with K = 32 sites (one 32-site z segment of a row).  The
// MFMA operands need 8 consecutive sites of one channel per lane, the
// transpose of the channels-last layout: the staging threads load 8 sites x
// 8 channels, transpose them in registers and store channel-major rows in LDS
// with 16-byte writes.
//
// A workgroup owns BY y-rows x 32 z-sites and marches along x over L planes
// (a.L).  Step t has in LDS the x plane X0 - 1 + t (BY + 2 rows, each channel
// row holding z0 - 8 .. z0 + 39 so that the z halo sits at slots 7 and 40)
// and the dz plane X0 + t; the next step's planes are loaded from global
// memory before the MFMAs and stored to the other LDS buffer after them, one
// barrier per step.  Wave w takes one (output block b, input block c) pair and
// all 27 offsets (when the layer has only two pairs, two waves share a pair,
// each over half the rows, and write separate partial sums).  It keeps the dz
// fragments of planes X0 + t - 2 .. X0 + t in registers; every x fragment it
// reads (three shifts in z built from three aligned chunks) feeds each
// (dx, dy) offset whose segment lies in its rows.
template <int CIN, int COS, int BY>
__global__ __launch_bounds__(256, 2) void conv_wgrad(WgradArgs a) {
    constexpr int NBI = CIN == 32 ? 2 : 1, NB = COS == 32 ? 2 : 1;
    constexpr int NP = NB * NBI, WPP = 4 / NP, RW = BY / WPP;
    constexpr int CINP = 16 * NBI, COUTP = 16 * NB;
    constexpr int XR = BY + 2, ZS = 48;
    constexpr int CGX = CIN / 8, CGD = COS / 8;
    constexpr int NX = XR * 4 * CGX;  // 8 x 8 transposes of x per plane
    constexpr int ND = BY * 4 * CGD;  // of dz
    constexpr int NE = XR * 2 * CGX;  // z-halo loads of x (8 channels of one site)
    static_assert(NP * WPP == 4 && RW * WPP == BY, "wave split");
    static_assert(NX + ND + NE <= 256, "staging tasks exceed the workgroup");
    __shared__ __align__(16) uint16_t xs[2][XR][CIN][ZS];
    __shared__ __align__(16) uint16_t ds[2][BY][COS][32];
    __shared__ float dbs[ND][8];
    const uint16_t* __restrict__ dz = reinterpret_cast<const uint16_t*>(a.dz);
    const uint16_t* __restrict__ x = reinterpret_cast<const uint16_t*>(a.x);
    const int N = a.N, L = a.L;
    const int nyb = N / BY, nzb = N / 32;
    int blk = blockIdx.x;
    const int y0 = (blk % nyb) * BY;
    blk /= nyb;
    const int z0 = (blk % nzb) * 32;
    const int X0 = (blk / nzb) * L;

    // staging task of this thread, fixed over the march
    const int tid = threadIdx.x;
    int kind = -1, trow = 0, tk = 0, tcg = 0;
    if (tid < NX) {
        kind = 0;
        trow = tid / (4 * CGX);
        tk = (tid / CGX) % 4;
        tcg = tid % CGX;
    } else if (tid < NX + ND) {
        const int u = tid - NX;
        kind = 1;
        trow = u / (4 * CGD);
        tk = (u / CGD) % 4;
        tcg = u % CGD;
    } else if (tid >= 256 - NE) {
        const int u = tid - (256 - NE);
        kind = 2;
        trow = u / (2 * CGX);
        tk = (u / CGX) % 2;
        tcg = u % CGX;
    }
    const int xrow_y = (y0 - 1 + trow + N) % N;  // x rows (kinds 0 and 2)
    const int zedge = tk == 0 ? (z0 - 1 + N) % N : (z0 + 32) % N;
    uint4 pre[8];
    float dbacc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) dbacc[j] = 0.f;

    // global loads of the x plane px and the dz plane qd (periodic in x)
    auto load_stage = [&](int px, int qd) {
        px = px < 0 ? px + N : (px >= N ? px - N : px);
        qd = qd >= N ? qd - N : qd;
        if (kind == 0) {
            const uint16_t* src = x + (static_cast<size_t>(px * N + xrow_y) * N + z0 + 8 * tk) * CIN + 8 * tcg;
#pragma unroll
            for (int j = 0; j < 8; ++j) pre[j] = *reinterpret_cast<const uint4*>(src + j * CIN);
        } else if (kind == 1) {
            const uint16_t* src = dz + (static_cast<size_t>(qd * N + y0 + trow) * N + z0 + 8 * tk) * COS + 8 * tcg;
#pragma unroll
            for (int j = 0; j < 8; ++j) pre[j] = *reinterpret_cast<const uint4*>(src + j * COS);
        } else if (kind == 2) {
            pre[0] = *reinterpret_cast<const uint4*>(x + (static_cast<size_t>(px * N + xrow_y) * N + zedge) * CIN + 8 * tcg);
        }
    };
    // word d of site j: channels 2d (low half) and 2d + 1 (high half)
    auto word = [&](int j, int d) -> uint32_t {
        return d == 0 ? pre[j].x : d == 1 ? pre[j].y : d == 2 ? pre[j].z : pre[j].w;
    };
    // channel ch of sites 2i, 2i + 1 packed in one word
    auto tword = [&](int ch, int i) -> uint32_t {
        const uint32_t lo = word(2 * i, ch >> 1), hi = word(2 * i + 1, ch >> 1);
        return (ch & 1) ? ((lo >> 16) | (hi & 0xFFFF0000u)) : ((lo & 0xFFFFu) | (hi << 16));
    };
    auto store_stage = [&](int buf, bool dz_counts) {
        if (kind == 0) {
#pragma unroll
            for (int ch = 0; ch < 8; ++ch)
                *reinterpret_cast<uint4*>(&xs[buf][trow][8 * tcg + ch][8 + 8 * tk]) =
                    make_uint4(tword(ch, 0), tword(ch, 1), tword(ch, 2), tword(ch, 3));
        } else if (kind == 1) {
#pragma unroll
            for (int ch = 0; ch < 8; ++ch) {
                const uint4 v = make_uint4(tword(ch, 0), tword(ch, 1), tword(ch, 2), tword(ch, 3));
                *reinterpret_cast<uint4*>(&ds[buf][trow][8 * tcg + ch][8 * tk]) = v;
                if (dz_counts) {
                    float s = 0.f;
                    const uint32_t wv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        s += bf2f(static_cast<uint16_t>(wv[i] & 0xFFFFu));
                        s += bf2f(static_cast<uint16_t>(wv[i] >> 16));
                    }
                    dbacc[ch] += s;
                }
            }
        } else if (kind == 2) {
            const int slot = tk == 0 ? 7 : 40;
#pragma unroll
            for (int ch = 0; ch < 8; ++ch) {
                const uint32_t wd = word(0, ch >> 1);
                xs[buf][trow][8 * tcg + ch][slot] = static_cast<uint16_t>((ch & 1) ? (wd >> 16) : (wd & 0xFFFFu));
            }
        }
    };

    const int lane = tid & 63, w = tid >> 6;
    const int n = lane & 15, g = lane >> 4;
    const int pr = w % NP, h = w / NP;
    const int b = pr / NBI, c = pr % NBI;
    const bool bl = CIN == 32 || n < 8;   // lane holds a real input channel
    const bool al = COS == 32 || n < 8;   // lane holds a real dz channel
    f32x4 acc[27];
#pragma unroll
    for (int o = 0; o < 27; ++o) acc[o] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 Ap[RW], Ac[RW], An[RW];
#pragma unroll
    for (int r = 0; r < RW; ++r) Ap[r] = Ac[r] = An[r] = zero8();

    load_stage(X0 - 1, X0);
    store_stage(0, true);
    __syncthreads();
    for (int t = 0; t < L + 2; ++t) {
        const int buf = t & 1;
        const bool more = t + 1 < L + 2;
        if (more) load_stage(X0 + t, X0 + t + 1);
        const bool qvalid = t < L;  // dz plane X0 + t lies in this chunk
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            Ap[r] = Ac[r];
            Ac[r] = An[r];
            An[r] = (qvalid && al) ? load8(&ds[buf][h * RW + r][16 * b + n][8 * g]) : zero8();
        }
#pragma unroll
        for (int yi = 0; yi < RW + 2; ++yi) {
            bf16x8 bm = zero8(), b0 = zero8(), bp = zero8();
            if (bl) {
                const uint16_t* base = &xs[buf][h * RW + yi][16 * c + n][8 * g];
                const uint4 c0 = *reinterpret_cast<const uint4*>(base);
                const uint4 c1 = *reinterpret_cast<const uint4*>(base + 8);
                const uint4 c2 = *reinterpret_cast<const uint4*>(base + 16);
                // z - 1: element 7 of c0, then elements 0..6 of c1; z + 1: 1..7 of c1, 0 of c2
                const uint4 m = make_uint4((c0.w >> 16) | (c1.x << 16), (c1.x >> 16) | (c1.y << 16),
                                           (c1.y >> 16) | (c1.z << 16), (c1.z >> 16) | (c1.w << 16));
                const uint4 p = make_uint4((c1.x >> 16) | (c1.y << 16), (c1.y >> 16) | (c1.z << 16),
                                           (c1.z >> 16) | (c1.w << 16), (c1.w >> 16) | (c2.x << 16));
                bm = __builtin_bit_cast(bf16x8, m);
                b0 = __builtin_bit_cast(bf16x8, c1);
                bp = __builtin_bit_cast(bf16x8, p);
            }
#pragma unroll
            for (int dy = -1; dy <= 1; ++dy) {
                const int ry = yi - 1 - dy;  // segment row fed by this x row at dy
                if (ry < 0 || ry >= RW) continue;
#pragma unroll
                for (int dx = -1; dx <= 1; ++dx) {
                    const bf16x8 af = dx == 1 ? Ap[ry] : (dx == 0 ? Ac[ry] : An[ry]);
                    const int o = 9 * (dx + 1) + 3 * (dy + 1);
                    acc[o] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, bm, acc[o], 0, 0, 0);
                    acc[o + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, b0, acc[o + 1], 0, 0, 0);
                    acc[o + 2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, bp, acc[o + 2], 0, 0, 0);
                }
            }
        }
        if (more) store_stage(buf ^ 1, t + 1 < L);
        __syncthreads();
    }

    // partial sums: [o][co][ci] then [co] for the bias, one slot per wave group
    float* out = a.partials + static_cast<size_t>(blockIdx.x * WPP + h) * a.partial_stride;
#pragma unroll
    for (int o = 0; o < 27; ++o)
#pragma unroll
        for (int r = 0; r < 4; ++r) out[(o * COUTP + 16 * b + 4 * g + r) * CINP + 16 * c + n] = acc[o][r];
    if (kind == 1) {
#pragma unroll
        for (int j = 0; j < 8; ++j) dbs[tid - NX][j] = dbacc[j];
    }
    __syncthreads();
    if (tid < COUTP) {
        float s = 0.f;
        if (tid < COS)
            for (int u = tid / 8; u < ND; u += CGD) s += dbs[u][tid % 8];
        out[27 * COUTP * CINP + tid] = s;
        if (WPP == 2) a.partials[static_cast<size_t>(blockIdx.x * WPP + 1) * a.partial_stride + 27 * COUTP * CINP + tid] = 0.f;
    }
}

// Fixed-order sum of the partials, then scatter into the flat gradient layout
// W[co][ci][dx][dy][dz] (FP32), b[co].  A block takes 64 consecutive
// elements; its four waves sum contiguous quarters of the partials in FP64
// (16 loads in flight per lane) and are combined in wave order.
__global__ __launch_bounds__(256) void wgrad_reduce(WgradReduceArgs a) {
    __shared__ double red[4][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int e = blockIdx.x * 64 + lane;
    const int nW = 27 * a.coutp * a.cinp;
    const int q = (a.nparts + 3) / 4;
    const int p0 = w * q, p1 = min(a.nparts, p0 + q);
    double s = 0.0;
    if (e < nW + a.coutp) {
        const float* src = a.partials + e;
        const size_t st = static_cast<size_t>(a.partial_stride);
        int p = p0;
        for (; p + 16 <= p1; p += 16) {
            float v[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) v[j] = src[static_cast<size_t>(p + j) * st];
#pragma unroll
            for (int j = 0; j < 16; ++j) s += static_cast<double>(v[j]);
        }
        for (; p < p1; ++p) s += static_cast<double>(src[static_cast<size_t>(p) * st]);
    }
    red[w][lane] = s;
    __syncthreads();
    if (w != 0 || e >= nW + a.coutp) return;
    const double tot = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
    if (e < nW) {
        const int o = e / (a.coutp * a.cinp), co = (e / a.cinp) % a.coutp, ci = e % a.cinp;
        if (co < a.cout && ci < a.cin) a.gW[(static_cast<size_t>(co) * a.cin + ci) * 27 + o] = static_cast<float>(tot);
    } else {
        const int co = e - nW;
        if (co < a.cout) a.gb[co] = static_cast<float>(tot);
    }
}

// ---------------------------------------------------------------- elementwise
// MSE against the target: y is [site][ystride] FP32 (cout channels used),
// t is [c][site] FP32; writes d loss / d y as BF16 [site][8] (channels >= cout
// zero) and per-workgroup partial sums of squares.
__global__ __launch_bounds__(256) void mse_grad(const float* __restrict__ y, int ystride, const float* __restrict__ t,
                                                int cout, size_t nsites, double scale, uint16_t* __restrict__ dy,
                                                double* __restrict__ partial) {
    __shared__ double red[256];
    double acc = 0.0;
    for (size_t s = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x; s < nsites;
         s += static_cast<size_t>(gridDim.x) * blockDim.x) {
        uint16_t h[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        for (int c = 0; c < cout; ++c) {
            const double d = static_cast<double>(y[s * ystride + c]) - static_cast<double>(t[c * nsites + s]);
            acc += d * d;
            h[c] = f2bf(static_cast<float>(2.0 * d * scale));
        }
        uint4 u;
        __builtin_memcpy(&u, h, 16);
        *reinterpret_cast<uint4*>(dy + s * 8) = u;
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

// Adam on the FP32 master parameters (Kingma and Ba 2015, bias-corrected).
__global__ void adam_update(float* __restrict__ theta, const float* __restrict__ grad, float* __restrict__ m,
                            float* __restrict__ v, int n, float lr, float b1, float b2, float eps, float c1, float c2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = grad[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float mh = mi / c1, vh = vi / c2;
    theta[i] = theta[i] - lr * mh / (sqrtf(vh) + eps);
}

// FP32 flat parameters of one layer -> BF16 forward weights w[o][coutp][cinp]
// (zero padded, 28th offset zero) and BF16 input-gradient weights
// wd[o'][cinp'][coutp'] = w[flip(o')][co][ci] with roles swapped, plus FP32 bias.
__global__ void prepare_layer(PrepArgs a) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    const int nf = a.no_f * a.coutp * a.cinp;
    if (e < nf) {
        const int o = e / (a.coutp * a.cinp), co = (e / a.cinp) % a.coutp, ci = e % a.cinp;
        float v = 0.f;
        if (o < 27 && co < a.cout && ci < a.cin) v = a.theta[(static_cast<size_t>(co) * a.cin + ci) * 27 + o];
        a.wf[e] = f2bf(v);
    }
    const int nd = a.no_d * a.cinp_d * a.coutp_d;  // input-gradient conv: inputs = co, outputs = ci
    if (a.wd && e < nd) {
        const int o = e / (a.coutp_d * a.cinp_d), ci = (e / a.cinp_d) % a.coutp_d, co = e % a.cinp_d;
        float v = 0.f;
        if (o < 27 && co < a.cout && ci < a.cin) {
            const int of = 26 - o;  // flipped offset: (-dx, -dy, -dz)
            v = a.theta[(static_cast<size_t>(co) * a.cin + ci) * 27 + of];
        }
        a.wd[e] = f2bf(v);
    }
    if (e < a.cout) a.bias[e] = a.theta[a.bias_offset + e];
}

// Lattice state (row-interleaved, T = float or double) -> network input,
// BF16 [site][8]: channels 0..2nf-1 = (field - mean) * inv_scale, then the
// broadcast features, the rest zero.  Also optionally stores the FP32
// fluctuations [c][site] (dataset recording).
template <typename T>
__global__ void pack_state(PackArgs a) {
    const size_t s = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    const size_t N = a.N, n3 = N * N * N;
    if (s >= n3) return;
    const size_t z = s % N, row = s / N;
    const T* st = static_cast<const T*>(a.state);
    const int na = 2 * a.nf;
    uint16_t h[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int c = 0; c < na; ++c) {
        const double v = static_cast<double>(st[(row * na + c) * N + z]) - a.mean[c];
        if (a.fluct_out) a.fluct_out[c * n3 + s] = static_cast<float>(v);
        if (a.fluct_sub) a.fluct_sub[c * n3 + s] = static_cast<float>(v) - a.fluct_sub_ref[c * n3 + s];
        h[c] = f2bf(static_cast<float>(v * a.inv_scale[c]));
    }
    for (int k = 0; k < a.nextra; ++k) h[na + k] = f2bf(a.extra[k]);
    if (a.x_out) {
        uint4 u;
        __builtin_memcpy(&u, h, 16);
        *reinterpret_cast<uint4*>(a.x_out + s * 8) = u;
    }
}

// Network input, FP32 [c][site], c <= 8, to BF16 [site][8].  One read and one
// 16-byte write per site, 7 us for 64^3; the same loop on one host core takes
// 630 us for 64^3.
__global__ __launch_bounds__(256) void pack_input(const float* __restrict__ x, int c, size_t n3, uint16_t* __restrict__ out) {
    const size_t s = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (s >= n3) return;
    uint16_t h[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) h[k] = k < c ? f2bf(x[k * n3 + s]) : 0;
    uint4 u;
    __builtin_memcpy(&u, h, 16);
    *reinterpret_cast<uint4*>(out + s * 8) = u;
}

// The first c channels of FP32 [site][stride], stride a multiple of 4, c <= 8,
// as [c][site]: the layout the host gets, so that only those values are copied.
__global__ __launch_bounds__(256) void channels_first(const float* __restrict__ in, int stride, int c, size_t n3,
                                                      float* __restrict__ out) {
    const size_t s = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (s >= n3) return;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        if (4 * b >= c) break;
        const f32x4 v = *reinterpret_cast<const f32x4*>(in + s * stride + 4 * b);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (4 * b + q < c) out[(4 * b + q) * n3 + s] = v[q];
    }
}

// Normalised dataset sample -> BF16 input [site][8] and FP32 target [c][site].
__global__ void pack_sample(SampleArgs a) {
    const size_t s = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (s >= a.n3) return;
    uint16_t h[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int c = 0; c < a.nfc; ++c) {
        h[c] = f2bf(a.fluct[c * a.n3 + s] * a.inv_in[c]);
        a.target[c * a.n3 + s] = a.incr[c * a.n3 + s] * a.inv_out[c];
    }
    for (int k = 0; k < a.nextra; ++k) h[a.nfc + k] = f2bf(a.extra[k]);
    uint4 u;
    __builtin_memcpy(&u, h, 16);
    *reinterpret_cast<uint4*>(a.x + s * 8) = u;
}

// Apply a predicted jump to the lattice state: for every field channel c,
// state = new_mean[c] + (state - old_mean[c]) + out_scale[c] * y[site][c].
template <typename T>
__global__ void unpack_jump(UnpackArgs a) {
    const size_t s = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    const size_t N = a.N, n3 = N * N * N;
    if (s >= n3) return;
    const size_t z = s % N, row = s / N;
    const T* st = static_cast<const T*>(a.state);
    T* out = static_cast<T*>(a.out);
    const int na = 2 * a.nf;
    for (int c = 0; c < na; ++c) {
        const size_t i = (row * na + c) * N + z;
        const double old = static_cast<double>(st[i]);
        const double v = a.new_mean[c] + (old - a.old_mean[c]) + a.out_scale[c] * static_cast<double>(a.y[s * a.ystride + c]);
        out[i] = static_cast<T>(v);
    }
}

// Host-side launchers ------------------------------------------------------
hipError_t launch_conv_fwd(const ConvArgs& a, int cin, int nb, hipStream_t s) {
    // the outputs of one of the epilogues, or of none of them
    const bool z = a.z_out && !a.zh_out && !a.a_out, act = !a.z_out && a.a_out;
    const int mode = z                                  ? kEpiZ
                     : act && a.gz && !a.zh_out         ? kEpiGeluGrad
                     : act && !a.gz && a.gelu           ? (a.zh_out ? kEpiGeluKeep : kEpiGelu)
                                                        : -1;
    if (mode < 0 || a.N < 16 || a.N % 16) return hipErrorInvalidValue;
    if (cin == 32 && (nb == 2 ? a.cout == 32 : nb == 1 && mode == kEpiZ && a.cout <= 16)) {
        // one column of 8 x 16 output sites per workgroup, its march in as many
        // pieces as fill the chip once: a workgroup has a CU to itself (115 KB of
        // LDS), and every piece pays for its weights, its first six planes and the
        // epilogue of its last step by itself
        constexpr int kCUs = 256;
        const int cols = (a.N / 8) * (a.N / 16), steps = a.N / 4;
        const int chunks = std::min(steps, std::max(1, kCUs / cols));
        const int L = (steps + chunks - 1) / chunks;
        auto k = nb == 1                 ? conv32_march<8, 1, kEpiZ>
                 : mode == kEpiZ         ? conv32_march<8, 2, kEpiZ>
                 : mode == kEpiGelu      ? conv32_march<8, 2, kEpiGelu>
                 : mode == kEpiGeluKeep  ? conv32_march<8, 2, kEpiGeluKeep>
                                         : conv32_march<8, 2, kEpiGeluGrad>;
        hipLaunchKernelGGL(k, dim3(cols * ((steps + L - 1) / L)), dim3(512), 0, s, a, L);
    } else if (cin == 8 && nb == 2 && a.cout == 32 && mode != kEpiZ) {
        // one workgroup per 4 x 8 x 16 block of output sites
        auto k = mode == kEpiGelu       ? conv8_fwd_tiled<8, kEpiGelu>
                 : mode == kEpiGeluKeep ? conv8_fwd_tiled<8, kEpiGeluKeep>
                                        : conv8_fwd_tiled<8, kEpiGeluGrad>;
        hipLaunchKernelGGL(k, dim3((a.N / 4) * (a.N / 8) * (a.N / 16)), dim3(512), 0, s, a);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

WgradShape wgrad_shape(int N, int cin, int cout_stride) {
    // x chunks double (L halves, kept >= 8) until about 512 workgroups
    const int base = (N / 4) * (N / 32);
    int L = N;
    while (base * (N / L) < 512 && L / 2 >= 8 && N % (L / 2) == 0) L /= 2;
    const int nbi = cin == 32 ? 2 : 1, nb = cout_stride == 32 ? 2 : 1;
    WgradShape sh;
    sh.L = L;
    sh.grid = base * (N / L);
    sh.parts = sh.grid * (4 / (nb * nbi));
    sh.stride = 27 * (16 * nb) * (16 * nbi) + 16 * nb;
    return sh;
}

hipError_t launch_conv_wgrad(const WgradArgs& a, int cin, hipStream_t s) {
    if (a.N % 32 || a.L < 1 || a.N % a.L) return hipErrorInvalidValue;
    const int grid = (a.N / 4) * (a.N / 32) * (a.N / a.L);
    if (cin == 32 && a.cout_stride == 32) hipLaunchKernelGGL((conv_wgrad<32, 32, 4>), dim3(grid), dim3(256), 0, s, a);
    else if (cin == 32 && a.cout_stride == 8) hipLaunchKernelGGL((conv_wgrad<32, 8, 4>), dim3(grid), dim3(256), 0, s, a);
    else if (cin == 8 && a.cout_stride == 32) hipLaunchKernelGGL((conv_wgrad<8, 32, 4>), dim3(grid), dim3(256), 0, s, a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_wgrad_reduce(const WgradReduceArgs& a, hipStream_t s) {
    const int n = 27 * a.coutp * a.cinp + a.coutp;
    hipLaunchKernelGGL(wgrad_reduce, dim3((n + 63) / 64), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_mse_grad(const float* y, int ystride, const float* t, int cout, size_t nsites, double scale,
                           void* dy, double* partial, int grid, hipStream_t s) {
    hipLaunchKernelGGL(mse_grad, dim3(grid), dim3(256), 0, s, y, ystride, t, cout, nsites, scale,
                       static_cast<uint16_t*>(dy), partial);
    return hipGetLastError();
}

hipError_t launch_adam(float* theta, const float* grad, float* m, float* v, int n, float lr, float b1, float b2,
                       float eps, float c1, float c2, hipStream_t s) {
    hipLaunchKernelGGL(adam_update, dim3((n + 255) / 256), dim3(256), 0, s, theta, grad, m, v, n, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

hipError_t launch_prepare_layer(const PrepArgs& a, hipStream_t s) {
    int n = a.no_f * a.coutp * a.cinp;
    if (a.wd) n = n > a.no_d * a.cinp_d * a.coutp_d ? n : a.no_d * a.cinp_d * a.coutp_d;
    if (n < a.cout) n = a.cout;
    hipLaunchKernelGGL(prepare_layer, dim3((n + 255) / 256), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_pack_state(const PackArgs& a, bool fp32, hipStream_t s) {
    const size_t n3 = static_cast<size_t>(a.N) * a.N * a.N;
    const dim3 grid(static_cast<unsigned>((n3 + 255) / 256));
    if (fp32) hipLaunchKernelGGL(pack_state<float>, grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL(pack_state<double>, grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_pack_sample(const SampleArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(pack_sample, dim3(static_cast<unsigned>((a.n3 + 255) / 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_pack_input(const float* x, int c, size_t n3, void* out, hipStream_t s) {
    hipLaunchKernelGGL(pack_input, dim3(static_cast<unsigned>((n3 + 255) / 256)), dim3(256), 0, s, x, c, n3,
                       static_cast<uint16_t*>(out));
    return hipGetLastError();
}

hipError_t launch_channels_first(const float* in, int stride, int c, size_t n3, float* out, hipStream_t s) {
    hipLaunchKernelGGL(channels_first, dim3(static_cast<unsigned>((n3 + 255) / 256)), dim3(256), 0, s, in, stride, c, n3, out);
    return hipGetLastError();
}

hipError_t launch_unpack_jump(const UnpackArgs& a, bool fp32, hipStream_t s) {
    const size_t n3 = static_cast<size_t>(a.N) * a.N * a.N;
    const dim3 grid(static_cast<unsigned>((n3 + 255) / 256));
    if (fp32) hipLaunchKernelGGL(unpack_jump<float>, grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL(unpack_jump<double>, grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace sg
}  // namespace cl
