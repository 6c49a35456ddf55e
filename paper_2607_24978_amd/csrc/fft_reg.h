// Line FFT of N = 64, 128 or 256 complex values in registers, with one
// exchange through LDS.
//
// The same decimation-in-time transform as fft_lds.h -- the same radix-2
// butterflies and twiddles in the same order, so the same rounding -- with
// its stages split in two: N = R1 R2, R2 threads share a line with R1 values
// each.  Thread t starts from the values n = t + R2 j (j < R1), which are R1
// consecutive positions of the bit-reversed line, runs the first log2 R1
// stages on them, exchanges, and runs the last log2 R2 stages on the
// positions i + R1 g (g < R2) of its S = R1 / R2 rows i = t + R2 s; it ends
// with value k = i + R1 g in register s R2 + g.  Those are the values
// t + R2 (s + S g), so a second transform can start from them in place.
// Against the radix passes over a line in LDS (a bit-reversed store, two or
// three sweeps and a final read, a barrier each) a value crosses LDS once.
#ifndef CL_FFT_REG_H
#define CL_FFT_REG_H

#include "fft_lds.h"
#include "static_for.h"

#include <hip/hip_runtime.h>
#include <type_traits>

namespace cl {

// Radices and threads per line.
template <int N>
struct RegPlan {
    static_assert(N == 64 || N == 128 || N == 256, "line lengths of the register transform");
    static constexpr int S1 = N == 64 ? 3 : 4, S2 = N == 256 ? 4 : 3;  // stages before and after the exchange
    static constexpr int R1 = 1 << S1, R2 = 1 << S2;
    static constexpr int S = R1 / R2;       // rows of the second part per thread
    static constexpr int ROW = R1 + 1;      // LDS row of one group of the first part (one pad value)
    static constexpr int SLOTS = R2 * ROW;  // LDS values of one line
};
inline bool reg_fft_size(int N) { return N == 64 || N == 128 || N == 256; }

template <typename V2> struct ScalarOf;
template <> struct ScalarOf<float2> { using type = float; };
template <> struct ScalarOf<double2> { using type = double; };

constexpr int rev_bits(int x, int bits) {
    int r = 0;
    for (int b = 0; b < bits; ++b) r |= ((x >> b) & 1) << (bits - 1 - b);
    return r;
}

// x times exp(-2 pi i K / 16), K < 8, or its conjugate: the twiddles of the
// first part.
template <int K, bool INV, typename V2>
__device__ __forceinline__ V2 rot16(V2 x) {
    using T = typename ScalarOf<V2>::type;
    V2 r;
    if constexpr (K == 0) {
        return x;
    } else if constexpr (K == 4) {
        r.x = INV ? -x.y : x.y;
        r.y = INV ? x.x : -x.x;
        return r;
    } else {
        constexpr double c1 = 0.92387953251128675613, c2 = 0.70710678118654752440, c3 = 0.38268343236508977173;
        constexpr double c = K == 1 ? c1 : K == 2 ? c2 : K == 3 ? c3 : K == 5 ? -c3 : K == 6 ? -c2 : -c1;
        constexpr double s = (K == 1 || K == 7) ? c3 : (K == 2 || K == 6) ? c2 : c1;
        r.x = static_cast<T>(c);
        r.y = static_cast<T>(INV ? s : -s);
        return cmul(x, r);
    }
}

template <typename V2>
__device__ __forceinline__ void butterfly(V2& a, V2& b, V2 v) {
    const V2 u = a;
    a.x = u.x + v.x;
    a.y = u.y + v.y;
    b.x = u.x - v.x;
    b.y = u.y - v.y;
}

// Stage K of the first part on the R values x (bit-reversed order).
template <int R, int K, int J, bool INV, typename V2>
__device__ __forceinline__ void first_stage(V2* x) {
    if constexpr (J < R) {
        constexpr int h = 1 << K;
        if constexpr (!(J & h)) butterfly(x[J], x[J + h], rot16<((J & (h - 1)) << (3 - K)), INV>(x[J + h]));
        first_stage<R, K, J + 1, INV>(x);
    }
}

// First part: x[j] = value t + R2 j of the line, through the first stages and
// out to LDS.  `ls` is the distance in LDS between consecutive values of a
// line, `buf` the line's first value.  A barrier belongs between the two
// parts, and another before the buffer is written again.
template <int N, bool INV, typename V2>
__device__ __forceinline__ void reg_first(const V2 (&in)[RegPlan<N>::R1], V2* buf, int ls, int t) {
    using P = RegPlan<N>;
    V2 x[P::R1];
#pragma unroll
    for (int i = 0; i < P::R1; ++i) x[i] = in[rev_bits(i, P::S1)];
    first_stage<P::R1, 0, 0, INV>(x);
    first_stage<P::R1, 1, 0, INV>(x);
    first_stage<P::R1, 2, 0, INV>(x);
    if constexpr (P::S1 == 4) first_stage<P::R1, 3, 0, INV>(x);
    V2* row = buf + rev_bits(t, P::S2) * P::ROW * ls;
#pragma unroll
    for (int i = 0; i < P::R1; ++i) row[i * ls] = x[i];
}

// Second part: x[s R2 + g] = value t + R2 s + R1 g of the transform.  tw: the
// N / 2 twiddles exp(-2 pi i k / N) (staged in LDS).
template <int N, bool INV, typename V2>
__device__ __forceinline__ void reg_second(V2 (&x)[RegPlan<N>::R1], const V2* buf, int ls, const V2* tw, int t) {
    using P = RegPlan<N>;
#pragma unroll
    for (int s = 0; s < P::S; ++s) {
        const int i = t + P::R2 * s;
        V2* y = x + s * P::R2;
#pragma unroll
        for (int g = 0; g < P::R2; ++g) y[g] = buf[(g * P::ROW + i) * ls];
#pragma unroll
        for (int k = 0; k < P::S2; ++k) {
            const int h = 1 << k;
#pragma unroll
            for (int q = 0; q < h; ++q) {
                V2 w = tw[(i + q * P::R1) << (P::S2 - 1 - k)];
                if (INV) w.y = -w.y;
#pragma unroll
                for (int j = q; j < P::R2; j += 2 * h) butterfly(y[j], y[j + h], cmul(y[j + h], w));
            }
        }
    }
}

// Index along the line of register r before and after a transform.
template <int N>
__device__ __forceinline__ int reg_n(int t, int r) { return t + RegPlan<N>::R2 * r; }
template <int N>
__device__ __forceinline__ int reg_k(int t, int r) {
    using P = RegPlan<N>;
    return t + P::R2 * (r / P::R2) + P::R1 * (r % P::R2);
}
// Register of a finished transform that holds value t + R2 j, the start of
// the next one.
template <int N>
__device__ __forceinline__ constexpr int reg_of_n(int j) {
    using P = RegPlan<N>;
    return (j % P::S) * P::R2 + j / P::S;
}

// A load of data that is read once: it is not kept in the memory-side cache,
// which then holds more of what the passes write.  256^3 FP32 with the state
// of a jump read this way: the y passes that follow 43 -> 41 us, the x pass
// with the modes 248 -> 224; the pass itself keeps its time.
template <typename T>
__device__ __forceinline__ T load_once(const T* p) { return __builtin_nontemporal_load(p); }
template <>
__device__ __forceinline__ float2 load_once(const float2* p) {
    typedef float v2 __attribute__((ext_vector_type(2)));
    const v2 v = __builtin_nontemporal_load(reinterpret_cast<const v2*>(p));
    return make_float2(v.x, v.y);
}
template <>
__device__ __forceinline__ double2 load_once(const double2* p) {
    typedef double v2 __attribute__((ext_vector_type(2)));
    const v2 v = __builtin_nontemporal_load(reinterpret_cast<const v2*>(p));
    return make_double2(v.x, v.y);
}

// The N / 2 twiddle factors into LDS (every thread of the block takes part).
template <int N, typename V2>
__device__ __forceinline__ void reg_twiddles(V2* t, const V2* __restrict__ tw) {
    for (int i = threadIdx.x; i < N / 2; i += blockDim.x) t[i] = tw[i];
}

}  // namespace cl

#endif  // CL_FFT_REG_H
