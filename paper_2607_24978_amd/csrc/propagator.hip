// Linear propagation of the fluctuations over a jump, mode by mode.
//
// About a homogeneous background, the lattice equations of motion of
// Sect. 2.1 (Eq. singletEOM in program variables: f' = a^(alpha-3) pi,
// pi' = a^(1+alpha) Lap f - a^(3+alpha) dV/df) are linear in the
// fluctuations to first order, with the 7-point Laplacian diagonal in the
// lattice Fourier modes (eigenvalue -kappa^2, kappa^2 = sum_i (2/dx)^2
// sin^2(pi n_i / N)) and the mass matrix d^2V/df_i df_j at the homogeneous
// values.  Every mode then follows the integrator's own kick-drift-kick
// sub-steps with the background's (a, fbar) at each kick and drift, which
// the host takes from its FP64 background predictor.
//
// The propagation over a jump is linear with real coefficients that depend on
// a mode only through kappa^2, which is even in every index and symmetric in
// their order: one 2 nf x 2 nf transfer matrix per sorted triple of folded
// indices (about N^3 / 48) is built first, then applied to every mode.
//
// Layout: the 2 nf real channels of a site, in the order f_0..f_{nf-1},
// pi_0..pi_{nf-1}, are packed pairwise into nf complex arrays (channel 2q in
// the real and 2q+1 in the imaginary part of array q), each transformed with
// the line FFT; a mode's channels are recovered from the array at k and at
// -k (Hermitian symmetry of real fields).  The packing is fused with the
// forward z pass and the unpacking with the inverse z pass (the inverse runs
// x, y, z), so the state is read once and written once per jump.  The
// transforms run in the state's precision: FP32 lattices use float2 values,
// whose rounding (relative to the fluctuations, from which the means are
// removed) is far below that of the FP32 state itself.  The transfer matrices
// are formed in FP64 and rounded once to that precision, in which they act.
#include "fft_lds.h"
#include "fft_reg.h"
#include "internal.h"
#include "xcd_order.h"

#include <hip/hip_runtime.h>
#include <cstdint>
#include <type_traits>
#include <vector>

namespace cl {
namespace {

template <typename V2>
__device__ __forceinline__ V2 make_v2(double x, double y) {
    V2 v;
    v.x = static_cast<decltype(v.x)>(x);
    v.y = static_cast<decltype(v.y)>(y);
    return v;
}

// Element idx = l N + e of a batch of L consecutive rows starting at row0:
// channel c of site (row0 + l, z = e) in the row-interleaved state.
__device__ __forceinline__ size_t chan_index(size_t row0, int idx, int logN, int c, int na) {
    const size_t N = size_t{1} << logN;
    return ((row0 + (idx >> logN)) * na + c) * N + (idx & (N - 1));
}

// Fluctuations of channels 2q, 2q+1 of L rows -> LDS, bit-reversed along z
// (every global load of a thread before its LDS stores), forward z
// transform, out to z[q].  K = L N / 256 elements per thread (K = 1: L N <=
// 256, the rest of the threads idle).
template <typename T, typename V2, int K>
__global__ __launch_bounds__(256) void prop_pack_fftz(PropZArgs a) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    V2* buf = reinterpret_cast<V2*>(lds_raw);
    const int N = a.N, logN = a.logN, L = a.L, total = L * N;
    const int q = blockIdx.y, na = 2 * a.nf;
    const size_t row0 = static_cast<size_t>(blockIdx.x) * L;
    const T* st = static_cast<const T*>(a.state);
    const double m0 = a.mean[2 * q], m1 = a.mean[2 * q + 1];
    T re[K], im[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int idx = static_cast<int>(threadIdx.x) + k * 256;
        if (K > 1 || idx < total) {
            const size_t i = chan_index(row0, idx, logN, 2 * q, na);
            re[k] = st[i];
            im[k] = st[i + N];
        }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int idx = static_cast<int>(threadIdx.x) + k * 256;
        if (K > 1 || idx < total) {
            const int l = idx >> logN, e = idx & (N - 1);
            buf[slot(l, bitrev(e, logN), N)] =
                make_v2<V2>(static_cast<double>(re[k]) - m0, static_cast<double>(im[k]) - m1);
        }
    }
    const V2* tws = stage_twiddles(buf, static_cast<const V2*>(a.tw), N, L);
    __syncthreads();
    fft_lds_stages(buf, tws, logN, L, false);
    V2* out = static_cast<V2*>(a.z[q]) + row0 * N;
    for (int idx = threadIdx.x; idx < total; idx += blockDim.x) out[idx] = buf[slot(idx >> logN, idx & (N - 1), N)];
}

// Rows of z[q] -> LDS bit-reversed, inverse z transform, then the means
// added back and channels 2q, 2q+1 of the rows written to `out`.
template <typename T, typename V2, int K>
__global__ __launch_bounds__(256) void prop_ifftz_unpack(PropZArgs a) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    V2* buf = reinterpret_cast<V2*>(lds_raw);
    const int N = a.N, logN = a.logN, L = a.L, total = L * N;
    const int q = blockIdx.y, na = 2 * a.nf;
    const size_t row0 = static_cast<size_t>(blockIdx.x) * L;
    const V2* in = static_cast<const V2*>(a.z[q]) + row0 * N;
    V2 v[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int idx = static_cast<int>(threadIdx.x) + k * 256;
        if (K > 1 || idx < total) v[k] = in[idx];
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int idx = static_cast<int>(threadIdx.x) + k * 256;
        if (K > 1 || idx < total) buf[slot(idx >> logN, bitrev(idx & (N - 1), logN), N)] = v[k];
    }
    const V2* tws = stage_twiddles(buf, static_cast<const V2*>(a.tw), N, L);
    __syncthreads();
    fft_lds_stages(buf, tws, logN, L, true);
    T* st = static_cast<T*>(a.out);
    const double m0 = a.mean[2 * q], m1 = a.mean[2 * q + 1];
    for (int idx = threadIdx.x; idx < total; idx += blockDim.x) {
        const V2 w = buf[slot(idx >> logN, idx & (N - 1), N)];
        const size_t i = chan_index(row0, idx, logN, 2 * q, na);
        st[i] = static_cast<T>(m0 + w.x);
        st[i + N] = static_cast<T>(m1 + w.y);
    }
}

// The same two passes for N = 64, 128 or 256 on the register transform
// (fft_reg.h), R2 threads per line: bound by HBM, 256^3 two fields FP32 97
// and 100 us (537 MB each, 5.5 TB/s; 107 and 106 with the passes over LDS
// above).  The unpacking goes through LDS once more for 16-byte stores
// (135 us with 4-byte ones).
template <typename T, typename V2, int N>
__global__ __launch_bounds__(256) void prop_pack_fftz_reg(PropZArgs a) {
    using P = RegPlan<N>;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int t = threadIdx.x % P::R2, l = threadIdx.x / P::R2, lines = blockDim.x / P::R2;
    V2* buf = reinterpret_cast<V2*>(lds_raw);
    V2* tws = buf + lines * P::SLOTS;
    const int q = blockIdx.y, na = 2 * a.nf;
    const size_t row = static_cast<size_t>(blockIdx.x) * lines + l;
    const T* st = static_cast<const T*>(a.state) + (row * na + 2 * q) * N;
    const double m0 = a.mean[2 * q], m1 = a.mean[2 * q + 1];
    T re[P::R1], im[P::R1];
#pragma unroll
    for (int r = 0; r < P::R1; ++r) {
        re[r] = load_once(st + reg_n<N>(t, r));
        im[r] = load_once(st + N + reg_n<N>(t, r));
    }
    reg_twiddles<N>(tws, static_cast<const V2*>(a.tw));
    V2 x[P::R1];
#pragma unroll
    for (int r = 0; r < P::R1; ++r)
        x[r] = make_v2<V2>(static_cast<double>(re[r]) - m0, static_cast<double>(im[r]) - m1);
    reg_first<N, false>(x, buf + l * P::SLOTS, 1, t);
    __syncthreads();
    reg_second<N, false>(x, buf + l * P::SLOTS, 1, tws, t);
    V2* out = static_cast<V2*>(a.z[q]) + row * N;
#pragma unroll
    for (int r = 0; r < P::R1; ++r) out[reg_k<N>(t, r)] = x[r];
}

template <typename T, typename V2, int N>
__global__ __launch_bounds__(256) void prop_ifftz_unpack_reg(PropZArgs a) {
    using P = RegPlan<N>;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int t = threadIdx.x % P::R2, l = threadIdx.x / P::R2, lines = blockDim.x / P::R2;
    V2* buf = reinterpret_cast<V2*>(lds_raw);
    V2* tws = buf + lines * P::SLOTS;
    const int q = blockIdx.y, na = 2 * a.nf;
    const size_t row = static_cast<size_t>(blockIdx.x) * lines + l;
    const V2* in = static_cast<const V2*>(a.z[q]) + row * N;
    V2 x[P::R1];
#pragma unroll
    for (int r = 0; r < P::R1; ++r) x[r] = load_once(in + reg_n<N>(t, r));
    reg_twiddles<N>(tws, static_cast<const V2*>(a.tw));
    reg_first<N, true>(x, buf + l * P::SLOTS, 1, t);
    __syncthreads();
    reg_second<N, true>(x, buf + l * P::SLOTS, 1, tws, t);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < P::R1; ++r) buf[l * P::SLOTS + reg_k<N>(t, r)] = x[r];
    __syncthreads();
    // 16-byte stores: a thread takes V consecutive z of both channels
    constexpr int V = 16 / sizeof(T);
    typedef T TV __attribute__((ext_vector_type(V)));
    const double m0 = a.mean[2 * q], m1 = a.mean[2 * q + 1];
    T* st = static_cast<T*>(a.out);
    for (int i = threadIdx.x; i < lines * (N / V); i += blockDim.x) {
        const int li = i / (N / V), z = (i % (N / V)) * V;
        const V2* src = buf + li * P::SLOTS + z;
        T* dst = st + ((static_cast<size_t>(blockIdx.x) * lines + li) * na + 2 * q) * N + z;
        TV re, im;
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const V2 w = src[v];
            re[v] = static_cast<T>(m0 + w.x);
            im[v] = static_cast<T>(m1 + w.y);
        }
        *reinterpret_cast<TV*>(dst) = re;
        *reinterpret_cast<TV*>(dst + N) = im;
    }
}

// Index of a sorted triple i0 <= i1 <= i2 of folded mode indices (each in
// [0, N/2]): i2(i2+1)(i2+2)/6 + i1(i1+1)/2 + i0, dense in [0, C(N/2 + 3, 3)).
__device__ __forceinline__ size_t triple_index(size_t i0, size_t i1, size_t i2) {
    return i2 * (i2 + 1) * (i2 + 2) / 6 + i1 * (i1 + 1) / 2 + i0;
}

// The transfer matrix of the jump for kappa^2 = kap2[i0] + kap2[i1] +
// kap2[i2], one thread per sorted triple (a.triples lists them in index
// order, packed 10 bits each): the 2 NF x 2 NF real matrix that maps a mode's
// (f, pi) at the start to the end, built by applying every sub-step to the
// unit vectors (the same operations as on a mode's values; the columns are
// independent chains).  Layout T[row][col] with a stride of 16 per entry,
// rows and columns in the channel order f_0.., pi_0...
template <int NF, typename TT>
__global__ __launch_bounds__(256) void prop_transfer(PropModeArgs a) {
    constexpr int NC = 2 * NF;
    const size_t t = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= a.ntriples) return;
    const uint32_t tr = a.triples[t];
    const double kap2 = a.kap2[tr & 1023u] + a.kap2[(tr >> 10) & 1023u] + a.kap2[(tr >> 20) & 1023u];
    double F[NC][NF], P[NC][NF];  // [column][field]
#pragma unroll
    for (int col = 0; col < NC; ++col)
#pragma unroll
        for (int j = 0; j < NF; ++j) {
            F[col][j] = (col == j) ? 1.0 : 0.0;
            P[col][j] = (col == NF + j) ? 1.0 : 0.0;
        }
    // kick by (ck kappa^2 + M) of the half-kick coefficients (ck, m)
    auto kick = [&](double ck, double m0, double m1, double m2) {
        const double g0 = ck * kap2 + m0;
#pragma unroll
        for (int col = 0; col < NC; ++col) {
            if (NF == 1) {
                P[col][0] -= g0 * F[col][0];
            } else {
                const double g1 = ck * kap2 + m2;
                const double f0 = F[col][0], f1 = F[col][NF - 1];
                P[col][0] -= g0 * f0 + m1 * f1;
                P[col][NF - 1] -= g1 * f1 + m1 * f0;
            }
        }
    };
    // The closing half kick of a sub-step and the opening one of the next act
    // on the same F: one kick with their sum (49 kicks instead of 96 for a
    // jump of 16 VV4 steps).
    kick(a.steps[0].ck0, a.steps[0].m0[0], a.steps[0].m0[1], a.steps[0].m0[2]);
    for (int i = 0; i < a.nsteps; ++i) {
        const PropStep& c = a.steps[i];
#pragma unroll
        for (int col = 0; col < NC; ++col)
#pragma unroll
            for (int j = 0; j < NF; ++j) F[col][j] += c.cd * P[col][j];
        double ck = c.ck1, m0 = c.m1[0], m1 = c.m1[1], m2 = c.m1[2];
        if (i + 1 < a.nsteps) {
            const PropStep& n = a.steps[i + 1];
            ck += n.ck0;
            m0 += n.m0[0];
            m1 += n.m0[1];
            m2 += n.m0[2];
        }
        kick(ck, m0, m1, m2);
    }
    // stored in the lattice's precision (FP32 lattices: the matrices' rounding
    // is that of the FP32 transforms they act between), rounded once
    TT* T = static_cast<TT*>(a.table) + t * (NC * NC);
#pragma unroll
    for (int col = 0; col < NC; ++col)
#pragma unroll
        for (int j = 0; j < NF; ++j) {
            T[j * NC + col] = static_cast<TT>(F[col][j]);
            T[(NF + j) * NC + col] = static_cast<TT>(P[col][j]);
        }
}

// A pair of modes k, -k of every packed array through the transfer matrix: the
// channels X = (A(k) + conj A(-k)) / 2, Y = (A(k) - conj A(-k)) / (2 i) of each
// array A (Hermitian symmetry of real fields), then A'(k) = X' + i Y' and
// A'(-k) = conj X' + i conj Y', times sc.  (The halves, exact, go with sc.)
template <int NF, typename TS, typename V2>
__device__ __forceinline__ void mode_pair(const TS (&Tm)[4 * NF * NF], TS sc, V2 (&vk)[NF], V2 (&vm)[NF]) {
    constexpr int NC = 2 * NF;
    const TS hs = TS(0.5) * sc;
    TS cx[NC], cy[NC];
#pragma unroll
    for (int q = 0; q < NF; ++q) {
        const TS ux = vk[q].x, uy = vk[q].y, rx = vm[q].x, ry = vm[q].y;
        cx[2 * q] = ux + rx;
        cy[2 * q] = uy - ry;
        cx[2 * q + 1] = uy + ry;
        cy[2 * q + 1] = rx - ux;
    }
    TS ox[NC], oy[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        TS vx = TS(0), vy = TS(0);
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            const TS tij = Tm[i * NC + j];
            vx += tij * cx[j];
            vy += tij * cy[j];
        }
        ox[i] = vx;
        oy[i] = vy;
    }
#pragma unroll
    for (int q = 0; q < NF; ++q) {
        const TS xx = ox[2 * q], xy = oy[2 * q], yx = ox[2 * q + 1], yy = oy[2 * q + 1];
        vk[q].x = hs * (xx - yy);
        vk[q].y = hs * (xy + yx);
        vm[q].x = hs * (xx + yy);
        vm[q].y = hs * (yx - xy);
    }
}

// One thread per folded index triple (i0, i1, i2): the up to eight modes
// (+-i0, +-i1, +-i2) share kappa^2, hence the transfer matrix, and form up to
// four pairs (k, -k), each through mode_pair with the inverse transform's
// 1/N^3.  Every mode is read and written once (the planes i2 = 0 and N/2, which are their
// own mirrors, twice with the same values).  A thread issues the matrix's
// and all its pairs' loads before the first use.
template <int NF, typename V2>
__global__ __launch_bounds__(256) void prop_modes(PropModeArgs a) {
    constexpr int NC = 2 * NF;
    const int N = a.N;
    const size_t M = static_cast<size_t>(N) / 2 + 1;
    const size_t t = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= M * M * M) return;
    const int i2 = static_cast<int>(t % M), i1 = static_cast<int>((t / M) % M), i0 = static_cast<int>(t / (M * M));
    int s0 = i0, s1 = i1, s2 = i2;  // sorted copy for the table
    if (s0 > s1) { const int x = s0; s0 = s1; s1 = x; }
    if (s1 > s2) { const int x = s1; s1 = s2; s2 = x; }
    if (s0 > s1) { const int x = s0; s0 = s1; s1 = x; }
    // the matrix in the table's precision (FP32 for FP32 lattices), 16-byte loads
    constexpr bool F32 = std::is_same<V2, float2>::value;
    using TS = typename std::conditional<F32, float, double>::type;
    using TV = typename std::conditional<F32, float4, double2>::type;
    constexpr int TPV = sizeof(TV) / sizeof(TS);  // table values per load
    const TV* T2 = reinterpret_cast<const TV*>(static_cast<const TS*>(a.table) + triple_index(s0, s1, s2) * (NC * NC));
    TV Tv[NC * NC / TPV];
#pragma unroll
    for (int e = 0; e < NC * NC / TPV; ++e) Tv[e] = T2[e];
    // representatives (sx, sy, +) of the pairs; an index equal to its mirror
    // (0 or N/2) has one sign only
    const bool x1 = i0 == 0 || 2 * i0 == N, y1 = i1 == 0 || 2 * i1 == N;
    size_t k[4], m[4];
    bool on[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const int sx = p >> 1, sy = p & 1;
        on[p] = !(sx && x1) && !(sy && y1);
        const int kx = sx ? (N - i0) & (N - 1) : i0, ky = sy ? (N - i1) & (N - 1) : i1, kz = i2;
        k[p] = (static_cast<size_t>(kx) * N + ky) * N + kz;
        m[p] = (static_cast<size_t>((N - kx) & (N - 1)) * N + ((N - ky) & (N - 1))) * N + ((N - kz) & (N - 1));
    }
    V2 vk[4][NF], vm[4][NF];
#pragma unroll
    for (int p = 0; p < 4; ++p)
        if (on[p])
#pragma unroll
            for (int q = 0; q < NF; ++q) {
                vk[p][q] = static_cast<const V2*>(a.in[q])[k[p]];
                vm[p][q] = static_cast<const V2*>(a.in[q])[m[p]];
            }
    // the channel arithmetic in the table's precision: FP32 for FP32 lattices
    // (values and matrices are FP32 already; half the registers), FP64 else
    TS Tm[NC * NC];
#pragma unroll
    for (int e = 0; e < NC * NC / TPV; ++e) {
        const TS* tv = reinterpret_cast<const TS*>(&Tv[e]);
#pragma unroll
        for (int u = 0; u < TPV; ++u) Tm[TPV * e + u] = tv[u];
    }
    const TS sc = static_cast<TS>(a.scale);
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        if (!on[p]) continue;
        mode_pair<NF>(Tm, sc, vk[p], vm[p]);
#pragma unroll
        for (int q = 0; q < NF; ++q) {
            V2* o = static_cast<V2*>(a.out[q]);
            o[k[p]] = vk[p][q];
            o[m[p]] = vm[p][q];
        }
    }
}

// The modes of an FP32 lattice with N = 64, 128 or 256 together with the x
// transforms on either side of them: a workgroup takes 16 consecutive z in
// 1 .. N / 2 of one y (or 16 consecutive y of z = 0) and their mirrors (-y, -z),
// transforms both sets of lines of every packed array along x in registers,
// applies prop_modes' arithmetic to the pairs (k, -k) -- after a transform
// the mirror of a thread's value x is held by the same thread, if the
// mirrored lines' thread t works on the rows of thread -t -- and transforms
// back.  One sweep over the arrays instead of five (x, modes, inverse x on
// each array); out of place, since the lines of z = 0 and N / 2 are their own
// mirror plane and are taken (with equal results) by two workgroups.  The
// transfer matrices come from the table through the caches, one per mode.
// 256^3, two fields: 197 us against 381 for the separate passes; what is left
// is VALU issue (about 70 us) and memory (about 100) that hardly overlap with
// two workgroups per CU, the table (its next matrix is prefetched), and the
// last 9 of the 2057 workgroups, which follow four full rounds of 512 by
// themselves (27 us; the lines of z = 0 do not fit into the others' lanes).
template <int NF, int N, int L>
__global__ __launch_bounds__(L * RegPlan<N>::R2, 2) void prop_x_modes(PropModeArgs a) {
    using P = RegPlan<N>;
    constexpr int NC = 2 * NF, R = P::R1, hN = N / 2;
    __shared__ float2 bufA[P::SLOTS * L], bufB[P::SLOTS * L], tws[N / 2];
    __shared__ uint2 tri[hN + 1];  // i (i + 1) / 2 and i (i + 1) (i + 2) / 6
    const int l = threadIdx.x % L, t = threadIdx.x / L, tb = (P::R2 - t) & (P::R2 - 1);
    // Neighbouring groups of z on one XCD: A's lines straddle two groups'
    // 128-byte segments (B's do not), which its L2 then moves once.  The rows y
    // and N - y follow each other (0, -1, 1, -2, 2, ...): they use the same
    // matrices, 0.5 MB a row for N = 256, which the L2 then reads once for both
    // (256^3, two fields: 197 us, rows in order of y 221).
    constexpr int nzb = hN / L;
    const int b = xcd_order(blockIdx.x, gridDim.x);
    const bool column = b >= N * nzb;  // the last hN / L + 1 workgroups: z = 0, 16 consecutive y
    const int row = b / nzb;
    const int y = column ? (b - N * nzb) * L + l : row & 1 ? N - (row + 1) / 2 : row / 2;
    const int z = column ? 0 : (b % nzb) * L + l + 1;
    const int yb = (N - y) & (N - 1), zb = (N - z) & (N - 1);
    // 32-bit byte offsets from the (uniform) array bases; formed again for the
    // stores, so that no address stays in registers in between
    constexpr unsigned plane = 8u * N * N, step = P::R2 * plane;
    unsigned offA = t * plane + 8u * (y * N + z), offB = t * plane + 8u * (yb * N + zb);
    float2 A[NF][R], B[NF][R];
#pragma unroll
    for (int q = 0; q < NF; ++q) {
        const char* in = static_cast<const char*>(a.in[q]);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            A[q][r] = load_once(reinterpret_cast<const float2*>(in + (r * step + offA)));
            B[q][r] = load_once(reinterpret_cast<const float2*>(in + (r * step + offB)));
        }
    }
    reg_twiddles<N>(tws, static_cast<const float2*>(a.tw));
    for (unsigned i = threadIdx.x; i <= hN; i += blockDim.x)
        tri[i] = make_uint2(i * (i + 1) / 2, i * (i + 1) * (i + 2) / 6);
#pragma unroll
    for (int q = 0; q < NF; ++q) {
        if (q) __syncthreads();
        reg_first<N, false>(A[q], bufA + l, L, t);
        __builtin_amdgcn_sched_barrier(0);
        reg_first<N, false>(B[q], bufB + l, L, t);
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        reg_second<N, false>(A[q], bufA + l, L, tws, t);
        __builtin_amdgcn_sched_barrier(0);
        reg_second<N, false>(B[q], bufB + l, L, tws, tb);
        __builtin_amdgcn_sched_barrier(0);
    }
    // The mirror of A's register r is B's register R - 1 - r, except in
    // thread 0, whose rows are their own mirrors: there B's registers are
    // brought into that order, and back below.
    // (Selects: a branch around this many registers makes the compiler spill.)
    const bool own = t == 0;
    auto order = [&](float2 (&b)[R], auto there) {
        float2 c[R];
#pragma unroll
        for (int g = 0; g < P::R2; ++g) {
            // rows i = 0 (register g: x = R1 g) and, with two rows per
            // thread, i = R2 (register R2 + g, already mirrored by 7 - g)
            constexpr int hi = P::S == 2 ? P::R2 : 0;
            if constexpr (decltype(there)::value) {
                c[hi + g] = b[(g + 1) % P::R2];
                if (P::S == 2) c[g] = b[R - P::R2 + g];
            } else {
                c[(g + 1) % P::R2] = b[hi + g];
                if (P::S == 2) c[R - P::R2 + g] = b[g];
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            b[r].x = own ? c[r].x : b[r].x;
            b[r].y = own ? c[r].y : b[r].y;
        }
    };
#pragma unroll
    for (int q = 0; q < NF; ++q) {
        order(B[q], std::true_type{});
        __builtin_amdgcn_sched_barrier(0);
    }
    const unsigned fy = y <= hN ? y : N - y;
    const float sc = static_cast<float>(a.scale);
    // Register r's matrix, triple_index of the sorted (fx, fy, z); the loads
    // of the next one go out before this one is used.
    const unsigned lo = min(fy, static_cast<unsigned>(z)), hi = max(fy, static_cast<unsigned>(z));
    auto matrix = [&](int r, float4 (&T)[NC * NC / 4]) {
        const int kx = reg_k<N>(t, r);
        const unsigned fx = kx <= hN ? kx : N - kx;
        const unsigned s1 = max(lo, min(fx, hi)), s2 = max(fx, hi);
        const unsigned at = tri[s2].y + tri[s1].x + min(fx, lo);
        const float4* Tm = static_cast<const float4*>(a.table) + at * (NC * NC / 4);
#pragma unroll
        for (int e = 0; e < NC * NC / 4; ++e) T[e] = Tm[e];
    };
    {
        float4 next[NC * NC / 4];
        matrix(0, next);
        static_for<R>([&](auto rc) {
            constexpr int r = decltype(rc)::value;
            float T[NC * NC];
#pragma unroll
            for (int e = 0; e < NC * NC / 4; ++e) {
                T[4 * e] = next[e].x;
                T[4 * e + 1] = next[e].y;
                T[4 * e + 2] = next[e].z;
                T[4 * e + 3] = next[e].w;
            }
            if constexpr (r + 1 < R) matrix(r + 1, next);
            __builtin_amdgcn_sched_barrier(0);
            float2 vk[NF], vm[NF];
#pragma unroll
            for (int q = 0; q < NF; ++q) {
                vk[q] = A[q][r];
                vm[q] = B[q][R - 1 - r];
            }
            mode_pair<NF>(T, sc, vk, vm);
#pragma unroll
            for (int q = 0; q < NF; ++q) {
                A[q][r] = vk[q];
                B[q][R - 1 - r] = vm[q];
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    }
#pragma unroll
    for (int q = 0; q < NF; ++q) {
        order(B[q], std::false_type{});
        __builtin_amdgcn_sched_barrier(0);
    }
    asm volatile("" : "+v"(offA), "+v"(offB));
#pragma unroll
    for (int q = 0; q < NF; ++q) {
        float2 u[R], v[R];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            u[j] = A[q][reg_of_n<N>(j)];
            v[j] = B[q][reg_of_n<N>(j)];
        }
        __syncthreads();
        reg_first<N, true>(u, bufA + l, L, t);
        __builtin_amdgcn_sched_barrier(0);
        reg_first<N, true>(v, bufB + l, L, tb);
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        reg_second<N, true>(u, bufA + l, L, tws, t);
        __builtin_amdgcn_sched_barrier(0);
        reg_second<N, true>(v, bufB + l, L, tws, t);
        __builtin_amdgcn_sched_barrier(0);
        char* out = static_cast<char*>(a.out[q]);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const unsigned k = (P::R2 * (r / P::R2) + P::R1 * (r % P::R2)) * plane;  // reg_k - t planes
            *reinterpret_cast<float2*>(out + (k + offA)) = u[r];
            *reinterpret_cast<float2*>(out + (k + offB)) = v[r];
        }
    }
}

template <typename T, typename V2, int K>
void launch_zk(bool inverse, const PropZArgs& a, dim3 grid, size_t lds, hipStream_t s) {
    if (inverse) hipLaunchKernelGGL((prop_ifftz_unpack<T, V2, K>), grid, dim3(256), lds, s, a);
    else hipLaunchKernelGGL((prop_pack_fftz<T, V2, K>), grid, dim3(256), lds, s, a);
}

template <typename T, typename V2, int N>
hipError_t launch_z_reg(bool inverse, const PropZArgs& a, hipStream_t s) {
    using P = RegPlan<N>;
    // 16 lines of 256 values (32 shorter ones) per workgroup, half in FP64
    constexpr int threads = sizeof(V2) == 8 ? 256 : 128, lines = threads / P::R2;
    const dim3 grid(N * N / lines, a.nf);
    constexpr size_t lds = (static_cast<size_t>(lines) * P::SLOTS + N / 2) * sizeof(V2);
    if (inverse) hipLaunchKernelGGL((prop_ifftz_unpack_reg<T, V2, N>), grid, dim3(threads), lds, s, a);
    else hipLaunchKernelGGL((prop_pack_fftz_reg<T, V2, N>), grid, dim3(threads), lds, s, a);
    return hipGetLastError();
}

// K = L N / 256 exactly (L N a power of two), or 1 for L N <= 256
template <typename T, typename V2>
hipError_t launch_z(bool inverse, const PropZArgs& a, hipStream_t s) {
    if (a.N == 256) return launch_z_reg<T, V2, 256>(inverse, a, s);
    if (a.N == 128) return launch_z_reg<T, V2, 128>(inverse, a, s);
    if (a.N == 64) return launch_z_reg<T, V2, 64>(inverse, a, s);
    const int total = a.L * a.N;
    const dim3 grid(static_cast<unsigned>(a.N) * a.N / a.L, a.nf);
    const size_t lds = fft_lds_bytes(a.N, a.L, sizeof(V2));
    switch (total) {
        case 2048: launch_zk<T, V2, 8>(inverse, a, grid, lds, s); break;
        case 1024: launch_zk<T, V2, 4>(inverse, a, grid, lds, s); break;
        case 512: launch_zk<T, V2, 2>(inverse, a, grid, lds, s); break;
        default: launch_zk<T, V2, 1>(inverse, a, grid, lds, s); break;
    }
    return hipGetLastError();
}

// Completes the z-pass shape (log2 N, rows per workgroup) and checks it: N a
// power of two <= 1024, L N <= 2048 elements (K <= 8 per thread).  z lines
// are contiguous, so both precisions take 2048-element batches (for float2
// half the LDS of the axis passes' batches, more workgroups per CU: measured
// faster than 4096 at 256^3).
bool z_shape(PropZArgs& a) {
    if (a.N < 2 || a.N > 1024 || (a.N & (a.N - 1)) != 0 || (a.nf != 1 && a.nf != 2)) return false;
    a.logN = 0;
    while ((1 << a.logN) < a.N) ++a.logN;
    a.L = fft_lines_per_block(a.N);
    return a.L * a.N <= 2048;
}

}  // namespace

hipError_t launch_prop_pack_fftz(const PropZArgs& args, bool fp32, hipStream_t s) {
    PropZArgs a = args;
    if (!z_shape(a)) return hipErrorInvalidValue;
    return fp32 ? launch_z<float, float2>(false, a, s) : launch_z<double, double2>(false, a, s);
}

hipError_t launch_prop_ifftz_unpack(const PropZArgs& args, bool fp32, hipStream_t s) {
    PropZArgs a = args;
    if (!z_shape(a)) return hipErrorInvalidValue;
    return fp32 ? launch_z<float, float2>(true, a, s) : launch_z<double, double2>(true, a, s);
}

size_t prop_table_entries(int N) {
    const size_t M = static_cast<size_t>(N) / 2 + 1;
    return M * (M + 1) * (M + 2) / 6;
}

std::vector<uint32_t> prop_triples(int N) {
    const uint32_t M = static_cast<uint32_t>(N) / 2 + 1;
    std::vector<uint32_t> out;
    out.reserve(prop_table_entries(N));
    for (uint32_t c = 0; c < M; ++c)
        for (uint32_t b = 0; b <= c; ++b)
            for (uint32_t a = 0; a <= b; ++a) out.push_back(a | (b << 10) | (c << 20));
    return out;
}

bool prop_modes_with_x(int N, bool fp32) { return fp32 && reg_fft_size(N); }

namespace {
template <int NF, int N, int L>
void launch_x_modes_n(const PropModeArgs& a, hipStream_t s) {
    // groups of L z, and of L y at z = 0
    const dim3 grid(N * (N / 2 / L) + N / 2 / L + 1), block(L * RegPlan<N>::R2);
    hipLaunchKernelGGL((prop_x_modes<NF, N, L>), grid, block, 0, s, a);
}
template <int NF>
void launch_x_modes(const PropModeArgs& a, hipStream_t s) {
    if (a.N == 256) launch_x_modes_n<NF, 256, 16>(a, s);
    else if (a.N == 128) launch_x_modes_n<NF, 128, 16>(a, s);
    else launch_x_modes_n<NF, 64, 16>(a, s);
}
}  // namespace

hipError_t launch_prop_modes(const PropModeArgs& a, bool fp32, hipStream_t s) {
    if (a.nf != 1 && a.nf != 2) return hipErrorInvalidValue;
    const bool with_x = prop_modes_with_x(a.N, fp32);
    if (with_x && !a.tw) return hipErrorInvalidValue;
    const unsigned tgrid = static_cast<unsigned>((a.ntriples + 255) / 256);
    const size_t M = a.N / 2 + 1;
    const unsigned mgrid = static_cast<unsigned>((M * M * M + 255) / 256);
    if (a.nf == 1) {
        if (fp32) {
            hipLaunchKernelGGL((prop_transfer<1, float>), dim3(tgrid), dim3(256), 0, s, a);
            if (with_x) launch_x_modes<1>(a, s);
            else hipLaunchKernelGGL((prop_modes<1, float2>), dim3(mgrid), dim3(256), 0, s, a);
        } else {
            hipLaunchKernelGGL((prop_transfer<1, double>), dim3(tgrid), dim3(256), 0, s, a);
            hipLaunchKernelGGL((prop_modes<1, double2>), dim3(mgrid), dim3(256), 0, s, a);
        }
    } else {
        if (fp32) {
            hipLaunchKernelGGL((prop_transfer<2, float>), dim3(tgrid), dim3(256), 0, s, a);
            if (with_x) launch_x_modes<2>(a, s);
            else hipLaunchKernelGGL((prop_modes<2, float2>), dim3(mgrid), dim3(256), 0, s, a);
        } else {
            hipLaunchKernelGGL((prop_transfer<2, double>), dim3(tgrid), dim3(256), 0, s, a);
            hipLaunchKernelGGL((prop_modes<2, double2>), dim3(mgrid), dim3(256), 0, s, a);
        }
    }
    return hipGetLastError();
}

}  // namespace cl
