// kernels_mr.h -- passes for mixed-radix lengths with the plan fixed at
// compile time, FP32 and FP64 (the Y / Z column passes and the X real-line
// passes of the transpose-based 3D FFT, Sec. 2).
//
// A length N = N1 N2 (N1 <= N2 <= 42, every factor 2, 3, 5 or 7) is done in
// two Cooley-Tukey steps with input index n = q + N2 m and output index
// k = k1 + N1 k2 (q, k2 < N2; m, k1 < N1):
//     Y[q][k1]          = W_N^{q k1} sum_m x[q + N2 m] W_N1^{m k1}      (step 1)
//     X[k1 + N1 k2]     = sum_q Y[q][k1] W_N2^{q k2}                    (step 2)
// (MrTwoStep: FP64, and FP32 16, 48 .. 320, 360, 480.)  The other FP32 lengths
// (MrStaged) cut the runtime-radix kernels' own sequence of radices and twiddles
// into two or three such steps.  Each step is one in-register DFT per thread whose
// radix structure is fixed at compile time; the only exchange between threads is
// the LDS tile between the steps.  A C2C tile (the columns of one
// 128-byte workspace row block: 16 FP32, 8 FP64) reads its first step's inputs
// straight from global memory into registers and stores the last step's outputs
// straight from registers: one or two LDS round trips per tile, against one per
// radix stage plus the staging of the load and the store in the runtime-radix
// kernels.  Lanes run along the columns of the tile on both sides.
//
// Bound by the HBM traffic of the pass; measured against the runtime-radix
// kernels, which staged the tile in LDS and read their twiddles per radix stage
// (ms per R2C + C2R pair): FP64 300 x 280 x 250 0.675 -> 0.365 (Y pass 2.55 ->
// 6.0 TB/s), FP64 600 x 400 x 450 3.95 -> 2.20, FP32 768 x 768 x 384 3.27 ->
// 2.37, FP32 384^3 in natural order 0.897 -> 0.616, FP32 36 x 20 x 24 0.049 ->
// 0.020 (8.2 against 2.9 us per pass on the device).
//
// Long lengths exchange the real and the imaginary parts one after the other
// through half the LDS (MrShape::SPLIT), so that several workgroups still fit
// on a CU and one's loads overlap another's transform.
//
// The backward transform is the forward one on conjugated values, conj(F(conj
// x)): the C2C kernel takes the sign at run time (one multiplication by +-1
// per element on each side, exact), the backward X kernel conjugates in its
// Hermitian fill and its stores.
//
// The X passes carry two real lines as one complex line (a + i b), as the
// runtime-radix X kernels do; their loads and stores run along the points of
// the lines, and the real/complex split (forward) or the Hermitian fill
// (backward) goes through LDS.
#pragma once

#include <type_traits>
#include <utility>

#include "fft_device.h"
#include "pf_internal.h"

namespace pf {

extern __shared__ __align__(16) unsigned char pf_smem[];

// ---- cos / sin of 2 pi m / n, evaluated by the compiler -----------------------
// The angle is reduced exactly in integers to a quarter turn plus an angle in
// [0, pi/4] (folded by the complement) and summed by its Taylor series in
// double-double arithmetic (Dekker's error-free sum and product; 14 terms,
// truncation below 1e-30), then rounded once: the constants carry no error of
// their own beyond the final rounding, in either precision.
struct CtDd {
    double h, l;
};
constexpr CtDd ct_fast2(double a, double b) {
    const double s = a + b;
    return CtDd{s, b - (s - a)};
}
constexpr CtDd ct_add(CtDd a, CtDd b) {
    const double s = a.h + b.h, t = s - a.h;
    const double e = (a.h - (s - t)) + (b.h - t);
    return ct_fast2(s, e + (a.l + b.l));
}
constexpr CtDd ct_mul(CtDd a, CtDd b) {
    const double p = a.h * b.h;
    const double ca = 134217729.0 * a.h, ah = ca - (ca - a.h), al = a.h - ah;
    const double cb = 134217729.0 * b.h, bh = cb - (cb - b.h), bl = b.h - bh;
    const double e = ((ah * bh - p) + ah * bl + al * bh) + al * bl;
    return ct_fast2(p, e + (a.h * b.l + a.l * b.h));
}
constexpr CtDd ct_div(CtDd a, double d) {  // two quotient digits
    const double q = a.h / d;
    const CtDd r = ct_add(a, ct_mul(CtDd{-q, 0.0}, CtDd{d, 0.0}));
    return ct_fast2(q, (r.h + r.l) / d);
}
constexpr double ct_trig(int m, int n, bool want_sin) {
    const long long r = ((long long)m % n + n) % n;
    const long long q = (4 * r) / n;     // quarter turns
    const long long rr = 4 * r - q * n;  // rest: (pi / 2) rr / n
    const bool flip = 2 * rr > n;
    const CtDd half_pi{1.5707963267948966, 6.123233995736766e-17};
    const CtDd x = ct_div(ct_mul(half_pi, CtDd{(double)(flip ? n - rr : rr), 0.0}), (double)n);
    const CtDd x2 = ct_mul(x, x), mx2{-x2.h, -x2.l};
    CtDd ts = x, ss = x, tc{1.0, 0.0}, sc{1.0, 0.0};
    for (int i = 1; i <= 14; ++i) {
        ts = ct_div(ct_mul(ts, mx2), (2.0 * i) * (2.0 * i + 1.0));
        tc = ct_div(ct_mul(tc, mx2), (2.0 * i - 1.0) * (2.0 * i));
        ss = ct_add(ss, ts);
        sc = ct_add(sc, tc);
    }
    const double s0 = flip ? sc.h : ss.h, c0 = flip ? ss.h : sc.h;
    const double c = q == 0 ? c0 : q == 1 ? -s0 : q == 2 ? -c0 : s0;
    const double s = q == 0 ? s0 : q == 1 ? c0 : q == 2 ? -s0 : -c0;
    return want_sin ? s : c;
}
template <int N>
struct CtTable {  // cos and sin of 2 pi m / N, m < N
    double c[N], s[N];
    constexpr CtTable() : c(), s() {
        for (int m = 0; m < N; ++m) c[m] = ct_trig(m, N, false), s[m] = ct_trig(m, N, true);
    }
};
template <int N>
struct CtTrig {
    static constexpr CtTable<N> t{};
};

// ---- in-register forward DFT of any 7-smooth size (natural order in and out) ---
// Sizes 2, 3, 4, 5, 7, 8, 16 use the fixed kernels; any other N = A B runs B
// DFTs of size A over x[B n1 + n2], twiddles by W_N^{n2 k1}, and A DFTs of size
// B, output k1 + A k2.  Backward passes conjugate their inputs and outputs.
template <int N>
struct MrSplit {
    static constexpr int A = (N % 16 == 0 && N > 16) ? 16
                           : (N % 8 == 0 && N > 8)   ? 8
                           : (N % 4 == 0 && N > 4)   ? 4
                           : (N % 2 == 0)            ? 2
                           : (N % 3 == 0)            ? 3
                           : (N % 5 == 0)            ? 5
                                                     : 7;
    static constexpr int B = N / A;
};

// ---- rounding --------------------------------------------------------------------
// A complex product is two multiply-adds per part, each of which rounds one of
// its two products by itself.  Left to the compiler, which one depends on the
// code around it, and so on every later change of a kernel.  On a large grid that
// is visible: a few energetic modes (amplitude 1 over noise of 0.2 at 768 x 768 x
// 384) leak their lines' rounding into the weak modes of the same lines at 1e-3
// of the noise, the same amount for any choice but never the same error.  So the
// choice is written out: FP32 results stay what they were bit for bit, and a batch
// gives the same bits fused and serial in either precision.
__device__ __forceinline__ float mr_fma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double mr_fma(double a, double b, double c) { return __builtin_fma(a, b, c); }

// a w, w read from a table (a of FIRST: the imaginary part rounds a.y w.x)
template <typename T, bool FIRST>
__device__ __forceinline__ cx<T> mr_cmul(cx<T> a, cx<T> w) {
    cx<T> r;
    r.x = mr_fma(a.x, w.x, -(a.y * w.y));
    r.y = FIRST ? mr_fma(a.x, w.y, a.y * w.x) : mr_fma(a.y, w.x, a.x * w.y);
    return r;
}

// Where an in-register DFT of the two-step plans stands: step 1 of the X and of
// the C2C kernels, step 2.
enum { MR_X1 = 0, MR_C1 = 1, MR_S2 = 2 };

// Rotation by W_N^{n2 k1} between the A- and the B-point DFTs of an N-point one:
// bit 0, the real part rounds the product of a.x (else of a.y); bit 1, the
// imaginary part rounds the product of a.y (else of a.x).
constexpr int mr_rounds(int N, int A, int where, int n2, int k1) {
    const int m = n2 * k1;
    if (N == 24 && where == MR_S2) {  // 8 x 3
        if (m == 3) return 2;
        if (k1 == 2) return 1;
    }
    if (2 * m > N) return N == 20 ? 3 : 2;  // negative sine
    const bool mixed = (N == 12 || N == 20) && where == MR_S2 && 2 * k1 != A;
    return mixed || 4 * m > N || 8 * m == N || where == MR_C1 ? 1 : 0;
}

template <typename T, int ROUNDS>
__device__ __forceinline__ cx<T> mr_rot(cx<T> a, T c, T s) {
    cx<T> r;
    r.x = (ROUNDS & 1) ? mr_fma(a.y, s, a.x * c) : mr_fma(a.x, c, a.y * s);
    r.y = (ROUNDS & 2) ? mr_fma(a.x, -s, a.y * c) : mr_fma(a.y, c, -(a.x * s));
    return r;
}

// v sgn, sgn = +-1.  FP32: hidden from the compiler, which would otherwise fold the
// product into the sums around it.
__device__ __forceinline__ float mr_flip(float v, float sgn) {
    asm("" : "+v"(v));
    v *= sgn;
    asm("" : "+v"(v));
    return v;
}
__device__ __forceinline__ double mr_flip(double v, double sgn) { return v * sgn; }

// 8 and 16 points as in Dft<T, 8, -1> and Dft<T, 16, -1>, the rounding written out
// (both parts round the product of a.x, of a.y where the sine is negative; step 1 of the
// X kernels: the real part that of a.y, sqrt(1/2) aside)
template <typename T>
__device__ __forceinline__ void mr_dft8(cx<T> *v) {
    cx<T> e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6];
    cx<T> o0 = v[1], o1 = v[3], o2 = v[5], o3 = v[7];
    dft4<T, -1>(e0, e1, e2, e3);
    dft4<T, -1>(o0, o1, o2, o3);
    const T h = T(kSqrtHalf);
    o1 = mr_rot<T, 1>(o1, h, h);
    o2 = cmuli<-1>(o2);
    o3 = mr_rot<T, 1>(o3, -h, h);
    v[0] = cadd(e0, o0), v[4] = csub(e0, o0);
    v[1] = cadd(e1, o1), v[5] = csub(e1, o1);
    v[2] = cadd(e2, o2), v[6] = csub(e2, o2);
    v[3] = cadd(e3, o3), v[7] = csub(e3, o3);
}
template <typename T, bool X1>
__device__ __forceinline__ void mr_dft16(cx<T> *v) {
    cx<T> a[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int k = 0; k < 4; ++k) a[i][k] = v[i + 4 * k];
        dft4<T, -1>(a[i][0], a[i][1], a[i][2], a[i][3]);
    }
    const T c = T(kCosPi8), s = T(kSinPi8), h = T(kSqrtHalf);
    a[1][1] = mr_rot<T, X1 ? 0 : 1>(a[1][1], c, s);
    a[1][2] = mr_rot<T, 1>(a[1][2], h, h);
    a[1][3] = mr_rot<T, X1 ? 0 : 1>(a[1][3], s, c);
    a[2][1] = mr_rot<T, 1>(a[2][1], h, h);
    a[2][2] = cmuli<-1>(a[2][2]);
    a[2][3] = mr_rot<T, 1>(a[2][3], -h, h);
    a[3][1] = mr_rot<T, X1 ? 0 : 1>(a[3][1], s, c);
    a[3][2] = mr_rot<T, 1>(a[3][2], -h, h);
    a[3][3] = mr_rot<T, 2>(a[3][3], -c, -s);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        dft4<T, -1>(a[0][k], a[1][k], a[2][k], a[3][k]);
#pragma unroll
        for (int i = 0; i < 4; ++i) v[k + 4 * i] = a[i][k];
    }
}

template <int K>
using MrInt = std::integral_constant<int, K>;
// f(MrInt<0>()), ..., f(MrInt<K - 1>())
template <typename F, int... I>
__device__ __forceinline__ void mr_each(std::integer_sequence<int, I...>, F f) {
    (f(MrInt<I>()), ...);
}

template <typename T, int N, int WHERE>
struct DftMR {
    __device__ __forceinline__ static void run(cx<T> *v) {
        if constexpr (N == 1) {
        } else if constexpr (N == 2 || N == 3 || N == 4 || N == 5 || N == 7) {
            Dft<T, N, -1>::run(v);
        } else if constexpr (N == 8) {
            mr_dft8<T>(v);
        } else if constexpr (N == 16) {
            mr_dft16<T, WHERE == MR_X1>(v);
        } else {
            constexpr int A = MrSplit<N>::A, B = MrSplit<N>::B;
            static_assert(A * B == N && B > 1, "size must be 7-smooth");
            constexpr CtTable<N> tab = CtTrig<N>::t;
            cx<T> t[B][A];
#pragma unroll
            for (int n2 = 0; n2 < B; ++n2) {
#pragma unroll
                for (int n1 = 0; n1 < A; ++n1) t[n2][n1] = v[B * n1 + n2];
                DftMR<T, A, WHERE>::run(t[n2]);
            }
            mr_each(std::make_integer_sequence<int, (B - 1) * (A - 1)>(), [&](auto i) {
                constexpr int n2 = 1 + decltype(i)::value / (A - 1), k1 = 1 + decltype(i)::value % (A - 1);
                t[n2][k1] = mr_rot<T, mr_rounds(N, A, WHERE, n2, k1)>(t[n2][k1], (T)tab.c[(n2 * k1) % N],
                                                                      (T)tab.s[(n2 * k1) % N]);
            });
            mr_each(std::make_integer_sequence<int, A>(), [&](auto i) {
                constexpr int k1 = decltype(i)::value;
                cx<T> u[B];
#pragma unroll
                for (int n2 = 0; n2 < B; ++n2) u[n2] = t[n2][k1];
                // (18 = 2 x 9: the odd outputs' 9-point DFT rounds as the X kernels' do)
                DftMR<T, B, (N == 18 && WHERE == MR_C1 && k1 == 1) ? MR_X1 : WHERE>::run(u);
#pragma unroll
                for (int k2 = 0; k2 < B; ++k2) v[k1 + A * k2] = u[k2];
            });
        }
    }
};

// ---- lengths -----------------------------------------------------------------------
// Lengths with a compile-time plan and their factors N1 <= N2, the pair
// closest to sqrt(N): every 7-smooth length from 16 to 1024 whose larger
// factor is at most 42 (all but 343 = 7 x 49 and 686 = 14 x 49, whose 49-point
// step would not fit the registers in FP64).
struct MrLen {
    short n, n1, n2;
};
constexpr MrLen kMrLen[] = {
    {16, 4, 4}, {18, 3, 6}, {20, 4, 5}, {21, 3, 7}, {24, 4, 6}, {25, 5, 5}, {27, 3, 9}, {28, 4, 7},
    {30, 5, 6}, {32, 4, 8}, {35, 5, 7}, {36, 6, 6}, {40, 5, 8}, {42, 6, 7}, {45, 5, 9}, {48, 6, 8},
    {49, 7, 7}, {50, 5, 10}, {54, 6, 9}, {56, 7, 8}, {60, 6, 10}, {63, 7, 9}, {64, 8, 8}, {70, 7, 10},
    {72, 8, 9}, {75, 5, 15}, {80, 8, 10}, {81, 9, 9}, {84, 7, 12}, {90, 9, 10}, {96, 8, 12}, {98, 7, 14},
    {100, 10, 10}, {105, 7, 15}, {108, 9, 12}, {112, 8, 14}, {120, 10, 12}, {125, 5, 25}, {126, 9, 14},
    {128, 8, 16}, {135, 9, 15}, {140, 10, 14}, {144, 12, 12}, {147, 7, 21}, {150, 10, 15}, {160, 10, 16},
    {162, 9, 18}, {168, 12, 14}, {175, 7, 25}, {180, 12, 15}, {189, 9, 21}, {192, 12, 16}, {196, 14, 14},
    {200, 10, 20}, {210, 14, 15}, {216, 12, 18}, {224, 14, 16}, {225, 15, 15}, {240, 15, 16}, {243, 9, 27},
    {245, 7, 35}, {250, 10, 25}, {252, 14, 18}, {256, 16, 16}, {270, 15, 18}, {280, 14, 20}, {288, 16, 18},
    {294, 14, 21}, {300, 15, 20}, {315, 15, 21}, {320, 16, 20}, {324, 18, 18}, {336, 16, 21}, {350, 14, 25},
    {360, 18, 20}, {375, 15, 25}, {378, 18, 21}, {384, 16, 24}, {392, 14, 28}, {400, 20, 20}, {405, 15, 27},
    {420, 20, 21}, {432, 18, 24}, {441, 21, 21}, {448, 16, 28}, {450, 18, 25}, {480, 20, 24}, {486, 18, 27},
    {490, 14, 35}, {500, 20, 25}, {504, 21, 24}, {512, 16, 32}, {525, 21, 25}, {540, 20, 27}, {560, 20, 28},
    {567, 21, 27}, {576, 24, 24}, {588, 21, 28}, {600, 24, 25}, {625, 25, 25}, {630, 21, 30}, {640, 20, 32},
    {648, 24, 27}, {672, 24, 28}, {675, 25, 27}, {700, 25, 28}, {720, 24, 30}, {729, 27, 27}, {735, 21, 35},
    {750, 25, 30}, {756, 27, 28}, {768, 24, 32}, {784, 28, 28}, {800, 25, 32}, {810, 27, 30}, {840, 28, 30},
    {864, 27, 32}, {875, 25, 35}, {882, 21, 42}, {896, 28, 32}, {900, 30, 30}, {945, 27, 35}, {960, 30, 32},
    {972, 27, 36}, {980, 28, 35}, {1000, 25, 40}, {1008, 28, 36}, {1024, 32, 32},
};
constexpr int kMrCount = (int)(sizeof(kMrLen) / sizeof(kMrLen[0]));

// index of length n in the table, -1 if it has no compile-time plan
constexpr int mr_index(int n) {
    for (int i = 0; i < kMrCount; ++i)
        if (kMrLen[i].n == n) return i;
    return -1;
}


// FP32 lengths on a staged plan (MrStaged); the others take MrTwoStep.
constexpr bool mr_staged(int n) { return n > 16 && (n < 48 || n > 320) && n != 360 && n != 480; }

// A staged plan: the radices of the runtime-radix kernels (16s first, then 8, 4,
// 2, 3, 5, 7), cut into two or three groups of consecutive radices, one group
// per step.  Two steps where some cut leaves at most 32 points on either side (36
// above 640 points), else three: 33 .. 36 points need 131 registers, one
// workgroup per CU, where the tile would let two in (420 points, Y pass 3.7
// TB/s in two steps, 4.9 in three; 864 points, whose tile is halved anyway,
// 4.5 against 4.1).  Of the cuts the one with the smallest largest step, then
// with the largest first step, then the earliest.
struct MrStages {
    int steps, g[3];         // steps, points of each step
    int count[3], r[3][10];  // each step's radices, in order
};
constexpr MrStages mr_stages(int n) {
    int r[10] = {}, m = n, c = 0;
    for (int x : {16, 8, 4, 2, 3, 5, 7})
        for (; m % x == 0; m /= x) r[c++] = x;
    int c1 = 0, c2 = c, best = 1 << 30;
    for (int three = 0; three < 2 && best > (n > 640 ? 36 : 32) * 4096 + 4095; ++three) {
        best = 1 << 30;
        for (int i = 1; i < c; ++i)
            for (int j = three ? i + 1 : c; j < c + 1 - three; ++j) {
                int x = 1, y = 1, z = 1;
                for (int k = 0; k < c; ++k) (k < i ? x : k < j ? y : z) *= r[k];
                const int v = (x > y ? x > z ? x : z : y > z ? y : z) * 4096 + 1024 - x;
                if (v < best) best = v, c1 = i, c2 = j;
            }
    }
    MrStages s{};
    s.steps = c2 < c ? 3 : 2;
    for (int k = 0; k < 3; ++k) s.g[k] = 1;
    for (int k = 0; k < c; ++k) {
        const int q = k < c1 ? 0 : k < c2 ? 1 : 2;
        s.g[q] *= r[k];
        s.r[q][s.count[q]++] = r[k];
    }
    return s;
}

// ---- global accesses -------------------------------------------------------------
// A workgroup-uniform base pointer and a 32-bit byte offset per lane: one address
// register per access in flight instead of two, which is what bounds how many
// waves fit (18 x 20 in FP32: 114 registers with 64-bit addresses, 84 so).  The planner
// keeps passes whose tiles span 4 GB or more on the runtime-radix kernels.  The bases are qualified as global memory: they come from the
// plan's arguments or a batch's table, so the compiler cannot tell that they are
// not LDS, and would make flat accesses, which also take the LDS path and its
// wait counter.
#define PF_GLOBAL __attribute__((address_space(1)))
// v passed through an empty asm statement: what is derived from it is computed
// again instead of being held in registers from its first use on
__device__ __forceinline__ int mr_fresh(int v) {
    asm volatile("" : "+v"(v));
    return v;
}
template <typename T>
__device__ __forceinline__ cx<T> mr_ld(const void *base, unsigned off) {
    typedef T v2 __attribute__((ext_vector_type(2)));
    const v2 u = *(const PF_GLOBAL v2 *)((const PF_GLOBAL char *)base + off);
    return cmk<T>(u.x, u.y);
}
template <typename T>
__device__ __forceinline__ T mr_ld1(const void *base, unsigned off) {
    return *(const PF_GLOBAL T *)((const PF_GLOBAL char *)base + off);
}
// PIN (FP64 values that travelled LDS in halves): the parts pass through an empty
// asm statement first, so that they are not held as one 4-register value from
// the first half's arrival on (25 x 40 points: 260 registers spilled, 9 so)
template <typename T, bool PIN = false, bool NT = false>
__device__ __forceinline__ void mr_st(void *base, unsigned off, cx<T> v) {
    typedef T v2 __attribute__((ext_vector_type(2)));
    if constexpr (PIN && sizeof(T) == 8) asm volatile("" : "+v"(v.x), "+v"(v.y));
    const v2 u = {v.x, v.y};
    PF_GLOBAL v2 *p = (PF_GLOBAL v2 *)((PF_GLOBAL char *)base + off);
    if constexpr (NT) __builtin_nontemporal_store(u, p);
    else *p = u;
}
// 16 bytes, aligned: two FP32 values or one FP64 value
template <typename T>
__device__ __forceinline__ void mr_ld16(const void *base, unsigned off, cx<T> (&v)[16 / sizeof(cx<T>)]) {
    typedef T vv __attribute__((ext_vector_type(16 / sizeof(T))));
    const vv u = *(const PF_GLOBAL vv *)((const PF_GLOBAL char *)base + off);
#pragma unroll
    for (int i = 0; i < (int)(16 / sizeof(cx<T>)); ++i) v[i] = cmk<T>(u[2 * i], u[2 * i + 1]);
}
template <typename T>
__device__ __forceinline__ void mr_st16(void *base, unsigned off, const cx<T> (&v)[16 / sizeof(cx<T>)]) {
    typedef T vv __attribute__((ext_vector_type(16 / sizeof(T))));
    vv u;
#pragma unroll
    for (int i = 0; i < (int)(16 / sizeof(cx<T>)); ++i) u[2 * i] = v[i].x, u[2 * i + 1] = v[i].y;
    *(PF_GLOBAL vv *)((PF_GLOBAL char *)base + off) = u;
}
template <typename T, bool NT>
__device__ __forceinline__ void mr_st1(void *base, unsigned off, T v) {
    PF_GLOBAL T *p = (PF_GLOBAL T *)((PF_GLOBAL char *)base + off);
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// f(k, tw[j k]) for 0 < k < N, the loads H ahead of their uses: where the compiler keeps
// the order of the source, one load at a time waits out its latency N times (360 points,
// forward X pass in FP32: 56 us on 360 x 360 x 200, 45.5 with 8 ahead).  FP64 4 ahead still
// waits (400 points: 117 us on 400 x 256 x 288, 105 with 6).  The C2C kernels hide it: 0.
template <typename T, int N, int H, typename F>
__device__ __forceinline__ void mr_twiddles(const cx<T> *tw, int j, F f) {
    cx<T> w[N];
#pragma unroll
    for (int k = 1; k < N + H; ++k) {
        if (k < N) w[k] = mr_ld<T>(tw, j * k * sizeof(cx<T>));
        if (k > H) f(k - H, w[k - H]);
    }
}

// ---- plans ----------------------------------------------------------------------
// What a step does with the points of one item, held in registers: step<S>(v, j,
// tw), j the item's index among the N / G(S) items of the step.  Item j of step S
// reads the positions j + p N / G(S), p < G(S); K(S), the product of the earlier
// steps, splits j = k + K h; output o goes to position k + K (h G(S) + o).  tw: W_N^m.
template <typename T, int N1, int N2>
struct MrTwoStep {
    static constexpr bool BOUNDED = true;  // see MrShape::XWAVES
    static constexpr int N = N1 * N2, STEPS = 2;
    static constexpr int G(int s) { return s == 0 ? N1 : s == 1 ? N2 : 1; }
    template <int S, bool XPASS>
    __device__ __forceinline__ static void step(cx<T> *v, int j, const cx<T> *tw) {
        if constexpr (S == 0) {
            DftMR<T, N1, !XPASS ? MR_C1 : N == 256 ? MR_S2 : MR_X1>::run(v);
            mr_twiddles<T, N1, !XPASS ? 0 : sizeof(T) == 4 ? 8 : 6>(tw, j, [&](int k, cx<T> w) {
                v[k] = mr_cmul<T, (N == 16 || (XPASS && N == 256))>(v[k], w);
            });
        } else {
            DftMR<T, N2, MR_S2>::run(v);
        }
    }
};

// FP32: the radix plan and the twiddles of the runtime-radix kernels, which ran
// these lengths before and give the same bits: before a radix-R butterfly on
// sub-transforms of Ns points, input r of output k < Ns is turned by W_{Ns
// R}^{r k}.  In step 0 these are constants, later they are read from the table.
template <int N_>
struct MrStaged {
    static constexpr bool BOUNDED = false;
    static constexpr int N = N_;
    static constexpr MrStages P = mr_stages(N);
    static constexpr int STEPS = P.steps;
    static constexpr int G(int s) { return P.g[s]; }
    static constexpr int K(int s) { return s == 0 ? 1 : s == 1 ? P.g[0] : P.g[0] * P.g[1]; }
    // radix I of step S; L: the product of the step's radices before it
    template <int S, int I, int L>
    __device__ __forceinline__ static void radix(float2 *v, unsigned k, const float2 *tw) {
        constexpr int M = G(S), R = P.r[S][I], Q = N / (K(S) * L * R);
        float2 u[M];
        mr_each(std::make_integer_sequence<int, L>(), [&](auto lc) {
            constexpr int l = decltype(lc)::value;
            float2 w[R];
            if constexpr (S > 0) {
#pragma unroll
                for (int r = 1; r < R; ++r) w[r] = mr_ld<float>(tw, (k * (r * Q) + r * Q * K(S) * l) * 8);
            } else if constexpr (l > 0) {
                constexpr CtTable<L * R> tab = CtTrig<L * R>::t;
#pragma unroll
                for (int r = 1; r < R; ++r) w[r] = cmk<float>((float)tab.c[(r * l) % (L * R)], (float)-tab.s[(r * l) % (L * R)]);
            }
#pragma unroll
            for (int b = 0; b < M / (R * L); ++b) {
                float2 t[R];
#pragma unroll
                for (int r = 0; r < R; ++r) t[r] = v[b * L + l + r * (M / R)];
                if constexpr (S > 0 || l > 0) {
#pragma unroll
                    for (int r = 1; r < R; ++r) t[r] = mr_cmul<float, true>(t[r], w[r]);
                }
                DftMR<float, R, MR_S2>::run(t);
#pragma unroll
                for (int r = 0; r < R; ++r) u[b * L * R + l + r * L] = t[r];
            }
        });
#pragma unroll
        for (int i = 0; i < M; ++i) v[i] = u[i];
        if constexpr (I + 1 < P.count[S]) radix<S, I + 1, L * R>(v, k, tw);
    }
    template <int S, bool XPASS>
    __device__ __forceinline__ static void step(float2 *v, int j, const float2 *tw) {
        radix<S, 0, 1>(v, S == 0 ? 0 : S + 1 == STEPS ? j : j % K(S), tw);
    }
};

template <typename T, int I, bool STAGED>
struct MrPick {
    typedef MrTwoStep<T, kMrLen[I].n1, kMrLen[I].n2> type;
};
template <int I>
struct MrPick<float, I, true> {
    typedef MrStaged<kMrLen[I].n> type;
};
// plan of table position I in precision T
template <typename T, int I>
using MrPlan = typename MrPick<T, I, sizeof(T) == 4 && mr_staged(kMrLen[I].n)>::type;

// ---- tile geometry -----------------------------------------------------------
// Tiles above this many bytes go through LDS in two halves: up to 80 KB two
// workgroups still fit on a CU, and the halves' two more barriers cost more
// than a third workgroup brings (FP32 Y pass, whole against halves: 384 points, 50
// KB, 5.14 against 4.64 TB/s; 500 points, 64 KB, 4.84 against 4.68; 600 points, 77
// KB, 4.83 against 4.89 and its Z passes 4.11 / 4.26 against 3.97 / 4.15).  Longer
// tiles fit one workgroup only when whole.
constexpr int kMrSplitAbove = 81920;

// Backward X kernel: 16-byte row accesses of each line in flight per thread (all
// of them up to 8; 4 of 8 bytes measured 3.79 TB/s at 1000 points, 8 of 16 bytes
// 4.41; 768 points 4.09 -> 4.52)
constexpr int kMrRowLoads = 8;

// columns of one C2C tile: a 128-byte workspace row
template <typename T>
__host__ __device__ constexpr int mr_cols() {
    return 128 / (int)sizeof(cx<T>);
}
constexpr int mr_max(int a, int b) { return a > b ? a : b; }
constexpr int mr_min(int a, int b) { return a < b ? a : b; }
constexpr int mr_ceil(int a, int b) { return (a + b - 1) / b; }

// Threads per column of the C2C kernel.  Two steps: as many as the larger step
// has items, rounded up to whole waves (one step-0 item per thread; two items in
// half the threads measured slower where N2 >= 2 N1: FP64 length 250 = 10 x 25,
// forward Z pass 81 against 71 us at 300 x 280 x 250).  Three steps (FP32): 64,
// the fewest rounds of items (in place of 48, Y / forward Z pass, TB/s: 768 points
// 3.99 / 3.31 -> 4.57 / 4.23, 1008 points 3.70 / 3.09 -> 3.89 / 3.20), but 48 where
// the tile goes through LDS in halves and 48 take the first step in one round and
// the others in at most three: two workgroups then fit the registers (640 points
// 4.00 / 3.32 -> 4.82 / 4.44).
template <typename T, class P>
__host__ __device__ constexpr int mr_c2c_cols() {
    const int w = 64 / mr_cols<T>();
    if (P::STEPS == 2) return mr_ceil(mr_max(P::G(0), P::G(1)), w) * w;
    const int J1 = P::N / P::G(1), J2 = P::N / P::G(2);
    const bool split = 128 * P::G(0) * (P::N / P::G(0) | 1) > kMrSplitAbove;
    return split && P::N / P::G(0) <= 48 && mr_max(J1, J2) <= 3 * 48 ? 48 : 64;
}
// X kernels: line pairs per tile (a power of two; the lines' workspace rows
// are separate, so the tile width does not change the row accesses): 4, more
// where 4 pairs' step-0 items would not fill a wave, 2 where the tile would
// exceed 40 KB (FP64 lengths above 640; fewer than 4 workgroups per CU)
template <typename T, class P>
__host__ __device__ constexpr int mr_xp() {
    const int m = P::STEPS == 3 ? 16 : mr_max(P::G(0), P::G(1)), xp = m >= 16 ? 4 : m >= 8 ? 8 : 16;
    return xp == 4 && 4 * P::N * (int)sizeof(cx<T>) > 40960 ? 2 : xp;
}
constexpr int kMrRows = 32;  // lines of the widest X tile
// X kernels: pairs x the items of the larger step (three steps: the C2C kernel's threads per column), whole waves
template <typename T, class P>
__host__ __device__ constexpr int mr_x_threads() {
    const int items = P::STEPS == 3 ? mr_c2c_cols<T, P>() : mr_max(P::G(0), P::G(1));
    return mr_ceil(mr_xp<T, P>() * items, 64) * 64;
}

template <typename T, class P>
struct MrShape {
    static constexpr int N = P::N;
    static constexpr int C = mr_cols<T>();
    static constexpr int G0 = P::G(0), G1 = P::G(1), G2 = P::G(2);
    // first exchange: output o of item q at o P2 + q, P2 odd so that the reads of
    // consecutive items fall on different banks; the second one in natural order
    static constexpr int J0 = N / G0, P2 = J0 % 2 == 0 ? J0 + 1 : J0;
    // X passes: XP line pairs per tile, XTHREADS threads; one complex line per
    // pair at pitch SP (= 16 mod 32, >= N)
    static constexpr int XP = mr_xp<T, P>();
    static constexpr int XTHREADS = mr_x_threads<T, P>();
    // Wavefronts per SIMD that the X kernels leave registers for.  Two steps in FP32: the
    // larger step's points and 24 more; unbounded, forward 20 x 24 took 89 registers (5
    // wavefronts) and 77 us on 480 x 360 x 250, bounded 71 .. 73.  FP64: 20 x 20 took 184 (2)
    // and 110 us forward on 400 x 256 x 288, with 3 105; 30 x 30 264 (1) and 203 us on 900 x
    // 300 x 200, with 2 (10 spilled) 195.  The staged plans lose by a bound (they spill up to 78).
    static constexpr int XWAVES = sizeof(T) == 8 ? mr_max(G0, G1) <= 21 ? 3 : 2
                                  : P::BOUNDED   ? mr_min(7, 512 / ((2 * mr_max(G0, G1) + 31) / 8 * 8))
                                                 : 1;
    static constexpr int NXH = N / 2 + 1, NKB = (NXH + C - 1) / C;  // modes and column blocks of a line
    static constexpr int SP = N + ((16 - N % 32) % 32 + 32) % 32;
    static constexpr int XLDS = mr_max(XP * G0 * P2, XP * SP) * (int)sizeof(cx<T>);
    // C2C pass with a line side: line-major tile copy at pitch SPZ >= N, written
    // by lanes along the points and read by lanes along the columns (C columns x
    // 64 / C points per wave): the residue gives the reads of one LDS cycle (256
    // bytes) distinct banks
    static constexpr int pitch(int bytes) {  // of elements of that many bytes
        const int e = 256 / bytes;
        return N + ((e / C - N % e) % e + e) % e;
    }
    static constexpr bool SPLIT =
        mr_max(128 * G0 * P2, C * pitch(sizeof(cx<T>)) * (int)sizeof(cx<T>)) > kMrSplitAbove;
    static constexpr int SPZ = pitch(SPLIT ? sizeof(T) : sizeof(cx<T>));
    static constexpr int XCHB = 128 * G0 * P2 / (SPLIT ? 2 : 1);
    static constexpr int SPZB = C * SPZ * (int)sizeof(cx<T>) / (SPLIT ? 2 : 1);
    static constexpr int CLDS = mr_max(XCHB, SPZB);
    // C2C kernel: threads per column, threads, and the points that one 32-bit offset
    // of a row side spans (the rounds of items are added to the base)
    static constexpr int CT = mr_c2c_cols<T, P>();
    static constexpr int CTHREADS = C * CT;
    static constexpr int SPAN = P::STEPS == 2 ? mr_max(G0, G1) : CT;
};

// ---- launch arguments --------------------------------------------------------------
// 64 bytes, the whole kernel argument segment: a launch with a larger one costs
// the host 3.6 .. 4.0 us against 2.65 us, and passes of small grids (3 us each
// on the device) wait for the host.  Read in one piece, they also shorten a
// pass by 0.4 us (FP64 64^3 replayed from a graph 24.7 -> 22.2 us per pair).
// Strides are in elements; every one of a
// grid up to 8192^3 fits 32 bits.
enum : unsigned { MR_BACKWARD = 1, MR_IN_LINES = 2, MR_OUT_LINES = 4, MR_BATCH = 8, MR_IN_USER = 16, MR_OUT_USER = 32,
                MR_XCD = 64, MR_OUTER_FAST = 128, MR_NT_STORES = 256 };
struct MrArgs {
    const void *in;
    void *out;
    const void *tw;  // W_n^m, m < n (forward sign)
    union {
        // C2C: per side (i, o) the strides of the outer index, of a column block and
        // of a point (rows) or a column (lines)
        struct {
            unsigned isa, isb, iss, osa, osb, oss;
        } c;
        // X: rows of the workspace between z planes and column blocks, row of line
        // y = 0, lines per plane, lines
        struct {
            unsigned zrows, kbrows, y0, ny, lines;
        } x;
        // spectral step: strides of the workspace as in c, and the grid
        struct {
            unsigned sa, sb, ss, nx, ny;
        } s;
        // MR_BATCH: in, out are the caller's arrays; transform i owns workgroups
        // first[i] .. first[i + 1] - 1 and runs with table[i], whose in (MR_IN_USER)
        // or out (MR_OUT_USER) is a byte offset into them
        struct {
            const MrArgs *table;
            const long long *first;
        } b;
    };
    int C, CB;       // C2C: valid columns, column blocks
    unsigned flags;
    int count;       // MR_BATCH: transforms
};
static_assert(sizeof(MrArgs) == 64, "one 64-byte argument segment");

__device__ __forceinline__ int mr_find(const long long *first, int count, long long blk) {
    int lo = 0, hi = count - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (first[mid] <= blk) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Workgroup b of a launch of n, dealt to XCD b mod 8: its tile, so that each XCD
// works through n / 8 consecutive tiles (the last n mod 8 in place).
__device__ __forceinline__ unsigned mr_xcd_tile(unsigned b, unsigned n) {
    const unsigned per = n >> 3;
    return b < per * 8 ? (b & 7) * per + (b >> 3) : b;
}

// The transform of this workgroup and its tile (returned): m itself, or the
// batch entry with its pointers resolved.
__device__ __forceinline__ unsigned mr_resolve(const MrArgs &m, MrArgs &a) {
    a = m;
    if (m.flags & MR_XCD) return mr_xcd_tile(blockIdx.x, (unsigned)m.count);
    if (!(m.flags & MR_BATCH)) return blockIdx.x;
    const int i = mr_find(m.b.first, m.count, blockIdx.x);
    a = m.b.table[i];
    if (m.flags & MR_IN_USER) a.in = (const char *)m.in + (size_t)a.in;
    if (m.flags & MR_OUT_USER) a.out = (char *)m.out + (size_t)a.out;
    return (unsigned)(blockIdx.x - m.b.first[i]);
}

// ---- a trip through LDS ---------------------------------------------------------
// One step's values travel between threads: every thread puts its values,
// synchronises, and gets its new ones -- whole complex values, or (SPLIT) the
// real parts and then the imaginary parts through the same words.  put(w) /
// get(g) call w(slot, value) / g(slot, value) for each of the thread's values.
// Ends with the reads; the caller synchronises before LDS is written again.
template <typename T, bool SPLIT, typename PUT, typename GET>
__device__ __forceinline__ void mr_trip(PUT put, GET get) {
    if constexpr (SPLIT) {
        T *lds = reinterpret_cast<T *>(pf_smem);
        put([&](int i, const cx<T> &v) { lds[i] = v.x; });
        __syncthreads();
        get([&](int i, cx<T> &v) { v.x = lds[i]; });
        __syncthreads();
        put([&](int i, const cx<T> &v) { lds[i] = v.y; });
        __syncthreads();
        get([&](int i, cx<T> &v) { v.y = lds[i]; });
    } else {
        cx<T> *lds = reinterpret_cast<cx<T> *>(pf_smem);
        put([&](int i, const cx<T> &v) { lds[i] = v; });
        __syncthreads();
        get([&](int i, cx<T> &v) { v = lds[i]; });
    }
}

template <typename T, int I, int K, bool ON>
__device__ __forceinline__ void mr_zero(cx<T> (&v)[I][K]) {
    if constexpr (ON) {
#pragma unroll
        for (int it = 0; it < I; ++it)
#pragma unroll
            for (int i = 0; i < K; ++i) v[it][i] = cmk<T>(T(0), T(0));
    }
}
// f(it, j) for the items j = j0 + it STEP < J of a thread, it < I
template <int J, int STEP, int I, typename F>
__device__ __forceinline__ void mr_items(int j0, F f) {
#pragma unroll
    for (int it = 0; it < I; ++it) {
        const int j = j0 + it * STEP;
        if (j < J) f(it, j);
    }
}

// One tile of the C2C pass: column block cb of outer index ta.
// CT threads per column, each with up to I items of a step.
template <typename T, class P, int CT>
__device__ __forceinline__ void mr_c2c_body(const MrArgs &a, unsigned ta, unsigned cb) {
    using S = MrShape<T, P>;
    constexpr int N = S::N, C = S::C, G0 = S::G0, G1 = S::G1, G2 = S::G2;
    constexpr int J0 = N / G0, J1 = N / G1, J2 = N / G2;  // items of the steps
    constexpr int I0 = mr_ceil(J0, CT), I1 = mr_ceil(J1, CT), I2 = mr_ceil(J2, CT);
    constexpr int NT = C * CT;
    constexpr int ITEMS = (C * N + NT - 1) / NT;  // tile points per thread
    constexpr unsigned CS = sizeof(cx<T>);
    const int tid = threadIdx.x;
    const int c = tid & (C - 1), j = tid / C;
    const int ncol = a.C - (int)cb * C;  // valid columns of the tile (may exceed C)
    const bool cv = c < ncol;
    const T sgn = (a.flags & MR_BACKWARD) ? T(-1) : T(1);
    const cx<T> *tw = reinterpret_cast<const cx<T> *>(a.tw);
    const cx<T> *in = reinterpret_cast<const cx<T> *>(a.in) + (size_t)ta * a.c.isa + (size_t)cb * a.c.isb;
    cx<T> *out = reinterpret_cast<cx<T> *>(a.out) + (size_t)ta * a.c.osa + (size_t)cb * a.c.osb;
    // a side whose columns are whole lines (points contiguous) goes through a
    // line-major LDS copy of the tile, so that its global accesses run along
    // the points; a row side is read / written by the first / last step's threads
    const bool in_lines = (a.flags & MR_IN_LINES) != 0;
    const bool out_lines = (a.flags & MR_OUT_LINES) != 0;
    // step 0: the points q + J0 m of column c (arrays zeroed before conditional
    // fills, SPLIT aside: the compiler otherwise keeps FP64 ones in scratch memory)
    cx<T> x[I0][G0];
    mr_zero<T, I0, G0, !S::SPLIT>(x);
    if (in_lines) {
        cx<T> r[ITEMS];
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const int f = tid + i * NT;
            const int cc = f / N, p = f - cc * N;
            r[i] = cmk<T>(T(0), T(0));
            if (f < C * N && cc < ncol) r[i] = mr_ld<T>(in, ((unsigned)cc * a.c.iss + p) * CS);
        }
        mr_trip<T, S::SPLIT>(
            [&](auto w) {
                const int tid = mr_fresh(threadIdx.x);
#pragma unroll
                for (int i = 0; i < ITEMS; ++i) {
                    const int f = tid + i * NT;
                    const int cc = f / N, p = f - cc * N;
                    if (f < C * N) w(cc * S::SPZ + p, r[i]);
                }
            },
            [&](auto g) {
                mr_items<J0, CT, I0>(j, [&](int it, int q) {
#pragma unroll
                    for (int m = 0; m < G0; ++m) g(c * S::SPZ + q + J0 * m, x[it][m]);
                });
            });
    } else {
        const unsigned off = ((unsigned)j * a.c.iss + c) * CS;
#pragma unroll
        for (int it = 0; it < I0; ++it) {
            if (j + it * CT < J0 && cv) {
#pragma unroll
                for (int m = 0; m < G0; ++m) x[it][m] = mr_ld<T>(in + (size_t)(it * CT + m * J0) * a.c.iss, off);
            }
        }
    }
    mr_items<J0, CT, I0>(j, [&](int it, int q) {
#pragma unroll
        for (int m = 0; m < G0; ++m) x[it][m].y = mr_flip(x[it][m].y, sgn);
        P::template step<0, false>(x[it], q, tw);
    });
    if (in_lines) __syncthreads();  // the staged lines are read before the exchange tile overwrites them
    cx<T> y[I1][G1];
    mr_zero<T, I1, G1, !S::SPLIT>(y);
    mr_trip<T, S::SPLIT>(
        [&](auto w) {
            mr_items<J0, CT, I0>(j, [&](int it, int q) {
#pragma unroll
                for (int o = 0; o < G0; ++o) w((o * S::P2 + q) * C + c, x[it][o]);
            });
        },
        [&](auto g) {
            mr_items<J1, CT, I1>(j, [&](int it, int i) {  // position i + p J1, J1 = G0 G2
                const int o = G2 == 1 ? i : i % G0, q = G2 == 1 ? 0 : i / G0;
#pragma unroll
                for (int p = 0; p < G1; ++p) g((o * S::P2 + q + p * G2) * C + c, y[it][p]);
            });
        });
    mr_items<J1, CT, I1>(j, [&](int it, int i) { P::template step<1, false>(y[it], i, tw); });
    // the last step's values v, output i + J o of item i
    auto put = [&](auto &v, auto jc, auto ic) {
        constexpr int J = decltype(jc)::value, I = decltype(ic)::value, G = N / J;
        if (out_lines) {
            __syncthreads();  // the exchange tile is read before the line-major copy overwrites it
            cx<T> r[1][ITEMS];
            mr_zero<T, 1, ITEMS, !S::SPLIT>(r);
            mr_trip<T, S::SPLIT>(
                [&](auto w) {
                    mr_items<J, CT, I>(j, [&](int it, int i) {
#pragma unroll
                        for (int o = 0; o < G; ++o) w(c * S::SPZ + i + J * o, v[it][o]);
                    });
                },
                [&](auto g) {
                    const int tid = mr_fresh(threadIdx.x);
#pragma unroll
                    for (int i = 0; i < ITEMS; ++i) {
                        const int f = tid + i * NT;
                        const int cc = f / N, p = f - cc * N;
                        if (f < C * N) g(cc * S::SPZ + p, r[0][i]);
                    }
                });
            const int tid = mr_fresh(threadIdx.x);
            auto store = [&](auto nt) {
#pragma unroll
                for (int i = 0; i < ITEMS; ++i) {
                    const int f = tid + i * NT;
                    const int cc = f / N, p = f - cc * N;
                    if (f < C * N && cc < ncol)
                        mr_st<T, S::SPLIT, decltype(nt)::value>(out, ((unsigned)cc * a.c.oss + p) * CS,
                                                                cmk<T>(r[0][i].x, mr_flip(r[0][i].y, sgn)));
                }
            };
            // FP64 tiles in halves have no room for two copies of the stores: with both, 960
            // points took 79 / 85 us forward / backward in place of 65 / 63 (60 x 300 x 960)
            // and 1000 and 1008 points spilled 14 and 2 registers in place of 9 and none, for
            // 1% at 768 points
            if constexpr (S::SPLIT && sizeof(T) == 8) store(std::false_type());
            else if (a.flags & MR_NT_STORES) store(std::true_type());
            else store(std::false_type());
        } else {
            const unsigned off = ((unsigned)j * a.c.oss + c) * CS;
#pragma unroll
            for (int it = 0; it < I; ++it) {
                if (j + it * CT < J && cv) {
#pragma unroll
                    for (int o = 0; o < G; ++o)
                        mr_st<T, S::SPLIT>(out + (size_t)(it * CT + o * J) * a.c.oss, off,
                                           cmk<T>(v[it][o].x, mr_flip(v[it][o].y, sgn)));
                }
            }
        }
    };
    if constexpr (P::STEPS == 2) {
        put(y, MrInt<J1>(), MrInt<I1>());
    } else {
        __syncthreads();  // the first exchange is read before the second overwrites it
        cx<T> z[I2][G2];
        mr_zero<T, I2, G2, !S::SPLIT>(z);
        mr_trip<T, S::SPLIT>(
            [&](auto w) {
                mr_items<J1, CT, I1>(j, [&](int it, int i) {
                    const int k = i % G0, h = i / G0;
#pragma unroll
                    for (int o = 0; o < G1; ++o) w((k + G0 * (h * G1 + o)) * C + c, y[it][o]);
                });
            },
            [&](auto g) {
                mr_items<J2, CT, I2>(j, [&](int it, int i) {
#pragma unroll
                    for (int p = 0; p < G2; ++p) g((i + J2 * p) * C + c, z[it][p]);
                });
            });
        mr_items<J2, CT, I2>(j, [&](int it, int i) { P::template step<2, false>(z[it], i, tw); });
        put(z, MrInt<J2>(), MrInt<I2>());
    }
}

// ---- spectral step along z (Chebyshev third transform), in place on the workspace --
// One tile (ky line ta, column block cb) of the step's z part: the type-I DCT of
// the nz = N / 2 + 1 rows (the N-point DFT of their even extension), the product
// with m = i mu, mu = -scale kx' / (kx'^2 + ky'^2 + kz'^2) (conj(m) with
// MR_BACKWARD, the adjoint), mu = 0 at k = 0, and the DFT of the product, again
// an even sequence, whose first nz points are the backward type-I DCT.  kx' = 2
// pi kx / nx, ky' = 2 pi ky / ny (ky signed), kz' = 2 pi kz / N.  The adjoint's
// end-node weights (1 at z = 0 and nz - 1, 2 inside) divide the rows on load and
// multiply them on store (they act along z alone, so they commute with X and
// Y).  The second DFT takes its factors in the other order, so that its step 1
// (N2 points, k1 + N1 k2) finds its inputs in the registers where the first one's
// step 2 left them: two trips through LDS for both.  The multiplier and the product
// with it are computed in FP64 for either precision and rounded once.
// Replaces a chain of Z pass, product, Z pass (and two weight passes of the
// adjoint), each over the whole array: the step and its adjoint at 320 x 300 x
// 181 took 768 us in FP32 and 1800 us in FP64, now 356 .. 369 and 615 .. 626; 24 x
// 70 x 71, 16 launches, 100 and 92 us, now 10 launches, 34 and 35 us.  The FP32
// extensions that are powers of two from 256 on stay on the power-of-two kernels:
// 512 x 512 x 257 takes 1.24 ms there (split DCT, 0.18 ms) against 1.51 here (0.33).
template <typename T, int N1, int N2>
__device__ __forceinline__ void mr_spec_body(const MrArgs &a, unsigned ta, unsigned cb) {
    using S = MrShape<T, MrTwoStep<T, N1, N2>>;
    constexpr int N = S::N, C = S::C, NZ = N / 2 + 1;
    static_assert(N % 2 == 0, "an even extension");
    constexpr unsigned CS = sizeof(cx<T>);
    const int tid = threadIdx.x;
    const int c = tid & (C - 1), j = tid / C;
    const int kx = (int)cb * C + c;
    const bool cv = kx <= (int)a.s.nx / 2, adj = (a.flags & MR_BACKWARD) != 0;
    const cx<T> *tw = reinterpret_cast<const cx<T> *>(a.tw);
    cx<T> *w = reinterpret_cast<cx<T> *>(a.out) + (size_t)ta * a.s.sa + (size_t)cb * a.s.sb;
    cx<T> x0[1][N1], y0[1][N2], *x = x0[0], *y = y0[0];
#pragma unroll
    for (int m = 0; m < N1; ++m) x[m] = cmk<T>(T(0), T(0));
    if (j < N2 && cv) {
#pragma unroll
        for (int m = 0; m < N1; ++m) {
            const int p = j + N2 * m, row = p < NZ ? p : N - p;
            x[m] = mr_ld<T>(w, ((unsigned)row * a.s.ss + c) * CS);
        }
    }
    if (j < N2) {
        if (adj) {
#pragma unroll
            for (int m = 0; m < N1; ++m) {
                const int p = j + N2 * m;
                x[m] = cscale(x[m], p == 0 || p == N / 2 ? T(1) : T(0.5));
            }
        }
        DftMR<T, N1, MR_X1>::run(x);
        mr_twiddles<T, N1, sizeof(T) == 4 ? 8 : 0>(tw, j, [&](int k, cx<T> w) { x[k] = cmul(x[k], w); });
    }
    mr_zero<T, 1, N2, !S::SPLIT>(y0);
    mr_trip<T, S::SPLIT>(
        [&](auto wr) {
            if (j < N2) {
#pragma unroll
                for (int k1 = 0; k1 < N1; ++k1) wr((k1 * S::P2 + j) * C + c, x[k1]);
            }
        },
        [&](auto g) {
            if (j < N1) {
#pragma unroll
                for (int q = 0; q < N2; ++q) g((j * S::P2 + q) * C + c, y[q]);
            }
        });
    if (j < N1) {  // first DFT, step 2: outputs k = j + N1 k2; product; second DFT, step 1
        DftMR<T, N2, MR_S2>::run(y);
        const double two_pi = 6.283185307179586476925286766559;
        const int kys = 2 * ta <= a.s.ny ? (int)ta : (int)ta - (int)a.s.ny;
        const double kxr = two_pi * kx / (int)a.s.nx, kyr = two_pi * kys / (int)a.s.ny, kxy = kxr * kxr + kyr * kyr;
        const double num = (adj ? kxr : -kxr) / ((double)a.s.nx * a.s.ny * N), dz = two_pi / N;
#pragma unroll
        for (int k2 = 0; k2 < N2; ++k2) {
            const int k = j + N1 * k2, kz = k < NZ ? k : N - k;
            const double kzr = dz * kz, d = kxy + kzr * kzr;
            double r;
            if constexpr (sizeof(T) == 8) {
                r = num / d;
            } else {  // the hardware reciprocal (error e, 2^-23) times 1 + e + e^2
                r = __builtin_amdgcn_rcp(d);
                const double e = __builtin_fma(-d, r, 1.0);
                r = num * __builtin_fma(__builtin_fma(e, e, e), r, r);
            }
            const double mu = d > 0.0 ? r : 0.0;
            y[k2] = cmk<T>((T)(-mu * (double)y[k2].y), (T)(mu * (double)y[k2].x));
        }
        DftMR<T, N2, MR_S2>::run(y);
        mr_twiddles<T, N2, sizeof(T) == 4 ? 8 : 0>(tw, j, [&](int k, cx<T> w) { y[k] = cmul(y[k], w); });
    }
    __syncthreads();  // the first exchange is read before the second overwrites it
    mr_zero<T, 1, N1, !S::SPLIT>(x0);
    mr_trip<T, S::SPLIT>(
        [&](auto wr) {
            if (j < N1) {
#pragma unroll
                for (int k = 0; k < N2; ++k) wr((j * S::P2 + k) * C + c, y[k]);
            }
        },
        [&](auto g) {
            if (j < N2) {
#pragma unroll
                for (int q = 0; q < N1; ++q) g((q * S::P2 + j) * C + c, x[q]);
            }
        });
    if (j < N2) {  // second DFT, step 2: outputs j + N2 b
        DftMR<T, N1, MR_X1>::run(x);
        if (cv) {
#pragma unroll
            for (int b = 0; b < N1; ++b) {
                const int row = j + N2 * b;
                if (row < NZ) {
                    const T f = adj && row != 0 && row != N / 2 ? T(2) : T(1);
                    mr_st<T, S::SPLIT>(w, ((unsigned)row * a.s.ss + c) * CS, cscale(x[b], f));
                }
            }
        }
    }
}

// ---- X passes: XP pairs of real lines per tile ----------------------------------
// Workspace rows (column block 0) of the 2 XP lines of the tile, relative to the
// first one's (returned): line g = z ny + y is row z zrows + y0 + y.
template <typename T, int XP>
__device__ __forceinline__ size_t mr_rows(const MrArgs &a, unsigned g0, unsigned *row) {
    const unsigned tid = threadIdx.x;
    const unsigned z0 = g0 / a.x.ny, y0 = g0 - z0 * a.x.ny;
    if (tid < 2 * XP) {
        const unsigned g = g0 + tid, z = g / a.x.ny;
        row[tid] = (z - z0) * a.x.zrows + (g - z * a.x.ny) - y0;
    }
    return (size_t)z0 * a.x.zrows + a.x.y0 + y0;
}

// f(it, c, j): item j < J of pair c, the items of a step dealt over NT threads
template <int XP, int J, int NT, typename F>
__device__ __forceinline__ void mr_x_items(F f) {
    constexpr int I = (XP * J + NT - 1) / NT;
#pragma unroll
    for (int it = 0; it < I; ++it) {
        const int i = (int)threadIdx.x + it * NT;
        const int c = i / J;
        if (i < XP * J) f(it, c, i - c * J);
    }
}

// Step-0 outputs x of item (c, q) to the exchange tile.
template <typename T, class P>
__device__ __forceinline__ void mr_x_put(const cx<T> (&x)[P::G(0)], int c, int q) {
    cx<T> *lds = reinterpret_cast<cx<T> *>(pf_smem);
#pragma unroll
    for (int o = 0; o < P::G(0); ++o) lds[(c * P::G(0) + o) * MrShape<T, P>::P2 + q] = x[o];
}

// From the exchange tile (mr_x_put of every item) to the last step's outputs, handed
// to put(v, J): v[it] of item (c, i) holds the points i + J o of line c.  Every thread calls this.
template <typename T, class P, int NT, typename PUT>
__device__ __forceinline__ void mr_x_steps(const cx<T> *tw, PUT put) {
    using S = MrShape<T, P>;
    constexpr int N = S::N, G0 = S::G0, G1 = S::G1, G2 = S::G2, J1 = N / G1, J2 = N / G2;
    constexpr int I1 = (S::XP * J1 + NT - 1) / NT, I2 = (S::XP * J2 + NT - 1) / NT;
    cx<T> *lds = reinterpret_cast<cx<T> *>(pf_smem);
    __syncthreads();
    cx<T> y[I1][G1];
    mr_x_items<S::XP, J1, NT>([&](int it, int c, int i) {
        const int o = G2 == 1 ? i : i % G0, q = G2 == 1 ? 0 : i / G0;
#pragma unroll
        for (int p = 0; p < G1; ++p) y[it][p] = lds[(c * G0 + o) * S::P2 + q + p * G2];
        P::template step<1, true>(y[it], i, tw);
    });
    if constexpr (P::STEPS == 2) {
        put(y, MrInt<J1>());
    } else {
        __syncthreads();  // the first exchange is read before the second overwrites it
        mr_x_items<S::XP, J1, NT>([&](int it, int c, int i) {
            const int k = i % G0, h = i / G0;
#pragma unroll
            for (int o = 0; o < G1; ++o) lds[c * S::SP + k + G0 * (h * G1 + o)] = y[it][o];
        });
        __syncthreads();
        cx<T> z[I2][G2];
        mr_x_items<S::XP, J2, NT>([&](int it, int c, int i) {
#pragma unroll
            for (int p = 0; p < G2; ++p) z[it][p] = lds[c * S::SP + i + J2 * p];
            P::template step<2, true>(z[it], i, tw);
        });
        put(z, MrInt<J2>());
    }
}

// forward: real lines -> half spectra in the blocked workspace
template <typename T, class P, int NT>
__device__ __forceinline__ void mr_r2c_body(const MrArgs &a, unsigned tile, unsigned *row) {
    using S = MrShape<T, P>;
    constexpr int N = S::N, C = S::C, G0 = S::G0, J0 = N / G0;
    constexpr unsigned CS = sizeof(cx<T>), RS = sizeof(T);
    cx<T> *lds = reinterpret_cast<cx<T> *>(pf_smem);
    const int tid = threadIdx.x;
    const unsigned g0 = tile * (2 * S::XP), lines = a.x.lines;
    const cx<T> *tw = reinterpret_cast<const cx<T> *>(a.tw);
    const T *in = reinterpret_cast<const T *>(a.in) + (size_t)g0 * N;
    cx<T> *out = reinterpret_cast<cx<T> *>(a.out) + mr_rows<T, S::XP>(a, g0, row) * C;
    mr_x_items<S::XP, J0, NT>([&](int, int c, int q) {  // step 0: lanes along the points of the lines
        const unsigned ga = g0 + 2 * c;
        cx<T> x[G0];
#pragma unroll
        for (int m = 0; m < G0; ++m) x[m] = cmk<T>(T(0), T(0));
        if (ga < lines) {
#pragma unroll
            for (int m = 0; m < G0; ++m) x[m].x = mr_ld1<T>(in, (2 * c * N + q + J0 * m) * RS);
        }
        if (ga + 1 < lines) {
#pragma unroll
            for (int m = 0; m < G0; ++m) x[m].y = mr_ld1<T>(in, ((2 * c + 1) * N + q + J0 * m) * RS);
        }
        P::template step<0, true>(x, q, tw);
        mr_x_put<T, P>(x, c, q);
    });
    mr_x_steps<T, P, NT>(tw, [&](auto &v, auto jc) {
        constexpr int J = decltype(jc)::value;
        __syncthreads();  // the exchange tile is read before the spectra overwrite it
        mr_x_items<S::XP, J, NT>([&](int it, int c, int i) {
#pragma unroll
            for (int o = 0; o < N / J; ++o) lds[c * S::SP + i + J * o] = v[it][o];
        });
    });
    __syncthreads();
    // split Z = A + i B into the half spectra of the two lines, row by row: 16 bytes
    // (V modes) per lane, 8 lanes along a row (kb, cc); the slots past the last
    // mode of the last row block are written with what LDS holds
    constexpr int V = C / 8, total = S::NKB * 8 * S::XP;
    const T h = T(0.5);
#pragma unroll 4
    for (int f = tid; f < total; f += NT) {
        const int kk = (f & 7) * V, cc = (f / 8) & (S::XP - 1), kb = f / (8 * S::XP);
        const int k = kb * C + kk;
        const unsigned ga = g0 + 2 * cc;
        if (k < S::NXH && ga < lines) {
            cx<T> za[V], zb[V];
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const cx<T> z = lds[cc * S::SP + k + v];
                const cx<T> w = lds[cc * S::SP + (k + v == 0 ? 0 : N - k - v)];
                za[v] = cmk<T>((z.x + w.x) * h, (z.y - w.y) * h);
                zb[v] = cmk<T>((z.y + w.y) * h, (w.x - z.x) * h);
            }
            const unsigned o = kb * a.x.kbrows;  // rows of 128 bytes
            mr_st16<T>(out, (row[2 * cc] + o) * 128 + kk * CS, za);
            if (ga + 1 < lines) mr_st16<T>(out, (row[2 * cc + 1] + o) * 128 + kk * CS, zb);
        }
    }
}

// backward: half spectra in the blocked workspace -> real lines
template <typename T, class P, int NT>
__device__ __forceinline__ void mr_c2r_body(const MrArgs &a, unsigned tile, unsigned *row) {
    using S = MrShape<T, P>;
    constexpr int N = S::N, C = S::C, G0 = S::G0, J0 = N / G0;
    constexpr unsigned CS = sizeof(cx<T>), RS = sizeof(T);
    cx<T> *lds = reinterpret_cast<cx<T> *>(pf_smem);
    const int tid = threadIdx.x;
    const unsigned g0 = tile * (2 * S::XP), lines = a.x.lines;
    const cx<T> *tw = reinterpret_cast<const cx<T> *>(a.tw);
    const cx<T> *in = reinterpret_cast<const cx<T> *>(a.in) + mr_rows<T, S::XP>(a, g0, row) * C;
    T *out = reinterpret_cast<T *>(a.out) + (size_t)g0 * N;
    __syncthreads();
    // conj(Z), Z = A + i B, on the whole line: modes k < nxh from the rows, the
    // rest by Hermitian symmetry; the imaginary parts of modes 0 and N / 2 are
    // dropped
    constexpr int V = C / 8, total = S::NKB * 8 * S::XP;  // 16 bytes (V modes) per lane
    constexpr int ROUNDS = (total + NT - 1) / NT, EH = ROUNDS < kMrRowLoads ? ROUNDS : kMrRowLoads;
    for (int f1 = tid; f1 < total; f1 += EH * NT) {
        cx<T> ra[EH][V], rb[EH][V];
#pragma unroll
        for (int i = 0; i < EH; ++i) {
#pragma unroll
            for (int v = 0; v < V; ++v) ra[i][v] = rb[i][v] = cmk<T>(T(0), T(0));
            const int f = f1 + i * NT;
            const int kk = (f & 7) * V, cc = (f / 8) & (S::XP - 1), kb = f / (8 * S::XP);
            const unsigned ga = g0 + 2 * cc;
            if (f < total && kb * C + kk < S::NXH && ga < lines) {
                const unsigned o = kb * a.x.kbrows;  // rows of 128 bytes
                mr_ld16<T>(in, (row[2 * cc] + o) * 128 + kk * CS, ra[i]);
                if (ga + 1 < lines) mr_ld16<T>(in, (row[2 * cc + 1] + o) * 128 + kk * CS, rb[i]);
            }
        }
#pragma unroll
        for (int i = 0; i < EH; ++i) {
            const int f = f1 + i * NT;
            const int kk = (f & 7) * V, cc = (f / 8) & (S::XP - 1), kb = f / (8 * S::XP);
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const int k = kb * C + kk + v;
                if (f < total && k < S::NXH) {
                    const cx<T> A = ra[i][v], B = rb[i][v];
                    cx<T> *col = lds + cc * S::SP;
                    if (k == 0 || 2 * k == N) {
                        col[k] = cmk<T>(A.x, -B.x);
                    } else {
                        col[k] = cmk<T>(A.x - B.y, -A.y - B.x);
                        col[N - k] = cmk<T>(A.x + B.y, A.y - B.x);
                    }
                }
            }
        }
    }
    __syncthreads();
    cx<T> x[(S::XP * J0 + NT - 1) / NT][G0];
    mr_x_items<S::XP, J0, NT>([&](int it, int c, int q) {  // step 0
#pragma unroll
        for (int m = 0; m < G0; ++m) x[it][m] = lds[c * S::SP + q + J0 * m];
        P::template step<0, true>(x[it], q, tw);
    });
    __syncthreads();  // the lines are read before the exchange tile overwrites them
    mr_x_items<S::XP, J0, NT>([&](int it, int c, int q) { mr_x_put<T, P>(x[it], c, q); });
    // last step: real parts to line 2c, minus imaginary to 2c + 1
    mr_x_steps<T, P, NT>(tw, [&](auto &v, auto jc) {
        constexpr int J = decltype(jc)::value;
        auto store = [&](auto nt) {
            constexpr bool NTS = decltype(nt)::value;
            mr_x_items<S::XP, J, NT>([&](int it, int c, int i) {
                const unsigned ga = g0 + 2 * c;
                if (ga < lines) {
#pragma unroll
                    for (int o = 0; o < N / J; ++o) mr_st1<T, NTS>(out, (2 * c * N + i + J * o) * RS, v[it][o].x);
                }
                if (ga + 1 < lines) {
#pragma unroll
                    for (int o = 0; o < N / J; ++o) mr_st1<T, NTS>(out, ((2 * c + 1) * N + i + J * o) * RS, -v[it][o].y);
                }
            });
        };
        if (a.flags & MR_NT_STORES) store(std::true_type());
        else store(std::false_type());
    });
}

// ---- kernels: one tile per workgroup, a plan's pass or a batch's ------------------
// C2C of a plan: grid (column blocks, outer indices), with MR_OUTER_FAST (outer
// indices, column blocks); the others: grid (tiles).
template <typename T, class P, int CT>
__device__ __forceinline__ void mr_c2c_tile(const MrArgs &m, const MrArgs &a, unsigned tile) {
    unsigned cb = tile, ta = blockIdx.y;
    if (m.flags & (MR_BATCH | MR_XCD)) {
        ta = tile / (unsigned)a.CB;
        cb = tile - ta * (unsigned)a.CB;
    } else if (m.flags & MR_OUTER_FAST) {
        ta = tile;
        cb = blockIdx.y;
    }
    mr_c2c_body<T, P, CT>(a, ta, cb);
}

template <class P, typename T>
__global__ __launch_bounds__((MrShape<T, P>::CTHREADS)) void k_mr_c2c(MrArgs m) {
    MrArgs a;
    const unsigned tile = mr_resolve(m, a);
    mr_c2c_tile<T, P, MrShape<T, P>::CT>(m, a, tile);
}

// grid (column blocks, ky)
template <int N1, int N2, typename T>
__global__ __launch_bounds__((MrShape<T, MrTwoStep<T, N1, N2>>::CTHREADS)) void k_mr_spec(MrArgs m) {
    mr_spec_body<T, N1, N2>(m, blockIdx.y, blockIdx.x);
}

template <class P, int FWD, typename T>
__global__ __launch_bounds__((MrShape<T, P>::XTHREADS), (MrShape<T, P>::XWAVES)) void k_mr_x(MrArgs m) {
    MrArgs a;
    const unsigned tile = mr_resolve(m, a);
    constexpr int NT = MrShape<T, P>::XTHREADS;
    __shared__ unsigned row[kMrRows];
    if constexpr (FWD) mr_r2c_body<T, P, NT>(a, tile, row);
    else mr_c2r_body<T, P, NT>(a, tile, row);
}

// The table's instantiations are dealt round-robin over PF_MR_UNITS
// compilation units per precision (kernels_mr_unit.hip, built once per unit).
#ifndef PF_MR_UNITS
#define PF_MR_UNITS 8
#endif
// C2C columns, forward X (real to half spectra), backward X, spectral step (even lengths)
enum { MR_C2C = 0, MR_R2C = 1, MR_C2R = 2, MR_SPEC = 3 };

typedef const void *(*mr_pick_fn)(int index, int what);

template <typename T, int I>
const void *mr_kernel_at(int what) {
    using P = MrPlan<T, I>;
    static_assert(MrShape<T, P>::XLDS <= kMaxLds && MrShape<T, P>::CLDS <= kMaxLds, "tile too large");
    static_assert(MrShape<T, P>::CTHREADS <= 1024 && MrShape<T, P>::XTHREADS <= 1024, "workgroup too large");
    switch (what) {
        case MR_C2C: return reinterpret_cast<const void *>(&k_mr_c2c<P, T>);
        case MR_R2C: return reinterpret_cast<const void *>(&k_mr_x<P, 1, T>);
        case MR_C2R: return reinterpret_cast<const void *>(&k_mr_x<P, 0, T>);
        case MR_SPEC:
            if constexpr (kMrLen[I].n % 2 == 0)
                return reinterpret_cast<const void *>(&k_mr_spec<kMrLen[I].n1, kMrLen[I].n2, T>);
    }
    return nullptr;
}

// ---- batched launches over several lengths -------------------------------------------
// One kernel per class of lengths (kMrLen positions first .. last - 1): the
// workgroups of every transform of the class in one launch, each branching to
// its length's code.  A launch per length (25 lengths in a batch of 32 grids: 144
// launches a pair of 5 .. 60 us, most with fewer tiles than would fill the
// chip) left the device to the tails; the classes keep lengths of similar
// register, LDS and thread needs together.  Measured per pair, a launch per
// length -> per class: 32 FP32 grids of 48 .. 320 points 2.04 -> 1.38 ms, 15 FP64
// grids of 24 .. 124 points 0.357 -> 0.147 ms.
struct MrClass {
    int first, last, cap;  // positions; threads per column (items beyond go to further rounds)
};
constexpr MrClass kMrClass[] = {{0, 36, 16},   {36, 60, 16},   {60, 72, 20},     // 16 .. 112, 120 .. 243, 245 .. 324
                                {72, 92, 36}, {92, 107, 36}, {107, 128, 36}};  // 336 .. 512, 525 .. 720, 729 .. 1024
constexpr int kMrLongClass = 3;  // from here on only for lengths with few workgroups (pf_batch_setup)
constexpr int kMrClasses = (int)(sizeof(kMrClass) / sizeof(kMrClass[0]));

constexpr int mr_class(int index) {
    for (int c = 0; c < kMrClasses; ++c)
        if (index >= kMrClass[c].first && index < kMrClass[c].last) return c;
    return -1;
}
template <typename T>
constexpr int mr_class_cols(int c) {  // threads per column: whole waves
    const int w = 64 / mr_cols<T>();
    return (kMrClass[c].cap + w - 1) / w * w;
}
template <typename T>
constexpr int mr_class_c2c_threads(int c) {
    return mr_cols<T>() * mr_class_cols<T>(c);
}
template <typename T, int F, int... I>
constexpr int mr_class_x_threads_of(std::integer_sequence<int, I...>) {
    int t = 0;
    ((t = mr_max(t, MrShape<T, MrPlan<T, F + I>>::XTHREADS)), ...);
    return t;
}
template <typename T, int CLS>
constexpr int mr_class_x_threads() {
    return mr_class_x_threads_of<T, kMrClass[CLS].first>(
        std::make_integer_sequence<int, kMrClass[CLS].last - kMrClass[CLS].first>());
}

// a.count of a batch entry: the transform's position in its class
template <typename T, int CLS, int... I>
__device__ __forceinline__ void mr_merged_c2c(const MrArgs &m, const MrArgs &a, unsigned tile,
                                              std::integer_sequence<int, I...>) {
    constexpr int F = kMrClass[CLS].first;
    (void)((a.count == I
                ? (mr_c2c_tile<T, MrPlan<T, F + I>, mr_class_cols<T>(CLS)>(m, a, tile), true)
                : false) || ...);
}
template <typename T, int CLS, int FWD, int... I>
__device__ __forceinline__ void mr_merged_x(const MrArgs &a, unsigned tile, unsigned *row,
                                            std::integer_sequence<int, I...>) {
    constexpr int F = kMrClass[CLS].first, NT = mr_class_x_threads<T, CLS>();
    auto one = [&](auto pos) {
        constexpr int P = F + decltype(pos)::value;
        if constexpr (FWD) mr_r2c_body<T, MrPlan<T, P>, NT>(a, tile, row);
        else mr_c2r_body<T, MrPlan<T, P>, NT>(a, tile, row);
        return true;
    };
    (void)((a.count == I ? one(std::integral_constant<int, I>()) : false) || ...);
}

template <int CLS, typename T>
__global__ __launch_bounds__(mr_class_c2c_threads<T>(CLS)) void k_mr_c2c_class(MrArgs m) {
    MrArgs a;
    const unsigned tile = mr_resolve(m, a);
    mr_merged_c2c<T, CLS>(m, a, tile, std::make_integer_sequence<int, kMrClass[CLS].last - kMrClass[CLS].first>());
}
template <int CLS, int FWD, typename T>
__global__ __launch_bounds__((mr_class_x_threads<T, CLS>())) void k_mr_x_class(MrArgs m) {
    MrArgs a;
    const unsigned tile = mr_resolve(m, a);
    __shared__ unsigned row[kMrRows];
    mr_merged_x<T, CLS, FWD>(a, tile, row,
                             std::make_integer_sequence<int, kMrClass[CLS].last - kMrClass[CLS].first>());
}

}  // namespace pf
