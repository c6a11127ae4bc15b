// Two-pass FFT of length n = R1 * R2 with the butterflies in registers: a
// thread loads the R1 inputs i + r*R2 of one butterfly from where the data
// are, transforms them, multiplies by the twiddles w^(i*k) and leaves them in
// LDS; after one barrier a thread reads the R2 values of one k, transforms
// them and stores the outputs k + R1*q where they go:
//
//   X[k + R1 q] = sum_i w_R2^(i q) ( w_n^(i k) sum_r x[i + r R2] w_R1^(r k) )
//
// (w_n = exp(-2 pi i/n), conjugated for the inverse). The data cross LDS once
// (one write, one read) with one barrier, where a Stockham transform of three
// radix-8/6 passes between LDS copies crosses it eight times with seven.
//
// Contraction is off and every fused multiply-add is written out, so the same
// input gives the same bits in whatever kernel the functions are inlined
// (single problems, batches, the transposes).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "fft_device.hpp"
#include "kernels.hpp"

namespace patk {

// cos and sin of 2 pi m/n at compile time: reduced exactly to the first
// octant, then the Taylor series (an argument of at most pi/4, so 12 terms
// leave less than an ulp of a double)
namespace ctrig {
constexpr double kTau = 6.283185307179586476925286766559;
constexpr double taylor_cos(double x) {
  double t = 1.0, s = 1.0;
  for (int i = 1; i <= 12; ++i) {
    t *= -x * x / double((2 * i - 1) * (2 * i));
    s += t;
  }
  return s;
}
constexpr double taylor_sin(double x) {
  double t = x, s = x;
  for (int i = 1; i <= 12; ++i) {
    t *= -x * x / double((2 * i) * (2 * i + 1));
    s += t;
  }
  return s;
}
constexpr double cos2pi(int m, int n) {
  m = ((m % n) + n) % n;
  if (2 * m > n) m = n - m;                                       // cos is even
  if (4 * m > n) return -cos2pi(n - 2 * m, 2 * n);                // pi - angle
  if (8 * m > n) return taylor_sin(kTau * double(n - 4 * m) / double(4 * n));  // pi/2 - angle
  return taylor_cos(kTau * double(m) / double(n));
}
constexpr double sin2pi(int m, int n) { return cos2pi(4 * m - n, 4 * n); }
constexpr int inverse_mod(int a, int m) {
  for (int i = 1; i < m; ++i)
    if (a * i % m == 1) return i;
  return 0;
}
}  // namespace ctrig

__host__ __device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__host__ __device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }

// a * b, a * conj(b)
template <typename T>
__host__ __device__ __forceinline__ cx<T> rmul(cx<T> a, cx<T> b) {
#pragma clang fp contract(off)
  return cx<T>{fma_(a.x, b.x, -(a.y * b.y)), fma_(a.x, b.y, a.y * b.x)};
}
template <typename T, bool INV>
__host__ __device__ __forceinline__ cx<T> twiddle(cx<T> a, cx<T> w) {
#pragma clang fp contract(off)
  if (INV) return cx<T>{fma_(a.x, w.x, a.y * w.y), fma_(a.y, w.x, -(a.x * w.y))};
  return rmul(a, w);
}

// a * exp(-+2 pi i M/N) with the multiplications that the angle leaves
template <typename T, int M, int N, bool INV>
__host__ __device__ __forceinline__ cx<T> const_twiddle(cx<T> a) {
#pragma clang fp contract(off)
  constexpr int m8 = (8 * M) % (8 * N);  // eighths of a turn, times N
  if constexpr (m8 == 0) {
    return a;
  } else if constexpr (m8 == 4 * N) {
    return cx<T>{-a.x, -a.y};
  } else if constexpr (m8 == 2 * N || m8 == 6 * N) {
    constexpr bool neg = (m8 == 2 * N) != INV;  // times -i
    return neg ? cx<T>{a.y, -a.x} : cx<T>{-a.y, a.x};
  } else if constexpr (m8 % N == 0) {  // odd eighths
    constexpr T h = T(0.70710678118654752440084436210485);
    constexpr T c = (m8 == N || m8 == 7 * N) ? h : -h;
    constexpr T s = ((m8 == N || m8 == 3 * N) != INV) ? -h : h;
    if constexpr (c * s > 0) return cx<T>{c * (a.x - a.y), c * (a.x + a.y)};
    return cx<T>{c * (a.x + a.y), c * (a.y - a.x)};
  } else {
    constexpr T c = T(ctrig::cos2pi(M, N));
    constexpr T s = T(INV ? ctrig::sin2pi(M, N) : -ctrig::sin2pi(M, N));
    return cx<T>{fma_(a.x, c, -(a.y * s)), fma_(a.x, s, a.y * c)};
  }
}

// DFT of N values in registers, natural order in and out. Coprime factors
// combine without twiddles (the index maps of Good and Thomas, free in
// registers), others by the Cooley-Tukey split.
template <int N>
struct RadixSplit;
#define PATK_SPLIT(n, a, b) \
  template <> struct RadixSplit<n> { static constexpr int A = a, B = b; };
PATK_SPLIT(6, 2, 3)
PATK_SPLIT(8, 2, 4)
PATK_SPLIT(9, 3, 3)
PATK_SPLIT(10, 2, 5)
PATK_SPLIT(12, 3, 4)
PATK_SPLIT(15, 3, 5)
PATK_SPLIT(16, 4, 4)
PATK_SPLIT(18, 2, 9)
PATK_SPLIT(20, 4, 5)
PATK_SPLIT(24, 3, 8)
PATK_SPLIT(25, 5, 5)
PATK_SPLIT(27, 3, 9)
PATK_SPLIT(30, 2, 15)
PATK_SPLIT(32, 4, 8)
#undef PATK_SPLIT

template <typename T, int N, bool INV>
struct RDft;

template <typename T, int N, bool INV, int A, int B, int I, int K>
__host__ __device__ __forceinline__ void split_twiddles(cx<T> (&t)[B][A]) {
  if constexpr (I < B) {
    if constexpr (K < A) {
      t[I][K] = const_twiddle<T, I * K, N, INV>(t[I][K]);
      split_twiddles<T, N, INV, A, B, I, K + 1>(t);
    } else {
      split_twiddles<T, N, INV, A, B, I + 1, 1>(t);
    }
  }
}

template <typename T, int N, bool INV>
struct RDft {
  __host__ __device__ __forceinline__ static void run(cx<T> (&a)[N]) {
    constexpr int A = RadixSplit<N>::A, B = RadixSplit<N>::B;
    constexpr int ia = ctrig::inverse_mod(A % B, B), ib = ctrig::inverse_mod(B % A, A);
    constexpr bool coprime = (A * ia) % B == 1 && (B * ib) % A == 1;
    cx<T> t[B][A];
#pragma unroll
    for (int i = 0; i < B; ++i) {
#pragma unroll
      for (int r = 0; r < A; ++r) t[i][r] = coprime ? a[(B * r + A * i) % N] : a[i + B * r];
      RDft<T, A, INV>::run(t[i]);
    }
    if constexpr (!coprime) split_twiddles<T, N, INV, A, B, 1, 1>(t);
#pragma unroll
    for (int k = 0; k < A; ++k) {
      cx<T> u[B];
#pragma unroll
      for (int i = 0; i < B; ++i) u[i] = t[i][k];
      RDft<T, B, INV>::run(u);
#pragma unroll
      for (int q = 0; q < B; ++q) a[coprime ? (B * ib * k + A * ia * q) % N : k + A * q] = u[q];
    }
  }
};

// The same sums, output e given to st(e, v) as each of the last butterflies
// ends: fewer values live where the outputs go to memory under conditions
// (with all of them held until the first store, radix 32 on 128 registers
// spilled 12 to 29 of them to scratch).
template <typename T, int N, bool INV, typename Store>
__device__ __forceinline__ void rdft_to(const cx<T> (&a)[N], Store st) {
  constexpr int A = RadixSplit<N>::A, B = RadixSplit<N>::B;
  constexpr int ia = ctrig::inverse_mod(A % B, B), ib = ctrig::inverse_mod(B % A, A);
  constexpr bool coprime = (A * ia) % B == 1 && (B * ib) % A == 1;
  cx<T> t[B][A];
#pragma unroll
  for (int i = 0; i < B; ++i) {
#pragma unroll
    for (int r = 0; r < A; ++r) t[i][r] = coprime ? a[(B * r + A * i) % N] : a[i + B * r];
    RDft<T, A, INV>::run(t[i]);
  }
  if constexpr (!coprime) split_twiddles<T, N, INV, A, B, 1, 1>(t);
#pragma unroll
  for (int k = 0; k < A; ++k) {
    cx<T> u[B];
#pragma unroll
    for (int i = 0; i < B; ++i) u[i] = t[i][k];
    RDft<T, B, INV>::run(u);
#pragma unroll
    for (int q = 0; q < B; ++q) st(coprime ? (B * ib * k + A * ia * q) % N : k + A * q, u[q]);
  }
}

template <typename T, bool INV>
struct RDft<T, 2, INV> {
  __host__ __device__ __forceinline__ static void run(cx<T> (&a)[2]) {
#pragma clang fp contract(off)
    const cx<T> t = a[0];
    a[0] = cx<T>{t.x + a[1].x, t.y + a[1].y};
    a[1] = cx<T>{t.x - a[1].x, t.y - a[1].y};
  }
};

template <typename T, bool INV>
struct RDft<T, 3, INV> {
  __host__ __device__ __forceinline__ static void run(cx<T> (&a)[3]) {
#pragma clang fp contract(off)
    constexpr T h = T(INV ? 0.86602540378443864676372317075294 : -0.86602540378443864676372317075294);
    const cx<T> t{a[1].x + a[2].x, a[1].y + a[2].y}, d{a[1].x - a[2].x, a[1].y - a[2].y};
    const cx<T> m{fma_(T(-0.5), t.x, a[0].x), fma_(T(-0.5), t.y, a[0].y)};
    a[0] = cx<T>{a[0].x + t.x, a[0].y + t.y};
    a[1] = cx<T>{fma_(-h, d.y, m.x), fma_(h, d.x, m.y)};
    a[2] = cx<T>{fma_(h, d.y, m.x), fma_(-h, d.x, m.y)};
  }
};

template <typename T, bool INV>
struct RDft<T, 4, INV> {
  __host__ __device__ __forceinline__ static void run(cx<T> (&a)[4]) {
#pragma clang fp contract(off)
    const cx<T> s0{a[0].x + a[2].x, a[0].y + a[2].y}, d0{a[0].x - a[2].x, a[0].y - a[2].y};
    const cx<T> s1{a[1].x + a[3].x, a[1].y + a[3].y}, d1{a[1].x - a[3].x, a[1].y - a[3].y};
    a[0] = cx<T>{s0.x + s1.x, s0.y + s1.y};
    a[2] = cx<T>{s0.x - s1.x, s0.y - s1.y};
    // d0 -+ i d1
    const cx<T> p{d0.x + d1.y, d0.y - d1.x}, m{d0.x - d1.y, d0.y + d1.x};
    a[1] = INV ? m : p;
    a[3] = INV ? p : m;
  }
};

template <typename T, bool INV>
struct RDft<T, 5, INV> {
  __host__ __device__ __forceinline__ static void run(cx<T> (&a)[5]) {
#pragma clang fp contract(off)
    constexpr T c1 = T(0.30901699437494742410229341718282);   // cos(2 pi/5)
    constexpr T c2 = T(-0.80901699437494742410229341718282);  // cos(4 pi/5)
    constexpr T s1 = T((INV ? 1 : -1) * 0.95105651629515357211643933337938);  // +-sin(2 pi/5)
    constexpr T s2 = T((INV ? 1 : -1) * 0.58778525229247312916870595463907);  // +-sin(4 pi/5)
    const cx<T> t1{a[1].x + a[4].x, a[1].y + a[4].y}, d1{a[1].x - a[4].x, a[1].y - a[4].y};
    const cx<T> t2{a[2].x + a[3].x, a[2].y + a[3].y}, d2{a[2].x - a[3].x, a[2].y - a[3].y};
    const cx<T> m1{fma_(c2, t2.x, fma_(c1, t1.x, a[0].x)), fma_(c2, t2.y, fma_(c1, t1.y, a[0].y))};
    const cx<T> m2{fma_(c1, t2.x, fma_(c2, t1.x, a[0].x)), fma_(c1, t2.y, fma_(c2, t1.y, a[0].y))};
    const cx<T> n1{fma_(s2, d2.x, s1 * d1.x), fma_(s2, d2.y, s1 * d1.y)};
    const cx<T> n2{fma_(-s1, d2.x, s2 * d1.x), fma_(-s1, d2.y, s2 * d1.y)};
    a[0] = cx<T>{a[0].x + (t1.x + t2.x), a[0].y + (t1.y + t2.y)};
    a[1] = cx<T>{m1.x - n1.y, m1.y + n1.x};
    a[4] = cx<T>{m1.x + n1.y, m1.y - n1.x};
    a[2] = cx<T>{m2.x - n2.y, m2.y + n2.x};
    a[3] = cx<T>{m2.x + n2.y, m2.y - n2.x};
  }
};

// Two-pass plan of one length on the device: the radices, the LDS layout
// (value k of sequence s, index i, at s*P + k*Q + i) and the twiddles
// tw[k*R2 + i] = exp(-2 pi i ik/n).
template <typename T>
struct Fft2 {
  int r1, r2;
  int P, Q;
  int ls;      // log2 of the sequences per work-group
  const cx<T>* tw;
};

template <typename T>
__host__ __device__ __forceinline__ Fft2<T> as_fft2(const Fft2Raw& f) {
  return Fft2<T>{f.r1, f.r2, f.P, f.Q, f.ls, static_cast<const cx<T>*>(f.tw)};
}

// Element at a 32-bit offset from a uniform base (one address register; the
// callers' arrays span less than 4 GiB from the base).
template <typename T>
__device__ __forceinline__ const cx<T>& cx_at(const cx<T>* base, unsigned at) {
  return *reinterpret_cast<const cx<T>*>(reinterpret_cast<const char*>(base) + at * unsigned(sizeof(cx<T>)));
}
template <typename T>
__device__ __forceinline__ cx<T>& cx_at(cx<T>* base, unsigned at) {
  return *reinterpret_cast<cx<T>*>(reinterpret_cast<char*>(base) + at * unsigned(sizeof(cx<T>)));
}

// Kernels of two-pass transforms come in three classes by the larger radix,
// since the largest radix a kernel holds sets its registers: up to 16 (76 to
// 80 registers in FP32: 6 waves per SIMD), 18 and 20 (5 waves), 24 to 32 (4
// waves). One kernel for all took 128 registers, and the batched x pass over
// lengths of 96 to 288 points 1.19 instead of 0.93 ms.
constexpr int reg_larger(const Fft2Raw& f) { return f.r1 > f.r2 ? f.r1 : f.r2; }
constexpr int reg_class(const Fft2Raw& f) { return reg_larger(f) <= 16 ? 16 : reg_larger(f) <= 20 ? 20 : 32; }
template <typename T, int CLS>
constexpr int reg_waves() { return sizeof(T) == 4 ? (CLS == 16 ? 6 : CLS == 20 ? 5 : 4) : (CLS == 16 ? 3 : 2); }
// kernels that also come for lengths without a two-pass transform (CLS 0)
template <typename T, int CLS>
constexpr int any_waves() { return CLS > 0 ? reg_waves<T, CLS ? CLS : 16>() : 1; }

// go(std::integral_constant<int, CLS>) for the class of a transform
template <class F>
static inline hipError_t class_pick(const Fft2Raw& f, F&& go) {
  switch (reg_class(f)) {
    case 16: return go(std::integral_constant<int, 16>{});
    case 20: return go(std::integral_constant<int, 20>{});
    default: return go(std::integral_constant<int, 32>{});
  }
}
// the same, 0 for a length without a two-pass transform
template <class F>
static inline hipError_t class_pick_any(const Fft2Raw& f, F&& go) {
  return f.r1 ? class_pick(f, go) : go(std::integral_constant<int, 0>{});
}

// tid / d for tid < 1024 and 1 < d <= 32 (exact: the error of m is below
// 1/1024 of a step)
__device__ __forceinline__ int small_div(int tid, int d) {
  const unsigned m = 65536u / unsigned(d) + 1u;
  return int((unsigned(tid) * m) >> 16);
}

// First pass for the butterfly i of the sequence whose LDS block is `seq`:
// ld(e) gives input element e.
template <typename T, int R, bool INV, typename Load>
__device__ __forceinline__ void reg_first(cx<T>* seq, int r2, int Q, const cx<T>* __restrict__ tw, int i, Load ld) {
  cx<T> v[R], w[R];
#pragma unroll
  for (int r = 0; r < R; ++r) v[r] = ld(i + r * r2);
#pragma unroll
  for (int r = 1; r < R; ++r) w[r] = tw[i + r * r2];
  RDft<T, R, INV>::run(v);
  seq[i] = v[0];
#pragma unroll
  for (int r = 1; r < R; ++r) seq[i + r * Q] = twiddle<T, INV>(v[r], w[r]);
}

// First pass of sequences that already sit in LDS in natural order (element e
// at seq[e]): every butterfly is in registers before the barrier, so the
// exchange takes the same LDS. Called by the whole work-group; `active`
// threads hold a butterfly.
template <typename T, int R, bool INV>
__device__ __forceinline__ void reg_first_in_lds(cx<T>* seq, int r2, int Q, const cx<T>* __restrict__ tw, int i,
                                                 bool active) {
  cx<T> v[R], w[R];
  if (active) {
#pragma unroll
    for (int r = 1; r < R; ++r) w[r] = tw[i + r * r2];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = seq[i + r * r2];
    RDft<T, R, INV>::run(v);
  }
  __syncthreads();
  if (active) {
    seq[i] = v[0];
#pragma unroll
    for (int r = 1; r < R; ++r) seq[i + r * Q] = twiddle<T, INV>(v[r], w[r]);
  }
}

// Second pass for the index k: st(q, v) takes output k + r1*q. PART: only part
// of the outputs is stored, and the larger radices hand them on as their
// butterflies end (rdft_to; passes that store them all need no more registers
// in one burst, and the transposed y pass over 432 points takes 16.8 us so,
// 21.0 with PART).
template <typename T, int R, bool INV, bool PART, typename Store>
__device__ __forceinline__ void reg_second(const cx<T>* seq, int Q, int k, Store st) {
  cx<T> v[R];
  const cx<T>* row = seq + k * Q;
#pragma unroll
  for (int r = 0; r < R; ++r) v[r] = row[r];
  if constexpr (PART && R >= 24) {
    rdft_to<T, R, INV>(v, st);
  } else {
    RDft<T, R, INV>::run(v);
#pragma unroll
    for (int q = 0; q < R; ++q) st(q, v[q]);
  }
}

// Three-pass transform of one length n = r1*r2*r3 (r3 = 1: two passes) for
// sequences whose whole spectrum ends in LDS in natural order (the temporal
// FFT): value k1 of sequence s, index i at s*P + k1*QA + i, within it value k2,
// index i at k1*QA + k2*QB + i; twA[k1*m + i] = w_n^(i k1), m = r2*r3, and
// twB[k2*r3 + i] = w_m^(i k2).
template <typename T>
struct Fft3 {
  int n, r1, r2, r3;
  int P, QA, QB;
  int ls;
  const cx<T>* twA;
  const cx<T>* twB;
};

template <typename T>
__host__ __device__ __forceinline__ Fft3<T> as_fft3(const Fft3Raw& f) {
  return Fft3<T>{f.r1 * f.r2 * f.r3, f.r1, f.r2, f.r3, f.P, f.QA, f.QB, f.ls, static_cast<const cx<T>*>(f.twA),
                 static_cast<const cx<T>*>(f.twB)};
}

// Pass over values in LDS at src[r*stride], R of them, by the `active`
// threads; after the barrier value k goes to st(k, v).
template <typename T, int R, bool INV, typename Store>
__device__ __forceinline__ void reg_in_lds(const cx<T>* src, int stride, bool active, Store st) {
  cx<T> v[R];
  if (active) {
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = src[r * stride];
    RDft<T, R, INV>::run(v);
  }
  __syncthreads();
  if (active) {
#pragma unroll
    for (int r = 0; r < R; ++r) st(r, v[r]);
  }
}

// Middle pass of three: the same in place (output k to dst[k*QB]), times the
// twiddles tw[k*step], which are loaded beside the values: after the barrier
// every wave of the group waited for them at once (sixteen uneven problems'
// temporal FFTs 404 us, 353 us so).
template <typename T, int R, bool INV>
__device__ __forceinline__ void reg_mid(const cx<T>* src, int stride, bool active, const cx<T>* __restrict__ tw,
                                        int step, cx<T>* dst, int QB) {
  cx<T> v[R], w[R];
  if (active) {
#pragma unroll
    for (int r = 0; r < R; ++r) w[r] = tw[r * step];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = src[r * stride];
    RDft<T, R, INV>::run(v);
  }
  __syncthreads();
  if (active) {
#pragma unroll
    for (int r = 0; r < R; ++r) dst[r * QB] = twiddle<T, INV>(v[r], w[r]);
  }
}

// Radix by a uniform switch over those of the class (the host's table of
// factorisations, two_pass_plan, pairs no others).
#define PATK_RADICES_16(X) X(2) X(3) X(4) X(5) X(6) X(8) X(9) X(10) X(12) X(15) X(16)
#define PATK_FIRST_20(X) X(9) X(10) X(12) X(15) X(16) X(18) X(20)
#define PATK_SECOND_20(X) X(16) X(18) X(20)
#define PATK_FIRST_32(X) X(10) X(16) X(18) X(20)
#define PATK_SECOND_32(X) X(24) X(25) X(27) X(30) X(32)

// and of the three-pass transforms (three_pass_plan): radices in ascending order
#define PATK_THREE_A16(X) X(5) X(8) X(9) X(10) X(12) X(15) X(16)
#define PATK_THREE_B16(X) X(8) X(9) X(10) X(12) X(15) X(16)
#define PATK_THREE_C16(X) X(9) X(10) X(12) X(15) X(16)
#define PATK_THREE_A20(X) X(9) X(10) X(12) X(15) X(16) X(18) X(20)
#define PATK_THREE_C20(X) X(18) X(20)
#define PATK_THREE_A32(X) X(5) X(9) X(10) X(15) X(16) X(18)
#define PATK_THREE_B32(X) X(10) X(15) X(16) X(18) X(20)
#define PATK_THREE_C32(X) X(24) X(25) X(27) X(32)

template <typename T, int CLS, bool INV, typename Load>
__device__ __forceinline__ void three_first_any(const Fft3<T>& f, cx<T>* seq, int i, Load ld) {
  const int m = f.r2 * f.r3;
#define PATK_CASE(R) case R: reg_first<T, R, INV>(seq, m, f.QA, f.twA, i, ld); break;
  if constexpr (CLS == 16) {
    switch (f.r1) { PATK_THREE_A16(PATK_CASE) default: break; }
  } else if constexpr (CLS == 20) {
    switch (f.r1) { PATK_THREE_A20(PATK_CASE) default: break; }
  } else {
    switch (f.r1) { PATK_THREE_A32(PATK_CASE) default: break; }
  }
#undef PATK_CASE
}

template <typename T, int CLS, bool INV>
__device__ __forceinline__ void three_mid_any(const Fft3<T>& f, cx<T>* row, int i2, bool active) {
#define PATK_CASE(R) \
  case R: reg_mid<T, R, INV>(row + i2, f.r3, active, f.twB + i2, f.r3, row + i2, f.QB); break;
  if constexpr (CLS == 16) {
    switch (f.r2) { PATK_THREE_B16(PATK_CASE) default: break; }
  } else if constexpr (CLS == 20) {
    switch (f.r2) { PATK_THREE_A20(PATK_CASE) default: break; }
  } else {
    switch (f.r2) { PATK_THREE_B32(PATK_CASE) default: break; }
  }
#undef PATK_CASE
}

template <typename T, int CLS, bool INV, typename Store>
__device__ __forceinline__ void three_last_any(const Fft3<T>& f, const cx<T>* src, bool active, Store st) {
#define PATK_CASE(R) case R: reg_in_lds<T, R, INV>(src, 1, active, st); break;
  if constexpr (CLS == 16) {
    switch (f.r3) { PATK_THREE_C16(PATK_CASE) default: break; }
  } else if constexpr (CLS == 20) {
    switch (f.r3) { PATK_THREE_C20(PATK_CASE) default: break; }
  } else {
    switch (f.r3) { PATK_THREE_C32(PATK_CASE) default: break; }
  }
#undef PATK_CASE
}

template <typename T, int CLS, bool INV, typename Load>
__device__ __forceinline__ void reg_first_any(const Fft2<T>& f, cx<T>* seq, int i, Load ld) {
#define PATK_CASE(R) case R: reg_first<T, R, INV>(seq, f.r2, f.Q, f.tw, i, ld); break;
  if constexpr (CLS == 16) {
    switch (f.r1) { PATK_RADICES_16(PATK_CASE) default: break; }
  } else if constexpr (CLS == 20) {
    switch (f.r1) { PATK_FIRST_20(PATK_CASE) default: break; }
  } else {
    switch (f.r1) { PATK_FIRST_32(PATK_CASE) default: break; }
  }
#undef PATK_CASE
}

template <typename T, int CLS, bool INV>
__device__ __forceinline__ void reg_first_in_lds_any(const Fft2<T>& f, cx<T>* seq, int i, bool active) {
#define PATK_CASE(R) case R: reg_first_in_lds<T, R, INV>(seq, f.r2, f.Q, f.tw, i, active); break;
  if constexpr (CLS == 16) {
    switch (f.r1) { PATK_RADICES_16(PATK_CASE) default: break; }
  } else if constexpr (CLS == 20) {
    switch (f.r1) { PATK_FIRST_20(PATK_CASE) default: break; }
  } else {
    switch (f.r1) { PATK_FIRST_32(PATK_CASE) default: break; }
  }
#undef PATK_CASE
}

template <typename T, int CLS, bool INV, bool PART = false, typename Store>
__device__ __forceinline__ void reg_second_any(const Fft2<T>& f, const cx<T>* seq, int k, Store st) {
#define PATK_CASE(R) case R: reg_second<T, R, INV, PART>(seq, f.Q, k, st); break;
  if constexpr (CLS == 16) {
    switch (f.r2) { PATK_RADICES_16(PATK_CASE) default: break; }
  } else if constexpr (CLS == 20) {
    switch (f.r2) { PATK_SECOND_20(PATK_CASE) default: break; }
  } else {
    switch (f.r2) { PATK_SECOND_32(PATK_CASE) default: break; }
  }
#undef PATK_CASE
}

// Second pass in place in LDS: `active` threads read the r2 values at src, and
// output q goes to st(q, v) after the barrier.
template <typename T, int CLS, bool INV, typename Store>
__device__ __forceinline__ void reg_second_in_lds_any(const Fft2<T>& f, const cx<T>* src, bool active, Store st) {
#define PATK_CASE(R) case R: reg_in_lds<T, R, INV>(src, 1, active, st); break;
  if constexpr (CLS == 16) {
    switch (f.r2) { PATK_RADICES_16(PATK_CASE) default: break; }
  } else if constexpr (CLS == 20) {
    switch (f.r2) { PATK_SECOND_20(PATK_CASE) default: break; }
  } else {
    switch (f.r2) { PATK_SECOND_32(PATK_CASE) default: break; }
  }
#undef PATK_CASE
}

}  // namespace patk
