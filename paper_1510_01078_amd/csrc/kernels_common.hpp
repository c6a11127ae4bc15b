// Helpers shared by the gfx950 stage kernels: FFT work-group shape, the
// in-LDS transform of a batch of sequences, dynamic-LDS opt-in and the
// device view of an FFT plan.
#pragma once
#include <hip/hip_runtime.h>

#include <mutex>
#include <type_traits>
#include <utility>

#include "fft_device.hpp"
#include "fft_reg.hpp"
#include "kernels.hpp"

namespace patk {

constexpr int kFftMaxV = 16;    // values per thread in the FFT kernels
constexpr int kFftThreads = 256; // threads per FFT work-group

// Sequences of length n per FFT work-group of nthr threads: at most kFftMaxV
// values per thread, at most `cap`, and (when possible) within 80 KiB of LDS
// so two work-groups share a CU.
template <typename T>
static inline int fft_batch(int n, int nthr, int cap) {
  int b = kFftMaxV * nthr / n;
  const int by_lds = int(81920 / (size_t(lseq(n)) * 2 * sizeof(T)));
  if (b > by_lds) b = by_lds;
  if (b > cap) b = cap;
  return b < 1 ? 1 : b;
}

// Sequences per work-group of an FFT stage: a power of two for lengths with a
// two-pass register transform (one butterfly per thread, so at most
// nthr / the larger radix of them, within 80 KiB of LDS so that two work-groups
// share a CU), else fft_batch.
template <typename T>
static inline int fft_seqs(const FftRaw& f, int nthr, int cap) {
  if (!f.two.r1) return fft_batch<T>(f.n, nthr, cap);
  int s = 1;
  const size_t seq = size_t(f.two.r1) * (f.two.r2 | 1) * 2 * sizeof(T);
  while (2 * s <= cap && 2 * s * reg_larger(f.two) <= nthr && 2 * s * seq <= 81920) s *= 2;
  return s;
}

// Bins per work-group of the y passes (the band ranges are whole groups of
// them): no more than the passes in LDS would hold, which leaves 4 from 540 to
// 640 points (8 there: y pass 17.0 -> 19.1 us at 640 points).
template <typename T>
static inline int fft_bins(const FftRaw& f, int nthr, int cap) {
  const int most = fft_batch<T>(f.n, nthr, cap);
  int s = fft_seqs<T>(f, nthr, cap);
  while (s > most) s /= 2;
  return s;
}

// Launch shape of a two-pass transform of S = fft_seqs sequences. Q is odd
// (lanes on consecutive k read distinct banks); P puts S consecutive
// sequences of one index on the banks that S neighbours leave free (a wave
// walks sequences fastest when it reads or writes columns).
template <typename T>
static inline Fft2Raw fft2_shape(const FftRaw& f, int S) {
  Fft2Raw t = f.two;
  constexpr int U = 256 / int(2 * sizeof(T));  // complex values across the 64 banks
  t.Q = t.r2 | 1;
  t.ls = 0;
  while ((1 << t.ls) < S) ++t.ls;
  t.P = t.r1 * t.Q;
  if (S > 1 && S <= U)
    while (t.P % (2 * U / S) != U / S) ++t.P;
  return t;
}
constexpr int three_class(const Fft3Raw& f) {
  const int r = f.r3 > 1 ? f.r3 : (f.r1 > f.r2 ? f.r1 : f.r2);  // radices ascend in three passes
  return r <= 16 ? 16 : r <= 20 ? 20 : 32;
}
// Threads of a temporal work-group: a butterfly each in every pass, up to 512.
// Where only the first pass (n / r1 butterflies, it does not work in place)
// takes more than 256 and its radices are of the larger classes, it runs in
// two rounds of 256 instead: 3200 points on five waves held 11 of 20 waves per
// CU (190 us for 22500 sensors, 207 us; at the smaller radices the rounds' own
// registers cost more).
static inline bool fft3_rounds(const Fft3Raw& f) {
  return f.r3 > 1 && three_class(f) > 16 && f.r2 * f.r3 > 256 && f.r1 * f.r3 <= 256;  // r2 <= r3
}
static inline int fft3_threads(const Fft3Raw& f) {
  const int most = f.r3 > 1 ? f.r2 * f.r3 : (f.r1 > f.r2 ? f.r1 : f.r2) << f.ls;  // radices ascend in three passes
  return fft3_rounds(f) ? 256 : (most + 63) / 64 * 64;
}
static inline size_t fft2_slots(const Fft2Raw& t) { return size_t(t.P) << t.ls; }
static inline int fft2_threads(const Fft2Raw& t) { return ((reg_larger(t) << t.ls) + 63) / 64 * 64; }

// Transform the nseq sequences of length fd.n in LDS. Sequences of at most
// 1024 points are each owned by one wave (no work-group barriers inside the
// transform); longer ones use the whole work-group. Callers synchronise the
// work-group before (after filling) and after (before reading).
constexpr int kWaveFftMax = 1024;

// FFT work-group shape: 256 threads, at most 8 sequences per group (measured
// best on MI355X among 128-512 threads and 4-16 sequences, block or wave mode)
constexpr int kFftCap = 8;
struct FftCfg {
  int threads = 256, cap = kFftCap, wave = 0;
};
static inline FftCfg fft_cfg() { return FftCfg{}; }
// The inverse 3-D FFT's x and y passes read and write the half spectrum in
// runs of `cap` consecutive z modes: 16 per group measured faster there.
constexpr int kInvCap = 16;
// z modes per work-group of the gather fused with the inverse x pass: 8
// (18 KiB of LDS at 256 points) leaves room for all the work-groups that the
// registers allow; the gather is bound by instruction issue (runs of 16 and 4
// took 0.083 and 0.088 ms where 8 took 0.077, on the passes in LDS)
constexpr int kGatherCap = 8;
static inline FftCfg inv_cfg() { return FftCfg{256, kInvCap, 0}; }

// Lengths with compile-time FFT instantiations (fft_ct), for the kernels that
// keep their passes in LDS: the position derivatives' (whose digits stay as they
// are) and the forward model's temporal transform and real-to-complex z pass,
// where they are the faster form. A launcher calls
// f(std::integral_constant<int, N>) for a listed length and
// f(std::integral_constant<int, 0>) (the runtime plan) otherwise.
template <int... Ns>
struct CtList {};
// sequences of length n a 256-thread group can hold, capped
__host__ __device__ constexpr int ct_maxb(int n, int cap) {
  return n > 0 && kFftMaxV * kFftThreads / n < cap ? kFftMaxV * kFftThreads / n : cap;
}
// 256 / 384 / 512 points: 128^3 .. 256^3 images at oversampling 1.5 or 2;
// 288 / 192 / 1920: a 192^3 image at oversampling 1.5 with 1536 samples
using CtLateral = CtList<256, 288, 384, 512>;
using CtInverse = CtList<128, 192, 256, 512>;
using CtTemporal = CtList<1920, 2048, 2560, 4096>;
// the forward model's real-to-complex z pass: of CtInverse the lengths whose
// compile-time form beats the register passes (image transforms 78 and 82 us
// at 256^3, a call 76.4 and 77.4 us at 128^3; at 192^3 41 and 38, at 128 x 128
// x 512 45 and 42 us)
using CtForwardZ = CtList<128, 256>;
// the forward model's fused x-FFT + interpolation (instantiated per footprint
// width and strip height as well) keeps the shorter list
using CtFused = CtList<256, 384, 512>;

template <class F>
static inline hipError_t ct_pick(CtList<>, int, F&& f) {
  return f(std::integral_constant<int, 0>{});
}
template <int N0, int... Ns, class F>
static inline hipError_t ct_pick(CtList<N0, Ns...>, int n, F&& f) {
  if (n == N0) return f(std::integral_constant<int, N0>{});
  return ct_pick(CtList<Ns...>{}, n, f);
}

template <typename T, bool INV>
__device__ __forceinline__ void fft_group(cx<T>* buf, const FftDesc<T>& fd, int nseq, int bstride, int tid, int nthr,
                                          int wave_mode) {
  if (wave_mode && fd.n <= kWaveFftMax) {
    const int lane = tid & 63, wave = tid >> 6, nwaves = nthr >> 6;
    for (int q = wave; q < nseq; q += nwaves) fft_lds<T, 16, INV, true>(buf + q * bstride, fd, 1, bstride, lane, 64);
  } else {
    fft_lds<T, kFftMaxV, INV, false>(buf, fd, nseq, bstride, tid, nthr);
  }
}

// The same transform with its twiddle table read from a copy in LDS (every
// pass reads the table between two barriers; from LDS the reads cost a few
// dozen cycles instead of a cache round trip).
template <typename T>
__device__ __forceinline__ FftDesc<T> lds_twiddles(FftDesc<T> fd, const cx<T>* twl) {
  fd.tw = twl;
  return fd;
}

// Allow a kernel more than the default dynamic LDS when a launch needs it.
// The largest size granted per (kernel, device) is remembered in a fixed
// table, so repeated launches (also inside a stream capture) make no runtime
// call and no host allocation.
static inline hipError_t allow_lds(const void* fn, size_t bytes) {
  if (bytes <= 65536) return hipSuccess;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return hipGetLastError();
  struct Grant {
    const void* fn;
    int dev;
    size_t bytes;
  };
  constexpr int kGrants = 256;
  static Grant granted[kGrants];
  static int used = 0;
  static std::mutex mu;
  std::lock_guard<std::mutex> lock(mu);
  int i = 0;
  while (i < used && !(granted[i].fn == fn && granted[i].dev == dev)) ++i;
  if (i < used && bytes <= granted[i].bytes) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes));
  if (e != hipSuccess) return e;
  if (i == used && used < kGrants) granted[used++] = Grant{fn, dev, 0};
  if (i < used) granted[i].bytes = bytes;  // a full table only means the attribute is set again next time
  return hipSuccess;
}

template <typename T>
static inline FftDesc<T> as_desc(const FftRaw& r) {
  FftDesc<T> d;
  static_assert(sizeof(FftPass) == sizeof(FftPassRaw), "pass layout");
  d.n = r.n;
  d.npass = r.npass;
  d.pass = static_cast<const FftPass*>(r.dpass);
  d.tw = static_cast<const cx<T>*>(r.tw);
  return d;
}

static inline FftView as_view(const FftRaw& r) {
  FftView v;
  v.n = r.n;
  v.npass = r.npass;
  v.pass = r.dpass;
  v.tw = r.tw;
  return v;
}

template <typename T>
__host__ __device__ inline FftDesc<T> view_desc(const FftView& v) {
  FftDesc<T> d;
  d.n = v.n;
  d.npass = v.npass;
  d.pass = static_cast<const FftPass*>(v.pass);
  d.tw = static_cast<const cx<T>*>(v.tw);
  return d;
}

// Problem of batched work item w (uniform over the work-group): the number of
// later problems whose first item is at or below w. prefix holds kGroupMax + 1
// entries (INT_MAX past the last problem), read by two wide scalar loads and
// compared without a branch, and the problem's arguments come by scalar loads
// as kernel arguments would: nothing waits on LDS, so a work-group per item
// costs two scalar round trips.
__device__ __forceinline__ int batch_locate(const int* __restrict__ prefix, int w) {
  int p = 0;
#pragma unroll
  for (int i = 1; i < kGroupMax; ++i) p += w >= prefix[i] ? 1 : 0;
  return p;
}

// Linear index of this work-group in a 2-D grid with the hardware's
// round-robin placement over the 8 XCDs undone: work-groups with consecutive
// results run on the same XCD and share its L2 (a partial tail keeps its
// own order).
__device__ __forceinline__ int xcd_linear() {
  const int b = blockIdx.x + gridDim.x * blockIdx.y;
  const int per = int(gridDim.x * gridDim.y) / 8;
  return b < per * 8 ? (b % 8) * per + b / 8 : b;
}

// LDS slots of a complex-to-real z work-group of `rows` real rows: two rows
// share one complex sequence, then the n twiddles.
__host__ __device__ constexpr int c2r_lds_slots(int rows, int n) { return (rows + 1) / 2 * lseq(n) + n; }
// complex pairs staged per thread in a runtime-length complex-to-real z pass:
// (rows + 1) / 2 pairs of n / 2 + 1 values with rows * n <= kFftMaxV * 256
// stay within 8 * 256 for every n <= 2048 (at most 1366; 1032 at n = 256)
constexpr int kC2rStage = 8;

// most threads of the inverse y pass: its work-groups take 16 z modes, whole
// 128-byte lines, also where that needs more than 256 butterflies (320 points:
// 58 us, 69 us with 8 modes)
constexpr int kInvYThreads = 512;
// pairs of rows per work-group of the two-pass complex-to-real z pass
constexpr int kC2rSeqs = 8;

// LDS slots of one temporal work-group (a sensor pair): the sequence, then
// the split twiddle tables (single-problem and batched launches).
__host__ __device__ constexpr int temporal_lds_slots(int n_t) { return lseq(n_t) + tw_split_slots(n_t); }

// The lane index, re-read inside a batched stage's persistent loop: values
// computed from it are then not hoisted out of the loop, where they stayed
// live across every work item (the batched temporal FFT held 94 registers
// against 72 for one item, 2 instead of 3 work-groups per CU).
__device__ __forceinline__ int loop_lane() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// Work item of a batched launch's slot L = blockIdx.x + i * gridDim.x (the
// i-th pass of a persistent grid). The hardware places work-groups on the 8
// XCDs round-robin, so with a grid that is a multiple of 8 slots L and L + 8
// share an XCD; items 2m and 2m + 1 (neighbouring blocks of one problem,
// which write the two halves of the same 128-byte lines) are given such a
// pair of slots, so that XCD's L2 merges the halves. A bijection on
// [0, total): the last total mod 16 items keep their slots.
__device__ __forceinline__ int batch_item(int L, int total) {
  if (L >= (total & ~15)) return L;
  const int r = L & 15;
  return (L & ~15) + 2 * (r & 7) + (r >> 3);
}

// Grid of a batched launch: one block per work item, or `st.grid` blocks
// striding over the items.
static inline unsigned batch_grid(const BatchStage& st) {
  return unsigned(st.grid > 0 && st.grid < st.total ? st.grid : st.total);
}

template <typename A, typename K>
static inline hipError_t launch_batch_kernel(K kern, const BatchStage& st, const BatchIO& io, hipStream_t s) {
  hipError_t e = allow_lds(reinterpret_cast<const void*>(kern), st.lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(batch_grid(st)), dim3(st.threads), st.lds, s, static_cast<const A*>(st.args),
                     st.prefix, st.total, io);
  return hipGetLastError();
}

}  // namespace patk
