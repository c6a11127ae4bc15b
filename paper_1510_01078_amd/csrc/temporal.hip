// Temporal stage of the reconstruction: the equispaced part of the
// non-equispaced-range NUFFT in time (Section 3.1), per sensor.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "kernels_common.hpp"

namespace patk {

// ---------------------------------------------------------------------------
// Stage 0: temporal FFT per sensor (the equispaced half of eq. NER_NUFFT).
// Two real traces share one complex FFT (re = sensor m0, im = sensor m1).
// Sample n sits at index (n - n0) mod n_t after multiplication by
// h_m*dt/phihat_t((n - n0)/n_t) (hw == nullptr: unit weight instead of
// h_m*dt); bins b_lo .. b_lo+nb-1 are kept per sensor.
// ---------------------------------------------------------------------------

constexpr int kTemporalThreads = 512;
// compile-time lengths (at most 4096 points): 256 threads, 16 values each,
// measured 5 % faster than 512 at 2560 points
constexpr int kTemporalCtThreads = 256;
template <int NCT>
constexpr int temporal_threads() { return NCT > 0 ? kTemporalCtThreads : kTemporalThreads; }

// Register form (fft_reg.hpp): the first pass loads the samples, in the last
// one only the slots of the band and its mirror are written to LDS, where the
// two sensors' bins are taken apart. 1 << ls sensor pairs per work-group
// (short traces: a pair is a few dozen butterflies). Bound by the vector ALU
// and by HBM in about equal parts.
enum { TEMPORAL_THREE = 0, TEMPORAL_TWO = 1, TEMPORAL_ROUNDS = 2 };  // passes; three with the first in rounds

template <typename T, int CLS, int FORM>
__device__ __forceinline__ void temporal_reg_body(const T* __restrict__ g, int M, int Nt, int n0,
                                                  const T* __restrict__ hw, const T* __restrict__ deap,
                                                  const Fft3<T>& f, int b_lo, int nb, int pitch,
                                                  cx<T>* __restrict__ Gt, int bx, int tid) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* buf = reinterpret_cast<cx<T>*>(smem_raw);
  const int n_t = f.n;
  const int S = 1 << f.ls;
  const int pairs = min(S, (M + 1) / 2 - (bx << f.ls));
  // thread -> (pair, butterfly) of a pass of `count` butterflies per pair
  auto split = [&](int t, int count, int& s, int& i) {
    s = S == 1 ? 0 : t / count;
    i = t - s * count;
    return s < pairs && i < count;
  };
  constexpr bool TWO = FORM == TEMPORAL_TWO;
  const Fft2<T> two{f.r1, f.r2, f.P, f.QA, f.ls, f.twA};
  int s, i;
  auto first = [&]() {
    const int m0 = 2 * ((bx << f.ls) + s);
    const bool has1 = m0 + 1 < M;
    const T w0 = hw ? hw[m0] : T(1);
    const T w1 = has1 ? (hw ? hw[m0 + 1] : T(1)) : T(0);
    const T* g0 = g + size_t(m0) * Nt;
    const T* g1 = g + size_t(has1 ? m0 + 1 : m0) * Nt;
    auto sample = [&](int e) {
      int n = e + n0;
      if (n >= n_t) n -= n_t;
      const bool in = n < Nt;  // else zero padding; the loads carry no branch, so they stay in flight together
      const int at = in ? n : 0;
      const T d = deap[at];
      const T a = g0[at] * w0 * d;
      const T b = g1[at] * w1 * d;
      return cx<T>{in ? a : T(0), in && has1 ? b : T(0)};
    };
    if constexpr (TWO)
      reg_first_any<T, CLS, false>(two, buf + s * f.P, i, sample);
    else
      three_first_any<T, CLS, false>(f, buf + s * f.P, i, sample);
  };
  if constexpr (FORM == TEMPORAL_ROUNDS) {
    for (int t = tid; split(t, n_t / f.r1, s, i); t += blockDim.x) first();
  } else if (split(tid, n_t / f.r1, s, i)) {
    first();
  }
  __syncthreads();
  // slots read below: bins b_lo .. b_lo + nb - 1 and their negatives
  const int reach = max(b_lo + nb - 1, -b_lo);
  cx<T>* seq;
  auto keep = [&](int e, cx<T> v) {
    if (e <= reach || e >= n_t - reach) seq[e] = v;
  };
  if constexpr (TWO) {
    const bool on = split(tid, f.r1, s, i);
    seq = buf + s * f.P;
    reg_second_in_lds_any<T, CLS, false>(two, seq + i * f.QA, on, [&](int q, cx<T> v) { keep(i + f.r1 * q, v); });
  } else {
    bool on = split(tid, f.r1 * f.r3, s, i);
    {
      const int k1 = small_div(i, f.r3), i2 = i - k1 * f.r3;
      seq = buf + s * f.P;
      three_mid_any<T, CLS, false>(f, seq + k1 * f.QA, i2, on);
    }
    __syncthreads();
    on = split(tid, f.r1 * f.r2, s, i);
    const int k2 = small_div(i, f.r1), k1 = i - k2 * f.r1;
    seq = buf + s * f.P;
    three_last_any<T, CLS, false>(f, seq + k1 * f.QA + k2 * f.QB, on,
                                  [&](int q, cx<T> v) { keep(k1 + f.r1 * (k2 + f.r2 * q), v); });
  }
  __syncthreads();
  for (int p = 0; p < pairs; ++p) {
    const int m0 = 2 * ((bx << f.ls) + p);
    const bool has1 = m0 + 1 < M;
    const cx<T>* x = buf + p * f.P;
    for (int j = tid; j < nb; j += blockDim.x) {
      const int b = b_lo + j;  // -n_t < b < n_t (the band fits in n_t bins)
      const cx<T> z = x[b < 0 ? b + n_t : b];
      const cx<T> zm = x[b > 0 ? n_t - b : -b];
      // transform of the real part: (Z_b + conj Z_-b)/2; of the imaginary part: (Z_b - conj Z_-b)/(2i)
      Gt[size_t(m0) * pitch + j] = cx<T>{T(0.5) * (z.x + zm.x), T(0.5) * (z.y - zm.y)};
      if (has1) Gt[size_t(m0 + 1) * pitch + j] = cx<T>{T(0.5) * (z.y + zm.y), T(-0.5) * (z.x - zm.x)};
    }
  }
}

template <typename T, int CLS, int FORM>
__global__ __launch_bounds__(kTemporalThreads, (reg_waves<T, CLS>())) void k_temporal_reg(
    const T* __restrict__ g, int M, int Nt, int n0, const T* __restrict__ hw, const T* __restrict__ deap, Fft3Raw f,
    int b_lo, int nb, int pitch, cx<T>* __restrict__ Gt) {
  temporal_reg_body<T, CLS, FORM>(g, M, Nt, n0, hw, deap, as_fft3<T>(f), b_lo, nb, pitch, Gt, blockIdx.x, threadIdx.x);
}

// Sensor pairs per work-group: one in three passes (hundreds of butterflies),
// in two as many (up to 4) as leave every CU several work-groups.
template <typename T>
Fft3Raw temporal_shape(const DevPlan& p) {
  Fft3Raw f = p.f_nt3;
  if (!f.r1) return f;
  const int pairs = (p.M + 1) / 2;
  f.ls = 0;
  if (f.r3 == 1)
    while (f.ls < 2 && (pairs >> (f.ls + 1)) >= 1024) ++f.ls;
  f.QB = f.r3 | 1;
  f.QA = (f.r3 > 1 ? f.r2 * f.QB : f.r2) | 1;
  f.P = std::max(f.r1 * f.QA, f.r1 * f.r2 * f.r3) | 1;
  return f;
}

// Other lengths: passes in LDS, runtime plan. The transform's twiddles come
// from the split tables (TwSplit) in LDS behind the sequence.
template <typename T>
__device__ __forceinline__ void temporal_body(const T* __restrict__ g, int M, int Nt, int n0,
                                              const T* __restrict__ hw, const T* __restrict__ deap,
                                              FftDesc<T> fd, int b_lo, int nb, int pitch, cx<T>* __restrict__ Gt, int bx,
                                              int tid = threadIdx.x) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* buf = reinterpret_cast<cx<T>*>(smem_raw);
  const int nthr = blockDim.x;
  const int n_t = fd.n;
  const int m0 = 2 * bx;  // the pair's first sensor (one pair per group measured fastest on MI355X)
  const bool has1 = m0 + 1 < M;
  // zero padding: only the slots no sample lands in, (n - n0) mod n_t for
  // n = Nt .. n_t-1; they are disjoint from the samples' slots, so the fill
  // and the sample stores need no barrier between them
  for (int i = tid; i < n_t - Nt; i += nthr) {
    int pos = Nt + i - n0;
    if (pos < 0) pos += n_t;
    buf[lpos(pos)] = cx<T>{T(0), T(0)};
  }
  const TwSplit<T> tw = tw_split_fill(buf + lseq(n_t), fd.tw, n_t, tid, nthr);
  const T w0 = hw ? hw[m0] : T(1);
  const T w1 = has1 ? (hw ? hw[m0 + 1] : T(1)) : T(0);
  const T* g0 = g + size_t(m0) * Nt;
  const T* g1 = g + size_t(has1 ? m0 + 1 : m0) * Nt;
  staged_copy<kFftMaxV>(
      Nt, tid, nthr,
      [&](int n) {
        const T d = deap[n];
        const T a = g0[n] * w0 * d;
        const T b = has1 ? g1[n] * w1 * d : T(0);
        return cx<T>{a, b};
      },
      [&](int n, cx<T> v) {
        int pos = n - n0;
        if (pos < 0) pos += n_t;
        buf[lpos(pos)] = v;
      });
  __syncthreads();
  fft_lds_tw<T, kFftMaxV, false, false>(buf, fd, tw, 1, lseq(n_t), tid, nthr);
  for (int i = tid; i < nb; i += nthr) {
    const int b = b_lo + i;  // -n_t < b < n_t (the band fits in n_t bins)
    const int pb = b < 0 ? b + n_t : b;
    const int mb = b > 0 ? n_t - b : -b;
    const cx<T> z = buf[lpos(pb)];
    const cx<T> zm = buf[lpos(mb)];
    // transform of the real part: (Z_b + conj Z_-b)/2; of the imaginary part: (Z_b - conj Z_-b)/(2i)
    Gt[size_t(m0) * pitch + i] = cx<T>{T(0.5) * (z.x + zm.x), T(0.5) * (z.y - zm.y)};
    if (has1) Gt[size_t(m0 + 1) * pitch + i] = cx<T>{T(0.5) * (z.y + zm.y), T(-0.5) * (z.x - zm.x)};
  }
}

template <typename T>
__global__ __launch_bounds__(kTemporalThreads) void k_temporal(const T* __restrict__ g, int M, int Nt, int n0,
                                                               const T* __restrict__ hw, const T* __restrict__ deap,
                                                               FftDesc<T> fd, int b_lo, int nb, int pitch,
                                                               cx<T>* __restrict__ Gt) {
  temporal_body<T>(g, M, Nt, n0, hw, deap, fd, b_lo, nb, pitch, Gt, blockIdx.x);
}

template <typename T>
hipError_t launch_temporal(const DevPlan& p, const T* g, void* Gt, bool weighted, hipStream_t s) {
  if (p.n_t > kFftMaxV * kTemporalThreads || p.Nt > p.n_t) return hipErrorInvalidValue;
  const int pairs = (p.M + 1) / 2;
  const T* hw = weighted ? static_cast<const T*>(p.hw) : nullptr;
  const T* deap = static_cast<const T*>(p.deap);
  cx<T>* out = static_cast<cx<T>*>(Gt);
  const Fft3Raw f = temporal_shape<T>(p);
  if (f.r1) {
    const size_t lds = (size_t(f.P) << f.ls) * sizeof(cx<T>);
    const dim3 grid((pairs + (1 << f.ls) - 1) >> f.ls), block(fft3_threads(f));
    auto go = [&](auto kern) {
      hipError_t e = allow_lds(reinterpret_cast<const void*>(kern), lds);
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL(kern, grid, block, lds, s, g, p.M, p.Nt, p.n0, hw, deap, f, p.b_lo, p.nb, p.pitch_t, out);
      return hipGetLastError();
    };
    switch (three_class(f)) {
      case 16: return f.r3 == 1 ? go(&k_temporal_reg<T, 16, 1>) : go(&k_temporal_reg<T, 16, 0>);
      case 20:
        return f.r3 == 1 ? go(&k_temporal_reg<T, 20, 1>)
               : fft3_rounds(f) ? go(&k_temporal_reg<T, 20, 2>) : go(&k_temporal_reg<T, 20, 0>);
      default:
        return f.r3 == 1 ? go(&k_temporal_reg<T, 32, 1>)
               : fft3_rounds(f) ? go(&k_temporal_reg<T, 32, 2>) : go(&k_temporal_reg<T, 32, 0>);
    }
  }
  const size_t lds = size_t(temporal_lds_slots(p.n_t)) * sizeof(cx<T>);
  hipError_t e = allow_lds(reinterpret_cast<const void*>(&k_temporal<T>), lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_temporal<T>, dim3(pairs), dim3(kTemporalThreads), lds, s, g, p.M, p.Nt, p.n0, hw, deap,
                     as_desc<T>(p.f_nt), p.b_lo, p.nb, p.pitch_t, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Transpose of k_temporal with unit weights (the forward model's last step):
//   g[m][n] = a_n Re sum_b Gt'[m][b] exp(+2 pi i b (n - n0)/n_t),
// a_n = 1/phihat_t((n - n0)/n_t). Two sensors share one inverse FFT: the
// spectrum Z[k] = (X0[k] + conj X0[-k])/2 + i (X1[k] + conj X1[-k])/2 (band
// bins placed at b mod n_t) transforms to Re x0 + i Re x1. The band never
// covers a bin twice (nb <= n_t), so each of the two placement passes
// writes distinct slots.
// ---------------------------------------------------------------------------
template <typename T, int NCT>
__global__ __launch_bounds__(temporal_threads<NCT>()) void k_temporal_t(const cx<T>* __restrict__ Gt, int M, int Nt,
                                                                        int n0,
                                                               const T* __restrict__ deap, FftDesc<T> fd, int b_lo,
                                                               int nb, T* __restrict__ g) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* buf = reinterpret_cast<cx<T>*>(smem_raw);
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int n_t = fd.n;
  const int m0 = 2 * blockIdx.x;
  const bool has1 = m0 + 1 < M;
  for (int q = tid; q < n_t; q += nthr) buf[lpos(q)] = cx<T>{T(0), T(0)};
  const TwSplit<T> tw = tw_split_fill(buf + lseq(n_t), fd.tw, n_t, tid, nthr);
  __syncthreads();
  const cx<T>* x0 = Gt + size_t(m0) * nb;
  const cx<T>* x1 = Gt + size_t(m0 + 1) * nb;
  const cx<T> zero{T(0), T(0)};
  for (int i = tid; i < nb; i += nthr) {
    const int b = b_lo + i;
    const int pb = b < 0 ? b + n_t : b;
    const cx<T> a = x0[i], c = has1 ? x1[i] : zero;
    buf[lpos(pb)] = cx<T>{T(0.5) * (a.x - c.y), T(0.5) * (a.y + c.x)};
  }
  __syncthreads();
  for (int i = tid; i < nb; i += nthr) {
    const int b = b_lo + i;
    const int mb = b > 0 ? n_t - b : -b;
    const cx<T> a = x0[i], c = has1 ? x1[i] : zero;
    cx<T>& z = buf[lpos(mb)];
    z = cx<T>{z.x + T(0.5) * (a.x + c.y), z.y + T(0.5) * (c.x - a.y)};
  }
  __syncthreads();
  if constexpr (NCT > 0)
    fft_ct_tw<T, NCT, temporal_threads<NCT>(), 1, true>(buf, 1, tw, tid);
  else
    fft_lds_tw<T, kFftMaxV, true, false>(buf, fd, tw, 1, lseq(n_t), tid, nthr);
  __syncthreads();
  for (int n = tid; n < Nt; n += nthr) {
    int pos = n - n0;
    if (pos < 0) pos += n_t;
    const cx<T> z = buf[lpos(pos)];
    const T d = deap[n];
    // the caller's traces: non-temporal stores (measured faster)
    __builtin_nontemporal_store(z.x * d, g + size_t(m0) * Nt + n);
    if (has1) __builtin_nontemporal_store(z.y * d, g + size_t(m0 + 1) * Nt + n);
  }
}

template <typename T>
hipError_t launch_temporal_t(const DevPlan& p, const void* Gt, T* g, hipStream_t s) {
  if (p.n_t > kFftMaxV * kTemporalThreads || p.Nt > p.n_t || p.nb > p.n_t) return hipErrorInvalidValue;
  const size_t lds = size_t(temporal_lds_slots(p.n_t)) * sizeof(cx<T>);
  return ct_pick(CtTemporal{}, p.n_t, [&](auto c) {
    constexpr int NCT = decltype(c)::value, NT = temporal_threads<NCT>();
    static_assert(NCT <= kFftMaxV * NT, "a thread holds at most kFftMaxV values");
    hipError_t e = allow_lds(reinterpret_cast<const void*>(&k_temporal_t<T, NCT>), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_temporal_t<T, NCT>), dim3((p.M + 1) / 2), dim3(NT), lds, s,
                       static_cast<const cx<T>*>(Gt), p.M, p.Nt, p.n0, static_cast<const T*>(p.deap),
                       as_desc<T>(p.f_nt), p.b_lo, p.nb, g);
    return hipGetLastError();
  });
}

// Batched form: the problems of one variant, the class of the register form
// (+ 64 * its form) or 0 for passes in LDS.
template <typename T, int CLS, int FORM>
__global__ __launch_bounds__(kTemporalThreads, (any_waves<T, CLS>())) void k_temporal_batch(
    const TemporalBA* __restrict__ args, const int* __restrict__ prefix, int total, BatchIO io) {
  for (int slot = blockIdx.x; slot < total; slot += gridDim.x) {
    if (slot != int(blockIdx.x)) __syncthreads();  // the previous item's LDS is done with
    const int w = batch_item(slot, total);
    const int p = batch_locate(prefix, w);
    const TemporalBA a = args[p];
    const T* g = static_cast<const T*>(io.in[a.problem]);
    if constexpr (CLS > 0)
      temporal_reg_body<T, CLS, FORM>(g, a.M, a.Nt, a.n0, static_cast<const T*>(a.hw), static_cast<const T*>(a.deap),
                                     as_fft3<T>(a.f3), a.b_lo, a.nb, a.pitch_t, static_cast<cx<T>*>(a.Gt),
                                     w - prefix[p], loop_lane());
    else
      temporal_body<T>(g, a.M, a.Nt, a.n0, static_cast<const T*>(a.hw), static_cast<const T*>(a.deap),
                       view_desc<T>(a.fd), a.b_lo, a.nb, a.pitch_t, static_cast<cx<T>*>(a.Gt), w - prefix[p],
                       loop_lane());
  }
}

template <typename T>
hipError_t launch_temporal_batch(const BatchStage& st, const BatchIO& io, hipStream_t s) {
  if (st.total <= 0) return hipSuccess;
  switch (st.variant) {
    case 16: return launch_batch_kernel<TemporalBA>(&k_temporal_batch<T, 16, 0>, st, io, s);
    case 20: return launch_batch_kernel<TemporalBA>(&k_temporal_batch<T, 20, 0>, st, io, s);
    case 32: return launch_batch_kernel<TemporalBA>(&k_temporal_batch<T, 32, 0>, st, io, s);
    case 64 + 16: return launch_batch_kernel<TemporalBA>(&k_temporal_batch<T, 16, 1>, st, io, s);
    case 64 + 20: return launch_batch_kernel<TemporalBA>(&k_temporal_batch<T, 20, 1>, st, io, s);
    case 128 + 20: return launch_batch_kernel<TemporalBA>(&k_temporal_batch<T, 20, 2>, st, io, s);
    case 64 + 32: return launch_batch_kernel<TemporalBA>(&k_temporal_batch<T, 32, 1>, st, io, s);
    case 128 + 32: return launch_batch_kernel<TemporalBA>(&k_temporal_batch<T, 32, 2>, st, io, s);
    default: return launch_batch_kernel<TemporalBA>(&k_temporal_batch<T, 0, 0>, st, io, s);
  }
}

#define PATK_INST(T)                                                                      \
  template Fft3Raw temporal_shape<T>(const DevPlan&);                                     \
  template hipError_t launch_temporal<T>(const DevPlan&, const T*, void*, bool, hipStream_t); \
  template hipError_t launch_temporal_t<T>(const DevPlan&, const void*, T*, hipStream_t); \
  template hipError_t launch_temporal_batch<T>(const BatchStage&, const BatchIO&, hipStream_t);
PATK_INST(float)
PATK_INST(double)
#undef PATK_INST

}  // namespace patk
