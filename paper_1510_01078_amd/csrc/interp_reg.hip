// Forward model's x transform fused with the interpolation to the sensors
// (the transpose of the lateral gridding and its x transform), with the rows'
// transforms as two register passes.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "interp_sensor.hpp"

namespace patk {

// ---------------------------------------------------------------------------
// As k_fft_x_interp: a work-group owns one strip of FS home-tile rows (plus
// the footprint's halo: R rows) and a run of bins. Per bin the first pass
// loads the kept x modes of every row from V' (a wave walks along y, zeros
// outside the bin's x-mode range), the second leaves the grid rows in LDS in
// natural order, and every sensor whose footprint origin lies in the strip
// sums its footprint there. The rows cross LDS three times before the
// footprint sums read them, eight times when they were staged and transformed
// by three passes in LDS.
// ---------------------------------------------------------------------------
// Threads: as the form with passes in LDS; radices above 20 take three waves
// per SIMD for their registers.
template <int CLS, int FS>
__host__ __device__ constexpr int reg_threads() { return FS == 2 && CLS == 32 ? 768 : kFusedThreads * FS; }

template <typename T, int W, int CLS, int FS>
__global__ __launch_bounds__((reg_threads<CLS, FS>())) void k_fft_x_interp_reg(
    const cx<T>* __restrict__ V, int nb, int pv, int Nx, int n_y, int tiles_x, int nchunks, int bins,
    const int* __restrict__ home_off, const int* __restrict__ home_sens, const int* __restrict__ sbx,
    const int* __restrict__ sby, const T* __restrict__ swx, const T* __restrict__ swy, Fft2Raw fr,
    const int* __restrict__ brange, cx<T>* __restrict__ Gt) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* buf = reinterpret_cast<cx<T>*>(smem_raw);
  const Fft2<T> f = as_fft2<T>(fr);
  constexpr int R = fused_rows<W, FS>();
  const int chunk = blockIdx.x % nchunks;  // bins vary fastest: neighbouring groups share the strip's sensors
  const int strip = blockIdx.x / nchunks;
  const int tiles_y = (n_y + kSpreadTile - 1) / kSpreadTile;
  const int q0 = home_off[strip * FS * tiles_x], q1 = home_off[min(strip * FS + FS, tiles_y) * tiles_x];
  if (q0 == q1) return;
  const int n_x = f.r1 * f.r2;
  const int py0 = strip * FS * kSpreadTile;
  const int b0 = chunk * bins, b1 = min(nb, b0 + bins);
  const int tid = threadIdx.x, nthr = blockDim.x;
  const size_t plane = size_t(Nx) * pv;
  constexpr int HELD = reg_held<T, W, CLS>();
  cx<T> held[HELD > 0 ? HELD : 1][kFusedBins];
  for (int b = b0; b < b1; ++b) {
    const cx<T>* src = V + size_t(b) * plane;
    // elements of the x modes this bin's range holds (others are zero and not written)
    const int J0 = brange ? brange[2 * b] : 0, J1 = brange ? brange[2 * b + 1] : Nx;
    const int p0 = J0, p1 = min(J1, Nx / 2 - 1);
    const int m0 = n_x - min(J1, Nx / 2), m1 = n_x - max(J0, 1);
    for (int t = tid; t < R * f.r2; t += nthr) {
      const int i = t / R, r = t - i * R;
      const unsigned py = unsigned((py0 + r) % n_y);  // periodic in y; short axes wrap more than once
      reg_first_any<T, CLS, true>(f, buf + r * f.P, i, [&](int e) {
        const bool pos = e >= p0 && e <= p1, neg = e >= m0 && e <= m1;
        const int jj = pos ? e : neg ? e - (n_x - Nx) : 0;  // the loads carry no branch
        const cx<T> v = cx_at(src, pos || neg ? unsigned(jj * pv) + py : 0u);
        return cx<T>{pos || neg ? v.x : T(0), pos || neg ? v.y : T(0)};
      });
    }
    __syncthreads();
    {
      const int k = tid / R, r = tid - k * R;
      cx<T>* seq = buf + r * f.P;
      reg_second_in_lds_any<T, CLS, true>(f, seq + k * f.Q, k < f.r1,
                                          [&](int q, cx<T> v) { seq[k + q * f.r1] = v; });
    }
    __syncthreads();
    // the first HELD sensors of every thread keep their values in registers
    // until the group's last bin (shifted one place per bin), so each
    // sensor's run of bins goes out in one burst
#pragma unroll
    for (int k = 0; k < HELD; ++k) {
      const int q = q0 + tid + k * nthr;
      cx<T> val{T(0), T(0)};
      if (q < q1) {
        FusedSensor<T, W> s;
        fused_sensor_load<T, W, false>(s, home_sens[q], py0, n_x, sbx, sby, swx, swy);
        val = fused_sensor_sum<T, W>(s, buf, f.P);
      }
#pragma unroll
      for (int j = 0; j + 1 < kFusedBins; ++j) held[k][j] = held[k][j + 1];
      held[k][kFusedBins - 1] = val;
    }
    for (int q = q0 + tid + HELD * nthr; q < q1; q += nthr) {
      FusedSensor<T, W> s;
      fused_sensor_load<T, W, false>(s, home_sens[q], py0, n_x, sbx, sby, swx, swy);
      Gt[size_t(s.m) * nb + b] = fused_sensor_sum<T, W>(s, buf, f.P);
    }
    __syncthreads();
  }
  // held[k][j] is bin b0 + j - (kFusedBins - nbin)
  const int nbin = b1 - b0;
#pragma unroll
  for (int k = 0; k < HELD; ++k) {
    const int q = q0 + tid + k * nthr;
    if (q < q1) {
      cx<T>* g = Gt + size_t(home_sens[q]) * nb + b0;  // bin b0 + i is held[k][i + kFusedBins - nbin]
#pragma unroll
      for (int j = 0; j < kFusedBins; ++j)
        if (j >= kFusedBins - nbin) g[j - (kFusedBins - nbin)] = held[k][j];
    }
  }
}

// LDS layout of the rows: the exchange and the natural order in turn, an odd
// pitch (a wave walks the rows of one index).
template <typename T>
static Fft2Raw fused_shape(const DevPlan& p) {
  Fft2Raw f = p.f_nx.two;
  f.Q = f.r2 | 1;
  f.P = std::max(f.r1 * f.Q, f.r1 * f.r2) | 1;
  return f;
}

template <typename T>
bool fused_reg_ok(const DevPlan& p, size_t lds_limit) {
  const int FS = p.fused_strip;
  const Fft2Raw f = fused_shape<T>(p);
  const int R = FS * kSpreadTile + p.w_xy - 1;
  // FP32 (in FP64 the radices spill); the second pass works in place: one
  // butterfly per thread
  const int threads = FS == 2 && reg_class(f) == 32 ? reg_threads<32, 2>() : kFusedThreads * FS;
  return sizeof(T) == 4 && f.r1 && R * f.r1 <= threads && size_t(R) * f.P * sizeof(cx<T>) <= lds_limit;
}

template <typename T, int W, int CLS, int FS>
static hipError_t launch_reg_wcs(const DevPlan& p, const void* V, void* Gt, hipStream_t s) {
  constexpr auto kern = &k_fft_x_interp_reg<T, W, CLS, FS>;
  const Fft2Raw f = fused_shape<T>(p);
  const size_t lds = size_t(fused_rows<W, FS>()) * f.P * sizeof(cx<T>);
  hipError_t e = allow_lds(reinterpret_cast<const void*>(kern), lds);
  if (e != hipSuccess) return e;
  const long long strips = (p.tiles_y + FS - 1) / FS;
  static std::atomic<unsigned long long> memo{0};
  const int bins =
      fused_bins(reinterpret_cast<const void*>(kern), reg_threads<CLS, FS>(), lds, strips, p.nb, p.tiles_y, memo);
  const int nchunks = (p.nb + bins - 1) / bins;
  hipLaunchKernelGGL(kern, dim3((unsigned)(strips * nchunks)), dim3(reg_threads<CLS, FS>()), lds, s,
                     static_cast<const cx<T>*>(V), p.nb, p.pitch_v, p.Nx, p.n_y, p.tiles_x, nchunks, bins, p.home_off,
                     p.home_sens, p.sbx, p.sby, static_cast<const T*>(p.swx), static_cast<const T*>(p.swy), f,
                     p.brange, static_cast<cx<T>*>(Gt));
  return hipGetLastError();
}

template <typename T, int W>
static hipError_t launch_reg_w(const DevPlan& p, const void* V, void* Gt, hipStream_t s) {
  return class_pick(p.f_nx.two, [&](auto c) {
    constexpr int CLS = decltype(c)::value;
    return p.fused_strip == 2 ? launch_reg_wcs<T, W, CLS, 2>(p, V, Gt, s) : launch_reg_wcs<T, W, CLS, 1>(p, V, Gt, s);
  });
}

template <typename T>
hipError_t launch_fft_x_interp_reg(const DevPlan& p, const void* V, void* Gt, hipStream_t s) {
  if (!p.f_nx.two.r1 || p.Nx > p.n_x) return hipErrorInvalidValue;
  switch (p.w_xy) {
    case 2: return launch_reg_w<T, 2>(p, V, Gt, s);
    case 4: return launch_reg_w<T, 4>(p, V, Gt, s);
    case 6: return launch_reg_w<T, 6>(p, V, Gt, s);
    case 8: return launch_reg_w<T, 8>(p, V, Gt, s);
    case 10: return launch_reg_w<T, 10>(p, V, Gt, s);
    case 12: return launch_reg_w<T, 12>(p, V, Gt, s);
    case 14: return launch_reg_w<T, 14>(p, V, Gt, s);
    case 16: return launch_reg_w<T, 16>(p, V, Gt, s);
    default: return hipErrorInvalidValue;
  }
}

#define PATK_INST(T) template hipError_t launch_fft_x_interp_reg<T>(const DevPlan&, const void*, void*, hipStream_t); \
  template bool fused_reg_ok<T>(const DevPlan&, size_t);
PATK_INST(float)
#undef PATK_INST
template bool fused_reg_ok<double>(const DevPlan&, size_t);
template <>
hipError_t launch_fft_x_interp_reg<double>(const DevPlan&, const void*, void*, hipStream_t) {
  return hipErrorInvalidValue;  // fused_reg_ok<double> is false
}

}  // namespace patk
