// Equispaced part of the lateral NUFFT (Section 3.2): FFTs of the
// oversampled grid along x and y, cropping and deconvolution.
#include <hip/hip_runtime.h>

#include <cmath>

#include "kernels_common.hpp"

namespace patk {

// ---------------------------------------------------------------------------
// Stage 2: FFT along x of every grid row, keeping the Nx centred modes.
// U[b][py][px] -> V[b][jj][py], jj = j mod Nx for j in [-Nx/2, Nx/2).
// ---------------------------------------------------------------------------
// Two-pass register transform: the first pass loads straight from the grid
// rows (a wave walks along a row), the second stores straight to the columns
// (a wave walks S rows of one mode, so S*8 bytes of one line). Bound by HBM
// (the grid is read once) and by the vector ALU's DFT arithmetic; LDS is
// crossed once. In double the grid's rows come by non-temporal loads, which
// leave the caches to the columns that the y pass reads next and to the next
// call's band values: 128^3 at the default windows 326 -> 312 us (x pass 117
// -> 111, temporal 32 -> 28, y pass 45 -> 41; with cached loads it was slower
// than the LDS passes' 319), 144^3 423 -> 406, 256^3 1208 -> 1204, 192^3 at
// oversampling 1.5 550 -> 555, batches of small problems 0.90 to 1.02 times.
// In single precision, half the bytes, the
// columns fit the cache beside the grid and the y pass loses more than the x
// pass gains (256^3 at the benchmark's windows 652 -> 662 us).
template <typename T, int CLS>
__device__ __forceinline__ void fft_x_reg_body(const cx<T>* __restrict__ U, int n_y, int pu, int pv, int Nx,
                                               int b_begin,
                                               const Fft2<T>& f, cx<T>* __restrict__ V, int bx, int by,
                                               const int* __restrict__ brange, int tid) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* buf = reinterpret_cast<cx<T>*>(smem_raw);
  const int S = 1 << f.ls;
  const int n_x = f.r1 * f.r2;
  const int b = b_begin + by;
  const int py0 = bx << f.ls;
  const int nr = min(S, n_y - py0);
  const cx<T>* src = U + (size_t(by) * n_y + py0) * pu;
  {
    const int s = small_div(tid, f.r2), i = tid - s * f.r2;
    if (s < nr)
      reg_first_any<T, CLS, false>(f, buf + s * f.P, i, [&](int e) {
        const cx<T>& u = cx_at(src, unsigned(s * pu + e));
        return sizeof(T) == 8 ? nt_load(&u) : u;
      });
  }
  __syncthreads();
  const int s = tid & (S - 1), k = tid >> f.ls;
  if (k < f.r1 && s < nr) {
    // modes j = 0 .. Nx/2-1 sit at column j, j = -Nx/2 .. -1 (element
    // n_x + j) at column Nx + j; only those whose band range holds bin b
    // (|j| in [J0, J1]) are written: the y-FFT and the interpolation read no
    // others
    const int J0 = brange ? brange[2 * b] : 0, J1 = brange ? brange[2 * b + 1] : Nx;
    const int p0 = J0, p1 = min(J1, Nx / 2 - 1);                    // elements of the non-negative modes
    const int m0 = n_x - min(J1, Nx / 2), m1 = n_x - max(J0, 1);    // and of the negative ones
    // one store per output from a uniform base, at offsets that differ by
    // uniform steps (an address pair and two branches per output cost
    // registers that radix 32 does not have)
    cx<T>* dst = V + size_t(b) * Nx * pv + py0;
    const unsigned at = unsigned(k * pv + s), step = unsigned(f.r1 * pv), back = unsigned((n_x - Nx) * pv);
    reg_second_any<T, CLS, false, true>(f, buf + s * f.P, k, [&](int q, cx<T> v) {
      const int e = k + q * f.r1;
      const bool neg = e >= m0 && e <= m1;
      if (neg || (e >= p0 && e <= p1)) cx_at(dst, at + unsigned(q) * step - (neg ? back : 0u)) = v;
    });
  }
}

// Longer lengths: passes in LDS, runtime plan.
template <typename T>
__device__ __forceinline__ void fft_x_body(const cx<T>* __restrict__ U, int n_y, int pu, int pv, int Nx, int rows,
                                           int b_begin, FftDesc<T> fd, cx<T>* __restrict__ V, int wm, int bx, int by,
                                           const int* __restrict__ brange = nullptr, int tid = threadIdx.x) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* buf = reinterpret_cast<cx<T>*>(smem_raw);
  const int nthr = blockDim.x;
  const int n_x = fd.n;
  const int bstride = lseq(n_x);
  const int b = b_begin + by;
  const int py0 = bx * rows;
  const int nr = min(rows, n_y - py0);
  const cx<T>* src = U + (size_t(b - b_begin) * n_y + py0) * pu;
  cx<T>* dst = V + size_t(b) * Nx * pv + py0;
  // output mode jj of the Nx kept, centred, at its slot of the n_x transform
  auto slot = [&](int jj) {
    const int j = jj < Nx / 2 ? jj : jj - Nx;
    return lpos(j < 0 ? j + n_x : j);
  };
  // only the x modes whose band range holds bin b (|j| in [J0, J1]) are
  // written: the y-FFT and the interpolation read no others
  const int J0 = brange ? brange[2 * b] : 0, J1 = brange ? brange[2 * b + 1] : Nx;
  auto kept = [&](int jj) {
    const int aj = jj < Nx / 2 ? jj : Nx - jj;
    return aj >= J0 && aj <= J1;
  };
  cx<T>* twl = buf + rows * bstride;
  const FastDiv div_nx(n_x), div_nr(nr);
  staged_copy<kFftMaxV>(
      nr * n_x, tid, nthr,
      [&](int q) {
        const int r = div_nx(q);
        return src[size_t(r) * pu + (q - r * n_x)];
      },
      [&](int q, cx<T> v) {
        const int r = div_nx(q);
        buf[r * bstride + lpos(q - r * n_x)] = v;
      });
  // the twiddles go to LDS behind the rows (every pass reads them)
  for (int t = tid; t < fd.n; t += nthr) twl[t] = fd.tw[t];
  __syncthreads();
  fft_group<T, false>(buf, lds_twiddles(fd, twl), nr, bstride, tid, nthr, wm);
  __syncthreads();
  staged_copy<kFftMaxV>(
      nr * Nx, tid, nthr,
      [&](int q) {
        const int jj = div_nr(q);
        return kept(jj) ? buf[(q - jj * nr) * bstride + slot(jj)] : cx<T>{T(0), T(0)};
      },
      [&](int q, cx<T> v) {
        const int jj = div_nr(q);
        if (kept(jj)) dst[size_t(jj) * pv + (q - jj * nr)] = v;
      });
}

template <typename T>
__global__ __launch_bounds__(kFftThreads) void k_fft_x(const cx<T>* __restrict__ U, int n_y, int pu, int pv, int Nx,
                                                       int rows,
                                                     int b_begin, FftDesc<T> fd, cx<T>* __restrict__ V, int wm,
                                                     const int* __restrict__ brange) {
  // neighbouring groups write the two halves of each 128-byte output line:
  // keep them on one XCD so its L2 merges the halves
  const int gl = xcd_linear();
  fft_x_body<T>(U, n_y, pu, pv, Nx, rows, b_begin, fd, V, wm, gl % gridDim.x, gl / gridDim.x, brange);
}

template <typename T, int CLS>
__global__ __launch_bounds__(kFftThreads, (reg_waves<T, CLS>())) void k_fft_x_reg(const cx<T>* __restrict__ U, int n_y,
                                                                                  int pu, int pv, int Nx, int b_begin,
                                                           Fft2Raw f, cx<T>* __restrict__ V,
                                                           const int* __restrict__ brange) {
  const int gl = xcd_linear();
  fft_x_reg_body<T, CLS>(U, n_y, pu, pv, Nx, b_begin, as_fft2<T>(f), V, gl % gridDim.x, gl / gridDim.x, brange,
                         threadIdx.x);
}

template <typename T>
hipError_t launch_fft_x(const DevPlan& p, const void* U, void* V, int b_begin, int b_end, hipStream_t s) {
  if (b_begin < 0 || b_end > p.nb || b_begin >= b_end) return hipErrorInvalidValue;
  const FftCfg cfg = fft_cfg();
  const int rows = fft_seqs<T>(p.f_nx, cfg.threads, cfg.cap);
  const dim3 grid((p.n_y + rows - 1) / rows, b_end - b_begin);
  if (p.f_nx.two.r1) {
    const Fft2Raw f = fft2_shape<T>(p.f_nx, rows);
    const size_t lds = fft2_slots(f) * sizeof(cx<T>);
    return class_pick(f, [&](auto c) {
      constexpr auto kern = &k_fft_x_reg<T, decltype(c)::value>;
      hipError_t e = allow_lds(reinterpret_cast<const void*>(kern), lds);
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL(kern, grid, dim3(fft2_threads(f)), lds, s, static_cast<const cx<T>*>(U), p.n_y, p.pitch_u,
                         p.pitch_v, p.Nx, b_begin,
                         f, static_cast<cx<T>*>(V), p.brange);
      return hipGetLastError();
    });
  }
  const size_t lds = (size_t(rows) * lseq(p.n_x) + p.n_x) * sizeof(cx<T>);
  if (size_t(rows) * p.n_x > size_t(kFftMaxV) * cfg.threads || size_t(rows) * p.Nx > size_t(kFftMaxV) * cfg.threads)
    return hipErrorInvalidValue;
  hipError_t e = allow_lds(reinterpret_cast<const void*>(&k_fft_x<T>), lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_fft_x<T>, grid, dim3(cfg.threads), lds, s, static_cast<const cx<T>*>(U), p.n_y, p.pitch_u,
                     p.pitch_v, p.Nx, rows,
                     b_begin, as_desc<T>(p.f_nx), static_cast<cx<T>*>(V), cfg.wave, p.brange);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Stage 3: FFT along y, keep the Ny centred modes and transpose so the bins
// of each lateral mode are contiguous: V[b][jj][py] -> Gh[jj][kk][b]. (The
// gather divides by the window transform in x and y, eq. NED_NUFFT's 1/Psi_j:
// one factor per interpolated point instead of one per mode and bin.)
// ---------------------------------------------------------------------------
// jrange (may be nullptr): groups of bins outside the x-mode's range are
// skipped (the interpolation never reads them).
//
// Two-pass register transform (as the x pass): rows in along a row, out with
// a wave on S bins of one mode. Non-temporal loads: each band row is read
// once, and keeping it out of the caches leaves them to the spectra this
// kernel writes, which the gather reads next.
template <typename T, int CLS>
__device__ __forceinline__ void fft_y_reg_body(const cx<T>* __restrict__ V, int nb, int pv, int pg, int Nx, int Ny,
                                               const Fft2<T>& f, cx<T>* __restrict__ Gh, int bx, int jj,
                                               const int* __restrict__ jrange, int tid) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* buf = reinterpret_cast<cx<T>*>(smem_raw);
  const int S = 1 << f.ls;
  const int n_y = f.r1 * f.r2;
  const int b0 = bx << f.ls;
  const int nbc = min(S, nb - b0);
  if (jrange && (b0 + nbc - 1 < jrange[2 * jj] || b0 > jrange[2 * jj + 1])) return;
  {
    const int s = small_div(tid, f.r2), i = tid - s * f.r2;
    if (s < nbc) {
      const cx<T>* src = V + (size_t(b0) * Nx + jj) * pv;  // bin b0 + s at src + s * Nx * pv
      const unsigned at = unsigned(s) * unsigned(Nx * pv);
      reg_first_any<T, CLS, false>(f, buf + s * f.P, i, [&](int e) { return nt_load(&cx_at(src, at + unsigned(e))); });
    }
  }
  __syncthreads();
  const int s = tid & (S - 1), k = tid >> f.ls;
  if (k < f.r1 && s < nbc) {
    cx<T>* dst = Gh + size_t(jj) * Ny * pg + b0;
    const unsigned at = unsigned(k * pg + s), step = unsigned(f.r1 * pg), back = unsigned((n_y - Ny) * pg);
    reg_second_any<T, CLS, false, true>(f, buf + s * f.P, k, [&](int q, cx<T> v) {
      // element e holds mode e below Ny/2 and e - n_y from -Ny/2 on
      const int e = k + q * f.r1;
      const bool neg = e >= n_y - Ny / 2;
      if (neg || e < Ny / 2) cx_at(dst, at + unsigned(q) * step - (neg ? back : 0u)) = v;
    });
  }
}

template <typename T>
__device__ __forceinline__ void fft_y_body(const cx<T>* __restrict__ V, int nb, int pv, int pg, int Nx, int Ny,
                                           int bins,
                                           FftDesc<T> fd, cx<T>* __restrict__ Gh, int wm, int bx, int by,
                                           const int* __restrict__ jrange = nullptr, int tid = threadIdx.x) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* buf = reinterpret_cast<cx<T>*>(smem_raw);
  const int nthr = blockDim.x;
  const int n_y = fd.n;
  const int bstride = lseq(n_y);
  const int jj = by;
  const int b0 = bx * bins;
  const int nbc = min(bins, nb - b0);
  if (jrange && (b0 + nbc - 1 < jrange[2 * jj] || b0 > jrange[2 * jj + 1])) return;
  const cx<T>* src = V + (size_t(b0) * Nx + jj) * pv;  // bin b0 + bi at src + bi * Nx * pv
  const size_t bin_stride = size_t(Nx) * pv;
  cx<T>* dst = Gh + size_t(jj) * Ny * pg + b0;
  // output mode kk of the Ny kept, centred, at its slot of the n_y transform
  auto slot = [&](int kk) {
    const int k = kk < Ny / 2 ? kk : kk - Ny;
    return lpos(k < 0 ? k + n_y : k);
  };
  cx<T>* twl = buf + bins * bstride;
  const FastDiv div_ny(n_y), div_nbc(nbc);
  staged_copy<kFftMaxV>(
      nbc * n_y, tid, nthr,
      [&](int q) {
        const int bi = div_ny(q);
        return src[bi * bin_stride + (q - bi * n_y)];
      },
      [&](int q, cx<T> v) {
        const int bi = div_ny(q);
        buf[bi * bstride + lpos(q - bi * n_y)] = v;
      });
  for (int t = tid; t < fd.n; t += nthr) twl[t] = fd.tw[t];
  __syncthreads();
  fft_group<T, false>(buf, lds_twiddles(fd, twl), nbc, bstride, tid, nthr, wm);
  __syncthreads();
  staged_copy<kFftMaxV>(
      nbc * Ny, tid, nthr,
      [&](int q) {
        const int kk = div_nbc(q);
        return buf[(q - kk * nbc) * bstride + slot(kk)];
      },
      [&](int q, cx<T> v) {
        const int kk = div_nbc(q);
        dst[size_t(kk) * pg + (q - kk * nbc)] = v;
      });
}

// (x mode, bin group) of a work-group: from the list of work items inside the
// ranges, or the two-dimensional grid of all
__device__ __forceinline__ void y_item(const int* __restrict__ ylist, int gl, int& bx, int& by) {
  if (ylist) {
    const int e = ylist[gl];
    by = e >> 16;
    bx = e & 0xffff;
  } else {
    bx = gl % gridDim.x;
    by = gl / gridDim.x;
  }
}

template <typename T>
__global__ __launch_bounds__(kFftThreads) void k_fft_y(const cx<T>* __restrict__ V, int nb, int pv, int pg, int Nx,
                                                       int Ny, int bins,
                                                     FftDesc<T> fd, cx<T>* __restrict__ Gh, int wm,
                                                     const int* __restrict__ jrange, const int* __restrict__ ylist) {
  // neighbouring groups write the two halves of each 128-byte output line:
  // keep them on one XCD so its L2 merges the halves
  int bx, by;
  y_item(ylist, xcd_linear(), bx, by);
  fft_y_body<T>(V, nb, pv, pg, Nx, Ny, bins, fd, Gh, wm, bx, by, jrange);
}

template <typename T, int CLS>
__global__ __launch_bounds__(kFftThreads, (reg_waves<T, CLS>())) void k_fft_y_reg(const cx<T>* __restrict__ V, int nb,
                                                                                  int pv, int pg, int Nx, int Ny,
                                                           Fft2Raw f, cx<T>* __restrict__ Gh,
                                                           const int* __restrict__ jrange,
                                                           const int* __restrict__ ylist) {
  int bx, by;
  y_item(ylist, xcd_linear(), bx, by);
  fft_y_reg_body<T, CLS>(V, nb, pv, pg, Nx, Ny, as_fft2<T>(f), Gh, bx, by, jrange, threadIdx.x);
}

template <typename T>
hipError_t launch_fft_y(const DevPlan& p, const void* V, void* Gh, hipStream_t s) {
  const FftCfg cfg = fft_cfg();
  const int bins = fft_bins<T>(p.f_ny, cfg.threads, cfg.cap);
  const bool listed = p.ylist && p.ylist_n > 0 && p.jrange;
  const dim3 grid = listed ? dim3(p.ylist_n) : dim3((p.nb + bins - 1) / bins, p.Nx);
  const int* ylist = listed ? p.ylist : nullptr;
  if (p.f_ny.two.r1) {
    const Fft2Raw f = fft2_shape<T>(p.f_ny, bins);
    const size_t lds = fft2_slots(f) * sizeof(cx<T>);
    return class_pick(f, [&](auto c) {
      constexpr auto kern = &k_fft_y_reg<T, decltype(c)::value>;
      hipError_t e = allow_lds(reinterpret_cast<const void*>(kern), lds);
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL(kern, grid, dim3(fft2_threads(f)), lds, s, static_cast<const cx<T>*>(V), p.nb, p.pitch_v,
                         p.pitch_g, p.Nx, p.Ny, f, static_cast<cx<T>*>(Gh),
                         p.jrange, ylist);
      return hipGetLastError();
    });
  }
  const size_t lds = (size_t(bins) * lseq(p.n_y) + p.n_y) * sizeof(cx<T>);
  if (size_t(bins) * p.n_y > size_t(kFftMaxV) * cfg.threads || size_t(bins) * p.Ny > size_t(kFftMaxV) * cfg.threads)
    return hipErrorInvalidValue;
  hipError_t e = allow_lds(reinterpret_cast<const void*>(&k_fft_y<T>), lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_fft_y<T>, grid, dim3(cfg.threads), lds, s, static_cast<const cx<T>*>(V), p.nb, p.pitch_v,
                     p.pitch_g, p.Nx, p.Ny,
                     bins, as_desc<T>(p.f_ny), static_cast<cx<T>*>(Gh), cfg.wave, p.jrange, ylist);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Transposes for the forward model (conjugate transposes of k_fft_y and
// k_fft_x: embed the cropped modes into the oversampled length with zeros,
// inverse FFT).
// Gh'[j][k][b] -> V'[b][j][py] = dcx_j sum_k dcy_k Gh'[j][k][b] e^{+2 pi i k py/n_y}
// ---------------------------------------------------------------------------
// Two-pass register form (the forward model): a wave of the first pass walks
// the S bins of one mode, the slots between the kept modes are zeros, and the
// second pass writes along the rows (of pv elements).
template <typename T, int CLS>
__global__ __launch_bounds__(kFftThreads, (reg_waves<T, CLS>())) void k_fft_y_t_reg(
    const cx<T>* __restrict__ Gh, int nb, int Nx, int Ny, const T* __restrict__ dcx, const T* __restrict__ dcy,
    Fft2Raw fr, cx<T>* __restrict__ V, int pv, const int* __restrict__ jrange, const int* __restrict__ ylist) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* buf = reinterpret_cast<cx<T>*>(smem_raw);
  const Fft2<T> f = as_fft2<T>(fr);
  const int tid = threadIdx.x;
  const int S = 1 << f.ls;
  const int n_y = f.r1 * f.r2;
  // (an XCD-grouped order measured slower here)
  const int jj = ylist ? ylist[blockIdx.x] >> 16 : int(blockIdx.y);
  const int b0 = (ylist ? ylist[blockIdx.x] & 0xffff : int(blockIdx.x)) << f.ls;
  const int nbc = min(S, nb - b0);
  // bins outside the x-mode's range hold zeros that nothing reads: skipped
  if (jrange && (b0 + nbc - 1 < jrange[2 * jj] || b0 > jrange[2 * jj + 1])) return;
  {
    const int s = tid & (S - 1), i = tid >> f.ls;
    if (i < f.r2 && s < nbc) {
      const T cxj = dcx[jj];
      const cx<T>* src = Gh + size_t(jj) * Ny * nb + b0 + s;
      reg_first_any<T, CLS, true>(f, buf + s * f.P, i, [&](int e) {
        const bool in = e < Ny / 2 || e >= n_y - Ny / 2;
        const int kk = e < Ny / 2 ? e : in ? e - (n_y - Ny) : 0;  // the loads carry no branch
        const T sc = in ? cxj * dcy[kk] : T(0);
        const cx<T> v = cx_at(src, unsigned(kk * nb));
        return cx<T>{in ? v.x * sc : T(0), in ? v.y * sc : T(0)};
      });
    }
  }
  __syncthreads();
  const int s = small_div(tid, f.r1), k = tid - s * f.r1;
  if (s < nbc) {
    cx<T>* v0 = V + (size_t(b0) * Nx + jj) * pv;  // bin b0 + s at v0 + s * Nx * pv
    const unsigned at = unsigned(s) * unsigned(Nx * pv) + unsigned(k);
    reg_second_any<T, CLS, true>(f, buf + s * f.P, k, [&](int q, cx<T> v) {
      // non-temporal: streams out once (measured faster for the fused reader)
      nt_store(&cx_at(v0, at + unsigned(q * f.r1)), v);
    });
  }
}

template <typename T>
hipError_t launch_fft_y_t_reg(const DevPlan& p, const void* Gh, void* V, hipStream_t s) {
  if (!p.f_ny.two.r1) return hipErrorInvalidValue;
  const FftCfg cfg = fft_cfg();
  const int bins = fft_bins<T>(p.f_ny, cfg.threads, cfg.cap);
  const bool listed = p.ylist && p.ylist_n > 0 && p.jrange;
  const dim3 grid = listed ? dim3(p.ylist_n) : dim3((p.nb + bins - 1) / bins, p.Nx);
  const Fft2Raw f = fft2_shape<T>(p.f_ny, bins);
  const size_t lds = fft2_slots(f) * sizeof(cx<T>);
  return class_pick(f, [&](auto c) {
    constexpr auto kern = &k_fft_y_t_reg<T, decltype(c)::value>;
    hipError_t e = allow_lds(reinterpret_cast<const void*>(kern), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, grid, dim3(fft2_threads(f)), lds, s, static_cast<const cx<T>*>(Gh), p.nb, p.Nx, p.Ny,
                       static_cast<const T*>(p.dcx), static_cast<const T*>(p.dcy), f, static_cast<cx<T>*>(V),
                       p.pitch_v, p.jrange, listed ? p.ylist : nullptr);
    return hipGetLastError();
  });
}

// Passes in LDS: other lengths, the two-kernel interpolation, and the position
// derivatives at every length (whose digits stay as they are).
template <typename T, int NCT>
__global__ __launch_bounds__(kFftThreads) void k_fft_y_t(const cx<T>* __restrict__ Gh, int nb, int Nx, int Ny,
                                                       int bins, const T* __restrict__ dcx,
                                                       const T* __restrict__ dcy, FftDesc<T> fd,
                                                       cx<T>* __restrict__ V, const int* __restrict__ jrange,
                                                       const int* __restrict__ ytlist) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* buf = reinterpret_cast<cx<T>*>(smem_raw);
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int n_y = NCT > 0 ? NCT : fd.n;
  const int bstride = lseq(n_y);
  // (an XCD-grouped order measured slower here); with ytlist a one-dimensional
  // grid over the ranges' bins (those outside hold zeros that nothing reads)
  const int item = ytlist ? ytlist[blockIdx.x] : 0;
  const int jj = ytlist ? item >> 16 : int(blockIdx.y);
  const int b0 = ytlist ? item & 0xffff : int(blockIdx.x) * bins;
  const int nbc = min(bins, (ytlist ? jrange[2 * jj + 1] + 1 : nb) - b0);
  const int gap = n_y - Ny;  // zero slots k = Ny/2 .. n_y - Ny/2 - 1
  const T cxj = dcx[jj];
  const cx<T>* src = Gh + size_t(jj) * Ny * nb + b0;
  auto slot = [&](int kk) {
    const int k = kk < Ny / 2 ? kk : kk - Ny;
    return lpos(k < 0 ? k + n_y : k);
  };
  cx<T>* twl = buf + bins * bstride;
  if constexpr (NCT > 0) {
    // compile-time geometry (bins = ROWS, 256 threads): no index divisions
    constexpr int ROWS = ct_maxb(NCT, kFftCap), BS = lseq(NCT);
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
      if (r < nbc)
        for (int c = tid; c < gap; c += kFftThreads) buf[r * BS + lpos(Ny / 2 + c)] = cx<T>{T(0), T(0)};
    const cx<T>* s0 = src + size_t(tid / ROWS) * nb + tid % ROWS;
    const size_t step = size_t(kFftThreads / ROWS) * nb;
    staged_cols<ROWS, kFftThreads, (NCT * ROWS + kFftThreads - 1) / kFftThreads>(  // Ny < n_y = NCT
        Ny, nbc, tid,
        [&](int kk, int, int u) {
          const T sc = cxj * dcy[kk];
          const cx<T> v = s0[u * step];
          return cx<T>{v.x * sc, v.y * sc};
        },
        [&](int kk, int bi, int, cx<T> v) { buf[bi * BS + slot(kk)] = v; });
    for (int t = tid; t < NCT; t += kFftThreads) twl[t] = fd.tw[t];
    __syncthreads();
    fft_ct<T, NCT, kFftThreads, ROWS, true>(buf, nbc, twl, tid);
    __syncthreads();
    cx<T>* v0 = V + (size_t(b0) * Nx + jj) * NCT;  // bin b0 + r at v0 + r * Nx * NCT
    const size_t bin_stride = size_t(Nx) * NCT;
    staged_rows<ROWS, NCT, kFftThreads>(
        nbc, tid, [&](int r, int c) { return buf[r * BS + lpos(c)]; },
        // non-temporal: streams out once (measured faster for the fused reader)
        [&](int r, int c, cx<T> v) { nt_store(v0 + r * bin_stride + c, v); });
  } else {
    const FastDiv div_gap(gap), div_nbc(nbc), div_ny(n_y);
    for (int q = tid; q < nbc * gap; q += nthr) {
      const int bi = div_gap(q);
      buf[bi * bstride + lpos(Ny / 2 + (q - bi * gap))] = cx<T>{T(0), T(0)};
    }
    staged_copy<kFftMaxV>(
        nbc * Ny, tid, nthr,
        [&](int q) {
          const int kk = div_nbc(q);
          const T sc = cxj * dcy[kk];
          const cx<T> v = src[size_t(kk) * nb + (q - kk * nbc)];
          return cx<T>{v.x * sc, v.y * sc};
        },
        [&](int q, cx<T> v) {
          const int kk = div_nbc(q);
          buf[(q - kk * nbc) * bstride + slot(kk)] = v;
        });
    for (int t = tid; t < fd.n; t += nthr) twl[t] = fd.tw[t];
    __syncthreads();
    fft_lds<T, kFftMaxV, true, false>(buf, lds_twiddles(fd, twl), nbc, bstride, tid, nthr);
    __syncthreads();
    staged_copy<kFftMaxV>(
        nbc * n_y, tid, nthr,
        [&](int q) {
          const int bi = div_ny(q);
          return buf[bi * bstride + lpos(q - bi * n_y)];
        },
        [&](int q, cx<T> v) {  // non-temporal: streams out once (measured faster for the fused reader)
          const int bi = div_ny(q);
          nt_store(V + (size_t(b0 + bi) * Nx + jj) * n_y + (q - bi * n_y), v);
        });
  }
}

template <typename T>
hipError_t launch_fft_y_t(const DevPlan& p, const void* Gh, void* V, hipStream_t s) {
  const FftCfg cfg = fft_cfg();
  const int bins = fft_batch<T>(p.n_y, cfg.threads, cfg.cap);  // the plan's ytlist is in these
  const size_t lds = (size_t(bins) * lseq(p.n_y) + p.n_y) * sizeof(cx<T>);
  if (size_t(bins) * p.n_y > size_t(kFftMaxV) * cfg.threads || size_t(bins) * p.Ny > size_t(kFftMaxV) * cfg.threads)
    return hipErrorInvalidValue;
  auto go = [&](auto kern, int nct) {
    // the compile-time kernels take their geometry from the length
    if (nct > 0 && (bins != ct_maxb(nct, kFftCap) || cfg.threads != kFftThreads)) return hipErrorInvalidValue;
    hipError_t e = allow_lds(reinterpret_cast<const void*>(kern), lds);
    if (e != hipSuccess) return e;
    const bool listed = p.ytlist && p.ytlist_n > 0 && p.jrange;
    const dim3 grid = listed ? dim3(p.ytlist_n) : dim3((p.nb + bins - 1) / bins, p.Nx);
    hipLaunchKernelGGL(kern, grid, dim3(cfg.threads), lds, s, static_cast<const cx<T>*>(Gh), p.nb, p.Nx, p.Ny,
                       bins, static_cast<const T*>(p.dcx), static_cast<const T*>(p.dcy), as_desc<T>(p.f_ny),
                       static_cast<cx<T>*>(V), p.jrange, listed ? p.ytlist : nullptr);
    return hipGetLastError();
  };
  return ct_pick(CtLateral{}, p.n_y, [&](auto c) { return go(&k_fft_y_t<T, decltype(c)::value>, decltype(c)::value); });
}

// V'[b][j][py] -> U'[b - b_begin][py][px] = sum_j V'[b][j][py] e^{+2 pi i j px/n_x}
template <typename T>
__global__ __launch_bounds__(kFftThreads) void k_fft_x_t(const cx<T>* __restrict__ V, int n_y, int Nx, int rows,
                                                       int b_begin, FftDesc<T> fd, cx<T>* __restrict__ U) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* buf = reinterpret_cast<cx<T>*>(smem_raw);
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int n_x = fd.n;
  const int bstride = lseq(n_x);
  const int b = b_begin + blockIdx.y;
  const int py0 = blockIdx.x * rows;
  const int nr = min(rows, n_y - py0);
  const int gap = n_x - Nx;
  const FastDiv div_gap(gap), div_nr(nr), div_nx(n_x);
  for (int q = tid; q < nr * gap; q += nthr) {
    const int r = div_gap(q);
    buf[r * bstride + lpos(Nx / 2 + (q - r * gap))] = cx<T>{T(0), T(0)};
  }
  const cx<T>* src = V + size_t(b) * Nx * n_y + py0;
  staged_copy<kFftMaxV>(
      nr * Nx, tid, nthr,
      [&](int q) {
        const int jj = div_nr(q);
        return src[size_t(jj) * n_y + (q - jj * nr)];
      },
      [&](int q, cx<T> v) {
        const int jj = div_nr(q);
        const int j = jj < Nx / 2 ? jj : jj - Nx;
        buf[(q - jj * nr) * bstride + lpos(j < 0 ? j + n_x : j)] = v;
      });
  __syncthreads();
  fft_lds<T, kFftMaxV, true, false>(buf, fd, nr, bstride, tid, nthr);
  __syncthreads();
  cx<T>* dst = U + (size_t(b - b_begin) * n_y + py0) * n_x;
  staged_copy<kFftMaxV>(
      nr * n_x, tid, nthr,
      [&](int q) {
        const int r = div_nx(q);
        return buf[r * bstride + lpos(q - r * n_x)];
      },
      [&](int q, cx<T> v) { dst[q] = v; });
}

template <typename T>
hipError_t launch_fft_x_t(const DevPlan& p, const void* V, void* U, int b_begin, int b_end, hipStream_t s) {
  const FftCfg cfg = fft_cfg();
  const int rows = fft_batch<T>(p.n_x, cfg.threads, cfg.cap);
  const size_t lds = size_t(rows) * lseq(p.n_x) * sizeof(cx<T>);
  if (size_t(rows) * p.n_x > size_t(kFftMaxV) * cfg.threads || size_t(rows) * p.Nx > size_t(kFftMaxV) * cfg.threads ||
      b_begin < 0 || b_end > p.nb || b_begin >= b_end)
    return hipErrorInvalidValue;
  hipError_t e = allow_lds(reinterpret_cast<const void*>(&k_fft_x_t<T>), lds);
  if (e != hipSuccess) return e;
  dim3 grid((p.n_y + rows - 1) / rows, b_end - b_begin);
  hipLaunchKernelGGL(k_fft_x_t<T>, grid, dim3(cfg.threads), lds, s, static_cast<const cx<T>*>(V), p.n_y, p.Nx, rows,
                     b_begin, as_desc<T>(p.f_nx), static_cast<cx<T>*>(U));
  return hipGetLastError();
}

// Batched forms of the x and y passes: a launch holds the problems of one
// variant, CLS the class of their two-pass transforms or 0 for the longer
// lengths.
template <typename T, int CLS>
__global__ __launch_bounds__(kFftThreads, (any_waves<T, CLS>())) void k_fft_x_batch(const FftXBA* __restrict__ args,
                                                             const int* __restrict__ prefix, int total,
                                                             BatchIO io) {
  for (int slot = blockIdx.x; slot < total; slot += gridDim.x) {
    if (slot != int(blockIdx.x)) __syncthreads();  // the previous item's LDS is done with
    const int w = batch_item(slot, total);
    const int p = batch_locate(prefix, w);
    const FftXBA a = args[p];
    const int local = w - prefix[p];
    const int by = local / a.gx;
    if constexpr (CLS > 0)
      fft_x_reg_body<T, CLS>(static_cast<const cx<T>*>(a.U), a.n_y, a.pitch_u, a.pitch_v, a.Nx, 0, as_fft2<T>(a.f2),
                             static_cast<cx<T>*>(a.V), local - by * a.gx, by, a.brange, loop_lane());
    else
      fft_x_body<T>(static_cast<const cx<T>*>(a.U), a.n_y, a.pitch_u, a.pitch_v, a.Nx, a.rows, 0, view_desc<T>(a.fd),
                    static_cast<cx<T>*>(a.V), 0, local - by * a.gx, by, a.brange, loop_lane());
  }
}

template <typename T, int CLS>
__global__ __launch_bounds__(kFftThreads, (any_waves<T, CLS>())) void k_fft_y_batch(const FftYBA* __restrict__ args,
                                                             const int* __restrict__ prefix, int total,
                                                             BatchIO io) {
  for (int slot = blockIdx.x; slot < total; slot += gridDim.x) {
    if (slot != int(blockIdx.x)) __syncthreads();  // the previous item's LDS is done with
    const int w = batch_item(slot, total);
    const int p = batch_locate(prefix, w);
    const FftYBA a = args[p];
    const int local = w - prefix[p];
    int by = local / a.gx, bx = local - by * a.gx;
    if (a.ylist) {  // the problem's work items inside its ranges
      const int e = a.ylist[local];
      by = e >> 16;
      bx = e & 0xffff;
    }
    if constexpr (CLS > 0)
      fft_y_reg_body<T, CLS>(static_cast<const cx<T>*>(a.V), a.nb, a.pitch_v, a.pitch_g, a.Nx, a.Ny, as_fft2<T>(a.f2),
                             static_cast<cx<T>*>(a.Gh), bx, by,
                             a.jrange, loop_lane());
    else
      fft_y_body<T>(static_cast<const cx<T>*>(a.V), a.nb, a.pitch_v, a.pitch_g, a.Nx, a.Ny, a.bins, view_desc<T>(a.fd),
                    static_cast<cx<T>*>(a.Gh), 0, bx, by, a.jrange,
                    loop_lane());
  }
}

template <typename T>
hipError_t launch_fft_x_batch(const BatchStage& st, const BatchIO& io, hipStream_t s) {
  if (st.total <= 0) return hipSuccess;
  switch (st.variant) {
    case 16: return launch_batch_kernel<FftXBA>(&k_fft_x_batch<T, 16>, st, io, s);
    case 20: return launch_batch_kernel<FftXBA>(&k_fft_x_batch<T, 20>, st, io, s);
    case 32: return launch_batch_kernel<FftXBA>(&k_fft_x_batch<T, 32>, st, io, s);
    default: return launch_batch_kernel<FftXBA>(&k_fft_x_batch<T, 0>, st, io, s);
  }
}

template <typename T>
hipError_t launch_fft_y_batch(const BatchStage& st, const BatchIO& io, hipStream_t s) {
  if (st.total <= 0) return hipSuccess;
  switch (st.variant) {
    case 16: return launch_batch_kernel<FftYBA>(&k_fft_y_batch<T, 16>, st, io, s);
    case 20: return launch_batch_kernel<FftYBA>(&k_fft_y_batch<T, 20>, st, io, s);
    case 32: return launch_batch_kernel<FftYBA>(&k_fft_y_batch<T, 32>, st, io, s);
    default: return launch_batch_kernel<FftYBA>(&k_fft_y_batch<T, 0>, st, io, s);
  }
}

#define PATK_INST(T)                                                                    \
  template hipError_t launch_fft_x<T>(const DevPlan&, const void*, void*, int, int, hipStream_t); \
  template hipError_t launch_fft_y<T>(const DevPlan&, const void*, void*, hipStream_t);          \
  template hipError_t launch_fft_y_t<T>(const DevPlan&, const void*, void*, hipStream_t);        \
  template hipError_t launch_fft_x_t<T>(const DevPlan&, const void*, void*, int, int, hipStream_t); \
  template hipError_t launch_fft_x_batch<T>(const BatchStage&, const BatchIO&, hipStream_t); \
  template hipError_t launch_fft_y_batch<T>(const BatchStage&, const BatchIO&, hipStream_t);
PATK_INST(float)
PATK_INST(double)
#undef PATK_INST
template hipError_t launch_fft_y_t_reg<float>(const DevPlan&, const void*, void*, hipStream_t);
template <>
hipError_t launch_fft_y_t_reg<double>(const DevPlan&, const void*, void*, hipStream_t) {
  return hipErrorInvalidValue;  // goes with the fused kernel: fused_reg_ok<double> is false
}

}  // namespace patk
