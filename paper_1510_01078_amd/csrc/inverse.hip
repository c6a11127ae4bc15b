// Equispaced inverse 3-D FFT of the weighted spectrum (the last step of the
// NEDNER list in Section 3), and its transpose for the forward model.
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "kernels_common.hpp"

namespace patk {

// ---------------------------------------------------------------------------
// Stage 5: equispaced inverse 3-D FFT (step 3 of the NEDNER list). The x pass
// runs with the gather; here the in-place inverse transform along y of
// F[jj][kk][l], l = 0..Nz/2-1 (rows of `pitch` elements; the plane l = Nz/2 is
// zero and not stored), then a complex-to-real transform along z. Of the
// transposes, the forward model's take the same rows and register passes, the
// position derivatives' packed rows with the plane and the passes in LDS.
// ---------------------------------------------------------------------------

// Two-pass register transform along x or y, in place: each pass's threads walk
// the nl <= S z modes at `base`, element e of mode s at base[e * stride + s]
// (one line of 128 bytes where S = 16). Bound by HBM.
template <typename T, int CLS, bool INV>
__device__ __forceinline__ void cfft_reg_body(cx<T>* __restrict__ base, unsigned stride, int nl, const Fft2<T>& f,
                                              int tid) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* buf = reinterpret_cast<cx<T>*>(smem_raw);
  const int s = tid & ((1 << f.ls) - 1), i = tid >> f.ls;
  const bool in = s < nl;
  cx<T>* b = base + s;
  if (in && i < f.r2)
    reg_first_any<T, CLS, INV>(f, buf + s * f.P, i, [&](int e) { return cx_at(b, unsigned(e) * stride); });
  __syncthreads();
  if (in && i < f.r1)
    reg_second_any<T, CLS, INV>(f, buf + s * f.P, i,
                                [&](int q, cx<T> v) { cx_at(b, unsigned(i + q * f.r1) * stride) = v; });
}

template <typename T, int CLS>
__device__ __forceinline__ void cfft_y_reg_body(cx<T>* __restrict__ F, int Lz, int pitch, const Fft2<T>& f, int bx,
                                                int jj, int tid) {
  const int l0 = bx << f.ls;
  cfft_reg_body<T, CLS, true>(F + size_t(jj) * (f.r1 * f.r2) * pitch + l0, unsigned(pitch),
                              min(1 << f.ls, Lz - l0), f, tid);
}

template <typename T, int CLS>
__global__ __launch_bounds__(kInvYThreads, (reg_waves<T, CLS>())) void k_cfft_y_reg(cx<T>* __restrict__ F, int Lz,
                                                                                   int pitch, Fft2Raw f) {
  // neighbouring groups share the 128-byte lines of the z runs: keep them on one XCD
  const int gl = xcd_linear();
  cfft_y_reg_body<T, CLS>(F, Lz, pitch, as_fft2<T>(f), gl % gridDim.x, gl / gridDim.x, threadIdx.x);
}

// Forward model: element stride and stride of the other axis' index (the grid's y)
template <typename T, int CLS>
__global__ __launch_bounds__(kInvYThreads, (reg_waves<T, CLS>())) void k_cfft_fwd_reg(cx<T>* __restrict__ F, int Lz,
                                                                                     unsigned stride, unsigned other,
                                                                                     Fft2Raw f) {
  const int gl = xcd_linear();
  const int by = gl / int(gridDim.x), l0 = (gl - by * int(gridDim.x)) << f.ls;
  cfft_reg_body<T, CLS, false>(F + size_t(by) * other + l0, stride, min(1 << f.ls, Lz - l0), as_fft2<T>(f),
                               threadIdx.x);
}

// Forward model's real-to-complex z pass: two real rows share one complex
// transform, Z = FFT(x0 + i x1), loaded as the first pass's inputs; from its
// natural order in LDS X0[l] = (Z[l] + conj Z[-l])/2 and X1[l] = (Z[l] - conj
// Z[-l])/(2i), l < Nz/2 (the transposed interpolation reads no l = Nz/2).
template <typename T, int CLS>
__global__ __launch_bounds__(kFftThreads, (reg_waves<T, CLS>())) void k_r2c_reg(const T* __restrict__ in,
                                                                               long long nrows, int pitch, Fft2Raw fr,
                                                                               cx<T>* __restrict__ D) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* buf = reinterpret_cast<cx<T>*>(smem_raw);
  const Fft2<T> f = as_fft2<T>(fr);
  const int tid = threadIdx.x;
  const int Nz = f.r1 * f.r2, Lz = Nz / 2;
  const long long r0 = (long long)blockIdx.x * (2 << f.ls);
  const int nr = (int)min((long long)(2 << f.ls), nrows - r0);
  const int np = (nr + 1) / 2;
  int s = small_div(tid, f.r2), i = tid - s * f.r2;
  if (s < np) {
    const T* row = in + (r0 + 2 * s) * Nz;
    const bool two = 2 * s + 1 < nr;
    const int next = two ? Nz : 0;
    reg_first_any<T, CLS, false>(f, buf + s * f.P, i, [&](int e) {
      const T a = row[e], c = row[e + next];
      return cx<T>{a, two ? c : T(0)};
    });
  }
  __syncthreads();
  s = small_div(tid, f.r1);
  i = tid - s * f.r1;
  {
    cx<T>* seq = buf + s * f.P;
    reg_second_in_lds_any<T, CLS, false>(f, seq + i * f.Q, s < np, [&](int q, cx<T> v) { seq[i + q * f.r1] = v; });
  }
  __syncthreads();
  const FastDiv div_lz(Lz);
  for (int q = tid; q < nr * Lz; q += blockDim.x) {
    const int r = div_lz(q), l = q - r * Lz;
    const cx<T>* seq = buf + (r >> 1) * f.P;
    const cx<T> z = seq[l], zm = seq[l == 0 ? 0 : Nz - l];
    D[(r0 + r) * pitch + l] = (r & 1) ? cx<T>{T(0.5) * (z.y + zm.y), T(-0.5) * (z.x - zm.x)}
                                      : cx<T>{T(0.5) * (z.x + zm.x), T(0.5) * (z.y - zm.y)};
  }
}

// Two-pass register transform of pairs of rows along z to real: two real rows
// share one complex transform, Z = X0 + i X1 (each Hermitian-extended)
// transforms to x0 + i x1. The DC bin keeps its real part only, as the real
// part of a single row's transform would; the Nyquist bin is zero. The rows go
// to LDS once and the first pass works there: loading its inputs from memory
// takes every value twice, for z and -z.
template <typename T, int CLS>
__device__ __forceinline__ void c2r_reg_body(const cx<T>* __restrict__ F, long long nrows, int pitch, const Fft2<T>& f,
                                             T* __restrict__ out, int bx, int tid) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* buf = reinterpret_cast<cx<T>*>(smem_raw);
  const int Nz = f.r1 * f.r2, Lz = Nz / 2;
  const long long r0 = (long long)bx * (2 << f.ls);  // the group's first row
  const int nr = (int)min((long long)(2 << f.ls), nrows - r0);
  const int np = (nr + 1) / 2;
  {
    const cx<T>* row = F + r0 * pitch;
    const FastDiv div_lz(Lz);
    struct Two {
      cx<T> a, c;
    };
    // Lz values per pair over the r1 or r2 threads a pair has: at most half the smaller radix each
    staged_copy<CLS == 16 ? 8 : 10>(
        np * Lz, tid, blockDim.x,
        [&](int q) {
          const int s = div_lz(q);
          const unsigned at = unsigned(2 * s * pitch + (q - s * Lz));
          return Two{cx_at(row, at), cx_at(row, at + (2 * s + 1 < nr ? unsigned(pitch) : 0u))};
        },
        [&](int q, Two v) {
          const int s = div_lz(q), l = q - s * Lz;
          if (2 * s + 1 >= nr) v.c = cx<T>{T(0), T(0)};
          cx<T>* seq = buf + s * f.P;
          if (l == 0) {
            seq[0] = cx<T>{v.a.x, v.c.x};
            seq[Lz] = cx<T>{T(0), T(0)};
          } else {
            seq[l] = cx<T>{v.a.x - v.c.y, v.a.y + v.c.x};
            seq[Nz - l] = cx<T>{v.a.x + v.c.y, v.c.x - v.a.y};
          }
        });
  }
  __syncthreads();
  int s = small_div(tid, f.r2), i = tid - s * f.r2;
  reg_first_in_lds_any<T, CLS, true>(f, buf + s * f.P, i, s < np);
  __syncthreads();
  s = small_div(tid, f.r1);
  i = tid - s * f.r1;
  if (s < np) {
    T* o = out + (r0 + 2 * s) * Nz + i;
    const bool two = 2 * s + 1 < nr;
    reg_second_any<T, CLS, true>(f, buf + s * f.P, i, [&](int q, cx<T> v) {
      o[q * f.r1] = v.x;
      if (two) o[q * f.r1 + Nz] = v.y;
    });
  }
}

template <typename T, int CLS>
__global__ __launch_bounds__(kFftThreads, (reg_waves<T, CLS>())) void k_c2r_reg(const cx<T>* __restrict__ F,
                                                                               long long nrows, int pitch, Fft2Raw f,
                                                                               T* __restrict__ out) {
  c2r_reg_body<T, CLS>(F, nrows, pitch, as_fft2<T>(f), out, blockIdx.x, threadIdx.x);
}

template <typename T, int NCT>
__device__ __forceinline__ void cfft_x_body(cx<T>* __restrict__ F, int Ny, int Lh, int lchunk,
                                            FftDesc<T> fd, int wm, int bx, int by) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* buf = reinterpret_cast<cx<T>*>(smem_raw);
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int Nx = NCT > 0 ? NCT : fd.n;
  const int bstride = lseq(Nx);
  const int kk = by;
  const int l0 = bx * lchunk;
  const int nl = min(lchunk, Lh - l0);
  cx<T>* base = F + size_t(kk) * Lh + l0;  // x mode jj, z mode l0 + li at base[jj * Ny * Lh + li]
  const size_t col = size_t(Ny) * Lh;
  cx<T>* twl = buf + lchunk * bstride;  // the twiddles go to LDS behind the rows
  if constexpr (NCT > 0) {
    // compile-time geometry (lchunk = ROWS z modes, 256 threads): no index divisions
    constexpr int ROWS = ct_maxb(NCT, kInvCap), BS = lseq(NCT), U = NCT * ROWS / kFftThreads;
    cx<T>* b0 = base + size_t(tid / ROWS) * col + tid % ROWS;
    const size_t step = size_t(kFftThreads / ROWS) * col;
    staged_cols<ROWS, kFftThreads, U>(
        NCT, nl, tid, [&](int, int, int u) { return b0[u * step]; },
        [&](int jj, int li, int, cx<T> v) { buf[li * BS + lpos(jj)] = v; });
    for (int t = tid; t < NCT; t += kFftThreads) twl[t] = fd.tw[t];
    __syncthreads();
    fft_ct<T, NCT, kFftThreads, ROWS, false>(buf, nl, twl, tid);
    __syncthreads();
    staged_cols<ROWS, kFftThreads, U>(
        NCT, nl, tid, [&](int jj, int li, int) { return buf[li * BS + lpos(jj)]; },
        [&](int, int, int u, cx<T> v) { b0[u * step] = v; });
  } else {
    const FastDiv div_nl(nl);
    staged_copy<kFftMaxV>(
        nl * Nx, tid, nthr,
        [&](int q) {
          const int jj = div_nl(q);
          return base[jj * col + (q - jj * nl)];
        },
        [&](int q, cx<T> v) {
          const int jj = div_nl(q);
          buf[(q - jj * nl) * bstride + lpos(jj)] = v;
        });
    for (int t = tid; t < fd.n; t += nthr) twl[t] = fd.tw[t];
    __syncthreads();
    fft_group<T, false>(buf, lds_twiddles(fd, twl), nl, bstride, tid, nthr, wm);
    __syncthreads();
    staged_copy<kFftMaxV>(
        nl * Nx, tid, nthr,
        [&](int q) {
          const int jj = div_nl(q);
          return buf[(q - jj * nl) * bstride + lpos(jj)];
        },
        [&](int q, cx<T> v) {
          const int jj = div_nl(q);
          base[jj * col + (q - jj * nl)] = v;
        });
  }
}

template <typename T, int NCT>
__global__ __launch_bounds__(kFftThreads) void k_cfft_x(cx<T>* __restrict__ F, int Ny, int Lh, int lchunk,
                                                      FftDesc<T> fd, int wm) {
  // neighbouring groups share the 128-byte lines of the z runs: keep them on one XCD
  const int gl = xcd_linear();
  cfft_x_body<T, NCT>(F, Ny, Lh, lchunk, fd, wm, gl % gridDim.x, gl / gridDim.x);
}

template <typename T, bool INV, int NCT = 0>
__device__ __forceinline__ void cfft_y_body(cx<T>* __restrict__ F, int Lh, int pitch, int lchunk, FftDesc<T> fd, int wm,
                                            int bx, int by, int tid = threadIdx.x) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* buf = reinterpret_cast<cx<T>*>(smem_raw);
  const int nthr = blockDim.x;
  const int Ny = NCT > 0 ? NCT : fd.n;
  const int bstride = lseq(Ny);
  const int jj = by;
  const int l0 = bx * lchunk;
  const int nl = min(lchunk, Lh - l0);
  cx<T>* base = F + size_t(jj) * Ny * pitch + l0;
  cx<T>* twl = buf + lchunk * bstride;  // the twiddles go to LDS behind the rows
  if constexpr (NCT > 0) {
    // compile-time geometry (lchunk = ROWS z modes, 256 threads): no index divisions
    constexpr int ROWS = ct_maxb(NCT, kInvCap), BS = lseq(NCT), U = NCT * ROWS / kFftThreads;
    cx<T>* b0 = base + size_t(tid / ROWS) * pitch + tid % ROWS;
    const size_t step = size_t(kFftThreads / ROWS) * pitch;
    staged_cols<ROWS, kFftThreads, U>(
        NCT, nl, tid, [&](int, int, int u) { return b0[u * step]; },
        [&](int kk, int li, int, cx<T> v) { buf[li * BS + lpos(kk)] = v; });
    for (int t = tid; t < NCT; t += kFftThreads) twl[t] = fd.tw[t];
    __syncthreads();
    fft_ct<T, NCT, kFftThreads, ROWS, INV>(buf, nl, twl, tid);
    __syncthreads();
    staged_cols<ROWS, kFftThreads, U>(
        NCT, nl, tid, [&](int kk, int li, int) { return buf[li * BS + lpos(kk)]; },
        [&](int, int, int u, cx<T> v) { b0[u * step] = v; });
  } else {
    const FastDiv div_nl(nl);
    staged_copy<kFftMaxV>(
        nl * Ny, tid, nthr,
        [&](int q) {
          const int kk = div_nl(q);
          return base[size_t(kk) * pitch + (q - kk * nl)];
        },
        [&](int q, cx<T> v) {
          const int kk = div_nl(q);
          buf[(q - kk * nl) * bstride + lpos(kk)] = v;
        });
    for (int t = tid; t < fd.n; t += nthr) twl[t] = fd.tw[t];
    __syncthreads();
    fft_group<T, INV>(buf, lds_twiddles(fd, twl), nl, bstride, tid, nthr, wm);
    __syncthreads();
    staged_copy<kFftMaxV>(
        nl * Ny, tid, nthr,
        [&](int q) {
          const int kk = div_nl(q);
          return buf[(q - kk * nl) * bstride + lpos(kk)];
        },
        [&](int q, cx<T> v) {
          const int kk = div_nl(q);
          base[size_t(kk) * pitch + (q - kk * nl)] = v;
        });
  }
}

template <typename T, bool INV, int NCT>
__global__ __launch_bounds__(kFftThreads) void k_cfft_y(cx<T>* __restrict__ F, int Lh, int pitch, int lchunk,
                                                      FftDesc<T> fd, int wm) {
  // neighbouring groups share the 128-byte lines of the z runs: keep them on one XCD
  const int gl = xcd_linear();
  cfft_y_body<T, INV, NCT>(F, Lh, pitch, lchunk, fd, wm, gl % gridDim.x, gl / gridDim.x);
}

// Longer lengths: passes in LDS, runtime plan. Two real rows share one complex
// transform as above.
template <typename T>
__device__ __forceinline__ void c2r_z_body(const cx<T>* __restrict__ F, long long nrows, int pitch, int rows,
                                           FftDesc<T> fd, T* __restrict__ f, int wm, int bx, int tid = threadIdx.x) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* buf = reinterpret_cast<cx<T>*>(smem_raw);
  const int nthr = blockDim.x;
  const int Nz = fd.n;
  const int Lz = Nz / 2;
  const int bstride = lseq(Nz);
  const long long r0 = (long long)bx * rows;
  const int nr = (int)min((long long)rows, nrows - r0);
  const int np = (nr + 1) / 2;
  const FastDiv div_lz(Lz), div_nz(Nz);
  struct Two {
    cx<T> a, c;
  };
  // kC2rStage pairs staged per thread (launches check np * (Nz/2 + 1) <= kC2rStage * threads)
  staged_copy<kC2rStage>(
      np * Lz, tid, nthr,
      [&](int q) {
        const int s = div_lz(q);
        const long long at = (r0 + 2 * s) * pitch + (q - s * Lz);
        return Two{F[at], 2 * s + 1 < nr ? F[at + pitch] : cx<T>{T(0), T(0)}};
      },
      [&](int q, Two v) {
        const int s = div_lz(q);
        const int l = q - s * Lz;
        cx<T>* row = buf + s * bstride;
        if (l == 0) {
          row[lpos(0)] = cx<T>{v.a.x, v.c.x};
          row[lpos(Lz)] = cx<T>{T(0), T(0)};
        } else {
          row[lpos(l)] = cx<T>{v.a.x - v.c.y, v.a.y + v.c.x};
          row[lpos(Nz - l)] = cx<T>{v.a.x + v.c.y, v.c.x - v.a.y};
        }
      });
  // the sequences hold (rows + 1) / 2 pairs: the twiddles go behind them
  cx<T>* twl = buf + (rows + 1) / 2 * bstride;
  for (int t = tid; t < fd.n; t += nthr) twl[t] = fd.tw[t];
  __syncthreads();
  fft_group<T, true>(buf, lds_twiddles(fd, twl), np, bstride, tid, nthr, wm);
  __syncthreads();
  staged_copy<kFftMaxV>(
      nr * Nz, tid, nthr,
      [&](int q) {
        const int r = div_nz(q);
        const cx<T> v = buf[(r >> 1) * bstride + lpos(q - r * Nz)];
        return (r & 1) ? v.y : v.x;
      },
      [&](int q, T v) { f[r0 * Nz + q] = v; });
}

template <typename T>
__global__ __launch_bounds__(kFftThreads) void k_c2r_z(const cx<T>* __restrict__ F, long long nrows, int pitch,
                                                     int rows, FftDesc<T> fd, T* __restrict__ f, int wm) {
  c2r_z_body<T>(F, nrows, pitch, rows, fd, f, wm, blockIdx.x);
}

// Transpose of the complex-to-real pass for the forward model: real rows f[r][e] ->
// Dh[r][l] = sum_e f[r][e] exp(-2 pi i l e/Nz), l = 0..Nz/2. Two real rows
// share one complex transform, Z = FFT(x0 + i x1): X0[l] = (Z[l] + conj
// Z[-l])/2 and X1[l] = (Z[l] - conj Z[-l])/(2i), so a work-group of `rows`
// rows transforms (rows + 1) / 2 sequences (half the transforms, LDS and
// registers of one sequence per row). PLANE: packed rows with the plane
// l = Nz/2, stored in one run (the row and mode of every value cost the
// position derivatives up to 3 % of this pass); else rows of `pitch` without it.
template <typename T, int NCT, bool PLANE>
__global__ __launch_bounds__(kFftThreads) void k_r2c_z(const T* __restrict__ f, long long nrows, int rows,
                                                     FftDesc<T> fd, cx<T>* __restrict__ D, int pitch) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* buf = reinterpret_cast<cx<T>*>(smem_raw);
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int Nz = NCT > 0 ? NCT : fd.n;
  const int Lh = Nz / 2 + 1;
  const int bstride = lseq(Nz);
  const long long r0 = (long long)blockIdx.x * rows;
  const int nr = (int)min((long long)rows, nrows - r0);
  const int np = (nr + 1) / 2;
  const FastDiv fdiv_lh(Lh), fdiv_nz(Nz);
  // compile-time lengths divide by constants (a shift for Nz)
  auto div_lh = [&](int q) { return NCT > 0 ? int(unsigned(q) / unsigned(NCT / 2 + 1)) : fdiv_lh(q); };
  auto div_nz = [&](int q) { return NCT > 0 ? int(unsigned(q) / unsigned(NCT > 0 ? NCT : 1)) : fdiv_nz(q); };
  struct Two {
    T a, b;
  };
  // values staged per thread: what a compile-time length needs, else
  // kFftMaxV (np * Nz <= rows * Nz / 2 + Nz / 2 <= 3 * 1024 by fft_batch)
  constexpr int ROWS = NCT > 0 ? ct_maxb(NCT, kInvCap) : 1;
  constexpr int UL = NCT > 0 ? ((ROWS + 1) / 2 * NCT + kFftThreads - 1) / kFftThreads : kFftMaxV;
  constexpr int UO = NCT > 0 ? (ROWS * (NCT / 2 + 1) + kFftThreads - 1) / kFftThreads : kFftMaxV;
  staged_copy<UL>(
      np * Nz, tid, nthr,
      [&](int q) {
        const int s = div_nz(q);
        const long long at = (r0 + 2 * s) * Nz + (q - s * Nz);
        return Two{f[at], 2 * s + 1 < nr ? f[at + Nz] : T(0)};
      },
      [&](int q, Two v) {
        const int s = div_nz(q);
        buf[s * bstride + lpos(q - s * Nz)] = cx<T>{v.a, v.b};
      });
  cx<T>* twl = buf + (rows + 1) / 2 * bstride;
  for (int t = tid; t < (NCT > 0 ? NCT : fd.n); t += nthr) twl[t] = fd.tw[t];
  __syncthreads();
  if constexpr (NCT > 0)
    fft_ct<T, NCT, kFftThreads, (ROWS + 1) / 2, false>(buf, np, twl, tid);
  else
    fft_lds<T, kFftMaxV, false, false>(buf, lds_twiddles(fd, twl), np, bstride, tid, nthr);
  __syncthreads();
  staged_copy<UO>(
      nr * Lh, tid, nthr,
      [&](int q) {
        const int r = div_lh(q);
        const int l = q - r * Lh;
        const cx<T>* row = buf + (r >> 1) * bstride;
        const cx<T> z = row[lpos(l)];
        const cx<T> zm = row[lpos(l == 0 ? 0 : Nz - l)];
        return (r & 1) ? cx<T>{T(0.5) * (z.y + zm.y), T(-0.5) * (z.x - zm.x)}
                       : cx<T>{T(0.5) * (z.x + zm.x), T(0.5) * (z.y - zm.y)};
      },
      [&](int q, cx<T> v) {
        if constexpr (PLANE) {
          D[r0 * Lh + q] = v;
        } else {
          const int r = div_lh(q);
          const int l = q - r * Lh;
          if (l < Nz / 2) D[(r0 + r) * pitch + l] = v;
        }
      });
}

// Forward model: in-place transforms of the half spectrum along y, then x.
template <typename T>
static hipError_t launch_forward_xy(const DevPlan& p, cx<T>* F, hipStream_t s) {
  const int Lh = p.Nz / 2 + 1;
  const FftCfg cfg = inv_cfg();
  const int ly = fft_batch<T>(p.Ny, cfg.threads, cfg.cap);
  const size_t lds_y = (size_t(ly) * lseq(p.Ny) + p.Ny) * sizeof(cx<T>);
  hipError_t e = ct_pick(CtInverse{}, p.Ny, [&](auto c) {
    constexpr int NCT = decltype(c)::value;
    // the compile-time kernels take their geometry from the length
    if (NCT > 0 && (ly != ct_maxb(NCT, kInvCap) || cfg.threads != kFftThreads)) return hipErrorInvalidValue;
    hipError_t e2 = allow_lds(reinterpret_cast<const void*>(&k_cfft_y<T, false, NCT>), lds_y);
    if (e2 != hipSuccess) return e2;
    hipLaunchKernelGGL((k_cfft_y<T, false, NCT>), dim3((Lh + ly - 1) / ly, p.Nx), dim3(cfg.threads), lds_y, s, F, Lh,
                       Lh, ly, as_desc<T>(p.f_Ny), cfg.wave);
    return hipGetLastError();
  });
  if (e != hipSuccess) return e;
  const int lx = fft_batch<T>(p.Nx, cfg.threads, cfg.cap);
  const size_t lds_x = (size_t(lx) * lseq(p.Nx) + p.Nx) * sizeof(cx<T>);
  return ct_pick(CtInverse{}, p.Nx, [&](auto c) {
    constexpr int NCT = decltype(c)::value;
    if (NCT > 0 && (lx != ct_maxb(NCT, kInvCap) || cfg.threads != kFftThreads)) return hipErrorInvalidValue;
    hipError_t e2 = allow_lds(reinterpret_cast<const void*>(&k_cfft_x<T, NCT>), lds_x);
    if (e2 != hipSuccess) return e2;
    hipLaunchKernelGGL((k_cfft_x<T, NCT>), dim3((Lh + lx - 1) / lx, p.Ny), dim3(cfg.threads), lds_x, s, F,
                       p.Ny, Lh, lx, as_desc<T>(p.f_Nx), cfg.wave);
    return hipGetLastError();
  });
}

template <typename T>
hipError_t launch_inverse(const DevPlan& p, void* Fh, T* f, hipStream_t s) {
  cx<T>* F = static_cast<cx<T>*>(Fh);
  const int Lz = p.Nz / 2;
  const FftCfg cfg = inv_cfg();
  hipError_t e;
  const int ly = fft_seqs<T>(p.f_Ny, p.f_Ny.two.r1 ? kInvYThreads : cfg.threads, cfg.cap);
  const dim3 gy((Lz + ly - 1) / ly, p.Nx);
  if (p.f_Ny.two.r1) {
    const Fft2Raw t = fft2_shape<T>(p.f_Ny, ly);
    const size_t lds = fft2_slots(t) * sizeof(cx<T>);
    e = class_pick(t, [&](auto c) {
      constexpr auto kern = &k_cfft_y_reg<T, decltype(c)::value>;
      hipError_t e2 = allow_lds(reinterpret_cast<const void*>(kern), lds);
      if (e2 != hipSuccess) return e2;
      hipLaunchKernelGGL(kern, gy, dim3(fft2_threads(t)), lds, s, F, Lz, p.pitch_f, t);
      return hipGetLastError();
    });
  } else {
    const size_t lds = (size_t(ly) * lseq(p.Ny) + p.Ny) * sizeof(cx<T>);
    e = allow_lds(reinterpret_cast<const void*>(&k_cfft_y<T, true, 0>), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_cfft_y<T, true, 0>), gy, dim3(cfg.threads), lds, s, F, Lz, p.pitch_f, ly,
                       as_desc<T>(p.f_Ny), cfg.wave);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return e;
  const long long nrows = (long long)p.Nx * p.Ny;
  if (p.f_Nz.two.r1) {
    const Fft2Raw t = fft2_shape<T>(p.f_Nz, fft_seqs<T>(p.f_Nz, cfg.threads, kC2rSeqs));
    const size_t lds = fft2_slots(t) * sizeof(cx<T>);
    const long long rows = 2LL << t.ls;
    return class_pick(t, [&](auto c) {
      constexpr auto kern = &k_c2r_reg<T, decltype(c)::value>;
      hipError_t e2 = allow_lds(reinterpret_cast<const void*>(kern), lds);
      if (e2 != hipSuccess) return e2;
      hipLaunchKernelGGL(kern, dim3((unsigned)((nrows + rows - 1) / rows)), dim3(fft2_threads(t)), lds, s, F, nrows,
                         p.pitch_f, t, f);
      return hipGetLastError();
    });
  }
  const int rows = fft_batch<T>(p.Nz, cfg.threads, cfg.cap);
  const size_t lds = size_t(c2r_lds_slots(rows, p.Nz)) * sizeof(cx<T>);
  if ((rows + 1) / 2 * (p.Nz / 2 + 1) > kC2rStage * cfg.threads) return hipErrorInvalidValue;
  e = allow_lds(reinterpret_cast<const void*>(&k_c2r_z<T>), lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_c2r_z<T>, dim3((unsigned)((nrows + rows - 1) / rows)), dim3(cfg.threads), lds, s, F, nrows,
                     p.pitch_f, rows, as_desc<T>(p.f_Nz), f, cfg.wave);
  return hipGetLastError();
}

// Real-to-complex z pass with its passes in LDS: packed rows with the plane
// l = Nz/2 at every length, or rows of pitch_f without it at the lengths of
// CtForwardZ (others return hipErrorInvalidValue).
template <typename T, bool PLANE>
static hipError_t launch_r2c_z(const DevPlan& p, const T* f, cx<T>* D, hipStream_t s) {
  const FftCfg cfg = inv_cfg();
  const int rows = fft_batch<T>(p.Nz, cfg.threads, cfg.cap);
  const size_t lds = size_t(c2r_lds_slots(rows, p.Nz)) * sizeof(cx<T>);  // (rows + 1) / 2 sequences
  const long long nrows = (long long)p.Nx * p.Ny;
  if ((rows + 1) / 2 * p.Nz > kFftMaxV * cfg.threads || rows * (p.Nz / 2 + 1) > kFftMaxV * cfg.threads)
    return hipErrorInvalidValue;
  return ct_pick(std::conditional_t<PLANE, CtInverse, CtForwardZ>{}, p.Nz, [&](auto c) {
    constexpr int NCT = decltype(c)::value;
    if constexpr (PLANE || NCT > 0) {
      constexpr auto kern = &k_r2c_z<T, NCT, PLANE>;
      hipError_t e2 = allow_lds(reinterpret_cast<const void*>(kern), lds);
      if (e2 != hipSuccess) return e2;
      hipLaunchKernelGGL(kern, dim3((unsigned)((nrows + rows - 1) / rows)), dim3(cfg.threads), lds, s, f, nrows, rows,
                         as_desc<T>(p.f_Nz), D, PLANE ? p.Nz / 2 + 1 : p.pitch_f);
      return hipGetLastError();
    } else {
      return hipErrorInvalidValue;
    }
  });
}

template <typename T>
hipError_t launch_forward3d(const DevPlan& p, const T* f, void* Dh, hipStream_t s) {
  cx<T>* D = static_cast<cx<T>*>(Dh);
  hipError_t e = launch_r2c_z<T, true>(p, f, D, s);
  if (e != hipSuccess) return e;
  return launch_forward_xy<T>(p, D, s);
}


// The forward transforms as register passes: Dh[jj][kk][l], l < Nz/2, rows of
// pitch_f; every axis of a length with two passes.
template <typename T>
hipError_t launch_forward3d_reg(const DevPlan& p, const T* f, void* Dh, hipStream_t s) {
  if (!p.f_Nx.two.r1 || !p.f_Ny.two.r1 || !p.f_Nz.two.r1) return hipErrorInvalidValue;
  cx<T>* D = static_cast<cx<T>*>(Dh);
  const int Lz = p.Nz / 2;
  const long long nrows = (long long)p.Nx * p.Ny;
  const Fft2Raw z = fft2_shape<T>(p.f_Nz, fft_seqs<T>(p.f_Nz, kFftThreads, kC2rSeqs));
  const size_t lds_z = fft2_slots(z) * sizeof(cx<T>);
  // the lengths of CtForwardZ stay with the compile-time form in the z pass
  bool fixed = false;
  (void)ct_pick(CtForwardZ{}, p.Nz, [&](auto c) {
    fixed = decltype(c)::value > 0;
    return hipSuccess;
  });
  hipError_t e = fixed ? launch_r2c_z<T, false>(p, f, D, s) : class_pick(z, [&](auto c) {
    constexpr auto kern = &k_r2c_reg<T, decltype(c)::value>;
    hipError_t e2 = allow_lds(reinterpret_cast<const void*>(kern), lds_z);
    if (e2 != hipSuccess) return e2;
    const long long rows = 2LL << z.ls;
    hipLaunchKernelGGL(kern, dim3((unsigned)((nrows + rows - 1) / rows)), dim3(fft2_threads(z)), lds_z, s, f, nrows,
                       p.pitch_f, z, D);
    return hipGetLastError();
  });
  if (e != hipSuccess) return e;
  auto pass = [&](const FftRaw& raw, unsigned stride, unsigned other, int count) {
    const Fft2Raw t = fft2_shape<T>(raw, fft_seqs<T>(raw, kInvYThreads, kInvCap));
    const size_t lds = fft2_slots(t) * sizeof(cx<T>);
    return class_pick(t, [&](auto c) {
      constexpr auto kern = &k_cfft_fwd_reg<T, decltype(c)::value>;
      hipError_t e2 = allow_lds(reinterpret_cast<const void*>(kern), lds);
      if (e2 != hipSuccess) return e2;
      hipLaunchKernelGGL(kern, dim3((Lz + (1 << t.ls) - 1) >> t.ls, count), dim3(fft2_threads(t)), lds, s, D, Lz,
                         stride,
                         other, t);
      return hipGetLastError();
    });
  };
  const unsigned row = unsigned(p.pitch_f), slab = unsigned(p.Ny) * row;
  e = pass(p.f_Ny, row, slab, p.Nx);
  if (e != hipSuccess) return e;
  return pass(p.f_Nx, slab, row, p.Ny);
}

// Batched forms of the inverse passes (one variant of problems per launch, as
// the lateral passes).
template <typename T, int CLS>
__global__ __launch_bounds__(kInvYThreads, (any_waves<T, CLS>())) void k_cfft_y_inv_batch(
    const CfftBA* __restrict__ args, const int* __restrict__ prefix, int total, BatchIO io) {
  for (int slot = blockIdx.x; slot < total; slot += gridDim.x) {
    if (slot != int(blockIdx.x)) __syncthreads();  // the previous item's LDS is done with
    const int w = batch_item(slot, total);
    const int p = batch_locate(prefix, w);
    const CfftBA a = args[p];
    const int local = w - prefix[p];
    const int by = local / a.gx;
    if constexpr (CLS > 0)
      cfft_y_reg_body<T, CLS>(static_cast<cx<T>*>(a.F), a.Lz, a.pitch, as_fft2<T>(a.f2), local - by * a.gx, by,
                              loop_lane());
    else
      cfft_y_body<T, true>(static_cast<cx<T>*>(a.F), a.Lz, a.pitch, a.lchunk, view_desc<T>(a.fd), 0,
                           local - by * a.gx, by, loop_lane());
  }
}

template <typename T, int CLS>
__global__ __launch_bounds__(kFftThreads, (any_waves<T, CLS>())) void k_c2r_z_batch(const C2rBA* __restrict__ args,
                                                                                   const int* __restrict__ prefix,
                                                                                   int total, BatchIO io) {
  for (int slot = blockIdx.x; slot < total; slot += gridDim.x) {
    if (slot != int(blockIdx.x)) __syncthreads();  // the previous item's LDS is done with
    const int w = batch_item(slot, total);
    const int p = batch_locate(prefix, w);
    const C2rBA a = args[p];
    T* out = static_cast<T*>(io.out[a.problem]);
    if constexpr (CLS > 0)
      c2r_reg_body<T, CLS>(static_cast<const cx<T>*>(a.F), a.nrows, a.pitch, as_fft2<T>(a.f2), out, w - prefix[p],
                           loop_lane());
    else
      c2r_z_body<T>(static_cast<const cx<T>*>(a.F), a.nrows, a.pitch, a.rows, view_desc<T>(a.fd), out, 0,
                    w - prefix[p]);
  }
}

template <typename T>
hipError_t launch_cfft_y_inv_batch(const BatchStage& st, const BatchIO& io, hipStream_t s) {
  if (st.total <= 0) return hipSuccess;
  switch (st.variant) {
    case 16: return launch_batch_kernel<CfftBA>(&k_cfft_y_inv_batch<T, 16>, st, io, s);
    case 20: return launch_batch_kernel<CfftBA>(&k_cfft_y_inv_batch<T, 20>, st, io, s);
    case 32: return launch_batch_kernel<CfftBA>(&k_cfft_y_inv_batch<T, 32>, st, io, s);
    default: return launch_batch_kernel<CfftBA>(&k_cfft_y_inv_batch<T, 0>, st, io, s);
  }
}

template <typename T>
hipError_t launch_c2r_z_batch(const BatchStage& st, const BatchIO& io, hipStream_t s) {
  if (st.total <= 0) return hipSuccess;
  switch (st.variant) {
    case 16: return launch_batch_kernel<C2rBA>(&k_c2r_z_batch<T, 16>, st, io, s);
    case 20: return launch_batch_kernel<C2rBA>(&k_c2r_z_batch<T, 20>, st, io, s);
    case 32: return launch_batch_kernel<C2rBA>(&k_c2r_z_batch<T, 32>, st, io, s);
    default: return launch_batch_kernel<C2rBA>(&k_c2r_z_batch<T, 0>, st, io, s);
  }
}

#define PATK_INST(T)                                                                \
  template hipError_t launch_inverse<T>(const DevPlan&, void*, T*, hipStream_t); \
  template hipError_t launch_forward3d<T>(const DevPlan&, const T*, void*, hipStream_t); \
  template hipError_t launch_forward3d_reg<T>(const DevPlan&, const T*, void*, hipStream_t); \
  template hipError_t launch_cfft_y_inv_batch<T>(const BatchStage&, const BatchIO&, hipStream_t); \
  template hipError_t launch_c2r_z_batch<T>(const BatchStage&, const BatchIO&, hipStream_t);
PATK_INST(float)
PATK_INST(double)
#undef PATK_INST

}  // namespace patk
