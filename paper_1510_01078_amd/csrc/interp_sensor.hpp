// Footprint sums and launch shape shared by the two forms of the forward
// model's fused x transform and interpolation to the sensors.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>

#include "kernels_common.hpp"

namespace patk {

constexpr int kFusedThreads = 512;  // per home-tile row of the strip
constexpr int kFusedBins = 8;       // most bins per work-group
// sensors per thread whose bins are held in registers: as many as fit the
// register budget (FP32 footprints up to 8 or 12 points; none of these forms
// spills)
template <typename T, int W>
__host__ __device__ constexpr int fused_held() {
  return sizeof(T) == 4 ? (W <= 8 ? 2 : (W <= 12 ? 1 : 0)) : 0;
}

template <int W, int FS>
__host__ __device__ constexpr int fused_rows() { return FS * kSpreadTile + W - 1; }

// the register transform leaves room for fewer: none beside radix 20 on 1024
// threads (128 registers, 2 of them spilled), as many on the 768 of the larger
// radices (168: the second costs 9 to 11 spilled registers up to 8-point
// footprints on two rows of home tiles, and without it the kernel takes 478 us
// instead of 405 for 16384 sensors on a 384^2 grid)
template <typename T, int W, int CLS>
__host__ __device__ constexpr int reg_held() {
  return sizeof(T) != 4 || W > 12 || CLS == 20 ? 0 : CLS == 32 && W <= 8 ? 2 : 1;
}

// One sensor of the strip: footprint origin row within the strip, the LDS
// slots of its footprint columns, and its weights.
template <typename T, int W>
struct FusedSensor {
  int m, oy;
  int col[W];
  T wx[W], wy[W];
};

template <typename T, int W, bool PADDED = true>
__device__ __forceinline__ void fused_sensor_load(FusedSensor<T, W>& f, int m, int py0, int n_x,
                                                  const int* __restrict__ sbx, const int* __restrict__ sby,
                                                  const T* __restrict__ swx, const T* __restrict__ swy) {
  f.m = m;
  const int ox = sbx[m];
  f.oy = sby[m] - py0;
#pragma unroll
  for (int t = 0; t < W; ++t) {
    f.wx[t] = swx[size_t(m) * W + t];
    f.wy[t] = swy[size_t(m) * W + t];
    int c = ox + t;
    if (c >= n_x) c -= n_x;
    f.col[t] = PADDED ? lpos(c) : c;
  }
}

// footprint sum in k_interp's order: rows of x-weighted sums, then y weights
template <typename T, int W>
__device__ __forceinline__ cx<T> fused_sensor_sum(const FusedSensor<T, W>& f, const cx<T>* buf, int bstride) {
  const cx<T>* rows = buf + f.oy * bstride;
  cx<T> acc{T(0), T(0)};
#pragma unroll
  for (int ty = 0; ty < W; ++ty) {
    cx<T> row{T(0), T(0)};
#pragma unroll
    for (int tx = 0; tx < W; ++tx) {
      const cx<T> v = rows[ty * bstride + f.col[tx]];
      row.x += f.wx[tx] * v.x;
      row.y += f.wx[tx] * v.y;
    }
    acc.x += f.wy[ty] * row.x;
    acc.y += f.wy[ty] * row.y;
  }
  return acc;
}

// Bins per work-group of a fused kernel: enough groups to fill the device
// several times over; where even 4 bins per group fill every resident slot at
// least twice, the count in 4..kFusedBins whose last wave of work-groups is
// fullest (the groups take about equal time, and a part-filled last wave idles
// the rest of the device: 0.98 -> 0.965 ms per forward call with 576 bins on a
// 384^2 grid, 7 bins instead of 6).
// `memo`, one per kernel, holds the last answer of the occupancy query: device,
// LDS bytes and resident groups in one word.
static inline int fused_bins(const void* kern, int threads, size_t lds, long long strips, int nb, int tiles_y,
                             std::atomic<unsigned long long>& memo) {
  int bins = int(std::min<long long>(kFusedBins, std::max<long long>(1, (long long)tiles_y * nb / 2048)));
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return bins;
  const unsigned long long key = (unsigned long long)(dev & 0xffff) << 48 | (unsigned long long)(lds & 0xffffff) << 24;
  unsigned long long word = memo.load(std::memory_order_relaxed);
  if ((word >> 24) != (key >> 24) || !(word & 0xffffff)) {
    int per_cu = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, threads, lds) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
      (void)hipGetLastError();
      return bins;
    }
    word = key | (unsigned long long)std::max(1, per_cu * cus);
    memo.store(word, std::memory_order_relaxed);
  }
  const long long slots = (long long)(word & 0xffffff);
  if (strips * ((nb + 3) / 4) >= 2 * slots) {
    double best = -1.0;
    for (int bb = 4; bb <= kFusedBins; ++bb) {
      const double waves = double(strips * ((nb + bb - 1) / bb)) / double(slots);
      const double fill = waves / std::ceil(waves);
      if (fill >= best - 1e-9) {
        best = fill;
        bins = bb;
      }
    }
  }
  return bins;
}

}  // namespace patk
