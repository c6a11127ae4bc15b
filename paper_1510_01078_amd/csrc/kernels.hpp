// Interface between the host plan code and the gfx950 stage kernels of the
// NEDNER-NUFFT reconstruction (Section 3: a non-equispaced-range NUFFT in
// time, a non-equispaced-data NUFFT over the sensor plane, then an
// equispaced inverse FFT).
//
// Order of the steps on the device. The temporal transform's equispaced part
// (deapodise, zero-pad, FFT) runs first, per sensor; the lateral NUFFT then
// runs once per kept temporal bin; the temporal interpolation at
// omega(K) = c|K| runs last, per lateral mode. This is the paper's
// composition with the two linear maps on different indices applied in the
// other order, which lets the lateral grid be built only for the band of
// temporal bins that the interpolation reads.
#pragma once
#include <hip/hip_runtime.h>
#include <cstddef>
#include <cstdint>

#include "plan_sizes.hpp"

namespace patk {

struct FftPassRaw {
  int R = 0, p = 0, nbf = 0, twstep = 0;
  uint32_t m_nbf = 0, m_p = 0;
};

// Two-pass register transform (fft_reg.hpp) of a length n = r1*r2; r1 = 0:
// the length has none. P, Q and ls (LDS strides, log2 of the sequences per
// work-group) depend on the kernel and are set where it is launched.
struct Fft2Raw {
  int r1, r2;
  int P, Q, ls;
  int pad;
  const void* tw;  // device, tw[k*r2 + i] = exp(-2 pi i ik/n), k < r1, i < r2
};

// Three-pass form (fft_reg.hpp) for the temporal FFT: n = r1*r2*r3, r3 = 1 for
// lengths with two passes, r1 = 0 for none. P, QA, QB and ls are set at launch.
struct Fft3Raw {
  int r1, r2, r3;
  int P, QA, QB, ls;
  int pad;
  const void* twA;  // device, [r1][r2*r3]
  const void* twB;  // device, [r2][r3] (r3 > 1)
};

struct FftRaw {
  int n = 0;
  int npass = 0;
  Fft2Raw two{0, 0, 0, 0, 0, 0, nullptr};
  FftPassRaw pass[12];           // host copy
  const void* dpass = nullptr;   // device copy of pass[0..npass)
  const void* tw = nullptr;      // device, n complex entries exp(-2 pi i t/n)
};

// Everything a launch needs, as plain values and device pointers.
struct DevPlan {
  int M = 0, Nt = 0, Nx = 0, Ny = 0, Nz = 0;
  int n_x = 0, n_y = 0, n_t = 0, n0 = 0, b_lo = 0, nb = 0;
  int w_xy = 0, w_t = 0, hdeg = 0;
  int tiles_x = 0, tiles_y = 0;
  int chunk_bins = 0;          // bins per spread / x-FFT round (the grid buffer holds this many)
  bool kahan = false;
  // row pitches (elements) of the reconstruction's intermediate arrays: grid
  // rows U, x-transformed rows V, lateral spectra Gh, band values Gt
  int pitch_u = 0, pitch_v = 0, pitch_g = 0, pitch_t = 0;
  int pitch_f = 0;             // z modes' rows of the x-transformed spectrum F
  double s_per_k = 0.0;        // c*dt*n_t/(2 pi): oversampled bin per unit |K|
  double kxu = 0, kyu = 0, kzu = 0;  // 2 pi/X, 2 pi/Y, 2 pi/Z
  double two_c = 0.0;          // 2c of W(K) = 2c|Kz|/|K|
  double n0_over_nt = 0.0;     // centring phase factor n0/n_t
  double inv_vol = 0.0;        // 1/(XYZ)
  double adj_scale = 0.0;      // dV/(2V) = 1/(2 Nx Ny Nz): the adjoint's constant weight with the 1/V of the inverse
  // device tables (element type T unless int)
  const void* hw = nullptr;       // [M]   h_m*dt
  const void* deap = nullptr;     // [Nt]  1/phihat_t((n - n0)/n_t)
  const int* sbx = nullptr;       // [M]   first x grid point of the footprint (mod n_x)
  const int* sby = nullptr;       // [M]
  const void* swx = nullptr;      // [M][w] x weights
  const void* swy = nullptr;      // [M][w]
  const int4* slot_rng = nullptr; // [tiles_x*patches_y] first and past-the-end packed slot of each 16 x kPatchRows
                                  // patch and the patch's index, patches of several rounds of slots first
  int spread_heavy = 0;           // patches (the first of slot_rng) that take one bin group per work item: those of
                                  // more than one round (kSlotBatch slots) where patsz::spread_split, else none
  const int* slot_sens = nullptr; // [slots][kSlotK] sensor ids of each slot, -1 for an empty place
  const void* slot_w = nullptr;   // [slots][64] each lane's weight wx*wy (0 where no sensor covers it)
  const unsigned* slot_k = nullptr;       // [slots][64] places in their slots of the lane's sensors for the
                                          // kSlotBatch slots from this one on (2 bits each, 0 past the patch)
  int patches_y = 0;
  const int* home_off = nullptr;  // [tiles+1] sensors whose footprint starts in each tile (CSR)
  const int* home_sens = nullptr; // [M]
  int fused_strip = 1;            // home-tile rows per strip of the fused forward kernel (1 or 2)
  const int* jrange = nullptr;    // [Nx][2] first and last band bin the interpolation reads per x-mode,
                                  // in whole groups of the y-FFT's bins; the y-FFT skips the others
  const int* brange = nullptr;    // [nb][2] per band bin the smallest and largest |j| whose range holds it
  const int* ylist = nullptr;     // the y-FFT's work items inside the ranges: jj << 16 | bin group
  int ylist_n = 0;
  const int* ytlist = nullptr;    // the same ranges for the transposed y pass with its passes in LDS, which takes
  int ytlist_n = 0;               // fft_batch bins per item: jj << 16 | first bin
  const void* dcx = nullptr;      // [Nx] 1/phihat(j/n_x), 0 at j = -Nx/2
  const void* dcy = nullptr;      // [Ny]
  const void* hcoef = nullptr;    // [w_t][hdeg+1] temporal tap polynomials
  FftRaw f_nt, f_nx, f_ny, f_Nx, f_Ny, f_Nz;
  Fft3Raw f_nt3{0, 0, 0, 0, 0, 0, 0, 0, nullptr, nullptr};  // temporal FFT
};

constexpr int kSpreadTile = 16;  // spread tile edge (grid points)
constexpr int kPatchRows = 4;    // rows of the spread's one-wave patch (16 x 4 grid points)
constexpr int kSlotK = 4;        // sensors per packed spread slot
constexpr int kSpreadGroups = 2; // most spread bin groups (16 bins each) per work-group
constexpr int kSlotBatch = 8;    // spread slots staged per round (their places fit one 32-bit word)

// Work items of the spread over `nchunks` bin groups: the first spread_heavy
// patches take one bin group per item (they read their lane tables again for
// every bin group anyway), the others `groups`.
inline long long spread_items(const DevPlan& p, int nchunks, int groups) {
  return (long long)p.spread_heavy * nchunks +
         ((long long)p.tiles_x * p.patches_y - p.spread_heavy) * ((nchunks + groups - 1) / groups);
}
// Two bin groups per item (one read of the lane tables for both) once that
// leaves enough one-wave items to fill the device; smaller problems spread the
// bin groups over more waves.
inline int spread_groups(const DevPlan& p, int nchunks) {
  return spread_items(p, nchunks, kSpreadGroups) >= patsz::kSpreadWaves ? kSpreadGroups : 1;
}

// Stage launchers; T = float or double. Buffers are device pointers.
//
// Reconstruction and adjoint: temporal -> spread -> fft_x -> fft_y -> gather
// -> inverse. Forward model (the exact transpose of the adjoint's stages, in
// reverse order): forward3d -> scatter -> fft_y_t -> fft_x_t -> interp ->
// temporal_t.

// Launch shape of the temporal FFT's register form (r1 = 0: passes in LDS).
template <typename T>
Fft3Raw temporal_shape(const DevPlan& p);
// weighted = true: traces scaled by h_m dt (reconstruction); false: unit
// weights (adjoint of the forward model).
template <typename T>
hipError_t launch_temporal(const DevPlan& p, const T* g, void* Gt, bool weighted, hipStream_t s);
// Bins [b_begin, b_end) of the band: U holds only those bins (U[b - b_begin]),
// V all bins.
template <typename T>
hipError_t launch_spread(const DevPlan& p, const void* Gt, void* U, int b_begin, int b_end, hipStream_t s);
template <typename T>
hipError_t launch_fft_x(const DevPlan& p, const void* U, void* V, int b_begin, int b_end, hipStream_t s);
template <typename T>
hipError_t launch_fft_y(const DevPlan& p, const void* V, void* Gh, hipStream_t s);
// GATHER_PHYSICAL: F(K) as defined (sign (-1)^(j+k), no 1/V); GATHER_IMAGE:
// the image-ready spectrum (-1)^(j+k) F(K) / (XYZ) consumed by
// launch_inverse; GATHER_ADJOINT: the adjoint's image-ready spectrum.
enum { GATHER_IMAGE = 0, GATHER_PHYSICAL = 1, GATHER_ADJOINT = 2 };
template <typename T>
hipError_t launch_gather(const DevPlan& p, const void* Gh, void* Fh, int mode, hipStream_t s);
template <typename T>
hipError_t launch_inverse(const DevPlan& p, void* F, T* f, hipStream_t s);
// Gather (GATHER_IMAGE or GATHER_ADJOINT) fused with the inverse transform
// along x into F[jj][kk][l], l < Nz/2 (rows of pitch_f); launch_inverse
// finishes along y and z.
template <typename T>
hipError_t launch_gather_x(const DevPlan& p, const void* Gh, void* F, int mode, hipStream_t s);

template <typename T>
void gather_shape(const DevPlan& p, int& lchunk, Fft2Raw& f2, size_t& slots);

// Forward model. f -> Dh (real-to-complex along z, forward FFTs along y, x)
template <typename T>
hipError_t launch_forward3d(const DevPlan& p, const T* f, void* Dh, hipStream_t s);
template <typename T>
hipError_t launch_forward3d_reg(const DevPlan& p, const T* f, void* Dh, hipStream_t s);
// Dh (rows of `pitch` z modes) -> Gh' (deriv 0: A; 1: d/dx_m; 2: d/dy_m); LDS bytes it needs
template <typename T>
hipError_t launch_scatter(const DevPlan& p, const void* Dh, int pitch, void* Gh, int deriv, hipStream_t s);
template <typename T>
size_t scatter_lds_bytes(const DevPlan& p);
// Gh'[j][k][b] -> V'[b][j][py]
template <typename T>
hipError_t launch_fft_y_t(const DevPlan& p, const void* Gh, void* V, hipStream_t s);
// V'[b][j][py] -> U'[b - b_begin][py][px] for bins [b_begin, b_end)
template <typename T>
hipError_t launch_fft_x_t(const DevPlan& p, const void* V, void* U, int b_begin, int b_end, hipStream_t s);
// U' (bins [b_begin, b_end)) -> Gt'[m][b] at the sensors
template <typename T>
hipError_t launch_interp(const DevPlan& p, const void* U, void* Gt, int b_begin, int b_end, hipStream_t s);
// k_fft_x_t and k_interp in one kernel over all bins (no grid buffer); usable
// when fused_interp_ok: n_x <= 1024 and the strip of 16 + w - 1 rows fits the
// work-group LDS limit.
template <typename T>
hipError_t launch_fft_x_interp(const DevPlan& p, const void* V, void* Gt, hipStream_t s);
// The two as register transforms (rows of pitch_v between them): lengths with
// two passes, and for the second fused_reg_ok.
template <typename T>
hipError_t launch_fft_y_t_reg(const DevPlan& p, const void* Gh, void* V, hipStream_t s);
template <typename T>
hipError_t launch_fft_x_interp_reg(const DevPlan& p, const void* V, void* Gt, hipStream_t s);
template <typename T>
bool fused_reg_ok(const DevPlan& p, size_t lds_limit);
// Static LDS that the fused kernel and the transposed interpolation hold
// beside their dynamic LDS (row and run tables); the plan's fit checks add it.
constexpr size_t kStaticLdsMargin = 512;

// LDS of the fused kernel for a strip of strip_tiles rows of home tiles
template <typename T>
size_t fused_interp_lds(const DevPlan& p, int strip_tiles);
template <typename T>
bool fused_interp_ok(const DevPlan& p, size_t lds_limit);
// Gt' -> g[m][n] (unit weights)
template <typename T>
hipError_t launch_temporal_t(const DevPlan& p, const void* Gt, T* g, hipStream_t s);

// ---------------------------------------------------------------------------
// Batched launches: one launch per stage and kernel variant (class of FFT
// lengths) serves up to kGroupMax problems of different sizes. The work items
// of a launch are the blocks of its problems, numbered problem after problem;
// prefix[p] is the first item of problem p (the total behind the last problem,
// then INT_MAX). Each problem's arguments sit in a device table; only the per-call input and output pointers travel in BatchIO (a
// kernel argument), so a batched call allocates and synchronises nothing.
// ---------------------------------------------------------------------------
constexpr int kBatchMax = 64;
constexpr int kGroupMax = 32;  // problems per batched launch

struct BatchIO {
  const void* in[kGroupMax];
  void* out[kGroupMax];
};

struct FftView {  // plain data, in the batch's argument tables
  int n, npass;
  const void* pass;
  const void* tw;
};

struct TemporalBA {
  const void* hw; const void* deap; FftView fd; Fft3Raw f3; int M, Nt, n0, b_lo, nb, pitch_t; void* Gt;
  int problem, pad;  // index into BatchIO
};
struct SpreadBA {
  const void* Gt; const int4* slot_rng; const int* slot_sens; const void* slot_w; const unsigned* slot_k;
  int nb, n_x, n_y, tiles_x, nchunks, heavy, groups, pitch_t, pitch_u, pad; void* U;
};
struct FftXBA {
  const void* U; FftView fd; Fft2Raw f2; int n_y, Nx, rows, gx, pitch_u, pitch_v; void* V; const int* brange;
};
struct FftYBA {
  const void* V; FftView fd; Fft2Raw f2; int nb, Nx, Ny, bins, gx, pitch_v, pitch_g; void* Gh;
  const int* jrange;  // per x-mode band range (bin groups outside it are skipped)
  const int* ylist;   // the work items inside the ranges (jj << 16 | bin group), or nullptr: gx * Nx items
};
struct GatherBA {  // the gather fused with the inverse transform along x
  const void* Gh; const void* hcoef; const void* dcx; const void* dcy; int nb, b_lo, Nx, Ny, Nz, wt, deg;
  int wt_ct, pitch_g;  // compile-time tap count to run (kBatchTaps member equal to wt, else 0: runtime taps)
  double s_per_k, kxu, kyu, kzu, two_c, n0_over_nt, scale; void* Fh;
  FftView fd; Fft2Raw f2; int lchunk, gx, pitch_f, pad;  // x transform (length Nx), z modes per group, groups along z
};
struct CfftBA {
  void* F; FftView fd; Fft2Raw f2; int Lz, pitch, lchunk, gx;
};
struct C2rBA {
  const void* F; FftView fd; Fft2Raw f2; long long nrows; int rows, pitch;
  int problem, pad;  // index into BatchIO
};

// One stage of a batched call: its argument table (one entry per problem),
// prefix sums of work items, the dynamic LDS bytes (maximum over problems)
// and the grid (0: one block per work item; otherwise blocks that loop over
// the work items).
struct BatchStage {
  const void* args = nullptr;
  const int* prefix = nullptr;
  int total = 0;
  size_t lds = 0;
  int grid = 0;
  bool kahan = false;  // spread with compensated summation
  int variant = 0;     // FFT stages: class of the problems' register transforms (0: passes in LDS), in the
                       // temporal stage + 64 * its form
  int threads = 256;   // FFT stages: work-group size
};

// tap counts the batched gather instantiates at compile time (each problem
// runs its own; other counts take the runtime-tap form)
constexpr int kBatchTaps[4] = {6, 8, 10, 12};

// temporal tap polynomials staged in LDS: at most 16 taps of degree <= 24
constexpr int kMaxTapCoefs = 16 * 25;

template <typename T> hipError_t launch_temporal_batch(const BatchStage& st, const BatchIO& io, hipStream_t s);
template <typename T> hipError_t launch_spread_batch(const BatchStage& st, const BatchIO& io, hipStream_t s);
template <typename T> hipError_t launch_fft_x_batch(const BatchStage& st, const BatchIO& io, hipStream_t s);
template <typename T> hipError_t launch_fft_y_batch(const BatchStage& st, const BatchIO& io, hipStream_t s);
template <typename T> hipError_t launch_gather_batch(const BatchStage& st, const BatchIO& io, hipStream_t s);
template <typename T> hipError_t launch_cfft_y_inv_batch(const BatchStage& st, const BatchIO& io, hipStream_t s);
template <typename T> hipError_t launch_c2r_z_batch(const BatchStage& st, const BatchIO& io, hipStream_t s);

}  // namespace patk
