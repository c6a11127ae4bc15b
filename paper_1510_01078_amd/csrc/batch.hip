// Batched reconstruction: up to kBatchMax independent problems (each its own
// sensor geometry, trace length and output grid) reconstructed with one
// launch per stage, kernel variant and group of problems. A stage's work items
// are the blocks of the variant's problems (problem after problem);
// per-problem arguments are uploaded once at creation, so a call only enqueues
// seven stages per group: one kernel for the spread, one per variant for the
// others (at most nine in the temporal stage, four in each later one).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cstdint>
#include <cstring>
#include <new>
#include <type_traits>
#include <utility>
#include <vector>

#include "kernels_common.hpp"
#include "pat_nufft.h"
#include "plan_internal.hpp"

using namespace patint;

namespace {
constexpr int kStages = 7;  // temporal, spread, fft x, fft y, gather + inverse x, inverse y, c2r z
// default grid: one work-group per work item (0), which finds its problem and
// arguments by scalar loads. A batch of 16 problems took 4.19 ms so, 4.22,
// 4.30, 4.50 and 4.73 ms on persistent grids of 65536, 16384, 4096 and 2048
// work-groups, which wait for an item's stores before they start the next.
constexpr int kDefaultGrid = 0;
}

// Problems are run in groups of at most kGroupMax, optionally also bounded by
// a byte budget on their oversampled grids (so that a group's stages could
// hand their intermediate arrays on through the last-level cache). Groups run
// one after another and share one workspace.
struct BatchGroup {
  std::vector<int> members;   // problem indices, ascending grid size
  void* tables = nullptr;     // argument tables and prefix sums
  size_t table_bytes = 0;
  // launches of each stage: one, or for the FFT stages one per class of
  // two-pass transform among the problems' lengths (fft_reg.hpp)
  std::vector<patk::BatchStage> st[kStages];
};

struct pat_batch {
  int count = 0;
  int device = 0;
  bool fp64 = false;
  pat_plan* plans[patk::kBatchMax] = {};
  pat_plan_desc alloc_desc{};  // allocator used for the batch's own memory
  std::vector<BatchGroup> groups;
  void* ws = nullptr;          // workspace of the largest group
  size_t ws_bytes = 0;
  size_t group_bytes = 0;
};

namespace {

struct Blob {
  std::vector<unsigned char> bytes;
  size_t add(const void* src, size_t n) {
    const size_t off = align_up(bytes.size());
    bytes.resize(off + n);
    if (n) std::memcpy(bytes.data() + off, src, n);
    return off;
  }
};

void destroy_batch(pat_batch* B) {
  if (!B) return;
  {
    DeviceGuard guard(B->device);
    (void)hipDeviceSynchronize();
    dev_free(B->alloc_desc, B->ws);
    for (auto& g : B->groups) dev_free(B->alloc_desc, g.tables);
  }
  for (int i = 0; i < B->count; ++i) nufft_plan_destroy(B->plans[i]);
  delete B;
}

// Workspace bytes of one problem: A = grid U (all bins) / lateral spectra,
// B = x rows / spectrum, C = band values (each 256-byte aligned).
template <typename T>
void problem_regions(const patk::DevPlan& d, size_t& a, size_t& b, size_t& cc) {
  const size_t c = sizeof(patk::cx<T>);
  const size_t lh = size_t(d.pitch_f);
  a = align_up(std::max(size_t(d.nb) * d.n_y * d.pitch_u * c, size_t(d.Nx) * d.Ny * d.pitch_g * c));
  b = align_up(std::max(size_t(d.nb) * d.Nx * d.pitch_v * c, size_t(d.Nx) * d.Ny * lh * c));
  cc = align_up(size_t(d.M) * d.pitch_t * c);
}

// Stage tables of one group, with workspace pointers into `ws`.
template <typename T>
pat_status build_group(pat_batch* B, BatchGroup& G, unsigned char* ws, hipStream_t stream) {
  using patk::cx;
  const int P = int(G.members.size());
  const size_t c = sizeof(cx<T>);
  const patk::FftCfg cfg = patk::fft_cfg();
  const patk::FftCfg icfg = patk::inv_cfg();
  std::vector<patk::TemporalBA> a0(P);
  std::vector<patk::SpreadBA> a1(P);
  std::vector<patk::FftXBA> a2(P);
  std::vector<patk::FftYBA> a3(P);
  std::vector<patk::GatherBA> a4(P);
  std::vector<patk::CfftBA> a5(P);
  std::vector<patk::C2rBA> a6(P);
  // per stage and problem: work items, LDS bytes, work-group size and variant
  std::vector<int> pre[kStages], threads[kStages], variant[kStages];
  std::vector<size_t> lds[kStages];
  for (int i = 0; i < kStages; ++i) {
    pre[i].assign(P, 0);
    threads[i].assign(P, 256);
    variant[i].assign(P, 0);
    lds[i].assign(P, 0);
  }
  const int kFft = patk::kFftMaxV * cfg.threads;
  size_t off = 0;
  for (int p = 0; p < P; ++p) {
    const patk::DevPlan& d = B->plans[G.members[p]]->dp;
    size_t ra, rb, rc;
    problem_regions<T>(d, ra, rb, rc);
    void* A = ws + off;
    void* Bw = ws + off + ra;
    void* C = ws + off + ra + rb;
    off += ra + rb + rc;
    const int Lz = d.Nz / 2;
    if (d.n_t > patk::kFftMaxV * 512) return PAT_ERR_UNSUPPORTED;
    // stage 0: temporal FFT, a block per sensor pair or a few
    const patk::Fft3Raw f0 = patk::temporal_shape<T>(d);
    a0[p] = patk::TemporalBA{d.hw, d.deap, patk::as_view(d.f_nt), f0, d.M, d.Nt, d.n0, d.b_lo, d.nb, d.pitch_t, C, p,
                             0};
    pre[0][p] = ((d.M + 1) / 2 + (1 << f0.ls) - 1) >> f0.ls;
    lds[0][p] = (f0.r1 ? size_t(f0.P) << f0.ls : size_t(patk::temporal_lds_slots(d.n_t))) * c;
    variant[0][p] = f0.r1 ? patk::three_class(f0) + 64 * (f0.r3 == 1 ? 1 : patk::fft3_rounds(f0) ? 2 : 0) : 0;
    threads[0][p] = f0.r1 ? patk::fft3_threads(f0) : 512;
    // stage 1: spread, all bins in one round
    const int nchunks = (d.nb + 15) / 16;
    a1[p] = patk::SpreadBA{C,     d.slot_rng, d.slot_sens, d.slot_w,       d.slot_k,          d.nb, d.n_x,
                           d.n_y, d.tiles_x,  nchunks,     d.spread_heavy, patk::kSpreadGroups, d.pitch_t, d.pitch_u, 0, A};
    const long long items1 = patk::spread_items(d, nchunks, patk::kSpreadGroups);
    if (items1 > 0x7fffffffLL) return PAT_ERR_UNSUPPORTED;
    pre[1][p] = int(items1);
    // stage 2: FFT along x
    const int rows = patk::fft_seqs<T>(d.f_nx, cfg.threads, cfg.cap);
    const patk::Fft2Raw fx = d.f_nx.two.r1 ? patk::fft2_shape<T>(d.f_nx, rows) : d.f_nx.two;
    if (!fx.r1 && (rows * d.n_x > kFft || rows * d.Nx > kFft)) return PAT_ERR_UNSUPPORTED;
    const int gx2 = (d.n_y + rows - 1) / rows;
    a2[p] = patk::FftXBA{A, patk::as_view(d.f_nx), fx, d.n_y, d.Nx, rows, gx2, d.pitch_u, d.pitch_v, Bw,
                         d.jrange ? d.brange : nullptr};
    pre[2][p] = gx2 * d.nb;
    lds[2][p] = (fx.r1 ? patk::fft2_slots(fx) : size_t(rows) * patk::lseq(d.n_x) + d.n_x) * c;
    variant[2][p] = fx.r1 ? patk::reg_class(fx) : 0;
    threads[2][p] = fx.r1 ? patk::fft2_threads(fx) : cfg.threads;
    // stage 3: FFT along y
    const int bins = patk::fft_bins<T>(d.f_ny, cfg.threads, cfg.cap);
    const patk::Fft2Raw fy = d.f_ny.two.r1 ? patk::fft2_shape<T>(d.f_ny, bins) : d.f_ny.two;
    if (!fy.r1 && (bins * d.n_y > kFft || bins * d.Ny > kFft)) return PAT_ERR_UNSUPPORTED;
    const int gx3 = (d.nb + bins - 1) / bins;
    const bool listed = d.ylist && d.ylist_n > 0 && d.jrange;
    a3[p] = patk::FftYBA{Bw, patk::as_view(d.f_ny), fy, d.nb, d.Nx, d.Ny, bins, gx3, d.pitch_v, d.pitch_g, A, d.jrange,
                         listed ? d.ylist : nullptr};
    pre[3][p] = listed ? d.ylist_n : gx3 * d.Nx;
    lds[3][p] = (fy.r1 ? patk::fft2_slots(fy) : size_t(bins) * patk::lseq(d.n_y) + d.n_y) * c;
    variant[3][p] = fy.r1 ? patk::reg_class(fy) : 0;
    threads[3][p] = fy.r1 ? patk::fft2_threads(fy) : cfg.threads;
    // stage 4: temporal interpolation and weight (image-ready spectrum) fused
    // with the inverse transform along x
    int lcx;
    patk::Fft2Raw f4;
    size_t slots4;
    patk::gather_shape<T>(d, lcx, f4, slots4);
    const int gx5 = (Lz + lcx - 1) / lcx;
    int wt_ct = 0;
    for (int t : patk::kBatchTaps)
      if (d.w_t == t && d.w_t * (d.hdeg + 1) <= patk::kMaxTapCoefs) wt_ct = t;
    a4[p] = patk::GatherBA{A, d.hcoef, d.dcx, d.dcy, d.nb, d.b_lo, d.Nx, d.Ny, d.Nz, d.w_t, d.hdeg, wt_ct, d.pitch_g,
                           d.s_per_k, d.kxu, d.kyu, d.kzu, d.two_c, d.n0_over_nt, d.inv_vol, Bw,
                           patk::as_view(d.f_Nx), f4, lcx, gx5, d.pitch_f, 0};
    pre[4][p] = gx5 * d.Ny;
    lds[4][p] = slots4 * c;
    variant[4][p] = f4.r1 ? patk::reg_class(f4) : 0;
    threads[4][p] = icfg.threads;
    // stage 5: inverse transform along y (in place on the spectrum)
    const int lcy = patk::fft_seqs<T>(d.f_Ny, d.f_Ny.two.r1 ? patk::kInvYThreads : icfg.threads, icfg.cap);
    const patk::Fft2Raw f5 = d.f_Ny.two.r1 ? patk::fft2_shape<T>(d.f_Ny, lcy) : d.f_Ny.two;
    const int gx6 = (Lz + lcy - 1) / lcy;
    a5[p] = patk::CfftBA{Bw, patk::as_view(d.f_Ny), f5, Lz, d.pitch_f, lcy, gx6};
    pre[5][p] = gx6 * d.Nx;
    lds[5][p] = (f5.r1 ? patk::fft2_slots(f5) : size_t(lcy) * patk::lseq(d.Ny) + d.Ny) * c;
    variant[5][p] = f5.r1 ? patk::reg_class(f5) : 0;
    threads[5][p] = f5.r1 ? patk::fft2_threads(f5) : icfg.threads;
    // stage 6: complex-to-real along z into the caller's image
    const long long nrows = (long long)d.Nx * d.Ny;
    int rz = patk::fft_batch<T>(d.Nz, icfg.threads, icfg.cap);
    patk::Fft2Raw f6 = d.f_Nz.two;
    if (f6.r1) {
      f6 = patk::fft2_shape<T>(d.f_Nz, patk::fft_seqs<T>(d.f_Nz, icfg.threads, patk::kC2rSeqs));
      rz = 2 << f6.ls;
    } else if ((rz + 1) / 2 * (d.Nz / 2 + 1) > patk::kC2rStage * icfg.threads) {
      return PAT_ERR_UNSUPPORTED;
    }
    a6[p] = patk::C2rBA{Bw, patk::as_view(d.f_Nz), f6, nrows, rz, d.pitch_f, p, 0};
    pre[6][p] = int((nrows + rz - 1) / rz);
    lds[6][p] = (f6.r1 ? patk::fft2_slots(f6) : size_t(patk::c2r_lds_slots(rz, d.Nz))) * c;
    variant[6][p] = f6.r1 ? patk::reg_class(f6) : 0;
    threads[6][p] = f6.r1 ? patk::fft2_threads(f6) : icfg.threads;
  }
  // each stage's launches: the problems of one variant, their arguments and
  // the running sums of their work items
  Blob blob;
  const bool kahan = B->plans[0]->dp.kahan;
  std::vector<std::pair<size_t, size_t>> at[kStages];
  auto add_stage = [&](int i, const auto& args) {
    std::vector<int> kinds(variant[i]);
    std::sort(kinds.begin(), kinds.end());
    kinds.erase(std::unique(kinds.begin(), kinds.end()), kinds.end());
    for (int kind : kinds) {
      std::vector<typename std::decay_t<decltype(args)>::value_type> part;
      std::vector<int> prefix(1, 0);
      patk::BatchStage st;
      for (int p = 0; p < P; ++p) {
        if (variant[i][p] != kind) continue;
        const long long next = (long long)prefix.back() + pre[i][p];
        if (next > 0x7fffffffLL) return false;
        part.push_back(args[p]);
        prefix.push_back(int(next));
        st.lds = std::max(st.lds, lds[i][p]);
        st.threads = std::max(part.size() == 1 ? 0 : st.threads, threads[i][p]);
      }
      st.total = prefix.back();
      st.grid = kDefaultGrid;
      st.kahan = kahan;
      st.variant = kind;
      const size_t oa = blob.add(part.data(), part.size() * sizeof(part[0]));
      prefix.resize(patk::kGroupMax + 1, INT_MAX);
      at[i].emplace_back(oa, blob.add(prefix.data(), prefix.size() * sizeof(int)));
      G.st[i].push_back(st);
    }
    return true;
  };
  if (!add_stage(0, a0) || !add_stage(1, a1) || !add_stage(2, a2) || !add_stage(3, a3) || !add_stage(4, a4) ||
      !add_stage(5, a5) || !add_stage(6, a6))
    return PAT_ERR_UNSUPPORTED;
  G.table_bytes = align_up(blob.bytes.size());
  G.tables = dev_alloc(B->alloc_desc, G.table_bytes);
  if (!G.tables) return PAT_ERR_ALLOC;
  if (hipMemcpyAsync(G.tables, blob.bytes.data(), blob.bytes.size(), hipMemcpyHostToDevice, stream) != hipSuccess ||
      hipStreamSynchronize(stream) != hipSuccess) {
    (void)hipGetLastError();
    return PAT_ERR_HIP;
  }
  unsigned char* tb = static_cast<unsigned char*>(G.tables);
  for (int i = 0; i < kStages; ++i)
    for (size_t v = 0; v < G.st[i].size(); ++v) {
      G.st[i][v].args = tb + at[i][v].first;
      G.st[i][v].prefix = reinterpret_cast<const int*>(tb + at[i][v].second);
    }
  return PAT_OK;
}

template <typename T>
pat_status build_batch(pat_batch* B, hipStream_t stream) {
  const int P = B->count;
  // group by the oversampled grid's size (the array handed from the spread to the x-FFT)
  std::vector<size_t> grid(P), total(P);
  for (int p = 0; p < P; ++p) {
    size_t a, b, c;
    problem_regions<T>(B->plans[p]->dp, a, b, c);
    const patk::DevPlan& d = B->plans[p]->dp;
    grid[p] = size_t(d.nb) * d.n_y * d.n_x * sizeof(patk::cx<T>);
    total[p] = a + b + c;
  }
  std::vector<int> order(P);
  for (int p = 0; p < P; ++p) order[p] = p;
  std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return grid[x] < grid[y]; });
  B->groups.clear();
  size_t sum = 0;
  for (int p : order) {
    if (B->groups.empty() || int(B->groups.back().members.size()) == patk::kGroupMax ||
        (sum + grid[p] > B->group_bytes && !B->groups.back().members.empty())) {
      B->groups.emplace_back();
      sum = 0;
    }
    B->groups.back().members.push_back(p);
    sum += grid[p];
  }
  size_t ws = 0;
  for (auto& g : B->groups) {
    size_t t = 0;
    for (int p : g.members) t += total[p];
    ws = std::max(ws, t);
  }
  B->ws_bytes = ws;
  B->ws = dev_alloc(B->alloc_desc, ws);
  if (!B->ws) return PAT_ERR_ALLOC;
  for (auto& g : B->groups) {
    const pat_status st = build_group<T>(B, g, static_cast<unsigned char*>(B->ws), stream);
    if (st != PAT_OK) return st;
  }
  return PAT_OK;
}

template <typename T>
pat_status run_batch(pat_batch* B, const void* const* g, void* const* f, hipStream_t s) {
  for (const BatchGroup& G : B->groups) {
    patk::BatchIO io{};
    for (size_t i = 0; i < G.members.size(); ++i) {
      io.in[i] = g[G.members[i]];
      io.out[i] = f[G.members[i]];
    }
    using Launch = hipError_t (*)(const patk::BatchStage&, const patk::BatchIO&, hipStream_t);
    const Launch launch[kStages] = {patk::launch_temporal_batch<T>, patk::launch_spread_batch<T>,
                                    patk::launch_fft_x_batch<T>, patk::launch_fft_y_batch<T>,
                                    patk::launch_gather_batch<T>, patk::launch_cfft_y_inv_batch<T>,
                                    patk::launch_c2r_z_batch<T>};
    for (int i = 0; i < kStages; ++i)
      for (const patk::BatchStage& st : G.st[i]) {
        const hipError_t e = launch[i](st, io, s);
        if (e != hipSuccess) return to_status(e);
      }
  }
  return PAT_OK;
}

}  // namespace

extern "C" {

pat_status pat_batch_create(const pat_plan_desc* descs, int32_t count, size_t group_bytes, void* stream,
                            pat_batch** out) {
  if (!out) return PAT_ERR_INVALID_ARGUMENT;
  *out = nullptr;
  if (!descs || count < 1 || count > patk::kBatchMax) return PAT_ERR_INVALID_ARGUMENT;
  for (int i = 1; i < count; ++i) {
    const bool fp64_i = descs[i].precision == PAT_FP64, fp64_0 = descs[0].precision == PAT_FP64;
    if (fp64_i != fp64_0 || (descs[i].precision == PAT_FP32_KAHAN) != (descs[0].precision == PAT_FP32_KAHAN))
      return PAT_ERR_INVALID_ARGUMENT;
  }
  pat_batch* B = new (std::nothrow) pat_batch();
  if (!B) return PAT_ERR_ALLOC;
  if (hipGetDevice(&B->device) != hipSuccess) {
    (void)hipGetLastError();
    delete B;
    return PAT_ERR_HIP;
  }
  B->alloc_desc = descs[0];
  B->alloc_desc.sensor_xy = nullptr;
  B->alloc_desc.sensor_h = nullptr;
  B->fp64 = descs[0].precision == PAT_FP64;
  B->group_bytes = group_bytes ? group_bytes : SIZE_MAX;
  for (int i = 0; i < count; ++i) {
    pat_status st = nufft_plan(&descs[i], stream, &B->plans[i]);
    if (st != PAT_OK) {
      destroy_batch(B);
      return st;
    }
    B->count = i + 1;
  }
  const pat_status st = B->fp64 ? build_batch<double>(B, static_cast<hipStream_t>(stream))
                                : build_batch<float>(B, static_cast<hipStream_t>(stream));
  if (st != PAT_OK) {
    destroy_batch(B);
    return st;
  }
  *out = B;
  return PAT_OK;
}

pat_status pat_batch_get_plan(const pat_batch* B, int32_t index, const pat_plan** plan) {
  if (!B || !plan || index < 0 || index >= B->count) return PAT_ERR_INVALID_ARGUMENT;
  *plan = B->plans[index];
  return PAT_OK;
}

pat_status pat_batch_set_grid(pat_batch* B, int32_t blocks) {
  if (!B || blocks < 0) return PAT_ERR_INVALID_ARGUMENT;
  for (auto& g : B->groups)
    for (auto& stage : g.st)
      for (auto& s : stage) s.grid = blocks;
  return PAT_OK;
}

pat_status pat_batch_groups(const pat_batch* B, int32_t* groups) {
  if (!B || !groups) return PAT_ERR_INVALID_ARGUMENT;
  *groups = int32_t(B->groups.size());
  return PAT_OK;
}

pat_status pat_batch_reconstruct(pat_batch* B, const void* const* g, void* const* f, void* stream) {
  if (!B || !g || !f) return PAT_ERR_INVALID_ARGUMENT;
  for (int p = 0; p < B->count; ++p)
    if (!g[p] || !f[p]) return PAT_ERR_INVALID_ARGUMENT;
  DeviceGuard guard(B->device);
  if (!guard.ok) return PAT_ERR_HIP;
  hipStream_t s = static_cast<hipStream_t>(stream);
  return B->fp64 ? run_batch<double>(B, g, f, s) : run_batch<float>(B, g, f, s);
}

pat_status pat_batch_destroy(pat_batch* B) {
  destroy_batch(B);
  return PAT_OK;
}

}  // extern "C"
