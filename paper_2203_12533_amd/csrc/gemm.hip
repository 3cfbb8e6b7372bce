// GEMM engine: C[M,N] = op(A)[M,K] . op(B)[K,N], fp32 accumulation, fused epilogues; argument checks and the
// choice of kernel for every problem (launch_gemm, launch_gemm_pair).
//
// bf16 problems made of full 256 x 256 tiles that fill the chip go to the ring-buffered kernel of gemm_ring.hip: that is
// most GEMMs of the large workloads.  Everything else in bf16 - any shape, ragged edges, few tiles - goes to gemm_tile.hip.
// Both fetch their operands global -> LDS directly.
//
// Launch mapping: one workgroup per output tile, 1-D grid.  Hardware deals consecutive workgroup ids
// round-robin to the 8 XCDs (each with its own L2), so ids are first regrouped so that every XCD owns a
// contiguous range of tiles, and within the range tiles are walked in groups of 8 tile-rows so that
// concurrently resident workgroups share A and B panels through that XCD's L2.
//
// fp32 problems go to gemm_f32.hip.
#include "common.hpp"
#include <algorithm>
#include <cmath>

#include "gemm_common.hpp"
#include "kernels.hpp"

#include <cstdlib>
#include <map>
#include <tuple>
#include <vector>

namespace pw {

static bool g_use_ring = true;

hipError_t gemm_init() {
  const char* env = getenv("PW_GEMM_RING");      // PW_GEMM_RING=0 selects the any-shape kernel everywhere
  g_use_ring = !(env && env[0] == '0');
  hipError_t e = gemm_ring_init();
  if (e == hipSuccess) e = gemm_tile_init();
  return e;
}

// ======================================================================================================
// host side
// ======================================================================================================
namespace {
struct ProfiledLaunch {
  hipEvent_t start, stop;
  double flops;
  bool optimizer = false;   // the launch carried the Adam epilogue: MFMA work plus 26 bytes per output element
  GemmShapeKey key{};       // shape, layouts and epilogue (of the first member of a shared launch)
};
struct ShapeLess {
  bool operator()(const GemmShapeKey& x, const GemmShapeKey& y) const {
    return std::tie(x.M, x.N, x.K, x.a_kmajor, x.b_kmajor, x.epilogue, x.members) <
           std::tie(y.M, y.N, y.K, y.a_kmajor, y.b_kmajor, y.epilogue, y.members);
  }
};
std::vector<GemmShapeRow> g_shape_rows;   // per-shape totals as of the last gemm_profile_end
GemmShapeKey shape_key(const GemmArgs& a, int members) {
  return GemmShapeKey{a.M, a.N, a.K, a.a_kmajor, a.b_kmajor, a.epilogue, members};
}
int64_t g_fused_launches = 0;   // what the last gemm_profile_end saw of such launches
double g_fused_ms = 0.0, g_fused_flops = 0.0;
bool g_profile_on = false;
std::vector<ProfiledLaunch> g_profile;
std::vector<hipEvent_t> g_profile_free;

hipEvent_t profile_event() {
  if (!g_profile_free.empty()) {
    hipEvent_t e = g_profile_free.back();
    g_profile_free.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  (void)hipEventCreate(&e);
  return e;
}
}  // namespace

void gemm_profile_begin() {
  for (auto& p : g_profile) {
    g_profile_free.push_back(p.start);
    g_profile_free.push_back(p.stop);
  }
  g_profile.clear();
  g_profile_on = true;
}

void gemm_profile_pause() { g_profile_on = false; }

hipError_t gemm_profile_end(int64_t* launches, double* total_ms, double* total_flops) {
  g_profile_on = false;
  double ms = 0.0, fl = 0.0;
  int64_t n = 0;
  g_fused_launches = 0;
  g_fused_ms = g_fused_flops = 0.0;
  hipError_t err = hipSuccess;
  std::map<GemmShapeKey, GemmShapeRow, ShapeLess> by_shape;
  for (auto& p : g_profile) {
    hipError_t e = hipEventSynchronize(p.stop);
    float t = 0.f;
    if (e == hipSuccess) e = hipEventElapsedTime(&t, p.start, p.stop);
    if (e != hipSuccess) err = e;
    GemmShapeRow& row = by_shape[p.key];
    row.key = p.key;
    row.launches++;
    row.total_ms += t;
    row.total_flops += p.flops;
    if (p.optimizer) {
      g_fused_launches++;
      g_fused_ms += t;
      g_fused_flops += p.flops;
    } else {
      n++;
      ms += t;
      fl += p.flops;
    }
    g_profile_free.push_back(p.start);
    g_profile_free.push_back(p.stop);
  }
  if (launches) *launches = n;
  if (total_ms) *total_ms = ms;
  if (total_flops) *total_flops = fl;
  g_profile.clear();
  g_shape_rows.clear();
  for (auto& kv : by_shape) g_shape_rows.push_back(kv.second);
  std::stable_sort(g_shape_rows.begin(), g_shape_rows.end(),
                   [](const GemmShapeRow& x, const GemmShapeRow& y) { return x.total_ms > y.total_ms; });
  return err;
}

int gemm_profile_shapes(GemmShapeRow* rows, int cap) {
  const int n = (int)g_shape_rows.size();
  for (int i = 0; rows && i < n && i < cap; ++i) rows[i] = g_shape_rows[i];
  return n;
}

void gemm_profile_fused(int64_t* launches, double* total_ms, double* total_flops) {
  if (launches) *launches = g_fused_launches;
  if (total_ms) *total_ms = g_fused_ms;
  if (total_flops) *total_flops = g_fused_flops;
}

static hipError_t launch_gemm_impl(hipStream_t s, const GemmArgs& a);

hipError_t launch_gemm(hipStream_t s, const GemmArgs& a) {
  const bool timed = g_profile_on && a.dtype == kBF16 && a.M > 0 && a.N > 0;
  if (!timed) return launch_gemm_impl(s, a);
  ProfiledLaunch p{profile_event(), profile_event(), 2.0 * (double)a.M * (double)a.N * (double)a.K, a.epilogue == kEpiAdam,
                   shape_key(a, 1)};
  if (!p.start || !p.stop) return hipErrorOutOfMemory;
  hipError_t e = hipEventRecord(p.start, s);
  if (e == hipSuccess) e = launch_gemm_impl(s, a);
  if (e == hipSuccess) e = hipEventRecord(p.stop, s);
  if (e == hipSuccess) g_profile.push_back(p);
  return e;
}

// Argument checks shared by every path; *empty is set when there is nothing to compute.
static hipError_t check_gemm_args(const GemmArgs& a, bool* empty) {
  *empty = false;
  const bool no_c = a.epilogue == kEpiAdam || a.epilogue == kEpiXentStats;   // C optional / unused there
  if (!a.A || !a.B || (!a.C && !no_c) || a.M < 0 || a.N < 0 || a.K < 0) return hipErrorInvalidValue;
  if (a.epilogue < kEpiStore || a.epilogue > kEpiXentGrad) return hipErrorInvalidValue;
  if (a.epilogue == kEpiAdam) {
    const AdamEpi& d = a.adam;
    if (!d.w || !d.m || !d.v || (!d.c_dev && d.t < 1) || a.out_dtype != kF32 || a.accumulate) return hipErrorInvalidValue;
    if (((uintptr_t)d.w | (uintptr_t)d.m | (uintptr_t)d.v | (uintptr_t)d.w_bf16 | (uintptr_t)d.c_dev) & 15) return hipErrorInvalidValue;
  }
  if (a.epilogue == kEpiXentStats || a.epilogue == kEpiXentGrad) {
    const XentEpi& x = a.xent;
    if (!x.tokens || x.T < 1 || a.M % x.T || a.accumulate) return hipErrorInvalidValue;
    if (a.epilogue == kEpiXentStats && (!x.part || !x.zt || ((uintptr_t)x.part & 7))) return hipErrorInvalidValue;
    if (a.epilogue == kEpiXentGrad && (!x.lse || a.out_dtype != kBF16)) return hipErrorInvalidValue;
  }
  if (a.lda < (a.a_kmajor ? a.M : a.K) || a.ldb < (a.b_kmajor ? a.N : a.K) || a.ldc < a.N) return hipErrorInvalidValue;
  if ((a.epilogue == kEpiBiasResidual || a.epilogue == kEpiGeluBwd) && !a.aux) return hipErrorInvalidValue;
  if (a.epilogue == kEpiBiasGelu && !a.C2) return hipErrorInvalidValue;
  if (a.accumulate && (a.out_dtype != kF32 || a.epilogue != kEpiStore)) return hipErrorInvalidValue;
  if (a.epilogue == kEpiBiasResidual && a.out_dtype != kF32) return hipErrorInvalidValue;
  if (a.out_dtype == kBF16 && a.dtype != kBF16) return hipErrorInvalidValue;
  if (a.M == 0 || a.N == 0) { *empty = true; return hipSuccess; }
  if (a.M > (1LL << 30) || a.N > (1LL << 30) || a.K > (1LL << 30)) return hipErrorInvalidValue;
  if (a.dtype == kF32) {
    if (a.out_dtype != kF32) return hipErrorInvalidValue;
    // vector epilogue accesses need 16-byte alignment; the kernel falls back to scalars when ldc % 4 != 0
    if (((uintptr_t)a.C | (uintptr_t)a.C2 | (uintptr_t)a.aux | (uintptr_t)a.bias) & 15) return hipErrorInvalidValue;
    return hipSuccess;
  }
  if (a.dtype != kBF16) return hipErrorInvalidValue;
  // 16-byte vector loads: every row start and every k offset of a piece must be 16-byte aligned
  if ((a.K % 8) || (a.lda % 8) || (a.ldb % 8)) return hipErrorInvalidValue;
  if ((a.a_kmajor && a.M % 8) || (a.b_kmajor && a.N % 8)) return hipErrorInvalidValue;
  if (((uintptr_t)a.A | (uintptr_t)a.B) & 15) return hipErrorInvalidValue;
  if (((uintptr_t)a.C | (uintptr_t)a.C2 | (uintptr_t)a.aux | (uintptr_t)a.bias) & 15) return hipErrorInvalidValue;
  if (a.ldc % 8) return hipErrorInvalidValue;
  return hipSuccess;
}

static EpiParams epi_of(const GemmArgs& a) {
  EpiParams e;
  e.mode = a.epilogue;
  e.out_bf16 = a.out_dtype == kBF16;
  e.accumulate = a.accumulate;
  e.bias = a.bias;
  e.aux = a.aux;
  e.C = a.C;
  e.C2 = a.C2;
  e.ldc = a.ldc;
  e.ad_w = a.adam.w; e.ad_m = a.adam.m; e.ad_v = a.adam.v; e.ad_wlp = (bf16*)a.adam.w_bf16; e.ad_c = a.adam.c_dev;
  e.ad_lr = a.adam.lr; e.ad_b1 = a.adam.b1; e.ad_b2 = a.adam.b2; e.ad_eps = a.adam.eps;
  e.ad_ic1 = e.ad_ic2 = 0.f;
  if (a.epilogue == kEpiAdam && !a.adam.c_dev) {   // the expressions of the Adam kernel
    e.ad_ic1 = 1.f / (1.f - powf(a.adam.b1, (float)a.adam.t));
    e.ad_ic2 = 1.f / (1.f - powf(a.adam.b2, (float)a.adam.t));
  }
  e.xe_tokens = a.xent.tokens; e.xe_part = a.xent.part; e.xe_zt = a.xent.zt; e.xe_lse = a.xent.lse;
  e.xe_inv_n = a.xent.inv_n; e.xe_T = a.xent.T; e.xe_V = (int)a.N; e.xe_groups = (int)(a.N / 64);
  return e;
}

static GemmBf16Params bf16_params_of(const GemmArgs& a, int tile) {
  GemmBf16Params p;
  p.A = (const bf16*)a.A;
  p.B = (const bf16*)a.B;
  p.M = a.M; p.N = a.N; p.K = a.K; p.lda = a.lda; p.ldb = a.ldb;
  p.tiles_m = (int)((a.M + tile - 1) / tile);
  p.tiles_n = (int)((a.N + tile - 1) / tile);
  p.b_colsum = a.b_colsum;
  p.colsum_accumulate = a.accumulate;
  p.epi = epi_of(a);
  return p;
}

// The ring-buffered kernel takes full 256 x 256 tiles only.
static bool ring_eligible(const GemmArgs& a) {
  return g_use_ring && a.dtype == kBF16 && gemm_ring_supported(a.M, a.N, a.K);
}

// The Adam epilogue lives in the ring kernel's weight-gradient instantiation (full 256 x 256 tiles, both operands
// k-major, fp32 product), alone when the problem fills most of the chip or as a member of a shared launch.
bool gemm_adam_fusable(const GemmArgs& a, bool grouped) {
  return ring_eligible(a) && a.a_kmajor && a.b_kmajor && a.out_dtype == kF32 && !a.accumulate &&
         (grouped || (a.M / 256) * (a.N / 256) >= 150);
}
// The loss epilogues live in the ring kernel's forward-layout instantiation.
bool gemm_xent_fusable(const GemmArgs& a) {
  return ring_eligible(a) && !a.a_kmajor && a.b_kmajor && (a.M / 256) * (a.N / 256) >= 150 && a.N <= (1 << 24);
}

bool gemm_colsum_fusable(const GemmArgs& a, bool paired) {
  return ring_eligible(a) && a.a_kmajor && a.b_kmajor && a.out_dtype == kF32 &&
         (a.epilogue == kEpiStore || a.epilogue == kEpiAdam) && (paired || (a.M / 256) * (a.N / 256) >= 150);
}

static hipError_t launch_gemm_impl(hipStream_t s, const GemmArgs& a) {
  bool empty;
  hipError_t err = check_gemm_args(a, &empty);
  if (err != hipSuccess || empty) return err;
  if (a.b_colsum && (!gemm_colsum_fusable(a, false) || ((uintptr_t)a.b_colsum & 3))) return hipErrorInvalidValue;
  if (a.epilogue == kEpiAdam)
    return gemm_adam_fusable(a, false) ? launch_gemm_ring(s, bf16_params_of(a, 256), true, true) : hipErrorInvalidValue;
  if (a.epilogue == kEpiXentStats || a.epilogue == kEpiXentGrad)
    return gemm_xent_fusable(a) ? launch_gemm_ring(s, bf16_params_of(a, 256), false, true) : hipErrorInvalidValue;

  if (a.dtype == kF32) {
    if ((a.M + 63) / 64 > 65535) return hipErrorInvalidValue;
    return launch_gemm_f32(s, a, epi_of(a));
  }
  // Full 256 x 256 tiles in rounds of one per compute unit: the ring-buffered kernel, which needs 1.4 times less of the chip
  // per FLOP than 128 x 128 tiles, and so
  //  * a single round from 150 tiles on if k is long (us, ring / tiles of 128: 2048 x 5120, 160 tiles, K 4096 79 / 92, K 2048 44 / 44,
  //    k-major 55 / 49; 2048 x 6144, 192 tiles, K 8192 159 / 178, K 4096 84 / 95, K 2048 46 / 48, k-major 56 / 54);
  //  * otherwise where at most a quarter of the rounds is idle (2048 x 8192 x 2048, 256 tiles, 57 / 64; 3072 x 6144 x 2048, 288 tiles,
  //    91 / 73);
  //  * and where the last round would be half full at most, the rounds before it, with that round's columns a problem of their
  //    own (2048 x 12288, 384 tiles, ring / 128 / both: K 8192 393 / 410 / 327, row-major A 314 / 342 / 296, K 4096 162 / 162 / 153,
  //    K 2048 87 / 92 / 86; K 1024 52 / 52 / 55; 8192 x 5120 x 2048, 640 tiles, 149 / - / 140).
  if (ring_eligible(a)) {
    const int64_t tm = a.M / 256, tiles = tm * (a.N / 256), slots = (tiles + 255) / 256 * 256, rest = tiles % 256;
    if (!a.b_colsum && a.K >= 2048 && tiles > 256 && rest > 0 && rest <= 128 && rest % tm == 0) {
      const int64_t n2 = rest / tm * 256, n1 = a.N - n2;
      const int64_t out_size = a.out_dtype == kBF16 ? 2 : 4, aux_size = a.epilogue == kEpiBiasResidual ? 4 : 2;
      GemmArgs head = a, tail = a;
      head.N = n1;
      tail.N = n2;
      tail.B = (const char*)a.B + (a.b_kmajor ? n1 : n1 * a.ldb) * 2;
      tail.C = (char*)a.C + n1 * out_size;
      if (a.bias) tail.bias = a.bias + n1;
      if (a.aux) tail.aux = (const char*)a.aux + n1 * aux_size;
      if (a.C2) tail.C2 = (char*)a.C2 + n1 * out_size;
      err = launch_gemm_impl(s, head);
      return err != hipSuccess ? err : launch_gemm_impl(s, tail);
    }
    if (a.b_colsum || (tiles >= 150 && (100 * tiles > 76 * slots || (tiles < 256 && a.K > 2048))))
      return launch_gemm_ring(s, bf16_params_of(a, 256), a.a_kmajor, a.b_kmajor);
  }
  return launch_gemm_tile(s, bf16_params_of(a, 256), a.a_kmajor, a.b_kmajor);
}

// Up to three independent GEMMs.  When all are ring-kernel problems of one operand layout, together fill at least
// most of the chip, and at least one of them would leave part of it idle (or miss the ring kernel) alone, they
// share a single launch (their tiles run side by side); otherwise one launch each.
bool gemm_group_shares_launch(const GemmArgs* a, int n) {
  if (n < 2 || n > kRingGroupMax) return false;
  int64_t total = 0;
  bool all_full_rounds = true;
  for (int i = 0; i < n; ++i) {
    if (a[i].M <= 0 || a[i].N <= 0 || !ring_eligible(a[i])) return false;
    if (a[i].a_kmajor != a[0].a_kmajor || a[i].b_kmajor != a[0].b_kmajor) return false;
    const int64_t t = (a[i].M / 256) * (a[i].N / 256);
    total += t;
    all_full_rounds = all_full_rounds && t % 256 == 0;
  }
  return total >= 150 && total <= (1 << 20) && !all_full_rounds;
}
bool gemm_pair_shares_launch(const GemmArgs& a0, const GemmArgs& a1) {
  const GemmArgs a[2] = {a0, a1};
  return gemm_group_shares_launch(a, 2);
}

hipError_t launch_gemm_group(hipStream_t s, const GemmArgs* a, int n) {
  if (n < 1 || n > kRingGroupMax || !a) return hipErrorInvalidValue;
  bool empty[kRingGroupMax], any_empty = false;
  for (int i = 0; i < n; ++i) {
    const hipError_t err = check_gemm_args(a[i], &empty[i]);
    if (err != hipSuccess) return err;
    any_empty = any_empty || empty[i];
  }
  const bool shared = !any_empty && gemm_group_shares_launch(a, n);
  for (int i = 0; i < n; ++i) {   // checked before anything is launched
    if (a[i].b_colsum && !gemm_colsum_fusable(a[i], shared)) return hipErrorInvalidValue;
    if (a[i].epilogue == kEpiAdam && !gemm_adam_fusable(a[i], shared)) return hipErrorInvalidValue;
    if (shared && (a[i].epilogue == kEpiAdam) != (a[0].epilogue == kEpiAdam)) return hipErrorInvalidValue;
    if (a[i].epilogue == kEpiXentStats || a[i].epilogue == kEpiXentGrad) return hipErrorInvalidValue;
  }
  if (!shared) {
    for (int i = 0; i < n; ++i) {
      const hipError_t err = launch_gemm(s, a[i]);
      if (err != hipSuccess) return err;
    }
    return hipSuccess;
  }
  // the larger problems' workgroups first
  int order[kRingGroupMax];
  double flops = 0.0;
  for (int i = 0; i < n; ++i) {
    order[i] = i;
    flops += 2.0 * (double)a[i].M * (double)a[i].N * (double)a[i].K;
  }
  std::stable_sort(order, order + n, [&](int x, int y) { return a[x].M * a[x].N > a[y].M * a[y].N; });
  GemmBf16Params p[kRingGroupMax];
  for (int i = 0; i < n; ++i) p[i] = bf16_params_of(a[order[i]], 256);
  const bool timed = g_profile_on;
  ProfiledLaunch pl{nullptr, nullptr, flops, a[0].epilogue == kEpiAdam, shape_key(a[order[0]], n)};
  hipError_t err = hipSuccess;
  if (timed) {
    pl.start = profile_event();
    pl.stop = profile_event();
    if (!pl.start || !pl.stop) return hipErrorOutOfMemory;
    err = hipEventRecord(pl.start, s);
    if (err != hipSuccess) return err;
  }
  err = launch_gemm_ring_group(s, p, n, a[0].a_kmajor, a[0].b_kmajor);
  if (timed && err == hipSuccess) {
    err = hipEventRecord(pl.stop, s);
    if (err == hipSuccess) g_profile.push_back(pl);
  }
  return err;
}

hipError_t launch_gemm_pair(hipStream_t s, const GemmArgs& a0, const GemmArgs& a1) {
  const GemmArgs a[2] = {a0, a1};
  return launch_gemm_group(s, a, 2);
}

}  // namespace pw
