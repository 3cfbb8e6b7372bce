// bf16 MFMA GEMM for any shape: the problems that do not fill the chip with full 256 x 256 tiles (gemm_ring.hip) - few
// tiles, ragged edges, a k that is no multiple of 64.
//
// What bounds such problems is latency and how many compute units take part, then the path from L2 into LDS.  A wave
// owns a 64 x 64 tile (16 accumulator blocks of v_mfma_f32_16x16x32_bf16); WM x WN waves form a group that shares its
// operand tiles in LDS, and WK groups of one workgroup split k between them, so that a problem of few tiles still has
// all its compute units' waves at work.  The groups' partial tiles meet in LDS and are added in group order (the same
// bits on every run); the epilogue reads the sum row-wise.
//
// Operands travel global -> LDS directly (global_load_lds_dwordx4: no staging registers, no LDS stores) and, stored
// k-major, come out of LDS through ds_read_b64_tr_b16 - the instruction facts are those of gemm_ring.hip.  Ragged
// problems take the same path: rows past the end are fetched from rows that exist (a product row depends on its own
// operand row only, and those rows are never stored), and in the last, partial k tile every 16-byte chunk past the end of
// k is fetched from a block of zeros.
//
#include "common.hpp"
#include "gemm_common.hpp"
#include "kernels.hpp"

#include <type_traits>

namespace pw {

namespace {

constexpr int kTBK = 64;   // k per stage
typedef __attribute__((address_space(3))) void* lds_ptr;
typedef short short4v __attribute__((ext_vector_type(4)));

__device__ __attribute__((aligned(16))) const uint32_t kZeros[4] = {0, 0, 0, 0};

__device__ __forceinline__ void dma16(const bf16* g, uint32_t lds_off) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(g), "s"(lds_off) : "memory", "m0");
}

// LDS layout of an operand tile of R rows x 64 k (16-byte chunks):
//  row-major: [R][8 chunks of 8 k], chunk c of row r at position c ^ ((r >> 1) & 7);
//  k-major:   [64 k][R / 8 chunks of 8 rows], chunk c of k-row k at c ^ kswz(k): the eight k-rows of 32 bytes that the
//             first 32 lanes of a transposing read touch (k0..k0+3, k0+8..k0+11) fall into eight different 32-byte windows
//             of the 256 bytes all banks hold - by the chunk alone where a k-row is 256 bytes, by the chunk and the
//             parity of k where it is 128.
template <int R> __device__ __forceinline__ int kswz(int k) {
  static_assert(R == 64 || R == 128, "tile heights in use");
  return R == 128 ? (4 * (k & 3)) ^ (2 * ((k >> 3) & 1)) : (2 * ((k >> 1) & 1)) ^ (4 * ((k >> 3) & 1));
}

// The same with a wave-uniform base and a 32-bit byte offset per lane.
__device__ __forceinline__ void dma16_s(const bf16* base, uint32_t off, uint32_t lds_off) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(base), "s"(lds_off) : "memory", "m0");
}

// One operand of a group's tile: R rows, fetched by G waves in pieces of 1 KiB.  A lane's byte offsets inside a k tile do
// not change from tile to tile (rows past the end are clamped); the tile's base is wave-uniform.  32-bit offsets reach as
// far as leading dimensions up to kMaxLd; WIDE has 64-bit ones.
constexpr int64_t kMaxLd = 1 << 23;
template <int R, int G, bool KMAJOR, bool WIDE>
struct Operand {
  typedef typename std::conditional<WIDE, uint64_t, uint32_t>::type offset;
  static constexpr int kPer = R / 8 / G;        // direct-load instructions per wave and k tile
  const bf16* base;                             // of the next tile to be issued
  int64_t step;                                 // elements per k tile
  offset off[kPer];
  __device__ __forceinline__ static int k_of(int instr, int lane) {   // first k of the lane's chunk inside the tile
    return KMAJOR ? instr * (512 / R) + lane / (R / 8) : ((lane & 7) ^ (((instr * 8 + (lane >> 3)) >> 1) & 7)) * 8;
  }
  __device__ __forceinline__ void init(const bf16* p, int64_t ld, int64_t row0, int64_t rows, int64_t first, int gw, int lane) {
    step = KMAJOR ? (int64_t)kTBK * ld : kTBK;
    base = p + (KMAJOR ? row0 : row0 * ld) + first * step;
    const int last = (int)(rows - row0 < R ? rows - row0 : R) - (KMAJOR ? 8 : 1);   // rows is a multiple of 8 if k-major
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const int instr = gw * kPer + j, k = k_of(instr, lane);
      if (KMAJOR) {
        const int r = min(((lane % (R / 8)) ^ kswz<R>(k)) * 8, last);
        off[j] = (offset)((k * ld + r) * 2);
      } else {
        const int r = min(instr * 8 + (lane >> 3), last);
        off[j] = (offset)((r * ld + k) * 2);
      }
    }
  }
  // Instruction j of the next k tile (a whole one) into LDS at lds_off.
  __device__ __forceinline__ void issue_one(int j, uint32_t lds_off, int gw) const {
    if constexpr (WIDE) dma16(at(j), lds_off + (gw * kPer + j) * 1024);
    else dma16_s(base, off[j], lds_off + (gw * kPer + j) * 1024);
  }
  __device__ __forceinline__ const bf16* at(int j) const {
    return reinterpret_cast<const bf16*>(reinterpret_cast<const char*>(base) + off[j]);
  }
  // The next k tile, of which `left` k exist (a multiple of 8).
  __device__ __forceinline__ void issue(int64_t left, uint32_t lds_off, int gw, int lane) const {
    if (left >= kTBK) {
#pragma unroll
      for (int j = 0; j < kPer; ++j) issue_one(j, lds_off, gw);
    } else {
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        const bf16* g = at(j);
        if (k_of(gw * kPer + j, lane) >= left) g = reinterpret_cast<const bf16*>(kZeros);
        dma16(g, lds_off + (gw * kPer + j) * 1024);
      }
    }
  }
  __device__ __forceinline__ void advance() { base += step; }
};

// The fragments of v_mfma_f32_16x16x32_bf16 that a lane reads from an operand tile: block j = rows row0 + 16 j + lane % 16,
// k = 32 kk + 8 (lane / 16) .. + 7.  The swizzle depends on the lane and - row-major - on kk or - k-major - on j, so two or
// four LDS addresses are kept; everything else (the other index, the second half of a transposing read, the stage) is an
// immediate offset.  (Row blocks are multiples of 16 and neither 32 kk nor the second half's + 4 reaches the bits of k
// that the swizzle looks at.)
template <int R, bool KMAJOR>
struct FragmentReader {
  uint32_t at[KMAJOR ? 4 : 2];
  __device__ __forceinline__ void init(uint32_t tile_off, int row0, int lane) {
    const int grp = lane >> 4, L = lane & 15;
    if (KMAJOR) {
      const int k = 8 * grp + (L >> 2);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int chunk = (row0 >> 3) + 2 * j + ((L & 3) >> 1);
        at[j] = tile_off + k * (2 * R) + ((chunk ^ kswz<R>(k)) << 4) + 8 * (L & 1);
      }
    } else {
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) at[kk] = tile_off + (row0 + L) * (2 * kTBK) + (((4 * kk + grp) ^ (L >> 1)) << 4);
    }
    // The addresses are kept as they are: left alone the compiler keeps one for every (stage, kk, j) instead.
#pragma unroll
    for (int j = 0; j < (KMAJOR ? 4 : 2); ++j) asm volatile("" : "+v"(at[j]));
  }
  __device__ __forceinline__ bf16x8 read(uint32_t stage_off, int kk, int j) const {
    if (!KMAJOR) {
      typedef __attribute__((address_space(3))) const bf16x8* p;
      return *(p)(uintptr_t)(at[kk] + stage_off + j * 16 * 2 * kTBK);
    } else {
      typedef __attribute__((address_space(3))) short4v* p;
      union { bf16x8 v; short4v h[2]; } u;
#pragma unroll
      for (int t = 0; t < 2; ++t)
        u.h[t] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((p)(uintptr_t)(at[j] + stage_off + kk * 64 * R + t * 8 * R));
      return u.v;
    }
  }
};

// WM x WN waves per group, WK groups, DEEP: see the main loop.
constexpr int NS = 2;   // stages of LDS per group (four, one workgroup per compute unit: no faster)
template <int WM_, int WN_, int WK_, bool DEEP_>
struct Shape {
  static constexpr int WM = WM_, WN = WN_, WK = WK_;
  static constexpr bool DEEP = DEEP_;
  static constexpr bool kSkew = WK > 1 && WM * WN > 1;               // the second group runs half a tile behind the first,
  static constexpr int kApartFrom = WM * WN == 4 ? 0 : 13;           // from this many k tiles on
  static constexpr int BM = 64 * WM, BN = 64 * WN, G = WM * WN, kThreads = 64 * G * WK;
  static constexpr int kWavesPerSimd = WK == 1 || kThreads == 512 ? 2 : 1;
  static constexpr int kStage = (BM + BN) * kTBK;                    // elements
  static constexpr int kLdP = BN + 4;                                // floats per row of a partial tile
  static constexpr size_t kRing = (size_t)WK * NS * kStage * 2, kParts = (size_t)WK * BM * kLdP * 4;
  static constexpr size_t kSmem = kRing > kParts ? kRing : kParts;
};

// Sum of the groups' partial tiles and the epilogue, 8 consecutive columns per lane and step.
template <class S, int KIND>
__device__ __forceinline__ void finish(const float* parts, const GemmBf16Params& p, int64_t m0, int64_t n0) {
  constexpr int kCols = S::BN / 8, kRows = S::kThreads / kCols;   // rows one step covers
  constexpr int kSteps = S::BM / kRows;
  const void* const src = epi_extra_src(p.epi, KIND);
  const int row0 = threadIdx.x / kCols, col = threadIdx.x % kCols * 8;
  const int64_t n = n0 + col;
  auto sum = [&](int row, float* v) {
#pragma unroll
    for (int g = 0; g < S::WK; ++g) {
      const float* q = parts + (g * S::BM + row) * S::kLdP + col;
      const f32x4 a = *reinterpret_cast<const f32x4*>(q), b = *reinterpret_cast<const f32x4*>(q + 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] = g == 0 ? a[e] : v[e] + a[e];
        v[e + 4] = g == 0 ? b[e] : v[e + 4] + b[e];
      }
    }
  };
  // The same columns in every step, of ragged tiles too (fetched per step there, 1672 x 1800 x 256 with GELU: 11.0 -> 10.0 us).  What is
  // left of a row behind its last vector goes by epilogue1.
  float bias[8] = {};
  if (epi_has_bias(p.epi.mode) && p.epi.bias && n + 7 < p.N) {
    const f32x4 a = *reinterpret_cast<const f32x4*>(p.epi.bias + n), b = *reinterpret_cast<const f32x4*>(p.epi.bias + n + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      bias[e] = a[e];
      bias[e + 4] = b[e];
    }
  }
  if (m0 + S::BM <= p.M && n0 + S::BN <= p.N) {
    EpiExtra x[kSteps] = {};                  // everything the epilogue reads is on its way before the tiles meet
    if (KIND != kExtraNone) {
#pragma unroll
      for (int i = 0; i < kSteps; ++i) epi_extra_load(KIND, src, (m0 + row0 + i * kRows) * p.epi.ldc + n, x[i]);
    }
    __syncthreads();                          // every partial tile is in LDS
#pragma unroll
    for (int i = 0; i < kSteps; ++i) {
      float v[8];
      sum(row0 + i * kRows, v);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] += bias[e];
      epilogue8<false>(p.epi, m0 + row0 + i * kRows, n, v, KIND, x[i]);
    }
    return;
  }
  __syncthreads();
#pragma unroll 1
  for (int i = 0; i < kSteps; ++i) {
    const int64_t m = m0 + row0 + i * kRows;
    float v[8];
    sum(row0 + i * kRows, v);
    if (m < p.M && n + 7 < p.N) {
      EpiExtra x = {};
      epi_extra_load(KIND, src, m * p.epi.ldc + n, x);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] += bias[e];
      epilogue8<false>(p.epi, m, n, v, KIND, x);
    } else if (m < p.M) {
#pragma unroll 1
      for (int e = 0; n + e < p.N && e < 8; ++e) epilogue1<true>(p.epi, m, n + e, v[e]);
    }
  }
}

template <class S, bool AK, bool BK_, bool WIDE = false>
__global__ __launch_bounds__(S::kThreads, S::kWavesPerSimd) void gemm_tile_kernel(GemmBf16Params p) {
  constexpr int G = S::G, WN = S::WN, WK = S::WK;
  constexpr bool kShared = G > 1;             // several waves read one operand tile: barriers; else every wave is on its own
  using OpA = Operand<S::BM, G, AK, WIDE>;
  using OpB = Operand<S::BN, G, BK_, WIDE>;
  constexpr int kPer = OpA::kPer + OpB::kPer;
  extern __shared__ __attribute__((aligned(1024))) bf16 smem[];
  int tm, tn;
  tile_of_block(blockIdx.x, p.tiles_m * p.tiles_n, p.tiles_m, p.tiles_n, tm, tn);
  const int64_t m0 = (int64_t)tm * S::BM, n0 = (int64_t)tn * S::BN;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int g = wave / G, gw = wave % G, wm = gw / WN, wn = gw % WN;

  f32x4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int total = (int)((p.K + kTBK - 1) / kTBK), per = (total + WK - 1) / WK;
  const int first = g * per, n = total - first < per ? (total - first < 0 ? 0 : total - first) : per;
  OpA oa;
  OpB ob;
  oa.init(p.A, p.lda, m0, p.M, first, gw, lane);
  ob.init(p.B, p.ldb, n0, p.N, first, gw, lane);
  const uint32_t ring_off = (uint32_t)(uintptr_t)(lds_ptr)smem + g * (NS * S::kStage * 2);
  FragmentReader<S::BM, AK> ra;
  FragmentReader<S::BN, BK_> rb;
  ra.init(ring_off, wm * 64, lane);
  rb.init(ring_off + S::BM * kTBK * 2, wn * 64, lane);
  auto issue = [&](int i) {
    const int64_t left = p.K - (int64_t)(first + i) * kTBK;
    const uint32_t st = ring_off + (uint32_t)(i % NS) * (S::kStage * 2);
    oa.issue(left, st, gw, lane);
    ob.issue(left, st + S::BM * kTBK * 2, gw, lane);
    oa.advance();
    ob.advance();
  };
  bf16x8 fa[2][2][4], fb[2][2][4];            // [tile parity][32-deep k step][16-row block]
  auto read_one = [&](int i, int kk, int m, bf16x8 (&a)[4], bf16x8 (&b)[4]) {   // m: 0..3 B blocks, 4..7 A blocks
    const uint32_t st = (uint32_t)(i % NS) * (S::kStage * 2);
    if (m < 4) b[m] = rb.read(st, kk, m);
    else a[m - 4] = ra.read(st, kk, m - 4);
  };
  auto read = [&](int i, int kk, bf16x8 (&a)[4], bf16x8 (&b)[4]) {
#pragma unroll
    for (int m = 0; m < 8; ++m) read_one(i, kk, m, a, b);
  };
  // 16 MFMAs; before(m) runs in front of the m-th and stays there.
  auto multiply = [&](const bf16x8 (&a)[4], const bf16x8 (&b)[4], auto&& before) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {        // back and forth: consecutive MFMAs share an operand
        const int j = (i & 1) ? 3 - jj : jj;
        __builtin_amdgcn_sched_barrier(0);
        before(4 * i + jj);
        __builtin_amdgcn_sched_barrier(0);
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a[i], acc[i][j], 0, 0, 0);
      }
    __builtin_amdgcn_sched_barrier(0);
  };
  // Instruction m of the next (whole) k tile, which goes to the stage of tile i.
  auto issue_one = [&](int i, int m) {
    const uint32_t st = ring_off + (uint32_t)(i % NS) * (S::kStage * 2);
    if (m < OpA::kPer) oa.issue_one(m, st, gw);
    else ob.issue_one(m - OpA::kPer, st + S::BM * kTBK * 2, gw);
    if (m == kPer - 1) {
      oa.advance();
      ob.advance();
    }
  };
  auto landed = [&](int after) {              // all direct loads but those of `after` later tiles
    if (after) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kPer) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  };
  auto reads_done = [&] { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); };
  auto meet = [&] {
    if (kShared) __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  auto idle = [](int) {};
  auto least = [](int x, int y) { return x < y ? x : y; };

#pragma unroll
  for (int i = 0; i < NS; ++i)
    if (i < n) issue(i);
  if (n > 0) landed(least(NS, n) - 1);
  meet();
  if (n > 0) {
    read(0, 0, fa[0][0], fb[0][0]);
    read(0, 1, fa[0][1], fb[0][1]);
  }
  // Direct loads go out one by one between MFMAs (issued in one go they hold the wave up until the load path has taken
  // them all: 2048 x 2048 x 8192 with both operands row-major 92 -> 66 us).
  // STREAM: what tile i asks for exists, and the tile to be loaded is a whole one.
  auto tile = [&](int i, auto index, auto streaming) {
    constexpr int c = decltype(index)::value & 1;
    constexpr bool STREAM = decltype(streaming)::value;
    if constexpr (S::DEEP) {
      // All of tile i + 1 is read under the first half of tile i, which frees its stage halfway for tile i + 1 + NS.
      if (STREAM) landed(NS - 1);
      else if (i + 1 < n) landed(least(NS - 1, n - 2 - i));
      meet();
      if (STREAM) {
        multiply(fa[c][0], fb[c][0], [&](int m) {
          if (m < 8) {
            read_one(i + 1, 0, m, fa[c ^ 1][0], fb[c ^ 1][0]);
            read_one(i + 1, 1, m, fa[c ^ 1][1], fb[c ^ 1][1]);
          }
        });
      } else {
        if (i + 1 < n) {
          read(i + 1, 0, fa[c ^ 1][0], fb[c ^ 1][0]);
          read(i + 1, 1, fa[c ^ 1][1], fb[c ^ 1][1]);
        }
        if (i < n) multiply(fa[c][0], fb[c][0], idle);
      }
      reads_done();
      meet();
      if (STREAM) {
        multiply(fa[c][1], fb[c][1], [&](int m) {
          if ((m + 1) * kPer / 16 > m * kPer / 16) issue_one(i + 1, m * kPer / 16);
        });
      } else {
        if (i + 1 + NS < n) issue(i + 1 + NS);
        if (i < n) multiply(fa[c][1], fb[c][1], idle);
      }
    } else {
      // One barrier: behind it tile i + 1 is visible and the stage of tile i is free for tile i + NS.
      if (STREAM) landed(NS - 2);
      else if (i + 1 < n) landed(least(NS - 2, n - 2 - i));
      reads_done();
      meet();
      if (STREAM) {
        multiply(fa[c][0], fb[c][0], [&](int m) {
          if (m & 1) read_one(i + 1, 0, m >> 1, fa[c ^ 1][0], fb[c ^ 1][0]);
          else issue_one(i, m >> 1);
        });
        multiply(fa[c][1], fb[c][1], [&](int m) {
          if (m < 8) read_one(i + 1, 1, m, fa[c ^ 1][1], fb[c ^ 1][1]);
        });
      } else {
        if (i + NS < n) issue(i + NS);
        if (i + 1 < n) read(i + 1, 0, fa[c ^ 1][0], fb[c ^ 1][0]);
        if (i < n) multiply(fa[c][0], fb[c][0], idle);
        if (i + 1 < n) read(i + 1, 1, fa[c ^ 1][1], fb[c ^ 1][1]);
        if (i < n) multiply(fa[c][1], fb[c][1], idle);
      }
    }
  };
  if constexpr (S::DEEP) {
    reads_done();
    meet();
    if (n > NS) issue(NS);
  }
  static_assert(S::DEEP ? kPer <= 16 : kPer == 8, "one direct load at most in front of each MFMA of a half");
  static_assert(NS == 2, "two stages: the waits leave at most one tile in flight, the loop goes two tiles a round");
  constexpr int kAhead = S::DEEP ? NS + 1 : NS;   // tile i loads tile i + kAhead
  // Two groups of several waves: one of them reads its operand tiles from LDS while the other multiplies.  In step, LDS and matrix
  // pipe take turns (us, 128 x 128 tiles, four waves alone / two groups in step / half a tile apart, profiles of one launch: the main
  // loop of 1000 x 3072 x 768 5.3 / 5.5 / 4.2, of 2048 x 2048 x 2048 13.8 / 14.3 / 11.6).  Apart, no unit is full: in 2048 x 2048 products
  // with k from 2048 to 6144, row-major, the matrix pipe is busy 34 % of a launch, LDS reads of the waves 18 %, and a wave waits to issue
  // 45 % of its time and on counters 39 % (with a transposing read and its spills 26, 14, 46 and 41 %).  Each group passes as many
  // barriers as the other.
  // The half tile at either end has to be earned back: two pairs of waves need 13 k tiles (128 x 64 tiles, in step / apart: 1280 x 1280 x
  // 256 6.7 / 6.9, 768 9.2 / 9.2, 1536 13.1 / 12.4; 1024 x 1536 x 832 8.9 / 8.8, 960 9.6 / 9.2), two groups of four waves none
  // (1536 x 1536 x 256, row-major, 7.1 / 7.0, 768 10.4 / 9.6).
  const bool apart = S::kSkew && total >= S::kApartFrom;
  if (apart && g == 1) meet();
  int i = 0;
  for (; i + NS - 1 + kAhead < n - 1; i += NS) {  // NS tiles, none of which loads the last one
    tile(i, std::integral_constant<int, 0>{}, std::true_type{});
    tile(i + 1, std::integral_constant<int, 1>{}, std::true_type{});
  }
  const int rounds = kShared ? per : n;           // with barriers inside, every group goes round equally often
  for (; i < rounds; i += 2) {
    tile(i, std::integral_constant<int, 0>{}, std::false_type{});
    if (i + 1 < rounds) tile(i + 1, std::integral_constant<int, 1>{}, std::false_type{});
  }

  if (apart && g == 0) meet();
  __syncthreads();                            // nobody reads operand tiles any more
  float* const parts = reinterpret_cast<float*>(smem);
  float* mine = parts + (g * S::BM + wm * 64 + (lane & 15)) * S::kLdP + wn * 64 + 4 * (lane >> 4);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) *reinterpret_cast<f32x4*>(mine + 16 * i * S::kLdP + 16 * j) = acc[i][j];
  switch (epi_extra_kind(p.epi)) {            // uniform over the launch
    case kExtraAuxBf16: finish<S, kExtraAuxBf16>(parts, p, m0, n0); break;
    case kExtraAuxF32: finish<S, kExtraAuxF32>(parts, p, m0, n0); break;
    case kExtraOldC: finish<S, kExtraOldC>(parts, p, m0, n0); break;
    default: finish<S, kExtraNone>(parts, p, m0, n0); break;
  }
}

template <class S, bool WIDE = false>
hipError_t prepare() {
  const void* const k[] = {reinterpret_cast<const void*>(gemm_tile_kernel<S, false, false, WIDE>),
                           reinterpret_cast<const void*>(gemm_tile_kernel<S, false, true, WIDE>),
                           reinterpret_cast<const void*>(gemm_tile_kernel<S, true, false, WIDE>),
                           reinterpret_cast<const void*>(gemm_tile_kernel<S, true, true, WIDE>)};
  for (const void* f : k) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::kSmem);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <class S, bool WIDE = false>
hipError_t launch(hipStream_t s, GemmBf16Params p, bool ak, bool bk) {
  const int64_t tm = (p.M + S::BM - 1) / S::BM, tn = (p.N + S::BN - 1) / S::BN;
  if (tm * tn > (1LL << 26)) return hipErrorInvalidValue;
  p.tiles_m = (int)tm;
  p.tiles_n = (int)tn;
  const int grid = (int)(tm * tn);
  if (!ak && !bk) gemm_tile_kernel<S, false, false, WIDE><<<grid, S::kThreads, S::kSmem, s>>>(p);
  else if (!ak) gemm_tile_kernel<S, false, true, WIDE><<<grid, S::kThreads, S::kSmem, s>>>(p);
  else if (!bk) gemm_tile_kernel<S, true, false, WIDE><<<grid, S::kThreads, S::kSmem, s>>>(p);
  else gemm_tile_kernel<S, true, true, WIDE><<<grid, S::kThreads, S::kSmem, s>>>(p);
  return hipGetLastError();
}

using Split = Shape<1, 1, 4, true>;     // 64 x 64 tiles, k over four waves of their own (one per SIMD: 300 registers)
using Half = Shape<2, 1, 2, true>;      // 128 x 64 tiles, k over two pairs of waves (likewise)
using Duo = Shape<2, 2, 2, true>;       // 128 x 128 tiles, k over two groups of four waves (two per SIMD)
using One = Shape<2, 2, 1, true>;       // 128 x 128 tiles, two workgroups per compute unit
using Two = Shape<2, 2, 1, false>;      // the same with the leaner loop

}  // namespace

hipError_t gemm_tile_init() {
  hipError_t e = prepare<Split>();
  if (e == hipSuccess) e = prepare<Split, true>();
  if (e == hipSuccess) e = prepare<Half>();
  if (e == hipSuccess) e = prepare<Duo>();
  if (e == hipSuccess) e = prepare<One>();
  if (e == hipSuccess) e = prepare<Two>();
  return e;
}

// Which shape (us per launch before: 128 x 128 tiles staged through registers, or full ring tiles on half the chip).
// The fewer tiles of 128 x 128 there are, the smaller the tile and the more waves share its k: 1000 x 768 x 3072 (48
// tiles) 51 -> 13 with Split (Half 20, One 24); 1280 x 1280 x 4096 (100) 72 -> 23 with Half (Split 30, One 30, Duo 28); up to one
// tile per compute unit One, or Duo where that wins (duo_pays).  Beyond that
// two workgroups share a compute unit and hide each other's waits; with a long k the leaner loop is ahead (2048 x 8000 x
// 8000: 216 against 251), with a short one it is not (4568 x 2240 x 1152: 32 against 29; 4096 x 4352 x 2048: 79 / 75).
//
// Duo saves a fifth of the main loop and pays with a second tile of partial sums through LDS (0.3 to 0.5 us).  One / Duo, us:
//   both operands row-major (without spills), from k = 1024 on: bf16 out 1536 x 1536 x 640 8.9 / 9.3, 768 9.6 / 9.5, 1024 10.9 / 10.6, 2048 17.4 /
//     16.3; residual 1024 x 3072 x 768 12.6 / 12.7, 1024 14.5 / 14.2; GELU 768 11.7 / 11.8, 1024 13.1 / 12.8;
//   ragged ones, whose rows wait for their old values or aux step by step and have half as many steps in Duo, from 256: 1000 x 3000 x 256 bf16
//     out 7.7 / 7.5, GELU' 9.7 / 8.8, residual 10.4 / 10.0; 768 GELU' 13.1 / 12.0; 192 residual 9.7 / 9.9;
//   plain fp32 out, where the stores come on top, from 1536: 1000 x 3000 x 768 12.1 / 12.2, 2000 x 2000 x 1024 14.2 / 14.4, 1536 x 1536 x 1536 15.6 /
//     15.6, 2048 18.6 / 17.9;
//   other layouts (a few registers spill, or transposing reads of both), whole tiles, from 2048: 2048 x 2048 x 1024, fp32 15.8 / 15.9, GELU
//     14.5 / 14.8, 1536 19.5 / 19.2, 18.6 / 18.5, 2048 22.9 / 22.3, 22.4 / 22.0, k-major 23.2 / 21.8;
//   ragged, from 4096: 2000 x 2000 x 2048 22.8 / 23.0, k-major 22.8 / 23.4, 1672 x 1800 x 3072 bf16 out 26.3 / 26.3, 4096 33.1 / 32.5, k-major
//     36.5 / 36.8, 1000 x 3000 x 4096 with a residual 35.9 / 34.5; but GELU' as above: x 256 9.7 / 9.1, 1024 15.8 / 14.8, 2048 22.9 / 21.2.
static bool duo_pays(const GemmBf16Params& p, bool ak, bool bk) {
  const bool whole = p.M % 128 == 0 && p.N % 128 == 0, rows = !ak && !bk;
  const bool plain = p.epi.mode == kEpiStore && !p.epi.out_bf16 && !p.epi.accumulate;
  if (!whole && (p.epi.mode == kEpiGeluBwd || (rows && !plain))) return p.K >= 256;
  if (rows) return p.K >= (plain ? 1536 : 1024);
  return p.K >= (whole ? 2048 : 4096);
}
hipError_t launch_gemm_tile(hipStream_t s, const GemmBf16Params& p, bool ak, bool bk) {
  if (p.lda > kMaxLd || p.ldb > kMaxLd) return launch<Split, true>(s, p, ak, bk);
  const int64_t t128 = ((p.M + 127) / 128) * ((p.N + 127) / 128);
  if (t128 <= 64) return launch<Split>(s, p, ak, bk);
  if (t128 <= 128) return launch<Half>(s, p, ak, bk);
  if (t128 <= 256 && duo_pays(p, ak, bk)) return launch<Duo>(s, p, ak, bk);
  if (t128 <= 256 || p.K <= 2048) return launch<One>(s, p, ak, bk);
  return launch<Two>(s, p, ak, bk);
}

}  // namespace pw
