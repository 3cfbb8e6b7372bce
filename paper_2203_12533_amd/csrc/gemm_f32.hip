// fp32 GEMM on the matrix cores: v_mfma_f32_16x16x4_f32 (fp32 products and sums), any M, N, K, strides and alignment.
//
// What bounds it: the matrix pipe gives 256 fp32 FLOP per clock and compute unit, so slowly against the bf16 shapes
// that operand fragments can come straight from global memory into registers - a wave tile of 32 x 32 needs 8 bytes
// per clock, a tile of 64 x 64 needs 4 - and there is neither an LDS tile nor a barrier in the main loop.  The
// problems of the fp32 configuration are small (512 x 256 outputs): what costs there is the length of the serial
// k-loop and how few compute units take part in it, so the k-range of an output tile is cut into slices, one wave
// each, whose partial tiles meet in LDS and are added in slice order (the same bits on every run).  The shorter sums
// also round less: against 64 bits 1.5e-7 ... 2.9e-7 where one long sum has 2.9e-7 ... 5.7e-7.
// Measured (us per launch, MI355X, the same operands again and again; before: 64 x 64 tiles on the vector ALU, one k-loop):
// 512 x 256 x 1024 133 -> 7.1, 512 x 1024 x 256 36 -> 7.6, 1024 x 256 x 512 (weight gradient) 72 -> 7.0, 1000 x 512 x 2048 360 -> 30,
// 2048^3 451 -> 156 (110 TFLOP/s of the 157 the fp32 matrix pipe has at 2.4 GHz), 4096 x 4096 x 1024 646 -> 289.  Behind other kernels,
// in a feed-forward block of 512 x 256 x 1024, the first three take 8.7, 9.1 (with the GELU epilogue) and 7.0.
//
// Fragments.  The instruction takes one value per lane and operand: row lane%16, k-slot lane/16.  Which k a slot stands
// for and which tile row a fragment row stands for is free as long as both operands (and the epilogue) agree:
//   step of 16 k: MFMA i (0..3) uses k = 4 (lane/16) + i;   block j of F: tile row F (lane%16) + j.
// An operand stored [row][k] is then read as 16-byte pieces along k, one stored [k][row] as F-value pieces along the
// rows.  Issued with the B fragment first, a lane ends up with row F (lane%16) + i and the 4 F consecutive columns
// 4 F (lane/16) .. of the product: vector stores without a detour.
#include "common.hpp"
#include "gemm_common.hpp"
#include "kernels.hpp"

#include <type_traits>

namespace pw {

namespace {

// Vectors of floats with the alignment of a float: global memory takes such accesses at any 4-byte boundary.
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x2u __attribute__((ext_vector_type(2), aligned(4)));
template <int F> struct PieceOf;
template <> struct PieceOf<1> { typedef float type __attribute__((ext_vector_type(1), aligned(4))); };
template <> struct PieceOf<2> { typedef f32x2u type; };
template <> struct PieceOf<4> { typedef f32x4u type; };

constexpr int kStepK = 16;

// One operand as a wave sees it.  rows: extent of the operand's row dimension, row0: first row of the wave tile.
template <int F, bool KMAJOR>
struct F32Operand {
  const float* p[KMAJOR ? 1 : F];
  const float* base;
  int64_t ld, row0, rows;
  int shift;
  // Rows past the end are fetched from rows that exist (their products are never stored): row-major clamps the row;
  // k-major pulls the piece of F rows back inside and `shift` says by how many places it moved.
  __device__ __forceinline__ void init(const float* b, int64_t ld_, int64_t row0_, int64_t rows_, int lane) {
    base = b; ld = ld_; row0 = row0_; rows = rows_;
    const int c = lane & 15, q = lane >> 4;
    shift = 0;
    if (KMAJOR) {
      int64_t r = row0 + F * c;
      if (r > rows - F) {
        const int64_t back = r - (rows - F);
        shift = back < F ? (int)back : F;
        r = rows - F;
      }
      p[0] = base + (int64_t)(4 * q) * ld + r;
    } else {
#pragma unroll
      for (int j = 0; j < F; ++j) {
        const int64_t r = row0 + F * c + j;
        p[j] = base + (r < rows ? r : rows - 1) * ld + 4 * q;
      }
    }
  }
  // A whole step (16 k, all of them inside).  EDGE: the wave tile reaches past the last row.
  template <bool EDGE>
  __device__ __forceinline__ void load(int64_t k0, float (&f)[4][F]) const {
    if (KMAJOR) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        typename PieceOf<F>::type v = *reinterpret_cast<const typename PieceOf<F>::type*>(p[0] + (k0 + i) * ld);
        if (EDGE) {
#pragma unroll
          for (int j = 0; j < F; ++j) {
            float t = v[j];
#pragma unroll
            for (int m = j + 1; m < F; ++m) t = shift == m - j ? v[m] : t;
            f[i][j] = t;
          }
        } else {
#pragma unroll
          for (int j = 0; j < F; ++j) f[i][j] = v[j];
        }
      }
    } else {
#pragma unroll
      for (int j = 0; j < F; ++j) {
        const f32x4u v = *reinterpret_cast<const f32x4u*>(p[j] + k0);
#pragma unroll
        for (int i = 0; i < 4; ++i) f[i][j] = v[i];
      }
    }
  }
  // Element by element, zero outside: the last, partial step of k, and operands of fewer than F rows.
  __device__ __forceinline__ void load_guarded(int64_t k0, int64_t K, int lane, float (&f)[4][F]) const {
    const int c = lane & 15, q = lane >> 4;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < F; ++j) {
        const int64_t k = k0 + 4 * q + i, r = row0 + F * c + j;
        f[i][j] = (k < K && r < rows) ? base[KMAJOR ? k * ld + r : r * ld + k] : 0.f;
      }
  }
};

struct GemmF32Params {
  const float* A;
  const float* B;
  int64_t M, N, K, lda, ldb;
  int tiles_m, tiles_n;
  EpiParams epi;
};

// One 16 FM x 16 F output tile per workgroup; its kWK waves take one slice of k each.
constexpr int kWK = 4;
template <int FM, int F, bool AK, bool BK_>
__global__ __launch_bounds__(64 * kWK) void gemm_f32_kernel(GemmF32Params p) {
  constexpr int TM = 16 * FM, T = 16 * F;
  // Steps in flight per wave.  Four or three on 16 x 32 tiles (us, 512 x 256 x 1024): A row-major and B k-major 7.3 / 7.7, both
  // k-major 7.5 / 7.5, both row-major 8.7 / 8.5, A k-major and B row-major 8.4 / 7.6.
  constexpr int kDepth = F == 2 ? 5 - FM : 2;
  int tm, tn;
  tile_of_block(blockIdx.x, p.tiles_m * p.tiles_n, p.tiles_m, p.tiles_n, tm, tn);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t m0 = (int64_t)tm * TM, n0 = (int64_t)tn * T;

  f32x4 acc[FM][F];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto multiply = [&](const float (&a)[4][FM], const float (&b)[4][F]) {
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < F; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[k][j], a[k][i], acc[i][j], 0, 0, 0);
  };

  const int64_t steps = (p.K + kStepK - 1) / kStepK, whole = p.K / kStepK;
  const int64_t per = (steps + kWK - 1) / kWK;
  const int64_t s0 = wave * per, s1 = (s0 + per < steps ? s0 + per : steps);
  if (s0 < s1) {
    F32Operand<FM, AK> oa;
    F32Operand<F, BK_> ob;
    oa.init(p.A, p.lda, m0, p.M, lane);
    ob.init(p.B, p.ldb, n0, p.N, lane);
    const bool tiny = p.M < FM || p.N < F;
    const bool edge = m0 + TM > p.M || n0 + T > p.N;
    const int64_t sw = tiny ? s0 : (s1 < whole ? s1 : whole);   // steps s0 .. sw-1 load whole pieces
    auto stream = [&](auto e) {
      constexpr bool EDGE = decltype(e)::value;
      float fa[kDepth][4][FM], fb[kDepth][4][F];
      int64_t s = s0;
#pragma unroll
      for (int d = 0; d < kDepth; ++d)
        if (s + d < sw) {
          oa.template load<EDGE>((s + d) * kStepK, fa[d]);
          ob.template load<EDGE>((s + d) * kStepK, fb[d]);
        }
      for (; s + 2 * kDepth <= sw; s += kDepth) {
#pragma unroll
        for (int d = 0; d < kDepth; ++d) {
          multiply(fa[d], fb[d]);
          oa.template load<EDGE>((s + d + kDepth) * kStepK, fa[d]);
          ob.template load<EDGE>((s + d + kDepth) * kStepK, fb[d]);
        }
      }
      for (; s < sw; s += kDepth) {
#pragma unroll
        for (int d = 0; d < kDepth; ++d)
          if (s + d < sw) {
            multiply(fa[d], fb[d]);
            if (s + d + kDepth < sw) {
              oa.template load<EDGE>((s + d + kDepth) * kStepK, fa[d]);
              ob.template load<EDGE>((s + d + kDepth) * kStepK, fb[d]);
            }
          }
      }
    };
    if (edge) stream(std::integral_constant<bool, true>{});
    else stream(std::integral_constant<bool, false>{});
    for (int64_t s = sw; s < s1; ++s) {
      float fa[4][FM], fb[4][F];
      oa.load_guarded(s * kStepK, p.K, lane, fa);
      ob.load_guarded(s * kStepK, p.K, lane, fb);
      multiply(fa, fb);
    }
  }

  auto put4 = [&](int64_t m, int64_t n, float v0, float v1, float v2, float v3) {
    if (m >= p.M) return;
    if (n + 3 < p.N && (p.epi.ldc & 3) == 0) {
      epilogue4<false>(p.epi, m, n, v0, v1, v2, v3);
    } else {
      const float v[4] = {v0, v1, v2, v3};
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (n + e < p.N) epilogue1<false>(p.epi, m, n + e, v[e]);
    }
  };
  // acc[i][j][r]: row FM (lane%16) + i, column 4 F (lane/16) + F r + j of the wave tile
  const int c = lane & 15, q = lane >> 4;
  auto value = [&](int i, int col) { return acc[i][col % F][col / F]; };   // col: 0 .. 4F-1 of this lane's columns
  // Partial tiles meet in LDS, [slice][row][column], rows padded by 4 floats: the 16 rows that the 16-byte
  // stores of one instruction touch then start in 8 different bank groups of 8 banks.
  constexpr int kLd = T + 4;
  __shared__ __attribute__((aligned(16))) float part[kWK * TM * kLd];
  float* mine = part + wave * (TM * kLd);
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int g = 0; g < F; ++g)
      *reinterpret_cast<float4*>(mine + (FM * c + i) * kLd + 4 * F * q + 4 * g) =
          make_float4(value(i, 4 * g), value(i, 4 * g + 1), value(i, 4 * g + 2), value(i, 4 * g + 3));
  __syncthreads();
  for (int piece = threadIdx.x; piece < TM * T / 4; piece += 64 * kWK) {
    const int row = piece / (T / 4), col = piece % (T / 4) * 4;
    const float* src = part + row * kLd + col;
    float4 t = *reinterpret_cast<const float4*>(src);
#pragma unroll
    for (int k = 1; k < kWK; ++k) {
      const float4 u = *reinterpret_cast<const float4*>(src + k * (TM * kLd));
      t.x += u.x; t.y += u.y; t.z += u.z; t.w += u.w;
    }
    put4(m0 + row, n0 + col, t.x, t.y, t.z, t.w);
  }
}

template <int FM, int F>
hipError_t launch_tile(hipStream_t s, GemmF32Params p, bool ak, bool bk) {
  const int64_t tm = (p.M + 16 * FM - 1) / (16 * FM), tn = (p.N + 16 * F - 1) / (16 * F);
  if (tm * tn > (1LL << 30)) return hipErrorInvalidValue;
  p.tiles_m = (int)tm;
  p.tiles_n = (int)tn;
  const int grid = (int)(tm * tn), block = 64 * kWK;
  if (!ak && !bk) gemm_f32_kernel<FM, F, false, false><<<grid, block, 0, s>>>(p);
  else if (!ak) gemm_f32_kernel<FM, F, false, true><<<grid, block, 0, s>>>(p);
  else if (!bk) gemm_f32_kernel<FM, F, true, false><<<grid, block, 0, s>>>(p);
  else gemm_f32_kernel<FM, F, true, true><<<grid, block, 0, s>>>(p);
  return hipGetLastError();
}

}  // namespace

// 64 x 64 tiles, which read half as much per FLOP, once there is one of them for every compute unit (2048 x 512 x 1000:
// 23 us against 34 with 32 x 32; 1000 x 2048 x 512: 33 against 36); below that the smaller tiles occupy more of the
// chip (1000 x 512 x 2048, 128 tiles of 64 x 64: 30 us against 44).  8 or 16 slices
// of k instead of 4 measured the same or slower at every size.
// 16 x 32 tiles where those of 32 x 32 leave half the compute units without one: the serial chain of a wave is half as long and
// twice as many units take part (us per launch, median of a kernel trace, 32 x 32 / 16 x 32: 512 x 256 x 1024, 128 tiles of 32 x 32,
// 9.7 / 7.1; 64 x 256 x 1024, 16 tiles, 10.0 / 6.9; 256 x 256 x 512 k-major, 64, 6.6 / 5.6; 512 x 256 x 256, 128, 4.9 / 4.2; beyond 128
// tiles no gain: 300 x 448 x 704, 140, 7.9 / 9.0; 512 x 512 x 512, 256, 6.8 / 7.6).
// Not for up to four tiles and a short k: more workgroups end later than these few waves compute (32 x 32 x 64 2.8 / 3.3, x 256 4.1 /
// 4.1; 64 x 64 x 16 3.1 / 3.5, x 160 4.1 / 4.0; from five tiles on no difference is left: 160 x 32 x 16 3.5 / 3.5).
// Nor where both operands are k-major, their rows straddle cache lines (a piece of one k is 64 bytes of A and 128 of B, and then comes
// from two lines) and they are more than an XCD's L2 of 4 MiB holds: the lower tile fetches each line of B twice as often (32 x 32 /
// 16 x 32: 130 x 620 x 2048 18.3 / 28.0, 160 x 590 x 3072 27.3 / 40.2, 480 x 250 x 4096 47.4 / 53.3, 41 x 151 x 6144 43.6 / 54.7).  A long k or
// few tiles move that further out: 300 x 300 x 1024 11.2 / 9.8, x 1280 13.2 / 11.1, 16 x 1000 x 4096 36.4 / 27.6, 558 x 32 x 4096 29.8 / 27.0.
// Whole lines have no such limit (496 x 256 x 8192 87.7 / 37.0), nor has one k-major operand (480 x 250 x 8192 79.8 / 37.8).
static bool low_tiles(const GemmArgs& a, int64_t t32) {
  if (t32 > 128) return false;
  if (t32 <= 4 && a.K <= (t32 == 1 ? 256 : 160)) return false;
  const bool straddles = a.a_kmajor && a.b_kmajor &&
                         (((uintptr_t)a.A | (uint64_t)a.lda * 4) % 64 != 0 || ((uintptr_t)a.B | (uint64_t)a.ldb * 4) % 128 != 0);
  return !straddles || (a.M + a.N) * a.K < (1 << 20) || a.K * t32 < (a.K > 4096 ? 60000 : 140000);
}
hipError_t launch_gemm_f32(hipStream_t s, const GemmArgs& a, const EpiParams& epi) {
  const GemmF32Params p{(const float*)a.A, (const float*)a.B, a.M, a.N, a.K, a.lda, a.ldb, 0, 0, epi};
  const int64_t t64 = ((a.M + 63) / 64) * ((a.N + 63) / 64);
  const int64_t t32 = ((a.M + 31) / 32) * ((a.N + 31) / 32);
  if (t64 >= 256) return launch_tile<4, 4>(s, p, a.a_kmajor, a.b_kmajor);
  return low_tiles(a, t32) ? launch_tile<1, 2>(s, p, a.a_kmajor, a.b_kmajor) : launch_tile<2, 2>(s, p, a.a_kmajor, a.b_kmajor);
}

}  // namespace pw
