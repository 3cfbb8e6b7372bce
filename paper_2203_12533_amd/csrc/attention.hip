// Multi-head attention, forward and backward: causal or unmasked, queries and keys/values from separate
// arrays with their own row strides and lengths (MhaArgs).  One definition serves a decoder's causal
// self-attention over packed [Q|K|V] rows, an encoder's unmasked self-attention and a decoder's attention over
// the encoder output.
//
// Two families:
//  * fp32 kernels (here): every product on the fp32 matrix pipe.  They serve the fp32 configuration (small, latency
//    bound) and whatever the bf16 kernels do not cover.
//  * bf16 MFMA kernels with direct global->LDS loads (attention_dma.hip): every layout and mask, both head widths -
//    the ones that matter for throughput.
// Scores and probabilities never touch HBM in any family: the forward keeps a running (max, sum)
// per row and writes only O and the row log-sum-exp; the backward recomputes P from Q, K and that
// log-sum-exp.  All reductions run in a fixed order: results are the same bits on every run.
#include <cstdlib>
#include <type_traits>

#include "attention_common.hpp"
#include "common.hpp"
#include "kernels.hpp"

namespace pw {

bool mha_dma_supported(const MhaArgs& a);
bool mha_dma_outputs_aligned(const void* dq, int64_t lddq, const void* dk, const void* dv, int64_t lddkv);
hipError_t launch_mha_fwd_dma(hipStream_t s, const MhaArgs& a, void* o, void* o_lo, float* lse, bool split);
hipError_t launch_mha_dq_dkv_dma(hipStream_t s, const MhaArgs& a, const void* o, const void* o_lo, const void* dout,
                                 const float* lse, float* delta, void* dq, int64_t lddq, void* dk, void* dv, int64_t lddkv,
                                 bool split);

// ---- the fp32 matrix-core family -----------------------------------------------------------------------
// v_mfma_f32_16x16x4_f32: A lane l = row l%16, k-slot l/16; B lane l = column l%16, the same k-slot; D lane l = column
// l%16, rows 4 (l/16) + r.  With c = l%16, q = l/16:
//   first product (scores):   step st, MFMA i: k-slot q stands for feature 16 st + 4 q + i, so a row's fragment is
//                             HD/16 pieces of 4 consecutive features;  D register r = row 4 q + r of the tile;
//   second product:           MFMA r: k-slot q stands for tile row 4 q + r, which makes D register r of the first product
//                             its B operand as it is; A row c of block j stands for feature 4 c + j of a group of 64, so
//                             the tile is read in pieces of 4 consecutive features once more, and a lane ends up with the
//                             16 consecutive features 16 q .. of its column (per group of 64).
// Everything is fp32 (bf16 operands are widened exactly), as a thread-per-row kernel on the vector ALU has it.
//
// What bounds it: at the sizes of the fp32 configuration (128 positions) the length of one workgroup's serial work and
// how many workgroups there are.  A workgroup owns 16 queries (or keys) only and its four waves take every fourth tile of
// 16 keys (queries); their partial results meet in LDS and are combined in wave order.  Fragments come straight from
// global memory (the pipe's 256 FLOP/clk per compute unit needs 8 bytes per clock and wave), so there is no barrier
// before that.  Measured against one thread per row on the vector ALU (us): 4 x 128 positions, 4 heads of 64, fp32,
// causal: forward 108 -> 6.4, delta + dQ 17 + 108 -> 8.0, dK and dV 166 + 105 -> 8.8; bf16, 4 x 333 queries over 520 keys,
// 8 heads of 64, all together 2510 -> 116.
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef __bf16 bf16x4u __attribute__((ext_vector_type(4), aligned(2)));
template <class T> __device__ __forceinline__ f32x4 load4f(const T* p);   // no alignment beyond the element's
template <> __device__ __forceinline__ f32x4 load4f<float>(const float* p) { return *reinterpret_cast<const f32x4u*>(p); }
template <> __device__ __forceinline__ f32x4 load4f<bf16>(const bf16* p) {
  const bf16x4u v = *reinterpret_cast<const bf16x4u*>(p);
  return f32x4{(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
}
__device__ __forceinline__ void store4f(float* p, f32x4 v) { *reinterpret_cast<f32x4u*>(p) = v; }
__device__ __forceinline__ void store4f(bf16* p, f32x4 v) {
  bf16x4u o = {(bf16)v[0], (bf16)v[1], (bf16)v[2], (bf16)v[3]};
  *reinterpret_cast<bf16x4u*>(p) = o;
}

constexpr int kFT = 16;        // rows of a tile: queries (or keys) of a workgroup, keys (queries) of a step
constexpr int kFWaves = 4;

// What the kernels need of an MhaArgs, typed.
template <class T> struct RowArgs {
  const T *q, *k, *v;
  int64_t ldq, ldkv;
  int Tq, Tk, H;
};

// 16 rows of one operand: row0 .. row0+15 of a sequence whose last valid row is `last`; rows past it are fetched from
// that row (in bounds) and, where they would be summed over (column_pieces with EDGE), replaced by zeros.
template <class T, int HD> struct RowTile {
  const T* base;
  int64_t ld;
  int last;
  // fragments of a first product: this lane's row row0 + c
  __device__ __forceinline__ void row_pieces(int row0, int lane, f32x4 (&f)[HD / 16]) const {
    const T* p = base + (int64_t)min(row0 + (lane & 15), last) * ld + 4 * (lane >> 4);
#pragma unroll
    for (int st = 0; st < HD / 16; ++st) f[st] = load4f(p + 16 * st);
  }
  // fragments of a second product: rows row0 + 4 q + r, features 64 g + 4 c ..
  template <bool EDGE>
  __device__ __forceinline__ void column_pieces(int row0, int lane, f32x4 (&f)[HD / 64][4]) const {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = row0 + 4 * (lane >> 4) + r;
      const T* p = base + (int64_t)min(row, last) * ld + 4 * (lane & 15);
#pragma unroll
      for (int g = 0; g < HD / 64; ++g) {
        f[g][r] = load4f(p + 64 * g);
        if (EDGE && row > last) f[g][r] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    }
  }
};

template <int HD>
__device__ __forceinline__ f32x4 row_product(const f32x4 (&a)[HD / 16], const f32x4 (&b)[HD / 16]) {
  f32x4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int st = 0; st < HD / 16; ++st)
#pragma unroll
    for (int i = 0; i < 4; ++i) d = __builtin_amdgcn_mfma_f32_16x16x4f32(a[st][i], b[st][i], d, 0, 0, 0);
  return d;
}

// acc[4 g + j] += (tile columns)^T . w, w = D registers of a first product (row 4 q + r, this lane's column).  `seen`
// (only looked at with MASKED): bit r says whether row 4 q + r counts for this lane's column; where it does not, w is
// zero, and a non-finite value in the tile must not turn that zero into a NaN: such a tile - none, in ordinary use - is
// added up pair by pair on the vector ALU.
template <int HD, bool MASKED>
__device__ __forceinline__ void column_product(const f32x4 (&t)[HD / 64][4], f32x4 w, unsigned seen, int lane, f32x4 (&acc)[HD / 16]) {
  if (MASKED) {
    bool odd = false;
#pragma unroll
    for (int g = 0; g < HD / 64; ++g)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int j = 0; j < 4; ++j) odd |= !(fabsf(t[g][r][j]) < INFINITY);
    if (__builtin_amdgcn_ballot_w64(odd) != 0) {
      const int c = lane & 15, q = lane >> 4;
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll 1
        for (int from = 0; from < 64; from += 16) {             // row 4 (from / 16) + r: its w and its bit sit in lane
          const float wr = __shfl(w[r], from + c, 64);          // from + c, its feature 64 g + 16 q + 4 e + j in register
          const bool sr = __shfl((int)seen, from + c, 64) >> r & 1;   // t[g][r][j] of lane from + 4 q + e
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int g = 0; g < HD / 64; ++g)
#pragma unroll
              for (int j = 0; j < 4; ++j) {
                const float v = __shfl(t[g][r][j], from + 4 * q + e, 64);
                if (sr) acc[4 * g + j][e] = __builtin_fmaf(wr, v, acc[4 * g + j][e]);
              }
        }
      return;
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int g = 0; g < HD / 64; ++g)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[4 * g + j] = __builtin_amdgcn_mfma_f32_16x16x4f32(t[g][r][j], w[r], acc[4 * g + j], 0, 0, 0);
}

// Where a wave parks its result for the combination: 16 rows (its lanes' columns) of HD features.
template <int HD> constexpr int kPartLd = HD + 4;
template <int HD>
__device__ __forceinline__ void park(float* part, int wave, int lane, const f32x4 (&acc)[HD / 16]) {
  float* row = part + (wave * kFT + (lane & 15)) * kPartLd<HD> + 16 * (lane >> 4);
#pragma unroll
  for (int g = 0; g < HD / 64; ++g)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      *reinterpret_cast<f32x4*>(row + 64 * g + 4 * e) = f32x4{acc[4 * g][e], acc[4 * g + 1][e], acc[4 * g + 2][e], acc[4 * g + 3][e]};
}
// out rows (valid of them) = scale * sum over the waves, in wave order.  All threads call; the caller has synchronised.
template <class T, int HD>
__device__ __forceinline__ void store_sum(const float* part, T* out, int64_t ld, int valid, float scale) {
  for (int idx = threadIdx.x; idx < kFT * HD / 4; idx += 64 * kFWaves) {
    const int row = idx / (HD / 4), col = idx % (HD / 4) * 4;
    f32x4 v = *reinterpret_cast<const f32x4*>(part + row * kPartLd<HD> + col);
#pragma unroll
    for (int w = 1; w < kFWaves; ++w) v += *reinterpret_cast<const f32x4*>(part + (w * kFT + row) * kPartLd<HD> + col);
    if (row < valid) store4f(out + (int64_t)row * ld + col, v * scale);
  }
}

// ---- forward: workgroup = 16 queries of one (batch, head) ----------------------------------------------
template <class T, int HD, bool CAUSAL>
__global__ __launch_bounds__(64 * kFWaves) void attention_fwd_f32_kernel(RowArgs<T> a, T* __restrict__ o, T* __restrict__ o_lo,
                                                                         float* __restrict__ lse) {
  __shared__ __attribute__((aligned(16))) float part[kFWaves * kFT * kPartLd<HD>];
  __shared__ float ms[kFWaves][kFT], ls[kFWaves][kFT];
  const int Tq = a.Tq, Tk = a.Tk, H = a.H, d = H * HD, nq = (Tq + kFT - 1) / kFT;
  int bh, qi;
  xcd_block_map(blockIdx.x, gridDim.x, nq, CAUSAL ? causal_group(nq, 64) : 1, bh, qi);
  const int qblk = CAUSAL ? nq - 1 - qi : qi, b = bh / H, h = bh - b * H, q0 = qblk * kFT;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, c = lane & 15, quad = lane >> 4;
  const RowTile<T, HD> K{a.k + (int64_t)b * Tk * a.ldkv + h * HD, a.ldkv, Tk - 1}, V{a.v + (int64_t)b * Tk * a.ldkv + h * HD, a.ldkv, Tk - 1};
  const RowTile<T, HD> Q{a.q + (int64_t)b * Tq * a.ldq + h * HD, a.ldq, Tq - 1};
  const float c2 = kLog2e / sqrtf((float)HD);
  f32x4 qf[HD / 16], acc[HD / 16];
  Q.row_pieces(q0, lane, qf);
#pragma unroll
  for (int i = 0; i < HD / 16; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;
  auto tile = [&](int t, auto e) {
    constexpr bool EDGE = decltype(e)::value;
    f32x4 kf[HD / 16], vf[HD / 64][4];
    K.row_pieces(t * kFT, lane, kf);
    V.template column_pieces<EDGE>(t * kFT, lane, vf);
    f32x4 s = row_product<HD>(kf, qf);
    unsigned seen = 15u;
    if (EDGE) {
      seen = 0;
      const int visible = (CAUSAL ? q0 + c : Tk - 1) - t * kFT - 4 * quad;   // last visible row of this lane's four
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (r <= visible) seen |= 1u << r;
        else s[r] = -INFINITY;
      }
    }
    float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64)) * c2;
    const float m_new = fmaxf(m, mx), alpha = m == m_new ? 1.f : __builtin_amdgcn_exp2f(m - m_new);   // (both -inf: see ref)
    m = m_new;
    // A wave that has met nothing but scores of -inf so far holds zeros: exp2(-inf - (-inf)) would turn them into NaN.
    const float ref = m == -INFINITY ? 0.f : m;
    f32x4 p;
    float sum = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      p[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], c2, -ref));
      sum += p[r];
    }
    l = l * alpha + sum;
#pragma unroll
    for (int i = 0; i < HD / 16; ++i) acc[i] *= alpha;
    column_product<HD, EDGE>(vf, p, seen, lane, acc);
  };
  const int n_tiles = CAUSAL ? qblk + 1 : (Tk + kFT - 1) / kFT;
  const int whole = CAUSAL ? qblk : Tk / kFT;
  int t = wave;
  for (; t < whole; t += kFWaves) tile(t, std::integral_constant<bool, false>{});
  if (t < n_tiles) tile(t, std::integral_constant<bool, true>{});
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  park<HD>(part, wave, lane, acc);
  if (quad == 0) {
    ms[wave][c] = m;
    ls[wave][c] = l;
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < kFT * HD / 4; idx += 64 * kFWaves) {
    const int row = idx / (HD / 4), col = idx % (HD / 4) * 4, query = q0 + row;
    float top = ms[0][row];
#pragma unroll
    for (int w = 1; w < kFWaves; ++w) top = fmaxf(top, ms[w][row]);
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    float total = 0.f;
#pragma unroll
    for (int w = 0; w < kFWaves; ++w) {
      const float f = ms[w][row] == top ? 1.f : __builtin_amdgcn_exp2f(ms[w][row] - top);   // a wave without a tile: exp2(-inf) = 0
      total = __builtin_fmaf(ls[w][row], f, total);
      v += *reinterpret_cast<const f32x4*>(part + (w * kFT + row) * kPartLd<HD> + col) * f;
    }
    if (query < Tq) {
      v *= 1.f / total;
      const int64_t at = ((int64_t)b * Tq + query) * d + h * HD + col;
      store4f(o + at, v);
      if (o_lo) {   // what the rounding of O left over (zero in fp32)
        f32x4 left;
#pragma unroll
        for (int i = 0; i < 4; ++i) left[i] = v[i] - to_f32(from_f32<T>(v[i]));
        store4f(o_lo + at, left);
      }
      if (col == 0) lse[(int64_t)bh * Tq + query] = (top + __builtin_amdgcn_logf(total)) * kLn2;   // v_log_f32 is log2
    }
  }
}

// ---- backward ------------------------------------------------------------------------------------------
// dq_i = scale * sum_j p_ij (dO_i.v_j - delta_i) k_j; workgroup = 16 queries.  Also leaves delta_i = sum_c dO_ic O_ic
// (every wave has the dO fragments at hand) for the dK/dV kernel behind it.
template <class T, int HD, bool CAUSAL>
__global__ __launch_bounds__(64 * kFWaves) void attention_dq_f32_kernel(RowArgs<T> a, const T* __restrict__ o, const T* __restrict__ o_lo,
                                                                        const T* __restrict__ dout, const float* __restrict__ lse,
                                                                        float* __restrict__ delta, T* __restrict__ dq_out, int64_t lddq) {
  __shared__ __attribute__((aligned(16))) float part[kFWaves * kFT * kPartLd<HD>];
  const int Tq = a.Tq, Tk = a.Tk, H = a.H, d = H * HD, nq = (Tq + kFT - 1) / kFT;
  int bh, qi;
  xcd_block_map(blockIdx.x, gridDim.x, nq, CAUSAL ? causal_group(nq, 64) : 1, bh, qi);
  const int qblk = CAUSAL ? nq - 1 - qi : qi, b = bh / H, h = bh - b * H, q0 = qblk * kFT;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, c = lane & 15, quad = lane >> 4;
  const RowTile<T, HD> K{a.k + (int64_t)b * Tk * a.ldkv + h * HD, a.ldkv, Tk - 1}, V{a.v + (int64_t)b * Tk * a.ldkv + h * HD, a.ldkv, Tk - 1};
  const RowTile<T, HD> Q{a.q + (int64_t)b * Tq * a.ldq + h * HD, a.ldq, Tq - 1};
  const int64_t dense = (int64_t)b * Tq * d + h * HD;
  const float scale = 1.f / sqrtf((float)HD), c2 = kLog2e * scale;
  f32x4 qf[HD / 16], gf[HD / 16], acc[HD / 16];
  Q.row_pieces(q0, lane, qf);
  RowTile<T, HD>{dout + dense, d, Tq - 1}.row_pieces(q0, lane, gf);
  float dl = 0.f;
  {
    f32x4 of[HD / 16];
    RowTile<T, HD>{o + dense, d, Tq - 1}.row_pieces(q0, lane, of);
    if (o_lo) {
      f32x4 lf[HD / 16];
      RowTile<T, HD>{o_lo + dense, d, Tq - 1}.row_pieces(q0, lane, lf);
#pragma unroll
      for (int st = 0; st < HD / 16; ++st) of[st] += lf[st];
    }
    // The diagonal of O . dO^T, from the same instructions as dP: where a query sees one key only, O is V and dP - delta
    // comes out as the exact zero that it is.
    const f32x4 od = row_product<HD>(of, gf);
    dl = (c & 2) ? ((c & 1) ? od[3] : od[2]) : ((c & 1) ? od[1] : od[0]);
    dl = __shfl(dl, c + 16 * (c >> 2), 64);
  }
  const int query = q0 + c;
  const float lse2 = lse[(int64_t)bh * Tq + min(query, Tq - 1)] * kLog2e;
  if (wave == 0 && quad == 0 && query < Tq) delta[(int64_t)bh * Tq + query] = dl;
#pragma unroll
  for (int i = 0; i < HD / 16; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto tile = [&](int t, auto e) {
    constexpr bool EDGE = decltype(e)::value;
    f32x4 kf[HD / 16], vf[HD / 16], kc[HD / 64][4];
    K.row_pieces(t * kFT, lane, kf);
    V.row_pieces(t * kFT, lane, vf);
    K.template column_pieces<EDGE>(t * kFT, lane, kc);
    const f32x4 s = row_product<HD>(kf, qf), dp = row_product<HD>(vf, gf);
    const int visible = (CAUSAL ? query : Tk - 1) - t * kFT - 4 * quad;
    unsigned seen = 15u;
    if (EDGE) seen = visible >= 3 ? 15u : visible < 0 ? 0u : (2u << visible) - 1u;
    f32x4 ds;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      ds[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], c2, -lse2)) * (dp[r] - dl);
      if (EDGE && !(seen >> r & 1)) ds[r] = 0.f;
    }
    column_product<HD, EDGE>(kc, ds, seen, lane, acc);
  };
  const int n_tiles = CAUSAL ? qblk + 1 : (Tk + kFT - 1) / kFT;
  const int whole = CAUSAL ? qblk : Tk / kFT;
  int t = wave;
  for (; t < whole; t += kFWaves) tile(t, std::integral_constant<bool, false>{});
  if (t < n_tiles) tile(t, std::integral_constant<bool, true>{});
  park<HD>(part, wave, lane, acc);
  __syncthreads();
  store_sum<T, HD>(part, dq_out + ((int64_t)b * Tq + q0) * lddq + h * HD, lddq, Tq - q0, scale);
}

// dv_j = sum_i p_ij dO_i, dk_j = scale * sum_i p_ij (dO_i.v_j - delta_i) q_i; workgroup = 16 keys, tiles of 16 queries.
template <class T, int HD, bool CAUSAL>
__global__ __launch_bounds__(64 * kFWaves, 2) void attention_dkv_f32_kernel(RowArgs<T> a, const T* __restrict__ dout,
                                                                         const float* __restrict__ lse, const float* __restrict__ delta,
                                                                         T* __restrict__ dk_out, T* __restrict__ dv_out, int64_t lddkv) {
  __shared__ __attribute__((aligned(16))) float part[kFWaves * kFT * kPartLd<HD>];
  const int Tq = a.Tq, Tk = a.Tk, H = a.H, d = H * HD, nk = (Tk + kFT - 1) / kFT;
  int bh, kblk;                                              // causal: the first keys see the most queries, they come first
  xcd_block_map(blockIdx.x, gridDim.x, nk, CAUSAL ? causal_group(nk, 64) : 1, bh, kblk);
  const int b = bh / H, h = bh - b * H, k0 = kblk * kFT;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, c = lane & 15, quad = lane >> 4;
  const RowTile<T, HD> Q{a.q + (int64_t)b * Tq * a.ldq + h * HD, a.ldq, Tq - 1}, G{dout + (int64_t)b * Tq * d + h * HD, d, Tq - 1};
  const float scale = 1.f / sqrtf((float)HD), c2 = kLog2e * scale;
  const float* lse_bh = lse + (int64_t)bh * Tq;
  const float* delta_bh = delta + (int64_t)bh * Tq;
  f32x4 kf[HD / 16], vf[HD / 16], dk[HD / 16], dv[HD / 16];
  RowTile<T, HD>{a.k + (int64_t)b * Tk * a.ldkv + h * HD, a.ldkv, Tk - 1}.row_pieces(k0, lane, kf);
  RowTile<T, HD>{a.v + (int64_t)b * Tk * a.ldkv + h * HD, a.ldkv, Tk - 1}.row_pieces(k0, lane, vf);
#pragma unroll
  for (int i = 0; i < HD / 16; ++i) dk[i] = dv[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto tile = [&](int t, auto e) {
    constexpr bool EDGE = decltype(e)::value;
    const int i0 = t * kFT + 4 * quad;                       // this lane's four queries
    f32x4 qr[HD / 16], gr[HD / 16], cols[HD / 64][4], lq, dq;
    Q.row_pieces(t * kFT, lane, qr);
    G.row_pieces(t * kFT, lane, gr);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = min(i0 + r, Tq - 1);
      lq[r] = lse_bh[i] * kLog2e;
      dq[r] = delta_bh[i];
    }
    const f32x4 s = row_product<HD>(qr, kf), dp = row_product<HD>(gr, vf);
    unsigned seen = 15u;
    if (EDGE) {
      seen = 0;
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (i0 + r < Tq && (!CAUSAL || i0 + r >= k0 + c)) seen |= 1u << r;
    }
    f32x4 p, ds;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      p[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], c2, -lq[r]));
      ds[r] = p[r] * (dp[r] - dq[r]);
      if (EDGE && !(seen >> r & 1)) p[r] = ds[r] = 0.f;
    }
    G.template column_pieces<EDGE>(t * kFT, lane, cols);
    column_product<HD, EDGE>(cols, p, seen, lane, dv);
    Q.template column_pieces<EDGE>(t * kFT, lane, cols);
    column_product<HD, EDGE>(cols, ds, seen, lane, dk);
  };
  // The tiles that need a mask - on the diagonal (wave 0's first), past the last query - come after the others.
  const int n_tiles = (Tq + kFT - 1) / kFT, whole = Tq / kFT;
  const bool diagonal = CAUSAL && wave == 0;
  int t = (CAUSAL ? kblk : 0) + wave + (diagonal ? kFWaves : 0);
  for (; t < whole; t += kFWaves) tile(t, std::integral_constant<bool, false>{});
#pragma unroll 1
  for (int e = diagonal ? 0 : 1; e < 2; ++e)
    if (e == 0 || t < n_tiles) tile(e == 0 ? kblk : t, std::integral_constant<bool, true>{});
  park<HD>(part, wave, lane, dv);
  __syncthreads();
  store_sum<T, HD>(part, dv_out + ((int64_t)b * Tk + k0) * lddkv + h * HD, lddkv, Tk - k0, 1.f);
  __syncthreads();
  park<HD>(part, wave, lane, dk);
  __syncthreads();
  store_sum<T, HD>(part, dk_out + ((int64_t)b * Tk + k0) * lddkv + h * HD, lddkv, Tk - k0, scale);
}

template <class T> static RowArgs<T> row_args(const MhaArgs& a) {
  return RowArgs<T>{(const T*)a.q, (const T*)a.k, (const T*)a.v, a.ldq, a.ldkv, a.Tq, a.Tk, a.H};
}
static bool f32_grid(const MhaArgs& a, int T, int* grid) {
  const int64_t g = ((int64_t)T + kFT - 1) / kFT * a.B * a.H;
  *grid = (int)g;
  return g <= 0x7fffffff;
}

template <class T, int HD>
static hipError_t fwd_f32(hipStream_t s, const MhaArgs& a, void* o, void* o_lo, float* lse) {
  int grid;
  if (!f32_grid(a, a.Tq, &grid)) return hipErrorInvalidValue;
  if (a.causal) attention_fwd_f32_kernel<T, HD, true><<<grid, 64 * kFWaves, 0, s>>>(row_args<T>(a), (T*)o, (T*)o_lo, lse);
  else attention_fwd_f32_kernel<T, HD, false><<<grid, 64 * kFWaves, 0, s>>>(row_args<T>(a), (T*)o, (T*)o_lo, lse);
  return hipGetLastError();
}
template <class T, int HD, bool CAUSAL>
static hipError_t bwd_f32_masked(hipStream_t s, const MhaArgs& a, const void* o, const void* o_lo, const void* dout, const float* lse,
                                 float* delta, void* dq, int64_t lddq, void* dk, void* dv, int64_t lddkv) {
  int grid_q, grid_k;
  if (!f32_grid(a, a.Tq, &grid_q) || !f32_grid(a, a.Tk, &grid_k)) return hipErrorInvalidValue;
  const RowArgs<T> r = row_args<T>(a);
  attention_dq_f32_kernel<T, HD, CAUSAL><<<grid_q, 64 * kFWaves, 0, s>>>(r, (const T*)o, (const T*)o_lo, (const T*)dout, lse, delta, (T*)dq, lddq);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  attention_dkv_f32_kernel<T, HD, CAUSAL><<<grid_k, 64 * kFWaves, 0, s>>>(r, (const T*)dout, lse, delta, (T*)dk, (T*)dv, lddkv);
  return hipGetLastError();
}
template <class T, int HD>
static hipError_t bwd_f32(hipStream_t s, const MhaArgs& a, const void* o, const void* o_lo, const void* dout, const float* lse,
                          float* delta, void* dq, int64_t lddq, void* dk, void* dv, int64_t lddkv) {
  return a.causal ? bwd_f32_masked<T, HD, true>(s, a, o, o_lo, dout, lse, delta, dq, lddq, dk, dv, lddkv)
                  : bwd_f32_masked<T, HD, false>(s, a, o, o_lo, dout, lse, delta, dq, lddq, dk, dv, lddkv);
}

static bool mha_args_ok(const MhaArgs& a) {
  if (!a.q || !a.k || !a.v || a.B <= 0 || a.Tq <= 0 || a.Tk <= 0 || a.H <= 0) return false;
  if (a.hd != 64 && a.hd != 128) return false;
  if (a.dtype != kF32 && a.dtype != kBF16) return false;
  if ((int64_t)a.B * a.H > 65535) return false;
  if (a.ldq < (int64_t)a.H * a.hd || a.ldkv < (int64_t)a.H * a.hd) return false;
  if (a.causal && a.Tq != a.Tk) return false;
  return true;
}

// bf16 runs the kernels of attention_dma.hip unless PW_ATTN_DMA=0 (A/B switch for measurements).
static bool use_dma_kernels() {
  static int v = -1;
  if (v < 0) {
    const char* e = getenv("PW_ATTN_DMA");
    v = !(e && e[0] == '0');
  }
  return v != 0;
}

// Packed causal self-attention: at head_dim 64 the one form whose probabilities are rounded to bf16 for the second
// products (as at head_dim 128 throughout); the others split them.
static bool is_packed_causal(const MhaArgs& a) {
  const int64_t d = (int64_t)a.H * a.hd;
  const size_t es = a.dtype == kBF16 ? 2 : 4;
  return a.causal && a.ldq == 3 * d && a.ldkv == 3 * d && (const char*)a.k == (const char*)a.q + d * es &&
         (const char*)a.v == (const char*)a.q + 2 * d * es;
}

hipError_t launch_mha_fwd(hipStream_t s, const MhaArgs& a, void* o, void* o_lo, float* lse) {
  if (!mha_args_ok(a) || !o || !lse) return hipErrorInvalidValue;
  const bool packed = a.dtype == kBF16 && is_packed_causal(a);
  if (packed && (((uintptr_t)a.q | (uintptr_t)o) & 15)) return hipErrorInvalidValue;
  if (use_dma_kernels() && mha_dma_supported(a) && !(((uintptr_t)o | (uintptr_t)o_lo) & 15))
    return launch_mha_fwd_dma(s, a, o, o_lo, lse, a.hd == 64 && !packed);
  if (a.dtype == kF32) return a.hd == 64 ? fwd_f32<float, 64>(s, a, o, o_lo, lse) : fwd_f32<float, 128>(s, a, o, o_lo, lse);
  return a.hd == 64 ? fwd_f32<bf16, 64>(s, a, o, o_lo, lse) : fwd_f32<bf16, 128>(s, a, o, o_lo, lse);
}

hipError_t launch_mha_bwd(hipStream_t s, const MhaArgs& a, const void* o, const void* o_lo, const void* dout,
                          const float* lse, float* delta, void* dq, int64_t lddq, void* dk, void* dv, int64_t lddkv) {
  if (!mha_args_ok(a) || !o || !dout || !lse || !delta || !dq || !dk || !dv) return hipErrorInvalidValue;
  const int64_t d = (int64_t)a.H * a.hd;
  if (lddq < d || lddkv < d) return hipErrorInvalidValue;
  const size_t es = a.dtype == kBF16 ? 2 : 4;
  const bool packed_out = lddq == 3 * d && lddkv == 3 * d && (char*)dk == (char*)dq + d * es && (char*)dv == (char*)dq + 2 * d * es;
  const bool packed = a.dtype == kBF16 && is_packed_causal(a) && packed_out;
  const bool dma = use_dma_kernels() && mha_dma_supported(a) && !(((uintptr_t)o | (uintptr_t)o_lo | (uintptr_t)dout) & 15) &&
                   (a.hd == 128 || mha_dma_outputs_aligned(dq, lddq, dk, dv, lddkv));
  // (at head_dim 128 the direct-to-LDS kernels have always taken gradients on 8-byte boundaries)
  if (packed && !(dma && a.hd == 128) && (((uintptr_t)a.q | (uintptr_t)o | (uintptr_t)dout | (uintptr_t)dq) & 15)) return hipErrorInvalidValue;
  if (dma) return launch_mha_dq_dkv_dma(s, a, o, o_lo, dout, lse, delta, dq, lddq, dk, dv, lddkv, a.hd == 64 && !packed);
  if (a.dtype == kF32)
    return a.hd == 64 ? bwd_f32<float, 64>(s, a, o, o_lo, dout, lse, delta, dq, lddq, dk, dv, lddkv)
                      : bwd_f32<float, 128>(s, a, o, o_lo, dout, lse, delta, dq, lddq, dk, dv, lddkv);
  return a.hd == 64 ? bwd_f32<bf16, 64>(s, a, o, o_lo, dout, lse, delta, dq, lddq, dk, dv, lddkv)
                    : bwd_f32<bf16, 128>(s, a, o, o_lo, dout, lse, delta, dq, lddq, dk, dv, lddkv);
}

static MhaArgs packed_args(int dtype, const void* qkv, int B, int T, int H, int hd) {
  const int64_t d = (int64_t)H * hd;
  const size_t es = dtype == kBF16 ? 2 : 4;
  const char* base = (const char*)qkv;
  return MhaArgs{dtype, base, base + d * es, base + 2 * d * es, 3 * d, 3 * d, B, T, T, H, hd, 1};
}

hipError_t launch_attention_fwd(hipStream_t s, int dtype, const void* qkv, void* o, float* lse, int B, int T, int H,
                                int hd) {
  if (!qkv || (dtype != kF32 && dtype != kBF16)) return hipErrorInvalidValue;
  return launch_mha_fwd(s, packed_args(dtype, qkv, B, T, H, hd), o, nullptr, lse);
}

hipError_t launch_attention_bwd(hipStream_t s, int dtype, const void* qkv, const void* o, const void* dout,
                                const float* lse, float* delta, void* dqkv, int B, int T, int H, int hd) {
  if (!qkv || !dqkv || (dtype != kF32 && dtype != kBF16)) return hipErrorInvalidValue;
  const int64_t d = (int64_t)H * hd;
  const size_t es = dtype == kBF16 ? 2 : 4;
  char* g = (char*)dqkv;
  return launch_mha_bwd(s, packed_args(dtype, qkv, B, T, H, hd), o, nullptr, dout, lse, delta, g, 3 * d, g + d * es, g + 2 * d * es, 3 * d);
}

}  // namespace pw
