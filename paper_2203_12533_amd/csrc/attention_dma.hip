// bf16 MFMA attention (head_dim 64 and 128) with direct global->LDS loads and transposing LDS reads.
//
// Register layout of v_mfma_f32_32x32x16_bf16 (D = A.B): A lane l supplies row l%32, k-slots 8 (l/32) .. +7; B lane l
// column l%32, the same k-slots; D lane l holds column l%32, register r row 8 (r/4) + 4 (l/32) + r%4.  The softmax row sits
// on the D column, i.e. on the lane (forward, dQ: S^T = K . Q^T; dK/dV: S = Q . K^T), so row statistics are one value per
// lane; the A tile of the first product is read with permuted rows, perm = [0-3, 8-11, 4-7, 12-15] within every 16, so that
// register r of half h stands for tile row 16 (r/8) + 8 h + r%8 and P (or dS) is the second product's B operand as it is.
// No atomics: dQ is summed by the block that owns the queries, dK/dV by the block that owns the keys, S recomputed in both.
//
// How operands travel:
//  * every tile (K, V, or Q, dO) is brought into LDS once, in its natural [row][head_dim] layout, by
//    global_load_lds_dwordx4 (each wave instruction deposits 1 KiB; no staging registers, no LDS
//    store instructions), double-buffered so the next tile is in flight while one is consumed;
//  * the second product needs the tile as [feature][row]; instead of keeping a transposed copy it is read
//    with ds_read_b64_tr_b16 (lane L of each 16-lane group points at [k0 + L/4][c0 + 4*(L%4)], lane i
//    receives rows k0..k0+3 of feature c0 + i).
// LDS swizzle, one rule for both access patterns: chunk c (8 features = 16 bytes) of row r sits at
// position c ^ (((r & 3) << 2) | ((r >> 2) & 3)).  16 consecutive (or permuted-within-16) rows of one chunk
// then hit 16 distinct 16-byte bank groups, and the 4 rows touched by one transposing read fall into 4
// different 64-byte windows.  At head_dim 64 a row is half of the 256 bytes all banks hold and its parity picks the half:
// c ^ ((((r >> 1) & 1) << 2) | ((r >> 2) & 3)) does the same.
// SPLIT (head_dim 64, all but packed causal self-attention): these calls have always been computed in fp32.  The forward's
// probabilities enter the second product as three bf16 values, which together are the fp32 ones: O with its remainder o_lo is
// as close to 64 bits as the fp32 kernels bring it (2.5e-6 in the norm, what the storage of the pair rounds off; with two
// values 3.4e-6).  In the backward two values do, 2^-17 of P and dS left out: dQ, dK and dV are stored in 8 bits, and their
// errors against 64 bits are those of the fp32 kernels to four digits (1.66e-3), also where keys and values share a component
// 64 times their spread.  Measured (us, forward and backward): 4 x 333 queries over 520 keys, 8 heads: 116 on the fp32
// matrix pipe -> 37; 2 x 2014 over 1092, 9 heads: 132.  The forward's third value: 10.3 -> 11.2 of the first, 8 x 700, 16 heads 40 -> 45.
// Packed causal, 4 x 1000, 12 heads: 131 with tiles staged through registers and a transposed copy in LDS -> 65.
// PARTS = 2, for few blocks: a wave alone takes 1.2 to 1.5 us per step whatever else the chip does (products, softmax and
// barrier one behind the other), so a launch that leaves units idle, or whose causal mask gives one block twice the average,
// lasts as long as its longest chain of steps.  Blocks of 64 rows then, two waves to 32 of them that take the halves of every
// tile in turn and add up through LDS at the end: half the steps, in the same fp32 sums.  The first above, whose dK/dV have too many
// blocks for it: forward 16.9 -> 10.8, backward 29.8 -> 25.8; the causal one 19.1 -> 17.2, 49.5 -> 48.1.
// Rows past the end of a sequence are fetched from a block of zeros; every use of such a row is masked or multiplied by an
// exact zero (P = exp2(-inf)).
// Values that are not finite.  A masked pair enters the second products with a probability of zero, and zero times infinity
// is NaN; so is a split probability times infinity where a part of it is zero or negative.  With SPLIT these calls give
// what a sum over the visible pairs alone gives: rows that did not come out finite are summed once more, pair by pair, at
// the end (nothing in the loop).  Without it (head_dim 128, packed causal) a masked value that is not finite spoils rows of
// its tile.
// Queries, keys and values come with their own pointers, row strides and lengths (MhaDev), so one set of kernels
// serves the packed causal self-attention of a decoder, the unmasked self-attention of an encoder and attention
// of decoder queries over encoder keys; CAUSAL is a template parameter (it decides which tiles are visited).
#include <algorithm>
#include <type_traits>

#include "attention_common.hpp"
#include "common.hpp"
#include "kernels.hpp"

namespace pw {

namespace {

constexpr int kNT = 256;                 // 4 waves
typedef __attribute__((address_space(3))) void* lds_ptr;
typedef short short4v __attribute__((ext_vector_type(4)));

// q, k, v: element (batch 0, row 0, feature 0); rows ldq / ldkv elements apart; batch b starts at row b*Tq / b*Tk.
struct MhaDev {
  const bf16 *q, *k, *v;
  int64_t ldq, ldkv;
  int Tq, Tk, H;
};

template <int HD> __device__ __forceinline__ int swz(int r) {
  return HD == 128 ? ((r & 3) << 2) | ((r >> 2) & 3) : (((r >> 1) & 1) << 2) | ((r >> 2) & 3);
}

__device__ __forceinline__ void dma16(const bf16* g, uint32_t lds_off) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(g), "s"(lds_off) : "memory", "m0");
}

// 4 bytes per lane straight into LDS at lds_off + 4*lane (per-row statistics of a tile).
__device__ __forceinline__ void dma4(const float* g, uint32_t lds_off) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" : : "v"(g), "s"(lds_off) : "memory", "m0");
}

// Same with a wave-uniform base pointer in scalar registers and a 32-bit per-lane byte offset.
__device__ __forceinline__ void dma16_s(const bf16* base, uint32_t voff, uint32_t lds_off) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(voff), "s"(base), "s"(lds_off) : "memory", "m0");
}

// Direct loads of a ROWS x HD tile, instructions of 1 KiB (512 / HD rows), dealt to WAVES waves.  Lane l
// fetches chunk (l % (HD/8)) ^ swz<HD>(row) of row l / (HD/8) of an instruction's rows.
// TileOffsets holds this lane's byte offsets inside a tile whose first row is row 0 (they do not depend on the
// tile), so a tile that lies fully inside the sequence costs no vector arithmetic: base + rows*ld is scalar.
template <int HD> constexpr int kRowsPerInstr = 512 / HD;
template <int ROWS, int HD, int WAVES = 4>
struct TileOffsets {
  static constexpr int kPerWave = ROWS * HD / (512 * WAVES);
  uint32_t off[kPerWave];
  __device__ __forceinline__ void init(int64_t ld, int wave, int lane) {
#pragma unroll
    for (int j = 0; j < kPerWave; ++j) {
      const int r = (wave * kPerWave + j) * kRowsPerInstr<HD> + lane / (HD / 8);
      off[j] = (uint32_t)((r * ld + (((lane % (HD / 8)) ^ swz<HD>(r)) << 3)) * 2);
    }
  }
};
// src: element (row 0 of the sequence, feature 0); tile rows row0 .. row0+ROWS-1; rows past `last` read as zero (the slow
// path, only for the one tile that straddles the end of the sequence).
template <int ROWS, int HD, int WAVES>
__device__ __forceinline__ void issue_tile(const bf16* __restrict__ src, int64_t ld, int row0, int last,
                                           const TileOffsets<ROWS, HD, WAVES>& to, uint32_t lds_off, int wave, int lane) {
  constexpr int kPerWave = TileOffsets<ROWS, HD, WAVES>::kPerWave;
  if (row0 + ROWS - 1 <= last) {
    const bf16* base = src + (int64_t)row0 * ld;
#pragma unroll
    for (int j = 0; j < kPerWave; ++j) dma16_s(base, to.off[j], lds_off + (wave * kPerWave + j) * 1024);
  } else {
#pragma unroll
    for (int j = 0; j < kPerWave; ++j) {
      const int instr = wave * kPerWave + j;
      const int r = instr * kRowsPerInstr<HD> + lane / (HD / 8);
      const int c = (lane % (HD / 8)) ^ swz<HD>(r);
      const bf16* g = src + (int64_t)(row0 + r) * ld + c * 8;
      if (row0 + r > last) g = reinterpret_cast<const bf16*>(kZeroRow);
      dma16(g, lds_off + instr * 1024);
    }
  }
}

// A wave's own 32 rows of an operand that stays in registers (fragments as load_row_frags has them), by way of LDS: read from global
// memory row by row, 16 bytes per lane, an instruction touches 32 lines for 32 bytes of each (about 64 clocks; Q, dO and O of the dQ
// kernel at width 128 took 4.8 us in front of its loop), direct loads touch whole rows.  tile: 32 * HD elements of the wave's.
template <int HD>
__device__ __forceinline__ void stage_rows(const bf16* src, int64_t ld, int row0, int limit, uint32_t lds_off, int lane) {
  TileOffsets<32, HD, 1> to;
  to.init(ld, 0, lane);
  issue_tile(src, ld, row0, limit - 1, to, lds_off, 0, lane);
}
template <int HD>
__device__ __forceinline__ void staged_frags(const bf16* __restrict__ tile, bf16x8* frag) {
  const int lane = threadIdx.x & 63, row = lane & 31, t = (lane >> 5) ^ swz<HD>(row);
#pragma unroll
  for (int kk = 0; kk < HD / 16; ++kk) frag[kk] = *reinterpret_cast<const bf16x8*>(tile + row * HD + ((2 * kk) ^ t) * 8);
  arrived<HD>(frag);
}

// 32x32 block of a first product: A rows (permuted) from a swizzled natural LDS tile, B from register fragments.
// The A fragments are fetched kDepth MFMAs ahead of their use (left alone the compiler fetches each one right
// before the MFMA that needs it, and every MFMA of the chain then waits out a full LDS round trip).
template <int HD>
__device__ __forceinline__ f32x16 first_product(const bf16* __restrict__ tile, int row_base, const bf16x8* bfrag) {
  constexpr int kDepth = 3, KK = HD / 16;   // 2 and 4 measured the same
  const int lane = threadIdx.x & 63;
  const int row = row_base + perm_row(lane & 31);
  const int t = (lane >> 5) ^ swz<HD>(row);                 // chunk (2 kk + half) ^ swz = (2 kk) ^ t
  const bf16* a = tile + row * HD;
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  bf16x8 af[kDepth];
#pragma unroll
  for (int kk = 0; kk < kDepth; ++kk) af[kk] = *reinterpret_cast<const bf16x8*>(a + ((2 * kk) ^ t) * 8);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[kk % kDepth], bfrag[kk], acc, 0, 0, 0);
    if (kk + kDepth < KK) af[kk % kDepth] = *reinterpret_cast<const bf16x8*>(a + ((2 * (kk + kDepth)) ^ t) * 8);
    __builtin_amdgcn_sched_barrier(0);
  }
  return acc;
}

// The second operand of a second product: 8 probabilities (or dS) per lane as a sum of TERMS bf16 values.  Three, each the
// upper half of what the ones before left over, are the fp32 value itself; two, rounded, leave 2^-17 of it.
template <int TERMS> struct Frag { bf16x8 v[TERMS]; };
template <int TERMS>
__device__ __forceinline__ Frag<TERMS> pack_frag(const f32x16& v, int first) {
  Frag<TERMS> f;
  if constexpr (TERMS == 3) {
    union { uint32_t w[4]; bf16x8 v; } u[3];
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      float x = v[first + e], y = v[first + e + 1];
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        u[t].w[e / 2] = __builtin_amdgcn_perm(__float_as_uint(y), __float_as_uint(x), 0x07060302u);   // both upper halves
        x -= __uint_as_float(__float_as_uint(x) & 0xffff0000u);
        y -= __uint_as_float(__float_as_uint(y) & 0xffff0000u);
      }
    }
#pragma unroll
    for (int t = 0; t < 3; ++t) f.v[t] = u[t].v;
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float left = v[first + e];
#pragma unroll
      for (int t = 0; t < TERMS; ++t) {
        f.v[t][e] = (bf16)left;
        left -= (float)f.v[t][e];
      }
    }
  }
  return f;
}
template <int TERMS>
__device__ __forceinline__ void mfma_frag(const bf16x8& a, const Frag<TERMS>& b, f32x16& acc) {
#pragma unroll
  for (int t = TERMS - 1; t >= 0; --t) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b.v[t], acc, 0, 0, 0);   // smallest first
}

// acc[cb] += Tile^T[features cb*32 ..][rows row_base .. row_base+15] . frag, the tile read transposed.
template <int HD, int TERMS>
__device__ __forceinline__ void second_product(const bf16* __restrict__ tile, int row_base, const Frag<TERMS>& frag, f32x16* acc) {
  const int lane = threadIdx.x & 63;
  const int grp = lane >> 4, L = lane & 15;
  const int row0 = row_base + 8 * (grp >> 1) + (L >> 2);          // tile row this lane points at for t = 0
  const int f0 = 16 * (grp & 1) + 4 * (L & 3);                    // first of its 4 features inside a 32-feature block
#pragma unroll
  for (int cb = 0; cb < HD / 32; ++cb) {
    union { bf16x8 v; short4v h[2]; } u;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int row = row0 + 4 * t;
      const int chunk = (cb * 32 + f0) >> 3;
      const bf16* p = tile + row * HD + ((chunk ^ swz<HD>(row)) << 3) + (f0 & 7);
      u.h[t] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)p);
    }
    mfma_frag<TERMS>(u.v, frag, acc[cb]);
  }
}

// Sums over the visible pairs one by one, from global memory: slow and sparing of registers.
template <int HD>
__device__ __forceinline__ float row_dot(const bf16* __restrict__ a, const bf16* __restrict__ b) {
  float s = 0.f;
#pragma unroll 1
  for (int c = 0; c < HD; c += 8) {
    const bf16x8 x = *reinterpret_cast<const bf16x8*>(a + c), y = *reinterpret_cast<const bf16x8*>(b + c);
#pragma unroll
    for (int e = 0; e < 8; ++e) s = fmaf((float)x[e], (float)y[e], s);
  }
  return s;
}
template <int HD>
__device__ __forceinline__ void add_row(float w, const bf16* __restrict__ row, f32x16* acc) {
  const int half = (threadIdx.x & 63) >> 5;
#pragma unroll
  for (int q = 0; q < HD / 8; ++q) {         // this lane's features 8 q + 4 half .. + 3
    const bf16x4 t = *reinterpret_cast<const bf16x4*>(row + 8 * q + 4 * half);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[q / 4][4 * (q % 4) + e] = fmaf(w, (float)t[e], acc[q / 4][4 * (q % 4) + e]);
  }
}
// Whether one of this lane's sums is NaN or infinite (zero times it is NaN).
template <int HD> __device__ __forceinline__ bool not_finite(const f32x16* acc) {
  float t[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int cb = 0; cb < HD / 32; ++cb)
#pragma unroll
    for (int r = 0; r < 16; ++r) t[r & 3] = fmaf(acc[cb][r], 0.f, t[r & 3]);
  const float u = (t[0] + t[1]) + (t[2] + t[3]);
  return u != u;
}
template <int HD> __device__ __forceinline__ void clear(f32x16* acc) {
#pragma unroll
  for (int cb = 0; cb < HD / 32; ++cb)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[cb][r] = 0.f;
}
// Forward and dQ: acc = the sum of weight(key, q.k) x[key] over the keys that this lane's query sees.
template <int HD, bool CAUSAL, class Weight>
__device__ __forceinline__ void sum_again(const bf16* q, int64_t ldq, const bf16* k, const bf16* x, int64_t ldkv, int q0, int Tq, int Tk,
                                          Weight weight, f32x16* acc) {
  const int query = min(q0 + ((int)threadIdx.x & 31), Tq - 1);      // (rows past the end are not stored)
  const bf16* mine = q + query * ldq;
  clear<HD>(acc);
#pragma unroll 1
  for (int j = 0; j < (CAUSAL ? min(q0 + 32, Tk) : Tk); ++j)
    if (!CAUSAL || j <= query) add_row<HD>(weight(j, row_dot<HD>(mine, k + j * ldkv)), x + j * ldkv, acc);
}

__device__ __forceinline__ void wait_and_sync() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's share of the tile in flight has landed
  __builtin_amdgcn_s_barrier();                      // ... and so has everyone else's; the other stage is free again
  asm volatile("" ::: "memory");
}

// Where two waves hold partial sums of the same rows (PARTS = 2): the second one's go through LDS to the first.
// box: this lane's word of a [HD / 2][64] array that both waves of a pair share.
template <int HD>
__device__ __forceinline__ void put_acc(float* box, const f32x16* acc) {
#pragma unroll
  for (int cb = 0; cb < HD / 32; ++cb)
#pragma unroll
    for (int r = 0; r < 16; ++r) box[(cb * 16 + r) * 64] = acc[cb][r];
}
// acc of part 0 += acc of part 1; true in the waves that hold the result.  Called by the whole workgroup.
template <int HD>
__device__ __forceinline__ bool sum_parts(float* box, int part, f32x16* acc) {
  __syncthreads();
  if (part == 1) put_acc<HD>(box, acc);
  __syncthreads();
  if (part == 1) return false;
#pragma unroll
  for (int cb = 0; cb < HD / 32; ++cb)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[cb][r] += box[(cb * 16 + r) * 64];
  return true;
}

// Tile rows per wave and iteration in the forward and dQ kernels.
template <int HD, int PARTS> constexpr int kSubRows = HD == 128 && PARTS == 2 ? 32 : 64;

// ===================================================================================================
// forward: block = 128 queries of one (batch, head); wave = 32 queries; key/value tiles of 64
// ===================================================================================================
template <int HD, bool CAUSAL, bool SPLIT, int PARTS>
__global__ __launch_bounds__(kNT, 2) void attn_fwd_dma_kernel(MhaDev a, bf16* __restrict__ o, bf16* __restrict__ o_lo,
                                                              float* __restrict__ lse) {
  constexpr int kSub = kSubRows<HD, PARTS>, BKV = kSub * PARTS, kRows = 128 / PARTS, kTerms = SPLIT ? 3 : 1;
  constexpr int kTile = BKV * HD;                       // elements per K (or V) tile
  extern __shared__ __attribute__((aligned(1024))) bf16 smem[];         // [stage][K | V]
  const int Tq = a.Tq, Tk = a.Tk, H = a.H;
  const int d = H * HD;
  const int64_t ld = a.ldkv;
  const int nq = (Tq + kRows - 1) / kRows;
  int bh, qi;
  if (CAUSAL) causal_block_map<HD>(blockIdx.x, gridDim.x, nq, (int64_t)Tk * (2 * HD * 2), 64, bh, qi);
  else xcd_block_map(blockIdx.x, gridDim.x, nq, 1, bh, qi);
  const int b = bh / H, h = bh - b * H;
  const int qblk = CAUSAL ? nq - 1 - qi : qi;           // causal: longest blocks of a problem first
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, half = lane >> 5;
  const int part = PARTS == 1 ? 0 : wave >> 1;         // which kSub rows of every tile are this wave's
  const int q0 = qblk * kRows + (PARTS == 1 ? wave : wave & 1) * 32;
  const int query = q0 + (lane & 31);
  const bf16* qbase = a.q + (int64_t)b * Tq * a.ldq + h * HD;
  const bf16* kbase = a.k + (int64_t)b * Tk * ld + h * HD;
  const bf16* vbase = a.v + (int64_t)b * Tk * ld + h * HD;
  const float c2 = kLog2e / sqrtf((float)HD);
  const uint32_t smem_off = (uint32_t)(uintptr_t)(lds_ptr)smem;

  const int last_q = min(Tq, (qblk + 1) * kRows) - 1;
  const int n_tiles = CAUSAL ? last_q / BKV + 1 : (Tk + BKV - 1) / BKV;
  TileOffsets<BKV, HD> to;
  to.init(ld, wave, lane);
  auto issue = [&](int t) {
    const uint32_t st = smem_off + (uint32_t)(t & 1) * (2 * kTile * 2);
    issue_tile(kbase, ld, t * BKV, Tk - 1, to, st, wave, lane);
    issue_tile(vbase, ld, t * BKV, Tk - 1, to, st + kTile * 2, wave, lane);
  };
  // The queries pass through the stage of tile 1, which is asked for behind the first barrier.
  static_assert(4 * 32 <= 2 * BKV, "a stage holds 32 rows for each wave");
  constexpr int kMine = 2 * kTile, kTileLoads = 2 * TileOffsets<BKV, HD>::kPerWave;
  stage_rows<HD>(qbase, a.ldq, q0, Tq, smem_off + (kMine + wave * 32 * HD) * 2, lane);
  issue(0);
  f32x16 acc[HD / 32];
  clear<HD>(acc);
  float m = -INFINITY, l = 0.f;
  bf16x8 qf[HD / 16];
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kTileLoads) : "memory");
  staged_frags<HD>(smem + kMine + wave * 32 * HD, qf);
  for (int t = 0; t < n_tiles; ++t) {
    const int j0 = t * BKV + part * kSub;
    wait_and_sync();
    if (t + 1 < n_tiles) issue(t + 1);
    if (CAUSAL ? j0 > q0 + 31 : PARTS > 1 && j0 >= Tk) continue;   // no key of the tile is this wave's to see
    const bf16* Ks = smem + (t & 1) * (2 * kTile) + part * (kSub * HD);
    const bf16* Vs = Ks + kTile;
    f32x16 s[kSub / 32];
#pragma unroll
    for (int kb = 0; kb < kSub / 32; ++kb) s[kb] = first_product<HD>(Ks, kb * 32, qf);
    // last visible key of this lane's query: itself (causal), else the last key there is
    const int last_key = CAUSAL ? query : Tk - 1;
    if (CAUSAL ? j0 + kSub - 1 > q0 : j0 + kSub > Tk) {   // the tile straddles the diagonal / the end of the keys
#pragma unroll
      for (int kb = 0; kb < kSub / 32; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (j0 + kb * 32 + reg_row(r, half) > last_key) s[kb][r] = -INFINITY;
    }
    float mx = max3(s[0][0], s[0][1], s[0][2]);
#pragma unroll
    for (int r = 3; r < 15; r += 2) mx = max3(mx, s[0][r], s[0][r + 1]);
    if constexpr (kSub == 64) {
#pragma unroll
      for (int r = 0; r < 16; r += 2) mx = max3(mx, s[1][r], s[1][r + 1]);
    }
    mx = max3(mx, s[0][15], s[0][15]);
    const float other = __shfl_xor(mx, 32, 64);
    mx = max3(mx, other, other) * c2;
    // Lazy rescaling: the running reference m only has to bound the exponents, not equal the maximum.  It is moved (and the
    // accumulators rescaled) only when some row's maximum grew by more than 2^8; otherwise exp2(s - m) <= 256.
    if (__builtin_amdgcn_ballot_w64(mx > m + 8.f) != 0) {
      const float m_new = fmaxf(m, mx);
      const float alpha = m == m_new ? 1.f : __builtin_amdgcn_exp2f(m - m_new);   // (both -inf: see ref)
      m = m_new;
      l *= alpha;
#pragma unroll
      for (int cb = 0; cb < HD / 32; ++cb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[cb][r] *= alpha;
    }
    // A row that has met nothing but scores of -inf so far holds zeros, which the tiles (or the part) to come add to.
    const float ref = m == -INFINITY ? 0.f : m;
    float sum = 0.f;
#pragma unroll
    for (int kb = 0; kb < kSub / 32; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = __builtin_amdgcn_exp2f(fmaf(s[kb][r], c2, -ref));
        s[kb][r] = p;
        sum += p;
      }
    l += sum;
#pragma unroll
    for (int kb = 0; kb < kSub / 32; ++kb)
#pragma unroll
      for (int b2 = 0; b2 < 2; ++b2) second_product<HD, kTerms>(Vs, kb * 32 + b2 * 16, pack_frag<kTerms>(s[kb], b2 * 8), acc);
  }
  l += __shfl_xor(l, 32, 64);
  if constexpr (PARTS > 1) {   // the second part hands its reference, sum and accumulators over through LDS
    float* const box = reinterpret_cast<float*>(smem) + (wave & 1) * ((HD / 2 + 2) * 64) + lane;
    __syncthreads();
    if (part == 1) {
      put_acc<HD>(box, acc);
      box[(HD / 2) * 64] = m;
      box[(HD / 2 + 1) * 64] = l;
    }
    __syncthreads();
    if (part == 1) return;
    const float m1 = box[(HD / 2) * 64], top = fmaxf(m, m1);
    const float w0 = m == top ? 1.f : __builtin_amdgcn_exp2f(m - top), w1 = m1 == top ? 1.f : __builtin_amdgcn_exp2f(m1 - top);
    m = top;
    l = l * w0 + box[(HD / 2 + 1) * 64] * w1;
#pragma unroll
    for (int cb = 0; cb < HD / 32; ++cb)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[cb][r] = acc[cb][r] * w0 + box[(cb * 16 + r) * 64] * w1;
  }
  auto store = [&](const f32x16* sum) {
    if (query >= Tq) return;
    const int64_t row = ((int64_t)b * Tq + query) * d + h * HD;
    if (o_lo)
      store_row_split<HD>(o + row, o_lo + row, sum, 1.f / l);
    else
      store_row<HD>(o + row, sum, 1.f / l);
    if (half == 0) lse[(int64_t)bh * Tq + query] = (m + __builtin_amdgcn_logf(l)) * kLn2;
  };
  // (Where l is NaN a visible score was, and the row is what it has to be.)
  if (SPLIT && __builtin_amdgcn_ballot_w64(query < Tq && l == l && not_finite<HD>(acc)) != 0) {
    f32x16 again[HD / 32];
    sum_again<HD, CAUSAL>(qbase, a.ldq, kbase, vbase, ld, q0, Tq, Tk,
                          [&](int, float s) { return __builtin_amdgcn_exp2f(fmaf(s, c2, m == -INFINITY ? 0.f : -m)); }, again);
    store(again);
  } else {
    store(acc);
  }
}

// ===================================================================================================
// dQ: same tiling as the forward.  dQ_i = scale * sum_j dS_ij K_j, dS = P (dP - delta)
// ===================================================================================================
// It also produces delta_i = sum_c dO_ic O_ic for its queries (each wave has the dO fragments of its 32 rows in
// registers anyway; O, plus the optional rounding remainder o_lo, is read the same way once) and leaves it in
// `delta` for the dK/dV kernel, which is launched behind this one.
template <int HD, bool CAUSAL, bool SPLIT, int PARTS>
__global__ __launch_bounds__(kNT, 2) void attn_dq_dma_kernel(MhaDev a, const bf16* __restrict__ o, const bf16* __restrict__ o_lo,
                                                             const bf16* __restrict__ dout, const float* __restrict__ lse,
                                                             float* __restrict__ delta, bf16* __restrict__ dq, int64_t lddq) {
  constexpr int kSub = kSubRows<HD, PARTS>, BKV = kSub * PARTS, kRows = 128 / PARTS, kTerms = SPLIT ? 2 : 1;
  constexpr int kTile = BKV * HD;
  extern __shared__ __attribute__((aligned(1024))) bf16 smem[];
  const int Tq = a.Tq, Tk = a.Tk, H = a.H;
  const int d = H * HD;
  const int64_t ld = a.ldkv;
  const int nq = (Tq + kRows - 1) / kRows;
  int bh, qi;
  if (CAUSAL) causal_block_map<HD>(blockIdx.x, gridDim.x, nq, (int64_t)Tk * (2 * HD * 2), 64, bh, qi);
  else xcd_block_map(blockIdx.x, gridDim.x, nq, 1, bh, qi);
  const int b = bh / H, h = bh - b * H;
  const int qblk = CAUSAL ? nq - 1 - qi : qi;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, half = lane >> 5;
  const int part = PARTS == 1 ? 0 : wave >> 1;         // which kSub rows of every tile are this wave's
  const int q0 = qblk * kRows + (PARTS == 1 ? wave : wave & 1) * 32;
  const int query = q0 + (lane & 31);
  const bf16* qbase = a.q + (int64_t)b * Tq * a.ldq + h * HD;
  const bf16* kbase = a.k + (int64_t)b * Tk * ld + h * HD;
  const bf16* vbase = a.v + (int64_t)b * Tk * ld + h * HD;
  const float scale = 1.f / sqrtf((float)HD);
  const float c2 = kLog2e * scale;
  const uint32_t smem_off = (uint32_t)(uintptr_t)(lds_ptr)smem;

  const int last_q = min(Tq, (qblk + 1) * kRows) - 1;
  const int n_tiles = CAUSAL ? last_q / BKV + 1 : (Tk + BKV - 1) / BKV;
  const int last_key = CAUSAL ? query : Tk - 1;
  TileOffsets<BKV, HD> to;
  to.init(ld, wave, lane);
  auto issue = [&](int t) {
    const uint32_t st = smem_off + (uint32_t)(t & 1) * (2 * kTile * 2);
    issue_tile(kbase, ld, t * BKV, Tk - 1, to, st, wave, lane);
    issue_tile(vbase, ld, t * BKV, Tk - 1, to, st + kTile * 2, wave, lane);
  };
  const float lse_in = lse[(int64_t)bh * Tq + min(query, Tq - 1)];
  // O and dO come through both stages, Q through that of tile 1 behind O; tile 0 follows when no wave reads its dO any more.
  static_assert(4 * 32 <= 2 * BKV, "a stage holds 32 rows for each wave");
  constexpr int kTileLoads = 2 * TileOffsets<BKV, HD>::kPerWave;
  const int mine = wave * 32 * HD, mine1 = 2 * kTile + mine;
  stage_rows<HD>(o + (int64_t)b * Tq * d + h * HD, d, q0, Tq, smem_off + mine1 * 2, lane);
  stage_rows<HD>(dout + (int64_t)b * Tq * d + h * HD, d, q0, Tq, smem_off + mine * 2, lane);
  bf16x8 qf[HD / 16], gf[HD / 16];
  float dl;
  {
    f32x16 od;
    bf16x8 of[HD / 16], lf[HD / 16];
    if (o_lo) load_row_frags<HD>(o_lo + (int64_t)b * Tq * d + h * HD, d, q0, Tq, lf);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    staged_frags<HD>(smem + mine1, of);
    staged_frags<HD>(smem + mine, gf);
    stage_rows<HD>(qbase, a.ldq, q0, Tq, smem_off + mine1 * 2, lane);
    __builtin_amdgcn_s_barrier();
    issue(0);
    // The diagonal of O . dO^T, from the same instructions as dP: where a query sees one key only, O is V and dP - delta
    // comes out as the exact zero that it is.
#pragma unroll
    for (int r = 0; r < 16; ++r) od[r] = 0.f;
#pragma unroll
    for (int kk = 0; kk < HD / 16; ++kk) od = __builtin_amdgcn_mfma_f32_32x32x16_bf16(of[kk], gf[kk], od, 0, 0, 0);
    if (o_lo) {
#pragma unroll
      for (int kk = 0; kk < HD / 16; ++kk) od = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lf[kk], gf[kk], od, 0, 0, 0);
    }
    // register r of half h holds row 8 (r/4) + 4 h + r%4: this column's own row is i = lane % 32
    const int i = lane & 31, reg = 4 * (i >> 3) + (i & 3);
    dl = od[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) dl = reg == r ? od[r] : dl;
    dl = __shfl(dl, i + 32 * ((i >> 2) & 1), 64);
    if (half == 0 && part == 0 && query < Tq) delta[(int64_t)bh * Tq + query] = dl;
  }
  f32x16 acc[HD / 32];
  clear<HD>(acc);
  const float lse2 = query < Tq ? lse_in * kLog2e : INFINITY;   // +inf: P = 0 for rows past the end
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kTileLoads) : "memory");
  staged_frags<HD>(smem + mine1, qf);
  for (int t = 0; t < n_tiles; ++t) {
    const int j0 = t * BKV + part * kSub;
    wait_and_sync();
    if (t + 1 < n_tiles) issue(t + 1);
    if (CAUSAL ? j0 > q0 + 31 : PARTS > 1 && j0 >= Tk) continue;
    const bf16* Ks = smem + (t & 1) * (2 * kTile) + part * (kSub * HD);
    const bf16* Vs = Ks + kTile;
    const bool diag = CAUSAL ? j0 + kSub - 1 > q0 : j0 + kSub > Tk;
#pragma unroll
    for (int kb = 0; kb < kSub / 32; ++kb) {
      f32x16 s = first_product<HD>(Ks, kb * 32, qf);      // S^T
      f32x16 dp = first_product<HD>(Vs, kb * 32, gf);     // dP^T = V . dO^T
      if (diag) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (j0 + kb * 32 + reg_row(r, half) > last_key) s[r] = -INFINITY;
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c2, -lse2)) * (dp[r] - dl);
#pragma unroll
      for (int b2 = 0; b2 < 2; ++b2) second_product<HD, kTerms>(Ks, kb * 32 + b2 * 16, pack_frag<kTerms>(s, b2 * 8), acc);   // dQ^T += K^T . dS^T
    }
  }
  if constexpr (PARTS > 1)
    if (!sum_parts<HD>(reinterpret_cast<float*>(smem) + (wave & 1) * (HD / 2 * 64) + lane, part, acc)) return;
  bf16* const row = dq + ((int64_t)b * Tq + query) * lddq + h * HD;
  if (SPLIT && __builtin_amdgcn_ballot_w64(query < Tq && lse2 == lse2 && dl == dl && not_finite<HD>(acc)) != 0) {
    f32x16 again[HD / 32];
    sum_again<HD, CAUSAL>(qbase, a.ldq, kbase, kbase, ld, q0, Tq, Tk, [&](int j, float s) {
      const float dp = row_dot<HD>(dout + ((int64_t)b * Tq + min(query, Tq - 1)) * d + h * HD, vbase + j * ld);
      return __builtin_amdgcn_exp2f(fmaf(s, c2, -lse2)) * (dp - dl);
    }, again);
    if (query < Tq) store_row<HD>(row, again, scale);
  } else if (query < Tq) {
    store_row<HD>(row, acc, scale);
  }
}

// ===================================================================================================
// dK, dV: block = 128 keys of one (batch, head); wave = 32 keys; query tiles of 64 as two 32-query blocks.
// Software-pipelined: the four phases of a block - first products S and dP, softmax / dS arithmetic on the
// vector ALU, second products into dV and dK - no longer run one after the other.  At width 128 a wave has one SIMD to
// itself here (its two output accumulators, the K / V fragments and the scores leave no room for a second wave), so
// nothing else hides the latencies: the first products of block n+1 are issued between the vector instructions
// of block n (one score element per MFMA: about as many vector cycles as the MFMA occupies the matrix pipe), and
// the transposed LDS reads of the second products run two MFMAs ahead.  Three tiles are resident (ring of
// three stages): the first products of the next tile start while the second products of the current one still
// read theirs.
// At width 128 these are the launches of few key blocks (PARTS = 2) and those of a single tile of queries (PARTS = 1, no next tile);
// attn_dkv_pair_kernel below has the others.
// ===================================================================================================
struct DkvStats { float lq[16], dq[16]; };

// This lane's log-sum-exp (scaled for exp2) and delta of the 16 queries its score registers stand for (block hb of
// the tile).
// (Raw values: the scaling of the log-sum-exp is left to the user, so that the reads can be issued a phase early.)
__device__ __forceinline__ void load_stats(const float* Ls, const float* Ds, int hb, int half, DkvStats& st) {
#pragma unroll
  for (int g = 0; g < 2; ++g)
#pragma unroll
    for (int v4 = 0; v4 < 2; ++v4) {
      const int base = hb * 32 + 16 * g + 8 * half + 4 * v4;
      const float4 l = *reinterpret_cast<const float4*>(Ls + base);
      const float4 d = *reinterpret_cast<const float4*>(Ds + base);
      const int r = 8 * g + 4 * v4;
      st.lq[r] = l.x; st.lq[r + 1] = l.y; st.lq[r + 2] = l.z; st.lq[r + 3] = l.w;
      st.dq[r] = d.x; st.dq[r + 1] = d.y; st.dq[r + 2] = d.z; st.dq[r + 3] = d.w;
    }
}

// First products of block `next` (sn = S, dpn = dP against the tile rows rbn .. rbn+31 of Qn / Gn), with - when
// HAVE_CUR - the arithmetic of block `cur` between the MFMAs: s becomes P = exp2(S c2 - lse), ds = P (dP - delta).
// (Masked scores are handled through the statistics: a log-sum-exp of +inf makes P an exact zero.)
template <int HD, int TERMS, bool HAVE_NEXT, bool HAVE_CUR>
__device__ __forceinline__ void dkv_front(const bf16* __restrict__ Qn, const bf16* __restrict__ Gn, int rbn,
                                          const bf16x8* kf, const bf16x8* vf, f32x16& sn, f32x16& dpn, f32x16& s,
                                          f32x16& dp, const DkvStats& st, float c2, Frag<TERMS>* pf, Frag<TERMS>* dsf) {
  constexpr int kDepth = 3, KK = HD / 16, kElems = 16 / (2 * KK);   // score elements per MFMA
  const int lane = threadIdx.x & 63;
  const int row = rbn + perm_row(lane & 31);
  const int t = (lane >> 5) ^ swz<HD>(row);
  const bf16* aq = Qn + row * HD;
  const bf16* ag = Gn + row * HD;
  bf16x8 fq[kDepth], fg[kDepth];
  if (HAVE_NEXT) {
#pragma unroll
    for (int r = 0; r < 16; ++r) sn[r] = dpn[r] = 0.f;
#pragma unroll
    for (int kk = 0; kk < kDepth; ++kk) {
      fq[kk] = *reinterpret_cast<const bf16x8*>(aq + ((2 * kk) ^ t) * 8);
      fg[kk] = *reinterpret_cast<const bf16x8*>(ag + ((2 * kk) ^ t) * 8);
    }
  }
  auto element = [&](int r) {
    if (HAVE_CUR) {
      s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c2, -st.lq[r]));
      dp[r] = s[r] * (dp[r] - st.dq[r]);
    }
  };
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    if (HAVE_NEXT) {
      sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fq[kk % kDepth], kf[kk], sn, 0, 0, 0);
      if (kk + kDepth < KK) fq[kk % kDepth] = *reinterpret_cast<const bf16x8*>(aq + ((2 * (kk + kDepth)) ^ t) * 8);
    }
#pragma unroll
    for (int e = 0; e < kElems; ++e) element(2 * kk * kElems + e);
    __builtin_amdgcn_sched_barrier(0);
    if (HAVE_NEXT) {
      dpn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fg[kk % kDepth], vf[kk], dpn, 0, 0, 0);
      if (kk + kDepth < KK) fg[kk % kDepth] = *reinterpret_cast<const bf16x8*>(ag + ((2 * (kk + kDepth)) ^ t) * 8);
    }
#pragma unroll
    for (int e = 0; e < kElems; ++e) element((2 * kk + 1) * kElems + e);
    __builtin_amdgcn_sched_barrier(0);
  }
  if (HAVE_CUR) {
#pragma unroll
    for (int b2 = 0; b2 < 2; ++b2) {
      pf[b2] = pack_frag<TERMS>(s, b2 * 8);
      dsf[b2] = pack_frag<TERMS>(dp, b2 * 8);
    }
  }
}

// Second products of a block: dv += Gs^T . P and dk += Qs^T . dS over the 32 queries at tile rows rb .. rb+31,
// TERMS * HD / 8 MFMAs whose transposed operand reads run kAhead steps ahead.
template <int HD, int TERMS>
__device__ __forceinline__ void dkv_back(const bf16* __restrict__ Qs, const bf16* __restrict__ Gs, int rb, const Frag<TERMS>* pf,
                                         const Frag<TERMS>* dsf, f32x16* dk, f32x16* dv) {
  constexpr int kAhead = 2, kBlocks = HD / 32, kSteps = 4 * kBlocks;
  const int lane = threadIdx.x & 63;
  const int grp = lane >> 4, L = lane & 15;
  const int f0 = 16 * (grp & 1) + 4 * (L & 3);
  // step j: b2 = 16-query half of the block, mat (0: dO -> dV, 1: Q -> dK), cb = 32-feature block
  auto read = [&](int j) {
    const int b2 = j / (2 * kBlocks), mat = (j / kBlocks) & 1, cb = j % kBlocks;
    const bf16* tile = mat ? Qs : Gs;
    const int row0 = rb + b2 * 16 + 8 * (grp >> 1) + (L >> 2);
    union { bf16x8 v; short4v h[2]; } u;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int row = row0 + 4 * t;
      const int chunk = (cb * 32 + f0) >> 3;
      const bf16* p = tile + row * HD + ((chunk ^ swz<HD>(row)) << 3) + (f0 & 7);
      u.h[t] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)p);
    }
    return u.v;
  };
  bf16x8 fr[kAhead + 1];
#pragma unroll
  for (int j = 0; j < kAhead; ++j) fr[j] = read(j);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int j = 0; j < kSteps; ++j) {
    if (j + kAhead < kSteps) fr[(j + kAhead) % (kAhead + 1)] = read(j + kAhead);
    const int b2 = j / (2 * kBlocks), mat = (j / kBlocks) & 1, cb = j % kBlocks;
    mfma_frag<TERMS>(fr[j % (kAhead + 1)], mat ? dsf[b2] : pf[b2], mat ? dk[cb] : dv[cb]);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// A wave's 32 keys over again (see the head of the file).
template <int HD, bool CAUSAL>
__device__ __forceinline__ void dkv_again(const MhaDev& a, const bf16* dout, const float* lse, const float* delta, bf16* dk_out, bf16* dv_out,
                                          int64_t lddkv, int bh, int k0) {
  const int T = a.Tq, Tk = a.Tk, H = a.H, b = bh / H, h = bh - b * H, d = H * HD;
  int key = k0 + ((int)threadIdx.x & 31);
  asm volatile("" : "+v"(key));                // nothing of this is worked out before the loop and kept in registers over it
  const bf16* q = a.q + (int64_t)b * T * a.ldq + h * HD;
  const bf16* g = dout + (int64_t)b * T * d + h * HD;
  const int64_t mine = ((int64_t)b * Tk + min(key, Tk - 1)) * a.ldkv + h * HD, row = ((int64_t)b * Tk + key) * lddkv + h * HD;
  const float scale = 1.f / sqrtf((float)HD), c2 = kLog2e * scale;
  lse += (int64_t)bh * T;
  delta += (int64_t)bh * T;
#pragma unroll 1
  for (int which = 0; which < 2; ++which) {    // dV, then dK
    f32x16 sum[HD / 32];
    clear<HD>(sum);
#pragma unroll 1
    for (int i = CAUSAL ? k0 : 0; i < T; ++i)
      if (!CAUSAL || i >= key) {
        const bf16 *qi = q + i * a.ldq, *gi = g + (int64_t)i * d;
        float w = __builtin_amdgcn_exp2f(fmaf(row_dot<HD>(qi, a.k + mine), c2, -lse[i] * kLog2e));
        if (which) w *= row_dot<HD>(gi, a.v + mine) - delta[i];
        add_row<HD>(w, which ? qi : gi, sum);
      }
    if (key < Tk) store_row<HD>((which ? dk_out : dv_out) + row, sum, which ? scale : 1.f);
  }
}

// ALONE: a compute unit has one workgroup at most, so a wave may have 512 registers.  In 256, which two workgroups need, head width 64
// spills (6 to 25 registers, unmasked 60): reloads in the loop, and each waits for the tiles in flight as well.  A few spills cost less than
// the wider form's moves between the two register files; bwd_dma has the figures.
template <int HD, bool CAUSAL, bool SPLIT, int PARTS, bool ALONE>
__global__ __launch_bounds__(kNT, ALONE ? 1 : 2) void attn_dkv_dma_kernel(MhaDev a, const bf16* __restrict__ dout,
                                                            const float* __restrict__ lse, const float* __restrict__ delta,
                                                            bf16* __restrict__ dk_out, bf16* __restrict__ dv_out, int64_t lddkv) {
  constexpr int BQ = 64, kStages = 3, kRows = 128 / PARTS, kTerms = SPLIT ? 2 : 1;
  constexpr int kTile = BQ * HD;
  extern __shared__ __attribute__((aligned(1024))) bf16 smem[];          // [stage][Q | dO], then the statistics
  float (*Ls)[BQ] = reinterpret_cast<float (*)[BQ]>(smem + kStages * 2 * kTile);
  float (*Ds)[BQ] = Ls + kStages;
  const int T = a.Tq, Tk = a.Tk, H = a.H;
  const int d = H * HD;
  const int64_t ld = a.ldq;
  int bh, kblk;                                         // causal: first key blocks see the most queries, they come first
  const int nk = (Tk + kRows - 1) / kRows;
  if (CAUSAL) causal_block_map<HD>(blockIdx.x, gridDim.x, nk, (int64_t)T * (2 * HD * 2), 32, bh, kblk);
  else xcd_block_map(blockIdx.x, gridDim.x, nk, 1, bh, kblk);
  const int b = bh / H, h = bh - b * H;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, half = lane >> 5;
  const int part = PARTS == 1 ? 0 : wave >> 1;          // which 32 rows of every tile are this wave's (PARTS = 1: all 64)
  const int k0 = kblk * kRows + (PARTS == 1 ? wave : wave & 1) * 32;
  const int key = k0 + (lane & 31);
  const bf16* qbase = a.q + (int64_t)b * T * ld + h * HD;
  const bf16* gbase = dout + (int64_t)b * T * d + h * HD;
  const float scale = 1.f / sqrtf((float)HD);
  const float c2 = kLog2e * scale;
  const uint32_t smem_off = (uint32_t)(uintptr_t)(lds_ptr)smem;

  TileOffsets<BQ, HD> to_q, to_g;
  to_q.init(ld, wave, lane);
  to_g.init(d, wave, lane);
  bf16x8 kf[HD / 16], vf[HD / 16];
  load_row_frags<HD>(a.k + (int64_t)b * Tk * a.ldkv + h * HD, a.ldkv, k0, Tk, kf);
  load_row_frags<HD>(a.v + (int64_t)b * Tk * a.ldkv + h * HD, a.ldkv, k0, Tk, vf);
  f32x16 dk[HD / 32], dv[HD / 32];
#pragma unroll
  for (int cb = 0; cb < HD / 32; ++cb)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      dk[cb][r] = 0.f;
      dv[cb][r] = 0.f;
    }

  const int first_tile = CAUSAL ? (kblk * kRows) / BQ : 0;
  const int n_tiles = (T + BQ - 1) / BQ;
  // A tile = 64 rows of Q and of dO plus the 64 queries' log-sum-exp and delta; all of it travels global -> LDS
  // directly (no destination registers: the compiler then has no pending load to wait for in the middle of the
  // pipeline, and the loads stay in flight until the explicit wait in front of the tile's barrier).  Statistics of
  // rows past the end are fetched from the last row and masked where they are used.
  const float* lse_bh = lse + (int64_t)bh * T;
  const float* delta_bh = delta + (int64_t)bh * T;
  const uint32_t stats_off = smem_off + kStages * 2 * kTile * 2;
  auto issue = [&](int t) {
    const uint32_t st = smem_off + (uint32_t)(t % kStages) * (2 * kTile * 2);
    issue_tile(qbase, ld, t * BQ, T - 1, to_q, st, wave, lane);
    issue_tile(gbase, d, t * BQ, T - 1, to_g, st + kTile * 2, wave, lane);
    if (wave == 0) {
      const int i = min(t * BQ + lane, T - 1);
      dma4(lse_bh + i, stats_off + (uint32_t)(t % kStages) * (BQ * 4));
      dma4(delta_bh + i, stats_off + (uint32_t)(kStages + t % kStages) * (BQ * 4));
    }
  };
  // Block n = 2 t + hb covers queries 32 n .. 32 n + 31.  Under the causal mask this wave's keys see the blocks from
  // k0 / 32 on; it starts with the tile that holds that block (waves 2 and 3 of a workgroup one tile after waves 0
  // and 1) and from there on runs every block - an odd first block's even neighbour is computed fully masked, which
  // keeps the pipeline below free of per-wave branches.
  // Without the sums over again (SPLIT) what that neighbour holds must not matter either: it is read as zeros.
  constexpr bool kHides = HD == 64 && CAUSAL && !SPLIT;
  constexpr int kZeros = kStages * 2 * kTile + 2 * kStages * BQ * 2;                // behind the statistics
  auto tile_q = [&](int n) { return smem + (kHides && 32 * n + 31 < k0 ? kZeros : ((n >> 1) % kStages) * (2 * kTile)); };
  auto first_stats = [&](int n, DkvStats& st) {
    load_stats(Ls[(n >> 1) % kStages], Ds[(n >> 1) % kStages], n & 1, half, st);
    if (kHides && 32 * n + 31 < k0) {                    // (every such wave writes the zeros for itself)
#pragma unroll
      for (int i = 0; i < 32 * HD / 512; ++i)
#pragma unroll
        for (int t = 0; t < 2; ++t) reinterpret_cast<uint4*>(smem + kZeros + t * kTile)[64 * i + lane] = make_uint4(0, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 16; ++r) st.dq[r] = 0.f;
    }
  };
  // What happens between the two blocks of tile t: tile t + 1 has to have landed, for every wave; behind the barrier
  // nobody reads tile t - 1 any more, so its stage takes tile t + 2.
  auto advance = [&](int t) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (t + 2 < n_tiles) issue(t + 2);
  };

  issue(first_tile);
  if (first_tile + 1 < n_tiles) {
    issue(first_tile + 1);
    // all but the second tile: its direct loads per wave, two more (the statistics) in wave 0
    constexpr int kLoads = 2 * TileOffsets<BQ, HD>::kPerWave;
    if (wave == 0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kLoads + 2) : "memory");
    else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kLoads) : "memory");
  } else {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");

  // Two sets of score registers: the even block of a tile lives in (s0, dp0), the odd one in (s1, dp1), so nothing is
  // ever copied from "next" to "current".
  f32x16 s0, dp0, s1, dp1;
  Frag<kTerms> pf[2], dsf[2];
  DkvStats st;
  // One step of the pipeline: the arithmetic of block n (scores in s, dp) between the first products of block n + 1
  // (into sn, dpn; NEXT: there is one), then the second products of block n.
  // The block behind block n of this wave is n + 1, or, where the other part has that one, n + 2.
  auto step = [&](int n, auto next, f32x16& s, f32x16& dp, f32x16& sn, f32x16& dpn) {
    constexpr bool NEXT = decltype(next)::value;
    const int hb = n & 1, nn = n + PARTS;
    const bf16* Qs = tile_q(n);
    const bf16* Qn = smem + ((nn >> 1) % kStages) * (2 * kTile);      // (a hidden block is a wave's first)
    // st holds the block's raw statistics, read from LDS during the previous step
#pragma unroll
    for (int r = 0; r < 16; ++r) st.lq[r] *= kLog2e;
    const int ib = 32 * n;
    // (The empty volatile statements tie the values to the rare branches below: without them the compiler turns the
    // two fix-ups into selects that every block pays for - some 130 vector instructions with their wait states.)
    if (CAUSAL && ib < k0 + 31) {        // a block on (or before) the diagonal: register r stands for query ib + reg_row(r, half)
      const int thr = key - ib - 8 * half;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if (16 * (r >> 3) + (r & 7) < thr) st.lq[r] = INFINITY;     // the key may not see this earlier query: P = 0
        asm volatile("" : "+v"(st.lq[r]));
      }
    }
    if (ib + 31 >= T) {                  // the block straddles the end of the queries
      const int thr = T - ib - 8 * half;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if (16 * (r >> 3) + (r & 7) >= thr) st.lq[r] = INFINITY;    // no such query: P = 0
        asm volatile("" : "+v"(st.lq[r]));
      }
    }
    dkv_front<HD, kTerms, NEXT, true>(Qn, Qn + kTile, (nn & 1) * 32, kf, vf, sn, dpn, s, dp, st, c2, pf, dsf);
    // the next block's statistics travel to registers under the second products (its tile is resident: see advance)
    if (NEXT) load_stats(Ls[(nn >> 1) % kStages], Ds[(nn >> 1) % kStages], nn & 1, half, st);
    dkv_back<HD, kTerms>(Qs, Qs + kTile, hb * 32, pf, dsf, dk, dv);
    // Register classes: the output accumulators and the K / V fragments are only ever touched by MFMAs and live in
    // the accumulation registers; the scores are worked on by the vector ALU and stay in ordinary registers, so no
    // MFMA result has to be copied across (with the wait states that costs).
#pragma unroll
    for (int cb = 0; cb < HD / 32; ++cb)
      if (HD == 128) asm volatile("" : "+a"(dk[cb]), "+a"(dv[cb]));
#pragma unroll
    for (int kk = 0; kk < HD / 16; ++kk)
      if (HD == 128) asm volatile("" : "+v"(kf[kk]), "+v"(vf[kk]));
  };
  using yes = std::integral_constant<bool, true>;
  using no = std::integral_constant<bool, false>;
  if constexpr (PARTS == 1) {
    int t0 = first_tile;
    bool any = true;
    if (CAUSAL && wave >= 2) {             // this wave's first tile is the next one
      any = first_tile + 1 < n_tiles;
      if (any) advance(first_tile);
      t0 = first_tile + 1;
    }
    if (any) {
      first_stats(2 * t0, st);
      dkv_front<HD, kTerms, true, false>(tile_q(2 * t0), tile_q(2 * t0) + kTile, 0, kf, vf, s0, dp0, s0, dp0, st, c2, pf, dsf);
      for (int t = t0; t + 1 < n_tiles; ++t) {
        step(2 * t, yes{}, s0, dp0, s1, dp1);
        advance(t);
        step(2 * t + 1, yes{}, s1, dp1, s0, dp0);
      }
      step(2 * (n_tiles - 1), yes{}, s0, dp0, s1, dp1);
      step(2 * (n_tiles - 1) + 1, no{}, s1, dp1, s0, dp0);
    }
  } else {
    // One block per tile and wave, the next one in the next tile: every step is led by the wait for it.
    first_stats(2 * first_tile + part, st);
    dkv_front<HD, kTerms, true, false>(tile_q(2 * first_tile + part), tile_q(2 * first_tile + part) + kTile, part * 32, kf, vf, s0, dp0, s0, dp0, st, c2, pf, dsf);
    int t = first_tile;
    for (; t + 2 < n_tiles; t += 2) {
      advance(t);
      step(2 * t + part, yes{}, s0, dp0, s1, dp1);
      advance(t + 1);
      step(2 * t + 2 + part, yes{}, s1, dp1, s0, dp0);
    }
    if (t + 1 < n_tiles) {
      advance(t);
      step(2 * t + part, yes{}, s0, dp0, s1, dp1);
      step(2 * t + 2 + part, no{}, s1, dp1, s0, dp0);
    } else {
      step(2 * t + part, no{}, s0, dp0, s1, dp1);
    }
    float* const box = reinterpret_cast<float*>(smem) + (wave & 1) * (HD / 2 * 64) + lane;
    (void)sum_parts<HD>(box, part, dk);
    if (!sum_parts<HD>(box, part, dv)) return;
  }
  if (SPLIT && __builtin_amdgcn_ballot_w64(key < Tk && (not_finite<HD>(dk) || not_finite<HD>(dv))) != 0) {
    dkv_again<HD, CAUSAL>(a, dout, lse, delta, dk_out, dv_out, lddkv, bh, k0);
    return;
  }
  if (key < Tk) {
    const int64_t row = ((int64_t)b * Tk + key) * lddkv + h * HD;
    store_row<HD>(dk_out + row, dk, scale);
    store_row<HD>(dv_out + row, dv, 1.f);
  }
}

// ===================================================================================================
// dK, dV for more than 128 blocks of 128 keys, at head_dim 128 and, unmasked, at 64 (but for a single tile of queries: bwd_dma): 8 waves,
// two to a SIMD, each pair with the same 32 keys; of every tile of 64 queries one wave takes the first 32, the other the rest, and
// their sums meet in LDS at the end (in a fixed order).
// What bounds the kernel above is that a SIMD has one wave: products, exponentials and LDS round trips of a block follow one
// another (3200 clocks for 1024 of matrix work).  A second wave needs each of them within 256 registers: K and V stay in LDS
// next to a ring of two tiles (129 KiB, one workgroup per compute unit) instead of in 64 registers, the addresses of LDS
// reads are worked out from one register each, the statistics come in under the last first products.  Half as many
// LDS bytes again per block is the price; two roles per pair (P and dV | dP, dS and dK over 64 keys each, P handed over through LDS:
// half the reads), halves of a pair one phase apart, and V in registers were all slower or the same, wave priorities no different.
// What bounds it: no unit is full (causal 8 x 1024, 16 heads, counters: matrix pipe 28 % of the time, before 24 %; LDS reads 28 %, no
// conflicts; vector issue 31 % of a SIMD); a wave waits on counters 37 % and to issue 32 % of its time, the barrier per tile keeps both
// waves of a SIMD in the same phase.  At width 64 (65 KiB, 175 registers; 4 x 333 over 520, 8 heads) the matrix pipe is busy 10 % and a wave
// waits on counters 38 %: six tiles between a prologue and the meeting of the sums.
// Measured (us, this kernel alone, kernel traces, before / now): in train steps causal 8 x 1024, 16 heads 123 / 101, 2 x 1024, 32 heads
// 97.8 / 79.2, unmasked 8 x 1024, 16 heads 179 / 153; by itself causal 2 x 1024, 16 heads 41.0 / 33.2, 16 x 128, 16 heads 16.4 / 14.6.
// Forward and backward: causal 4 x 1000, 8 heads 89.1 / 84.3; 8 x 300, 12 heads 59.8 / 58.1; 4 x 333 queries over 520 keys, 16 heads
// 80.7 / 76.9.  The dispatch (bwd_dma) has both limits' figures.
// ===================================================================================================
constexpr int kPairWaves = 8, kPairBQ = 64;
template <int HD> constexpr int kSmemPair = (2 * 128 * HD + 2 * 2 * kPairBQ * HD) * 2 + 2 * 2 * kPairBQ * 4;
template <int HD, bool CAUSAL, bool SPLIT>
__global__ __launch_bounds__(64 * kPairWaves, 2) void attn_dkv_pair_kernel(MhaDev a, const bf16* __restrict__ dout,
                                                                           const float* __restrict__ lse, const float* __restrict__ delta,
                                                                           bf16* __restrict__ dk_out, bf16* __restrict__ dv_out, int64_t lddkv) {
  constexpr int KK = HD / 16, kRows = 128, kDepth = 2, kPairTile = kPairBQ * HD, kTerms = SPLIT ? 2 : 1;
  extern __shared__ __attribute__((aligned(1024))) bf16 smem[];          // K | V | [stage][Q | dO] | statistics
  bf16* const ring = smem + 2 * kRows * HD;
  float (*Ls)[kPairBQ] = reinterpret_cast<float (*)[kPairBQ]>(ring + 2 * 2 * kPairTile);
  float (*Ds)[kPairBQ] = Ls + 2;
  const int T = a.Tq, Tk = a.Tk, H = a.H, d = H * HD;
  const int64_t ld = a.ldq;
  int bh, kblk;
  const int nk = (Tk + kRows - 1) / kRows;
  if (CAUSAL) causal_block_map<HD>(blockIdx.x, gridDim.x, nk, (int64_t)T * (2 * HD * 2), 32, bh, kblk);
  else xcd_block_map(blockIdx.x, gridDim.x, nk, 1, bh, kblk);
  const int b = bh / H, h = bh - b * H;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, half = lane >> 5;
  const int part = wave >> 2, kw = (wave & 3) * 32;
  const int k0 = kblk * kRows + kw, key = k0 + (lane & 31);
  const bf16* qbase = a.q + (int64_t)b * T * ld + h * HD;
  const bf16* gbase = dout + (int64_t)b * T * d + h * HD;
  const float scale = 1.f / sqrtf((float)HD), c2 = kLog2e * scale;
  const uint32_t smem_off = (uint32_t)(uintptr_t)(lds_ptr)smem;
  const uint32_t ring_off = smem_off + 2 * kRows * HD * 2, stats_off = ring_off + 2 * 2 * kPairTile * 2;
  const float* lse_bh = lse + (int64_t)bh * T;
  const float* delta_bh = delta + (int64_t)bh * T;
  {
    TileOffsets<kRows, HD, kPairWaves> to;
    to.init(a.ldkv, wave, lane);
    issue_tile(a.k + (int64_t)b * Tk * a.ldkv + h * HD, a.ldkv, kblk * kRows, Tk - 1, to, smem_off, wave, lane);
    issue_tile(a.v + (int64_t)b * Tk * a.ldkv + h * HD, a.ldkv, kblk * kRows, Tk - 1, to, smem_off + kRows * HD * 2, wave, lane);
  }
  TileOffsets<kPairBQ, HD, kPairWaves> to_q, to_g;
  to_q.init(ld, wave, lane);
  to_g.init(d, wave, lane);
  auto issue = [&](int t) {
    const uint32_t st = ring_off + (uint32_t)(t & 1) * (2 * kPairTile * 2);
    issue_tile(qbase, ld, t * kPairBQ, T - 1, to_q, st, wave, lane);
    issue_tile(gbase, d, t * kPairBQ, T - 1, to_g, st + kPairTile * 2, wave, lane);
    if (wave < 2) {                            // statistics of rows past the end: the last row's, masked where they are used
      const int i = min(t * kPairBQ + lane, T - 1);
      dma4((wave ? delta_bh : lse_bh) + i, stats_off + (uint32_t)(2 * wave + (t & 1)) * (kPairBQ * 4));
    }
  };
  f32x16 dk[HD / 32], dv[HD / 32];
  clear<HD>(dk);
  clear<HD>(dv);
  const int first_tile = CAUSAL ? (kblk * kRows) / kPairBQ : 0, n_tiles = (T + kPairBQ - 1) / kPairBQ;
  // Where this lane's row of a first operand starts in LDS: features 16 kk + 8 half .. are at that address ^ (kk << 5).
  const int qrow = part * 32 + perm_row(lane & 31), krow = kw + (lane & 31);
  const uint32_t q_at = ring_off + qrow * (HD * 2) + ((half ^ swz<HD>(qrow)) << 4);
  uint32_t k_at = smem_off + krow * (HD * 2) + ((half ^ swz<HD>(krow)) << 4);
  // ... and of the second ones, read transposed: features 32 cb .. of queries 16 b2 .. at that address ^ (cb << 6), + 32 HD b2.
  const int trow = part * 32 + 8 * (lane >> 5) + ((lane & 15) >> 2);
  const uint32_t back_at = ring_off + trow * (HD * 2) + (((2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ swz<HD>(trow)) << 4) + 8 * (lane & 1);
  issue(first_tile);
  for (int t = first_tile; t < n_tiles; ++t) {
    wait_and_sync();
    if (t + 1 < n_tiles) issue(t + 1);
    const int ib = t * kPairBQ + part * 32;    // first query of this wave's block
    if ((CAUSAL && ib + 31 < k0) || ib >= T) continue;
    uint32_t qa = q_at + (uint32_t)(t & 1) * (2 * kPairTile * 2);
    asm volatile("" : "+v"(qa), "+v"(k_at));   // (the addresses below are worked out anew: 16 registers kept for them spill)
    f32x16 s, dp;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = dp[r] = 0.f;
    bf16x8 fq[kDepth], fk[kDepth], fg[kDepth], fv[kDepth];
    auto fetch = [&](int kk) {
      typedef __attribute__((address_space(3))) const bf16x8* chunk;
      const uint32_t aq = qa ^ (kk << 5), ak = k_at ^ (kk << 5);
      fq[kk % kDepth] = *(chunk)(uintptr_t)aq;
      fk[kk % kDepth] = *(chunk)(uintptr_t)ak;
      fg[kk % kDepth] = *(chunk)(uintptr_t)(aq + kPairTile * 2);
      fv[kk % kDepth] = *(chunk)(uintptr_t)(ak + kRows * HD * 2);
    };
#pragma unroll
    for (int kk = 0; kk < kDepth; ++kk) fetch(kk);
    __builtin_amdgcn_sched_barrier(0);
    DkvStats st;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      if (kk == KK - 1) load_stats(Ls[t & 1], Ds[t & 1], part, half, st);
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fq[kk % kDepth], fk[kk % kDepth], s, 0, 0, 0);
      dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fg[kk % kDepth], fv[kk % kDepth], dp, 0, 0, 0);
      if (kk + kDepth < KK) fetch(kk + kDepth);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) st.lq[r] *= kLog2e;
    if ((CAUSAL && ib < k0 + 31) || ib + 31 >= T) {   // the diagonal, or the end of the queries
      const int from = CAUSAL ? key - ib : -1, to = T - ib;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if (reg_row(r, half) < from || reg_row(r, half) >= to) st.lq[r] = INFINITY;   // no such pair: P = 0
        asm volatile("" : "+v"(st.lq[r]));
      }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c2, -st.lq[r]));
      dp[r] = s[r] * (dp[r] - st.dq[r]);
    }
    uint32_t ba = back_at + (uint32_t)(t & 1) * (2 * kPairTile * 2);
    asm volatile("" : "+v"(ba));
    auto read = [&](int j) {                   // j: (2 b2 + (0: dO -> dV, 1: Q -> dK)) * HD / 32 + cb
      const int cb = j % (HD / 32), mat = j / (HD / 32) & 1, b2 = j / (HD / 16);
      typedef __attribute__((address_space(3))) short4v* piece;
      union { bf16x8 v; short4v h[2]; } u;
#pragma unroll
      for (int e = 0; e < 2; ++e)
        u.h[e] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (piece)(uintptr_t)((ba ^ (cb << 6) ^ (e << 4)) + 8 * HD * e + 32 * HD * b2 + (mat ? 0 : kPairTile * 2)));
      return u.v;
    };
    constexpr int kAhead = 2, kBlocks = HD / 32, kSteps = 4 * kBlocks;
    bf16x8 fr[kAhead + 1];
#pragma unroll
    for (int j = 0; j < kAhead; ++j) fr[j] = read(j);
    Frag<kTerms> w[2][2];
#pragma unroll
    for (int b2 = 0; b2 < 2; ++b2) {
      w[b2][0] = pack_frag<kTerms>(s, b2 * 8);
      w[b2][1] = pack_frag<kTerms>(dp, b2 * 8);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < kSteps; ++j) {
      if (j + kAhead < kSteps) fr[(j + kAhead) % (kAhead + 1)] = read(j + kAhead);
      const int cb = j % kBlocks, mat = j / kBlocks & 1;
      mfma_frag<kTerms>(fr[j % (kAhead + 1)], w[j / (2 * kBlocks)][mat], mat ? dk[cb] : dv[cb]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  float* const box = reinterpret_cast<float*>(smem) + (wave & 3) * (HD / 2 * 64) + lane;
  (void)sum_parts<HD>(box, part, dk);          // (its barriers: every wave is done with the tiles)
  if (!sum_parts<HD>(box, part, dv)) return;
  if (SPLIT && __builtin_amdgcn_ballot_w64(key < Tk && (not_finite<HD>(dk) || not_finite<HD>(dv))) != 0) {
    dkv_again<HD, CAUSAL>(a, dout, lse, delta, dk_out, dv_out, lddkv, bh, k0);
    return;
  }
  if (key < Tk) {
    const int64_t row = ((int64_t)b * Tk + key) * lddkv + h * HD;
    store_row<HD>(dk_out + row, dk, scale);
    store_row<HD>(dv_out + row, dv, 1.f);
  }
}

}  // namespace

// Dynamic LDS: two stages of two 64-row tiles (64 KiB at head_dim 128); dK/dV three stages and their statistics (97.5 KiB;
// attn_dkv_pair_kernel has kSmemPair, 129 KiB, at width 64 65).
template <int HD, int PARTS> constexpr int kSmemTiles = 2 * 2 * kSubRows<HD, PARTS> * PARTS * HD * 2;
template <int HD, bool HIDES> constexpr int kSmemDkv = 3 * 2 * 64 * HD * 2 + 6 * 64 * 4 + (HIDES ? (64 + 32) * HD * 2 : 0);   // (tile_q)

template <int HD, bool CAUSAL, bool SPLIT>
static hipError_t prepare_dma() {
  hipError_t e = hipSuccess;
  auto raise = [&](auto kernel, int bytes) {
    if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  };
  raise(attn_fwd_dma_kernel<HD, CAUSAL, SPLIT, 1>, kSmemTiles<HD, 1>);
  raise(attn_fwd_dma_kernel<HD, CAUSAL, SPLIT, 2>, kSmemTiles<HD, 2>);
  raise(attn_dq_dma_kernel<HD, CAUSAL, SPLIT, 1>, kSmemTiles<HD, 1>);
  raise(attn_dq_dma_kernel<HD, CAUSAL, SPLIT, 2>, kSmemTiles<HD, 2>);
  constexpr int kDkv = kSmemDkv<HD, HD == 64 && CAUSAL && !SPLIT>;       // (which of these there are: bwd_dma)
  raise(attn_dkv_dma_kernel<HD, CAUSAL, SPLIT, 1, HD == 128>, kDkv);
  if constexpr (HD == 128 || SPLIT) raise(attn_dkv_dma_kernel<HD, CAUSAL, SPLIT, 2, true>, kDkv);
  if constexpr (HD == 64 && CAUSAL) raise(attn_dkv_dma_kernel<HD, CAUSAL, SPLIT, 2, false>, kDkv);
  if constexpr (HD == 128 || !CAUSAL) raise(attn_dkv_pair_kernel<HD, CAUSAL, SPLIT>, kSmemPair<HD>);
  return e;
}

// Raises the dynamic-LDS limit of the kernels (once; called at context creation, never inside a capture).
hipError_t attention_dma_init() {
  static bool done = false;
  if (done) return hipSuccess;
  hipError_t e = prepare_dma<128, true, false>();
  if (e == hipSuccess) e = prepare_dma<128, false, false>();
  if (e == hipSuccess) e = prepare_dma<64, true, false>();
  if (e == hipSuccess) e = prepare_dma<64, true, true>();
  if (e == hipSuccess) e = prepare_dma<64, false, true>();
  if (e == hipSuccess) done = true;
  return e;
}

static MhaDev dev_of(const MhaArgs& a) {
  return MhaDev{(const bf16*)a.q, (const bf16*)a.k, (const bf16*)a.v, a.ldq, a.ldkv, a.Tq, a.Tk, a.H};
}

// Whether the kernels of this file take the problem: bf16, 16-byte aligned rows, no farther apart than a lane's 32-bit byte
// offset into a tile of up to 128 rows reaches (128 * 2^24 * 2 bytes = 2^32).
constexpr int64_t kMaxLd = 1 << 24;
bool mha_dma_supported(const MhaArgs& a) {
  if (a.dtype != kBF16 || (a.hd != 128 && a.hd != 64)) return false;
  if (a.ldq > kMaxLd || a.ldkv > kMaxLd) return false;
  if (((uintptr_t)a.q | (uintptr_t)a.k | (uintptr_t)a.v) & 15) return false;
  return a.ldq % 8 == 0 && a.ldkv % 8 == 0;
}

// (problem, block) pairs, see xcd_block_map
template <int PARTS> static int blocks_of(int rows, const MhaArgs& a) { return (rows + 128 / PARTS - 1) / (128 / PARTS) * a.B * a.H; }
// Whether two waves share 32 rows (PARTS = 2: blocks of 64 rows, half the steps each, every tile loaded twice as often).
// It pays where the blocks of 128 leave compute units idle (twice as many still find one each: 128 of them), and under the
// causal mask also up to a block per unit, at head_dim 64, where units hold several, up to one and a half, since the longest
// blocks, twice the average, then decide - if those are long enough.  Both ways in us (one wave / two):
//   forward: causal, T x 64: 64 (any number) 4.7 / 5.2; 128 blocks: 128 5.7 / 5.3, 192 6.2 / 6.3, 320 8.0 / 7.3; 256 blocks: 320 8.1 / 8.6, 384
//     9.6 / 8.5, 448 9.9 / 10.0, 512 11.5 / 9.4; 384 blocks: 448 12.7 / 15.1, 512 15.3 / 14.0, 1024 23.7 / 19.7; 512 blocks: 512 13.6 / 14.8, 768
//     17.8 / 23.7.  T x 128: 64 5.4 / 6.0; 256 blocks: 256 12.4 / 10.9, 320 11.9 / 13.0, 384 15.0 / 12.9, 448 14.9 / 15.4, 512 17.4 / 14.8, 1024
//     28.2 / 22.0; 384 blocks: 512 22.9 / 22.3, 768 27.5 / 29.6.
//     Unmasked, 192 blocks over keys of 64: 64 7.0 / 7.9, 100 8.7 / 8.1, 512 16.9 / 13.9; of 128: 128 10.8 / 11.7, 192 12.2 / 13.0, 256 13.8 / 14.2, 384
//     18.3 / 17.4; 256 blocks, 1024 35.6 / 32.4; 512 blocks, 16 x 512 x 64 25.3 / 25.5.
//   backward (dQ and dK/dV): causal, T x 64: 64 10.7 / 12.4; 128 blocks: 128 15.2 / 13.5; 256 blocks: 320 22.5 / 23.6, 384 25.7 / 24.7, 512 30.2 / 27.6;
//     384 blocks: 448 36.2 / 39.4, 768 50.8 / 51.6, 1024 62.2 / 55.1; 512 blocks: 768 51.5 / 60.3, 1024 61.8 / 61.1.  T x 128: 64 15.4 / 17.9, 128
//     blocks: 128 23.4 / 21.1, 1024 69 / 48.
//   dQ alone: causal 2 x 1024, 16 x 128 (256) 70.6 / 66.0; unmasked 1 x 1000 over 2000, 16 x 128 (128) 93 / 81, 4 x 700 over 500, 8 x 128 (192) 50.0 / 51.9.
//   dK/dV alone: unmasked 1 x 2048 over 256, 16 x 128 (32) 83 / 60.6.  At head_dim 128, and unmasked at 64, the other side of the 128
//   blocks is attn_dkv_pair_kernel, see bwd_dma.
// (Forward and dQ have since lost 0.5 to 5 us in front of their loops, with one wave and with two.)
// most: the largest number of blocks, for rows whose other side is at least `from` long (where it is shorter, 128; under the
// causal mask 256 between 384 and `from`, none up to 64: one tile has no halves worth sharing).
static bool two_parts(const MhaArgs& a, int rows, int other, int from, int most) {
  const int blocks = blocks_of<1>(rows, a);
  if (a.causal && other <= 64) return false;
  if (other >= from) return blocks <= most;
  return blocks <= (a.causal && other >= 384 ? std::min(most, 256) : 128);
}

template <int HD, bool CAUSAL, bool SPLIT>
static hipError_t fwd_dma(hipStream_t s, const MhaArgs& a, void* o, void* o_lo, float* lse) {
  auto run = [&](auto kernel, int grid, int lds) { kernel<<<grid, kNT, lds, s>>>(dev_of(a), (bf16*)o, (bf16*)o_lo, lse); };
  if (CAUSAL ? two_parts(a, a.Tq, a.Tk, 512, HD == 64 ? 384 : 256) : two_parts(a, a.Tq, a.Tk, HD == 64 ? 65 : 256, 256)) run(attn_fwd_dma_kernel<HD, CAUSAL, SPLIT, 2>, blocks_of<2>(a.Tq, a), kSmemTiles<HD, 2>);
  else run(attn_fwd_dma_kernel<HD, CAUSAL, SPLIT, 1>, blocks_of<1>(a.Tq, a), kSmemTiles<HD, 1>);
  return hipGetLastError();
}
// split: probabilities and dS enter the second products as sums of bf16 values (SPLIT; head_dim 64 only).
hipError_t launch_mha_fwd_dma(hipStream_t s, const MhaArgs& a, void* o, void* o_lo, float* lse, bool split) {
  const hipError_t e = attention_dma_init();
  if (e != hipSuccess) return e;
  if (a.hd == 128) return a.causal ? fwd_dma<128, true, false>(s, a, o, o_lo, lse) : fwd_dma<128, false, false>(s, a, o, o_lo, lse);
  if (!a.causal) return fwd_dma<64, false, true>(s, a, o, o_lo, lse);
  return split ? fwd_dma<64, true, true>(s, a, o, o_lo, lse) : fwd_dma<64, true, false>(s, a, o, o_lo, lse);
}

struct MhaGrads { const void *o, *o_lo, *dout; const float* lse; float* delta; void* dq; int64_t lddq; void *dk, *dv; int64_t lddkv; };
template <int HD, bool CAUSAL, bool SPLIT>
static hipError_t bwd_dma(hipStream_t s, const MhaArgs& a, const MhaGrads& g) {
  auto run_q = [&](auto kernel, int grid, int lds) {
    kernel<<<grid, kNT, lds, s>>>(dev_of(a), (const bf16*)g.o, (const bf16*)g.o_lo, (const bf16*)g.dout, g.lse, g.delta, (bf16*)g.dq, g.lddq);
  };
  if (CAUSAL ? two_parts(a, a.Tq, a.Tk, 768, HD == 64 ? 384 : 256) : two_parts(a, a.Tq, a.Tk, 0, 128)) run_q(attn_dq_dma_kernel<HD, CAUSAL, SPLIT, 2>, blocks_of<2>(a.Tq, a), kSmemTiles<HD, 2>);
  else run_q(attn_dq_dma_kernel<HD, CAUSAL, SPLIT, 1>, blocks_of<1>(a.Tq, a), kSmemTiles<HD, 1>);
  auto run_kv = [&](auto kernel, int grid) {
    kernel<<<grid, kNT, kSmemDkv<HD, HD == 64 && CAUSAL && !SPLIT>, s>>>(dev_of(a), (const bf16*)g.dout, g.lse, g.delta, (bf16*)g.dk, (bf16*)g.dv, g.lddkv);
  };
  // Width 128, dK/dV alone (us, kernel traces, attn_dkv_dma_kernel of one wave / of two parts / attn_dkv_pair_kernel): causal 112 blocks,
  // T 192 15.7 / 12.9 / 13.6, 512 24.9 / 18.6 / 20.4, 1024 38.9 / 27.6 / 30.9; 136, T 100 12.7 / 18.3 / 12.8, 192 15.9 / 13.3 / 13.4, 512 24.9 / 26.7 / 20.6,
  // 1024 39.0 / 35.8 / 31.3; 216, 700 31.4 / 37.7 / 25.7; 256, 65 12.2 / 17.1 / 11.7, 2048 70.0 / 58.0 / 56.4; 512, 256 33.8 / 45.5 / 30.8.  Unmasked 128
  // blocks, 256 queries over 500 keys 16.5 / 14.9 / 14.8, 1000 38.3 / 28.6 / 30.9; 136, 256 16.3 / 25.2 / 14.6, 1000 38.2 / 52.9 / 31.0.  Past 128 blocks
  // two parts win only where their blocks of 64 still find a unit each (138 blocks of T 700 are 253 of 64: 30.0 / 22.3 / 24.4).  One
  // tile of queries gives pairs nothing to overlap and more waves to start: 64 over 100 keys, 256 blocks 11.2 / 18.0 / 12.5, over 500 13.3
  // / 19.0 / 13.2.  Of what pairs have, 128 queries (two whole tiles) over up to 48 keys lose on 130 to 224 blocks: 160, 32 keys 8.4 / - / 8.7;
  // 96 queries 8.8 / - / 8.7, 160 10.8 / - / 10.5, and all of these on 256 blocks and more gain, so no line is drawn for them.
  // Width 64, unmasked (one wave with the registers of two / pairs): 4 x 333 over 520, 8 heads, 160 blocks 16.1 / 12.2; 8 x 512, 16 heads, 512 blocks
  // 40.3 / 33.4; 2 x 2014 over 1092, 9 heads, 162 blocks 65.7 / 49.6.  One tile of queries loses where a second round of workgroups of eight waves starts, past
  // 256 blocks (backward, registers of one workgroup of two / pairs: 70 x 1 over 100, 4 heads, 280 blocks 18.2 / 21.0, 64 queries 18.9 / 22.0, 65 25.1 / 24.7; 16
  // x 33 over 500, 8 heads, 512 blocks 24.0 / 25.5; 5 x 33 over 500, 8 heads, 160 blocks 17.3 / 17.4, 1 query 17.2 / 16.8).  Two parts up to 128
  // blocks (those / pairs): 1 x 700, 6 heads 16.7 / 19.8; 4 x 600 over 60, 12 heads 15.5 / 17.7.  Packed causal pairs gain and lose: 1 x 2048, 16 heads 37.5 / 35.1, 8 x
  // 1024 52.9 / 56.3, 4 x 1000, 12 heads 26.8 / 27.1.
  // Two parts of width 64, registers of one workgroup of two on a unit / of both: 1 x 700, 6 heads, unmasked 27.0 / 17.8; 4 x 600 over 60, 12 heads
  // 25.5 / 16.4; causal with split dS (25 registers spill) 1 x 2048, 8 heads 47.8 / 42.4, 8 x 300, 4 heads 12.3 / 11.4, 1 x 1024, 16 heads 27.6 / 24.5;
  // packed causal (10 spill) 1 x 2048, 8 heads 31.8 / 33.4, 1 x 1024, 16 heads 18.8 / 20.1, 8 x 775, 2 heads 16.2 / 17.1.  One wave per 32 keys
  // gains nothing: 16 x 128, 16 heads 10.3 / 10.7, with split dS forward and backward 17.6 / 17.8, 40 x 64, 6 heads 12.1 / 12.4.
  constexpr bool kManyParts = HD == 64 && CAUSAL;            // more than 256 blocks of two parts occur
  if (CAUSAL ? two_parts(a, a.Tk, a.Tq, 768, HD == 64 ? 384 : 128) : two_parts(a, a.Tk, a.Tq, 0, 128)) {
    const int blocks = blocks_of<2>(a.Tk, a);
    if constexpr (!kManyParts) run_kv(attn_dkv_dma_kernel<HD, CAUSAL, SPLIT, 2, true>, blocks);
    else if constexpr (!SPLIT) run_kv(attn_dkv_dma_kernel<HD, CAUSAL, SPLIT, 2, false>, blocks);
    else run_kv(blocks <= 256 ? attn_dkv_dma_kernel<HD, CAUSAL, SPLIT, 2, true> : attn_dkv_dma_kernel<HD, CAUSAL, SPLIT, 2, false>, blocks);
    return hipGetLastError();
  }
  const int blocks = blocks_of<1>(a.Tk, a);
  if ((HD == 64 && CAUSAL) || (a.Tq <= kPairBQ && (HD == 128 || blocks > 256)))
    run_kv(attn_dkv_dma_kernel<HD, CAUSAL, SPLIT, 1, HD == 128>, blocks);
  else if constexpr (HD == 128 || !CAUSAL)
    attn_dkv_pair_kernel<HD, CAUSAL, SPLIT><<<blocks, 64 * kPairWaves, kSmemPair<HD>, s>>>(
        dev_of(a), (const bf16*)g.dout, g.lse, g.delta, (bf16*)g.dk, (bf16*)g.dv, g.lddkv);
  return hipGetLastError();
}
bool mha_dma_outputs_aligned(const void* dq, int64_t lddq, const void* dk, const void* dv, int64_t lddkv) {
  return !((((uintptr_t)dq | (uintptr_t)dk | (uintptr_t)dv) & 7) || lddq % 4 || lddkv % 4);
}
hipError_t launch_mha_dq_dkv_dma(hipStream_t s, const MhaArgs& a, const void* o, const void* o_lo, const void* dout,
                                 const float* lse, float* delta, void* dq, int64_t lddq, void* dk, void* dv, int64_t lddkv,
                                 bool split) {
  const hipError_t e = attention_dma_init();
  if (e != hipSuccess) return e;
  if (!mha_dma_outputs_aligned(dq, lddq, dk, dv, lddkv)) return hipErrorInvalidValue;
  const MhaGrads g{o, o_lo, dout, lse, delta, dq, lddq, dk, dv, lddkv};
  if (a.hd == 128) return a.causal ? bwd_dma<128, true, false>(s, a, g) : bwd_dma<128, false, false>(s, a, g);
  if (!a.causal) return bwd_dma<64, false, true>(s, a, g);
  return split ? bwd_dma<64, true, true>(s, a, g) : bwd_dma<64, true, false>(s, a, g);
}

}  // namespace pw
