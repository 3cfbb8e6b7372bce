// Embedding lookup (forward, backward) and fused softmax cross-entropy.  HBM-bound kernels.
#include "common.hpp"
#include "kernels.hpp"

namespace pw {

// Token id of flat position p = b*T + t in a token array whose rows are `stride` ids apart (T+1 for the
// [B, T+1] arrays that carry inputs and next-token targets together), clamped into [0, V) so that a bad id
// can never index outside the tables (forward and backward clamp identically).
__device__ __forceinline__ int token_at(const int32_t* __restrict__ tokens, int p, int T, int stride, int V, int shift = 0) {
  const int b = p / T, t = p - b * T;
  const int id = tokens[(size_t)b * stride + t + shift];
  return id < 0 ? 0 : (id >= V ? V - 1 : id);
}

// ---- embedding forward: x[b*T+t,:] = wte[tok[b,t],:] + wpe[t,:] (one fp32 add per element: exact) ----
__global__ void embedding_fwd_kernel(const int32_t* __restrict__ tokens, const float* __restrict__ wte,
                                     const float* __restrict__ wpe, float* __restrict__ x, int B, int T, int d, int V,
                                     int stride) {
  const int n = blockIdx.x;
  const int t = n % T;
  const int id = token_at(tokens, n, T, stride, V);
  const float4* we = reinterpret_cast<const float4*>(wte + (size_t)id * d);
  const float4* pe = reinterpret_cast<const float4*>(wpe + (size_t)t * d);
  float4* xo = reinterpret_cast<float4*>(x + (size_t)n * d);
  for (int c = threadIdx.x; c < (d >> 2); c += blockDim.x) {
    const float4 a = we[c], p = pe[c];
    xo[c] = make_float4(a.x + p.x, a.y + p.y, a.z + p.z, a.w + p.w);
  }
}

hipError_t launch_embedding_fwd(hipStream_t s, const int32_t* tokens, const float* wte, const float* wpe, float* x,
                                int B, int T, int d, int V, int tok_stride) {
  const int stride = tok_stride > 0 ? tok_stride : T + 1;
  if (stride < T) return hipErrorInvalidValue;
  if (!tokens || !wte || !wpe || !x || B < 0 || T <= 0 || d <= 0 || d % 4 || V <= 0) return hipErrorInvalidValue;
  if (((uintptr_t)wte | (uintptr_t)wpe | (uintptr_t)x) & 15) return hipErrorInvalidValue;
  if (B == 0) return hipSuccess;
  embedding_fwd_kernel<<<B * T, 256, 0, s>>>(tokens, wte, wpe, x, B, T, d, V, stride);
  return hipGetLastError();
}

// ---- embedding backward -------------------------------------------------------------------------------
// dwte is a scatter-add with repeated ids; every id's rows of dx are added in ascending order of their positions, without
// floating-point atomics: the same bits on every run.  The positions of an id are gathered first, in the id's own row of
// dwte - a count and, as far as they fit, the positions in whatever order integer atomics deal the slots - which the last
// kernel sorts and overwrites.  That kernel writes each row once: zeros for an unused id, else the sum of its rows.
// HBM-bound by the write of dwte (268 of the 345 MB that 8192 positions, 32768 ids of 2048 columns cannot do without).
// Measured there 85 us; a fill of dwte and a search through all tokens by the workgroup of every position took 143 (1024
// ids: 32 against 60; 256 columns: 23 against 77).
__device__ __forceinline__ int id_slots(int d) { return d - 1 < 2047 ? d - 1 : 2047; }   // positions that fit the row

__global__ __launch_bounds__(256) void embedding_ids_reset_kernel(float* __restrict__ dwte, int d, int V) {
  const int id = blockIdx.x * 256 + threadIdx.x;
  if (id < V) *reinterpret_cast<int4*>(dwte + (size_t)id * d) = make_int4(0, 0, 0, 0);
}
__global__ __launch_bounds__(256) void embedding_ids_gather_kernel(const int32_t* __restrict__ tokens, float* __restrict__ dwte,
                                                                   int N, int T, int d, int V, int stride) {
  const int p = blockIdx.x * 256 + threadIdx.x;
  if (p >= N) return;
  int* row = reinterpret_cast<int*>(dwte + (size_t)token_at(tokens, p, T, stride, V) * d);
  const int slot = atomicAdd(row, 1);
  if (slot < id_slots(d)) row[1 + slot] = p;
}

// VEC float4 per thread cover a row (d <= 1024 * VEC).  The first blocks take kEbRows rows of dwte each (what is known about
// them is read in one go: with a row of its own a block spends as long waiting for it as writing), the last T blocks one
// row of dwpe (the sum over the batch).
// SCAN, for at most kEbScan positions: nothing has been gathered; every block looks through all tokens for its ids, which
// takes less time than two more launches (512 positions, 5000 ids of 1012 columns, with the forward lookup: 9.4 us against
// 17.8, and 15.8 with the fill and search).
constexpr int kEbRows = 4;
constexpr int kEbScan = 2048;
template <int VEC, bool SCAN>
__global__ __launch_bounds__(256) void embedding_bwd_kernel(const int32_t* __restrict__ tokens, const float* __restrict__ dx,
                                                            float* __restrict__ dwte, float* __restrict__ dwpe, int B, int T,
                                                            int d, int V, int stride, int id_blocks) {
  constexpr int kAhead = VEC <= 2 ? 8 : 8 / VEC;          // rows of dx in flight
  constexpr int kList = 2048;
  __shared__ int list[kList], sorted[kList], wave_cnt[4];
  const int d4 = d >> 2, nt = blockDim.x, N = B * T;
  float4 acc[VEC];
  auto clear = [&] {
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  };
  auto load = [&](int p, float4 (&v)[VEC]) {
    const float4* row = reinterpret_cast<const float4*>(dx + (size_t)p * d);
#pragma unroll
    for (int i = 0; i < VEC; ++i)
      if ((int)threadIdx.x + i * nt < d4) v[i] = row[threadIdx.x + i * nt];
  };
  auto add = [&](const float4 (&v)[VEC]) {
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
      acc[i].x += v[i].x; acc[i].y += v[i].y; acc[i].z += v[i].z; acc[i].w += v[i].w;
    }
  };
  auto add_all = [&](int n, auto&& position) {            // rows position(0), position(1), ... in this order
    int k = 0;
    for (; k + kAhead <= n; k += kAhead) {
      float4 v[kAhead][VEC];
#pragma unroll
      for (int j = 0; j < kAhead; ++j) load(position(k + j), v[j]);
#pragma unroll
      for (int j = 0; j < kAhead; ++j) add(v[j]);
    }
    for (; k < n; ++k) {
      float4 v[VEC];
      load(position(k), v);
      add(v);
    }
  };
  auto store = [&](float* out) {
#pragma unroll
    for (int i = 0; i < VEC; ++i)
      if ((int)threadIdx.x + i * nt < d4) reinterpret_cast<float4*>(out)[threadIdx.x + i * nt] = acc[i];
  };
  clear();
  if ((int)blockIdx.x >= id_blocks) {
    const int t = blockIdx.x - id_blocks;
    add_all(B, [&](int b) { return b * T + t; });
    store(dwpe + (size_t)t * d);
    return;
  }
  const int id0 = blockIdx.x * kEbRows;
  auto sort = [&](int n) {                                // list -> sorted; elements differ: a place is how many are below
    for (int i = threadIdx.x; i < n; i += nt) {
      int place = 0;
      for (int j = 0; j < n; ++j) place += list[j] < list[i];
      sorted[place] = list[i];
    }
    __syncthreads();
  };
  if constexpr (SCAN) {
    __shared__ int found[kEbRows + 1];                    // per row, and altogether
    if (threadIdx.x <= kEbRows) found[threadIdx.x] = 0;
    __syncthreads();
    for (int p = threadIdx.x; p < N; p += nt) {
      const int r = token_at(tokens, p, T, stride, V) - id0;
      if (r >= 0 && r < kEbRows) {
        atomicAdd(&found[r], 1);
        list[atomicAdd(&found[kEbRows], 1)] = r * kEbScan + p;
      }
    }
    __syncthreads();
    if (found[kEbRows] > 0) sort(found[kEbRows]);
    int from = 0;
#pragma unroll
    for (int r = 0; r < kEbRows; ++r) {
      if (id0 + r >= V) break;
      if (r > 0) clear();
      add_all(found[r], [&](int k) { return sorted[from + k] & (kEbScan - 1); });
      from += found[r];
      store(dwte + (size_t)(id0 + r) * d);
    }
    return;
  }
  int4 use[kEbRows];                                      // the count and the first three slots
#pragma unroll
  for (int r = 0; r < kEbRows; ++r)
    if (id0 + r < V) use[r] = *reinterpret_cast<const int4*>(dwte + (size_t)(id0 + r) * d);
  __syncthreads();                                        // every wave has read the first 16 bytes of the block's rows
#pragma unroll
  for (int r = 0; r < kEbRows; ++r) {
    const int id = id0 + r;
    if (id >= V) break;                                   // uniform, as everything that depends on a count
    const int count = use[r].x;
    if (r > 0) clear();
    if (count <= 3) {
      const int a = use[r].y, b = count > 1 ? use[r].z : 0x7fffffff, c = count > 2 ? use[r].w : 0x7fffffff;
      const int lo = min(a, min(b, c)), hi = max(a, max(b, c));
      const int mid = count == 2 ? max(a, b) : max(min(a, b), min(max(a, b), c));
      add_all(count, [&](int k) { return k == 0 ? lo : k == 1 ? mid : hi; });
    } else if (count <= id_slots(d)) {
      const int* row = reinterpret_cast<const int*>(dwte + (size_t)id * d) + 1;
      for (int i = threadIdx.x; i < count; i += nt) list[i] = row[i];
      __syncthreads();
      sort(count);
      add_all(count, [&](int k) { return sorted[k]; });
    } else {                                              // more than the row holds: look through all tokens, in order
      int have = 0;
      for (int base = 0; base < N; base += nt) {
        const int p = base + threadIdx.x;
        const bool hit = p < N && token_at(tokens, p, T, stride, V) == id;
        const uint64_t mask = __ballot(hit);
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        if (lane == 0) wave_cnt[w] = __popcll(mask);
        __syncthreads();
        int before = 0, total = 0;
        for (int i = 0; i < (nt >> 6); ++i) {
          if (i < w) before += wave_cnt[i];
          total += wave_cnt[i];
        }
        if (hit) list[have + before + __popcll(mask & ((1ull << lane) - 1))] = p;
        have += total;
        __syncthreads();
        if (have + nt > kList || base + nt >= N) {
          add_all(have, [&](int k) { return list[k]; });
          have = 0;
          __syncthreads();
        }
      }
    }
    store(dwte + (size_t)id * d);
  }
}

template <bool SCAN>
static void launch_embedding_bwd_rows(hipStream_t s, int block, const int32_t* tokens, const float* dx, float* dwte, float* dwpe,
                                      int B, int T, int d, int V, int stride) {
  const int id_blocks = (V + kEbRows - 1) / kEbRows, grid = id_blocks + T;
  if (d <= 1024) embedding_bwd_kernel<1, SCAN><<<grid, block, 0, s>>>(tokens, dx, dwte, dwpe, B, T, d, V, stride, id_blocks);
  else if (d <= 2048) embedding_bwd_kernel<2, SCAN><<<grid, block, 0, s>>>(tokens, dx, dwte, dwpe, B, T, d, V, stride, id_blocks);
  else if (d <= 4096) embedding_bwd_kernel<4, SCAN><<<grid, block, 0, s>>>(tokens, dx, dwte, dwpe, B, T, d, V, stride, id_blocks);
  else embedding_bwd_kernel<8, SCAN><<<grid, block, 0, s>>>(tokens, dx, dwte, dwpe, B, T, d, V, stride, id_blocks);
}

hipError_t launch_embedding_bwd(hipStream_t s, const int32_t* tokens, const float* dx, float* dwte, float* dwpe,
                                int B, int T, int d, int V, int tok_stride) {
  const int stride = tok_stride > 0 ? tok_stride : T + 1;
  if (stride < T) return hipErrorInvalidValue;
  if (!tokens || !dx || !dwte || !dwpe || B < 0 || T <= 0 || d <= 0 || d % 4 || d > 8192 || V <= 0) return hipErrorInvalidValue;
  if (((uintptr_t)dx | (uintptr_t)dwte | (uintptr_t)dwpe) & 15) return hipErrorInvalidValue;
  if (B == 0) {
    const hipError_t e = launch_fill_f32(s, dwte, (int64_t)V * d, 0.f);
    return e != hipSuccess ? e : launch_fill_f32(s, dwpe, (int64_t)T * d, 0.f);
  }
  int block = ((d >> 2) + 63) / 64 * 64;                  // one float4 per thread, whole waves, at most 256
  if (block > 256) block = 256;
  if ((int64_t)B * T <= kEbScan) {
    launch_embedding_bwd_rows<true>(s, block, tokens, dx, dwte, dwpe, B, T, d, V, stride);
  } else {
    embedding_ids_reset_kernel<<<(V + 255) / 256, 256, 0, s>>>(dwte, d, V);
    embedding_ids_gather_kernel<<<(B * T + 255) / 256, 256, 0, s>>>(tokens, dwte, B * T, T, d, V, stride);
    launch_embedding_bwd_rows<false>(s, block, tokens, dx, dwte, dwpe, B, T, d, V, stride);
  }
  return hipGetLastError();
}

// ---- softmax cross-entropy ----------------------------------------------------------------------------
// One block per row of logits, HBM-bound.  A row of up to kXeThreads * 16 bytes * 8 (32768 columns in bf16) stays in
// registers between the statistics and the gradient, (softmax - onehot)/N, that overwrites it: one read, one write.
// Longer rows are read twice.  Row losses are added in a fixed order by a one-block kernel.  8192 x 32768 in bf16: 257 us
// with two reads -> 215 (5.0 TB/s, the rate of a plain copy).
constexpr int kXeThreads = 512;

template <class T> struct Vec8;
template <> struct Vec8<bf16> {
  static constexpr int n = 8;
  static __device__ __forceinline__ void load(const bf16* p, float* o) {
    const bf16x8 v = *reinterpret_cast<const bf16x8*>(p);
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = (float)v[i];
  }
  static __device__ __forceinline__ void store(bf16* p, const float* o) {
    bf16x8 v;
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = (bf16)o[i];
    *reinterpret_cast<bf16x8*>(p) = v;
  }
};
template <> struct Vec8<float> {
  static constexpr int n = 4;
  static __device__ __forceinline__ void load(const float* p, float* o) {
    const float4 v = *reinterpret_cast<const float4*>(p);
    o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
  }
  static __device__ __forceinline__ void store(float* p, const float* o) {
    *reinterpret_cast<float4*>(p) = make_float4(o[0], o[1], o[2], o[3]);
  }
};

// The row in registers, as it is stored: CH chunks of 16 bytes per thread.
template <class T, int CH>
__global__ __launch_bounds__(kXeThreads) void softmax_xent_held_kernel(T* __restrict__ z, const int32_t* __restrict__ tokens,
                                                                       float* __restrict__ row_loss, int T_, int V, float inv_n) {
  __shared__ float red[kXeThreads / 64];
  constexpr int W = Vec8<T>::n;
  const int n = blockIdx.x;
  T* zr = z + (size_t)n * V;
  uint4 raw[CH];
#pragma unroll
  for (int i = 0; i < CH; ++i) {
    const int c = (threadIdx.x + i * kXeThreads) * W;
    if (c < V) raw[i] = *reinterpret_cast<const uint4*>(zr + c);
  }
  const int tgt = token_at(tokens, n, T_, T_ + 1, V, 1);
  float m = -INFINITY;
#pragma unroll
  for (int i = 0; i < CH; ++i)
    if ((threadIdx.x + i * kXeThreads) * W < V) {
      float v[W];
      Vec8<T>::load(reinterpret_cast<const T*>(&raw[i]), v);
#pragma unroll
      for (int k = 0; k < W; ++k) m = fmaxf(m, v[k]);
    }
  const float gm = block_max(m, red);
  float l = 0.f;
#pragma unroll
  for (int i = 0; i < CH; ++i)
    if ((threadIdx.x + i * kXeThreads) * W < V) {
      float v[W];
      Vec8<T>::load(reinterpret_cast<const T*>(&raw[i]), v);
#pragma unroll
      for (int k = 0; k < W; ++k) l += __expf(v[k] - gm);
    }
  const float lse = gm + logf(block_sum(l, red));
#pragma unroll
  for (int i = 0; i < CH; ++i) {
    const int c = (threadIdx.x + i * kXeThreads) * W;
    if (c < V) {
      float v[W];
      Vec8<T>::load(reinterpret_cast<const T*>(&raw[i]), v);
#pragma unroll
      for (int k = 0; k < W; ++k) {
        if (c + k == tgt) row_loss[n] = lse - v[k];
        v[k] = (__expf(v[k] - lse) - (c + k == tgt ? 1.f : 0.f)) * inv_n;
      }
      Vec8<T>::store(zr + c, v);
    }
  }
}

// Longer rows: the second pass reads the row again.
template <class T>
__global__ __launch_bounds__(kXeThreads) void softmax_xent_kernel(T* __restrict__ z, const int32_t* __restrict__ tokens,
                                                                  float* __restrict__ row_loss, int T_, int V, float inv_n) {
  __shared__ float red[kXeThreads / 64];
  constexpr int W = Vec8<T>::n;
  const int n = blockIdx.x;
  const int tgt = token_at(tokens, n, T_, T_ + 1, V, 1);
  T* zr = z + (size_t)n * V;
  float m = -INFINITY, l = 0.f;
  for (int c = threadIdx.x * W; c < V; c += kXeThreads * W) {
    float v[W];
    Vec8<T>::load(zr + c, v);
    float cm = v[0];
#pragma unroll
    for (int i = 1; i < W; ++i) cm = fmaxf(cm, v[i]);
    const float nm = fmaxf(m, cm);
    float add = 0.f;
#pragma unroll
    for (int i = 0; i < W; ++i) add += __expf(v[i] - nm);
    l = l * __expf(m - nm) + add;
    m = nm;
  }
  const float gm = block_max(m, red);
  const float gl = block_sum(l * __expf(m - gm), red);   // threads with no column have l = 0, m = -inf: exp(-inf) = 0
  const float lse = gm + logf(gl);
  if (threadIdx.x == 0) row_loss[n] = lse - to_f32(zr[tgt]);
  __syncthreads();   // zr[tgt] was read before anyone overwrites the row
  for (int c = threadIdx.x * W; c < V; c += kXeThreads * W) {
    float v[W];
    Vec8<T>::load(zr + c, v);
#pragma unroll
    for (int i = 0; i < W; ++i) v[i] = (__expf(v[i] - lse) - (c + i == tgt ? 1.f : 0.f)) * inv_n;
    Vec8<T>::store(zr + c, v);
  }
}

// thread i adds rows i, i + 1024, ... in order (eight in flight), then the block's sum in its fixed order
constexpr int kMrThreads = 1024;
__global__ __launch_bounds__(kMrThreads) void mean_rows_kernel(const float* __restrict__ row_loss, float* __restrict__ loss, int N) {
  __shared__ float red[kMrThreads / 64];
  float s = 0.f;
#pragma unroll 8
  for (int n = threadIdx.x; n < N; n += kMrThreads) s += row_loss[n];
  const float total = block_sum(s, red);
  if (threadIdx.x == 0) *loss = total / (float)N;
}

// Loss from the per-group statistics that the LM-head GEMM's kEpiXentStats epilogue leaves (the logits themselves
// were never stored): one wave per row merges the (max, sum exp(z - max)) pairs of the row's 64-column groups.
__global__ __launch_bounds__(256) void xent_from_stats_kernel(const float* __restrict__ part, const float* __restrict__ zt,
                                                               float* __restrict__ lse, float* __restrict__ row_loss,
                                                               int N, int groups) {
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= N) return;   // whole waves leave together
  const float2* pr = reinterpret_cast<const float2*>(part) + (size_t)r * groups;
  float m = -INFINITY, l = 0.f;
  for (int g = lane; g < groups; g += 64) {
    const float2 p = pr[g];
    const float nm = fmaxf(m, p.x);
    l = l * __expf(m - nm) + p.y * __expf(p.x - nm);
    m = nm;
  }
  const float gm = wave_max(m);
  const float gl = wave_sum(l * __expf(m - gm));   // lanes without a group: l = 0, exp(-inf) = 0
  if (lane == 0) {
    const float v = gm + logf(gl);
    lse[r] = v;
    row_loss[r] = v - zt[r];
  }
}

hipError_t launch_xent_from_stats(hipStream_t s, const float* part, const float* zt, float* lse, float* row_loss,
                                  float* loss, int N, int groups) {
  if (!part || !zt || !lse || !row_loss || !loss || N <= 0 || groups <= 0 || ((uintptr_t)part & 7)) return hipErrorInvalidValue;
  xent_from_stats_kernel<<<(N + 3) / 4, 256, 0, s>>>(part, zt, lse, row_loss, N, groups);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  mean_rows_kernel<<<1, kMrThreads, 0, s>>>(row_loss, loss, N);
  return hipGetLastError();
}

template <class T>
static void launch_xent_rows(hipStream_t s, T* z, const int32_t* tokens, float* row_loss, int N, int T_, int V) {
  const int per = kXeThreads * Vec8<T>::n;           // columns per chunk
  const float inv_n = 1.f / (float)N;
  if (V <= per) softmax_xent_held_kernel<T, 1><<<N, kXeThreads, 0, s>>>(z, tokens, row_loss, T_, V, inv_n);
  else if (V <= 2 * per) softmax_xent_held_kernel<T, 2><<<N, kXeThreads, 0, s>>>(z, tokens, row_loss, T_, V, inv_n);
  else if (V <= 4 * per) softmax_xent_held_kernel<T, 4><<<N, kXeThreads, 0, s>>>(z, tokens, row_loss, T_, V, inv_n);
  else if (V <= 8 * per) softmax_xent_held_kernel<T, 8><<<N, kXeThreads, 0, s>>>(z, tokens, row_loss, T_, V, inv_n);
  else softmax_xent_kernel<T><<<N, kXeThreads, 0, s>>>(z, tokens, row_loss, T_, V, inv_n);
}

hipError_t launch_softmax_xent(hipStream_t s, int dtype, void* z, const int32_t* tokens, float* loss, float* row_loss,
                               int B, int T, int V) {
  if (!z || !tokens || !loss || !row_loss || B <= 0 || T <= 0 || V <= 0) return hipErrorInvalidValue;
  const int W = dtype == kBF16 ? 8 : 4;
  if (V % W || ((uintptr_t)z & 15)) return hipErrorInvalidValue;
  const int N = B * T;
  if (dtype == kF32) launch_xent_rows<float>(s, (float*)z, tokens, row_loss, N, T, V);
  else if (dtype == kBF16) launch_xent_rows<bf16>(s, (bf16*)z, tokens, row_loss, N, T, V);
  else return hipErrorInvalidValue;
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  mean_rows_kernel<<<1, kMrThreads, 0, s>>>(row_loss, loss, N);
  return hipGetLastError();
}

}  // namespace pw
