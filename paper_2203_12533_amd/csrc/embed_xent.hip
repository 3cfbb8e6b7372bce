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
// A fill of dwte and a search through all tokens by the workgroup of every position took twice as long there.
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

// A row of dwte or dwpe belongs to a group of TPR threads (16 to 256, VEC float4 each: d <= 4 * TPR * VEC); the 256 / TPR
// groups of a block work side by side, so that narrow rows fill it too.  The first `id_blocks` blocks take kEbRows rows of dwte
// each (what is known about them is read in one go: with a row of its own a block spends as long waiting for it as writing),
// rows id_blocks apart: frequent ids are often neighbours, and a block adds its long rows one after the other.  The other
// blocks take dwpe (sums over the batch).
// SCAN, for at most kEbScan positions: nothing has been gathered; every block looks through all tokens for its ids.  That
// takes a time that grows with positions x blocks, two more launches about 5 us.  Both ways, us, at 2048 | 3000 positions: 32768
// ids of 64 columns 9.2 / 12.0 | 11.6 / 12.2, of 256 16 / 20 | 20 / 20, of 2048 46 / 47 | 55 / 56; 100000 ids of 128 33 / 31 | 44 / 31,
// of 1024 73 / 167 | 96 / 173; 1024 ids of 512 9 / 14 | 11 / 16.
// Order of an id's positions: up to three by comparison; up to kPart by counting for each how many are below, all rows of the
// block at once; more of them the same way row by row (n^2 / 256 steps of a thread) as long as that takes less than a look
// through all N tokens in order (a step for every 256).
// Measured (us; before: d / 4 threads for four neighbouring rows; before that: fill and search): 2048 positions over 32768 ids of
// 64 columns 7.3 (31.1; 12.6), of 2048 columns 43 (42; 54); 8192 over 32768 x 2048 64 (65; 123); drawn log-uniformly 156 (241; 430),
// over 1024 x 256 90 (338; 219).
template <int TPR> constexpr int kEbGroups = 256 / TPR;
template <int TPR> constexpr int kEbRows = TPR >= 256 ? 4 : TPR >= 64 ? 8 : 16;
constexpr int kEbScan = 2048;
template <int TPR, int VEC, bool SCAN>
__global__ __launch_bounds__(256) void embedding_bwd_kernel(const int32_t* __restrict__ tokens, const float* __restrict__ dx,
                                                            float* __restrict__ dwte, float* __restrict__ dwpe, int B, int T,
                                                            int d, int V, int stride, int id_blocks, uint32_t id_magic) {
  constexpr int kAhead = VEC <= 2 ? 8 : 8 / VEC;          // rows of dx in flight
  constexpr int kList = 2048, G = kEbGroups<TPR>, R = kEbRows<TPR>, kPart = kList / R;
  __shared__ int list[kList], sorted[kList], count[R + 1], wave_cnt[4];
  const int d4 = d >> 2, N = B * T, group = threadIdx.x / TPR, lane_in = threadIdx.x % TPR;
  float4 acc[VEC];
  auto clear = [&] {
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  };
  auto load = [&](int p, float4 (&v)[VEC]) {
    const float4* row = reinterpret_cast<const float4*>(dx + (size_t)p * d);
#pragma unroll
    for (int i = 0; i < VEC; ++i)
      if (lane_in + i * TPR < d4) v[i] = row[lane_in + i * TPR];
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
      if (lane_in + i * TPR < d4) reinterpret_cast<float4*>(out)[lane_in + i * TPR] = acc[i];
  };
  clear();
  if ((int)blockIdx.x >= id_blocks) {
    const int t = (blockIdx.x - id_blocks) * G + group;
    if (t >= T) return;
    add_all(B, [&](int b) { return b * T + t; });
    store(dwpe + (size_t)t * d);
    return;
  }
  auto id_of = [&](int r) { return (int)blockIdx.x + r * id_blocks; };
  // from -> to, by `threads` threads; elements differ: a place is how many are below
  auto sort = [](const int* from, int* to, int n, int thread, int threads) {
    for (int i = thread; i < n; i += threads) {
      const int mine = from[i];
      int place = 0;
      for (int j = 0; j < n; ++j) place += from[j] < mine;
      to[place] = mine;
    }
  };
  // A look through all tokens in order for row r; its group adds and stores.  The whole block calls.
  auto search = [&](int r) {
    const int id = id_of(r);
    const bool owner = group == r % G;
    clear();
    int have = 0;
    for (int base = 0; base < N; base += 256) {
      const int p = base + threadIdx.x;
      const bool hit = p < N && token_at(tokens, p, T, stride, V) == id;
      const uint64_t mask = __ballot(hit);
      const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
      if (lane == 0) wave_cnt[w] = __popcll(mask);
      __syncthreads();
      int before = 0, total = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (i < w) before += wave_cnt[i];
        total += wave_cnt[i];
      }
      if (hit) list[have + before + __popcll(mask & ((1ull << lane) - 1))] = p;
      have += total;
      __syncthreads();
      if (have + 256 > kList || base + 256 >= N) {
        if (owner) add_all(have, [&](int k) { return list[k]; });
        have = 0;
        __syncthreads();
      }
    }
    if (owner) store(dwte + (size_t)id * d);
  };
  if constexpr (SCAN) {
    if (threadIdx.x <= R) count[threadIdx.x] = 0;         // per row, and altogether
    __syncthreads();
    const int rows_on = 256 / T, on = 256 - rows_on * T;  // positions 256 apart, as (row, column) of the token array
    int t = threadIdx.x % T;
    const int32_t* tok = tokens + (size_t)(threadIdx.x / T) * stride;
    constexpr int kLook = 4;                              // tokens in flight (one: 2046 positions x 5000 ids x 512 6.4 us, four: 6.1)
    for (int p = threadIdx.x; p < N; p += kLook * 256) {
      int ids[kLook];
#pragma unroll
      for (int j = 0; j < kLook; ++j) {
        if (p + j * 256 < N) ids[j] = tok[t];
        tok += (size_t)rows_on * stride;
        t += on;
        if (t >= T) t -= T, tok += stride;
      }
#pragma unroll
      for (int j = 0; j < kLook; ++j) {
        if (p + j * 256 >= N) break;
        const int id = min(max(ids[j], 0), V - 1);
        int r = (int)__umulhi((uint32_t)id, id_magic), rest = id - r * id_blocks;   // id / id_blocks, one off at most
        if (rest < 0) rest += id_blocks, --r;
        if (rest >= id_blocks) rest -= id_blocks, ++r;
        if (rest == (int)blockIdx.x) {
          atomicAdd(&count[r], 1);
          const int slot = atomicAdd(&count[R], 1);
          if (slot < kList) list[slot] = r * kEbScan + p + j * 256;
        }
      }
    }
    __syncthreads();
    const int all = count[R];                             // (those behind kList are not in the list)
    if (all > 256) {
      for (int r = 0; r < R && id_of(r) < V; ++r) {
        if (count[r] > 0) search(r);
        else if (group == r % G) clear(), store(dwte + (size_t)id_of(r) * d);
      }
      return;
    }
    if (all > 0) {
      sort(list, sorted, all, threadIdx.x, 256);
      __syncthreads();
    }
    int from = 0;
#pragma unroll
    for (int k = 0; k < R / G; ++k) {
      const int r = group + k * G;
      if (id_of(r) >= V) break;
      for (int q = k == 0 ? 0 : r - G; q < r; ++q) from += count[q];
      if (k > 0) clear();
      add_all(count[r], [&](int j) { return sorted[from + j] & (kEbScan - 1); });
      store(dwte + (size_t)id_of(r) * d);
    }
    return;
  }
  int4 use[R / G];                                        // the count and the first three slots
#pragma unroll
  for (int k = 0; k < R / G; ++k) {
    const int r = group + k * G;
    use[k] = id_of(r) < V ? *reinterpret_cast<const int4*>(dwte + (size_t)id_of(r) * d) : make_int4(-1, 0, 0, 0);
    if (lane_in == 0) count[r] = use[k].x;
  }
  __syncthreads();                                        // every wave has read the first 16 bytes of the block's rows
#pragma unroll
  for (int k = 0; k < R / G; ++k) {
    const int n = use[k].x;
    if (n < 0 || n > 3) continue;
    const int a = use[k].y, b = n > 1 ? use[k].z : 0x7fffffff, c = n > 2 ? use[k].w : 0x7fffffff;
    const int lo = min(a, min(b, c)), hi = max(a, max(b, c));
    const int mid = n == 2 ? max(a, b) : max(min(a, b), min(max(a, b), c));
    clear();
    add_all(n, [&](int j) { return j == 0 ? lo : j == 1 ? mid : hi; });
    store(dwte + (size_t)id_of(group + k * G) * d);
  }
  int longest = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) longest = max(longest, count[r]);
  if (longest <= 3) return;
  // Rows whose positions fit a part of the list, all of them at once; then the others, the whole block row by row.
  auto shared_part = [&](int n) { return n > 3 && n <= kPart && n <= id_slots(d); };
#pragma unroll 1
  for (int r = group; r < R; r += G)
    if (shared_part(count[r]))
      for (int i = lane_in; i < count[r]; i += TPR) list[r * kPart + i] = reinterpret_cast<const int*>(dwte + (size_t)id_of(r) * d)[1 + i];
  __syncthreads();
#pragma unroll 1
  for (int r = group; r < R; r += G)
    if (shared_part(count[r])) sort(list + r * kPart, sorted + r * kPart, count[r], lane_in, TPR);
  __syncthreads();
#pragma unroll 1
  for (int r = group; r < R; r += G)
    if (shared_part(count[r])) {
      clear();
      add_all(count[r], [&](int k) { return sorted[r * kPart + k]; });
      store(dwte + (size_t)id_of(r) * d);
    }
  __syncthreads();
#pragma unroll 1
  for (int r = 0; r < R; ++r) {
    const int n = count[r];
    if (n <= 3 || shared_part(n)) continue;
    if (n > id_slots(d) || (int64_t)n * n > 128 * (int64_t)N) {
      search(r);
      continue;
    }
    float* const row = dwte + (size_t)id_of(r) * d;
    for (int i = threadIdx.x; i < n; i += 256) list[i] = reinterpret_cast<const int*>(row)[1 + i];
    __syncthreads();
    sort(list, sorted, n, threadIdx.x, 256);
    __syncthreads();
    if (group == r % G) {
      clear();
      add_all(n, [&](int k) { return sorted[k]; });
      store(row);
    }
    __syncthreads();
  }
}

template <bool SCAN>
static void launch_embedding_bwd_rows(hipStream_t s, const int32_t* tokens, const float* dx, float* dwte, float* dwpe, int B, int T,
                                      int d, int V, int stride) {
  auto run = [&](auto kernel, int rows, int groups) {
    const int id_blocks = (V + rows - 1) / rows;
    const uint64_t magic = (1ull << 32) / (uint64_t)id_blocks + 1;
    kernel<<<id_blocks + (T + groups - 1) / groups, 256, 0, s>>>(tokens, dx, dwte, dwpe, B, T, d, V, stride, id_blocks,
                                                                 (uint32_t)(magic < 0xffffffffull ? magic : 0xffffffffull));
  };
#define PW_EMBEDDING_BWD(TPR, VEC) run(embedding_bwd_kernel<TPR, VEC, SCAN>, kEbRows<TPR>, kEbGroups<TPR>)
  if (d <= 64) PW_EMBEDDING_BWD(16, 1);
  else if (d <= 128) PW_EMBEDDING_BWD(32, 1);
  else if (d <= 256) PW_EMBEDDING_BWD(64, 1);
  else if (d <= 512) PW_EMBEDDING_BWD(128, 1);
  else if (d <= 1024) PW_EMBEDDING_BWD(256, 1);
  else if (d <= 2048) PW_EMBEDDING_BWD(256, 2);
  else if (d <= 4096) PW_EMBEDDING_BWD(256, 4);
  else PW_EMBEDDING_BWD(256, 8);
#undef PW_EMBEDDING_BWD
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
  if ((int64_t)B * T <= kEbScan) {
    launch_embedding_bwd_rows<true>(s, tokens, dx, dwte, dwpe, B, T, d, V, stride);
  } else {
    embedding_ids_reset_kernel<<<(V + 255) / 256, 256, 0, s>>>(dwte, d, V);
    embedding_ids_gather_kernel<<<(B * T + 255) / 256, 256, 0, s>>>(tokens, dwte, B * T, T, d, V, stride);
    launch_embedding_bwd_rows<false>(s, tokens, dx, dwte, dwpe, B, T, d, V, stride);
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
