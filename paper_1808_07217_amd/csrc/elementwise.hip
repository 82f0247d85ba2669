// Bandwidth- and latency-bound kernels of the local-SGD step: index
// sampling, softmax cross-entropy, bias gradient + update, the fused
// momentum-SGD update, and the K-way replica average.
#include "kernels.h"
#include "device_common.h"

namespace lsgd {
namespace {

// One thread per (worker k, group of 4 slots): a Philox block gives the four
// uniform words of slots 4q .. 4q+3 of worker k at local step `step`.
__global__ void k_sample(uint32_t key0, uint32_t key1, uint32_t s_lo,
                         uint32_t s_hi, int K, long long N, int B,
                         int32_t* idx) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (4 * q < B) sample_iid4(key0, key1, s_lo, s_hi, blockIdx.y, K, N, B, q, idx);
}

// One thread per (worker k = blockIdx.y, slot b): row pi_e(lo_k + jB + b).
__global__ void k_sample_epoch(uint32_t key0, uint32_t key1, uint32_t e, long long j,
                               int K, long long N, int B, int m, int32_t* idx) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  const int k = blockIdx.y;
  if (b >= B) return;
  const uint32_t q = (uint32_t)((long long)k * N / K + j * B + b);
  idx[(long long)k * B + b] = epoch_row(q, N, m, key0, key1, e);
}

// ------------------------------------------------------------------ loss
// Softmax cross-entropy over C classes for the B rows of replica k
// (blockIdx.x): dZ = (softmax(z) - onehot(y)) / B and the mean loss, summed
// in a fixed order (per-thread rows ascending, then a fixed LDS tree).
__global__ __launch_bounds__(256) void k_xent(const float* Z, const int32_t* y,
                                              const int32_t* idx, int B, int C,
                                              void* dZ, int dz_bf16,
                                              float* loss, int* nonfinite) {
  __shared__ float red[256];
  const int k = blockIdx.x;
  const float invB = 1.0f / (float)B;
  float part = 0.f;
  for (int b = threadIdx.x; b < B; b += blockDim.x) {
    const long long row = (long long)k * B + b;
    const float* z = Z + row * C;
    const int lab = y[idx[row]];
    float m = z[0];
    for (int j = 1; j < C; ++j) m = fmaxf(m, z[j]);
    float s = 0.f, rest = 0.f;
    for (int j = 0; j < C; ++j) {
      const float e = __expf(z[j] - m);
      s += e;
      if (j != lab) rest += e;
    }
    const float zy = z[lab];
    part += zy >= m ? log1pf(rest) : (m - zy) + logf(s);
    const float inv_s = 1.0f / s;
    for (int j = 0; j < C; ++j) {
      const float p = __expf(z[j] - m) * inv_s;
      const float d = (p - (j == lab ? 1.f : 0.f)) * invB;
      if (dz_bf16)
        ((bf16_t*)dZ)[row * C + j] = f32_to_bf16(d);
      else
        ((float*)dZ)[row * C + j] = d;
    }
  }
  red[threadIdx.x] = part;
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const float mean = red[0] * invB;
    if (loss) loss[k] = mean;
    if (nonfinite && !isfinite(mean)) *nonfinite = 1;
  }
}

// ------------------------------------------------------------------ update
__device__ __forceinline__ void sgd(float& w, float& u, float grad, float lr,
                                    float mom, float wd, int nesterov) {
  const float g = __builtin_fmaf(wd, w, grad);
  u = __builtin_fmaf(mom, u, g);
  const float d = step_dir(u, g, mom, nesterov);
  w = __builtin_fmaf(-lr, d, w);
}

__global__ void k_sgd_update4(float4* W, float4* U, const float4* G,
                              long long n4, float lr, float mom, float wd,
                              int nesterov) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n4;
       i += (long long)gridDim.x * blockDim.x) {
    float4 w = W[i], u = U[i];
    const float4 g = G[i];
    sgd(w.x, u.x, g.x, lr, mom, wd, nesterov);
    sgd(w.y, u.y, g.y, lr, mom, wd, nesterov);
    sgd(w.z, u.z, g.z, lr, mom, wd, nesterov);
    sgd(w.w, u.w, g.w, lr, mom, wd, nesterov);
    W[i] = w;
    U[i] = u;
  }
}

__global__ void k_sgd_update1(float* W, float* U, const float* G, long long n,
                              float lr, float mom, float wd, int nesterov) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    float w = W[i], u = U[i];
    sgd(w, u, G[i], lr, mom, wd, nesterov);
    W[i] = w;
    U[i] = u;
  }
}

// ------------------------------------------------------------------ average
// Fixed summation tree over replicas lo .. lo+n-1: split at the largest power
// of two below n, left part first. For a power-of-two K this is the pairwise
// tree ((0+1)+(2+3))+..., under which identical replicas sum exactly.
__host__ __device__ constexpr int split_of(int n) {
  int h = 1;
  while (2 * h < n) h *= 2;
  return h;
}

template <int N>
struct Tree {
  template <typename F>
  __device__ __forceinline__ static auto sum(const F& ld, int k0) {
    constexpr int H = split_of(N);
    return Tree<H>::sum(ld, k0) + Tree<N - H>::sum(ld, k0 + H);
  }
};
template <>
struct Tree<1> {
  template <typename F>
  __device__ __forceinline__ static auto sum(const F& ld, int k0) {
    return ld(k0);
  }
};

// Same tree for a run-time K: blocks of eight through a binary counter of
// power-of-two sums, then the K % 8 left over, folded from the right. The
// counter's levels are unrolled, so that it stays in registers: LV of them hold
// 8 (2^LV - 1) + 7 replicas.
template <int LV, typename F>
__device__ __forceinline__ auto tree_sum_rt(const F& ld, int K) {
  using V = decltype(ld(0));
  const int q = K / 8, r = K % 8;
  V st[LV];
  for (int c = 0; c < q; ++c) {
    V v = Tree<8>::sum(ld, 8 * c);
    bool carry = true;
#pragma unroll
    for (int l = 0; l < LV; ++l) {
      if (!carry) continue;
      if (c >> l & 1) {
        v = st[l] + v;
      } else {
        st[l] = v;
        carry = false;
      }
    }
  }
  V v{};
  bool any = false;  // (uniform, as K is)
  auto left = [&](const V& w) __attribute__((always_inline)) {
    v = any ? w + v : w;
    any = true;
  };
  if (r & 1) left(ld(K - 1));
  if (r & 2) left(Tree<2>::sum(ld, K - r % 4));
  if (r & 4) left(Tree<4>::sum(ld, K - r));
#pragma unroll
  for (int l = 0; l < LV; ++l)
    if (q >> l & 1) left(st[l]);
  return v;
}
// KT > 0: KT replicas; 0 and -1: any K up to 127, any K.
template <int KT, typename F>
__device__ __forceinline__ auto tree_sum(const F& ld, int K) {
  if constexpr (KT > 0)
    return Tree<KT>::sum(ld, 0);
  else
    return tree_sum_rt<KT == 0 ? 4 : 28>(ld, K);
}

// Four floats, and four bf16 values, at any element's alignment: the row
// pitch of caller-owned arrays need not be a multiple of four.
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x2_any __attribute__((ext_vector_type(2), aligned(2)));

// NT: streams beyond the Infinity Cache bypass it (loads and stores without
// allocation); smaller ones keep their lines, which the next kernel reads.
template <bool NT>
__device__ __forceinline__ v4f ld4(const float* p) {
  if constexpr (NT) return __builtin_nontemporal_load((const v4f_any*)p);
  return *(const v4f_any*)p;
}
template <bool NT>
__device__ __forceinline__ void st4(float* p, v4f v) {
  if constexpr (NT)
    __builtin_nontemporal_store(v, (v4f_any*)p);
  else
    *(v4f_any*)p = v;
}
__device__ __forceinline__ void store_bf16x4(bf16_t* p, v4f v) {
  const uint32_t a = f32_to_bf16(v.x) | ((uint32_t)f32_to_bf16(v.y) << 16);
  const uint32_t b = f32_to_bf16(v.z) | ((uint32_t)f32_to_bf16(v.w) << 16);
  *(u32x2_any*)p = u32x2_any{a, b};
}

// The replica average: item i owns elements 4i .. 4i+3 of every replica; the
// n % 4 elements left over are an item each (one thread taking them in turn
// would chain their K loads: 82 us instead of 7 for 24 rows of 100003).
// The grid's y index picks a block of K consecutive replicas (hierarchical
// averaging; a single block is the global average).
// mean_out != nullptr (one block): write the mean there (and its bf16 copy to
// Wb [n] when given) and leave W untouched.
// HBM-bound. 16 x 16.8M (2.1 GB read and written): 455 us, with the NT
// form 366 us (5.9 TB/s). The plain form keeps eight wavefronts a SIMD: with more
// registers (74 for 16 rows) rows in the cache whose pitch is a power of two lose
// up to 10% (16 x 1M 21.2 -> 23.4 us, 32 x 1M 41.7 -> 46.5), others 1%.
template <int KT, bool NT>
__global__ __launch_bounds__(256, !NT && KT > 0 && KT <= 32 ? 8 : 1) void k_average4(float* W, bf16_t* Wb, int K, long long n,
                                                  long long ld, float* mean_out) {
  W += blockIdx.y * (long long)K * ld;
  if (Wb) Wb += blockIdx.y * (long long)K * ld;
  const float Kf = (float)K;
  const long long n4 = n / 4, items = n4 + n % 4;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < items;
       i += (long long)gridDim.x * blockDim.x) {
    if (i < n4) {
      const long long e = 4 * i;
      const v4f s = tree_sum<KT>([&](int k) { return ld4<NT>(W + k * ld + e); }, K);
      const v4f mean = v4f{s.x / Kf, s.y / Kf, s.z / Kf, s.w / Kf};
      if (mean_out) {
        *(v4f_any*)(mean_out + e) = mean;
        if (Wb) store_bf16x4(Wb + e, mean);
        continue;
      }
      for (int k = 0; k < K; ++k) {
        st4<NT>(W + k * ld + e, mean);
        if (Wb) store_bf16x4(Wb + k * ld + e, mean);
      }
      continue;
    }
    const long long e = 3 * n4 + i;
    const float mean = tree_sum<KT>([&](int k) { return W[k * ld + e]; }, K) / Kf;
    if (mean_out) {
      mean_out[e] = mean;
      if (Wb) Wb[e] = f32_to_bf16(mean);
      continue;
    }
    for (int k = 0; k < K; ++k) {
      W[k * ld + e] = mean;
      if (Wb) Wb[k * ld + e] = f32_to_bf16(mean);
    }
  }
}

// Synchronisation with global momentum: the replica mean (the tree of
// k_average4), then u = mg u + (ws - mean) / lr and ws = ws - lr u, where ws
// holds the model of the previous synchronisation; every replica gets ws.
__device__ __forceinline__ float gm_step(float mean, float& ws, float& u,
                                         float mg, float lr) {
  u = mg * u + (ws - mean) / lr;
  ws = ws - lr * u;
  return ws;
}

template <int KT, bool NT>
__global__ __launch_bounds__(256) void k_average_gm4(float* W, bf16_t* Wb, int K, long long n,
                                                     long long ld, float* ws, float* ug,
                                                     float mg, float lr) {
  const float Kf = (float)K;
  const long long n4 = n / 4, items = n4 + n % 4;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < items;
       i += (long long)gridDim.x * blockDim.x) {
    if (i < n4) {
      const long long e = 4 * i;
      const v4f s = tree_sum<KT>([&](int k) { return ld4<NT>(W + k * ld + e); }, K);
      v4f w = *(const v4f_any*)(ws + e), u = *(const v4f_any*)(ug + e);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float wj = w[j], uj = u[j];
        gm_step(s[j] / Kf, wj, uj, mg, lr);
        w[j] = wj;
        u[j] = uj;
      }
      *(v4f_any*)(ws + e) = w;
      *(v4f_any*)(ug + e) = u;
      for (int k = 0; k < K; ++k) {
        st4<NT>(W + k * ld + e, w);
        if (Wb) store_bf16x4(Wb + k * ld + e, w);
      }
      continue;
    }
    const long long e = 3 * n4 + i;
    const float mean = tree_sum<KT>([&](int k) { return W[k * ld + e]; }, K) / Kf;
    float w = ws[e], u = ug[e];
    gm_step(mean, w, u, mg, lr);
    ws[e] = w;
    ug[e] = u;
    for (int k = 0; k < K; ++k) {
      W[k * ld + e] = w;
      if (Wb) Wb[k * ld + e] = f32_to_bf16(w);
    }
  }
}

__global__ void k_broadcast(const float* src, float* W, bf16_t* Wb, int K,
                            long long n, long long ld, int replica) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    const float v = src[i];
    for (int k = 0; k < K; ++k) {
      if (replica >= 0 && k != replica) continue;
      W[k * ld + i] = v;
      if (Wb) Wb[k * ld + i] = f32_to_bf16(v);
    }
  }
}

__global__ void k_to_bf16(const float* x, bf16_t* y, long long n) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x)
    y[i] = f32_to_bf16(x[i]);
}

// rows x n floats from src (row pitch spitch) to dst (row pitch dpitch): the
// sections of the state blob against the padded replica rows (whose pitches
// differ by less than a vector, so most rows are unaligned on one side). Four
// floats per thread: 64 x 10.5M floats (5.4 GB moved) 1677 us at one each,
// now 852 us each (6.3 TB/s).
template <bool NT>
__global__ __launch_bounds__(256) void k_copy_rows(float* dst, long long dpitch, const float* src,
                                                   long long spitch, long long n) {
  // (parts of 2^23 workgroups on the grid's z axis)
  const long long e0 = 4 * ((((long long)blockIdx.z << 23) + blockIdx.x) * 256 + threadIdx.x);
  float* d = dst + blockIdx.y * dpitch;
  const float* q = src + blockIdx.y * spitch;
  if (e0 + 4 <= n) {
    st4<NT>(d + e0, ld4<NT>(q + e0));
  } else {
    for (long long e = e0; e < n; ++e) d[e] = q[e];
  }
}

__global__ void k_put_words(unsigned long long* dst, Words8 v) {
  if (threadIdx.x < 8) dst[threadIdx.x] = v.w[threadIdx.x];
}

__global__ void k_fill(float* x, float v, long long n) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x)
    x[i] = v;
}

// One element (or float4) per thread over the whole range: measured on the
// fused update at 1 GB, a full grid streams 15% faster than a grid capped at
// 16384 workgroups with grid-stride loops. An axis of the grid holds fewer than
// 2^32 threads (a longer one is cut short without an error): longer ranges fall
// back to the grid-stride loop the kernels keep.
int grid_for(long long n, int threads) {
  const long long b = (n + threads - 1) / threads, most = 0xffffffffLL / threads;
  return (int)(b < 1 ? 1 : b < most ? b : most);
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

}  // namespace

hipError_t launch_sample(uint64_t seed, int64_t step, int K, int64_t N, int B,
                         int32_t* idx, hipStream_t s) {
  const int groups = (B + 3) / 4;
  dim3 grid((groups + 63) / 64, K);
  hipLaunchKernelGGL(k_sample, grid, dim3(64), 0, s, (uint32_t)seed,
                     (uint32_t)(seed >> 32), (uint32_t)step,
                     (uint32_t)((uint64_t)step >> 32), K, (long long)N, B, idx);
  return hipGetLastError();
}

hipError_t launch_sample_epoch(uint64_t seed, int64_t step, int K, int64_t N,
                               int B, int32_t* idx, hipStream_t s) {
  const long long S = (N / K) / B;  // batches per worker and epoch
  if (S < 1 || N > 0x7fffffffLL) return hipErrorInvalidValue;
  int m = 1;
  while ((1LL << (2 * m)) < N) ++m;
  const long long e = step / S, j = step % S;
  dim3 grid((B + 63) / 64, K);
  hipLaunchKernelGGL(k_sample_epoch, grid, dim3(64), 0, s, (uint32_t)seed,
                     (uint32_t)(seed >> 32), (uint32_t)e, j, K, (long long)N, B,
                     m, idx);
  return hipGetLastError();
}

hipError_t launch_xent(const float* Z, const int32_t* y, const int32_t* idx,
                       int K, int B, int C, void* dZ, int dz_bf16, float* loss,
                       int* nonfinite, hipStream_t s) {
  hipLaunchKernelGGL(k_xent, dim3(K), dim3(256), 0, s, Z, y, idx, B, C, dZ,
                     dz_bf16, loss, nonfinite);
  return hipGetLastError();
}

hipError_t launch_sgd_update(float* W, float* U, const float* G, long long n,
                             float lr, float mom, float wd, int nesterov,
                             hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (n % 4 == 0 && aligned16(W) && aligned16(U) && aligned16(G))
    hipLaunchKernelGGL(k_sgd_update4, dim3(grid_for(n / 4, 256)), dim3(256), 0,
                       s, (float4*)W, (float4*)U, (const float4*)G, n / 4, lr,
                       mom, wd, nesterov);
  else
    hipLaunchKernelGGL(k_sgd_update1, dim3(grid_for(n, 256)), dim3(256), 0, s,
                       W, U, G, n, lr, mom, wd, nesterov);
  return hipGetLastError();
}

// The averages' instances: up to 16 replicas, and 32 and 64, with every load of
// an item in flight at once; other counts by blocks of eight, each waiting for
// the one before (32 rows of 100003: 6.6 us, by blocks 8.1; 64 of 1841162: 203
// against 216; 24 of 100003: 6.6 by blocks).
#define LSGD_FOR_REPLICAS(K, LAUNCH) \
  switch (K) {                       \
    case 1: LAUNCH(1); break;        \
    case 2: LAUNCH(2); break;        \
    case 3: LAUNCH(3); break;        \
    case 4: LAUNCH(4); break;        \
    case 5: LAUNCH(5); break;        \
    case 6: LAUNCH(6); break;        \
    case 7: LAUNCH(7); break;        \
    case 8: LAUNCH(8); break;        \
    case 9: LAUNCH(9); break;        \
    case 10: LAUNCH(10); break;      \
    case 11: LAUNCH(11); break;      \
    case 12: LAUNCH(12); break;      \
    case 13: LAUNCH(13); break;      \
    case 14: LAUNCH(14); break;      \
    case 15: LAUNCH(15); break;      \
    case 16: LAUNCH(16); break;      \
    case 32: LAUNCH(32); break;      \
    case 64: LAUNCH(64); break;      \
    default:                         \
      if (K < 128) {                 \
        LAUNCH(0);                   \
      } else {                       \
        LAUNCH(-1);                  \
      }                              \
  }

hipError_t launch_average_blocks(float* W, bf16_t* Wb, int Kb, int blocks,
                                 long long n, long long ld, float* mean_out,
                                 long long nt_bytes, hipStream_t s) {
  if (n <= 0 || Kb <= 0 || blocks <= 0) return hipSuccess;
  if (blocks > 65535 || (mean_out && blocks != 1)) return hipErrorInvalidValue;
  const int K = Kb;
  const bool nt = 4LL * K * blocks * n >= nt_bytes;
  const dim3 grid(grid_for(n / 4 + n % 4, 256), blocks), block(256);
#define LSGD_AVG(KK)                                                               \
  if (nt)                                                                          \
    hipLaunchKernelGGL((k_average4<KK, true>), grid, block, 0, s, W, Wb, K, n, ld, \
                       mean_out);                                                  \
  else                                                                             \
    hipLaunchKernelGGL((k_average4<KK, false>), grid, block, 0, s, W, Wb, K, n, ld, \
                       mean_out)
  LSGD_FOR_REPLICAS(K, LSGD_AVG)
#undef LSGD_AVG
  return hipGetLastError();
}

hipError_t launch_average(float* W, bf16_t* Wb, int K, long long n,
                          long long ld, float* mean_out, long long nt_bytes, hipStream_t s) {
  return launch_average_blocks(W, Wb, K, 1, n, ld, mean_out, nt_bytes, s);
}

hipError_t launch_average_gm(float* W, bf16_t* Wb, int K, long long n,
                             long long ld, float* ws, float* ug, float mg,
                             float lr, long long nt_bytes, hipStream_t s) {
  if (n <= 0 || K <= 0) return hipSuccess;
  const bool nt = 4LL * K * n >= nt_bytes;
  const dim3 grid(grid_for(n / 4 + n % 4, 256)), block(256);
#define LSGD_AVG_GM(KK)                                                                \
  if (nt)                                                                              \
    hipLaunchKernelGGL((k_average_gm4<KK, true>), grid, block, 0, s, W, Wb, K, n, ld,  \
                       ws, ug, mg, lr);                                                \
  else                                                                                 \
    hipLaunchKernelGGL((k_average_gm4<KK, false>), grid, block, 0, s, W, Wb, K, n, ld, \
                       ws, ug, mg, lr)
  LSGD_FOR_REPLICAS(K, LSGD_AVG_GM)
#undef LSGD_AVG_GM
  return hipGetLastError();
}

hipError_t launch_broadcast(const float* src, float* W, bf16_t* Wb, int K,
                            long long n, long long ld, int replica,
                            hipStream_t s) {
  hipLaunchKernelGGL(k_broadcast, dim3(grid_for(n, 256)), dim3(256), 0, s, src,
                     W, Wb, K, n, ld, replica);
  return hipGetLastError();
}

hipError_t launch_to_bf16(const float* x, bf16_t* y, long long n,
                          hipStream_t s) {
  hipLaunchKernelGGL(k_to_bf16, dim3(grid_for(n, 256)), dim3(256), 0, s, x, y,
                     n);
  return hipGetLastError();
}

hipError_t launch_copy_rows(float* dst, long long dpitch, const float* src,
                            long long spitch, long long n, int rows,
                            hipStream_t s) {
  if (rows <= 0 || n <= 0) return hipSuccess;
  if (rows > 65535) return hipErrorInvalidValue;
  const long long b = (n + 1023) / 1024, part = 1LL << 23;
  const dim3 grid((unsigned)(b < part ? b : part), rows, (unsigned)((b + part - 1) / part));
  if (8LL * rows * n >= kNtBytes)
    hipLaunchKernelGGL(k_copy_rows<true>, grid, dim3(256), 0, s, dst,
                       dpitch, src, spitch, n);
  else
    hipLaunchKernelGGL(k_copy_rows<false>, grid, dim3(256), 0, s, dst,
                       dpitch, src, spitch, n);
  return hipGetLastError();
}

hipError_t launch_put_words(void* dst, const Words8& v, hipStream_t s) {
  hipLaunchKernelGGL(k_put_words, dim3(1), dim3(64), 0, s,
                     (unsigned long long*)dst, v);
  return hipGetLastError();
}

hipError_t launch_fill(float* x, float v, long long n, hipStream_t s) {
  hipLaunchKernelGGL(k_fill, dim3(grid_for(n, 256)), dim3(256), 0, s, x, v, n);
  return hipGetLastError();
}

}  // namespace lsgd
