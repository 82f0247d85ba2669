// The output layer of the network with few classes (C <= 32), fused around
// the loss: the mean mini-batch cross-entropy whose gradient is the bracket of
// eq. 2 in the paper.
//
// k_head_fwd: one workgroup per few sample rows of a replica: its four waves
//   split the D inputs, then softmax cross-entropy (stable form), dZ = (p -
//   onehot)/B, and, below the top layer, the input gradient dA[d] = sum_c
//   dZ[c] W[d][c] masked by the ReLU derivative (A > 0).
// k_head_wgrad: one workgroup per (replica, 64 inputs d): dW[d][c] =
//   sum_b A[b][d] dZ[b][c], fused with the momentum-SGD update; workgroup 0 of
//   each replica also updates the bias (sum_b dZ[b][c]) and reduces the
//   per-row losses.
#include <type_traits>

#include "kernels.h"

namespace lsgd {
namespace {

template <typename T>
__device__ __forceinline__ float ld(const T* p, long long i);
template <>
__device__ __forceinline__ float ld<float>(const float* p, long long i) {
  return p[i];
}
template <>
__device__ __forceinline__ float ld<bf16_t>(const bf16_t* p, long long i) {
  return bf16_to_f32(p[i]);
}
__device__ __forceinline__ void st(float* p, long long i, float v) { p[i] = v; }
__device__ __forceinline__ void st(bf16_t* p, long long i, float v) {
  p[i] = f32_to_bf16(v);
}
__device__ __forceinline__ float round_like(float v, const float*) { return v; }
__device__ __forceinline__ float round_like(float v, const bf16_t*) {
  return bf16_to_f32(f32_to_bf16(v));
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

__device__ __forceinline__ void sgd_step(float& w, float& u, float grad,
                                         const HeadArgs& h) {
  const float g = __builtin_fmaf(h.wd, w, grad);
  u = __builtin_fmaf(h.mom, u, g);
  const float d = step_dir(u, g, h.mom, h.nesterov);
  w = __builtin_fmaf(-h.lr, d, w);
}

// The CM classes of one row of W_L from p on, in vector loads at any element
// alignment. Classes past the real count are whatever follows the row (the
// bias or padding lies behind the last one): the callers drop what they form
// from them.
typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x2_any __attribute__((ext_vector_type(2), aligned(2)));
template <int CM>
__device__ __forceinline__ void load_row(const float* p, float (&w)[CM]) {
#pragma unroll
  for (int c = 0; c < CM; c += 4) {
    const v4f_any t = *(const v4f_any*)(p + c);
#pragma unroll
    for (int e = 0; e < 4; ++e) w[c + e] = t[e];
  }
}
template <int CM>
__device__ __forceinline__ void load_row(const bf16_t* p, float (&w)[CM]) {
#pragma unroll
  for (int c = 0; c < CM; c += 4) {
    const u32x2_any t = *(const u32x2_any*)(p + c);
    w[c] = __uint_as_float(t.x << 16);
    w[c + 1] = __uint_as_float(t.x & 0xffff0000u);
    w[c + 2] = __uint_as_float(t.y << 16);
    w[c + 3] = __uint_as_float(t.y & 0xffff0000u);
  }
}

// Sums of v[0 .. N) over a wavefront (N / 32 whole): five exchanges that each
// halve what a lane keeps (lanes with the exchanged bit set keep the upper
// half), then one plain exchange; v[0 .. N/32) of lane l are the sums from
// index first(l) on. 31 N / 32 + N / 32 = N exchanges instead of the 6 N of a
// butterfly per value.
template <int N, int OFF>
__device__ __forceinline__ void scatter_sum(float* v, int lane, int& first) {
  if constexpr (OFF == 1) {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] += __shfl_xor(v[i], 1, 64);
  } else {
    const bool up = (lane & OFF) != 0;
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
      const float give = up ? v[i] : v[i + N / 2], keep = up ? v[i + N / 2] : v[i];
      v[i] = keep + __shfl_xor(give, OFF, 64);
    }
    if (up) first += N / 2;
    scatter_sum<N / 2, OFF / 2>(v, lane, first);
  }
}

// Rows per workgroup of k_head_fwd: R x CM partial logits per lane.
template <int CM>
constexpr int head_rows() { return CM <= 16 ? 8 : 4; }

// Logits, loss, dZ and the input gradient of R rows of replica k. The four
// waves take inputs d = 256 i + 64 wave + lane: a lane reads the rows' values
// and its row of W_L straight from memory, four strides in flight, and keeps R
// x CM partial logits; the waves' sums are added in order. Bound by the rows'
// bytes and, for small D, by its chain of three memory round trips. 3072
// gathered inputs, 16 x 128 rows, 10 classes: 50 us with W_L staged through
// LDS and two rows per wave, now 14.9 us; 5 x 50 rows of 100 inputs: 16
// us, now 8.5.
template <typename T, int CM, bool GATHER>
__global__ __launch_bounds__(256) void k_head_fwd(HeadArgs h) {
  constexpr int R = head_rows<CM>(), N = R * CM;
  constexpr int LPR = CM <= 16 ? 16 : 32;  // softmax lanes per row
  static_assert(N % 32 == 0 && R * LPR <= 256, "exchange and softmax shapes");
  __shared__ float zs[4][N];
  __shared__ __attribute__((aligned(16))) float dzs[N];
  const int k = blockIdx.y, row0 = blockIdx.x * R;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int D = h.D, C = h.C;
  const T* Wg = (const T*)h.W + (long long)k * h.sW;
  const T* arow[R];
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int row = min(row0 + q, h.B - 1);
    arow[q] = GATHER ? (const T*)h.A + (long long)h.rowmap[(long long)k * h.B + row] * D
                     : (const T*)h.A + (long long)k * h.sA + (long long)row * D;
  }
  // softmax thread t: row t / LPR, class t % LPR; its label on its way
  const int sq = (int)threadIdx.x / LPR, sc = (int)threadIdx.x % LPR;
  const bool smx = sq < R;
  const long long srr = (long long)k * h.B + min(row0 + sq, h.B - 1);
  const int lab = smx ? h.y[h.rowmap[srr]] : 0;
  const float bias = smx && sc < C ? h.bias[(long long)k * h.sBias + sc] : 0.f;

  float z[N];
#pragma unroll
  for (int i = 0; i < N; ++i) z[i] = 0.f;
  for (int d0 = wave * 64 + lane; d0 - lane < D; d0 += 1024) {
    float av[4][R], w[4][CM];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int d = min(d0 + 256 * u, D - 1);
      load_row<CM>(Wg + (long long)d * C, w[u]);
#pragma unroll
      for (int q = 0; q < R; ++q) av[u][q] = ld(arow[q], d);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool in = d0 + 256 * u < D;
#pragma unroll
      for (int q = 0; q < R; ++q) {
        const float x = in ? av[u][q] : 0.f;
#pragma unroll
        for (int c = 0; c < CM; ++c) {
          const float wc = in ? w[u][c] : 0.f;
          z[q * CM + c] = __builtin_fmaf(x, wc, z[q * CM + c]);
        }
      }
    }
  }
  int first = 0;
  scatter_sum<N, 32>(z, lane, first);
  if ((lane & 1) == 0) {
#pragma unroll
    for (int i = 0; i < N / 32; ++i) zs[wave][first + i] = z[i];
  }
  __syncthreads();
  if (smx) {  // whole wavefronts: R LPR is a multiple of 64
    float zc = -INFINITY;
    if (sc < C) {
      const int i = sq * CM + sc;
      zc = (((zs[0][i] + zs[1][i]) + zs[2][i]) + zs[3][i]) + bias;
    }
    float m = zc;
#pragma unroll
    for (int off = LPR / 2; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
    const float e = sc < C ? __expf(zc - m) : 0.f;
    float s = e, rest = sc != lab ? e : 0.f;
#pragma unroll
    for (int off = LPR / 2; off > 0; off >>= 1) {
      s += __shfl_xor(s, off, 64);
      rest += __shfl_xor(rest, off, 64);
    }
    const float zy = __shfl(zc, (lane & ~(LPR - 1)) + lab, 64);
    const float loss = zy >= m ? log1pf(rest) : (m - zy) + logf(s);
    const float p = e * (1.0f / s);
    const float dz =
        round_like((p - (sc == lab ? 1.f : 0.f)) * (1.0f / (float)h.B), (const T*)nullptr);
    if (row0 + sq < h.B) {
      if (sc < C) st((T*)h.dZ, srr * C + sc, dz);
      if (sc == 0) h.rowloss[srr] = loss;
    }
    if (sc < CM) dzs[sq * CM + sc] = sc < C ? dz : 0.f;
  }
  if (!h.dZprev) return;  // uniform over the workgroup
  __syncthreads();
  // input gradient, ReLU-masked: the rows and W_L again (from cache)
  float dz[N];
#pragma unroll
  for (int i = 0; i < N; i += 4) *(float4*)&dz[i] = *(const float4*)&dzs[i];
  T* out = (T*)h.dZprev + ((long long)k * h.B + row0) * D;
  for (int d = wave * 64 + lane; d < D; d += 256) {
    float w[CM], mk[R];
    load_row<CM>(Wg + (long long)d * C, w);
#pragma unroll
    for (int q = 0; q < R; ++q) mk[q] = h.nomask ? 1.f : ld(arow[q], d);
#pragma unroll
    for (int c = 0; c < CM; ++c)
      if (c >= C) w[c] = 0.f;
#pragma unroll
    for (int q = 0; q < R; ++q) {
      float v = 0.f;
#pragma unroll
      for (int c = 0; c < CM; ++c) v = __builtin_fmaf(dz[q * CM + c], w[c], v);
      if (row0 + q < h.B) st(out, (long long)q * D + d, mk[q] > 0.f ? v : 0.f);
    }
  }
}

// Weight gradient of the output layer and its update: workgroup (x, k) owns
// inputs d = 64 x .. 64 x + 63 of replica k (lane d), its four waves the batch
// rows grp, grp + 4, ... Per 128 rows, the 32 activations of each thread and dZ
// (zero-padded to CM classes, in LDS) are loaded at once; this slice of W_L and
// U_L is on its way from the start. A row of dZ is read as CM / 4 broadcast
// float4; the waves' partials are added in order and the SGD step applied.
// Workgroup 0 of each replica also updates the bias and reduces the loss.
// 3072 gathered inputs, 16 x 128 rows, 10 classes (floor 5 us for the rows):
// 21 us with a class loop of runtime length, now 12.0 us.
template <typename T, int CM, bool GATHER>
__global__ __launch_bounds__(256) void k_head_wgrad(HeadArgs h) {
  constexpr int RPG = 32, RB = 4 * RPG;       // rows per wave / workgroup and pass
  constexpr int WPT = (64 * CM + 255) / 256;  // weights per thread
  constexpr int ZPT = RB * CM / 256;          // dZ values per thread and pass
  __shared__ __attribute__((aligned(16))) float dzs[RB * CM];
  __shared__ float part[4][64][CM + 1];
  __shared__ float red[256];
  const int k = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  const int grp = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int D = h.D, C = h.C, B = h.B;
  const int dbase = blockIdx.x * 64, d = min(dbase + lane, D - 1);
  const int nw = min(64, D - dbase) * C;  // this slice's weights
  const bool first = blockIdx.x == 0;
  const T* dZ = (const T*)h.dZ + (long long)k * B * C;
  const long long wbase = (long long)k * h.sP + (long long)dbase * C;
  float wv[WPT], uv[WPT];
#pragma unroll
  for (int q = 0; q < WPT; ++q) {
    const int e = min(tid + 256 * q, nw - 1);
    wv[q] = h.Wsrc[(long long)k * h.sSrc + (long long)dbase * C + e];
    uv[q] = h.Um[wbase + e];
  }
  float rl = 0.f;  // per-row losses: strided partial sums, then a fixed tree
  if (first)
    for (int b = tid; b < B; b += 256) rl += h.rowloss[(long long)k * B + b];

  float acc[CM];
#pragma unroll
  for (int c = 0; c < CM; ++c) acc[c] = 0.f;
  float bsum = 0.f;  // bias gradient of class tid (first workgroup)
  for (int b0 = 0; b0 < B; b0 += RB) {
    const int nb = min(RB, B - b0);
    float av[RPG], zv[ZPT];
#pragma unroll
    for (int r = 0; r < RPG; ++r) {
      const int b = b0 + min(grp + 4 * r, nb - 1);
      const long long row = GATHER ? (long long)h.rowmap[(long long)k * B + b] * D
                                   : (long long)k * h.sA + (long long)b * D;
      av[r] = ld((const T*)h.A, row + d);
    }
#pragma unroll
    for (int q = 0; q < ZPT; ++q) {
      const int i = tid + 256 * q, b = i / CM, c = i - b * CM;
      zv[q] = b < nb && c < C ? ld(dZ, (long long)(b0 + b) * C + c) : 0.f;
    }
    if (b0) __syncthreads();  // the previous pass's dZ is no longer read
#pragma unroll
    for (int q = 0; q < ZPT; ++q) dzs[tid + 256 * q] = zv[q];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RPG; ++r) {
      if (grp + 4 * r >= nb) break;  // uniform over the wave
      const float* zr = dzs + (grp + 4 * r) * CM;
#pragma unroll
      for (int c = 0; c < CM; c += 4) {
        const float4 z4 = *(const float4*)(zr + c);
        acc[c] = __builtin_fmaf(av[r], z4.x, acc[c]);
        acc[c + 1] = __builtin_fmaf(av[r], z4.y, acc[c + 1]);
        acc[c + 2] = __builtin_fmaf(av[r], z4.z, acc[c + 2]);
        acc[c + 3] = __builtin_fmaf(av[r], z4.w, acc[c + 3]);
      }
    }
    if (first && tid < C) {
#pragma unroll 8
      for (int b = 0; b < nb; ++b) bsum += dzs[b * CM + tid];
    }
  }
#pragma unroll
  for (int c = 0; c < CM; ++c) part[grp][lane][c] = acc[c];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < WPT; ++q) {
    const int e = tid + 256 * q;
    if (e < nw) {
      const int dl = e / C, c = e - dl * C;
      const float g = ((part[0][dl][c] + part[1][dl][c]) + part[2][dl][c]) + part[3][dl][c];
      float w = wv[q], u = uv[q];
      sgd_step(w, u, g, h);
      h.Wm[wbase + e] = w;
      h.Um[wbase + e] = u;
      if (h.Wb) h.Wb[wbase + e] = f32_to_bf16(w);
    }
  }
  if (!first) return;  // uniform over the workgroup
  if (tid < C) {
    const long long o = (long long)k * h.sP + tid;
    float w = h.bsrc[(long long)k * h.sSrc + tid], u = h.bias_u[o];
    sgd_step(w, u, bsum, h);
    h.bias_w[o] = w;
    h.bias_u[o] = u;
  }
  red[tid] = rl;
  __syncthreads();
  for (int w2 = 128; w2 > 0; w2 >>= 1) {
    if (tid < w2) red[tid] += red[tid + w2];
    __syncthreads();
  }
  if (tid == 0) {
    const float mean = red[0] / (float)B;
    if (h.loss) h.loss[k] = mean;
    // a non-finite loss raises the context's flag (a plain store: every
    // writer stores the same value)
    if (h.nonfinite && !isfinite(mean)) *h.nonfinite = 1;
  }
}

// Register-resident variant for fp32, a class count fixed at compile time,
// D % 256 == 0 and D <= 512: lane l
// owns inputs d = 256 j + 4 l .. +3 (j < D / 256) of two sample rows and the
// matching rows W_L[d][0..C-1]; all of them are loaded in one batch, so the
// logits, the loss, dZ and the masked input gradient cost one memory round
// trip. The loss and gradient formulas are those of k_head_fwd; only the
// split of the logit sums over lanes differs (each lane's inputs in ascending
// d, then an xor butterfly).
template <int C, int NJ>
__global__ __launch_bounds__(256) void k_head_fwd_vec(HeadArgs h) {
  constexpr int RPW = 2;
  const int k = blockIdx.y;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int D = h.D;
  const float* Wg = (const float*)h.W + (long long)k * h.sW;
  long long rr[RPW];
  bool live[RPW];
  float4 a[RPW][NJ];
#pragma unroll
  for (int q = 0; q < RPW; ++q) {
    const int row = (blockIdx.x * 4 + wave) * RPW + q;
    live[q] = row < h.B;
    rr[q] = (long long)k * h.B + (live[q] ? row : 0);
    const float* arow = (const float*)h.A + (long long)k * h.sA +
                        (long long)(live[q] ? row : 0) * D;
#pragma unroll
    for (int j = 0; j < NJ; ++j) a[q][j] = *(const float4*)(arow + 256 * j + 4 * lane);
  }
  // W rows d .. d+3 are 4*C consecutive floats (C float4 when C is even)
  static_assert(C % 2 == 0 && C <= 16, "class count");
  float wr[NJ][4 * C];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const float* wp = Wg + (long long)(256 * j + 4 * lane) * C;
#pragma unroll
    for (int v = 0; v < C; ++v) {
      const float4 t = *(const float4*)(wp + 4 * v);
      wr[j][4 * v] = t.x;
      wr[j][4 * v + 1] = t.y;
      wr[j][4 * v + 2] = t.z;
      wr[j][4 * v + 3] = t.w;
    }
  }
  float z[RPW][C];
#pragma unroll
  for (int q = 0; q < RPW; ++q)
#pragma unroll
    for (int c = 0; c < C; ++c) {
      float acc = 0.f;
      {
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          acc = __builtin_fmaf(a[q][j].x, wr[j][0 * C + c], acc);
          acc = __builtin_fmaf(a[q][j].y, wr[j][1 * C + c], acc);
          acc = __builtin_fmaf(a[q][j].z, wr[j][2 * C + c], acc);
          acc = __builtin_fmaf(a[q][j].w, wr[j][3 * C + c], acc);
        }
      }
      z[q][c] = acc;
    }
  const float* bias = h.bias + (long long)k * h.sBias;
  const float invB = 1.0f / (float)h.B;
  float dz[RPW][C];
#pragma unroll
  for (int q = 0; q < RPW; ++q) {
#pragma unroll
    for (int c = 0; c < C; ++c)
      z[q][c] = wave_sum(z[q][c]) + bias[c];
    const int lab = h.y[h.rowmap[rr[q]]];
    float m = z[q][0];
#pragma unroll
    for (int c = 1; c < C; ++c)
      m = fmaxf(m, z[q][c]);
    float sum = 0.f, rest = 0.f, zy = 0.f;
#pragma unroll
    for (int c = 0; c < C; ++c)
      {
        const float e = __expf(z[q][c] - m);
        sum += e;
        if (c != lab) rest += e;
        else zy = z[q][c];
      }
    const float loss = zy >= m ? log1pf(rest) : (m - zy) + logf(sum);
    const float inv_s = 1.0f / sum;
    float mine = 0.f;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      dz[q][c] = 0.f;
      {
        const float p = __expf(z[q][c] - m) * inv_s;
        dz[q][c] = (p - (c == lab ? 1.f : 0.f)) * invB;
        if (c == lane) mine = dz[q][c];
      }
    }
    if (live[q]) {
      if (lane < C) ((float*)h.dZ)[rr[q] * C + lane] = mine;
      if (lane == 0) h.rowloss[rr[q]] = loss;
    }
  }
  if (!h.dZprev) return;
#pragma unroll
  for (int q = 0; q < RPW; ++q) {
    if (!live[q]) continue;
    float* out = (float*)h.dZprev + rr[q] * D;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float acc = 0.f;
#pragma unroll
        for (int c = 0; c < C; ++c)
          acc = __builtin_fmaf(dz[q][c], wr[j][e * C + c], acc);
        v[e] = acc;
      }
      const float4 av = a[q][j];
      float4 o;
      o.x = (h.nomask || av.x > 0.f) ? v[0] : 0.f;
      o.y = (h.nomask || av.y > 0.f) ? v[1] : 0.f;
      o.z = (h.nomask || av.z > 0.f) ? v[2] : 0.f;
      o.w = (h.nomask || av.w > 0.f) ? v[3] : 0.f;
      *(float4*)(out + 256 * j + 4 * lane) = o;
    }
  }
}

// bf16 form: the bf16 copy of W_L and bf16 activations, a class count C
// fixed at compile time and D = 512 NJ. The replica's W_L ([D][C] bf16, D C / 8
// 16-byte words) is copied into LDS unchanged, every word loaded before the
// first is stored; lane l of a wave owns inputs d = 512 j + 8 l .. +7 of two
// sample rows, loaded in the same batch. The logits, the loss, dZ and the
// masked input gradient then need no further global read. Formulas and
// rounding points (dZ and the input gradient rounded to bf16) are those of
// k_head_fwd; each lane adds its inputs in ascending d before the xor
// butterfly.
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) {
  return __uint_as_float(w & 0xFFFF0000u);
}
__device__ __forceinline__ float bf16_at(const uint4& v, int e) {
  const uint32_t w = e < 2 ? v.x : (e < 4 ? v.y : (e < 6 ? v.z : v.w));
  return (e & 1) ? bf16_hi(w) : bf16_lo(w);
}

template <int C, int NJ>
__global__ __launch_bounds__(256) void k_head_fwd_bf16(HeadArgs h) {
  constexpr int RPW = 2;
  constexpr int D = 512 * NJ;
  constexpr int WV = D * C / 8;            // 16-byte words of W_L
  constexpr int WPT = (WV + 255) / 256;    // per thread
  __shared__ uint4 Ws[WV];
  const int k = blockIdx.y;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const uint4* Wg = (const uint4*)((const bf16_t*)h.W + (long long)k * h.sW);
  uint4 wv[WPT];
#pragma unroll
  for (int u = 0; u < WPT; ++u) {
    const int i = u * 256 + (int)threadIdx.x;
    wv[u] = i < WV ? Wg[i] : make_uint4(0u, 0u, 0u, 0u);
  }
  long long rr[RPW];
  bool live[RPW];
  uint4 a[RPW][NJ];
#pragma unroll
  for (int q = 0; q < RPW; ++q) {
    const int row = (blockIdx.x * 4 + wave) * RPW + q;
    live[q] = row < h.B;
    rr[q] = (long long)k * h.B + (live[q] ? row : 0);
    const bf16_t* arow = (const bf16_t*)h.A + (long long)k * h.sA +
                         (long long)(live[q] ? row : 0) * D;
#pragma unroll
    for (int j = 0; j < NJ; ++j) a[q][j] = *(const uint4*)(arow + 512 * j + 8 * lane);
  }
#pragma unroll
  for (int u = 0; u < WPT; ++u) {
    const int i = u * 256 + (int)threadIdx.x;
    if (i < WV) Ws[i] = wv[u];
  }
  __syncthreads();
  // W_L[d][c] for the lane's d = 512 j + 8 l + t: element t C + c of the C
  // words starting at word (64 j + l) C
  float z[RPW][C];
#pragma unroll
  for (int q = 0; q < RPW; ++q)
#pragma unroll
    for (int c = 0; c < C; ++c) z[q][c] = 0.f;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    uint4 w[C];
#pragma unroll
    for (int v = 0; v < C; ++v) w[v] = Ws[(64 * j + lane) * C + v];
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
      for (int c = 0; c < C; ++c) {
        const int e = t * C + c;
        const float wdc = bf16_at(w[e / 8], e % 8);
#pragma unroll
        for (int q = 0; q < RPW; ++q)
          z[q][c] = __builtin_fmaf(bf16_at(a[q][j], t), wdc, z[q][c]);
      }
    __builtin_amdgcn_sched_barrier(0);  // one slice of W_L in registers at a time
  }
  const float* bias = h.bias + (long long)k * h.sBias;
  const float invB = 1.0f / (float)h.B;
  float dz[RPW][C];
#pragma unroll
  for (int q = 0; q < RPW; ++q) {
#pragma unroll
    for (int c = 0; c < C; ++c) z[q][c] = wave_sum(z[q][c]) + bias[c];
    const int lab = h.y[h.rowmap[rr[q]]];
    float m = z[q][0];
#pragma unroll
    for (int c = 1; c < C; ++c) m = fmaxf(m, z[q][c]);
    float sum = 0.f, rest = 0.f, zy = 0.f;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const float e = __expf(z[q][c] - m);
      sum += e;
      if (c != lab) rest += e;
      else zy = z[q][c];
    }
    const float loss = zy >= m ? log1pf(rest) : (m - zy) + logf(sum);
    const float inv_s = 1.0f / sum;
    float mine = 0.f;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const float p = __expf(z[q][c] - m) * inv_s;
      dz[q][c] = round_like((p - (c == lab ? 1.f : 0.f)) * invB, (const bf16_t*)nullptr);
      if (c == lane) mine = dz[q][c];
    }
    if (live[q]) {
      if (lane < C) ((bf16_t*)h.dZ)[rr[q] * C + lane] = f32_to_bf16(mine);
      if (lane == 0) h.rowloss[rr[q]] = loss;
    }
  }
  if (!h.dZprev) return;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    uint4 w[C];
#pragma unroll
    for (int v = 0; v < C; ++v) w[v] = Ws[(64 * j + lane) * C + v];
#pragma unroll
    for (int q = 0; q < RPW; ++q) {
      if (!live[q]) continue;
      uint32_t o[4];
#pragma unroll
      for (int t2 = 0; t2 < 4; ++t2) {
        uint32_t pair = 0u;
#pragma unroll
        for (int hb = 0; hb < 2; ++hb) {
          const int t = 2 * t2 + hb;
          float acc = 0.f;
#pragma unroll
          for (int c = 0; c < C; ++c) {
            const int e = t * C + c;
            acc = __builtin_fmaf(dz[q][c], bf16_at(w[e / 8], e % 8), acc);
          }
          const float out = (h.nomask || bf16_at(a[q][j], t) > 0.f) ? acc : 0.f;
          pair |= (uint32_t)f32_to_bf16(out) << (16 * hb);
        }
        o[t2] = pair;
      }
      *(uint4*)((bf16_t*)h.dZprev + rr[q] * D + 512 * j + 8 * lane) =
          make_uint4(o[0], o[1], o[2], o[3]);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

template <typename T, int CM>
hipError_t launch_pair(const HeadArgs& h, hipStream_t s, int which) {
  const bool gather = h.gather != 0;  // the top layer is layer 1
  if (which == 0) {
    dim3 grid((h.B + head_rows<CM>() - 1) / head_rows<CM>(), h.K);
    if (gather)
      hipLaunchKernelGGL((k_head_fwd<T, CM, true>), grid, dim3(256), 0, s, h);
    else
      hipLaunchKernelGGL((k_head_fwd<T, CM, false>), grid, dim3(256), 0, s, h);
  } else {
    // (behind hidden layers gemm_update has this layer with the others; only
    // ResNet-20's, in fp32, comes here)
    dim3 grid((h.D + 63) / 64, h.K);
    if (gather)
      hipLaunchKernelGGL((k_head_wgrad<T, CM, true>), grid, dim3(256), 0, s, h);
    else if constexpr (std::is_same_v<T, float>)
      hipLaunchKernelGGL((k_head_wgrad<T, CM, false>), grid, dim3(256), 0, s, h);
    else
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// the smallest instance with room for C classes
template <typename T>
hipError_t launch_any(const HeadArgs& h, hipStream_t s, int which) {
  if (h.C <= 12) return launch_pair<T, 12>(h, s, which);
  if (h.C <= 16) return launch_pair<T, 16>(h, s, which);
  return launch_pair<T, 32>(h, s, which);
}

bool al16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

hipError_t launch_head(int dtype, const HeadArgs& h, hipStream_t s, int which) {
  if (h.C < 1 || h.C > kHeadMaxClasses) return hipErrorInvalidValue;
  if (h.K > 65535 || h.B < 1 || h.D < 1) return hipErrorInvalidValue;
  // register-resident forward when the shapes and alignment allow it
  if (which == 0 && dtype == 0 && !h.gather && h.C == 10 && h.D % 256 == 0 &&
      h.D <= 512 && h.sA % 4 == 0 && h.sW % 4 == 0 && al16(h.A) && al16(h.W) &&
      (h.dZprev == nullptr || al16(h.dZprev))) {
    dim3 grid((h.B + 7) / 8, h.K);
    if (h.D == 256)
      hipLaunchKernelGGL((k_head_fwd_vec<10, 1>), grid, dim3(256), 0, s, h);
    else
      hipLaunchKernelGGL((k_head_fwd_vec<10, 2>), grid, dim3(256), 0, s, h);
    return hipGetLastError();
  }
  // the same for bf16 operands, D a multiple of 512 up to 2048
  if (which == 0 && dtype == 1 && !h.gather && h.C == 10 && h.D % 512 == 0 &&
      h.D <= 2048 && h.sA % 8 == 0 && h.sW % 8 == 0 && al16(h.A) && al16(h.W) &&
      (h.dZprev == nullptr || al16(h.dZprev))) {
    dim3 grid((h.B + 7) / 8, h.K);
    switch (h.D / 512) {
      case 1: hipLaunchKernelGGL((k_head_fwd_bf16<10, 1>), grid, dim3(256), 0, s, h); break;
      case 2: hipLaunchKernelGGL((k_head_fwd_bf16<10, 2>), grid, dim3(256), 0, s, h); break;
      case 3: hipLaunchKernelGGL((k_head_fwd_bf16<10, 3>), grid, dim3(256), 0, s, h); break;
      default: hipLaunchKernelGGL((k_head_fwd_bf16<10, 4>), grid, dim3(256), 0, s, h); break;
    }
    return hipGetLastError();
  }
  return dtype == 1 ? launch_any<bf16_t>(h, s, which) : launch_any<float>(h, s, which);
}

}  // namespace

hipError_t launch_head_fwd(int dtype, const HeadArgs& h, hipStream_t s) {
  return launch_head(dtype, h, s, 0);
}
hipError_t launch_head_wgrad(int dtype, const HeadArgs& h, hipStream_t s) {
  return launch_head(dtype, h, s, 1);
}

}  // namespace lsgd
