// Grouped (replica-batched) GEMM on the gfx950 matrix cores.
//
// Each of the G groups is one replica's layer contraction of the gradient in
// eq. 2 of the paper: forward Z = A W (+ bias, ReLU), the input gradient
// dA = dZ W^T (masked by the ReLU derivative), and the weight gradient
// G = A^T dZ, whose epilogue applies the local momentum-SGD update directly so
// the gradient never goes to memory; the same kernel sums dZ over the batch
// for the bias gradient and updates the bias.
//
// Every product runs on v_mfma_f32_32x32x16_bf16. bf16 operands feed it as
// they are. An fp32 operand x is taken as three bf16 pieces, x = x1 + x2 + x3
// (each the round-to-nearest bf16 of what the ones before leave, so the sum is
// exact: 3 x 8 significant bits), and x y as the six products x1 y1, x1 y2,
// x2 y1, x2 y2, x1 y3, x3 y1, each exact in fp32; the three left out are below
// 2^-26 |x y| together. x1 y1 has an accumulator of its own and the five small
// ones share another, added at the end: a k range of 16 then rounds once at the
// sum's own magnitude where v_mfma_f32_32x32x2f32 rounds 16 times. Measured
// against fp64 (normwise, normal operands, K = 64 / 512 / 3072): 5.0e-8 /
// 1.3e-7 / 3.4e-7, the fp32 instruction 1.4e-7 / 4.0e-7 / 1.0e-6; the six
// products issue at 290 TFLOP/s, the fp32 instruction at 122.
// Infinities: x1 of an infinity (or of a finite value that rounds to one)
// leaves NaN pieces, so a wave whose result holds any NaN forms its tile again
// with the fp32 instruction and keeps that.
//
// Work distribution: a 1-D grid of G * S * tilesM * tilesN workgroups. The
// hardware deals consecutive workgroup ids round-robin to the 8 XCDs (each
// with its own L2), so the id is remapped to give every XCD a contiguous range
// of tiles: the tiles of one replica then share that XCD's L2.
// Split-K (S > 1) gives skinny GEMMs enough workgroups: split s covers K range
// [s*kchunk, (s+1)*kchunk) and writes a raw fp32 partial; a second kernel sums
// the S partials in ascending s and applies the epilogue.
#include <type_traits>

#include "kernels.h"

namespace lsgd {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
// four elements at any element's alignment (one global load)
typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x2_any __attribute__((ext_vector_type(2), aligned(2)));

constexpr int kThreads = 256;
constexpr int kXcds = 8;

struct Tile {
  int g, s, m0, n0;
};

__device__ __forceinline__ Tile decode_tile(const GemmArgs& a, int BM, int BN) {
  const int tn = (a.N + BN - 1) / BN, tm = (a.M + BM - 1) / BM;
  const int per_split = tn * tm, per_g = per_split * a.splits;
  const int total = per_g * a.G;
  const int p = blockIdx.x;
  int l = (total % kXcds == 0) ? (p % kXcds) * (total / kXcds) + p / kXcds : p;
  Tile t;
  t.g = l / per_g;
  l -= t.g * per_g;
  t.s = l / per_split;
  l -= t.s * per_split;
  t.m0 = (l / tn) * BM;
  t.n0 = (l % tn) * BN;
  return t;
}

__device__ __forceinline__ void sgd_step(float& w, float& u, float grad,
                                         const GemmArgs& a) {
  const float g = __builtin_fmaf(a.wd, w, grad);
  u = __builtin_fmaf(a.mom, u, g);
  const float d = step_dir(u, g, a.mom, a.nesterov);
  w = __builtin_fmaf(-a.lr, d, w);
}

// Epilogue applied to a finished value of C[g][m][n] (split-K's second
// kernel). OUTBF: activations are bf16 (bf16 workloads) and so are the mask
// operand and the output.
template <int EPI, bool OUTBF>
__device__ __forceinline__ void finish(const GemmArgs& a, int g, int m, int n,
                                       float v) {
  const long long o = (long long)g * a.sC + (long long)m * a.ldc + n;
  if constexpr (EPI == EPI_BIAS || EPI == EPI_BIAS_RELU)
    v += a.bias[(long long)g * a.sBias + n];
  if constexpr (EPI == EPI_BIAS_RELU) v = v > 0.f ? v : 0.f;
  if constexpr (EPI == EPI_RELU_MASK) {
    const float mk = OUTBF ? bf16_to_f32(((const bf16_t*)a.mask)[o])
                           : ((const float*)a.mask)[o];
    v = mk > 0.f ? v : 0.f;
  }
  if constexpr (OUTBF)
    ((bf16_t*)a.C)[o] = f32_to_bf16(v);
  else
    ((float*)a.C)[o] = v;
}

// Bias of the weight-gradient workgroups with m0 == 0: db[n] = sum_b dZ[b][n],
// then the same update as the weights.
__device__ __forceinline__ void bias_update(const GemmArgs& a, int g, int n, float colsum) {
  const long long o = (long long)g * a.sBiasP + n;
  float w = a.bias_src ? a.bias_src[(long long)g * a.sBiasSrc + n] : a.bias_w[o];
  float u = a.bias_u[o];
  sgd_step(w, u, colsum, a);
  a.bias_w[o] = w;
  a.bias_u[o] = u;
}

// ------------------------------------------------------------ operand pieces
// Two fp32 values as packed bf16 pairs p[0] + p[1] + p[2] (see the top).
__device__ __forceinline__ void split3(float x, float y, uint32_t (&p)[3]) {
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    p[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(v2f{x, y}, bf16x2));
    x -= __uint_as_float(p[i] << 16);
    y -= __uint_as_float(p[i] & 0xffff0000u);
  }
}

// Four consecutive elements of an operand as loaded, and their bf16 planes.
template <bool BF>
struct Quad;
template <>
struct Quad<false> {
  using E = float;
  static constexpr int kPlanes = 3;
  v4f v;
  __device__ __forceinline__ void load(const E* p) { v = *(const v4f_any*)p; }
  __device__ __forceinline__ void set(int e, const E* p, bool ok) { v[e] = ok ? *p : 0.f; }
  __device__ __forceinline__ void zero() { v = v4f{0.f, 0.f, 0.f, 0.f}; }
  __device__ __forceinline__ void planes(u32x2 (&q)[3]) const {
    uint32_t a[3], b[3];
    split3(v[0], v[1], a);
    split3(v[2], v[3], b);
#pragma unroll
    for (int i = 0; i < 3; ++i) q[i] = u32x2{a[i], b[i]};
  }
  __device__ __forceinline__ v4f f32() const { return v; }
};
template <>
struct Quad<true> {
  using E = bf16_t;
  static constexpr int kPlanes = 1;
  u32x2 v;
  __device__ __forceinline__ void load(const E* p) { v = *(const u32x2_any*)p; }
  __device__ __forceinline__ void set(int e, const E* p, bool ok) {
    const uint32_t h = ok ? *p : 0u;
    uint32_t w = e < 2 ? v.x : v.y;
    w = (e & 1) ? (w & 0xffffu) | (h << 16) : (w & 0xffff0000u) | h;
    if (e < 2)
      v.x = w;
    else
      v.y = w;
  }
  __device__ __forceinline__ void zero() { v = u32x2{0u, 0u}; }
  __device__ __forceinline__ void planes(u32x2 (&q)[1]) const { q[0] = v; }
  __device__ __forceinline__ v4f f32() const {
    return v4f{__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u),
               __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xffff0000u)};
  }
};

// ------------------------------------------------------------------ the GEMM
// Block tile BM x BN, K slabs of BK, 4 wavefronts in a 2 x 2 layout, each
// owning (BM/2) x (BN/2) as 32 x 32 MFMA blocks (lane l takes 8 k from
// 8 (l / 32) of row / column l % 32; accumulator v of lane l is
// C[8 (v/4) + 4 (l/32) + v%4][l%32]). Operands go global -> registers -> bf16
// planes in a double-buffered LDS ring; D register sets, so D slabs' loads
// are in flight while one computes. An operand stored with k contiguous lies
// in LDS as [row][k] (16-byte fragment reads; a pitch of BK + 8 spreads eight
// rows over all banks); one stored with k as the slow index lies as [k][column]
// -- no transposition on the way in -- and is read with ds_read_b64_tr_b16,
// which gives each lane of 16 its column's four k from a 4 x 16 block (pitch
// + 64 bytes: four rows of a block in disjoint banks).
// FULL: whole tiles and whole slabs (checked at launch). Otherwise rows past
// the end are clamped, and slabs or tiles that reach past K or past the
// columns of a k-slow operand take element loads (a uniform branch).
template <bool BF, bool AT, bool BT, int EPI, bool GATHER, int BM, int BN, int BK, int D,
          bool FULL>
__global__ __launch_bounds__(kThreads, BM * BN > 128 * 64 ? 1 : 2) void gemm_mm(GemmArgs a) {
  using Q = Quad<BF>;
  using E = typename Q::E;
  constexpr int NPL = Q::kPlanes;
  constexpr int WM = BM / 2, WN = BN / 2, FM = WM / 32, FN = WN / 32;
  constexpr bool AK = !AT, BKc = BT;  // k contiguous in storage
  constexpr int PA = AK ? BK + 8 : BM + 32, PB = BKc ? BK + 8 : BN + 32;
  constexpr int SA = (AK ? BM : BK) * PA, SB = (BKc ? BN : BK) * PB;  // one plane
  constexpr int NA = BM * BK / 4 / kThreads, NB = BN * BK / 4 / kThreads;
  static_assert(NA >= 1 && NB >= 1 && D % 2 == 0, "tile too small");
  __shared__ __attribute__((aligned(16))) bf16_t sA[2 * NPL * SA];
  __shared__ __attribute__((aligned(16))) bf16_t sB[2 * NPL * SB];
  constexpr bool kRows = AT && GATHER;  // the k rows of A come from a row map
  __shared__ int32_t srmap[kRows ? 512 : 1];  // beyond: read the map itself

  const Tile t = decode_tile(a, BM, BN);
  const int g = t.g, m0 = t.m0, n0 = t.n0;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lk = lane >> 5, lr = lane & 31;
  const int wm0 = (wave >> 1) * WM, wn0 = (wave & 1) * WN;
  const E* A = (const E*)a.A + (long long)g * a.sA;
  const E* B = (const E*)a.B + (long long)g * a.sB;
  const int32_t* rmap = GATHER ? a.rowmap + (long long)g * a.sRow : nullptr;
  const int M = a.M, N = a.N;
  const int kbeg = t.s * a.kchunk, kend = min(a.Kd, kbeg + a.kchunk);
  const int nk = (kend - kbeg + BK - 1) / BK;

  // EPI_SGD: the tile's W and U, in accumulator layout, on their way while
  // the k loop runs (clamped where the tile ends)
  constexpr bool kUpd = EPI == EPI_SGD;
  float wv[kUpd ? FM : 1][kUpd ? FN : 1][16], uv[kUpd ? FM : 1][kUpd ? FN : 1][16];
  auto out_row = [&](int i, int v) __attribute__((always_inline)) {
    return m0 + wm0 + i * 32 + (v >> 2) * 8 + lk * 4 + (v & 3);
  };
  if constexpr (kUpd) {
    const float* Wr = a.Wsrc ? a.Wsrc + (long long)g * a.sWsrc : a.W + (long long)g * a.sC;
    const float* Ur = a.U + (long long)g * a.sC;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          int m = out_row(i, v), n = n0 + wn0 + j * 32 + lr;
          if constexpr (!FULL) {
            m = min(m, M - 1);
            n = min(n, N - 1);
          }
          const long long o = (long long)m * a.ldc + n;
          wv[i][j][v] = Wr[o];
          uv[i][j][v] = Ur[o];
        }
  }

  if constexpr (kRows) {
    for (int i = tid; i < 512 && kbeg + i < kend; i += kThreads) srmap[i] = rmap[kbeg + i];
    __syncthreads();
  }
  // per quad of this thread: the storage offset that does not depend on k
  long long offA[NA], offB[NB];
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    const int q = tid + i * kThreads;
    if constexpr (AK) {
      int r = m0 + q / (BK / 4);
      if constexpr (!FULL) r = min(r, M - 1);
      offA[i] = (GATHER ? (long long)rmap[r] : (long long)r) * a.lda + (q % (BK / 4)) * 4;
    } else {
      offA[i] = m0 + (q % (BM / 4)) * 4;
    }
  }
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int q = tid + i * kThreads;
    if constexpr (BKc) {
      int r = n0 + q / (BK / 4);
      if constexpr (!FULL) r = min(r, N - 1);
      offB[i] = (long long)r * a.ldb + (q % (BK / 4)) * 4;
    } else {
      offB[i] = n0 + (q % (BN / 4)) * 4;
    }
  }
  auto arow = [&](int k) __attribute__((always_inline)) {  // storage row of A's k
    if constexpr (kRows) return (long long)(k - kbeg < 512 ? srmap[k - kbeg] : rmap[k]);
    return (long long)k;
  };
  auto gload = [&](int k0, Q(&xa)[NA], Q(&xb)[NB]) __attribute__((always_inline)) {
    const bool ktail = !FULL && k0 + BK > kend;
    if (ktail || (!FULL && !AK && m0 + BM > M)) {
#pragma unroll
      for (int i = 0; i < NA; ++i) {
        const int q = tid + i * kThreads;
        xa[i].zero();
        if constexpr (AK) {
          const int k = k0 + (q % (BK / 4)) * 4;
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (k + e < kend) xa[i].set(e, A + offA[i] + k0 + e, true);
        } else {
          const int k = k0 + q / (BM / 4);
          if (k < kend) {
            const E* p = A + arow(k) * a.lda;
#pragma unroll
            for (int e = 0; e < 4; ++e)
              xa[i].set(e, p + min((int)offA[i] + e, M - 1), true);
          }
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < NA; ++i) {
        if constexpr (AK)
          xa[i].load(A + offA[i] + k0);
        else
          xa[i].load(A + arow(k0 + (tid + i * kThreads) / (BM / 4)) * a.lda + offA[i]);
      }
    }
    if (ktail || (!FULL && !BKc && n0 + BN > N)) {
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const int q = tid + i * kThreads;
        xb[i].zero();
        if constexpr (BKc) {
          const int k = k0 + (q % (BK / 4)) * 4;
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (k + e < kend) xb[i].set(e, B + offB[i] + k0 + e, true);
        } else {
          const int k = k0 + q / (BN / 4);
          if (k < kend) {
            const E* p = B + (long long)k * a.ldb;
#pragma unroll
            for (int e = 0; e < 4; ++e)
              xb[i].set(e, p + min((int)offB[i] + e, N - 1), true);
          }
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        if constexpr (BKc)
          xb[i].load(B + offB[i] + k0);
        else
          xb[i].load(B + (long long)(k0 + (tid + i * kThreads) / (BN / 4)) * a.ldb + offB[i]);
      }
    }
  };
  // bias gradient: this thread's share of four columns' sums over k (k-slow B)
  const bool do_bias = kUpd && a.bias_w && m0 == 0;
  v4f colsum = v4f{0.f, 0.f, 0.f, 0.f};
  auto lstore = [&](int buf, const Q(&xa)[NA], const Q(&xb)[NB]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const int q = tid + i * kThreads;
      const int o = AK ? (q / (BK / 4)) * PA + (q % (BK / 4)) * 4
                       : (q / (BM / 4)) * PA + (q % (BM / 4)) * 4;
      u32x2 p[NPL];
      xa[i].planes(p);
#pragma unroll
      for (int l = 0; l < NPL; ++l) *(u32x2*)&sA[(buf * NPL + l) * SA + o] = p[l];
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int q = tid + i * kThreads;
      const int o = BKc ? (q / (BK / 4)) * PB + (q % (BK / 4)) * 4
                        : (q / (BN / 4)) * PB + (q % (BN / 4)) * 4;
      u32x2 p[NPL];
      xb[i].planes(p);
#pragma unroll
      for (int l = 0; l < NPL; ++l) *(u32x2*)&sB[(buf * NPL + l) * SB + o] = p[l];
    }
  };
  auto colsums = [&](const Q(&xb)[NB]) __attribute__((always_inline)) {
    if constexpr (kUpd) {
      if (do_bias) {
#pragma unroll
        for (int i = 0; i < NB; ++i) colsum += xb[i].f32();
      }
    }
  };
  floatx16 hi[FM][FN], lo[BF ? 1 : FM][BF ? 1 : FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        hi[i][j][v] = 0.f;
        if constexpr (!BF) lo[i][j][v] = 0.f;
      }
  // fragment of rows (columns) r0 .. r0 + 31, k kk .. kk + 15, of one plane
  const int trow = 8 * lk + ((lane & 15) >> 2), tcol = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  auto frag = [&](const bf16_t* p, bool kc, int pitch, int r0, int kk)
      __attribute__((always_inline)) -> bf16x8 {
    if (kc) return *(const bf16x8*)&p[(r0 + lr) * pitch + kk + 8 * lk];
    using L = __attribute__((address_space(3))) s16x4;
    const bf16_t* b = p + (kk + trow) * pitch + r0 + tcol;
    const s16x4 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16((L*)b);
    const s16x4 y = __builtin_amdgcn_ds_read_tr16_b64_v4i16((L*)(b + 4 * pitch));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    return __builtin_bit_cast(bf16x8, s16x8{x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]});
  };
  auto compute = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int kk = 0; kk < BK; kk += 16) {
      bf16x8 fa[FM][NPL], fb[FN][NPL];
#pragma unroll
      for (int l = 0; l < NPL; ++l) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
          fa[i][l] = frag(sA + (buf * NPL + l) * SA, AK, PA, wm0 + i * 32, kk);
#pragma unroll
        for (int j = 0; j < FN; ++j)
          fb[j][l] = frag(sB + (buf * NPL + l) * SB, BKc, PB, wn0 + j * 32, kk);
      }
      auto mm = [&](int x, int y, bool low) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j) {
            floatx16& c = low ? lo[BF ? 0 : i][BF ? 0 : j] : hi[i][j];
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i][x], fb[j][y], c, 0, 0, 0);
          }
      };
      if constexpr (!BF) {
        mm(NPL - 1, 0, true);
        mm(0, 0, false);
        mm(0, NPL - 1, true);
        mm(1 % NPL, 1 % NPL, true);
        mm(1 % NPL, 0, true);
        mm(0, 1 % NPL, true);
      } else {
        mm(0, 0, false);
      }
    }
  };
  // slab t: register set t % D, LDS buffer t % 2; loads past the last slab
  // repeat it (unused)
  if (nk > 0) {
    Q ra[D][NA], rb[D][NB];
    auto slab = [&](int s) __attribute__((always_inline)) { return kbeg + min(s, nk - 1) * BK; };
#pragma unroll
    for (int d = 0; d < D; ++d) gload(slab(d), ra[d], rb[d]);
    colsums(rb[0]);
    lstore(0, ra[0], rb[0]);
    __syncthreads();
    int it = 0;
    for (; it + D < nk; it += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        gload(slab(it + d + D), ra[d], rb[d]);
        __builtin_amdgcn_sched_barrier(0);
        compute(d & 1);
        colsums(rb[(d + 1) % D]);
        lstore((d + 1) & 1, ra[(d + 1) % D], rb[(d + 1) % D]);
        __syncthreads();
      }
    }
#pragma unroll
    for (int d = 0; d < D; ++d) {
      if (it + d >= nk) break;
      compute(d & 1);
      if (it + d + 1 < nk) {
        colsums(rb[(d + 1) % D]);
        lstore((d + 1) & 1, ra[(d + 1) % D], rb[(d + 1) % D]);
      }
      __syncthreads();
    }
  }
  if constexpr (!BF) {
    bool bad = false;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          hi[i][j][v] += lo[i][j][v];
          bad |= hi[i][j][v] != hi[i][j][v];
        }
    if (__builtin_expect(__any(bad), 0)) {
      // infinities (or NaN) among the operands: the fp32 instruction, from
      // memory
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          floatx16 acc;
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[v] = 0.f;
          const int m = min(m0 + wm0 + i * 32 + lr, M - 1), n = min(n0 + wn0 + j * 32 + lr, N - 1);
          for (int k = kbeg; k < kend; k += 2) {
            const int kx = k + lk, kc = min(kx, kend - 1);
            const long long oa = AT ? (GATHER ? (long long)rmap[kc] : (long long)kc) * a.lda + m
                                    : (GATHER ? (long long)rmap[m] : (long long)m) * a.lda + kc;
            const long long ob = BT ? (long long)n * a.ldb + kc : (long long)kc * a.ldb + n;
            const float x = kx < kend ? ((const float*)A)[oa] : 0.f;
            const float y = kx < kend ? ((const float*)B)[ob] : 0.f;
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x, y, acc, 0, 0, 0);
          }
          hi[i][j] = acc;
        }
    }
  }

  // epilogue
  constexpr bool OUTBF = BF && (EPI == EPI_BIAS_RELU || EPI == EPI_RELU_MASK);
  if constexpr (kUpd) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int m = out_row(i, v), n = n0 + wn0 + j * 32 + lr;
          if (!FULL && (m >= M || n >= N)) continue;
          const long long o = (long long)g * a.sC + (long long)m * a.ldc + n;
          sgd_step(wv[i][j][v], uv[i][j][v], hi[i][j][v], a);
          a.W[o] = wv[i][j][v];
          a.U[o] = uv[i][j][v];
          if (a.Wb) a.Wb[o] = f32_to_bf16(wv[i][j][v]);
        }
    if (do_bias) {
      // the threads that share a column's quad, in ascending thread order
      constexpr int RQ = BN / 4, TPC = kThreads / RQ;
      float* red = (float*)sA;  // [TPC][BN] floats (the k loop is done with it)
      static_assert(TPC * BN * 4 <= 2 * NPL * SA * 2, "column sums fit");
      __syncthreads();
      *(v4f*)&red[(tid / RQ) * BN + (tid % RQ) * 4] = colsum;
      __syncthreads();
      if (tid < BN && n0 + tid < N) {
        float s = red[tid];
#pragma unroll
        for (int q = 1; q < TPC; ++q) s += red[q * BN + tid];
        bias_update(a, g, n0 + tid, s);
      }
    }
  } else if (a.splits > 1) {  // raw partial sums, [s][g][M][N]
    float* P = a.part + ((long long)t.s * a.G + g) * M * N;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int m = out_row(i, v), n = n0 + wn0 + j * 32 + lr;
          if (FULL || (m < M && n < N)) P[(long long)m * N + n] = hi[i][j][v];
        }
  } else {
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int n = n0 + wn0 + j * 32 + lr;
      float bias = 0.f;
      if constexpr (EPI == EPI_BIAS || EPI == EPI_BIAS_RELU)
        bias = a.bias[(long long)g * a.sBias + (FULL ? n : min(n, N - 1))];
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        float mk[16];
        if constexpr (EPI == EPI_RELU_MASK) {  // the mask first: 16 loads in flight
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            int m = out_row(i, v);
            if constexpr (!FULL) m = min(m, M - 1);
            const long long o = (long long)g * a.sC + (long long)m * a.ldc + (FULL ? n : min(n, N - 1));
            mk[v] = OUTBF ? bf16_to_f32(((const bf16_t*)a.mask)[o]) : ((const float*)a.mask)[o];
          }
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int m = out_row(i, v);
          if (!FULL && (m >= M || n >= N)) continue;
          const long long o = (long long)g * a.sC + (long long)m * a.ldc + n;
          float r = hi[i][j][v] + bias;
          if constexpr (EPI == EPI_STORE) r = hi[i][j][v];
          if constexpr (EPI == EPI_BIAS_RELU) r = r > 0.f ? r : 0.f;
          if constexpr (EPI == EPI_RELU_MASK) r = mk[v] > 0.f ? hi[i][j][v] : 0.f;
          if constexpr (OUTBF)
            ((bf16_t*)a.C)[o] = f32_to_bf16(r);
          else
            ((float*)a.C)[o] = r;
        }
      }
    }
  }
}

// ------------------------------------------------- fp32 update, specialised
// Fused weight gradient + momentum-SGD update over the 128 x 128 tiles of one
// or several layers (a list of problems whose tiles are concatenated). A
// workgroup of 8 wavefronts stays resident and walks its share of the tile
// list; its waves have two roles that run concurrently:
//   MFMA waves 0-3 each compute a 64 x 64 quarter of tile j. A lane loads its
//     operands straight from global memory as float2 pairs along m (resp. n);
//     the two halves of a pair feed two different 32 x 32 MFMA blocks, so
//     block i's MFMA row r is m = 2 r + i (columns likewise) and no LDS
//     staging (and so no barrier among the MFMA waves) is needed. A ring of
//     D k-pairs of registers keeps D loads in flight.
//   Update waves 4-7 apply the SGD step to tile j-1 from the gradient tile
//     in LDS (float4 runs along n: coalesced W/U rows), then issue the W/U
//     reads of tile j, which arrive while tile j's MFMAs run.
// Two workgroup barriers per tile hand the LDS gradient buffer over. The
// HBM-bound update of one tile thus overlaps the MFMA phase of the next,
// where separate workgroups doing both phases in turn fall into step and
// alternate between compute-only and memory-only periods across the chip.
// Every problem needs M % 128 == 0, N % 128 == 0, 8-byte aligned operand
// rows, 16-byte aligned W/U rows and (gathered rows) Kd <= 512; all share
// lr, momentum, weight decay and Nesterov.
constexpr int kWsThreads = 512;
constexpr int kWsMaxRows = 512;
constexpr int kWsDepth = 8;        // k-pairs of operands in flight per lane
constexpr int kWsMinTiles = 1024;  // below: one tile per workgroup is as good

struct WsArgs {
  GemmArgs p[kWsMaxProblems];
  int start[kWsMaxProblems + 1];  // first tile of each problem; [np] = total
  int np;
};

struct WsTile {
  int pi, g, m0, n0;
};

__device__ __forceinline__ bool ws_tile(const WsArgs& w, int j, WsTile& t) {
  const int total = w.start[w.np];
  const int p = blockIdx.x, nwg = gridDim.x;
  int l;
  if (total % kXcds == 0 && nwg % kXcds == 0) {
    // XCD x = p % 8 owns tiles [x * total/8, (x+1) * total/8)
    const int chunk = total / kXcds, q = p / kXcds + j * (nwg / kXcds);
    if (q >= chunk) return false;
    l = (p % kXcds) * chunk + q;
  } else {
    const long long ll = p + (long long)j * nwg;
    if (ll >= total) return false;
    l = (int)ll;
  }
  int pi = 0;
  while (pi + 1 < w.np && l >= w.start[pi + 1]) ++pi;
  l -= w.start[pi];
  const int tn = w.p[pi].N / 128, per_g = tn * (w.p[pi].M / 128);
  t.pi = pi;
  t.g = l / per_g;
  l -= t.g * per_g;
  t.m0 = (l / tn) * 128;
  t.n0 = (l % tn) * 128;
  return true;
}

// Row list (sampled dataset indices) of a gathered tile: thread t < 256 of
// the MFMA role holds entries t and t + 256 (clamped to the last row).
struct WsRows {
  int32_t r0, r1;
};
__device__ __forceinline__ WsRows ws_rows_load(const WsArgs& w, const WsTile& t) {
  const GemmArgs& a = w.p[t.pi];
  const int32_t* rm = a.rowmap + (long long)t.g * a.sRow;
  const int last = a.Kd - 1, i = threadIdx.x;
  return WsRows{rm[min(i, last)], rm[min(i + 256, last)]};
}
__device__ __forceinline__ void ws_rows_store(int32_t* buf, const WsRows& r) {
  buf[threadIdx.x] = r.r0;
  buf[threadIdx.x + 256] = r.r1;
}

// Operand pairs of the MFMA role: two consecutive fp32 values (float2), or
// two consecutive bf16 values in one 32-bit word, widened to fp32 at use
// (bf16 x bf16 products are exact in fp32, so the fp32 MFMA computes what a
// bf16 MFMA with fp32 accumulation does, up to the order of the sums).
template <bool BF>
struct WsOp;
template <>
struct WsOp<false> {
  using E = float;
  using P = float2;
  __device__ static P ld(const E* p) { return *(const float2*)p; }
  __device__ static float lo(P v) { return v.x; }
  __device__ static float hi(P v) { return v.y; }
};
template <>
struct WsOp<true> {
  using E = bf16_t;
  using P = uint32_t;
  __device__ static P ld(const E* p) { return *(const uint32_t*)p; }
  __device__ static float lo(P v) { return __uint_as_float(v << 16); }
  __device__ static float hi(P v) { return __uint_as_float(v & 0xffff0000u); }
};

// k loop of one MFMA wave over a tile (its 64 x 64 quarter): rows
// k = 2 kp + lk, kp < nkp. A points at column m0 + wm0 + 2 lr of row 0
// (gathered: row srm[k]), B at column n0 + wn0 + 2 lr of row 0.
template <bool BF, int D>
struct WsK {
  using Op = WsOp<BF>;
  using E = typename Op::E;
  using P = typename Op::P;

  __device__ static void mfma(floatx16 (&acc)[2][2], P ra, P rb, float& cs0, float& cs1) {
    const float a0 = Op::lo(ra), a1 = Op::hi(ra), b0 = Op::lo(rb), b1 = Op::hi(rb);
    acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b0, acc[0][0], 0, 0, 0);
    acc[0][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b1, acc[0][1], 0, 0, 0);
    acc[1][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, b0, acc[1][0], 0, 0, 0);
    acc[1][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, b1, acc[1][1], 0, 0, 0);
    cs0 += b0;
    cs1 += b1;
  }

  // Any batch size. Rows past the end are clamped to the last one and their
  // values replaced by zero at use, so the loads carry no branches and stay
  // countable in flight; a runtime loop's back edge still makes the compiler
  // wait for all of them at the top of each block.
  __device__ static void generic(floatx16 (&acc)[2][2], const E* A, const E* B,
                                 long long lda, long long ldb, int Kd, bool gather,
                                 const int32_t* srm, int lk, float& cs0, float& cs1) {
    P ra[D], rb[D];
    auto load = [&](int kp, P& x, P& y) __attribute__((always_inline)) {
      const int k = min(2 * kp + lk, Kd - 1);
      const int sr = srm[min(k, kWsMaxRows - 1)];
      const long long row = gather ? (long long)sr : (long long)k;
      x = Op::ld(A + row * lda);
      y = Op::ld(B + (long long)k * ldb);
    };
#pragma unroll
    for (int d = 0; d < D; ++d) load(d, ra[d], rb[d]);
    const int nblk = ((Kd + 1) / 2 + D - 1) / D;
    for (int blk = 0; blk < nblk; ++blk) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        const int kp = blk * D + d;
        const bool live = 2 * kp + lk < Kd;
        const P za = live ? ra[d] : P{}, zb = live ? rb[d] : P{};
        mfma(acc, za, zb, cs0, cs1);
        load(kp + D, ra[d], rb[d]);
        // keep each refill right behind its slot's MFMAs: left alone, the
        // scheduler sinks the refills to the end of the block, where they
        // have no time left to arrive
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }

  // ROWS (64 or 128) rows in straight-line code: the wait before each slot's
  // MFMAs counts exactly the D - 1 younger refills. The row indices sit in
  // ROWS / 64 registers per lane (rows lane, lane + 64) and a refill takes
  // its row by readlane at a compile-time lane instead of waiting on an LDS
  // read between MFMAs; B rows walk with one running pointer.
  template <int ROWS>
  __device__ static void unrolled(floatx16 (&acc)[2][2], const E* A, const E* B,
                                  long long lda, long long ldb, bool gather,
                                  const int32_t* srm, int lane, int lk, float& cs0,
                                  float& cs1) {
    static_assert(ROWS == 64 || ROWS == 128, "one or two index registers per lane");
    constexpr int NKP = ROWS / 2;
    P ra[D], rb[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int k = 2 * d + lk;
      const long long row = gather ? (long long)srm[k] : (long long)k;
      ra[d] = Op::ld(A + row * lda);
      rb[d] = Op::ld(B + (long long)k * ldb);
    }
    const int r_lo = srm[lane], r_hi = ROWS > 64 ? srm[lane + 64] : 0;
    const E* bq = B + (long long)(2 * D + lk) * ldb;
    const long long bstep = 2 * ldb;
#pragma unroll
    for (int kp = 0; kp < NKP; ++kp) {
      const int d = kp % D;
      const P ca = ra[d], cb = rb[d];
      const float a0 = Op::lo(ca), a1 = Op::hi(ca), b0 = Op::lo(cb), b1 = Op::hi(cb);
      acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b0, acc[0][0], 0, 0, 0);
      if (kp + D < NKP) {
        // refill of this slot with k-pair kp + D, between the MFMAs
        const int ke = 2 * (kp + D);
        const int src = ke < 64 ? r_lo : r_hi;
        const int se = __builtin_amdgcn_readlane(src, ke & 63);
        const int so = __builtin_amdgcn_readlane(src, (ke + 1) & 63);
        const long long row = gather ? (long long)(lk ? so : se) : (long long)(ke + lk);
        ra[d] = Op::ld(A + row * lda);
      }
      acc[0][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b1, acc[0][1], 0, 0, 0);
      if (kp + D < NKP) {
        rb[d] = Op::ld(bq);
        bq += bstep;
      }
      acc[1][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, b0, acc[1][0], 0, 0, 0);
      acc[1][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, b1, acc[1][1], 0, 0, 0);
      cs0 += b0;
      cs1 += b1;
      __builtin_amdgcn_sched_barrier(0);
    }
  }
};

// Both roles walk the same tile list and execute the same barriers: one
// before the first tile, then two per tile.
template <bool BF, int D>
__global__ __launch_bounds__(kWsThreads) void gemm_f32_sgd_ws(WsArgs w) {
  using K = WsK<BF, D>;
  using E = typename K::E;
  constexpr int T = 128, CP = T + 4;  // gradient tile pitch (16-byte rows)
  constexpr int PER = T * T / 4 / 256;  // float4 per update thread
  __shared__ __attribute__((aligned(16))) float Gs[T * CP];
  // row lists, double-buffered: tile j reads buffer j % 2 while the MFMA
  // role writes tile j+1's list into the other one after its k loop
  __shared__ int32_t srmap[2][kWsMaxRows];
  // wave index as a scalar: the role branch below is uniform per wave
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  WsTile cur, prev;
  bool prev_ok = false;

  if (wave < 4) {
    // ---- MFMA role: gradient tile j into LDS
    const int lk = lane >> 5, lr = lane & 31;
    const int wm0 = (wave >> 1) * 64, wn0 = (wave & 1) * 64;
    {
      WsTile t0;
      if (ws_tile(w, 0, t0) && w.p[t0.pi].rowmap) ws_rows_store(srmap[0], ws_rows_load(w, t0));
    }
    __syncthreads();  // row list of the first tile
    for (int j = 0;; ++j) {
      const bool ok = ws_tile(w, j, cur);  // uniform over the workgroup
      if (!ok && !prev_ok) break;
      floatx16 acc[2][2];
      if (ok) {
        // next tile's row list: issued now, stored after the k loop
        WsTile nxt;
        const bool nxt_rows = ws_tile(w, j + 1, nxt) && w.p[nxt.pi].rowmap;
        WsRows nr{0, 0};
        if (nxt_rows) nr = ws_rows_load(w, nxt);

        const GemmArgs& a = w.p[cur.pi];
        const int Kd = a.Kd;
        const bool gather = a.rowmap != nullptr;
        const int32_t* srm = srmap[j & 1];
        const E* A = (const E*)a.A + (long long)cur.g * a.sA + cur.m0 + wm0 + 2 * lr;
        const E* B = (const E*)a.B + (long long)cur.g * a.sB + cur.n0 + wn0 + 2 * lr;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int jj = 0; jj < 2; ++jj)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][jj][v] = 0.f;
        float cs0 = 0.f, cs1 = 0.f;
        if (Kd == 128)
          K::template unrolled<128>(acc, A, B, a.lda, a.ldb, gather, srm, lane, lk, cs0, cs1);
        else if (Kd == 64)
          K::template unrolled<64>(acc, A, B, a.lda, a.ldb, gather, srm, lane, lk, cs0, cs1);
        else
          K::generic(acc, A, B, a.lda, a.ldb, Kd, gather, srm, lk, cs0, cs1);
        if (nxt_rows) ws_rows_store(srmap[(j + 1) & 1], nr);
        if (a.bias_w && cur.m0 == 0 && wm0 == 0) {
          // lanes < 32 summed the even batch rows, lanes >= 32 the odd ones
          cs0 += __shfl_xor(cs0, 32, 64);
          cs1 += __shfl_xor(cs1, 32, 64);
          if (lk == 0) {
            const int n = cur.n0 + wn0 + 2 * lr;
            bias_update(a, cur.g, n, cs0);
            bias_update(a, cur.g, n + 1, cs1);
          }
        }
      }
      __syncthreads();  // the update role has consumed gradient tile j-1
      if (ok) {
        // accumulator v of block (i, jj): row 8(v/4) + 4 lk + v%4, column lr
        // of the block, i.e. tile row wm0 + 2 R + i, column wn0 + 2 lr + jj
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int R = (v >> 2) * 8 + lk * 4 + (v & 3);
            *(float2*)&Gs[(wm0 + 2 * R + i) * CP + wn0 + 2 * lr] =
                make_float2(acc[i][0][v], acc[i][1][v]);
          }
      }
      __syncthreads();  // gradient tile j (and tile j+1's row list) in LDS
      prev_ok = ok;
    }
  } else {
    // ---- update role: SGD step of tile j-1, then tile j's W/U reads
    const int u = (int)threadIdx.x - 256;
    float4 wv[PER], uv[PER];
    __syncthreads();  // row list of the first tile
    for (int j = 0;; ++j) {
      const bool ok = ws_tile(w, j, cur);
      if (!ok && !prev_ok) break;
      if (prev_ok) {
        const GemmArgs& a = w.p[prev.pi];
#pragma unroll
        for (int p = 0; p < PER; ++p) {
          const int r = u / 32 + 8 * p, c = (u % 32) * 4;
          const long long off = (long long)prev.g * a.sC +
                                (long long)(prev.m0 + r) * a.ldc + prev.n0 + c;
          const float4 gr = *(const float4*)&Gs[r * CP + c];
          float4 wq = wv[p], uq = uv[p];
          sgd_step(wq.x, uq.x, gr.x, a);
          sgd_step(wq.y, uq.y, gr.y, a);
          sgd_step(wq.z, uq.z, gr.z, a);
          sgd_step(wq.w, uq.w, gr.w, a);
          *(float4*)(a.W + off) = wq;
          *(float4*)(a.U + off) = uq;
          if (a.Wb) {
            const uint32_t lo = f32_to_bf16(wq.x) | ((uint32_t)f32_to_bf16(wq.y) << 16);
            const uint32_t hi = f32_to_bf16(wq.z) | ((uint32_t)f32_to_bf16(wq.w) << 16);
            *(uint2*)(a.Wb + off) = make_uint2(lo, hi);
          }
        }
      }
      if (ok) {
        const GemmArgs& a = w.p[cur.pi];
#pragma unroll
        for (int p = 0; p < PER; ++p) {
          const int r = u / 32 + 8 * p, c = (u % 32) * 4;
          const long long in = (long long)(cur.m0 + r) * a.ldc + cur.n0 + c;
          const long long off = (long long)cur.g * a.sC + in;
          wv[p] = *(const float4*)(a.Wsrc ? a.Wsrc + (long long)cur.g * a.sWsrc + in
                                          : a.W + off);
          uv[p] = *(const float4*)(a.U + off);
        }
      }
      __syncthreads();  // gradient tile j-1 consumed
      __syncthreads();  // gradient tile j is in LDS
      prev = cur;
      prev_ok = ok;
    }
  }
}

// Shape and alignment rules of the specialised kernel for one problem.
// fp32 operands are read as float2, bf16 operands as pairs in one 32-bit word.
bool ws_eligible(int dtype, const GemmArgs& a) {
  auto al = [](const void* p, uintptr_t m) { return ((uintptr_t)p & m) == 0; };
  const uintptr_t pair = dtype == 0 ? 7 : 3;
  return (dtype == 0 || dtype == 1) && a.splits <= 1 && a.G > 0 && a.M > 0 &&
         a.N > 0 && a.Kd > 0 && a.M % 128 == 0 && a.N % 128 == 0 &&
         (a.rowmap == nullptr || a.Kd <= kWsMaxRows) &&
         a.lda % 2 == 0 && a.sA % 2 == 0 && al(a.A, pair) &&
         a.ldb % 2 == 0 && a.sB % 2 == 0 && al(a.B, pair) &&
         a.ldc % 4 == 0 && a.sC % 4 == 0 && al(a.W, 15) && al(a.U, 15) &&
         (a.Wb == nullptr || al(a.Wb, 7)) &&
         (a.Wsrc == nullptr || (al(a.Wsrc, 15) && a.sWsrc % 4 == 0));
}


// ------------------------------------------------------------------ split-K
// C[g][m][n] = epilogue(sum_{s=0}^{S-1} part[s][g][m][n]), s ascending. S is
// a template argument so all S loads are issued before the sum.
template <int EPI, bool OUTBF, int S>
__global__ void k_splitk_reduce(GemmArgs a) {
  const long long MN = (long long)a.M * a.N, total = MN * a.G;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x) {
    float p[S];
#pragma unroll
    for (int s = 0; s < S; ++s) p[s] = a.part[i + s * total];
    float v = p[0];
#pragma unroll
    for (int s = 1; s < S; ++s) v += p[s];
    const int g = (int)(i / MN);
    const long long r = i - g * MN;
    finish<EPI, OUTBF>(a, g, (int)(r / a.N), (int)(r % a.N), v);
  }
}

template <int EPI, bool OUTBF>
hipError_t launch_reduce(const GemmArgs& a, hipStream_t s) {
  const long long n = (long long)a.G * a.M * a.N;
  const int blocks = (int)((n + 255) / 256 < 8192 ? (n + 255) / 256 : 8192);
  switch (a.splits) {
    case 2: hipLaunchKernelGGL((k_splitk_reduce<EPI, OUTBF, 2>), dim3(blocks), dim3(256), 0, s, a); break;
    case 4: hipLaunchKernelGGL((k_splitk_reduce<EPI, OUTBF, 4>), dim3(blocks), dim3(256), 0, s, a); break;
    case 8: hipLaunchKernelGGL((k_splitk_reduce<EPI, OUTBF, 8>), dim3(blocks), dim3(256), 0, s, a); break;
    case 3: hipLaunchKernelGGL((k_splitk_reduce<EPI, OUTBF, 3>), dim3(blocks), dim3(256), 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Compute units and resident specialised-update workgroups per CU on the
// current device, queried once per device.
template <bool BF>
hipError_t ws_grid(long long tiles, int& grid) {
  struct Shape {
    int cus = 0, per_cu = 0;
  };
  static Shape cache[64];
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  if (cache[dev].cus == 0) {
    Shape sh;
    e = hipDeviceGetAttribute(&sh.cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &sh.per_cu, reinterpret_cast<const void*>(gemm_f32_sgd_ws<BF, kWsDepth>),
        kWsThreads, 0);
    if (e != hipSuccess) return e;
    if (sh.per_cu < 1) sh.per_cu = 1;
    cache[dev] = sh;
  }
  long long g = (long long)cache[dev].cus * cache[dev].per_cu;
  if (g > tiles) g = tiles;
  if (g >= kXcds) g -= g % kXcds;
  grid = (int)g;
  return hipSuccess;
}

}  // namespace

int gemm_sgd_multi_tiles(int dtype, const GemmArgs* list, int n) {
  if (n < 1 || n > kWsMaxProblems) return -1;
  long long total = 0;
  for (int i = 0; i < n; ++i) {
    if (!ws_eligible(dtype, list[i])) return -1;
    total += (long long)(list[i].M / 128) * (list[i].N / 128) * list[i].G;
  }
  return total < (1LL << 30) ? (int)total : -1;
}

hipError_t launch_gemm_sgd_multi(int dtype, const GemmArgs* list, int n,
                                 hipStream_t s) {
  const int total = gemm_sgd_multi_tiles(dtype, list, n);
  if (total < 0) return hipErrorInvalidValue;
  if (total == 0) return hipSuccess;
  WsArgs w{};
  w.np = n;
  w.start[0] = 0;
  for (int i = 0; i < n; ++i) {
    w.p[i] = list[i];
    w.p[i].splits = 1;
    w.start[i + 1] = w.start[i] + (list[i].M / 128) * (list[i].N / 128) * list[i].G;
    if (i > 0 && (list[i].lr != list[0].lr || list[i].mom != list[0].mom ||
                  list[i].wd != list[0].wd || list[i].nesterov != list[0].nesterov))
      return hipErrorInvalidValue;
  }
  int grid = 0;
  hipError_t e = dtype == 1 ? ws_grid<true>(total, grid) : ws_grid<false>(total, grid);
  if (e != hipSuccess) return e;
  if (dtype == 1)
    hipLaunchKernelGGL((gemm_f32_sgd_ws<true, kWsDepth>), dim3(grid), dim3(kWsThreads),
                       0, s, w);
  else
    hipLaunchKernelGGL((gemm_f32_sgd_ws<false, kWsDepth>), dim3(grid), dim3(kWsThreads),
                       0, s, w);
  return hipGetLastError();
}

namespace {

// Tile of a forward, input-gradient or plain product. Larger tiles read less
// from LDS per MFMA, but a launch should have a workgroup for each of the 256
// CUs (two of the 128 x 64 ones): 128 x 128 (fp32) or 128 x 64 tiles where the
// output has that many, or where the inner dimension is long enough for
// split-K to get there; else 64 x 64. Measured, 16 replicas of 128 x 512 x
// 3072, fp32 with the partials' sum: 128 x 128 split 4 46 us, 128 x 64 split 4
// 51-58, 64 x 64 split 2 53; 128 x 512 x 512: 64 x 64 12 us, 128 x 64 18.
struct Shape {
  int BM, BN;
};
Shape tile_shape(bool bf, int M, int N, int G, int Kd) {
  if (M <= 64 || N <= 64) return {64, 64};
  const bool deep = Kd >= 2048;
  const long long t128 = (long long)((M + 127) / 128) * ((N + 127) / 128) * G;
  if (!bf && (t128 >= 256 || (deep && t128 >= 32))) return {128, 128};
  const long long t64 = (long long)((M + 127) / 128) * ((N + 63) / 64) * G;
  if (t64 >= 512 || deep) return {128, 64};
  return {64, 64};
}

// Whole tiles, whole slabs per split: the FULL kernel variant.
bool full(const GemmArgs& a, int BM, int BN, int BK) {
  return a.M % BM == 0 && a.N % BN == 0 && a.kchunk % BK == 0 &&
         (long long)a.kchunk * a.splits == a.Kd;
}

template <bool BF, bool AT, bool BT, int EPI, bool GATHER, int BM, int BN, int BK, int D>
hipError_t run_tile(const GemmArgs& a, hipStream_t s) {
  const long long total =
      (long long)((a.N + BN - 1) / BN) * ((a.M + BM - 1) / BM) * a.G * a.splits;
  if (total > 0x7fffffffLL) return hipErrorInvalidValue;
  if (full(a, BM, BN, BK))
    hipLaunchKernelGGL((gemm_mm<BF, AT, BT, EPI, GATHER, BM, BN, BK, D, true>), dim3(total),
                       dim3(kThreads), 0, s, a);
  else
    hipLaunchKernelGGL((gemm_mm<BF, AT, BT, EPI, GATHER, BM, BN, BK, D, false>), dim3(total),
                       dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

template <bool BF, bool AT, bool BT, int EPI, bool GATHER>
hipError_t run_type(const GemmArgs& a, hipStream_t s) {
  if constexpr (EPI == EPI_SGD) {
    return run_tile<BF, AT, BT, EPI, GATHER, 64, 64, 32, 2>(a, s);
  } else {
    const Shape sh = tile_shape(BF, a.M, a.N, a.G, a.Kd);
    hipError_t e;
    if (sh.BM == 64)
      e = run_tile<BF, AT, BT, EPI, GATHER, 64, 64, BF ? 64 : 32, 2>(a, s);
    else if (BF || sh.BN == 64)
      e = run_tile<BF, AT, BT, EPI, GATHER, 128, 64, BF ? 32 : 16, 2>(a, s);
    else
      e = run_tile<BF, AT, BT, EPI, GATHER, 128, BF ? 64 : 128, BF ? 32 : 16, 2>(a, s);
    if (e != hipSuccess || a.splits == 1) return e;
    constexpr bool OUTBF = BF && (EPI == EPI_BIAS_RELU || EPI == EPI_RELU_MASK);
    return launch_reduce<EPI, OUTBF>(a, s);
  }
}

template <bool AT, bool BT, int EPI, bool GATHER>
hipError_t run(int dtype, const GemmArgs& a, hipStream_t s) {
  if constexpr (AT && !BT && EPI == EPI_SGD) {
    // one large layer: the specialised update kernel with a one-item list
    if (ws_eligible(dtype, a) &&
        (long long)(a.M / 128) * (a.N / 128) * a.G >= kWsMinTiles)
      return launch_gemm_sgd_multi(dtype, &a, 1, s);
  }
  return dtype == 1 ? run_type<true, AT, BT, EPI, GATHER>(a, s)
                    : run_type<false, AT, BT, EPI, GATHER>(a, s);
}

template <bool AT, bool BT, int EPI>
hipError_t dispatch(int dtype, const GemmArgs& a, hipStream_t s) {
  if (a.rowmap) {  // gathered rows: the first layer's forward and update
    if constexpr (EPI == EPI_STORE || EPI == EPI_RELU_MASK)
      return hipErrorInvalidValue;
    else
      return run<AT, BT, EPI, true>(dtype, a, s);
  }
  return run<AT, BT, EPI, false>(dtype, a, s);
}

}  // namespace

int gemm_splits(int dtype, int M, int N, int Kd, int G, int epi) {
  if (epi == EPI_SGD) return 1;
  const Shape sh = tile_shape(dtype == 1, M, N, G, Kd);
  const long long tiles = (long long)((N + sh.BN - 1) / sh.BN) * ((M + sh.BM - 1) / sh.BM) * G;
  const int want = sh.BM * sh.BN == 128 * 64 ? 512 : 256;
  int s = 1;
  // up to 8 splits while the grid has fewer workgroups than that and every
  // split keeps at least 128 of K
  while (s < 8 && tiles * s < want && Kd / (s * 2) >= 128) s *= 2;
  return s;
}

hipError_t launch_gemm(int dtype, int trans_a, int trans_b, int epi,
                       int out_bf16, const GemmArgs& args, hipStream_t s) {
  if (args.G <= 0 || args.M <= 0 || args.N <= 0 || args.Kd <= 0) return hipSuccess;
  GemmArgs a = args;
  if (a.splits < 1) a.splits = 1;
  if (a.splits > 1 && (a.part == nullptr || epi == EPI_SGD)) return hipErrorInvalidValue;
  a.kchunk = (a.Kd + a.splits - 1) / a.splits;
  a.kchunk = (a.kchunk + 31) / 32 * 32;
  // activations are bf16 exactly when the operands are
  if ((epi == EPI_BIAS_RELU || epi == EPI_RELU_MASK) && out_bf16 != (dtype == 1))
    return hipErrorInvalidValue;
  const int key = trans_a * 2 + trans_b;
  switch (epi) {
    case EPI_STORE:
      switch (key) {
        case 0: return dispatch<false, false, EPI_STORE>(dtype, a, s);
        case 1: return dispatch<false, true, EPI_STORE>(dtype, a, s);
        case 2: return dispatch<true, false, EPI_STORE>(dtype, a, s);
        default: return dispatch<true, true, EPI_STORE>(dtype, a, s);
      }
    case EPI_BIAS:
      if (key == 0) return dispatch<false, false, EPI_BIAS>(dtype, a, s);
      break;
    case EPI_BIAS_RELU:
      if (key == 0) return dispatch<false, false, EPI_BIAS_RELU>(dtype, a, s);
      break;
    case EPI_RELU_MASK:
      if (key == 1) return dispatch<false, true, EPI_RELU_MASK>(dtype, a, s);
      break;
    case EPI_SGD:
      if (key == 2) return dispatch<true, false, EPI_SGD>(dtype, a, s);
      break;
    default:
      break;
  }
  return hipErrorInvalidValue;
}

}  // namespace lsgd
