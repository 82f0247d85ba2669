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
// (each the round-to-nearest bf16 of what the ones before leave: 3 x 8
// significant bits), and x y as the six products x1 y1, x1 y2, x2 y1, x2 y2,
// x1 y3, x3 y1, each exact in fp32. The three left out reach 2^-24 |x y| at
// worst (|x2| <= 2^-8 |x|, |x3| <= 2^-17 |x|); their rms over normal operands is
// 2^-27.4 |x y|. x1 y1 has an accumulator of its own and the five small
// ones share another, added at the end: a k range of 16 then rounds once at the
// sum's own magnitude where v_mfma_f32_32x32x2f32 rounds 16 times. Measured
// against fp64 (normwise, normal operands, K = 3 / 64 / 512 / 3072): 2.7e-8 /
// 5.0e-8 / 1.3e-7 / 3.4e-7, kernels on the fp32 instruction 3.6e-8 / 1.1e-7 /
// 2.9e-7 / 7.0e-7.
// An inner range of one or two, where the products left out would show (largest
// error over |x y| 9.4e-8 against 6.0e-8 at K = 1), takes the fp32 instruction.
// So does a wave whose result holds an infinity or a NaN: x1 of an infinity, or
// of a finite value that rounds to one, leaves NaN pieces, and x1 y1 may
// overflow where x y does not.
// The pieces of a value below 2^-110 fall under bf16's smallest subnormal, an
// error of up to 2^-134 |y| of its product. The plain product (EPI_STORE), whose
// operands may be anything, splits 2^16 x and 2^16 y instead, exact down to the
// smallest subnormal (2^-149, whose image is bf16's), and takes 2^-32 of the sum;
// what overflows by that (results of 2^96, operands of 2^112) takes the fp32
// instruction. The products of a local step
// do not: a step of normal size does not see 1e-40 of an activation or a
// weight, and the multiplications cost it 2 to 4% (the 512-wide MLP's round of
// 16 steps 3.24 -> 3.35 ms, 784-300-100-10 at a batch of 50 55 -> 57 us a step).
//
// Work distribution: a 1-D grid of G * S * tilesM * tilesN workgroups. The
// hardware deals consecutive workgroup ids round-robin to the 8 XCDs (each
// with its own L2), so the id is remapped to give every XCD a contiguous range
// of tiles: the tiles of one replica then share that XCD's L2.
// Split-K (S > 1) gives skinny GEMMs enough workgroups: split s covers K range
// [s*kchunk, (s+1)*kchunk) and writes a raw fp32 partial; a second kernel sums
// the S partials in ascending s and applies the epilogue.
#include <type_traits>

#include "device_common.h"
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
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));

constexpr int kThreads = 256;
constexpr int kXcds = 8;

struct Tile {
  int g, s, m0, n0;
};

// A launch of n workgroups in order: on the grid's x axis, and past 2^23 of them
// in rows of that (an axis holds fewer than 2^32 threads; a longer one is cut
// short without an error).
constexpr int kGridShift = 23;
dim3 grid_of(long long n) {
  if (n <= 1LL << kGridShift) return dim3((unsigned)n);
  return dim3(1u << kGridShift, (unsigned)((n + (1LL << kGridShift) - 1) >> kGridShift));
}
__device__ __forceinline__ unsigned workgroup_id() {
  return (blockIdx.y << kGridShift) + blockIdx.x;
}

// (g < 0: past the last tile)
__device__ __forceinline__ Tile decode_tile(const GemmArgs& a, int BM, int BN) {
  const int tn = (a.N + BN - 1) / BN, tm = (a.M + BM - 1) / BM;
  const int per_split = tn * tm, per_g = per_split * a.splits;
  const int total = per_g * a.G;
  if (workgroup_id() >= (unsigned)total) return Tile{-1, 0, 0, 0};
  const int p = workgroup_id();
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
// Two fp32 values (SCALED: times kSplitScale) as packed bf16 pairs
// p[0] + p[1] + p[2] (see the top).
constexpr float kSplitScale = 0x1p16f, kSplitUnscale = 0x1p-32f;
template <bool SCALED>
__device__ __forceinline__ void split3(float x, float y, uint32_t (&p)[3]) {
  if constexpr (SCALED) {
    x *= kSplitScale;
    y *= kSplitScale;
  }
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
  v4f v;
  __device__ __forceinline__ void load(const E* p) { v = *(const v4f_any*)p; }
  __device__ __forceinline__ void set(int e, const E* p, bool ok) { v[e] = ok ? *p : 0.f; }
  __device__ __forceinline__ void zero() { v = v4f{0.f, 0.f, 0.f, 0.f}; }
  // elements s .. s + 3 of the quad and whatever follows (s >= 4: none of it)
  __device__ __forceinline__ void shift(int s) {
    if (s & 1) v = v4f{v[1], v[2], v[3], v[3]};
    if (s & 2) v = v4f{v[2], v[3], v[3], v[3]};
  }
  // the first n elements, zeros behind them
  __device__ __forceinline__ void keep(int n) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = e < n ? v[e] : 0.f;
  }
  template <bool SCALED>
  __device__ __forceinline__ void planes(u32x2 (&q)[3]) const {
    uint32_t a[3], b[3];
    split3<SCALED>(v[0], v[1], a);
    split3<SCALED>(v[2], v[3], b);
#pragma unroll
    for (int i = 0; i < 3; ++i) q[i] = u32x2{a[i], b[i]};
  }
  __device__ __forceinline__ v4f f32() const { return v; }
};
template <>
struct Quad<true> {
  using E = bf16_t;
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
  __device__ __forceinline__ void shift(int s) {
    if (s & 1) v = u32x2{(v.x >> 16) | (v.y << 16), v.y >> 16};
    if (s & 2) v = u32x2{v.y, v.y};
  }
  __device__ __forceinline__ void keep(int n) {
    v.x = n > 1 ? v.x : n > 0 ? v.x & 0xffffu : 0u;
    v.y = n > 3 ? v.y : n > 2 ? v.y & 0xffffu : 0u;
  }
  template <bool SCALED>
  __device__ __forceinline__ void planes(u32x2 (&q)[1]) const { q[0] = v; }
  __device__ __forceinline__ v4f f32() const {
    return v4f{__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u),
               __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xffff0000u)};
  }
};

// Eight bf16 elements: one load and one LDS store of 16 bytes (products in whole
// tiles: 8192 x 512 x 8192 123 us in quads, 101; 64 x 64 x 65536 389, 281).
struct Oct {
  using E = bf16_t;
  u32x4 v;
  __device__ __forceinline__ void load(const E* p) { v = *(const u32x4_any*)p; }
  template <bool SCALED>
  __device__ __forceinline__ void planes(u32x4 (&q)[1]) const { q[0] = v; }
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
// FULL: whole tiles and whole slabs (checked at launch). Otherwise every load
// still is one vector load at a clamped address, and what a ragged edge needs
// (a shift, zeros) is done as the quad goes to LDS: loads behind a branch would
// each be waited for.
// NT: 1, the update's W and U pass by the caches; 2, all but the W it reads (see
// gemm_update).
// LDS: one plane of an operand of R rows (columns) and its pitch, in elements;
// two buffers of an operand's planes.
constexpr int kMapRows = 512;
constexpr int plane_pitch(bool kc, int R, int BK) { return kc ? BK + 8 : R + 32; }
constexpr int plane_size(bool kc, int R, int BK) { return (kc ? R : BK) * plane_pitch(kc, R, BK); }
constexpr int ring_size(bool bf, bool kc, int R, int BK) {
  return 2 * (bf ? 1 : 3) * plane_size(kc, R, BK);
}
template <bool BF, bool AT, bool BT, int EPI, bool GATHER, int BM, int BN, int BK, int D,
          bool FULL, int NT = 0>
__device__ __forceinline__ void gemm_tile(const GemmArgs& a, const Tile t, bf16_t* sA,
                                          bf16_t* sB, int32_t* srmap) {
  constexpr bool kOct = BF && FULL && EPI != EPI_SGD;
  constexpr int VE = kOct ? 8 : 4;  // elements of a vector load
  using Q = std::conditional_t<kOct, Oct, Quad<BF>>;
  using E = typename Q::E;
  using P = std::conditional_t<kOct, u32x4, u32x2>;
  constexpr int NPL = BF ? 1 : 3;
  constexpr int WM = BM / 2, WN = BN / 2, FM = WM / 32, FN = WN / 32;
  constexpr bool AK = !AT, BKc = BT;  // k contiguous in storage
  constexpr int PA = plane_pitch(AK, BM, BK), PB = plane_pitch(BKc, BN, BK);
  constexpr int SA = plane_size(AK, BM, BK), SB = plane_size(BKc, BN, BK);
  constexpr int NA = BM * BK / VE / kThreads, NB = BN * BK / VE / kThreads;
  static_assert(NA >= 1 && NB >= 1 && D % 2 == 0, "tile too small");
  // the k rows of A come from a row map (an update's may have none: its rows
  // in order), the first kMapRows of it in LDS
  constexpr bool kRows = AT && GATHER;
  constexpr bool kScaled = EPI == EPI_STORE;

  const int g = t.g, m0 = t.m0, n0 = t.n0;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lk = lane >> 5, lr = lane & 31;
  const int wm0 = (wave >> 1) * WM, wn0 = (wave & 1) * WN;
  const E* A = (const E*)a.A + (long long)g * a.sA;
  const E* B = (const E*)a.B + (long long)g * a.sB;
  const int32_t* rmap = GATHER && a.rowmap ? a.rowmap + (long long)g * a.sRow : nullptr;
  const int M = a.M, N = a.N;
  const int kbeg = t.s * a.kchunk, kend = min(a.Kd, kbeg + a.kchunk);
  const int nk = (kend - kbeg + BK - 1) / BK;

  // EPI_SGD: the tile's W and U, in accumulator layout, at 32-bit offsets from
  // the tile's corner (clamped where the tile ends); loaded before the last D
  // slabs, when the operand registers fall free (from the start on they cost a
  // fourth workgroup per CU: 107 against 90 us, see gemm_update)
  constexpr bool kUpd = EPI == EPI_SGD;
  float wv[kUpd ? FM : 1][kUpd ? FN : 1][16], uv[kUpd ? FM : 1][kUpd ? FN : 1][16];
  auto out_row = [&](int i, int v) __attribute__((always_inline)) {
    return m0 + wm0 + i * 32 + (v >> 2) * 8 + lk * 4 + (v & 3);
  };
  const long long tile0 = (long long)m0 * a.ldc + n0;
  auto tile_off = [&](int i, int j, int v) __attribute__((always_inline)) {
    int m = out_row(i, v), n = n0 + wn0 + j * 32 + lr;
    if constexpr (!FULL) {
      m = min(m, M - 1);
      n = min(n, N - 1);
    }
    return (unsigned)((m - m0) * (int)a.ldc + (n - n0));
  };
  auto wu_load = [&]() __attribute__((always_inline)) {
    if constexpr (kUpd) {
      const float* Wr =
          (a.Wsrc ? a.Wsrc + (long long)g * a.sWsrc : a.W + (long long)g * a.sC) + tile0;
      const float* Ur = a.U + (long long)g * a.sC + tile0;
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const float* wp = Wr + tile_off(i, j, v);
            const float* up = Ur + tile_off(i, j, v);
            wv[i][j][v] = NT == 1 ? __builtin_nontemporal_load(wp) : *wp;
            uv[i][j][v] = NT != 0 ? __builtin_nontemporal_load(up) : *up;
          }
    }
  };

  if constexpr (kRows) {
    for (int i = tid; i < kMapRows && kbeg + i < kend; i += kThreads)
      srmap[i] = rmap ? rmap[kbeg + i] : kbeg + i;
    __syncthreads();
  }
  // per quad of this thread: the storage offset that does not depend on k
  // (ragged tiles: rows clamped; a quad that reaches past the columns of a
  // k-slow operand is read four before their end and shifted into place)
  long long offA[NA], offB[NB];
  int shA[NA], shB[NB];
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    const int q = tid + i * kThreads;
    shA[i] = 0;
    if constexpr (AK) {
      int r = m0 + q / (BK / VE);
      if constexpr (!FULL) r = min(r, M - 1);
      offA[i] = (GATHER ? (long long)rmap[r] : (long long)r) * a.lda;
    } else {
      const int c = m0 + (q % (BM / VE)) * VE, cc = FULL ? c : max(min(c, M - 4), 0);
      offA[i] = cc;
      shA[i] = c - cc;
    }
  }
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int q = tid + i * kThreads;
    shB[i] = 0;
    if constexpr (BKc) {
      int r = n0 + q / (BK / VE);
      if constexpr (!FULL) r = min(r, N - 1);
      offB[i] = (long long)r * a.ldb;
    } else {
      const int c = n0 + (q % (BN / VE)) * VE, cc = FULL ? c : max(min(c, N - 4), 0);
      offB[i] = cc;
      shB[i] = c - cc;
    }
  }
  auto arow = [&](int k) __attribute__((always_inline)) {  // storage row of A's k
    if constexpr (kRows)
      return (long long)(k - kbeg < kMapRows ? srmap[k - kbeg] : rmap ? rmap[k] : k);
    return (long long)k;
  };
  // fewer than four elements along the contiguous axis: element loads
  const bool thin = !FULL && ((AK || BKc ? a.Kd < 4 : false) || (!AK && M < 4) || (!BKc && N < 4));
  auto gload = [&](int k0, Q(&xa)[NA], Q(&xb)[NB]) __attribute__((always_inline)) {
    if constexpr (!FULL) {
      if (__builtin_expect(thin, 0)) {
#pragma unroll
        for (int i = 0; i < NA; ++i) {
          const int q = tid + i * kThreads;
          const int k = AK ? k0 + (q % (BK / VE)) * VE : k0 + q / (BM / VE);
          const int c = AK ? 0 : (int)offA[i] + shA[i];
          xa[i].zero();
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int ke = AK ? k + e : k;
            if (ke < kend && (AK || c + e < M))
              xa[i].set(e, AK ? A + offA[i] + ke : A + arow(ke) * a.lda + c + e, true);
          }
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
          const int q = tid + i * kThreads;
          const int k = BKc ? k0 + (q % (BK / VE)) * VE : k0 + q / (BN / VE);
          const int c = BKc ? 0 : (int)offB[i] + shB[i];
          xb[i].zero();
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int ke = BKc ? k + e : k;
            if (ke < kend && (BKc || c + e < N))
              xb[i].set(e, BKc ? B + offB[i] + ke : B + (long long)ke * a.ldb + c + e, true);
          }
        }
        return;
      }
    }
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const int q = tid + i * kThreads;
      int k = AK ? k0 + (q % (BK / VE)) * VE : k0 + q / (BM / VE);
      if constexpr (!FULL) k = min(k, kend - (AK ? 4 : 1));
      xa[i].load(AK ? A + offA[i] + k : A + arow(k) * a.lda + offA[i]);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int q = tid + i * kThreads;
      int k = BKc ? k0 + (q % (BK / VE)) * VE : k0 + q / (BN / VE);
      if constexpr (!FULL) k = min(k, kend - (BKc ? 4 : 1));
      xb[i].load(BKc ? B + offB[i] + k : B + (long long)k * a.ldb + offB[i]);
    }
  };
  // ragged tiles: shifted quads into place, zeros past the last k
  const bool edge_m = !FULL && !AK && m0 + BM > M, edge_n = !FULL && !BKc && n0 + BN > N;
  auto fix = [&](int k0, Q(&xa)[NA], Q(&xb)[NB]) __attribute__((always_inline)) {
    if constexpr (!FULL) {
      if (thin) return;
      if (edge_m) {
#pragma unroll
        for (int i = 0; i < NA; ++i) xa[i].shift(shA[i]);
      }
      if (edge_n) {
#pragma unroll
        for (int i = 0; i < NB; ++i) xb[i].shift(shB[i]);
      }
      if (k0 + BK > kend) {
#pragma unroll
        for (int i = 0; i < NA; ++i) {
          const int q = tid + i * kThreads;
          const int k = AK ? k0 + (q % (BK / VE)) * VE : k0 + q / (BM / VE);
          if constexpr (AK) xa[i].shift(max(k - (kend - 4), 0));
          xa[i].keep(AK ? kend - k : (k < kend ? 4 : 0));
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
          const int q = tid + i * kThreads;
          const int k = BKc ? k0 + (q % (BK / VE)) * VE : k0 + q / (BN / VE);
          if constexpr (BKc) xb[i].shift(max(k - (kend - 4), 0));
          xb[i].keep(BKc ? kend - k : (k < kend ? 4 : 0));
        }
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
      const int o = AK ? (q / (BK / VE)) * PA + (q % (BK / VE)) * VE
                       : (q / (BM / VE)) * PA + (q % (BM / VE)) * VE;
      P p[NPL];
      xa[i].template planes<kScaled>(p);
#pragma unroll
      for (int l = 0; l < NPL; ++l) *(P*)&sA[(buf * NPL + l) * SA + o] = p[l];
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int q = tid + i * kThreads;
      const int o = BKc ? (q / (BK / VE)) * PB + (q % (BK / VE)) * VE
                        : (q / (BN / VE)) * PB + (q % (BN / VE)) * VE;
      P p[NPL];
      xb[i].template planes<kScaled>(p);
#pragma unroll
      for (int l = 0; l < NPL; ++l) *(P*)&sB[(buf * NPL + l) * SB + o] = p[l];
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
    auto put = [&](int sl, int buf, Q(&xa)[NA], Q(&xb)[NB]) __attribute__((always_inline)) {
      fix(slab(sl), xa, xb);
      colsums(xb);
      lstore(buf, xa, xb);
    };
    put(0, 0, ra[0], rb[0]);
    __syncthreads();
    int it = 0;
    for (; it + D < nk; it += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        gload(slab(it + d + D), ra[d], rb[d]);
        __builtin_amdgcn_sched_barrier(0);
        compute(d & 1);
        put(it + d + 1, (d + 1) & 1, ra[(d + 1) % D], rb[(d + 1) % D]);
        __syncthreads();
      }
    }
    wu_load();  // on their way while the last slabs compute
#pragma unroll
    for (int d = 0; d < D; ++d) {
      if (it + d >= nk) break;
      compute(d & 1);
      if (it + d + 1 < nk) put(it + d + 1, (d + 1) & 1, ra[(d + 1) % D], rb[(d + 1) % D]);
      __syncthreads();
    }
  }
  if constexpr (!BF) {
    float sum = 0.f;  // an infinity or a NaN among the results shows in it
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          hi[i][j][v] += lo[i][j][v];
          sum += hi[i][j][v];
          if constexpr (kScaled) hi[i][j][v] *= kSplitUnscale;
        }
    if (__builtin_expect(__any(!__builtin_isfinite(sum)) || kend - kbeg <= 2, 0)) {
      // the fp32 instruction, from memory
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          const int m = min(m0 + wm0 + i * 32 + lr, M - 1), n = min(n0 + wn0 + j * 32 + lr, N - 1);
          const int kmid = kbeg + (kend - kbeg) / 4 * 2;
#pragma unroll
          for (int v = 0; v < 16; ++v) hi[i][j][v] = 0.f;
#pragma unroll 1
          for (int half = 0; half < 2; ++half) {  // (two sums round less than one)
            const int ke = half ? kend : kmid;
            floatx16 acc;
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] = 0.f;
            for (int k = half ? kmid : kbeg; k < ke; k += 2) {
              const int kx = k + lk, kc = min(kx, ke - 1);
              const long long oa = AT ? arow(kc) * a.lda + m
                                      : (GATHER ? (long long)rmap[m] : (long long)m) * a.lda + kc;
              const long long ob = BT ? (long long)n * a.ldb + kc : (long long)kc * a.ldb + n;
              const float x = kx < ke ? ((const float*)A)[oa] : 0.f;
              const float y = kx < ke ? ((const float*)B)[ob] : 0.f;
              acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x, y, acc, 0, 0, 0);
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) hi[i][j][v] += acc[v];
          }
        }
    }
  }

  // epilogue
  constexpr bool OUTBF = BF && (EPI == EPI_BIAS_RELU || EPI == EPI_RELU_MASK);
  if constexpr (kUpd) {
    const long long t0 = (long long)g * a.sC + tile0;
    float* Wt = a.W + t0;
    float* Ut = a.U + t0;
    bf16_t* Wbt = a.Wb + t0;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int m = out_row(i, v), n = n0 + wn0 + j * 32 + lr;
          if (!FULL && (m >= M || n >= N)) continue;
          const unsigned o = tile_off(i, j, v);
          sgd_step(wv[i][j][v], uv[i][j][v], hi[i][j][v], a);
          if constexpr (NT != 0) {
            __builtin_nontemporal_store(wv[i][j][v], Wt + o);
            __builtin_nontemporal_store(uv[i][j][v], Ut + o);
          } else {
            Wt[o] = wv[i][j][v];
            Ut[o] = uv[i][j][v];
          }
          if (a.Wb) Wbt[o] = f32_to_bf16(wv[i][j][v]);
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

template <bool BF, bool AT, bool BT, int EPI, bool GATHER, int BM, int BN, int BK, int D,
          bool FULL>
__global__ __launch_bounds__(kThreads, BM * BN > 128 * 64 ? 1 : 2) void gemm_mm(GemmArgs a) {
  __shared__ __attribute__((aligned(16))) bf16_t sA[ring_size(BF, !AT, BM, BK)];
  __shared__ __attribute__((aligned(16))) bf16_t sB[ring_size(BF, BT, BN, BK)];
  const Tile t = decode_tile(a, BM, BN);
  if (t.g < 0) return;
  gemm_tile<BF, AT, BT, EPI, GATHER, BM, BN, BK, D, FULL>(a, t, sA, sB, nullptr);
}

// Weight gradients fused with their momentum-SGD step, of one or several
// layers: their 64 x 64 tiles concatenated in one launch. HBM-bound (W and U
// read and written, 16 B per weight): a workgroup's k loop and its update
// stream are short, so what counts is how many are in flight -- four per CU
// (37 KB of LDS at BK = 16, 128 registers) drift apart and keep both busy.
// 16 x 3072 x 512 from 128 gathered rows: 90 us, 4.7 TB/s with the operands;
// at three workgroups per CU 101-107, BK = 32 and two 116, and a persistent
// form of eight waves (four computing 128 x 128 tiles, four updating the tile
// before) 105 on the fp32 instruction. Ragged tiles (FULL false) need the
// registers of two slabs for their addresses: D = 2 (12 x 1537 x 771 from 90
// rows: 69 us, D = 4 77, spilling). NT: a state beyond the 256 MB Infinity
// Cache is streamed past the caches (64 x 3072 x 2048: fp32 1292 -> 1190 us,
// bf16 1427 -> 1347 us, 5.4 TB/s; a state that fits loses the lines the next
// step reads: 86 -> 92 us); the one mean that all replicas read while a lazy
// average is pending stays in the caches (NT 2: 64 x 3072-2048-2048-10, all
// layers, bf16 2229 -> 1979 us, fp32 1956 -> 1812).
struct UpdArgs {
  GemmArgs p[kUpdMaxProblems];
  int start[kUpdMaxProblems + 1];  // first tile of each problem; [np] = total
  int np;
  unsigned whole;  // bit i: problem i has whole tiles and slabs only
  StepTail tail;
  int nloss, ntail;  // workgroups of the losses; of the tail (a multiple of 8)
};

// The tail's workgroup p: a replica's loss, or 256 threads of the sampler. They
// come first in the grid, so they end long before the tiles do. (As launches of
// their own on a side stream, behind an event each way, they cost the step
// about 16 us.)
__device__ __forceinline__ void step_tail(const UpdArgs& w, int p, float* red) {
  const StepTail& t = w.tail;
  const int tid = threadIdx.x;
  if (p < w.nloss) {
    float part = 0.f;  // strided partial sums, then a fixed tree
    for (int b = tid; b < t.B; b += kThreads) part += t.rowloss[(long long)p * t.B + b];
    red[tid] = part;
    __syncthreads();
    for (int n = kThreads / 2; n > 0; n >>= 1) {
      if (tid < n) red[tid] += red[tid + n];
      __syncthreads();
    }
    if (tid == 0) {
      const float mean = red[0] / (float)t.B;
      if (t.loss) t.loss[p] = mean;
      // a plain store: every writer stores the same value
      if (t.nonfinite && !isfinite(mean)) *t.nonfinite = 1;
    }
    return;
  }
  if (!t.idx) return;
  const long long i = (long long)(p - w.nloss) * kThreads + tid;
  if (t.epoch) {
    if (i >= (long long)t.K * t.B) return;
    const int k = (int)(i / t.B), b = (int)(i - (long long)k * t.B);
    const uint32_t q = (uint32_t)((long long)k * t.N / t.K + t.j * t.B + b);
    t.idx[i] = epoch_row(q, t.N, t.m, t.key0, t.key1, t.e);
  } else {
    const int quads = (t.B + 3) / 4;
    if (i >= (long long)t.K * quads) return;
    const int k = (int)(i / quads);
    sample_iid4(t.key0, t.key1, t.s_lo, t.s_hi, k, t.K, t.N, t.B, (int)(i - (long long)k * quads),
                t.idx);
  }
}

// (bf16: whole tiles in slabs of 64, 94 against 95 us for 16 x 3072 x 512)
template <bool BF, int NT>
__global__ __launch_bounds__(kThreads, BF ? 3 : 4) void gemm_update(UpdArgs w) {
  constexpr int BK = BF ? 64 : 16;
  __shared__ __attribute__((aligned(16))) bf16_t sA[ring_size(BF, false, 64, BK)];
  __shared__ __attribute__((aligned(16))) bf16_t sB[ring_size(BF, false, 64, BK)];
  __shared__ int32_t srmap[kMapRows];
  const unsigned id = workgroup_id();
  if (id < (unsigned)w.ntail) {
    step_tail(w, id, (float*)sA);
    return;
  }
  const int total = w.start[w.np];
  if (id - w.ntail >= (unsigned)total) return;
  const int p = id - w.ntail;
  int l = (total % kXcds == 0) ? (p % kXcds) * (total / kXcds) + p / kXcds : p;
  int pi = 0;
  while (pi + 1 < w.np && l >= w.start[pi + 1]) ++pi;
  l -= w.start[pi];
  const GemmArgs& a = w.p[pi];
  const int tn = (a.N + 63) / 64, per_g = tn * ((a.M + 63) / 64);
  Tile t;
  t.s = 0;
  t.g = l / per_g;
  l -= t.g * per_g;
  t.m0 = (l / tn) * 64;
  t.n0 = (l % tn) * 64;
  if (w.whole >> pi & 1u)  // uniform
    gemm_tile<BF, true, false, EPI_SGD, true, 64, 64, BK, BF ? 2 : 4, true, NT>(a, t, sA, sB, srmap);
  else
    gemm_tile<BF, true, false, EPI_SGD, true, 64, 64, BF ? 32 : 16, 2, false, NT>(a, t, sA, sB,
                                                                                  srmap);
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

// Tile of a forward, input-gradient or plain product. Larger tiles read less
// from LDS per MFMA, but a launch should have a workgroup for each of the 256
// CUs (two of the 128 x 64 ones): 128 x 128 (fp32) or 128 x 64 tiles where the
// output has that many, or where the inner dimension is long enough for
// split-K to get there; else 64 x 64. Measured, 16 replicas of 128 x 512 x
// 3072, fp32 with the partials' sum: 128 x 128 split 4 46 us, 128 x 64 split 4
// 51-58, 64 x 64 split 2 53; 128 x 512 x 512: 64 x 64 12 us, 128 x 64 18.
// Between one and nearly two rounds of 128 x 128 tiles (one a CU) 64 x 64 ones
// leave less of the chip idle at the end: fp32 5 x 700 x 1100 x 784 (270 tiles)
// 96 us, 59 as 64 x 64; 28 x 128 x 2048 x 256 (448) 35.7, 35.4; 31 x 256 x 1024
// x 512 (496) 61, 68.
// A caller's product without split-K takes larger tiles only where they fill the
// chip by themselves (16 x 128 x 512 x 3072 in bf16: 31 us as 128 x 64, 16 as 64 x 64).
struct Shape {
  int BM, BN;
};
Shape tile_shape(bool bf, int M, int N, int G, int Kd, bool split = true) {
  if (M <= 64 || N <= 64) return {64, 64};
  const bool deep = split && Kd >= 2048;
  const long long t128 = (long long)((M + 127) / 128) * ((N + 127) / 128) * G;
  if (!bf && !deep && t128 > 256 && t128 < 480) return {64, 64};
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
    hipLaunchKernelGGL((gemm_mm<BF, AT, BT, EPI, GATHER, BM, BN, BK, D, true>), grid_of(total),
                       dim3(kThreads), 0, s, a);
  else
    hipLaunchKernelGGL((gemm_mm<BF, AT, BT, EPI, GATHER, BM, BN, BK, D, false>), grid_of(total),
                       dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

template <bool BF, bool AT, bool BT, int EPI, bool GATHER>
hipError_t run_type(const GemmArgs& a, hipStream_t s) {
  const Shape sh = tile_shape(BF, a.M, a.N, a.G, a.Kd, a.splits > 1);
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

template <bool AT, bool BT, int EPI, bool GATHER>
hipError_t run(int dtype, const GemmArgs& a, hipStream_t s) {
  return dtype == 1 ? run_type<true, AT, BT, EPI, GATHER>(a, s)
                    : run_type<false, AT, BT, EPI, GATHER>(a, s);
}

template <bool AT, bool BT, int EPI>
hipError_t dispatch(int dtype, const GemmArgs& a, hipStream_t s) {
  if (a.rowmap) {  // gathered rows: the first layer's forward
    if constexpr (EPI == EPI_STORE || EPI == EPI_RELU_MASK)
      return hipErrorInvalidValue;
    else
      return run<AT, BT, EPI, true>(dtype, a, s);
  }
  return run<AT, BT, EPI, false>(dtype, a, s);
}

}  // namespace

void step_tail_sample(StepTail& t, int epoch, uint64_t seed, int64_t step, int64_t N,
                      int32_t* idx) {
  t.idx = idx;
  t.epoch = epoch;
  t.key0 = (uint32_t)seed;
  t.key1 = (uint32_t)(seed >> 32);
  t.s_lo = (uint32_t)step;
  t.s_hi = (uint32_t)((uint64_t)step >> 32);
  t.N = N;
  if (epoch) {
    const long long S = (N / t.K) / t.B;  // batches per worker and epoch, >= 1
    t.e = (uint32_t)(step / S);
    t.j = step % S;
    t.m = 1;
    while ((1LL << (2 * t.m)) < N) ++t.m;
  }
}

hipError_t launch_gemm_update(int dtype, const GemmArgs* list, int n, const StepTail& tail,
                              hipStream_t s) {
  if (n < 1 || n > kUpdMaxProblems) return hipErrorInvalidValue;
  UpdArgs w{};
  w.np = n;
  w.tail = tail;
  w.nloss = tail.rowloss ? tail.K : 0;
  const long long slots = !tail.idx ? 0 : (long long)tail.K * (tail.epoch ? tail.B : (tail.B + 3) / 4);
  const long long extra = w.nloss + (slots + kThreads - 1) / kThreads;
  if (extra > 0x7fffffffLL - kXcds) return hipErrorInvalidValue;
  w.ntail = (int)((extra + kXcds - 1) / kXcds * kXcds);
  long long total = 0, state = 0;  // tiles; bytes of W, U and the bf16 copy
  bool shared = false;             // W is read from one model for all replicas
  for (int i = 0; i < n; ++i) {
    GemmArgs& a = w.p[i];
    a = list[i];
    if (a.G <= 0 || a.M <= 0 || a.N <= 0 || a.Kd <= 0) return hipErrorInvalidValue;
    a.splits = 1;
    a.kchunk = (a.Kd + 31) / 32 * 32;
    if (full(a, 64, 64, dtype == 1 ? 64 : 16)) w.whole |= 1u << i;
    state += (long long)a.G * a.M * a.N * (a.Wb ? 10 : 8);
    shared |= a.Wsrc && a.sWsrc == 0;
    w.start[i] = (int)total;
    total += (long long)((a.M + 63) / 64) * ((a.N + 63) / 64) * a.G;
    if (total > 0x7fffffffLL) return hipErrorInvalidValue;
  }
  w.start[n] = (int)total;
  const int nt = state < kNtBytes ? 0 : shared ? 2 : 1;
  if (total + w.ntail > 0x7fffffffLL) return hipErrorInvalidValue;
  const dim3 grid = grid_of(total + w.ntail), block(kThreads);
#define LSGD_UPDATE(BF, NT) \
  hipLaunchKernelGGL((gemm_update<BF, NT>), grid, block, 0, s, w)
  if (dtype == 1) {
    if (nt == 0) LSGD_UPDATE(true, 0);
    if (nt == 1) LSGD_UPDATE(true, 1);
    if (nt == 2) LSGD_UPDATE(true, 2);
  } else {
    if (nt == 0) LSGD_UPDATE(false, 0);
    if (nt == 1) LSGD_UPDATE(false, 1);
    if (nt == 2) LSGD_UPDATE(false, 2);
  }
#undef LSGD_UPDATE
  return hipGetLastError();
}

int gemm_splits(int dtype, int M, int N, int Kd, int G) {
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
  if (a.splits > 1 && a.part == nullptr) return hipErrorInvalidValue;
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
    default:
      break;
  }
  return hipErrorInvalidValue;
}

}  // namespace lsgd
