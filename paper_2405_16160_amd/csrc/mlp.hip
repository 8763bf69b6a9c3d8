// Warm-start network on the GPU: bfloat16 matrix products on MFMA with FP32
// accumulation, fused bias / ReLU / ReLU-derivative epilogues, MSE gradient,
// bias-gradient column sums and Adam on FP32 master weights.  Host side of
// include/pdhcg_mlp.h at the end of the file.
#include <hip/hip_runtime.h>
#include <math.h>
#include <string.h>

#include <string>
#include <vector>

#include "../../include/pdhcg.h"
#include "../../include/pdhcg_mlp.h"
#include "internal.hpp"

namespace pdhcg {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// float -> bfloat16, round to nearest, ties to even (NaN kept quiet)
__device__ __forceinline__ uint16_t to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float from_bf16(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

// k per LDS stage (four K = 32 MFMA steps per round trip to memory; 256 would
// leave two workgroups per CU instead of three: 256 x 5500 x 512 18.3 us against
// 16.7 us)
constexpr int GK = 128;
constexpr int GP = 8;    // LDS row padding (bf16 elements): the 16-byte fragment reads of 16 rows fall on all 64 banks once

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
// vectors at any element address (a row of an odd-sized matrix starts at one):
// the hardware takes unaligned global accesses
typedef uint16_t u16x8u __attribute__((ext_vector_type(8), aligned(2)));
typedef uint16_t u16x4u __attribute__((ext_vector_type(4), aligned(2)));
typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));
typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));

// One operand's R x GK tile on its way from memory to LDS, R / 4 elements per
// thread held in registers while earlier stages are multiplied.  The matrix is
// rows x k; KC: k is the contiguous direction (element (r, k) at r * ld + k, 16
// bytes per load); else r is (element at k * ld + r): a thread then takes 4 k by
// 4 r, 8 bytes per load, and turns them so that its 4 k of a row are one 8-byte
// LDS store.  Loads are unconditional (a branch around them would make the
// compiler wait for one before the next): the direction across the rows of
// memory is clamped into the matrix, along a row they may run past its end by
// less than a stage, which every operand's buffer has behind its last row
// (kPad).  What lies beyond the matrix stays in rows whose results are not
// stored; k beyond the range is cleared in LDS (gemm_tile).
constexpr int kPad = GK + 8;
template <int R, bool KC>
struct TileStage {
  static constexpr int NV = KC ? R * GK / 2048 : R * GK / 4096;
  u16x8 v8[KC ? NV : 1];
  u16x4 v4[KC ? 1 : NV][4];

  __device__ __forceinline__ void load(const uint16_t* __restrict__ M, uint32_t ld, int r0, int k0, int nr, int ke) {
    const int tid = threadIdx.x;
    if constexpr (KC) {
#pragma unroll
      for (int u = 0; u < NV; ++u) {
        const int q = tid + u * 256, gr = min(r0 + q / (GK / 8), nr - 1), gk = k0 + (q % (GK / 8)) * 8;
        v8[u] = *reinterpret_cast<const u16x8u*>(M + (uint64_t)(uint32_t)gr * ld + gk);
      }
    } else {
#pragma unroll
      for (int u = 0; u < NV; ++u) {
        const int q = tid + u * 256, gr = r0 + (q % (R / 4)) * 4, gk = k0 + (q / (R / 4)) * 4;
#pragma unroll
        for (int j = 0; j < 4; ++j)
          v4[u][j] = *reinterpret_cast<const u16x4u*>(M + (uint64_t)(uint32_t)min(gk + j, ke - 1) * ld + gr);
      }
    }
  }

  __device__ __forceinline__ void store(uint16_t (*T)[GK + GP]) const {
    const int tid = threadIdx.x;
    if constexpr (KC) {
#pragma unroll
      for (int u = 0; u < NV; ++u) {
        const int q = tid + u * 256;
        *reinterpret_cast<u16x8*>(&T[q / (GK / 8)][(q % (GK / 8)) * 8]) = v8[u];
      }
    } else {
#pragma unroll
      for (int u = 0; u < NV; ++u) {
        const int q = tid + u * 256, r = (q % (R / 4)) * 4, k = (q / (R / 4)) * 4;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          *reinterpret_cast<u16x4*>(&T[r + e][k]) = u16x4{v4[u][0][e], v4[u][1][e], v4[u][2][e], v4[u][3][e]};
      }
    }
  }
};

// Where a product's values go: with part set, the raw partial product of k
// chunk z to part[z][m][n]; else v + bias[n], ReLU, zero where mask(m, n) <= 0
// (the ReLU derivative), and then, by what is set: decoded start points (x0,
// decode_value); the mean-squared error against T (loss, mse_value); cf (FP32)
// and/or cb (bfloat16).
struct GemmOut {
  const float* bias;
  int relu;
  const uint16_t* mask;
  float* cf;
  uint16_t* cb;
  int64_t ldc;
  float* part;
  // decoded outputs
  const double *mu, *sd;
  int n, n_pair, m;
  const int32_t *plus, *minus, *rest;
  double *x0, *y0;
  // mean-squared error: row m of T is its row rows[m] when rows is given;
  // loss[workgroup] receives the workgroup's sum of (v - T)^2
  const float* T;
  const int32_t* rows;
  float scale;
  double* loss;
};

typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef double f64x2u __attribute__((ext_vector_type(2), aligned(8)));

// v + bias, ReLU, zero where masked
__device__ __forceinline__ float epilogue(const GemmOut& o, float v, float bias, bool masked) {
  if (o.bias) v += bias;
  if (o.relu) v = v > 0.f ? v : 0.f;
  return masked ? 0.f : v;
}

// Column c of the network's output as it enters the start point, in rows of the
// packed x0 (n per row) and y0 (m per row): c < n gives x_c = z sd_c + mu_c;
// column n + p (p < n_pair) the multiplier lam of the p-th equality pair,
// y[plus_p] = max(lam, 0) and y[minus_p] = max(-lam, 0); column n + n_pair + q
// gives y[rest_q] = max(v, 0).
struct DecodeColumn {
  double sd, mu;
  double *a, *b;  // its first element in x0 or y0, and (of a pair) the second in y0
  int ld;
  bool dual;
  __device__ __forceinline__ void set(const GemmOut& o, int c) {
    sd = o.sd[c];
    mu = o.mu[c];
    b = nullptr;
    dual = c >= o.n;
    ld = dual ? o.m : o.n;
    if (!dual) {
      a = o.x0 + c;
    } else if (c < o.n + o.n_pair) {
      a = o.y0 + o.plus[c - o.n];
      b = o.y0 + o.minus[c - o.n];
    } else {
      a = o.y0 + o.rest[c - o.n - o.n_pair];
    }
  }
  // The product and the sum are rounded separately (contraction into a fused
  // multiply-add is switched off here), as a host computation of the same
  // formula does.
  __device__ __forceinline__ double value(float z) const {
#pragma clang fp contract(off)
    return (double)z * sd + mu;
  }
  __device__ __forceinline__ double first(double v) const { return dual ? (v > 0.0 ? v : 0.0) : v; }
  __device__ __forceinline__ double second(double v) const { return -v > 0.0 ? -v : 0.0; }
};

struct Gemm {
  int M, N, K;
  const uint16_t* A;
  uint32_t lda;
  const uint16_t* B;
  uint32_t ldb;
  int kchunk;
  int gx, gy, gz;  // workgroups along n, m and (out.part) the k chunks
  GemmOut out;
};

template <int BM, int BN>
struct GemmLds {
  uint16_t As[BM][GK + GP];
  uint16_t Bt[BN][GK + GP];  // B tile stored as [n][k]
};

// The epilogue's per-element inputs of a thread of a 64 x 64 tile (its four
// columns of every 16th row): the targets or the mask, loaded before the product
// starts so that the epilogue does not wait for them.
struct EpilogueIn {
  f32x4 t[4];
  u16x4 k[4];
  __device__ __forceinline__ void load(const Gemm& g, int m0, int n0) {
    const GemmOut& o = g.out;
    const int tid = threadIdx.x, n = n0 + (tid % 16) * 4;
    if (o.loss) {
      int row[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int m = min(m0 + tid / 16 + 16 * u, g.M - 1);
        row[u] = o.rows ? o.rows[m] : m;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const float* p = o.T + (int64_t)row[u] * o.ldc;
        if (n + 4 <= g.N) {
          t[u] = *reinterpret_cast<const f32x4u*>(p + n);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) t[u][e] = p[min(n + e, g.N - 1)];
        }
      }
    }
    if (o.mask && !o.part) {  // (past a row's end: inside the buffer's padding)
#pragma unroll
      for (int u = 0; u < 4; ++u)
        k[u] = *reinterpret_cast<const u16x4u*>(o.mask + (int64_t)min(m0 + tid / 16 + 16 * u, g.M - 1) * o.ldc + n);
    }
  }
};

// The epilogue of a BM x BN tile C: a thread keeps its four columns and takes
// every 1024 / BN-th row.  pre: its inputs (64 x 64 tiles).
template <int BM, int BN>
__device__ __forceinline__ void emit(const Gemm& g, int m0, int n0, int wg, int bz, float (*C)[BN + 4],
                                     const EpilogueIn& pre) {
  constexpr bool kPre = BM == 64 && BN == 64;
  constexpr int kRows = BM * BN / 1024, kUnroll = kPre ? kRows : 2;
  const GemmOut& o = g.out;
  const int tid = threadIdx.x, c = (tid % (BN / 4)) * 4, n = n0 + c;
  const int w = min(4, g.N - n);  // columns in range (<= 0: none)
  const bool full = w == 4;
  double loss = 0.0;
  float bias[4] = {0.f, 0.f, 0.f, 0.f};
  DecodeColumn dc[4];
  bool vec = full;  // decoded columns side by side in one array
  if (w > 0 && !o.part) {
    if (o.bias) {
#pragma unroll
      for (int e = 0; e < 4; ++e) bias[e] = o.bias[min(n + e, g.N - 1)];
    }
    if (o.x0) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        dc[e].set(o, min(n + e, g.N - 1));
        vec = vec && dc[e].a == dc[0].a + e && dc[e].dual == dc[0].dual && (dc[0].b ? dc[e].b == dc[0].b + e : !dc[e].b);
      }
    }
  }
#pragma unroll kUnroll
  for (int u = 0; u < kRows; ++u) {
    const int row = tid / (BN / 4) + u * (1024 / BN), m = m0 + row;
    if (m >= g.M || w <= 0) continue;
    float v[4];
    {
      const f32x4 t = *reinterpret_cast<const f32x4*>(&C[row][c]);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = t[e];
    }
    if (o.part) {
      float* p = o.part + ((int64_t)bz * g.M + m) * g.N + n;
      if (full) {
        *reinterpret_cast<f32x4u*>(p) = f32x4u{v[0], v[1], v[2], v[3]};
      } else {
#pragma unroll
        for (int e = 0; e < 3; ++e)
          if (e < w) p[e] = v[e];
      }
      continue;
    }
    const int64_t at = (int64_t)m * o.ldc + n;
    bool masked[4] = {false, false, false, false};
    if (o.mask) {  // (read past a row's end: inside the buffer's padding)
      u16x4 k;
      if constexpr (kPre) k = pre.k[u];
      else k = *reinterpret_cast<const u16x4u*>(o.mask + at);
#pragma unroll
      for (int e = 0; e < 4; ++e) masked[e] = !(from_bf16(k[e]) > 0.f);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = epilogue(o, v[e], bias[e], masked[e]);
    if (o.x0) {
      double d[4], f[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        d[e] = dc[e].value(v[e]);
        f[e] = dc[e].first(d[e]);
      }
      if (vec) {
        double* p = dc[0].a + (int64_t)m * dc[0].ld;
        *reinterpret_cast<f64x2u*>(p) = f64x2u{f[0], f[1]};
        *reinterpret_cast<f64x2u*>(p + 2) = f64x2u{f[2], f[3]};
        if (dc[0].b) {
          p = dc[0].b + (int64_t)m * dc[0].ld;
          *reinterpret_cast<f64x2u*>(p) = f64x2u{dc[0].second(d[0]), dc[1].second(d[1])};
          *reinterpret_cast<f64x2u*>(p + 2) = f64x2u{dc[2].second(d[2]), dc[3].second(d[3])};
        }
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (e < w) {
            dc[e].a[(int64_t)m * dc[e].ld] = f[e];
            if (dc[e].b) dc[e].b[(int64_t)m * dc[e].ld] = dc[e].second(d[e]);
          }
      }
      continue;
    }
    if (o.loss) {
      float tv[4];
      if constexpr (kPre) {
#pragma unroll
        for (int e = 0; e < 4; ++e) tv[e] = pre.t[u][e];
      } else {
        const float* t = o.T + (int64_t)(o.rows ? o.rows[m] : m) * o.ldc;
#pragma unroll
        for (int e = 0; e < 4; ++e) tv[e] = t[min(n + e, g.N - 1)];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float d = v[e] - tv[e];
        if (e < w) loss += (double)d * (double)d;
        v[e] = 2.0f * d * o.scale;
      }
    }
    if (full) {
      if (o.cf) *reinterpret_cast<f32x4u*>(o.cf + at) = f32x4u{v[0], v[1], v[2], v[3]};
      if (o.cb) *reinterpret_cast<u16x4u*>(o.cb + at) = u16x4u{to_bf16(v[0]), to_bf16(v[1]), to_bf16(v[2]), to_bf16(v[3])};
    } else {
#pragma unroll
      for (int e = 0; e < 3; ++e)
        if (e < w) {
          if (o.cf) o.cf[at + e] = v[e];
          if (o.cb) o.cb[at + e] = to_bf16(v[e]);
        }
    }
  }
  if (o.loss) {  // the workgroup's squared error, in a fixed order
    double* const red = reinterpret_cast<double*>(C);
    __syncthreads();
    red[tid] = loss;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
      if (tid < k) red[tid] += red[tid + k];
      __syncthreads();
    }
    if (tid == 0) o.loss[wg] = red[0];
  }
}

// C = A B on bfloat16 operands with FP32 accumulation, A(m,k) and B(k,n) each
// contiguous along k (AKC, BKC) or along m, n, so transposed operands need no
// copy.  A workgroup of four waves forms a BM x BN tile, each wave a quarter as
// tiles of the gfx950 MFMA 16x16x32 (eight bfloat16 per lane and operand).
//
// What bounds it: at these sizes (256 rows, 512 hidden units) a workgroup's
// chain of k stages, each a round trip to the last-level cache (about 1 us: a
// kernel starts with cold L2s), not the matrix cores.  So a stage is deep, the
// next one is on its way in registers while this one is multiplied, and the
// epilogue's inputs are loaded at the start.  256 x 5500 x 512 with the MSE
// gradient in its epilogue: 16.7 us; with a 32-deep stage loaded, stored and
// multiplied in turn 32.9 us, and 11.0 us for the gradient's own kernel.
//
// The k range is taken in chunks of kchunk; every chunk is summed from zero and
// the chunks' sums are added in order.  With out.part, workgroup z takes chunk z
// alone and splitk_finish adds them (few output tiles and a long k: more CUs
// take part); without it one workgroup takes them all, to the same bits (in 64 x
// 64 tiles: the second set of sums would leave a 128 x 128 tile one wave per
// SIMD).
template <int BM, int BN, bool AKC, bool BKC>
__device__ __forceinline__ void gemm_tile(const Gemm& g, int bx, int by, int bz, GemmLds<BM, BN>& L) {
  constexpr int MI = BM / 32, NJ = BN / 32;
  constexpr bool kFold = BM == 64 && BN == 64;
  const GemmOut& out = g.out;
  const int M = g.M, N = g.N, K = g.K, kchunk = g.kchunk;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave >> 1) * (BM / 2), wn = (wave & 1) * (BN / 2);
  const int m0 = by * BM, n0 = bx * BN;
  f32x4 acc[MI][NJ], sum[kFold ? MI : 1][kFold ? NJ : 1];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      if constexpr (kFold) sum[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  const int kstart = out.part ? bz * kchunk : 0;
  const int kend = out.part ? min(K, kstart + kchunk) : K;
  const bool folds = kFold && kstart + kchunk < kend;
  // a stage: k from kb, its chunk ending at ke (kb >= kend: none)
  struct Stage {
    int kb, ke;
  };
  auto after = [&](Stage t) {
    t.kb += GK;
    if (t.kb >= t.ke) {
      t.kb = t.ke;
      t.ke = min(kend, t.ke + kchunk);
    }
    return t;
  };
  EpilogueIn pre;
  if constexpr (BM == 64 && BN == 64) pre.load(g, m0, n0);
  TileStage<BM, AKC> sa;
  TileStage<BN, BKC> sb;
  Stage cur{kstart, min(kend, kstart + kchunk)};
  sa.load(g.A, g.lda, m0, cur.kb, M, cur.ke);
  sb.load(g.B, g.ldb, n0, cur.kb, N, cur.ke);
  for (;;) {
    sa.store(L.As);
    sb.store(L.Bt);
    const int depth = min(GK, cur.ke - cur.kb);
    if (depth & 31) {  // the last step's k beyond the range: zero in both operands
      __syncthreads();
      const int k = (depth & ~31) + (tid & 31);
      if (k >= depth) {
        for (int r = tid >> 5; r < BM; r += 8) L.As[r][k] = 0;
        for (int r = tid >> 5; r < BN; r += 8) L.Bt[r][k] = 0;
      }
    }
    __syncthreads();
    const Stage nxt = after(cur);
    const bool more = nxt.kb < kend;
    if (more) {
      sa.load(g.A, g.lda, m0, nxt.kb, M, nxt.ke);
      sb.load(g.B, g.ldb, n0, nxt.kb, N, nxt.ke);
    }
#pragma unroll 2
    for (int ks = 0; ks < depth; ks += 32) {
      bf16x8 a[MI], b[NJ];
#pragma unroll
      for (int i = 0; i < MI; ++i)
        a[i] = *reinterpret_cast<const bf16x8*>(&L.As[wm + i * 16 + (lane & 15)][ks + 8 * (lane >> 4)]);
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        b[j] = *reinterpret_cast<const bf16x8*>(&L.Bt[wn + j * 16 + (lane & 15)][ks + 8 * (lane >> 4)]);
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    if constexpr (kFold) {
      if (folds && nxt.kb == cur.ke) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j) {
            sum[i][j] += acc[i][j];
            acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
          }
      }
    }
    if (!more) break;
    __syncthreads();
    cur = nxt;
  }
  // the tile through LDS, so that the epilogue is a short loop (code that runs
  // once is fetched from memory once per CU: with the epilogue unrolled over the
  // accumulators a kernel of one stage took 8 us) and stores whole vectors
  __syncthreads();
  float(*const C)[BN + 4] = reinterpret_cast<float(*)[BN + 4]>(&L);
  static_assert(sizeof(float) * BM * (BN + 4) <= sizeof(L), "the tile fits the staging area");
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float v = acc[i][j][r];
        if constexpr (kFold) v = folds ? sum[i][j][r] : v;
        C[wm + i * 16 + 4 * (lane >> 4) + r][wn + j * 16 + (lane & 15)] = v;
      }
  __syncthreads();
  emit<BM, BN>(g, m0, n0, by * g.gx + bx, bz, C, pre);
}

template <int BM, int BN, bool AKC, bool BKC>
__global__ void __launch_bounds__(256) gemm_bf16(Gemm g) {
  __shared__ __attribute__((aligned(16))) GemmLds<BM, BN> L;
  gemm_tile<BM, BN, AKC, BKC>(g, blockIdx.x, blockIdx.y, blockIdx.z, L);
}

// Two independent products of one layer's backward pass in one launch: the
// weight gradient H' G (w) and the gradient of the layer's input G W' (h).  Each
// alone is a latency chain that leaves most of the GPU idle (output layer, 256
// rows, 512 x 5500: 21.4 and 42.7 us apart before, 19.0 us together).
__global__ void __launch_bounds__(256) gemm_backward(Gemm w, Gemm h) {
  __shared__ __attribute__((aligned(16))) GemmLds<64, 64> L;
  const int nh = h.gx * h.gy * h.gz;
  int b = blockIdx.x;
  if (b < nh) {  // (the longer chain first)
    const int bx = b % h.gx, q = b / h.gx;
    gemm_tile<64, 64, true, true>(h, bx, q % h.gy, q / h.gy, L);
  } else {
    b -= nh;
    gemm_tile<64, 64, false, false>(w, b % w.gx, b / w.gx, 0, L);
  }
}

// sum of the split-K partials in order z = 0 .. S-1, then the epilogue
__global__ void splitk_finish(const float* __restrict__ Cpart, int S, int M, int N, GemmOut out) {
  const int64_t mn = (int64_t)M * N;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < mn; e += (int64_t)gridDim.x * blockDim.x) {
    float v = 0.f;
#pragma unroll 8
    for (int z = 0; z < S; ++z) v += Cpart[z * mn + e];
    const int m = (int)(e / N), n = (int)(e - (int64_t)m * N);
    const bool masked = out.mask && !(from_bf16(out.mask[(int64_t)m * out.ldc + n]) > 0.f);
    v = epilogue(out, v, out.bias ? out.bias[n] : 0.f, masked);
    if (out.x0) {
      DecodeColumn d;
      d.set(out, n);
      const double z = d.value(v);
      d.a[(int64_t)m * d.ld] = d.first(z);
      if (d.b) d.b[(int64_t)m * d.ld] = d.second(z);
      continue;
    }
    if (out.cf) out.cf[(int64_t)m * out.ldc + n] = v;
    if (out.cb) out.cb[(int64_t)m * out.ldc + n] = to_bf16(v);
  }
}

__global__ void f32_to_bf16(const float* __restrict__ in, uint16_t* __restrict__ out, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    out[i] = to_bf16(in[i]);
}

// out (batch x cols, bfloat16) = rows rows[0..batch) of in (FP32, cols per row)
__global__ void rows_to_bf16(const float* __restrict__ in, const int32_t* __restrict__ rows, int batch, int cols,
                             uint16_t* __restrict__ out) {
  const int64_t n = (int64_t)batch * cols;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = i / cols, c = i - r * cols;
    out[i] = to_bf16(in[(int64_t)rows[r] * cols + c]);
  }
}

// a step's loss from the workgroups' squared errors, and its running sum over
// the training steps (acc[0]) with their count (acc[1]); one workgroup of 256
// threads: strided partial sums, then a fixed-order tree
struct LossJob {
  const double* partial;
  int n;
  double scale;
  float* out;
  double* acc;
};
__device__ __forceinline__ void sum_loss(const LossJob& J) {
  __shared__ double red[256];
  double s = 0.0;
  for (int i = threadIdx.x; i < J.n; i += 256) s += J.partial[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double t = red[0] * J.scale;
    *J.out = (float)t;
    J.acc[0] += t;
    J.acc[1] += 1.0;
  }
}

// out[c] = sum_r M[r, c] (bias gradients): a workgroup takes 16 columns, its
// 16 row groups sum rows g, g + 16, ... and the groups' sums are added in a
// fixed order.  The three layers' sums and the step's loss (the last workgroup)
// are one launch (each alone is a few workgroups' chain of reads: 6.5 us apiece
// and 4.3 us, one after another).
constexpr int CS_COLS = 16, CS_GROUPS = 16;
struct ColsumJob {
  const float* in;
  float* out;
  int cols;
  int first;  // first workgroup of the job
};
__global__ void __launch_bounds__(CS_COLS * CS_GROUPS) colsum3(ColsumJob j0, ColsumJob j1, ColsumJob j2, int rows,
                                                                LossJob loss) {
  if (blockIdx.x == gridDim.x - 1) {
    sum_loss(loss);
    return;
  }
  __shared__ float part[CS_GROUPS][CS_COLS];
  const int b = blockIdx.x;
  const ColsumJob J = b >= j2.first ? j2 : (b >= j1.first ? j1 : j0);
  const int cl = threadIdx.x % CS_COLS, g = threadIdx.x / CS_COLS;
  const int c = (b - J.first) * CS_COLS + cl;
  float s = 0.f;
  if (c < J.cols) {
#pragma unroll 8
    for (int r = g; r < rows; r += CS_GROUPS) s += J.in[(int64_t)r * J.cols + c];
  }
  part[g][cl] = s;
  __syncthreads();
  if (g == 0 && c < J.cols) {
    float t = part[0][cl];
    for (int k = 1; k < CS_GROUPS; ++k) t += part[k][cl];
    J.out[c] = t;
  }
}

// Adam on FP32 masters; refreshes the bfloat16 copy
__device__ __forceinline__ void adam_one(float& w, float g, float& m, float& v, float lr, float b1, float b2, float eps,
                                         float c1, float c2) {
  m = fmaf(1.f - b1, g, b1 * m);
  v = fmaf(g, (1.f - b2) * g, b2 * v);
  w = w - lr * (m / c1) / (sqrtf(v / c2) + eps);
}

// Bound by its traffic, 30 bytes per parameter: four parameters per thread and
// load, every load of a thread before its arithmetic.
__global__ void __launch_bounds__(256) adam(float* __restrict__ w, const float* __restrict__ g, float* __restrict__ m,
                                            float* __restrict__ v, int64_t n, float lr, float b1, float b2, float eps,
                                            float c1, float c2, uint16_t* __restrict__ wb) {
  const int64_t stride = (int64_t)gridDim.x * 256;
  for (int64_t q = blockIdx.x * (int64_t)256 + threadIdx.x; q < n / 4; q += stride) {
    f32x4 wi = reinterpret_cast<const f32x4*>(w)[q], mi = reinterpret_cast<const f32x4*>(m)[q],
          vi = reinterpret_cast<const f32x4*>(v)[q];
    const f32x4 gi = reinterpret_cast<const f32x4*>(g)[q];
    u16x4 bi;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float we = wi[e], me = mi[e], ve = vi[e];
      adam_one(we, gi[e], me, ve, lr, b1, b2, eps, c1, c2);
      wi[e] = we;
      mi[e] = me;
      vi[e] = ve;
      bi[e] = to_bf16(we);
    }
    reinterpret_cast<f32x4*>(m)[q] = mi;
    reinterpret_cast<f32x4*>(v)[q] = vi;
    reinterpret_cast<f32x4*>(w)[q] = wi;
    reinterpret_cast<u16x4*>(wb)[q] = bi;
  }
  const int64_t i = n / 4 * 4 + threadIdx.x;  // the last n mod 4 parameters
  if (blockIdx.x == 0 && i < n) {
    float wi = w[i], mi = m[i], vi = v[i];
    adam_one(wi, g[i], mi, vi, lr, b1, b2, eps, c1, c2);
    w[i] = wi;
    m[i] = mi;
    v[i] = vi;
    wb[i] = to_bf16(wi);
  }
}

int grid_for(int64_t n) {
  int64_t g = (n + 255) / 256;
  if (g < 1) g = 1;
  if (g > 2048) g = 2048;
  return (int)g;
}

}  // namespace
}  // namespace pdhcg

using namespace pdhcg;

struct pdhcg_mlp {
  int n_in = 0, n_hid = 0, n_out = 0, cap = 0;
  int rows = 0;  // rows of the input and activation buffers (>= cap)
  hipStream_t stream = nullptr;
  int64_t np = 0;
  int64_t off[6] = {0, 0, 0, 0, 0, 0};  // W1 b1 W2 b2 W3 b3 in the packed vector
  float *w = nullptr, *g = nullptr, *m = nullptr, *v = nullptr;
  uint16_t* wb = nullptr;               // bfloat16 copy of the packed vector (weights used)
  int64_t t = 0;
  uint16_t *xb = nullptr, *h1 = nullptr, *h2 = nullptr, *gob = nullptr, *d2b = nullptr, *d1b = nullptr;
  float *go = nullptr, *d2 = nullptr, *d1 = nullptr, *loss = nullptr;
  double* partial = nullptr;
  double* loss_acc = nullptr;  // [sum of step losses, steps] since the last pdhcg_mlp_take_loss
  float* kpart = nullptr;      // split-K partial products (kSplitMax x kSplitTiles tiles of 64 x 64)
  std::vector<void*> allocs;
  ~pdhcg_mlp() {
    for (void* p : allocs) (void)hipFree(p);
  }
  template <typename T>
  bool alloc(T** p, int64_t count) {
    if (hipMalloc((void**)p, sizeof(T) * (size_t)(count > 0 ? count : 1)) != hipSuccess) {
      (void)hipGetLastError();
      return false;
    }
    allocs.push_back(*p);
    return true;
  }
};

namespace {

#define MLPX(call)                                                                                  \
  do {                                                                                              \
    hipError_t e_ = (call);                                                                         \
    if (e_ != hipSuccess) return set_error(PDHCG_ERR_HIP, (std::string(#call) + ": " + hipGetErrorString(e_)).c_str()); \
  } while (0)

// The k range of a product with fewer than kSplitTiles output tiles of 64 x 64
// and k >= 512 is cut into at most kSplitMax chunks of >= 256 k each, summed
// apart (the sums' rounding follows from this rule alone, whichever kernel
// takes the chunks).
constexpr int kSplitTiles = 128, kSplitMax = 8, kTile = 64;

int k_chunk(int M, int N, int K) {
  const int tiles = ((N + kTile - 1) / kTile) * ((M + kTile - 1) / kTile);
  if (tiles >= kSplitTiles || K < 512) return K;
  const int S = std::min(std::min(kSplitMax, (2 * kSplitTiles + tiles - 1) / tiles), K / 256);
  return ((K + S - 1) / S + 31) / 32 * 32;
}

// one operand: element (r, k) at r * ld + k (kc) or at k * ld + r
struct Operand {
  const uint16_t* p;
  int64_t ld;
  bool kc;
};

// the launch of C = A B with chunked sums, tiles of t x t
Gemm gemm_job(int M, int N, int K, const Operand& A, const Operand& B, int kchunk, const GemmOut& o, int t = kTile) {
  Gemm g{M, N, K, A.p, (uint32_t)A.ld, B.p, (uint32_t)B.ld, kchunk, (N + t - 1) / t, (M + t - 1) / t, 1, o};
  return g;
}

template <int BM, int BN>
void launch_gemm(hipStream_t s, const Gemm& g, const Operand& A, const Operand& B) {
  const dim3 grid(g.gx, g.gy, g.gz);
  if (A.kc && B.kc) hipLaunchKernelGGL((gemm_bf16<BM, BN, true, true>), grid, dim3(256), 0, s, g);
  else if (A.kc) hipLaunchKernelGGL((gemm_bf16<BM, BN, true, false>), grid, dim3(256), 0, s, g);
  else hipLaunchKernelGGL((gemm_bf16<BM, BN, false, false>), grid, dim3(256), 0, s, g);
}

// the chunks of a product that go to workgroups of their own (their sums in
// `work`, added by finish_split): more than one, over a k beyond kFoldK; a
// product of 256 x 512 over k = 5500 keeps 32 CUs busy otherwise
constexpr int kFoldK = 1024;
int split_chunks(const float* work, int K, int kchunk) {
  const int S = (K + kchunk - 1) / kchunk;
  return S > 1 && K > kFoldK && work ? S : 1;
}

hipError_t finish_split(hipStream_t s, const float* work, int S, int M, int N, const GemmOut& o) {
  const int64_t mn = (int64_t)M * N;
  hipLaunchKernelGGL(splitk_finish, dim3((int)std::min<int64_t>((mn + 255) / 256, 2048)), dim3(256), 0, s, work, S, M,
                     N, o);
  return hipGetLastError();
}

// C = A B with the sums chunked by kchunk.  Tiles of 128 x 128 once they give
// every CU four (kBigTiles): half the operand traffic; below that 64 x 64, whose
// shorter k chain and larger count win while CUs are idle.
constexpr int kBigTiles = 1024;

bool big_tiles(int M, int N, int K, int kchunk) {
  return kchunk >= K && (int64_t)((N + 127) / 128) * ((M + 127) / 128) >= kBigTiles;
}

hipError_t gemm(hipStream_t s, float* work, int M, int N, int K, const Operand& A, const Operand& B, int kchunk,
                const GemmOut& o) {
  const int S = split_chunks(work, K, kchunk);
  if (S > 1) {
    Gemm g = gemm_job(M, N, K, A, B, kchunk, o);
    g.gz = S;
    g.out.part = work;
    launch_gemm<64, 64>(s, g, A, B);
    hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : finish_split(s, work, S, M, N, o);
  }
  if (big_tiles(M, N, K, kchunk))
    launch_gemm<128, 128>(s, gemm_job(M, N, K, A, B, kchunk, o, 128), A, B);
  else
    launch_gemm<64, 64>(s, gemm_job(M, N, K, A, B, kchunk, o), A, B);
  return hipGetLastError();
}

GemmOut plain_out(const float* bias, int relu, const uint16_t* mask, float* cf, uint16_t* cb, int64_t ldc) {
  GemmOut o{};
  o.bias = bias;
  o.relu = relu;
  o.mask = mask;
  o.cf = cf;
  o.cb = cb;
  o.ldc = ldc;
  return o;
}

int check_batch(const pdhcg_mlp* h, int32_t batch) {
  if (!h) return set_error(PDHCG_ERR_INVALID_ARGUMENT, "null network handle");
  if (batch < 1 || batch > h->cap) return set_error(PDHCG_ERR_INVALID_ARGUMENT, "batch outside 1..max_batch");
  return 0;
}

// workgroups of the output layer of `batch` rows: the squared errors it leaves
int loss_groups(int batch, int n_out, int n_hid) {
  const int t = big_tiles(batch, n_out, n_hid, k_chunk(batch, n_out, n_hid)) ? 128 : kTile;
  return ((n_out + t - 1) / t) * ((batch + t - 1) / t);
}

// The two hidden layers for `rows` rows of xb into h1 and h2, then the output
// layer into `o`.  A workspace of many rows is one pass; its k chunks are those
// of passes of `step` rows (the network's max_batch), so a row's outputs do not
// depend on how many others share its pass; the last, shorter step is launched
// apart only if its chunks differ.
int run_layers(pdhcg_mlp* h, int rows, int step, const GemmOut& o) {
  const int a = h->n_in, d = h->n_hid, no = h->n_out;
  struct Layer {
    const uint16_t *in, *w;
    int k, n;
    GemmOut out;
  };
  const Layer L[3] = {{h->xb, h->wb + h->off[0], a, d, plain_out(h->w + h->off[1], 1, nullptr, nullptr, h->h1, d)},
                      {h->h1, h->wb + h->off[2], d, d, plain_out(h->w + h->off[3], 1, nullptr, nullptr, h->h2, d)},
                      {h->h2, h->wb + h->off[4], d, no, o}};
  for (const Layer& l : L) {
    const int full = rows / step * step, tail = rows - full;
    const int cf = k_chunk(step, l.n, l.k), ct = tail ? k_chunk(tail, l.n, l.k) : cf;
    const bool one = full == 0 || tail == 0 || cf == ct;
    for (int part = 0; part < (one ? 1 : 2); ++part) {
      const int r0 = part ? full : 0, nr = one ? rows : (part ? tail : full);
      GemmOut po = l.out;
      if (po.cf) po.cf += (int64_t)r0 * po.ldc;
      if (po.cb) po.cb += (int64_t)r0 * po.ldc;
      if (po.x0) po.x0 += (int64_t)r0 * po.n, po.y0 += (int64_t)r0 * po.m;
      // (the split-K workspace holds a product of fewer than kSplitTiles tiles, so a step's rows at most; the
      // squared errors are formed by the product's own workgroups)
      MLPX(gemm(h->stream, nr <= step && !po.loss ? h->kpart : nullptr, nr, l.n, l.k, Operand{l.in + (int64_t)r0 * l.k, l.k, true},
                Operand{l.w, l.n, false}, r0 >= full ? ct : cf, po));
    }
  }
  return 0;
}

// forward pass of `batch` rows of X (device FP32: the first batch rows, or
// rows[0..batch) when rows is given), the output layer into `o`; keeps the
// bfloat16 activations for the backward pass
int run_forward(pdhcg_mlp* h, const float* X, const int32_t* rows, int batch, const GemmOut& o) {
  const int a = h->n_in;
  if (rows)
    hipLaunchKernelGGL(rows_to_bf16, dim3(grid_for((int64_t)batch * a)), dim3(256), 0, h->stream, X, rows, batch, a,
                       h->xb);
  else
    hipLaunchKernelGGL(f32_to_bf16, dim3(grid_for((int64_t)batch * a)), dim3(256), 0, h->stream, X, h->xb,
                       (int64_t)batch * a);
  MLPX(hipGetLastError());
  return run_layers(h, batch, batch, o);
}

// the backward products of one layer in one launch: dW = H' G (M x N over k =
// batch) and the layer input's gradient G W' into `oh`
int backward_layer(pdhcg_mlp* h, int batch, int n_in, int n_out, const uint16_t* H, const uint16_t* G,
                   const uint16_t* W, float* dW, const GemmOut& oh) {
  Gemm w = gemm_job(n_in, n_out, batch, Operand{H, n_in, false}, Operand{G, n_out, false},
                    k_chunk(n_in, n_out, batch), plain_out(nullptr, 0, nullptr, dW, nullptr, n_out));
  const int kc = k_chunk(batch, n_in, n_out), S = split_chunks(h->kpart, n_out, kc);
  Gemm d = gemm_job(batch, n_in, n_out, Operand{G, n_out, true}, Operand{W, n_out, true}, kc, oh);
  if (S > 1) {
    d.gz = S;
    d.out.part = h->kpart;
  }
  hipLaunchKernelGGL(gemm_backward, dim3(d.gx * d.gy * d.gz + w.gx * w.gy), dim3(256), 0, h->stream, w, d);
  MLPX(hipGetLastError());
  if (S > 1) MLPX(finish_split(h->stream, h->kpart, S, batch, n_in, oh));
  return 0;
}

// forward pass, MSE gradient and backward pass of one batch, queued on the
// network's stream (no wait); the gradient stays in h->g, the loss in h->loss
int queue_loss_grad(pdhcg_mlp* h, const float* X, const float* T, const int32_t* rows, int batch) {
  int rc;
  const int a = h->n_in, d = h->n_hid, o = h->n_out;
  const int64_t no = (int64_t)batch * o;
  // the output layer forms the error's gradient G = 2 (O - T) / count (FP32 and
  // bfloat16) and its workgroups' squared errors
  GemmOut mse = plain_out(h->w + h->off[5], 0, nullptr, h->go, h->gob, o);
  mse.T = T;
  mse.rows = rows;
  mse.scale = (float)(1.0 / (double)no);
  mse.loss = h->partial;
  if ((rc = run_forward(h, X, rows, batch, mse))) return rc;
  float* g = h->g;
  if ((rc = backward_layer(h, batch, d, o, h->h2, h->gob, h->wb + h->off[4], g + h->off[4],
                           plain_out(nullptr, 0, h->h2, h->d2, h->d2b, d))))
    return rc;
  if ((rc = backward_layer(h, batch, d, d, h->h1, h->d2b, h->wb + h->off[2], g + h->off[2],
                           plain_out(nullptr, 0, h->h1, h->d1, h->d1b, d))))
    return rc;
  MLPX(gemm(h->stream, h->kpart, a, d, batch, Operand{h->xb, a, false}, Operand{h->d1b, d, false}, k_chunk(a, d, batch),
            plain_out(nullptr, 0, nullptr, g + h->off[0], nullptr, d)));
  // db = column sums of the three layers' output gradients; the step's loss
  const int wo = (o + CS_COLS - 1) / CS_COLS, wd = (d + CS_COLS - 1) / CS_COLS;
  hipLaunchKernelGGL(colsum3, dim3(wo + 2 * wd + 1), dim3(CS_COLS * CS_GROUPS), 0, h->stream,
                     ColsumJob{h->go, g + h->off[5], o, 0}, ColsumJob{h->d2, g + h->off[3], d, wo},
                     ColsumJob{h->d1, g + h->off[1], d, wo + wd}, batch,
                     LossJob{h->partial, loss_groups(batch, o, d), 1.0 / (double)no, h->loss, h->loss_acc});
  MLPX(hipGetLastError());
  return 0;
}

int queue_adam(pdhcg_mlp* h, float lr, float beta1, float beta2, float eps) {
  h->t += 1;
  const float c1 = (float)(1.0 - pow((double)beta1, (double)h->t));
  const float c2 = (float)(1.0 - pow((double)beta2, (double)h->t));
  hipLaunchKernelGGL(adam, dim3((int)std::max<int64_t>(1, std::min<int64_t>((h->np / 4 + 255) / 256, 4096))), dim3(256), 0, h->stream, h->w, h->g, h->m, h->v, h->np, lr, beta1,
                     beta2, eps, c1, c2, h->wb);
  MLPX(hipGetLastError());
  return 0;
}

}  // namespace

extern "C" {

int pdhcg_mlp_create(pdhcg_mlp** out, int32_t n_in, int32_t n_hid, int32_t n_out, int32_t max_batch,
                     void* hip_stream) {
  if (!out) return set_error(PDHCG_ERR_INVALID_ARGUMENT, "null handle pointer");
  *out = nullptr;
  if (n_in < 1 || n_hid < 1 || n_out < 1 || max_batch < 1)
    return set_error(PDHCG_ERR_INVALID_ARGUMENT, "network sizes and max_batch must be >= 1");
  pdhcg_mlp* h = new pdhcg_mlp();
  h->n_in = n_in;
  h->n_hid = n_hid;
  h->n_out = n_out;
  h->cap = max_batch;
  h->stream = (hipStream_t)hip_stream;
  const int64_t sizes[6] = {(int64_t)n_in * n_hid, n_hid, (int64_t)n_hid * n_hid, n_hid, (int64_t)n_hid * n_out, n_out};
  int64_t acc = 0;
  for (int k = 0; k < 6; ++k) {
    h->off[k] = acc;
    acc += sizes[k];
  }
  h->np = acc;
  const int64_t B = max_batch;
  // inputs and activations of a pass of pdhcg_mlp_predict_start: up to 4 096
  // rows at once while they stay within 32 MB per activation
  h->rows = (int)std::max<int64_t>(B, std::min<int64_t>(4096, (int64_t)(16 << 20) / std::max(n_hid, n_in)));
  const int64_t R = h->rows;
  bool ok = h->alloc(&h->w, acc) && h->alloc(&h->g, acc) && h->alloc(&h->m, acc) && h->alloc(&h->v, acc) &&
            h->alloc(&h->wb, acc + kPad) && h->alloc(&h->xb, R * n_in + kPad) &&
            h->alloc(&h->h1, R * n_hid + kPad) &&
            h->alloc(&h->h2, R * n_hid + kPad) && h->alloc(&h->gob, B * n_out + kPad) &&
            h->alloc(&h->d2b, B * n_hid + kPad) &&
            h->alloc(&h->d1b, B * n_hid + kPad) && h->alloc(&h->go, B * n_out) &&
            h->alloc(&h->d2, B * n_hid) && h->alloc(&h->d1, B * n_hid) && h->alloc(&h->loss, 1) &&
            h->alloc(&h->partial, (int64_t)((n_out + kTile - 1) / kTile) * ((B + kTile - 1) / kTile)) && h->alloc(&h->loss_acc, 2) &&
            h->alloc(&h->kpart, (int64_t)kSplitMax * kSplitTiles * kTile * kTile);
  if (!ok) {
    delete h;
    return set_error(PDHCG_ERR_OUT_OF_MEMORY, "hipMalloc failed for the network");
  }
  if (hipMemsetAsync(h->w, 0, sizeof(float) * acc, h->stream) != hipSuccess ||
      hipMemsetAsync(h->wb, 0, sizeof(uint16_t) * acc, h->stream) != hipSuccess ||
      hipMemsetAsync(h->loss_acc, 0, sizeof(double) * 2, h->stream) != hipSuccess ||
      hipStreamSynchronize(h->stream) != hipSuccess) {
    delete h;
    return set_error(PDHCG_ERR_HIP, "initialising the network failed");
  }
  *out = h;
  return 0;
}

int64_t pdhcg_mlp_num_params(const pdhcg_mlp* h) { return h ? h->np : 0; }

int pdhcg_mlp_set_params(pdhcg_mlp* h, const float* params) {
  if (!h || !params) return set_error(PDHCG_ERR_INVALID_ARGUMENT, "null argument");
  MLPX(hipMemcpyAsync(h->w, params, sizeof(float) * h->np, hipMemcpyHostToDevice, h->stream));
  MLPX(hipMemsetAsync(h->m, 0, sizeof(float) * h->np, h->stream));
  MLPX(hipMemsetAsync(h->v, 0, sizeof(float) * h->np, h->stream));
  hipLaunchKernelGGL(f32_to_bf16, dim3(grid_for(h->np)), dim3(256), 0, h->stream, h->w, h->wb, h->np);
  MLPX(hipGetLastError());
  MLPX(hipStreamSynchronize(h->stream));
  h->t = 0;
  return 0;
}

int pdhcg_mlp_get_params(const pdhcg_mlp* h, float* params) {
  if (!h || !params) return set_error(PDHCG_ERR_INVALID_ARGUMENT, "null argument");
  MLPX(hipMemcpyAsync(params, h->w, sizeof(float) * h->np, hipMemcpyDeviceToHost, h->stream));
  MLPX(hipStreamSynchronize(h->stream));
  return 0;
}

int pdhcg_mlp_forward(pdhcg_mlp* h, const float* X, int32_t batch, float* Y) {
  int rc;
  if ((rc = check_batch(h, batch))) return rc;
  if (!X || !Y) return set_error(PDHCG_ERR_INVALID_ARGUMENT, "null X or Y");
  if ((rc = run_forward(h, X, nullptr, batch, plain_out(h->w + h->off[5], 0, nullptr, Y, nullptr, h->n_out)))) return rc;
  MLPX(hipStreamSynchronize(h->stream));
  return 0;
}

int pdhcg_mlp_predict_start(pdhcg_mlp* h, const float* X, int32_t batch, const double* out_mu,
                            const double* out_sd, int32_t n, int32_t n_pair, const int32_t* plus,
                            const int32_t* minus, int32_t n_rest, const int32_t* rest, int32_t m, double* x0,
                            double* y0) {
  if (!h) return set_error(PDHCG_ERR_INVALID_ARGUMENT, "null network handle");
  if (batch < 1) return set_error(PDHCG_ERR_INVALID_ARGUMENT, "batch must be >= 1");
  if (!X || !out_mu || !out_sd || !x0 || (m > 0 && !y0))
    return set_error(PDHCG_ERR_INVALID_ARGUMENT, "null input or output array");
  if (n < 0 || n_pair < 0 || n_rest < 0 || m < 0 || n + n_pair + n_rest != h->n_out || 2 * n_pair + n_rest != m)
    return set_error(PDHCG_ERR_INVALID_ARGUMENT,
                     "need n + n_pair + n_rest = n_out and 2 n_pair + n_rest = m (every row of y once)");
  if ((n_pair > 0 && (!plus || !minus)) || (n_rest > 0 && !rest))
    return set_error(PDHCG_ERR_INVALID_ARGUMENT, "null row index array");
  int rc;
  GemmOut o = plain_out(h->w + h->off[5], 0, nullptr, nullptr, nullptr, h->n_out);
  o.mu = out_mu;
  o.sd = out_sd;
  o.n = n;
  o.n_pair = n_pair;
  o.m = m;
  o.plus = plus;
  o.minus = minus;
  o.rest = rest;
  // passes of the workspace's rows, a whole number of max_batch steps each; the
  // output layer writes the start points itself
  const int64_t pass = (int64_t)(h->rows / h->cap) * h->cap;
  for (int64_t r0 = 0; r0 < batch; r0 += pass) {
    const int rows = (int)std::min<int64_t>(pass, batch - r0);
    const int64_t cnt = (int64_t)rows * h->n_in;
    hipLaunchKernelGGL(f32_to_bf16, dim3(grid_for(cnt)), dim3(256), 0, h->stream, X + r0 * h->n_in, h->xb, cnt);
    MLPX(hipGetLastError());
    o.x0 = x0 + r0 * n;
    o.y0 = y0 + r0 * m;
    if ((rc = run_layers(h, rows, std::min(h->cap, rows), o))) return rc;
  }
  MLPX(hipStreamSynchronize(h->stream));
  return 0;
}

int pdhcg_mlp_loss_grad(pdhcg_mlp* h, const float* X, const float* T, int32_t batch, float* loss, float* grads) {
  int rc;
  if ((rc = check_batch(h, batch))) return rc;
  if (!X || !T) return set_error(PDHCG_ERR_INVALID_ARGUMENT, "null X or T");
  if ((rc = queue_loss_grad(h, X, T, nullptr, batch))) return rc;
  if (loss) MLPX(hipMemcpyAsync(loss, h->loss, sizeof(float), hipMemcpyDeviceToHost, h->stream));
  if (grads) MLPX(hipMemcpyAsync(grads, h->g, sizeof(float) * h->np, hipMemcpyDeviceToHost, h->stream));
  MLPX(hipStreamSynchronize(h->stream));
  return 0;
}

int pdhcg_mlp_train_step(pdhcg_mlp* h, const float* X, const float* T, const int32_t* rows, int32_t batch, float lr,
                         float beta1, float beta2, float eps) {
  int rc;
  if ((rc = check_batch(h, batch))) return rc;
  if (!X || !T) return set_error(PDHCG_ERR_INVALID_ARGUMENT, "null X or T");
  if ((rc = queue_loss_grad(h, X, T, rows, batch))) return rc;
  return queue_adam(h, lr, beta1, beta2, eps);
}

int pdhcg_mlp_take_loss(pdhcg_mlp* h, double* sum, int64_t* steps) {
  if (!h) return set_error(PDHCG_ERR_INVALID_ARGUMENT, "null network handle");
  double acc[2] = {0.0, 0.0};
  MLPX(hipMemcpyAsync(acc, h->loss_acc, sizeof(acc), hipMemcpyDeviceToHost, h->stream));
  MLPX(hipMemsetAsync(h->loss_acc, 0, sizeof(double) * 2, h->stream));
  MLPX(hipStreamSynchronize(h->stream));
  if (sum) *sum = acc[0];
  if (steps) *steps = (int64_t)acc[1];
  return 0;
}

int pdhcg_mlp_adam_step(pdhcg_mlp* h, float lr, float beta1, float beta2, float eps) {
  if (!h) return set_error(PDHCG_ERR_INVALID_ARGUMENT, "null network handle");
  int rc;
  if ((rc = queue_adam(h, lr, beta1, beta2, eps))) return rc;
  MLPX(hipStreamSynchronize(h->stream));
  return 0;
}

void pdhcg_mlp_destroy(pdhcg_mlp* h) {
  if (!h) return;
  (void)hipStreamSynchronize(h->stream);
  delete h;
}

}  // extern "C"
