// Fourier neural operator surrogate: BF16 MFMA training and inference on gfx950.
//
// The learned form beside the method: a classic FNO maps the state
// (c, eta_1..3) on an n^3 grid to the increment of the state a fixed time
// later.  Architecture (width w, modes m, L layers, hidden h):
//   v0 = x W_lift + b_lift;  v_{l+1} = act(K_l v_l + v_l W_l + b_l);
//   out = GELU(v_L P1 + c1) P2 + c2,
//   K_l v = inverse truncated DFT( R_l . forward truncated DFT(v) ),
// retained modes kx < m and ky, kz in the m lowest positive and negative
// frequencies.  Activations are channel-last [point][channel] BF16.
//
// Dense contractions run on MFMA (gfx950 v_mfma_f32_32x32x16_bf16, FP32 accumulate):
//  * a layer along whole x lines (width <= 64, at most 16 modes): channel
//    mixing, the inverse x stage, the activation and the next layer's x stage
//    in one pass (k_xline); else channel mixing as [points x K] x [K x N] GEMMs
//    (k_cm_gemm) and the x stages as GEMMs of their own (k_lm_gemm);
//  * the y and z stages of the truncated DFT as a small constant matrix G times
//    batched activation blocks, Out_b = G X_b (k_lm_rows; backward: G^T);
//  * the projection with the loss and its backward pass in one kernel (width
//    <= 32, k_proj), else as GEMMs through the hidden layer;
//  * the weight gradients, reductions over points (k_wgrad_mfma).
// The per-mode complex w x w mixing and its gradients run on FP32 vector ALUs.
// Adam updates FP32 master weights and refreshes the BF16 working copies.
#include <hip/hip_runtime.h>

#include <chrono>
#include <cmath>
#include <cstring>
#include <mutex>
#include <new>
#include <type_traits>
#include <vector>

#include "../../include/pf.h"
#include "pf_context.hpp"
#include "pf_fno_sizes.hpp"

namespace {

typedef unsigned short u16;
typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

// gfx950's 32 x 32 x 16 BF16 MFMA (FP32 accumulate).  Lane l holds row l % 32
// of A and column l % 32 of B at k = 8 (l / 32) .. 8 (l / 32) + 7; the
// accumulator layout is that of every 32 x 32 MFMA (lane l, element i: row
// 8 (i / 4) + 4 (l / 32) + i % 4, column l % 32).
__device__ inline f32x16 mfma16(bf16x4 a_lo, bf16x4 a_hi, bf16x4 b_lo, bf16x4 b_hi, f32x16 acc) {
  const s16x8 a = {a_lo[0], a_lo[1], a_lo[2], a_lo[3], a_hi[0], a_hi[1], a_hi[2], a_hi[3]};
  const s16x8 b = {b_lo[0], b_lo[1], b_lo[2], b_lo[3], b_hi[0], b_hi[1], b_hi[2], b_hi[3]};
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc,
                                                 0, 0, 0);
}
__device__ inline f32x16 mfma32(u32x4 a, u32x4 b, f32x16 acc) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc,
                                                 0, 0, 0);
}
// 16 x 16 x 32: lane l holds row / column l % 16 at k = 8 (l / 16) ..; element
// i of the accumulator: row 4 (l / 16) + i, column l % 16.
__device__ inline f32x4 mfma16x16(u32x4 a, u32x4 b, f32x4 acc) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc,
                                                 0, 0, 0);
}
__device__ inline f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = 0.0f;
  return z;
}

// two values to BF16, round to nearest even (v_cvt_pk_bf16_f32)
__device__ inline unsigned pack2(float a, float b) {
  const bf16x2 v = {(__bf16)a, (__bf16)b};
  return __builtin_bit_cast(unsigned, v);
}

// A 32 x 32 accumulator tile as BF16 operands of the next MFMA: lane l keeps
// its column l % 32, with the tile's rows as that operand's k (op[s]: rows
// 16 s .. 16 s + 15).  The two half-waves exchange the row groups they hold.
__device__ inline void to_operand(const f32x16& v, u32x4 (&op)[2]) {
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const unsigned d0 = pack2(v[8 * s], v[8 * s + 1]), d1 = pack2(v[8 * s + 2], v[8 * s + 3]);
    const unsigned e0 = pack2(v[8 * s + 4], v[8 * s + 5]), e1 = pack2(v[8 * s + 6], v[8 * s + 7]);
    const auto p = __builtin_amdgcn_permlane32_swap(d0, e0, false, false);
    const auto q = __builtin_amdgcn_permlane32_swap(d1, e1, false, false);
    op[s] = u32x4{p[0], q[0], p[1], q[1]};
  }
}

// The identity's rows k = 16 s .. 16 s + 15 as a B operand: op x identity puts
// an operand (lane = row) into the accumulator with lane = k, i.e. transposes
// it, exactly (BF16 values times one).
__device__ inline u32x4 identity_operand(int s, int lr, int lg) {
  u32x4 w;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int k = 16 * s + 8 * lg + 2 * j;
    w[j] = (k == lr ? 0x3F80u : 0u) | (k + 1 == lr ? 0x3F800000u : 0u);
  }
  return w;
}
// op (lane = row, k) -> operands with lane = k and k = row; t: the same in FP32
__device__ inline f32x16 transpose_operand(const u32x4 (&op)[2], const u32x4 (&id)[2], u32x4 (&out)[2]) {
  f32x16 t = mfma32(op[0], id[0], zero16());
  t = mfma32(op[1], id[1], t);
  to_operand(t, out);
  return t;
}

__host__ __device__ inline u16 f2bf(float f) {
  unsigned int u;
  std::memcpy(&u, &f, 4);
  u += 0x7FFFu + ((u >> 16) & 1u);  // round to nearest even
  return (u16)(u >> 16);
}
__host__ __device__ inline float bf2f(u16 h) {
  unsigned int u = ((unsigned int)h) << 16;
  float f;
  std::memcpy(&f, &u, 4);
  return f;
}

__device__ inline float gelu_f(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }
__device__ inline float gelu_g(float x) {
  return 0.5f * (1.0f + erff(x * 0.70710678118654752f)) + x * 0.39894228040143268f * expf(-0.5f * x * x);
}

__device__ inline bf16x4 ld4(const u16* p) { return *reinterpret_cast<const bf16x4*>(p); }

// A second contraction along the x lines that a channel-mixing GEMM can carry:
// for point p = line * R + x, adds sum_k G[x][k] X[line * xbs + k * ldx + n]
// (the truncated-DFT x stage whose result the GEMM would otherwise read back
// as a residual).  G row-major R x K (K % 4 == 0, zero beyond K); R % 32 == 0
// so that a wave's 32 points lie in one line.  G == nullptr: none.
struct LineTerm {
  const u16* G = nullptr;
  int K = 0, R = 0;
  const u16* X = nullptr;
  long long xbs = 0;
  int ldx = 0;
};

// Eight values of a row at k = kb .. kb + 7, zero beyond K (K % 4 == 0); v16:
// the row is 16-byte aligned and K % 8 == 0.
__device__ inline u32x4 ld8(const u16* row, int kb, int K, bool v16) {
  u32x4 r = {0, 0, 0, 0};
  if (v16) {
    if (kb < K) r = *reinterpret_cast<const u32x4*>(row + kb);
  } else {
    if (kb < K) {
      const u32x2 a = *reinterpret_cast<const u32x2*>(row + kb);
      r[0] = a[0], r[1] = a[1];
    }
    if (kb + 4 < K) {
      const u32x2 a = *reinterpret_cast<const u32x2*>(row + kb + 4);
      r[2] = a[0], r[3] = a[1];
    }
  }
  return r;
}
// the same for a store of n values starting at column c of the row
__device__ inline void st8(u16* row, int c, int N, bool v16, u32x4 v) {
  if (v16) {
    if (c < N) *reinterpret_cast<u32x4*>(row + c) = v;
  } else {
    if (c < N) *reinterpret_cast<u32x2*>(row + c) = u32x2{v[0], v[1]};
    if (c + 4 < N) *reinterpret_cast<u32x2*>(row + c + 4) = u32x2{v[2], v[3]};
  }
}

// ---- channel-mixing GEMM: Out[p][n] = epi(sum_k In[p][k] Bt[n][k] [+ line term]) ----
// K % 4 == 0 (zero beyond K), P % 128 == 0, N <= 32 * NT.  Epilogue: + bias[n] + resid[p][n],
// times GELU'(gpre[p][n]) (a data gradient through the activation; GELU' from a
// table over the BF16 values), stores any of: f32 result, bf16 pre-activation,
// bf16 GELU(pre).
// The weights are the A operand and the points the B operand, so a lane holds
// one point and reads and writes its channels 16 bytes at a time (with the
// roles exchanged every store was two bytes wide).
template <int NT>
__global__ void __launch_bounds__(256)
k_cm_gemm(const u16* __restrict__ In, int ldin, int K, const u16* __restrict__ Bt, int N,
          const float* __restrict__ bias, const float* __restrict__ resid, int ldres, float* __restrict__ outf,
          u16* __restrict__ outpre, u16* __restrict__ outact, int ldout, LineTerm lt,
          const u16* __restrict__ gpre, const float* __restrict__ gtab) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const long long p0 = ((long long)blockIdx.x * 4 + wave) * 32;
  const int lr = lane & 31, lg = lane >> 5;
  f32x16 acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = zero16();
  const bool in16 = K % 8 == 0 && ldin % 8 == 0, k16 = K % 8 == 0;
  for (int kk = 0; kk < K; kk += 16) {
    const int kb = kk + lg * 8;
    const u32x4 b = ld8(In + (p0 + lr) * ldin, kb, K, in16);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int n = t * 32 + lr;
      u32x4 a = {0, 0, 0, 0};
      if (n < N) a = ld8(Bt + (long long)n * K, kb, K, k16);
      acc[t] = mfma32(a, b, acc[t]);
    }
  }
  if (lt.G) {
    const long long line = p0 / lt.R;
    const int x = (int)(p0 % lt.R) + lr;
    const u16* Xb = lt.X + line * lt.xbs;
    const bool g16 = lt.K % 8 == 0;
    for (int kk = 0; kk < lt.K; kk += 16) {
      const int kb = kk + lg * 8;
      const u32x4 b = ld8(lt.G + (long long)x * lt.K, kb, lt.K, g16);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int n = t * 32 + lr;
        u32x4 a = {0, 0, 0, 0};
        if (n < N) {
#pragma unroll
          for (int j = 0; j < 8; ++j)
            if (kb + j < lt.K) a[j >> 1] |= (unsigned)Xb[(long long)(kb + j) * lt.ldx + n] << (16 * (j & 1));
        }
        acc[t] = mfma32(a, b, acc[t]);
      }
    }
  }
  const long long p = p0 + lr;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    f32x16 v = acc[t];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int c = t * 32 + 8 * q + 4 * lg;  // this lane's channels c .. c + 3
      if (c >= N) continue;
      if (N % 4 == 0) {
        const f32x4 bb = bias ? *reinterpret_cast<const f32x4*>(bias + c) : f32x4{0.f, 0.f, 0.f, 0.f};
        f32x4 rr = {0.f, 0.f, 0.f, 0.f};
        if (resid) rr = *reinterpret_cast<const f32x4*>(resid + p * ldres + c);
        u32x2 gp = {0, 0};
        if (gpre) gp = *reinterpret_cast<const u32x2*>(gpre + p * ldout + c);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float r = v[4 * q + j] + bb[j];
          if (resid) r += rr[j];
          if (gpre) r *= gtab[(gp[j >> 1] >> (16 * (j & 1))) & 0xffffu];
          v[4 * q + j] = r;
        }
        if (outf) {
          *reinterpret_cast<f32x4*>(outf + p * ldout + c) =
              f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
        }
      } else {  // f32 results of a channel count that 4 does not divide
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (c + j >= N) continue;
          float r = v[4 * q + j] + (bias ? bias[c + j] : 0.0f);
          if (resid) r += resid[p * ldres + c + j];
          if (outf) outf[p * ldout + c + j] = r;
        }
      }
    }
    const bool o16 = N % 8 == 0 && ldout % 8 == 0;
    u32x4 op[2];
    if (outpre) {
      to_operand(v, op);
#pragma unroll
      for (int s = 0; s < 2; ++s) st8(outpre + p * ldout, t * 32 + 16 * s + 8 * lg, N, o16, op[s]);
    }
    if (outact) {
#pragma unroll
      for (int i = 0; i < 16; ++i) v[i] = gelu_f(v[i]);
      to_operand(v, op);
#pragma unroll
      for (int s = 0; s < 2; ++s) st8(outact + p * ldout, t * 32 + 16 * s + 8 * lg, N, o16, op[s]);
    }
  }
}

// ---- projection: out = GELU(v P1 + c1) P2 + c2 (w <= 32, h <= 32 HT, co <= 8) ----
// One pass over the points from v_L to the network's output; the hidden layer
// stays in registers.  At 128^3, h = 128 the separate GEMMs moved 1.6 GB per
// sample through the hidden layer (0.92 ms for two samples).  TRAIN goes on to the loss against
// (y - x) / scale, the data gradient d v_L (dpre) and the gradients of P1, c1, P2
// and c2 (one partial set per block: part1 rows k = 0 .. w, part2 rows
// 0 .. h, the last row the bias's): with the hidden layer's activations and
// gradients in HBM that took 4.6 GB and 3.9 ms per sample.  Now 0.17 ms per
// sample, bound by the exact GELUs (the vector units issue in 62 % of the
// cycles), and 0.58 with TRAIN, by its registers (two waves per SIMD, 35 %).
// A wave takes 32 points at a time; points are the B operand throughout, so
// every product's accumulator holds one point per lane, and the next product
// takes it as an operand (to_operand).  The weight gradients contract over
// points: their operands are transposed through an identity product.
// P % 32 == 0.  The sums over channels run in the order of k_cm_gemm's.
struct ProjArgs {
  const u16* v;        // [P][w]
  const u16 *P1T, *P2T, *P1, *P2;  // [h][w], [co][h], [w][h], [h][8]
  const float *c1, *c2;
  long long P;
  int w, h, co;
  float* outf;         // !TRAIN: [P][co]
  const float *x, *y;  // TRAIN: planar [..][P]
  const float* scale;
  float inv;           // 2 / (P co)
  const float* gtab;
  u16* dpre;           // [P][w]
  float *part1, *part2;
  double* dpart;
};

template <bool TRAIN, int HT>
__global__ void __launch_bounds__(256, 2) k_proj(ProjArgs pa) {
  constexpr int H = 32 * HT, LH = H + 8;
  __shared__ __attribute__((aligned(16))) u16 sP1T[H * 40];
  __shared__ __attribute__((aligned(16))) u16 sP2T[8 * LH];
  __shared__ __attribute__((aligned(16))) u16 sP1[TRAIN ? 32 * LH : 8];
  __shared__ __attribute__((aligned(16))) u16 sP2[TRAIN ? H * 8 : 8];
  __shared__ __attribute__((aligned(16))) float sc1[H];
  // TRAIN: the hidden activations' operands (each lane's own slots: 32 registers
  // fewer, which keeps two waves per SIMD), and the block sums at the end
  __shared__ u32x4 shop[TRAIN ? 2 * HT * 256 : 1];
  float* red = reinterpret_cast<float*>(shop);
  const int w = pa.w, h = pa.h, co = pa.co;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, lr = lane & 31, lg = lane >> 5;
  for (int e = tid; e < H * 40; e += 256) {
    const int r = e / 40, k = e % 40;
    sP1T[e] = (r < h && k < w) ? pa.P1T[r * w + k] : (u16)0;
  }
  for (int e = tid; e < 8 * LH; e += 256) {
    const int r = e / LH, k = e % LH;
    sP2T[e] = (r < co && k < h) ? pa.P2T[r * h + k] : (u16)0;
  }
  for (int e = tid; e < H; e += 256) sc1[e] = e < h ? pa.c1[e] : 0.0f;
  if constexpr (TRAIN) {
    for (int e = tid; e < 32 * LH; e += 256) {
      const int r = e / LH, k = e % LH;
      sP1[e] = (r < w && k < h) ? pa.P1[r * h + k] : (u16)0;
    }
    for (int e = tid; e < H * 8; e += 256) sP2[e] = e < h * 8 ? pa.P2[e] : (u16)0;
  }
  __syncthreads();
  float c2[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) c2[j] = 4 * lg + j < co ? pa.c2[4 * lg + j] : 0.0f;
  const bool v16 = w % 8 == 0;
  const long long ntile = pa.P / 32;
  u32x4 id[2];
  f32x16 g1[TRAIN ? HT : 1];
  f32x4 g2[TRAIN ? 2 * HT : 1];
  float b1[TRAIN ? HT : 1], b2 = 0.0f, scl[4];
  double loss = 0.0;
  if constexpr (TRAIN) {
#pragma unroll
    for (int s = 0; s < 2; ++s) id[s] = identity_operand(s, lr, lg);
#pragma unroll
    for (int t = 0; t < HT; ++t) g1[t] = zero16(), b1[t] = 0.0f;
#pragma unroll
    for (int t = 0; t < 2 * HT; ++t) g2[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 4; ++j) scl[j] = 4 * lg + j < co ? pa.scale[4 * lg + j] : 1.0f;
  }
  // pre-activations of hidden channels 32 t .. 32 t + 31 at this lane's point
  auto hidden = [&](int t, const u32x4(&vop)[2]) {
    f32x16 a = zero16();
#pragma unroll
    for (int s = 0; s < 2; ++s)
      if (16 * s < w) a = mfma32(*reinterpret_cast<const u32x4*>(sP1T + (32 * t + lr) * 40 + 16 * s + 8 * lg), vop[s], a);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 bb = *reinterpret_cast<const f32x4*>(sc1 + 32 * t + 8 * q + 4 * lg);
#pragma unroll
      for (int j = 0; j < 4; ++j) a[4 * q + j] = a[4 * q + j] + bb[j];
    }
    return a;
  };
  for (long long tile = (long long)blockIdx.x * 4 + wave; tile < ntile; tile += (long long)gridDim.x * 4) {
    const long long p = tile * 32 + lr;
    u32x4 vop[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) vop[s] = ld8(pa.v + p * w, 16 * s + 8 * lg, w, v16);
    float xv[4], yv[4];
    if constexpr (TRAIN) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int c = 4 * lg + j;
        xv[j] = c < co ? pa.x[c * pa.P + p] : 0.0f;
        yv[j] = c < co ? pa.y[c * pa.P + p] : 0.0f;
      }
    }
    f32x16 o = zero16();
#pragma unroll
    for (int t = 0; t < HT; ++t) {
      f32x16 a = hidden(t, vop);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        a[i] = gelu_f(a[i]);
        if (TRAIN && i % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // four erfs in flight: registers
      }
      u32x4 hop[2];
      to_operand(a, hop);
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        if constexpr (TRAIN) shop[(2 * t + s) * 256 + tid] = hop[s];
        u32x4 q = {0, 0, 0, 0};
        if (lr < 8) q = *reinterpret_cast<const u32x4*>(sP2T + lr * LH + 32 * t + 16 * s + 8 * lg);
        o = mfma32(q, hop[s], o);
      }
      __builtin_amdgcn_sched_barrier(0);  // one tile at a time: registers
    }
    if constexpr (!TRAIN) {
      float* of = pa.outf + p * co + 4 * lg;
      if (co % 4 == 0) {
        if (4 * lg < co)
          *reinterpret_cast<f32x4*>(of) = f32x4{o[0] + c2[0], o[1] + c2[1], o[2] + c2[2], o[3] + c2[3]};
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (4 * lg + j < co) of[j] = o[j] + c2[j];
      }
    } else {
      float g[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        g[j] = 0.0f;
        if (4 * lg + j < co) {
          const float tgt = (yv[j] - xv[j]) / scl[j];
          const float d = (o[j] + c2[j]) - tgt;
          loss += (double)d * d;
          g[j] = d * pa.inv;
        }
      }
      // output gradients as an operand (lane = point, k = output channel < 8)
      const auto e0 = __builtin_amdgcn_permlane32_swap(pack2(g[0], g[1]), 0u, false, false);
      const auto e1 = __builtin_amdgcn_permlane32_swap(pack2(g[2], g[3]), 0u, false, false);
      const u32x4 dop = {e0[0], e1[0], e0[1], e1[1]};
      u32x4 vT[2], dT[2];
      transpose_operand(vop, id, vT);
      u32x4 d16;  // lane % 16 = output channel, k = the 32 points in permlane16 order
      {
        const f32x16 t = mfma32(dop, id[0], zero16());
        to_operand(t, dT);
#pragma unroll
        for (int i = 0; i < 16; ++i) b2 += t[i];
#pragma unroll
        for (int j = 0; j < 4; ++j) d16[j] = __builtin_amdgcn_permlane16_swap(dT[0][j], dT[1][j], false, false)[0];
      }
      f32x16 dv = zero16();
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < HT; ++t) {
        u32x4 q = {0, 0, 0, 0};
        if (lg == 0) q = *reinterpret_cast<const u32x4*>(sP2 + (32 * t + lr) * 8);
        f32x16 dh = mfma32(q, dop, zero16());
        const f32x16 a = hidden(t, vop);
#pragma unroll
        for (int i = 0; i < 16; i += 2) {
          const unsigned hb = pack2(a[i], a[i + 1]);
          dh[i] *= pa.gtab[hb & 0xffffu];
          dh[i + 1] *= pa.gtab[hb >> 16];
          if (i % 8 == 6) __builtin_amdgcn_sched_barrier(0);
        }
        u32x4 dhop[2], tr[2];
        to_operand(dh, dhop);
#pragma unroll
        for (int s = 0; s < 2; ++s)
          dv = mfma32(*reinterpret_cast<const u32x4*>(sP1 + lr * LH + 32 * t + 16 * s + 8 * lg), dhop[s], dv);
        __builtin_amdgcn_sched_barrier(0);
        const f32x16 dt = transpose_operand(dhop, id, tr);
#pragma unroll
        for (int i = 0; i < 16; ++i) b1[t] += dt[i];
#pragma unroll
        for (int s = 0; s < 2; ++s) g1[t] = mfma32(vT[s], tr[s], g1[t]);
        __builtin_amdgcn_sched_barrier(0);
        dhop[0] = shop[2 * t * 256 + tid];
        dhop[1] = shop[(2 * t + 1) * 256 + tid];
        transpose_operand(dhop, id, tr);
        u32x4 h0, h1;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const auto z = __builtin_amdgcn_permlane16_swap(tr[0][j], tr[1][j], false, false);
          h0[j] = z[0];
          h1[j] = z[1];
        }
        g2[2 * t] = mfma16x16(d16, h0, g2[2 * t]);
        g2[2 * t + 1] = mfma16x16(d16, h1, g2[2 * t + 1]);
        __builtin_amdgcn_sched_barrier(0);
      }
      u32x4 op[2];
      to_operand(dv, op);
#pragma unroll
      for (int s = 0; s < 2; ++s) st8(pa.dpre + p * w, 16 * s + 8 * lg, w, v16, op[s]);
    }
  }
  if constexpr (TRAIN) {
    // the four waves' sums, tile by tile, into this block's partial sets
    float* d1 = pa.part1 + (long long)blockIdx.x * (w + 1) * h;
    float* d2 = pa.part2 + (long long)blockIdx.x * (h + 1) * co;
#pragma unroll
    for (int t = 0; t < HT; ++t) {
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 16; ++i) red[wave * 1024 + (8 * (i >> 2) + 4 * lg + (i & 3)) * 32 + lr] = g1[t][i];
      __syncthreads();
      for (int e = tid; e < 1024; e += 256) {
        const int k = e >> 5, n = 32 * t + (e & 31);
        if (k < w && n < h) d1[k * h + n] = (red[e] + red[1024 + e]) + (red[2048 + e] + red[3072 + e]);
      }
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 2 * HT; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int c = 4 * (lane >> 4) + i;  // output channel
        if (c < 8) red[wave * 1024 + c * H + 16 * t + (lane & 15)] = g2[t][i];
      }
    __syncthreads();
    for (int e = tid; e < 8 * H; e += 256) {
      const int c = e / H, k = e % H;
      if (c < co && k < h) d2[k * co + c] = (red[e] + red[1024 + e]) + (red[2048 + e] + red[3072 + e]);
    }
    __syncthreads();
    // bias rows: the two half-waves hold different points of a channel
#pragma unroll
    for (int t = 0; t < HT; ++t) red[wave * 256 + lg * 128 + 32 * t + lr] = b1[t];
    red[1024 + wave * 64 + lane] = b2;
    __syncthreads();
    for (int e = tid; e < h; e += 256) {
      float s = 0.0f;
      for (int k = 0; k < 8; ++k) s += red[128 * k + e];
      d1[w * h + e] = s;
    }
    if (tid < co) {
      float s = 0.0f;
      for (int k = 0; k < 8; ++k) s += red[1024 + 32 * k + tid];
      d2[h * co + tid] = s;
    }
    for (int q = 32; q > 0; q >>= 1) loss += __shfl_xor(loss, q, 64);
    __syncthreads();
    double* rl = reinterpret_cast<double*>(red);
    if (lane == 0) rl[wave] = loss;
    __syncthreads();
    if (tid == 0) pa.dpart[blockIdx.x] = (rl[0] + rl[1]) + (rl[2] + rl[3]);
  }
}

// ---- small-matrix GEMM: Out_b[r][n] = sum_k G[r][k] X_b[k][n] ---------------
// G row-major R x K (K % 4 == 0, zero beyond K), X_b rows of stride ldx,
// batch stride xbs.
// Each wave owns 32 columns and 4 row tiles (128 rows); blockIdx.z picks the
// 128-row band, so stages with many rows (the inverse stages: 2n rows) spread
// over more waves.  A block's four waves cover wpb column groups of
// `bpb = 4 / wpb` batches (wpb = 1 for the 32-column x stages, so no wave of a
// block idles there).
__global__ void __launch_bounds__(256)
k_lm_gemm(const u16* __restrict__ G, int R, int K, const u16* __restrict__ X, long long xbs, int ldx, int Nc,
          float* __restrict__ outf, u16* __restrict__ outb, long long obs, int ldo, int accumulate, int wpb,
          long long batches) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int lr = lane & 31, lg = lane >> 5;
  const long long b = (long long)blockIdx.y * (4 / wpb) + wave / wpb;
  if (b >= batches) return;  // no block-level synchronisation in this kernel
  const int n = (blockIdx.x * wpb + wave % wpb) * 32 + lr;
  const bool valid = n < Nc;
  const u16* Xb = X + b * xbs;
  {
    const int r0 = blockIdx.z * 128;
    f32x16 acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[t][i] = 0.0f;
    for (int kk = 0; kk < K; kk += 16) {
      const int kb = kk + lg * 8;
      const bool in0 = kb < K, in1 = kb + 4 < K;  // K % 4 == 0
      bf16x4 b0 = {0, 0, 0, 0}, b1 = {0, 0, 0, 0};
      if (valid && in0) {
#pragma unroll
        for (int j = 0; j < 4; ++j) b0[j] = (short)Xb[(long long)(kb + j) * ldx + n];
      }
      if (valid && in1) {
#pragma unroll
        for (int j = 0; j < 4; ++j) b1[j] = (short)Xb[(long long)(kb + 4 + j) * ldx + n];
      }
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int r = r0 + t * 32 + lr;
        if (r0 + t * 32 < R) {
          bf16x4 a0 = {0, 0, 0, 0}, a1 = {0, 0, 0, 0};
          if (r < R && in0) a0 = ld4(G + (long long)r * K + kb);
          if (r < R && in1) a1 = ld4(G + (long long)r * K + kb + 4);
          acc[t] = mfma16(a0, a1, b0, b1, acc[t]);
        }
      }
    }
    if (valid) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int row = r0 + t * 32 + 8 * (i >> 2) + 4 * lg + (i & 3);
          if (row >= R) continue;
          const long long o = b * obs + (long long)row * ldo + n;
          const float v = acc[t][i];
          if (outf) outf[o] = accumulate ? outf[o] + v : v;
          if (outb) outb[o] = f2bf(v);
        }
    }
  }
}

// ---- small-matrix GEMM with the slow index contracted: y and z stages ----------
// The same product as k_lm_gemm for X whose rows (the contracted index) are
// long: a wave takes 32 columns and RT * 32 rows of G, reads 32 x 32 tiles of X
// 16 bytes per lane and transposes them in registers (transpose_operand), where
// k_lm_gemm gathers eight 2-byte values per lane and operand.  A lane then holds
// one row of the result and stores eight columns at a time.  blockIdx.z picks
// the band of RT * 32 rows.  Needs K, Nc, ldx, xbs, ldo, obs % 8 == 0.
template <int RT>
__global__ void __launch_bounds__(256)
k_lm_rows(const u16* __restrict__ G, int R, int K, const u16* __restrict__ X, long long xbs, int ldx, int Nc,
          float* __restrict__ outf, u16* __restrict__ outb, long long obs, int ldo, long long items) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, lr = lane & 31, lg = lane >> 5;
  const long long item = (long long)blockIdx.x * 4 + wave;  // (batch, 32-column group)
  if (item >= items) return;  // no block-level synchronisation in this kernel
  const int groups = (Nc + 31) / 32;
  const long long b = item / groups;
  const int n0 = (int)(item % groups) * 32, r0 = blockIdx.z * (32 * RT);
  const u16* Xb = X + b * xbs;
  u32x4 id[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) id[s] = identity_operand(s, lr, lg);
  f32x16 acc[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) acc[t] = zero16();
  auto load = [&](int k0, u32x4(&x)[2]) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int n = n0 + 16 * s + 8 * lg;
      x[s] = u32x4{0, 0, 0, 0};
      if (k0 + lr < K && n < Nc) x[s] = *reinterpret_cast<const u32x4*>(Xb + (long long)(k0 + lr) * ldx + n);
    }
  };
  u32x4 nx[2];
  load(0, nx);
  for (int k0 = 0; k0 < K; k0 += 32) {
    const u32x4 x[2] = {nx[0], nx[1]};
    u32x4 xt[2];
    if (k0 + 32 < K) load(k0 + 32, nx);
    transpose_operand(x, id, xt);
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const int r = r0 + 32 * t + lr;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        if (k0 + 16 * s >= K) continue;
        const u32x4 g = r < R ? ld8(G + (long long)r * K, k0 + 16 * s + 8 * lg, K, true) : u32x4{0, 0, 0, 0};
        acc[t] = mfma32(xt[s], g, acc[t]);
      }
    }
  }
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const int r = r0 + 32 * t + lr;
    const long long o = b * obs + (long long)r * ldo + n0;
    if (outf) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = 8 * q + 4 * lg;
        if (r < R && n0 + c < Nc)
          *reinterpret_cast<f32x4*>(outf + o + c) = f32x4{acc[t][4 * q], acc[t][4 * q + 1], acc[t][4 * q + 2],
                                                          acc[t][4 * q + 3]};
      }
    } else {
      u32x4 op[2];
      to_operand(acc[t], op);
#pragma unroll
      for (int s = 0; s < 2; ++s)
        if (r < R) st8(outb + o - n0, n0 + 16 * s + 8 * lg, Nc, true, op[s]);
    }
  }
}

// ---- one layer along x lines: pointwise product, inverse x stage, activation, next x stage ----
// A wave takes one x line, 32 points at a time: v W (+ the inverse x stage of
// the line's spectral block X) + bias, the activation (or, backward, times
// GELU' of gpre), stored; and, contracted over the line's points with Gd, the
// x stage the next spectral path starts with - from the registers, so the
// activations are not read again for it (134 MB per layer at 128^3) nor
// gathered 2 bytes at a time.  With k_lm_rows it took an advance of two 128^3
// samples from 3.34 to 2.18 ms, a gradient over four from 21.2 to 16.9 ms.  Bt == nullptr: only the x stage of In.
// SEP: the inverse x stage is summed apart and added last (the order of the
// unfused path, which grids that 32 does not divide took).
// K, N <= 32 NT, N % 4 == 0, n % 8 == 0, 2m <= 32.
struct XLineArgs {
  const u16* In;       // [point][ldin]
  int ldin, K, N;
  const u16* Bt;       // [N][K]
  const float* bias;
  const u16 *G, *X;    // [n][2m]; [line][2m][N] (null: no line term)
  int m2;              // 2m
  const u16* gpre;     // [point][N]
  const float* gtab;
  u16 *outpre, *outact;
  const u16* Gd;       // [2m][n] (null: no x stage)
  u16* A1;             // [line][2m][N]
  int n;
  long long lines;
};

template <int NT, bool SEP>
__global__ void __launch_bounds__(256, NT == 1 ? (SEP ? 3 : 4) : 2) k_xline(XLineArgs a) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, lr = lane & 31, lg = lane >> 5;
  const long long line = (long long)blockIdx.x * 4 + wave;
  if (line >= a.lines) return;  // no block-level synchronisation in this kernel
  const int n = a.n, K = a.K, N = a.N, m2 = a.m2;
  const bool in16 = K % 8 == 0 && a.ldin % 8 == 0, k16 = K % 8 == 0, o16 = N % 8 == 0, g16 = m2 % 8 == 0;
  u32x4 bt[NT][2 * NT], xt[NT][2];
  f32x16 spec[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int c = 32 * t + lr;
#pragma unroll
    for (int s = 0; s < 2 * NT; ++s) {
      bt[t][s] = u32x4{0, 0, 0, 0};
      if (a.Bt && c < N) bt[t][s] = ld8(a.Bt + c * K, 16 * s + 8 * lg, K, k16);
    }
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      u32x4 x = {0, 0, 0, 0};
      if (a.G && c < N) {
        const u16* Xb = a.X + line * m2 * N + c;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int k = 16 * s + 8 * lg + j;
          if (k < m2) x[j >> 1] |= (unsigned)Xb[k * N] << (16 * (j & 1));
        }
      }
      xt[t][s] = x;
    }
    spec[t] = zero16();
  }
  u32x4 id[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) id[s] = identity_operand(s, lr, lg);
  // the next 32 points' channels are loaded while these are worked on
  auto point = [&](int x0) { return line * n + (x0 + lr < n ? x0 + lr : 0); };
  u32x4 vn[2 * NT];
#pragma unroll
  for (int s = 0; s < 2 * NT; ++s) vn[s] = ld8(a.In + point(0) * a.ldin, 16 * s + 8 * lg, K, in16);
  for (int x0 = 0; x0 < n; x0 += 32) {
    const bool in = x0 + lr < n;
    const long long p = point(x0);
    u32x4 src[NT][2];  // what the x stage contracts (lane = point)
    u32x4 vin[2 * NT];
#pragma unroll
    for (int s = 0; s < 2 * NT; ++s) vin[s] = vn[s];
    if (x0 + 32 < n) {
#pragma unroll
      for (int s = 0; s < 2 * NT; ++s) vn[s] = ld8(a.In + point(x0 + 32) * a.ldin, 16 * s + 8 * lg, K, in16);
    }
    if (a.Bt) {
      u32x2 gp[NT][4];
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int c = t * 32 + 8 * q + 4 * lg;
          gp[t][q] = u32x2{0, 0};
          if (a.gpre && c < N) gp[t][q] = *reinterpret_cast<const u32x2*>(a.gpre + p * N + c);
        }
      f32x16 acc[NT], acx[SEP ? NT : 1];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        acc[t] = zero16();
        if constexpr (SEP) acx[t] = zero16();
      }
#pragma unroll
      for (int s = 0; s < 2 * NT; ++s)
        if (16 * s < K) {
#pragma unroll
          for (int t = 0; t < NT; ++t) acc[t] = mfma32(bt[t][s], vin[s], acc[t]);
        }
      if (a.G) {
#pragma unroll
        for (int s = 0; s < 2; ++s)
          if (16 * s < m2) {
            const u32x4 g = in ? ld8(a.G + (x0 + lr) * m2, 16 * s + 8 * lg, m2, g16) : u32x4{0, 0, 0, 0};
#pragma unroll
            for (int t = 0; t < NT; ++t) {
              if constexpr (SEP)
                acx[t] = mfma32(xt[t][s], g, acx[t]);
              else
                acc[t] = mfma32(xt[t][s], g, acc[t]);
            }
          }
      }
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        f32x16 v = acc[t];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int c = t * 32 + 8 * q + 4 * lg;
          if (c >= N) continue;
          const f32x4 bb = a.bias ? *reinterpret_cast<const f32x4*>(a.bias + c) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            float r = v[4 * q + j] + bb[j];
            if constexpr (SEP) r += acx[t][4 * q + j];
            if (a.gpre) r *= a.gtab[(gp[t][q][j >> 1] >> (16 * (j & 1))) & 0xffffu];
            v[4 * q + j] = r;
          }
        }
        if (a.outpre || !a.outact) {
          to_operand(v, src[t]);
          if (a.outpre && in) {
#pragma unroll
            for (int s = 0; s < 2; ++s) st8(a.outpre + p * N, 32 * t + 16 * s + 8 * lg, N, o16, src[t][s]);
          }
        }
        if (a.outact) {
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            v[i] = gelu_f(v[i]);
            if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // four erfs in flight: registers
          }
          to_operand(v, src[t]);
          if (in) {
#pragma unroll
            for (int s = 0; s < 2; ++s) st8(a.outact + p * N, 32 * t + 16 * s + 8 * lg, N, o16, src[t][s]);
          }
        }
      }
    } else {
#pragma unroll
      for (int t = 0; t < NT; ++t) src[t][0] = vin[2 * t], src[t][1] = vin[2 * t + 1];
    }
    if (a.Gd) {
      u32x4 gd[2];
#pragma unroll
      for (int s = 0; s < 2; ++s)
        gd[s] = lr < m2 ? ld8(a.Gd + lr * n, x0 + 16 * s + 8 * lg, n, true) : u32x4{0, 0, 0, 0};
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        u32x4 tr[2];
        transpose_operand(src[t], id, tr);
#pragma unroll
        for (int s = 0; s < 2; ++s)
          if (x0 + 16 * s < n) spec[t] = mfma32(tr[s], gd[s], spec[t]);
      }
    }
  }
  if (a.Gd) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      u32x4 op[2];
      to_operand(spec[t], op);
#pragma unroll
      for (int s = 0; s < 2; ++s)
        if (lr < m2) st8(a.A1 + (line * m2 + lr) * N, 32 * t + 16 * s + 8 * lg, N, o16, op[s]);
    }
  }
}

// ---- per-mode complex mixing (FP32) -------------------------------------------
// S: [2][modes][w] (real block, imaginary block); R: [modes][w][w] (in, out),
// BF16.  `batches` spectra one after another (stride 2 modes w), the same
// weights.  Bound by reading R (28 MB a layer at width 32, 12 modes): V weights
// per load (V = 8: 16 bytes, where w % 8 == 0).
template <int V>
__device__ inline void ldw(const u16* p, float (&r)[V]) {
  if constexpr (V == 8) {
    const u32x4 v = *reinterpret_cast<const u32x4*>(p);
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = bf2f((u16)(v[e >> 1] >> (16 * (e & 1))));
  } else {
    r[0] = bf2f(p[0]);
  }
}

// T = R S: V outputs per thread
template <int V>
__global__ void __launch_bounds__(256)
k_mix_fwd(const float* __restrict__ S, const u16* __restrict__ Rr, const u16* __restrict__ Ri, int modes, int w,
          u16* __restrict__ Tb, int batches) {
  const long long gid = blockIdx.x * 256LL + threadIdx.x;
  const long long mo = (long long)modes * w, per = mo / V;
  if (gid >= per * batches) return;
  const long long bo = (gid / per) * 2 * mo;  // this spectrum's offset
  S += bo;
  Tb += bo;
  const long long id = gid % per;
  const long long md = id / (w / V);
  const int o = V * (int)(id % (w / V));
  float tr[V], ti[V];
#pragma unroll
  for (int e = 0; e < V; ++e) tr[e] = ti[e] = 0.f;
  for (int i = 0; i < w; ++i) {
    const float sr = S[md * w + i], si = S[mo + md * w + i];
    float rr[V], ri[V];
    ldw<V>(Rr + (md * w + i) * w + o, rr);
    ldw<V>(Ri + (md * w + i) * w + o, ri);
#pragma unroll
    for (int e = 0; e < V; ++e) {
      tr[e] += rr[e] * sr - ri[e] * si;
      ti[e] += rr[e] * si + ri[e] * sr;
    }
  }
#pragma unroll
  for (int e = 0; e < V; ++e) {
    Tb[md * w + o + e] = f2bf(tr[e]);
    Tb[mo + md * w + o + e] = f2bf(ti[e]);
  }
}

// dS = R^H dT: V weights per load
template <int V>
__global__ void __launch_bounds__(256)
k_mix_bwd_data(const float* __restrict__ dT, const u16* __restrict__ Rr, const u16* __restrict__ Ri,
               u16* __restrict__ dSb, int modes, int w) {
  const long long id = blockIdx.x * 256LL + threadIdx.x;
  if (id >= (long long)modes * w) return;
  const long long md = id / w;
  const int i = (int)(id % w);
  const long long mo = (long long)modes * w;
  float sr = 0.f, si = 0.f;
  for (int o = 0; o < w; o += V) {
    float rr[V], ri[V];
    ldw<V>(Rr + (md * w + i) * w + o, rr);
    ldw<V>(Ri + (md * w + i) * w + o, ri);
#pragma unroll
    for (int e = 0; e < V; ++e) {
      const float tr = dT[md * w + o + e], ti = dT[mo + md * w + o + e];
      sr += rr[e] * tr + ri[e] * ti;
      si += rr[e] * ti - ri[e] * tr;
    }
  }
  dSb[md * w + i] = f2bf(sr);
  dSb[mo + md * w + i] = f2bf(si);
}

__global__ void __launch_bounds__(256)
k_mix_bwd_w(const float* __restrict__ S, const float* __restrict__ dT, float* __restrict__ gRr,
            float* __restrict__ gRi, int modes, int w) {
  const long long id = blockIdx.x * 256LL + threadIdx.x;
  if (id >= (long long)modes * w * w) return;
  const long long md = id / (w * w);
  const int i = (int)((id / w) % w), o = (int)(id % w);
  const long long mo = (long long)modes * w;
  const float sr = S[md * w + i], si = S[mo + md * w + i];
  const float tr = dT[md * w + o], ti = dT[mo + md * w + o];
  gRr[id] += sr * tr + si * ti;
  gRi[id] += sr * ti - si * tr;
}

// ---- weight gradients on MFMA: G[k][n] += sum_p A[p][k] D[p][n], gb[n] += sum_p D[p][n] ----
// The reduction runs over points, the slow index of both operands.  A wave
// reads 32 points' channels 16 bytes per lane, transposes them in registers
// (an identity product, transpose_operand) and feeds them to the MFMA as
// operands over k = points, for the KT x NT output tiles at (k0, n0); the next
// 32 points are loaded meanwhile.  Each block writes one partial set
// part[block * KN + k * N + n] (KN = (K + 1) * N; row k = K holds the bias
// sums, written with k0 == 0); k_sum_partials adds the sets.  Streaming: at
// 128^3 a 32 x 32 gradient reads 268 MB.  lda, ldd % 4 == 0 and cover K, N
// rounded up to 4; P % 32 == 0.
template <int KT, int NT>
__global__ void __launch_bounds__(256)
k_wgrad_mfma(const u16* __restrict__ A, int lda, int K, const u16* __restrict__ D, int ldd, int N, long long P,
             int k0, int n0, float* __restrict__ part) {
  __shared__ float red[4 * 1024];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, lr = lane & 31, lg = lane >> 5;
  const bool a16 = lda % 8 == 0 && K % 8 == 0, d16 = ldd % 8 == 0 && N % 8 == 0;
  const long long ntile = P / 32, step = (long long)gridDim.x * 4;
  u32x4 id[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) id[s] = identity_operand(s, lr, lg);
  f32x16 acc[KT][NT];
  float bs[NT];
#pragma unroll
  for (int i = 0; i < KT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = zero16();
#pragma unroll
  for (int j = 0; j < NT; ++j) bs[j] = 0.0f;
  u32x4 an[KT][2], dn[NT][2];
  auto load = [&](long long tile) {
    const long long p = tile * 32 + lr;
#pragma unroll
    for (int i = 0; i < KT; ++i)
#pragma unroll
      for (int s = 0; s < 2; ++s) an[i][s] = ld8(A + p * lda, k0 + 32 * i + 16 * s + 8 * lg, K, a16);
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int s = 0; s < 2; ++s) dn[j][s] = ld8(D + p * ldd, n0 + 32 * j + 16 * s + 8 * lg, N, d16);
  };
  long long tile = (long long)blockIdx.x * 4 + wave;
  if (tile < ntile) load(tile);
  for (; tile < ntile; tile += step) {
    u32x4 a[KT][2], d[NT][2], aT[KT][2], dT[2];
#pragma unroll
    for (int i = 0; i < KT; ++i) a[i][0] = an[i][0], a[i][1] = an[i][1];
#pragma unroll
    for (int j = 0; j < NT; ++j) d[j][0] = dn[j][0], d[j][1] = dn[j][1];
    if (tile + step < ntile) load(tile + step);
#pragma unroll
    for (int i = 0; i < KT; ++i) transpose_operand(a[i], id, aT[i]);
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const f32x16 t = transpose_operand(d[j], id, dT);
#pragma unroll
      for (int e = 0; e < 16; ++e) bs[j] += t[e];
#pragma unroll
      for (int i = 0; i < KT; ++i)
#pragma unroll
        for (int s = 0; s < 2; ++s) acc[i][j] = mfma32(aT[i][s], dT[s], acc[i][j]);
    }
  }
  float* dst = part + (long long)blockIdx.x * (K + 1) * N;
#pragma unroll
  for (int i = 0; i < KT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      __syncthreads();
#pragma unroll
      for (int e = 0; e < 16; ++e) red[wave * 1024 + (8 * (e >> 2) + 4 * lg + (e & 3)) * 32 + lr] = acc[i][j][e];
      __syncthreads();
      for (int e = tid; e < 1024; e += 256) {
        const int k = k0 + 32 * i + (e >> 5), n = n0 + 32 * j + (e & 31);
        if (k < K && n < N) dst[k * N + n] = (red[e] + red[1024 + e]) + (red[2048 + e] + red[3072 + e]);
      }
    }
  if (k0 == 0) {
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NT; ++j) red[(wave * 2 + lg) * 32 * NT + 32 * j + lr] = bs[j];
    __syncthreads();
    if (tid < 32 * NT && n0 + tid < N) {
      float s = 0.0f;
      for (int k = 0; k < 8; ++k) s += red[k * 32 * NT + tid];
      dst[K * N + n0 + tid] = s;
    }
  }
}

// Adds nsets partial sets into gW / gb.  A block sums 16 consecutive entries:
// its 16 groups of 16 threads take every sixteenth set, then combine in LDS.
__global__ void __launch_bounds__(256) k_sum_partials(const float* __restrict__ part, int nsets, int K, int N,
                                                      float* __restrict__ gW, float* __restrict__ gb) {
  __shared__ float sh[16][17];
  const int KN = (K + 1) * N;
  const int el = threadIdx.x & 15, grp = threadIdx.x >> 4;
  const int e = blockIdx.x * 16 + el;
  float s = 0.f;
  if (e < KN)
    for (int b = grp; b < nsets; b += 16) s += part[(long long)b * KN + e];
  sh[grp][el] = s;
  __syncthreads();
  if (grp != 0 || e >= KN) return;
  s = 0.f;
#pragma unroll
  for (int g = 0; g < 16; ++g) s += sh[g][el];
  const int k = e / N, n = e % N;
  if (k < K)
    gW[k * N + n] += s;
  else
    gb[n] += s;
}

// ---- elementwise ------------------------------------------------------------------
// dpre = dpost * GELU'(pre) (or dpost when linear), in bf16.
__global__ void __launch_bounds__(256) k_gelu_bwd(const float* __restrict__ dpost, const u16* __restrict__ pre,
                                                  const float* __restrict__ gtab, u16* __restrict__ dpreb,
                                                  long long n, int linear) {
  const long long i = blockIdx.x * 256LL + threadIdx.x;
  if (i >= n) return;
  dpreb[i] = f2bf(linear ? dpost[i] : dpost[i] * gtab[pre[i]]);
}

// GELU' over every bf16 value (65536 entries, 256 KiB): the backward pass takes
// it at BF16 pre-activations, of which few distinct values occur, so a lookup
// (from the L1) replaces an erf and an exp.
__global__ void __launch_bounds__(256) k_gelu_table(float* __restrict__ gtab) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  gtab[i] = gelu_g(bf2f((u16)i));
}

// per-channel input normalisation (x - shift) * inv, applied before rounding to bf16
struct InNorm {
  float shift[8];
  float inv[8];
};

// planar f32 [cin][P] (or f64) -> normalised bf16 [P][ld] zero padded
template <typename TI>
__global__ void __launch_bounds__(256) k_pack_input(const TI* __restrict__ x, long long P, int cin, int ld,
                                                    InNorm nm, u16* __restrict__ out) {
  const long long p = blockIdx.x * 256LL + threadIdx.x;
  if (p >= P) return;
  for (int c = 0; c < ld; ++c)
    out[p * ld + c] = c < cin ? f2bf((float)((x[c * P + p] - (TI)nm.shift[c]) * (TI)nm.inv[c])) : (u16)0;
}

// loss: out f32 [P][co] vs target (y - x) / scale (planar f32); writes dout
// (bf16 [P][ldd] padded) and per-block squared-error partials
__global__ void __launch_bounds__(256) k_loss(const float* __restrict__ out, const float* __restrict__ x,
                                              const float* __restrict__ y, const float* __restrict__ scale,
                                              long long P, int co, int ldd, u16* __restrict__ doutb, double* __restrict__ part) {
  __shared__ double sh[4];
  const long long p = blockIdx.x * 256LL + threadIdx.x;
  double s = 0.0;
  if (p < P) {
    const float inv = 2.0f / (float)((double)P * co);
    for (int c = 0; c < ldd; ++c) {
      float g = 0.f;
      if (c < co) {
        const float tgt = (y[c * P + p] - x[c * P + p]) / scale[c];
        const float d = out[p * co + c] - tgt;
        s += (double)d * d;
        g = d * inv;
      }
      doutb[p * ldd + c] = f2bf(g);
    }
  }
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = sh[0] + sh[1] + sh[2] + sh[3];
}

__global__ void __launch_bounds__(256) k_sum_d(const double* __restrict__ part, int n, double* __restrict__ out) {
  __shared__ double sh[4];
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) s += part[i];
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) out[0] = sh[0] + sh[1] + sh[2] + sh[3];
}

// Adam on FP32 master weights; the gradient buffer is consumed (zeroed).
__global__ void __launch_bounds__(256) k_adam(float* __restrict__ th, float* __restrict__ m, float* __restrict__ v,
                                              float* __restrict__ g, long long n, float lr, float b1, float b2,
                                              float eps, float gscale, float c1, float c2) {
  const long long i = blockIdx.x * 256LL + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i] * gscale;
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  th[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  g[i] = 0.f;
}

// bf16 working copies: dst[r][c] = src[r*sr + c*sc] (transposes and padding)
__global__ void __launch_bounds__(256) k_to_bf16(const float* __restrict__ src, int rows, int cols, int ld_dst,
                                                 long long sr, long long sc, u16* __restrict__ dst) {
  const long long i = blockIdx.x * 256LL + threadIdx.x;
  if (i >= (long long)rows * ld_dst) return;
  const int r = (int)(i / ld_dst), c = (int)(i % ld_dst);
  dst[i] = c < cols ? f2bf(src[r * sr + c * sc]) : (u16)0;
}

// new_state[f][p] = state[f][p] + scale[f] * out[p][f]  (f64 planar state).
// st and res may be the same array (in-place advance): each element is read
// and then written by the same thread, so neither carries __restrict__.
__global__ void __launch_bounds__(256) k_apply(const double* st, const float* __restrict__ out,
                                               const float* __restrict__ scale, long long P, int co,
                                               double* res, double* __restrict__ part) {
  __shared__ double sh[4];
  const long long p = blockIdx.x * 256LL + threadIdx.x;
  double dc = 0.0;
  if (p < P) {
    for (int f = 0; f < co; ++f) {
      const double d = (double)scale[f] * (double)out[p * co + f];
      res[f * P + p] = st[f * P + p] + d;
      if (f == 0) dc = d;
    }
  }
  for (int o = 32; o > 0; o >>= 1) dc += __shfl_xor(dc, o, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = dc;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = sh[0] + sh[1] + sh[2] + sh[3];
}

// mass correction: c -= mean increment of c (the composition is conserved)
__global__ void __launch_bounds__(256) k_shift(double* __restrict__ c, long long P, const double* __restrict__ sum) {
  const long long p = blockIdx.x * 256LL + threadIdx.x;
  if (p < P) c[p] -= sum[0] / (double)P;
}

// partial sums of (a - b)^2 and b^2
__global__ void __launch_bounds__(256) k_rel_l2(const double* __restrict__ a, const double* __restrict__ b,
                                                long long n, double* __restrict__ part) {
  __shared__ double sh[2][4];
  double d2 = 0.0, b2 = 0.0;
  for (long long i = blockIdx.x * 256LL + threadIdx.x; i < n; i += 256LL * gridDim.x) {
    const double d = a[i] - b[i];
    d2 += d * d;
    b2 += b[i] * b[i];
  }
  for (int o = 32; o > 0; o >>= 1) {
    d2 += __shfl_xor(d2, o, 64);
    b2 += __shfl_xor(b2, o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    sh[0][threadIdx.x >> 6] = d2;
    sh[1][threadIdx.x >> 6] = b2;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = sh[0][0] + sh[0][1] + sh[0][2] + sh[0][3];
    part[2 * blockIdx.x + 1] = sh[1][0] + sh[1][1] + sh[1][2] + sh[1][3];
  }
}

}  // namespace

// ---- host side ----------------------------------------------------------------
// Kinds of work for the accounting of algorithmic bytes and flops
// (pf_fno_work): each launch counts its operands read once and its results
// written once, at their storage widths.
enum FnoKind { FK_LM = 0, FK_CM, FK_WGRAD, FK_WSUM, FK_MIX, FK_GELU, FK_ELEM, FK_COUNT };

struct pf_fno {
  pf_fno_config cfg;
  hipStream_t stream = nullptr;
  int acct = 0;  // accounting on
  bool fuse_x = false;  // x stages carried by the channel-mixing GEMMs (n % 32 == 0)
  bool xlines = false;     // layers as passes along x lines (k_xline: width <= 64, 16 modes at most)
  bool fuse_proj = false;  // the projection in one pass (width <= 32, one MFMA tile)
  double acct_bytes[FK_COUNT] = {}, acct_flops[FK_COUNT] = {};
  long long acct_n[FK_COUNT] = {};
  long long P = 0;
  int mode_count = 0;   // (2m)^2 m
  int cinp = 8, coutp = 8;  // padded channel counts (K % 8)
  int64_t nparams = 0;
  // parameter offsets in the flat FP32 vector
  long long o_Wl, o_bl, o_P1, o_c1, o_P2, o_c2;
  std::vector<long long> o_Rr, o_Ri, o_W, o_b;
  float *th = nullptr, *gr = nullptr, *am = nullptr, *av = nullptr;
  long long adam_t = 0;
  // bf16 working weights
  u16 *bWliftT = nullptr, *bP1T = nullptr, *bP1 = nullptr, *bP2T = nullptr, *bP2 = nullptr;
  std::vector<u16*> bWT, bW, bRr, bRi;
  // DFT matrices (forward and inverse stages, and their transposes)
  u16 *Gxf, *Gyf, *Gzf, *Gxi, *Gyi, *Gzi, *GxfT, *GyfT, *GzfT, *GxiT, *GyiT, *GziT;
  float* scale = nullptr;  // output scale per channel
  InNorm innorm;           // input normalisation (identity by default)
  // activations
  u16* xin = nullptr;
  std::vector<u16*> v, pre;
  std::vector<float*> S;
  u16 *hpre = nullptr, *hact = nullptr;
  u16 *A1 = nullptr, *A2 = nullptr, *Tb = nullptr, *B3 = nullptr, *B2 = nullptr;
  float *B1 = nullptr, *outf = nullptr;
  // backward buffers
  float *dvf = nullptr, *dT = nullptr;
  u16 *dpreb = nullptr, *dpreb2 = nullptr, *douthb = nullptr, *dhb = nullptr, *dSb = nullptr;
  float* gtab = nullptr;  // GELU' over the bf16 values
  float* part = nullptr;
  double* dpart = nullptr;
  double* dsum = nullptr;
  double* hsum = nullptr;  // pinned
  // batched inference over `bcap` samples (allocated on first use, grown on demand)
  int bcap = 0;
  std::vector<void*> ballocs;
  u16 *bxin = nullptr, *bv0 = nullptr, *bv1 = nullptr, *bA1 = nullptr, *bA2 = nullptr, *bTb = nullptr, *bB3 = nullptr,
      *bB2 = nullptr, *bhact = nullptr;
  float *bS = nullptr, *bB1 = nullptr, *boutf = nullptr;
  double *bdpart = nullptr, *bdsum = nullptr;
  // ensemble surrogate advance: current, network and plain states of `ecap` members
  int ecap = 0;
  std::vector<void*> eallocs;
  double *eX = nullptr, *eY = nullptr, *eP = nullptr;
  // checked-advance buffers (allocated on first use)
  double* adv_next = nullptr;
  double* adv_ref = nullptr;
  double* l2_part = nullptr;
  double* l2_host = nullptr;  // pinned
  std::vector<void*> allocs;
};

#define FH(call)                                     \
  do {                                               \
    if ((call) != hipSuccess) return PF_ERR_HIP;     \
  } while (0)

static pf_status falloc(pf_fno* F, void** p, size_t bytes) {
  if (hipMalloc(p, bytes) != hipSuccess) {
    *p = nullptr;
    return PF_ERR_OOM;
  }
  F->allocs.push_back(*p);
  return PF_OK;
}

static inline unsigned gdiv(long long n, int b) { return (unsigned)((n + b - 1) / b); }

static inline void account(pf_fno* F, int kind, double bytes, double flops) {
  if (!F->acct) return;
  F->acct_bytes[kind] += bytes;
  F->acct_flops[kind] += flops;
  F->acct_n[kind] += 1;
}

// Real DFT matrices for the six stages (see the header comment of this file).
static void build_dft(int n, int m, std::vector<std::vector<float>>& out) {
  const double pi = 3.14159265358979323846;
  std::vector<int> kx(m), kyz(2 * m);
  for (int i = 0; i < m; ++i) kx[i] = i;
  for (int i = 0; i < m; ++i) kyz[i] = i, kyz[m + i] = n - m + i;
  const int m2 = 2 * m;
  // x forward: rows (ri, kx) 2m, cols x n
  std::vector<float> xf(2 * m * n), xi(n * 2 * m), yf(2 * m2 * 2 * n), yi(2 * n * 2 * m2);
  for (int k = 0; k < m; ++k)
    for (int x = 0; x < n; ++x) {
      const double a = 2 * pi * kx[k] * x / n;
      xf[(0 * m + k) * n + x] = (float)cos(a);
      xf[(1 * m + k) * n + x] = (float)(-sin(a));
      const double w = (kx[k] == 0 ? 1.0 : 2.0) / ((double)n * n * n);
      xi[x * 2 * m + 0 * m + k] = (float)(w * cos(a));
      xi[x * 2 * m + 1 * m + k] = (float)(-w * sin(a));
    }
  // y / z forward: rows (ro, k) 2*m2, cols (y, ri) 2n ; inverse: rows (y, ro) 2n, cols (ri, k) 2*m2
  for (int k = 0; k < m2; ++k)
    for (int y = 0; y < n; ++y) {
      const double a = 2 * pi * kyz[k] * y / n;
      const float C = (float)cos(a), S = (float)sin(a);
      const int K2 = 2 * n;
      yf[(0 * m2 + k) * K2 + y * 2 + 0] = C;
      yf[(0 * m2 + k) * K2 + y * 2 + 1] = S;
      yf[(1 * m2 + k) * K2 + y * 2 + 0] = -S;
      yf[(1 * m2 + k) * K2 + y * 2 + 1] = C;
      const int Kq = 2 * m2;
      yi[(y * 2 + 0) * Kq + 0 * m2 + k] = C;
      yi[(y * 2 + 0) * Kq + 1 * m2 + k] = -S;
      yi[(y * 2 + 1) * Kq + 0 * m2 + k] = S;
      yi[(y * 2 + 1) * Kq + 1 * m2 + k] = C;
    }
  out = {xf, yf, yf, xi, yi, yi};
}

static std::vector<float> transpose(const std::vector<float>& a, int R, int K) {
  std::vector<float> t((size_t)R * K);
  for (int r = 0; r < R; ++r)
    for (int k = 0; k < K; ++k) t[(size_t)k * R + r] = a[(size_t)r * K + k];
  return t;
}

static pf_status upload_bf16(pf_fno* F, const std::vector<float>& h, u16** d) {
  std::vector<u16> b(h.size());
  for (size_t i = 0; i < h.size(); ++i) b[i] = f2bf(h[i]);
  pf_status s = falloc(F, (void**)d, sizeof(u16) * b.size());
  if (s != PF_OK) return s;
  if (hipMemcpy(*d, b.data(), sizeof(u16) * b.size(), hipMemcpyHostToDevice) != hipSuccess) return PF_ERR_HIP;
  return PF_OK;
}

// algorithmic bytes of one channel-mixing GEMM over `points` points
static double cm_bytes(double points, int K, int N, const float* bias, const float* resid, const float* outf,
                       const u16* outpre, const u16* outact) {
  double b = points * K * 2.0 + 2.0 * N * K + (bias ? 4.0 * N : 0.0);
  if (resid) b += points * N * 4.0;
  if (outf) b += points * N * 4.0;
  if (outpre) b += points * N * 2.0;
  if (outact) b += points * N * 2.0;
  return b;
}

static void lm(pf_fno* F, const u16* G, int R, int K, const u16* X, long long xbs, int ldx, int Nc, int batches,
               float* outf, u16* outb, long long obs, int ldo, int accumulate) {
  const int wpb = Nc <= 32 ? 1 : (Nc <= 64 ? 2 : 4);  // waves per batch
  const double cols = (double)Nc * batches;
  account(F, FK_LM, 2.0 * R * K + 2.0 * K * cols + (outf ? (accumulate ? 8.0 : 4.0) : 2.0) * R * cols,
          2.0 * R * K * cols);
  // the batches in launches of at most 65535 blocks along y
  const long long per = 65535LL * (4 / wpb);
  for (long long b0 = 0; b0 < batches; b0 += per) {
    const long long nb = std::min<long long>(per, batches - b0);
    dim3 grid(gdiv(Nc, 32 * wpb), gdiv(nb, 4 / wpb), gdiv(R, 128));
    k_lm_gemm<<<grid, 256, 0, F->stream>>>(G, R, K, X + b0 * xbs, xbs, ldx, Nc, outf ? outf + b0 * obs : nullptr,
                                           outb ? outb + b0 * obs : nullptr, obs, ldo, accumulate, wpb, nb);
  }
}

// y and z stages of the truncated DFT (G: R x K, K % 8 == 0; columns % 8 == 0)
static void lm_rows(pf_fno* F, const u16* G, int R, int K, const u16* X, long long xbs, int ldx, int Nc, int batches,
                    float* outf, u16* outb, long long obs, int ldo) {
  const double cols = (double)Nc * batches;
  account(F, FK_LM, 2.0 * R * K + 2.0 * K * cols + (outf ? 4.0 : 2.0) * R * cols, 2.0 * R * K * cols);
  const long long items = (long long)batches * gdiv(Nc, 32);
  // 64 rows per wave where that fills the chip (four waves per SIMD), else 32
  const bool two = R > 32 && items * gdiv(R, 64) >= 4096;
  dim3 grid(gdiv(items, 4), 1, gdiv(R, two ? 64 : 32));
  if (two)
    k_lm_rows<2><<<grid, 256, 0, F->stream>>>(G, R, K, X, xbs, ldx, Nc, outf, outb, obs, ldo, items);
  else
    k_lm_rows<1><<<grid, 256, 0, F->stream>>>(G, R, K, X, xbs, ldx, Nc, outf, outb, obs, ldo, items);
}

// one pass along the x lines of `samples` grids (see k_xline)
static void xline(pf_fno* F, XLineArgs a, long long samples) {
  const pf_fno_config& c = F->cfg;
  a.m2 = 2 * c.modes;
  a.n = c.n;
  a.lines = samples * c.n * c.n;
  a.gtab = F->gtab;
  const double points = (double)F->P * samples;
  if (a.Bt) {
    double bytes = cm_bytes(points, a.K, a.N, a.bias, nullptr, nullptr, a.outpre, a.outact);
    double flops = 2.0 * points * a.K * a.N;
    if (a.G) {
      bytes += 2.0 * a.n * a.m2 + (double)a.lines * a.m2 * a.N * 2.0;
      flops += 2.0 * points * a.m2 * a.N;
    }
    if (a.gpre) bytes += points * a.N * 2.0;
    account(F, FK_CM, bytes, flops);
  }
  if (a.Gd)
    account(F, FK_LM, 2.0 * a.n * a.m2 + 2.0 * a.lines * a.m2 * a.N + (a.Bt ? 0.0 : 2.0 * points * a.K),
            2.0 * points * a.m2 * a.N);
  const unsigned grid = gdiv(a.lines, 4);
  if (a.N <= 32)
    F->fuse_x ? k_xline<1, false><<<grid, 256, 0, F->stream>>>(a) : k_xline<1, true><<<grid, 256, 0, F->stream>>>(a);
  else
    F->fuse_x ? k_xline<2, false><<<grid, 256, 0, F->stream>>>(a) : k_xline<2, true><<<grid, 256, 0, F->stream>>>(a);
}

static void cm_launch(pf_fno* F, long long points, const u16* In, int ldin, int K, const u16* Bt, int N,
                      const float* bias, const float* resid, int ldres, float* outf, u16* outpre, u16* outact,
                      int ldout, const LineTerm& lt, const u16* gpre = nullptr) {
  const unsigned grid = (unsigned)(points / 128);
  double bytes = cm_bytes((double)points, K, N, bias, resid, outf, outpre, outact);
  double flops = 2.0 * points * K * N;
  if (lt.G) {
    bytes += 2.0 * lt.R * lt.K + (double)(points / lt.R) * lt.K * N * 2.0;
    flops += 2.0 * points * lt.K * N;
  }
  if (gpre) bytes += points * N * 2.0;
  account(F, FK_CM, bytes, flops);
  auto go = [&](auto NC) {
    k_cm_gemm<decltype(NC)::value><<<grid, 256, 0, F->stream>>>(In, ldin, K, Bt, N, bias, resid, ldres, outf, outpre,
                                                                outact, ldout, lt, gpre, F->gtab);
  };
  if (N <= 32)
    go(std::integral_constant<int, 1>{});
  else if (N <= 64)
    go(std::integral_constant<int, 2>{});
  else
    go(std::integral_constant<int, 4>{});
}

static void cm(pf_fno* F, const u16* In, int ldin, int K, const u16* Bt, int N, const float* bias, const float* resid,
               int ldres, float* outf, u16* outpre, u16* outact, int ldout,
               const LineTerm& lt = LineTerm(), const u16* gpre = nullptr) {
  cm_launch(F, F->P, In, ldin, K, Bt, N, bias, resid, ldres, outf, outpre, outact, ldout, lt, gpre);
}

static void sum_partials(pf_fno* F, const float* part, int nb, int K, int N, float* gW, float* gb) {
  const double kn = (double)(K + 1) * N;
  account(F, FK_WSUM, 4.0 * nb * kn + 8.0 * kn, (double)nb * kn);
  k_sum_partials<<<gdiv((K + 1) * N, 16), 256, 0, F->stream>>>(part, nb, K, N, gW, gb);
}

static void wgrad(pf_fno* F, const u16* A, int lda, int K, const u16* D, int ldd, int N, float* gW, float* gb) {
  const int nb = pf::wgrad_blocks(F->P);
  for (int k0 = 0; k0 < K; k0 += 64)
    for (int n0 = 0; n0 < N; n0 += 64) {
      const int kk = std::min(64, K - k0), nn = std::min(64, N - n0);
      account(F, FK_WGRAD, (double)F->P * 2.0 * (kk + nn) + 4.0 * nb * kk * nn, 2.0 * F->P * kk * nn);
      auto go = [&](auto KC, auto NC) {
        k_wgrad_mfma<decltype(KC)::value, decltype(NC)::value>
            <<<nb, 256, 0, F->stream>>>(A, lda, K, D, ldd, N, F->P, k0, n0, F->part);
      };
      using one = std::integral_constant<int, 1>;
      using two = std::integral_constant<int, 2>;
      if (kk <= 32)
        nn <= 32 ? go(one{}, one{}) : go(one{}, two{});
      else
        nn <= 32 ? go(two{}, one{}) : go(two{}, two{});
    }
  sum_partials(F, F->part, nb, K, N, gW, gb);
}

// The fused projection over `points` points.
static ProjArgs proj_args(const pf_fno* F, const u16* v, long long points) {
  ProjArgs a = {};
  a.v = v;
  a.P1T = F->bP1T;
  a.P2T = F->bP2T;
  a.P1 = F->bP1;
  a.P2 = F->bP2;
  a.c1 = F->th + F->o_c1;
  a.c2 = F->th + F->o_c2;
  a.P = points;
  a.w = F->cfg.width;
  a.h = F->cfg.hidden;
  a.co = F->cfg.cout;
  a.gtab = F->gtab;
  return a;
}

template <bool TRAIN>
static int proj_launch(pf_fno* F, const ProjArgs& a) {
  const int nb = pf::proj_blocks(a.P);
  if (a.h <= 64)
    k_proj<TRAIN, 2><<<nb, 256, 0, F->stream>>>(a);
  else if (a.h <= 96)
    k_proj<TRAIN, 3><<<nb, 256, 0, F->stream>>>(a);
  else
    k_proj<TRAIN, 4><<<nb, 256, 0, F->stream>>>(a);
  return nb;
}

// out (f32 [points][cout]) of v_L (bf16 [points][width])
static void project(pf_fno* F, const u16* v, long long points, float* out) {
  const pf_fno_config& c = F->cfg;
  ProjArgs a = proj_args(F, v, points);
  a.outf = out;
  // accounted as its two products; the hidden layer moves no bytes
  account(F, FK_CM, 2.0 * points * c.width + 2.0 * c.hidden * c.width, 2.0 * points * c.hidden * c.width);
  account(F, FK_CM, 4.0 * points * c.cout + 2.0 * c.hidden * c.cout, 2.0 * points * c.hidden * c.cout);
  proj_launch<false>(F, a);
}

// Projection, loss and the projection's backward pass: d v_L into dpre, the
// gradients of P1, c1, P2, c2 added to the gradient buffer, the summed squared
// error into F->dsum.
static void project_train(pf_fno* F, const float* x, const float* y, u16* dpre) {
  const pf_fno_config& c = F->cfg;
  const int w = c.width, h = c.hidden, co = c.cout;
  ProjArgs a = proj_args(F, F->pre[c.layers - 1], F->P);
  a.x = x;
  a.y = y;
  a.scale = F->scale;
  a.inv = 2.0f / (float)((double)F->P * co);
  a.dpre = dpre;
  a.part1 = F->part;
  a.part2 = F->part + pf::proj_parts(F->P, w, h, co).second;
  a.dpart = F->dpart;
  account(F, FK_CM, (double)F->P * (4.0 * w + 8.0 * co) + 4.0 * h * (w + co), 6.0 * F->P * h * (w + co));
  const int nb = proj_launch<true>(F, a);
  k_sum_d<<<1, 256, 0, F->stream>>>(F->dpart, nb, F->dsum);
  sum_partials(F, a.part1, nb, w, h, F->gr + F->o_P1, F->gr + F->o_c1);
  sum_partials(F, a.part2, nb, h, co, F->gr + F->o_P2, F->gr + F->o_c2);
}

// refresh the bf16 working weights from the FP32 master vector
static void refresh(pf_fno* F) {
  const pf_fno_config& c = F->cfg;
  const int w = c.width, h = c.hidden;
  hipStream_t s = F->stream;
  auto cvt = [&](long long off, int rows, int cols, int ld, long long sr, long long sc, u16* dst) {
    k_to_bf16<<<gdiv((long long)rows * ld, 256), 256, 0, s>>>(F->th + off, rows, cols, ld, sr, sc, dst);
  };
  // W_lift^T [w][cinp]: dst[o][c] = W_lift[c][o]
  cvt(F->o_Wl, w, c.cin, F->cinp, 1, w, F->bWliftT);
  for (int l = 0; l < c.layers; ++l) {
    cvt(F->o_W[l], w, w, w, 1, w, F->bWT[l]);   // W^T[o][i] = W[i][o]
    cvt(F->o_W[l], w, w, w, w, 1, F->bW[l]);    // W[i][o]
    const long long nr = (long long)F->mode_count * w * w;
    k_to_bf16<<<gdiv(nr, 256), 256, 0, s>>>(F->th + F->o_Rr[l], 1, (int)nr, (int)nr, 0, 1, F->bRr[l]);
    k_to_bf16<<<gdiv(nr, 256), 256, 0, s>>>(F->th + F->o_Ri[l], 1, (int)nr, (int)nr, 0, 1, F->bRi[l]);
  }
  cvt(F->o_P1, h, w, w, 1, h, F->bP1T);        // P1^T [h][w]
  cvt(F->o_P1, w, h, h, h, 1, F->bP1);         // P1 [w][h]
  cvt(F->o_P2, c.cout, h, h, 1, c.cout, F->bP2T);  // P2^T [cout][h]
  cvt(F->o_P2, h, c.cout, F->coutp, c.cout, 1, F->bP2);  // P2 [h][coutp]
}

// per-mode mixing of `batches` spectra: S (f32) and R (bf16) in, T (bf16) out
static double mix_fwd_bytes(int modes, int w, int batches) {
  const double mo = (double)modes * w;
  return batches * (2.0 * mo * 4.0 + 2.0 * mo * 2.0) + 2.0 * modes * (double)w * w * 2.0;
}

// the inverse x stage of a layer's spectral path as a line term (B2: the
// inverse y stage's output, one 2m x w block per x line)
static LineTerm x_inverse(const pf_fno* F, const u16* B2) {
  LineTerm lt;
  lt.G = F->Gxi;
  lt.K = 2 * F->cfg.modes;
  lt.R = F->cfg.n;
  lt.X = B2;
  lt.xbs = (long long)2 * F->cfg.modes * F->cfg.width;
  lt.ldx = F->cfg.width;
  return lt;
}

// Buffers of a forward pass over `B` samples.
struct FwdBufs {
  const u16* xin;
  u16 *A1, *A2, *Tb, *B3, *B2;
  float* B1;
};

// One layer's spectral path from the x stage's output (A1) to the inverse y
// stage's (B2); S: the spectrum before the mixing (f32).
static void spectral_fwd(pf_fno* F, const FwdBufs& u, int l, int B, float* S) {
  const pf_fno_config& c = F->cfg;
  const int n = c.n, w = c.width, m = c.modes, m2 = 2 * m;
  const int Nz = m2 * m * w;
  const long long spec = 2LL * F->mode_count * w;
  // y (batch sample, z), z (batch sample)
  lm_rows(F, F->Gyf, 2 * m2, 2 * n, u.A1, (long long)n * 2 * m * w, m * w, m * w, B * n, nullptr, u.A2,
          (long long)2 * m2 * m * w, m * w);
  lm_rows(F, F->Gzf, 2 * m2, 2 * n, u.A2, 2LL * n * Nz, Nz, Nz, B, S, nullptr, spec, Nz);
  account(F, FK_MIX, mix_fwd_bytes(F->mode_count, w, B), 8.0 * F->mode_count * w * w * B);
  auto mix = [&](auto VC) {
    constexpr int V = decltype(VC)::value;
    k_mix_fwd<V><<<gdiv((long long)F->mode_count * w / V * B, 256), 256, 0, F->stream>>>(S, F->bRr[l], F->bRi[l],
                                                                                         F->mode_count, w, u.Tb, B);
  };
  w % 8 == 0 ? mix(std::integral_constant<int, 8>{}) : mix(std::integral_constant<int, 1>{});
  lm_rows(F, F->Gzi, 2 * n, 2 * m2, u.Tb, spec, Nz, Nz, B, nullptr, u.B3, 2LL * n * Nz, Nz);
  lm_rows(F, F->Gyi, 2 * n, 2 * m2, u.B3, (long long)2 * m2 * m * w, m * w, m * w, B * n, nullptr, u.B2,
          (long long)2 * n * m * w, m * w);
}

// Lift and layers over B samples.  v(l): the layer's input, pre(l): where its
// pre-activation is kept (null: not kept; the last layer's, v_L, always is),
// S(l): its spectrum.
template <class V, class Pre, class Sp>
static void forward_layers(pf_fno* F, const FwdBufs& u, int B, V v, Pre pre, Sp S) {
  const pf_fno_config& c = F->cfg;
  const int n = c.n, w = c.width, m = c.modes;
  const float* th = F->th;
  const long long points = F->P * B;
  if (F->xlines) {
    XLineArgs a = {};
    a.In = u.xin;
    a.ldin = a.K = F->cinp;
    a.N = w;
    a.Bt = F->bWliftT;
    a.bias = th + F->o_bl;
    a.outpre = v(0);
    a.Gd = F->Gxf;
    a.A1 = u.A1;
    xline(F, a, B);
  } else {
    cm_launch(F, points, u.xin, F->cinp, F->cinp, F->bWliftT, w, th + F->o_bl, nullptr, 0, nullptr, v(0), nullptr, w,
              LineTerm());
  }
  for (int l = 0; l < c.layers; ++l) {
    const bool last = l == c.layers - 1;  // linear
    if (!F->xlines)
      lm(F, F->Gxf, 2 * m, n, v(l), (long long)n * w, w, w, B * n * n, nullptr, u.A1, (long long)2 * m * w, w, 0);
    spectral_fwd(F, u, l, B, S(l));
    // pointwise path, bias, the spectral part's inverse x stage, activation, and
    // the next layer's x stage
    if (F->xlines) {
      XLineArgs a = {};
      a.In = v(l);
      a.ldin = a.K = a.N = w;
      a.Bt = F->bWT[l];
      a.bias = th + F->o_b[l];
      a.G = F->Gxi;
      a.X = u.B2;
      a.outpre = pre(l);
      a.outact = last ? nullptr : v(l + 1);
      a.Gd = last ? nullptr : F->Gxf;
      a.A1 = u.A1;
      xline(F, a, B);
    } else if (F->fuse_x) {
      cm_launch(F, points, v(l), w, w, F->bWT[l], w, th + F->o_b[l], nullptr, 0, nullptr, pre(l),
                last ? nullptr : v(l + 1), w, x_inverse(F, u.B2));
    } else {
      lm(F, F->Gxi, n, 2 * m, u.B2, (long long)2 * m * w, w, w, B * n * n, u.B1, nullptr, (long long)n * w, w, 0);
      cm_launch(F, points, v(l), w, w, F->bWT[l], w, th + F->o_b[l], u.B1, w, nullptr, pre(l),
                last ? nullptr : v(l + 1), w, LineTerm());
    }
  }
}

// forward pass for the packed input F->xin up to v_L (F->pre[layers - 1]);
// keep: with the other layers' pre-activations, for the backward pass
static void forward_layers(pf_fno* F, bool keep) {
  const int L = F->cfg.layers;
  const FwdBufs u = {F->xin, F->A1, F->A2, F->Tb, F->B3, F->B2, F->B1};
  forward_layers(
      F, u, 1, [&](int l) { return F->v[l]; },
      [&](int l) { return keep || l == L - 1 ? F->pre[l] : (u16*)nullptr; }, [&](int l) { return F->S[l]; });
}

// the projection as GEMMs through the hidden layer (width > 32)
static void project_gemms(pf_fno* F) {
  const pf_fno_config& c = F->cfg;
  const int w = c.width, h = c.hidden;
  const float* th = F->th;
  cm(F, F->pre[c.layers - 1], w, w, F->bP1T, h, th + F->o_c1, nullptr, 0, nullptr, F->hpre, F->hact, h);
  cm(F, F->hact, h, h, F->bP2T, c.cout, th + F->o_c2, nullptr, 0, F->outf, nullptr, nullptr, c.cout);
}

// forward pass for the packed input F->xin; leaves the result in F->outf
static void forward(pf_fno* F) {
  forward_layers(F, false);
  if (F->fuse_proj)
    project(F, F->pre[F->cfg.layers - 1], F->P, F->outf);
  else
    project_gemms(F);
}

// Projection, loss (sum of squares into F->dsum) and backward pass for the
// state pair x, y.  Every gradient that a weight gradient reads is BF16, as the
// MFMA takes it.
static void loss_backward(pf_fno* F, const float* x, const float* y) {
  const pf_fno_config& c = F->cfg;
  const int n = c.n, w = c.width, m = c.modes, m2 = 2 * m, h = c.hidden, co = c.cout;
  const long long P = F->P;
  float* g = F->gr;
  u16* db[2] = {F->dpreb, F->dpreb2};  // d pre of the layer, and of the one before
  if (F->fuse_proj) {
    project_train(F, x, y, db[0]);
  } else {
    project_gemms(F);
    const unsigned nb = pf::pointwise_blocks(P);
    account(F, FK_ELEM, (double)P * co * (4.0 * 3) + (double)P * F->coutp * 2.0, 0.0);
    k_loss<<<nb, 256, 0, F->stream>>>(F->outf, x, y, F->scale, P, co, F->coutp, F->douthb, F->dpart);
    k_sum_d<<<1, 256, 0, F->stream>>>(F->dpart, (int)nb, F->dsum);
    // out = hact P2 + c2
    wgrad(F, F->hact, h, h, F->douthb, F->coutp, co, g + F->o_P2, g + F->o_c2);
    // d hpre = (d out P2^T) GELU'(hpre), formed in the GEMM's epilogue
    cm(F, F->douthb, F->coutp, F->coutp, F->bP2, h, nullptr, nullptr, 0, nullptr, F->dhb, nullptr, h, LineTerm(),
       F->hpre);
    wgrad(F, F->pre[c.layers - 1], w, w, F->dhb, h, h, g + F->o_P1, g + F->o_c1);
    cm(F, F->dhb, h, h, F->bP1, w, nullptr, nullptr, 0, nullptr, db[0], nullptr, w);
  }
  const int Nz = m2 * m * w;
  // the spectral path's transposed stages from the x stage's output (B2) down to A1
  auto spectral_back = [&](int l) {
    lm_rows(F, F->GyiT, 2 * m2, 2 * n, F->B2, (long long)2 * n * m * w, m * w, m * w, n, nullptr, F->B3,
            (long long)2 * m2 * m * w, m * w);
    lm_rows(F, F->GziT, 2 * m2, 2 * n, F->B3, 0, Nz, Nz, 1, F->dT, nullptr, 0, Nz);
    account(F, FK_MIX, 2.0 * F->mode_count * w * 4.0 * 2 + 2.0 * F->mode_count * (double)w * w * 8.0,
            8.0 * F->mode_count * w * w);
    account(F, FK_MIX, 2.0 * F->mode_count * w * (4.0 + 2.0) + 2.0 * F->mode_count * (double)w * w * 2.0,
            8.0 * F->mode_count * w * w);
    k_mix_bwd_w<<<gdiv((long long)F->mode_count * w * w, 256), 256, 0, F->stream>>>(
        F->S[l], F->dT, g + F->o_Rr[l], g + F->o_Ri[l], F->mode_count, w);
    auto mix = [&](auto VC) {
      k_mix_bwd_data<decltype(VC)::value><<<gdiv((long long)F->mode_count * w, 256), 256, 0, F->stream>>>(
          F->dT, F->bRr[l], F->bRi[l], F->dSb, F->mode_count, w);
    };
    w % 8 == 0 ? mix(std::integral_constant<int, 8>{}) : mix(std::integral_constant<int, 1>{});
    lm_rows(F, F->GzfT, 2 * n, 2 * m2, F->dSb, 0, Nz, Nz, 1, nullptr, F->A2, 0, Nz);
    lm_rows(F, F->GyfT, 2 * n, 2 * m2, F->A2, (long long)2 * m2 * m * w, m * w, m * w, n, nullptr, F->A1,
            (long long)2 * n * m * w, m * w);
  };
  if (F->xlines) {
    XLineArgs a = {};
    a.In = db[0];
    a.ldin = a.K = a.N = w;
    a.Gd = F->GxiT;
    a.A1 = F->B2;
    xline(F, a, 1);
  }
  for (int l = c.layers - 1; l >= 0; --l) {
    wgrad(F, F->v[l], w, w, db[0], w, w, g + F->o_W[l], g + F->o_b[l]);
    if (!F->xlines)
      lm(F, F->GxiT, 2 * m, n, db[0], (long long)n * w, w, w, n * n, nullptr, F->B2, (long long)2 * m * w, w, 0);
    spectral_back(l);
    // d v_l = d pre_l W^T + (transposed x stage of A1), times GELU'(pre_{l-1}) to
    // give d pre_{l-1} (d v_0 for l = 0)
    const u16* gp = l > 0 ? F->pre[l - 1] : nullptr;
    if (F->xlines) {
      XLineArgs a = {};
      a.In = db[0];
      a.ldin = a.K = a.N = w;
      a.Bt = F->bW[l];
      a.G = F->GxfT;
      a.X = F->A1;
      a.gpre = gp;
      a.outpre = db[1];
      a.Gd = l > 0 ? F->GxiT : nullptr;  // and the next spectral path's x stage
      a.A1 = F->B2;
      xline(F, a, 1);
      std::swap(db[0], db[1]);
    } else if (F->fuse_x) {
      LineTerm lt;
      lt.G = F->GxfT;
      lt.K = 2 * m;
      lt.R = n;
      lt.X = F->A1;
      lt.xbs = (long long)2 * m * w;
      lt.ldx = w;
      cm(F, db[0], w, w, F->bW[l], w, nullptr, nullptr, 0, nullptr, db[1], nullptr, w, lt, gp);
      std::swap(db[0], db[1]);
    } else {
      cm(F, db[0], w, w, F->bW[l], w, nullptr, nullptr, 0, F->dvf, nullptr, nullptr, w);
      lm(F, F->GxfT, n, 2 * m, F->A1, (long long)2 * m * w, w, w, n * n, F->dvf, nullptr, (long long)n * w, w, 1);
      account(F, FK_GELU, (double)P * w * (4.0 + 2.0 + 2.0), 20.0 * P * w);
      k_gelu_bwd<<<gdiv(P * w, 256), 256, 0, F->stream>>>(F->dvf, gp, F->gtab, db[0], P * w, l > 0 ? 0 : 1);
    }
  }
  // lift: v0 = x W_lift + b_lift (db[0]: d v0)
  wgrad(F, F->xin, F->cinp, c.cin, db[0], w, w, g + F->o_Wl, g + F->o_bl);
}

extern "C" {

pf_status pf_fno_create(const pf_fno_config* cfg, void* stream, pf_fno** out) {
  if (!cfg || !out) return PF_ERR_ARG;
  *out = nullptr;
  const pf_fno_config c = *cfg;
  if (c.n < 8 || c.n > 256 || c.n % 8 || c.width < 4 || c.width > 128 || c.width % 4 || c.modes < 2 ||
      c.modes % 2 || 2 * c.modes > c.n || c.layers < 1 || c.layers > 8 || c.hidden < 8 || c.hidden > 128 || c.hidden % 8 ||
      c.cin < 1 || c.cin > 8 || c.cout < 1 || c.cout > 8)
    return PF_ERR_ARG;
  int ndev = 0;  // no usable device: a HIP error, before any allocation
  if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1) return PF_ERR_HIP;
  pf_fno* F = new (std::nothrow) pf_fno();
  if (!F) return PF_ERR_OOM;
  F->cfg = c;
  F->stream = (hipStream_t)stream;
  F->P = (long long)c.n * c.n * c.n;
  for (int i = 0; i < 8; ++i) F->innorm.shift[i] = 0.f, F->innorm.inv[i] = 1.f;
  const int w = c.width, m = c.modes, m2 = 2 * m, h = c.hidden, n = c.n;
  F->mode_count = m2 * m2 * m;
  F->fuse_x = n % 32 == 0;
  F->fuse_proj = w <= 32;
  F->xlines = w <= 64 && m <= 16;
  // parameter layout (same order as the oracle)
  long long off = 0;
  F->o_Wl = off; off += (long long)c.cin * w;
  F->o_bl = off; off += w;
  for (int l = 0; l < c.layers; ++l) {
    F->o_Rr.push_back(off); off += (long long)F->mode_count * w * w;
    F->o_Ri.push_back(off); off += (long long)F->mode_count * w * w;
    F->o_W.push_back(off); off += (long long)w * w;
    F->o_b.push_back(off); off += w;
  }
  F->o_P1 = off; off += (long long)w * h;
  F->o_c1 = off; off += h;
  F->o_P2 = off; off += (long long)h * c.cout;
  F->o_c2 = off; off += c.cout;
  F->nparams = off;
  const long long P = F->P;
  pf_status s = PF_OK;
  auto A = [&](void** p, size_t b) {
    if (s == PF_OK) s = falloc(F, p, b);
  };
  A((void**)&F->th, 4 * off);
  A((void**)&F->gr, 4 * off);
  A((void**)&F->am, 4 * off);
  A((void**)&F->av, 4 * off);
  A((void**)&F->bWliftT, 2 * w * F->cinp);
  F->bWT.resize(c.layers);
  F->bW.resize(c.layers);
  F->bRr.resize(c.layers);
  F->bRi.resize(c.layers);
  for (int l = 0; l < c.layers; ++l) {
    A((void**)&F->bWT[l], 2 * w * w);
    A((void**)&F->bW[l], 2 * w * w);
    A((void**)&F->bRr[l], 2 * (size_t)F->mode_count * w * w);
    A((void**)&F->bRi[l], 2 * (size_t)F->mode_count * w * w);
  }
  A((void**)&F->bP1T, 2 * h * w);
  A((void**)&F->bP1, 2 * w * h);
  A((void**)&F->bP2T, 2 * c.cout * h);
  A((void**)&F->bP2, 2 * h * F->coutp);
  A((void**)&F->scale, 4 * 8);
  A((void**)&F->xin, 2 * P * F->cinp);
  F->v.resize(c.layers + 1);
  F->pre.resize(c.layers);
  F->S.resize(c.layers);
  for (int l = 0; l <= c.layers; ++l) A((void**)&F->v[l], 2 * P * w);
  const size_t spec = (size_t)2 * F->mode_count * w;
  for (int l = 0; l < c.layers; ++l) {
    A((void**)&F->pre[l], 2 * P * w);
    A((void**)&F->S[l], 4 * spec);
  }
  if (!F->fuse_proj) A((void**)&F->hpre, 2 * P * h);
  if (!F->fuse_proj) A((void**)&F->hact, 2 * P * h);
  A((void**)&F->gtab, 4 * 65536);
  const size_t a1 = (size_t)n * n * 2 * m * w, a2 = (size_t)n * 2 * m2 * m * w, b2 = (size_t)n * 2 * n * m * w;
  A((void**)&F->A1, 2 * std::max(a1, b2));
  A((void**)&F->A2, 2 * std::max(a2, (size_t)2 * n * m2 * m * w));
  A((void**)&F->Tb, 2 * spec);
  A((void**)&F->B3, 2 * std::max((size_t)2 * n * m2 * m * w, a2));
  A((void**)&F->B2, 2 * std::max(b2, a1));
  if (!F->fuse_x && !F->xlines) A((void**)&F->B1, 4 * P * w);
  A((void**)&F->outf, 4 * P * c.cout);
  if (!F->fuse_x && !F->xlines) A((void**)&F->dvf, 4 * P * w);
  A((void**)&F->dT, 4 * spec);
  if (!F->fuse_proj) A((void**)&F->dhb, 2 * P * h);
  A((void**)&F->dpreb, 2 * P * w);
  if (F->fuse_x || F->xlines) A((void**)&F->dpreb2, 2 * P * w);
  if (!F->fuse_proj) A((void**)&F->douthb, 2 * P * F->coutp);
  A((void**)&F->dSb, 2 * spec);
  A((void**)&F->part, 4 * pf::part_elems(P, w, h, c.cin, c.cout, F->fuse_proj));
  A((void**)&F->dpart, 8 * pf::dpart_elems(P, F->fuse_proj));
  A((void**)&F->dsum, 8);
  if (s == PF_OK && hipHostMalloc((void**)&F->hsum, 8, 0) != hipSuccess) s = PF_ERR_OOM;
  if (s == PF_OK) {
    std::vector<std::vector<float>> G;
    build_dft(n, m, G);
    const int R[6] = {2 * m, 2 * m2, 2 * m2, n, 2 * n, 2 * n};
    const int K[6] = {n, 2 * n, 2 * n, 2 * m, 2 * m2, 2 * m2};
    u16** dst[6] = {&F->Gxf, &F->Gyf, &F->Gzf, &F->Gxi, &F->Gyi, &F->Gzi};
    u16** dstT[6] = {&F->GxfT, &F->GyfT, &F->GzfT, &F->GxiT, &F->GyiT, &F->GziT};
    for (int i = 0; i < 6 && s == PF_OK; ++i) {
      s = upload_bf16(F, G[i], dst[i]);
      if (s == PF_OK) s = upload_bf16(F, transpose(G[i], R[i], K[i]), dstT[i]);
    }
  }
  if (s == PF_OK) {
    std::vector<float> one(8, 1.0f);
    if (hipMemcpy(F->scale, one.data(), 32, hipMemcpyHostToDevice) != hipSuccess) s = PF_ERR_HIP;
    if (hipMemset(F->th, 0, 4 * off) != hipSuccess || hipMemset(F->gr, 0, 4 * off) != hipSuccess ||
        hipMemset(F->am, 0, 4 * off) != hipSuccess || hipMemset(F->av, 0, 4 * off) != hipSuccess)
      s = PF_ERR_HIP;
  }
  if (s == PF_OK) {
    k_gelu_table<<<256, 256, 0, F->stream>>>(F->gtab);
    if (hipGetLastError() != hipSuccess) s = PF_ERR_HIP;
  }
  if (s != PF_OK) {
    pf_fno_destroy(F);
    return s;
  }
  *out = F;
  return PF_OK;
}

void pf_fno_destroy(pf_fno* F) {
  if (!F) return;
  if (F->stream) hipStreamSynchronize(F->stream);
  for (void* p : F->allocs) hipFree(p);
  for (void* p : F->ballocs) hipFree(p);
  for (void* p : F->eallocs) hipFree(p);
  if (F->hsum) hipHostFree(F->hsum);
  if (F->l2_host) hipHostFree(F->l2_host);
  delete F;
}

int64_t pf_fno_num_params(const pf_fno* F) { return F ? F->nparams : 0; }

pf_status pf_fno_set_params(pf_fno* F, const float* host) {
  if (!F || !host) return PF_ERR_ARG;
  FH(hipMemcpyAsync(F->th, host, 4 * F->nparams, hipMemcpyHostToDevice, F->stream));
  refresh(F);
  FH(hipMemsetAsync(F->am, 0, 4 * F->nparams, F->stream));
  FH(hipMemsetAsync(F->av, 0, 4 * F->nparams, F->stream));
  FH(hipMemsetAsync(F->gr, 0, 4 * F->nparams, F->stream));
  F->adam_t = 0;
  FH(hipStreamSynchronize(F->stream));
  return PF_OK;
}

pf_status pf_fno_get_params(pf_fno* F, float* host) {
  if (!F || !host) return PF_ERR_ARG;
  FH(hipMemcpyAsync(host, F->th, 4 * F->nparams, hipMemcpyDeviceToHost, F->stream));
  FH(hipStreamSynchronize(F->stream));
  return PF_OK;
}

pf_status pf_fno_get_grad(pf_fno* F, float* host) {
  if (!F || !host) return PF_ERR_ARG;
  FH(hipMemcpyAsync(host, F->gr, 4 * F->nparams, hipMemcpyDeviceToHost, F->stream));
  FH(hipStreamSynchronize(F->stream));
  return PF_OK;
}

pf_status pf_fno_load(pf_fno* F, const void* host, size_t bytes) {
  if (!F || !host) return PF_ERR_ARG;
  const size_t np = (size_t)F->nparams;
  if (bytes == 4 * np) return pf_fno_set_params(F, (const float*)host);
  if (bytes != 2 * np) return PF_ERR_ARG;
  // bfloat16 -> float32 is exact (the upper half of the float's bits)
  std::vector<float> w(np);
  const u16* h = (const u16*)host;
  for (size_t i = 0; i < np; ++i) w[i] = bf2f(h[i]);
  return pf_fno_set_params(F, w.data());
}
pf_status pf_fno_train_step(pf_fno* F, const float* x, const float* y, int32_t batch, float lr, float* loss) {
  if (!F || !x || !y || batch < 1 || !(lr > 0.f) || !std::isfinite(lr)) return PF_ERR_ARG;
  pf_status s = pf_fno_zero_grad(F);
  if (s != PF_OK) return s;
  const size_t per = (size_t)F->cfg.cin * (size_t)F->P;
  double tot = 0.0;
  for (int b = 0; b < batch; ++b) {
    double l = 0.0;
    s = pf_fno_grad(F, x + b * per, y + b * per, &l);
    if (s != PF_OK) return s;
    tot += l;
  }
  s = pf_fno_adam_step(F, lr, 0.9f, 0.999f, 1e-8f, 1.0f / (float)batch);
  if (s != PF_OK) return s;
  FH(hipStreamSynchronize(F->stream));
  if (loss) *loss = (float)(tot / batch);
  return PF_OK;
}
pf_status pf_fno_zero_grad(pf_fno* F) {
  if (!F) return PF_ERR_ARG;
  FH(hipMemsetAsync(F->gr, 0, 4 * F->nparams, F->stream));
  return PF_OK;
}

pf_status pf_fno_set_scale(pf_fno* F, const float* host_scale) {
  if (!F || !host_scale) return PF_ERR_ARG;
  FH(hipMemcpyAsync(F->scale, host_scale, 4 * F->cfg.cout, hipMemcpyHostToDevice, F->stream));
  FH(hipStreamSynchronize(F->stream));
  return PF_OK;
}

pf_status pf_fno_set_input_norm(pf_fno* F, const float* shift, const float* scale) {
  if (!F || !shift || !scale) return PF_ERR_ARG;
  for (int c = 0; c < F->cfg.cin; ++c)
    if (!(scale[c] > 0.f) || !std::isfinite(shift[c]) || !std::isfinite(scale[c])) return PF_ERR_ARG;
  for (int c = 0; c < 8; ++c) {
    F->innorm.shift[c] = c < F->cfg.cin ? shift[c] : 0.f;
    F->innorm.inv[c] = c < F->cfg.cin ? 1.f / scale[c] : 1.f;
  }
  return PF_OK;
}

pf_status pf_fno_forward(pf_fno* F, const float* x, float* out) {
  if (!F || !x || !out) return PF_ERR_ARG;
  account(F, FK_ELEM, (double)F->P * (4.0 * F->cfg.cin + 2.0 * F->cinp), 0.0);
  k_pack_input<float><<<gdiv(F->P, 256), 256, 0, F->stream>>>(x, F->P, F->cfg.cin, F->cinp, F->innorm, F->xin);
  forward(F);
  FH(hipMemcpyAsync(out, F->outf, 4 * F->P * F->cfg.cout, hipMemcpyDeviceToDevice, F->stream));
  FH(hipGetLastError());
  FH(hipStreamSynchronize(F->stream));
  return PF_OK;
}

pf_status pf_fno_grad(pf_fno* F, const float* x, const float* y, double* loss) {
  if (!F || !x || !y) return PF_ERR_ARG;
  account(F, FK_ELEM, (double)F->P * (4.0 * F->cfg.cin + 2.0 * F->cinp), 0.0);
  k_pack_input<float><<<gdiv(F->P, 256), 256, 0, F->stream>>>(x, F->P, F->cfg.cin, F->cinp, F->innorm, F->xin);
  forward_layers(F, true);
  loss_backward(F, x, y);
  FH(hipMemcpyAsync(F->hsum, F->dsum, 8, hipMemcpyDeviceToHost, F->stream));
  FH(hipGetLastError());
  FH(hipStreamSynchronize(F->stream));
  if (loss) *loss = F->hsum[0] / ((double)F->P * F->cfg.cout);
  return PF_OK;
}

pf_status pf_fno_adam_step(pf_fno* F, float lr, float beta1, float beta2, float eps, float grad_scale) {
  if (!F) return PF_ERR_ARG;
  F->adam_t += 1;
  const float c1 = 1.f - powf(beta1, (float)F->adam_t), c2 = 1.f - powf(beta2, (float)F->adam_t);
  account(F, FK_ELEM, 7.0 * 4.0 * F->nparams, 0.0);
  k_adam<<<gdiv(F->nparams, 256), 256, 0, F->stream>>>(F->th, F->am, F->av, F->gr, F->nparams, lr, beta1, beta2,
                                                       eps, grad_scale, c1, c2);
  refresh(F);
  FH(hipGetLastError());
  return PF_OK;
}

static constexpr int kL2Blocks = 512;
// pf_rel_l2_noalloc: devices it keeps a scratch address for, and the largest
// count it takes (the per-thread partial sums of 512 x 256 threads then add at
// most 2^24 squares each)
static constexpr int kMaxDevices = 64;
static constexpr int64_t kNoallocMaxN = (int64_t)1 << 41;

// ||a - b|| / ||b|| with caller-provided partials (device) and staging (pinned host)
static pf_status rel_l2_impl(hipStream_t s, const double* a, const double* b, long long n, double* part,
                             double* host, double* out) {
  k_rel_l2<<<kL2Blocks, 256, 0, s>>>(a, b, n, part);
  FH(hipGetLastError());
  FH(hipMemcpyAsync(host, part, sizeof(double) * 2 * kL2Blocks, hipMemcpyDeviceToHost, s));
  FH(hipStreamSynchronize(s));
  double d2 = 0.0, b2 = 0.0;
  for (int i = 0; i < kL2Blocks; ++i) {
    d2 += host[2 * i];
    b2 += host[2 * i + 1];
  }
  *out = b2 > 0.0 ? std::sqrt(d2 / b2) : std::sqrt(d2);
  return PF_OK;
}

// ---- allocation-free relative L2 ------------------------------------------------
// The partial sums of pf_rel_l2_noalloc live in a file-scope device array (one
// copy per GPU, held until the process ends).  In host code `scratch` names a
// host-side stand-in, not device memory: the array is only ever reached
// through the address hipGetSymbolAddress returns for the current device,
// looked up once per device on the entry point's first call there.
static __device__ __align__(256) double scratch[2 * kL2Blocks];
static std::mutex g_scratch_mu;
static double* g_scratch_ptr[kMaxDevices] = {nullptr};

static pf_status scratch_for_current_device(double** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return PF_ERR_HIP;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return PF_ERR_HIP;
    g_scratch_ptr[dev] = (double*)p;
  }
  *out = g_scratch_ptr[dev];
  return PF_OK;
}

pf_status pf_rel_l2_noalloc(const double* a, const double* b, int64_t n, void* stream, double* out) {
  if (!a || !b || n < 1 || !out) return PF_ERR_ARG;
  if (n > kNoallocMaxN) return PF_ERR_ARG;
  double* part = nullptr;
  pf_status st = scratch_for_current_device(&part);
  if (st != PF_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  // the same kernel and host-side summation order as pf_rel_l2; the host copy of
  // the partials is a stack array (no pinned or device allocation)
  double host[2 * kL2Blocks];
  k_rel_l2<<<kL2Blocks, 256, 0, s>>>(a, b, n, part);
  FH(hipGetLastError());
  FH(hipMemcpyAsync(host, part, sizeof(host), hipMemcpyDeviceToHost, s));
  FH(hipStreamSynchronize(s));
  double d2 = 0.0, b2 = 0.0;
  for (int i = 0; i < kL2Blocks; ++i) {
    d2 += host[2 * i];
    b2 += host[2 * i + 1];
  }
  *out = b2 > 0.0 ? std::sqrt(d2 / b2) : std::sqrt(d2);
  return PF_OK;
}

pf_status pf_rel_l2(const double* a, const double* b, int64_t n, void* stream, double* out) {
  if (!a || !b || n < 1 || !out) return PF_ERR_ARG;
  double* part = nullptr;
  double* host = nullptr;
  if (hipMalloc((void**)&part, sizeof(double) * 2 * kL2Blocks) != hipSuccess) return PF_ERR_OOM;
  if (hipHostMalloc((void**)&host, sizeof(double) * 2 * kL2Blocks, 0) != hipSuccess) {
    hipFree(part);
    return PF_ERR_OOM;
  }
  pf_status st = rel_l2_impl((hipStream_t)stream, a, b, n, part, host, out);
  hipStreamSynchronize((hipStream_t)stream);
  hipHostFree(host);
  hipFree(part);
  return st;
}

}  // extern "C"

// ---- batched inference ---------------------------------------------------------
static pf_status grow(std::vector<void*>& list, void** p, size_t bytes) {
  if (hipMalloc(p, bytes) != hipSuccess) {
    *p = nullptr;
    return PF_ERR_OOM;
  }
  list.push_back(*p);
  return PF_OK;
}

// Inference buffers for B samples (the forward pass's activations, B times;
// no pre-activations or gradients are kept).
static pf_status ensure_batch(pf_fno* F, int B) {
  if (B <= F->bcap) return PF_OK;
  hipStreamSynchronize(F->stream);
  for (void* p : F->ballocs) hipFree(p);
  F->ballocs.clear();
  F->bcap = 0;
  const pf_fno_config& c = F->cfg;
  const size_t w = c.width, m = c.modes, m2 = 2 * m, h = c.hidden, n = c.n, P = (size_t)F->P, Bs = (size_t)B;
  const size_t Nz = m2 * m * w, spec = 2 * (size_t)F->mode_count * w;
  const size_t a1 = std::max(n * n * 2 * m * w, n * 2 * n * m * w);
  pf_status s = PF_OK;
  auto A = [&](void** p, size_t bytes) {
    if (s == PF_OK) s = grow(F->ballocs, p, bytes);
  };
  A((void**)&F->bxin, Bs * 2 * P * F->cinp);
  A((void**)&F->bv0, Bs * 2 * P * w);
  A((void**)&F->bv1, Bs * 2 * P * w);
  A((void**)&F->bA1, Bs * 2 * a1);
  A((void**)&F->bA2, Bs * 2 * 2 * n * Nz);
  A((void**)&F->bS, Bs * 4 * spec);
  A((void**)&F->bTb, Bs * 2 * spec);
  A((void**)&F->bB3, Bs * 2 * 2 * n * Nz);
  A((void**)&F->bB2, Bs * 2 * a1);
  if (!F->fuse_x && !F->xlines) A((void**)&F->bB1, Bs * 4 * P * w);
  if (!F->fuse_proj) A((void**)&F->bhact, Bs * 2 * P * h);
  A((void**)&F->boutf, Bs * 4 * P * c.cout);
  A((void**)&F->bdpart, Bs * 8 * pf::pointwise_blocks(F->P));
  A((void**)&F->bdsum, Bs * 8);
  if (s != PF_OK) {
    for (void* p : F->ballocs) hipFree(p);
    F->ballocs.clear();
    return s;
  }
  F->bcap = B;
  return PF_OK;
}

static void cm_points(pf_fno* F, long long points, const u16* In, int ldin, int K, const u16* Bt, int N,
                      const float* bias, const float* resid, int ldres, float* outf, u16* outpre, u16* outact,
                      int ldout, const LineTerm& lt = LineTerm()) {
  cm_launch(F, points, In, ldin, K, Bt, N, bias, resid, ldres, outf, outpre, outact, ldout, lt);
}

// The forward pass of B samples at once (inputs packed in bxin, outputs in
// boutf): every channel-mixing GEMM runs over the B n^3 points together and
// every truncated-DFT stage takes the B samples' lines as more batches of the
// same small GEMM, so the sums are those of the one-sample pass.
static void forward_batch(pf_fno* F, int B) {
  const pf_fno_config& c = F->cfg;
  const int w = c.width, h = c.hidden, L = c.layers;
  const long long PB = F->P * B;
  const float* th = F->th;
  const FwdBufs u = {F->bxin, F->bA1, F->bA2, F->bTb, F->bB3, F->bB2, F->bB1};
  u16* vb[2] = {F->bv0, F->bv1};
  forward_layers(
      F, u, B, [&](int l) { return vb[l & 1]; }, [&](int l) { return l == L - 1 ? vb[(l + 1) & 1] : (u16*)nullptr; },
      [&](int) { return F->bS; });
  const u16* v = vb[L & 1];
  if (F->fuse_proj) {
    project(F, v, PB, F->boutf);
    return;
  }
  cm_points(F, PB, v, w, w, F->bP1T, h, th + F->o_c1, nullptr, 0, nullptr, nullptr, F->bhact, h);
  cm_points(F, PB, F->bhact, h, h, F->bP2T, c.cout, th + F->o_c2, nullptr, 0, F->boutf, nullptr, nullptr, c.cout);
}

// next_b = state_b + scale * net(state_b), mean of c restored, for b < B
// (states / nexts: [B][cin][n^3] float64; next may equal state).
static pf_status apply_batch(pf_fno* F, const double* states, double* nexts, int B) {
  pf_status s = ensure_batch(F, B);
  if (s != PF_OK) return s;
  const long long P = F->P;
  const int ci = F->cfg.cin, co = F->cfg.cout;
  const unsigned nb = pf::pointwise_blocks(P);
  for (int b = 0; b < B; ++b) {
    account(F, FK_ELEM, (double)P * (8.0 * ci + 2.0 * F->cinp), 0.0);
    k_pack_input<double><<<nb, 256, 0, F->stream>>>(states + (long long)b * ci * P, P, ci, F->cinp, F->innorm,
                                                    F->bxin + (long long)b * P * F->cinp);
  }
  forward_batch(F, B);
  for (int b = 0; b < B; ++b) {
    double* nx = nexts + (long long)b * co * P;
    account(F, FK_ELEM, (double)P * co * (8.0 + 4.0 + 8.0), 0.0);
    k_apply<<<nb, 256, 0, F->stream>>>(states + (long long)b * ci * P, F->boutf + (long long)b * P * co, F->scale, P,
                                       co, nx, F->bdpart + (long long)b * nb);
    k_sum_d<<<1, 256, 0, F->stream>>>(F->bdpart + (long long)b * nb, (int)nb, F->bdsum + b);
    account(F, FK_ELEM, (double)P * 16.0, 0.0);
    k_shift<<<nb, 256, 0, F->stream>>>(nx, P, F->bdsum + b);
  }
  FH(hipGetLastError());
  FH(hipStreamSynchronize(F->stream));
  return PF_OK;
}

extern "C" {

pf_status pf_fno_work(pf_fno* F, int32_t enable, double* bytes, double* flops, int64_t* launches, int32_t kinds) {
  if (!F || kinds < 0 || (kinds > 0 && (!bytes || !flops || !launches))) return PF_ERR_ARG;
  for (int k = 0; k < kinds && k < FK_COUNT; ++k) {
    bytes[k] = F->acct_bytes[k];
    flops[k] = F->acct_flops[k];
    launches[k] = F->acct_n[k];
  }
  for (int k = FK_COUNT; k < kinds; ++k) {
    bytes[k] = flops[k] = 0.0;
    launches[k] = 0;
  }
  if (enable >= 0) {
    F->acct = enable ? 1 : 0;
    for (int k = 0; k < FK_COUNT; ++k) {
      F->acct_bytes[k] = F->acct_flops[k] = 0.0;
      F->acct_n[k] = 0;
    }
  }
  return PF_OK;
}

pf_status pf_fno_apply_batch(pf_fno* F, const double* states, double* nexts, int32_t batch) {
  if (!F || !states || !nexts || batch < 1 || F->cfg.cin != F->cfg.cout) return PF_ERR_ARG;
  return apply_batch(F, states, nexts, batch);
}

pf_status pf_fno_apply(pf_fno* F, const double* state, double* next) {
  if (!F || !state || !next || F->cfg.cin != F->cfg.cout) return PF_ERR_ARG;
  account(F, FK_ELEM, (double)F->P * (8.0 * F->cfg.cin + 2.0 * F->cinp), 0.0);
  k_pack_input<double><<<gdiv(F->P, 256), 256, 0, F->stream>>>(state, F->P, F->cfg.cin, F->cinp, F->innorm, F->xin);
  forward(F);
  const unsigned nb = pf::pointwise_blocks(F->P);
  account(F, FK_ELEM, (double)F->P * F->cfg.cout * (8.0 + 4.0 + 8.0), 0.0);
  k_apply<<<nb, 256, 0, F->stream>>>(state, F->outf, F->scale, F->P, F->cfg.cout, next, F->dpart);
  k_sum_d<<<1, 256, 0, F->stream>>>(F->dpart, (int)nb, F->dsum);
  account(F, FK_ELEM, (double)F->P * 16.0, 0.0);
  k_shift<<<nb, 256, 0, F->stream>>>(next, F->P, F->dsum);
  FH(hipGetLastError());
  FH(hipStreamSynchronize(F->stream));
  return PF_OK;
}

// one plain-solver interval: out = plain(state) over [0, delta]
static pf_status plain_interval(pf_ctx* plain, const double* in, double* out, long long P, double delta) {
  pf_status s = pf_set_state(plain, in, in + P, 1, 0.0);
  if (s != PF_OK) return s;
  s = pf_advance(plain, delta, nullptr);
  if (s != PF_OK) return s;
  return pf_get_state(plain, out, out + P, 1);
}

pf_status pf_fno_advance(pf_fno* F, pf_ctx* plain, double* state, int32_t n_adv, double delta,
                         int32_t check_every, double tol, pf_fno_stats* st) {
  if (!F || !plain || !state || !st || n_adv < 0 || !(delta > 0.0) || check_every < 1 || !(tol >= 0.0) ||
      F->cfg.cin != 4 || F->cfg.cout != 4)
    return PF_ERR_ARG;
  const long long P = F->P;
  const size_t bytes = sizeof(double) * 4 * P;
  if (!F->adv_next) {
    pf_status s = falloc(F, (void**)&F->adv_next, bytes);
    if (s == PF_OK) s = falloc(F, (void**)&F->adv_ref, bytes);
    if (s == PF_OK) s = falloc(F, (void**)&F->l2_part, sizeof(double) * 2 * kL2Blocks);
    if (s == PF_OK && hipHostMalloc((void**)&F->l2_host, sizeof(double) * 2 * kL2Blocks, 0) != hipSuccess)
      s = PF_ERR_OOM;
    if (s != PF_OK) return s;
  }
  using clk = std::chrono::steady_clock;
  auto ms_since = [](clk::time_point t0) {
    return std::chrono::duration<double, std::milli>(clk::now() - t0).count();
  };
  for (int32_t a = 0; a < n_adv; ++a) {
    if (st->plain_left > 0) {
      const auto t0 = clk::now();
      pf_status s = plain_interval(plain, state, state, P, delta);
      st->ms_plain += ms_since(t0);
      if (s != PF_OK) return s;
      st->plain += 1;
      st->plain_left -= 1;
      continue;
    }
    const bool check = st->since_check + 1 >= check_every;
    auto t0 = clk::now();
    pf_status s = pf_fno_apply(F, state, check ? F->adv_next : state);
    st->ms_surrogate += ms_since(t0);
    if (s != PF_OK) return s;
    st->surrogate += 1;
    st->since_check += 1;
    if (!check) continue;
    st->since_check = 0;
    st->checks += 1;
    t0 = clk::now();
    s = plain_interval(plain, state, F->adv_ref, P, delta);
    double err = 0.0;
    if (s == PF_OK) s = rel_l2_impl(F->stream, F->adv_next, F->adv_ref, P, F->l2_part, F->l2_host, &err);
    if (s != PF_OK) return s;
    st->err_last = err;
    if (!(err <= st->err_max)) st->err_max = err;
    const bool fail = !(err <= tol);
    if (fail) {
      st->fallbacks += 1;
      st->plain_left = check_every;
    }
    FH(hipMemcpyAsync(state, fail ? F->adv_ref : F->adv_next, bytes, hipMemcpyDeviceToDevice, F->stream));
    FH(hipStreamSynchronize(F->stream));
    st->ms_plain += ms_since(t0);
  }
  return PF_OK;
}

pf_status pf_fno_ensemble_advance(pf_fno* F, pf_ens* E, const int32_t* members, int32_t count, int32_t n_adv,
                                  double delta, int32_t check_every, double tol, pf_fno_stats* st) {
  if (!F || !E || !members || !st || count < 1 || n_adv < 0 || !(delta > 0.0) || check_every < 1 || !(tol >= 0.0) ||
      F->cfg.cin != 4 || F->cfg.cout != 4)
    return PF_ERR_ARG;
  const int M = pf::ens_members(E);
  for (int i = 0; i < count; ++i) {
    if (members[i] < 0 || members[i] >= M || pf::ens_member_n(E, members[i]) != F->cfg.n) return PF_ERR_ARG;
    for (int j = 0; j < i; ++j)
      if (members[j] == members[i]) return PF_ERR_ARG;
  }
  const long long P = F->P;
  const size_t per = 4 * (size_t)P;
  if (count > F->ecap) {
    hipStreamSynchronize(F->stream);
    for (void* p : F->eallocs) hipFree(p);
    F->eallocs.clear();
    F->ecap = 0;
    pf_status s = grow(F->eallocs, (void**)&F->eX, sizeof(double) * per * count);
    if (s == PF_OK) s = grow(F->eallocs, (void**)&F->eY, sizeof(double) * per * count);
    if (s == PF_OK) s = grow(F->eallocs, (void**)&F->eP, sizeof(double) * per * count);
    if (s != PF_OK) return s;
    F->ecap = count;
  }
  if (!F->l2_part) {
    pf_status s = falloc(F, (void**)&F->l2_part, sizeof(double) * 2 * kL2Blocks);
    if (s == PF_OK && hipHostMalloc((void**)&F->l2_host, sizeof(double) * 2 * kL2Blocks, 0) != hipSuccess)
      s = PF_ERR_OOM;
    if (s != PF_OK) return s;
  }
  using clk = std::chrono::steady_clock;
  auto ms_since = [](clk::time_point t0) {
    return std::chrono::duration<double, std::milli>(clk::now() - t0).count();
  };
  hipStream_t es = pf::ens_stream(E);
  std::vector<double> t0(count), tf(M);
  for (int i = 0; i < count; ++i) {
    t0[i] = pf::ens_member_time(E, members[i]);
    pf_status s = pf_ensemble_get_state(E, members[i], F->eX + i * per, F->eX + i * per + P, 1);
    if (s != PF_OK) return s;
  }
  double ms_net = 0.0, ms_plain = 0.0;
  std::vector<char> due(count), plainm(count);
  for (int32_t a = 0; a < n_adv; ++a) {
    bool any_net = false, any_plain = false;
    for (int i = 0; i < count; ++i) {
      plainm[i] = st[i].plain_left > 0;
      due[i] = !plainm[i] && st[i].since_check + 1 >= check_every;
      any_net = any_net || !plainm[i];
      any_plain = any_plain || plainm[i] || due[i];
    }
    auto t1 = clk::now();
    if (any_net) {  // every member through the network in one batched pass
      pf_status s = apply_batch(F, F->eX, F->eY, count);
      if (s != PF_OK) return s;
    }
    ms_net += ms_since(t1);
    t1 = clk::now();
    if (any_plain) {  // the checks and the plain intervals: one ensemble advance
      for (int m = 0; m < M; ++m) tf[m] = pf::ens_member_time(E, m);
      for (int i = 0; i < count; ++i) {
        if (!(plainm[i] || due[i])) continue;
        pf_status s = pf::ens_member_set(E, members[i], F->eX + i * per, 0.0);
        if (s != PF_OK) return s;
        tf[members[i]] = delta;
      }
      pf_status s = pf_ensemble_advance(E, tf.data(), 1 << 30, nullptr);
      if (s != PF_OK) return s;
      for (int i = 0; i < count; ++i) {
        if (!(plainm[i] || due[i])) continue;
        s = pf_ensemble_get_state(E, members[i], F->eP + i * per, F->eP + i * per + P, 1);
        if (s != PF_OK) return s;
      }
      FH(hipStreamSynchronize(es));
    }
    for (int i = 0; i < count; ++i) {
      pf_fno_stats& x = st[i];
      const double* src;
      if (plainm[i]) {
        x.plain += 1;
        x.plain_left -= 1;
        src = F->eP + i * per;
      } else {
        x.surrogate += 1;
        x.since_check += 1;
        src = F->eY + i * per;
        if (due[i]) {
          x.since_check = 0;
          x.checks += 1;
          double err = 0.0;
          pf_status s = rel_l2_impl(F->stream, F->eY + i * per, F->eP + i * per, P, F->l2_part, F->l2_host, &err);
          if (s != PF_OK) return s;
          x.err_last = err;
          if (!(err <= x.err_max)) x.err_max = err;
          if (!(err <= tol)) {
            x.fallbacks += 1;
            x.plain_left = check_every;
            src = F->eP + i * per;
          }
        }
      }
      FH(hipMemcpyAsync(F->eX + i * per, src, sizeof(double) * per, hipMemcpyDeviceToDevice, F->stream));
    }
    FH(hipStreamSynchronize(F->stream));
    ms_plain += ms_since(t1);
  }
  for (int i = 0; i < count; ++i) {
    pf_status s = pf::ens_member_set(E, members[i], F->eX + i * per, t0[i] + n_adv * delta);
    if (s != PF_OK) return s;
    st[i].ms_surrogate += ms_net;
    st[i].ms_plain += ms_plain;
  }
  FH(hipStreamSynchronize(es));
  return PF_OK;
}

}  // extern "C"
