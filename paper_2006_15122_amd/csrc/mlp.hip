// Spectrum surrogate: 2 -> 256 -> 256 -> 256 -> 64 perceptron with GELU,
// trained and evaluated on the matrix cores.
//
// Every product is C[M][N] = A[M][K] Bt[N][K]^T with BF16 operands stored
// K-contiguous and FP32 accumulation (v_mfma_f32_16x16x32_bf16):
//   forward          a_l   = h_{l-1} W_l^T            (A = h_{l-1},  Bt = W_l)
//   input gradient   dh    = da_l W_l                 (A = da_l,     Bt = W_l^T)
//   weight gradient  gW_l  = da_l^T h_{l-1}           (A = da_l^T,   Bt = h_{l-1}^T)
// A training step is two kernels.  The first takes 16 batch rows per block
// through the forward pass, the loss and the input-gradient chain with the
// activations in LDS (all of that is local to a row), and writes BF16 copies
// of h_l and da_l in blocks of 16 batch rows, each unit's 16 values together.
// The second computes the weight gradients (KSPLIT rows per split, the splits
// of a tile in the waves of one block), sums every partial (splits, bias
// columns, loss) in a fixed order and applies Adam, so a training step is
// deterministic.
//
// Operand layout of one 16x16x32 product on a 64-lane wave (verified on the
// device): lane l holds A[l%16][8(l/16) .. 8(l/16)+7] and
// Bt[l%16][8(l/16) .. 8(l/16)+7] (8 BF16 each) and receives
// C[4(l/16) + e][l%16], e = 0..3.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "common.hpp"
#include "../../include/surrogate.h"

using namespace cl;

struct surrogate_t;

namespace {

constexpr int NIN = SURR_N_IN, WID = SURR_WIDTH, NOUT = SURR_N_OUT, NPAR = SURR_NPARAMS;
constexpr int NFQ0 = SURR_N_FREQ0, NFQ1 = SURR_N_FREQ1, NFEAT = SURR_N_FEAT;
static_assert(NFEAT == NIN + 2 * (NFQ0 + NFQ1), "feature count");
// offsets of the tensors in the flat parameter vector
constexpr int OW1 = 0, OB1 = OW1 + WID * NFEAT, OW2 = OB1 + WID, OB2 = OW2 + WID * WID, OW3 = OB2 + WID,
              OB3 = OW3 + WID * WID, OW4 = OB3 + WID, OB4 = OW4 + NOUT * WID;
static_assert(OB4 + NOUT == NPAR, "parameter count");

constexpr int KSPLIT = 256;      // batch rows per split of a weight-gradient product
constexpr int MAX_BATCH = 16384;
constexpr int MAX_STEPS = 65536;
constexpr int LDH = WID + 8;     // LDS row pitch of the fused forward (BF16), 16 B skew per row

typedef uint16_t bf16_t;
typedef __bf16 bf16x8 __attribute__((__vector_size__(8 * sizeof(__bf16))));
typedef float f4 __attribute__((__vector_size__(4 * sizeof(float))));
typedef f4 f4_any __attribute__((aligned(4)));  // at any FP32 address

// FP32 -> BF16, round to nearest, ties to even (one v_cvt_pk_bf16_f32 for two)
__device__ __forceinline__ bf16_t to_bf16(float f) { return __builtin_bit_cast(bf16_t, (__bf16)f); }
typedef __bf16 bf16x2 __attribute__((__vector_size__(2 * sizeof(__bf16))));
__device__ __forceinline__ uint32_t to_bf16x2(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, bf16x2{(__bf16)lo, (__bf16)hi});
}
__device__ __forceinline__ float from_bf16(bf16_t b) { return __uint_as_float((uint32_t)b << 16); }

// erfc(z) for z >= 0 by the Chebyshev fit of Press et al., Numerical Recipes
// (Sec. 6.2, erfcc): t exp(-z^2 + P(t)) with t = 1 / (1 + z/2), fractional
// error below 1.2e-7 in exact arithmetic (about 1e-6 in FP32 for z < 9).
__device__ __forceinline__ float erfc_pos(float z) {
  const float t = __builtin_amdgcn_rcpf(fmaf(0.5f, z, 1.0f));
  float p = 0.17087277f;
  p = fmaf(p, t, -0.82215223f);
  p = fmaf(p, t, 1.48851587f);
  p = fmaf(p, t, -1.13520398f);
  p = fmaf(p, t, 0.27886807f);
  p = fmaf(p, t, -0.18628806f);
  p = fmaf(p, t, 0.09678418f);
  p = fmaf(p, t, 0.37409196f);
  p = fmaf(p, t, 1.00002368f);
  return t * __expf(fmaf(t, p, fmaf(-z, z, -1.26551223f)));
}
// 1 + erf(z): 2 - erfc(z) for z >= 0 and erfc(-z) below, so that the left
// tail keeps its relative precision (1 + erf(z) cancels there), which is what
// the BF16 rounding of the activation sees.
__device__ __forceinline__ float one_plus_erf(float z) {
  const float ec = erfc_pos(fabsf(z));
  return z >= 0.0f ? 2.0f - ec : ec;
}
// GELU(a) = a Phi(a) = a (1 + erf(a / sqrt 2)) / 2 and its derivative
// Phi(a) + a exp(-a^2/2) / sqrt(2 pi)
__device__ __forceinline__ float gelu(float a) { return 0.5f * a * one_plus_erf(a * 0.70710678118654752f); }
__device__ __forceinline__ float gelu_grad(float a) {
  return 0.5f * one_plus_erf(a * 0.70710678118654752f) + a * 0.39894228040143268f * __expf(-0.5f * a * a);
}

__device__ __forceinline__ bf16x8 load8(const bf16_t* p) {
  return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(p));
}
__device__ __forceinline__ f4 mma(bf16x8 a, bf16x8 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// BF16 weight copies lie as the products read them: a wave's fragment of 16
// outputs and 32 inputs is 1 KB on end (lane l's eight values at 8 l), the
// fragments of 16 outputs follow each other.  Place of output o, input i of K.
// (In rows of K a fragment is sixteen 64-byte pieces, half a cache line each: a
// block that reads a hidden layer's 128 KB waited 3.2 us for it.)
constexpr int FRAG = 512;
__device__ __forceinline__ int wpos(int o, int i, int K) {
  return (o / 16 * (K / 32) + i / 32) * FRAG + ((i % 32) / 8 * 16 + o % 16) * 8 + i % 8;
}

// normalisation constants on the device
struct Norm {
  float in_shift[NIN], in_scale[NIN], out_shift[NOUT], out_scale[NOUT], enc_freq[NIN];
};

// The first layer's inputs of a raw row (x0, x1): the normalised inputs u_c,
// then sin and cos of 2^k enc_freq[c] u_c for the octaves of input 0, then
// those of input 1.  One call gives one octave o (0 .. NOCT - 1) of a row; the
// call with o = 0 also stores u_0, that with o = NFQ0 u_1.  The angle is held as
// an FP32 number p and its rounding error e: the octave scales both exactly, and
// the first-order term 2^k e keeps the high octaves as accurate as the low ones
// (the rounding of the angle would otherwise grow with 2^k).
constexpr int NOCT = NFQ0 + NFQ1;
__device__ __forceinline__ void feature(const float* X, int o, const Norm* nm, float* f) {
  const int c = o < NFQ0 ? 0 : 1, k = c ? o - NFQ0 : o;
  const float u = (X[c] - nm->in_shift[c]) * nm->in_scale[c], fr = nm->enc_freq[c];
  const float p = fr * u, q = (float)(1 << k);
  const float e = fmaf(fr, u, -p) * q;
  float sn, cs;
  sincosf(p * q, &sn, &cs);
  if (k == 0) f[c] = u;
  f[NIN + 2 * o] = fmaf(e, cs, sn);
  f[NIN + 2 * o + 1] = fmaf(-e, sn, cs);
}
// the features of NR rows (row r at X + 2 src(r), padding rows past nvalid zero)
// by a block of NT threads, one octave of one row per thread and turn: a row's
// 11 octaves on one thread were a chain of 22 library calls, 8 us
template <int NR, int NT, typename Src>
__device__ __forceinline__ void block_features(const float* X, const Norm* nm, int t, Src src, float (*xs)[NFEAT]) {
  static_assert(NT % NR == 0 && NIN == 2, "whole rows per turn");
  const int r = t % NR;
  const int64_t i = src(r);
  for (int o = t / NR; o < NOCT; o += NT / NR) {
    if (i >= 0) {
      feature(X + 2 * i, o, nm, xs[r]);
    } else {
      if (o == 0 || o == NFQ0) xs[r][o ? 1 : 0] = 0.0f;
      xs[r][NIN + 2 * o] = xs[r][NIN + 2 * o + 1] = 0.0f;
    }
  }
}

// ---------------------------------------------------------------------------
// training step, part 1: everything that is local to a batch row.  One block
// takes RB = 16 rows through the forward pass, the loss and the backward pass
// down to the input layer; the 16 x 256 activations and gradients stay in
// LDS between layers.  Sixteen waves; wave w owns hidden units 16w .. 16w+15
// (waves 0-3 also output units 16w .. 16w+15), so the pre-activations that
// GELU'(a_l) needs on the way down stay in the registers of the thread that
// formed them.  It writes what the
// weight-gradient products need (h_l, da_l, BF16) and per-block partial
// sums of the bias gradients, of the first layer's weight gradient and of the
// loss.
//
// Bound by latency (one block a CU at a batch of 2048 rows, each layer waits for
// the one before): each layer's weights are requested while the previous layer's
// activations are formed.  2048 rows: 19 us, 16384 rows 63 us; with row-major
// weights requested in place 29 and 103.
// ---------------------------------------------------------------------------
constexpr int RB = 16;          // batch rows per block of the fused step kernel
constexpr int LDY = NOUT + 8;   // LDS pitch of dL/dy (BF16)

struct RowArgs {
  const float* X;        // raw inputs [*][2], rows selected by `rows` (or the first n)
  const float* T;        // raw targets [*][NOUT]
  const int32_t* rows;
  int nvalid;            // rows >= nvalid are padding (zero gradient)
  float dscale;          // 2 / (nvalid * NOUT)
  const Norm* nm;
  const bf16_t *W1b, *W2b, *W3b, *W4b, *W2t, *W3t, *W4t;
  const float *b1, *b2, *b3, *b4;
  bf16_t *H1t, *H2t, *H3t;          // BF16 h_l, [R][WID][RB]
  bf16_t *DYt, *D3t, *D2t;          // BF16 dL/dy [R][NOUT][RB], dL/da_l [R][WID][RB]
  float *bp1, *bp2, *bp3, *bp4;     // per-block bias-gradient columns [R][width]
  float* w1p;                       // per-block first-layer weight gradient [R][NFEAT][WID]
  double* lpart;                    // per-block sum of squared residuals [R]
};

// sum over the block's 16 rows of per-lane column values (lanes l, l^16, l^32,
// l^48 share a column; every one of them returns the column sum).  The lane
// swaps are vector instructions, where a shuffle is a trip through LDS.
typedef uint32_t u32x2 __attribute__((__vector_size__(2 * sizeof(uint32_t))));
__device__ __forceinline__ float col_sum16(float v) {
  const u32x2 a = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false));
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const u32x2 b = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false));
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// one 16 x 16 tile of C = A Bt^T, K = 32 NK: A is the block's 16 rows in LDS
// (pitch lda), Bt the fragments of the wave's 16 columns, which it has requested
// before (while the previous layer's activations were formed)
constexpr int CT = 1;  // 16-column tiles per wave
template <int NK>
struct Weights {
  bf16x8 b[NK];
  __device__ __forceinline__ Weights() {}
  __device__ __forceinline__ Weights(const bf16_t* __restrict__ W, int tile, int lane) { request(W, tile, lane); }
  __device__ __forceinline__ void request(const bf16_t* __restrict__ W, int tile, int lane) {
    const bf16_t* p = W + (size_t)tile * NK * FRAG + 8 * lane;
#pragma unroll
    for (int s = 0; s < NK; ++s) b[s] = load8(p + FRAG * s);
  }
  __device__ __forceinline__ f4 times(const bf16_t* As, int lda, int lane) const {
    const int r16 = lane & 15, kq = (lane >> 4) * 8;
    f4 acc = f4{0.0f, 0.0f, 0.0f, 0.0f};
    bf16x8 a[NK];
#pragma unroll
    for (int s = 0; s < NK; ++s) a[s] = load8(As + r16 * lda + 32 * s + kq);
#pragma unroll
    for (int s = 0; s < NK; ++s) acc = mma(a[s], b[s], acc);
    return acc;
  }
};

// four rows i0 .. i0+3 of unit j into a block's [units][RB] copy
__device__ __forceinline__ void store_t4(bf16_t* Ht, int j, int i0, const float (&v)[4]) {
  *reinterpret_cast<uint2*>(Ht + j * RB + i0) = uint2{to_bf16x2(v[0], v[1]), to_bf16x2(v[2], v[3])};
}

constexpr int NWAVE = WID / (16 * CT);       // 16
static_assert(RB * WID == 4 * 64 * NWAVE && CT == 1, "four rows of one unit per thread");

__global__ __launch_bounds__(64 * NWAVE) void step_rows_kernel(RowArgs g) {
  __shared__ __align__(16) bf16_t HA[RB * LDH];
  __shared__ __align__(16) bf16_t HB[RB * LDH];
  __shared__ __align__(16) bf16_t DY[RB * LDY];
  __shared__ __align__(16) float xs[RB][NFEAT];
  __shared__ double lred[4];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int rq = (lane >> 4) * 4;  // first of this lane's 4 rows in a 16-row tile
  const int rb = blockIdx.x, r0 = rb * RB;
  const int j = 16 * w + (lane & 15);  // this lane's unit
  auto row_of = [&](int r) -> int64_t {
    const int i = r0 + r;
    return i < g.nvalid ? (g.rows ? (int64_t)g.rows[i] : (int64_t)i) : -1;
  };
  auto blk = [&](bf16_t* p, int width) { return p + (size_t)rb * width * RB; };

  constexpr int KH = WID / 32, KO = NOUT / 32;
  // requested ahead of their use: the first two layers' weights and, behind the
  // features' inputs (loads return in order), the targets
  const Weights<KH> w2(g.W2b, w, lane);
  bf16x8 w1[NFEAT / 8];
#pragma unroll
  for (int c = 0; c < NFEAT / 8; ++c) w1[c] = load8(g.W1b + NFEAT * j + 8 * c);
  const float bj1 = g.b1[j];
  block_features<RB, 64 * NWAVE>(g.X, g.nm, t, row_of, xs);
  float tv[4];
  if (w < NOUT / 16) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int64_t src = row_of(rq + e);
      tv[e] = src >= 0 ? g.T[src * NOUT + j] : 0.0f;
    }
  }
  __syncthreads();
  // layer 1 (K = NFEAT, plain FMA); padding rows (past nvalid) have zero features
  float a1[4], a2[4], a3[4];
  {
    float wf[NFEAT], hv[4];
#pragma unroll
    for (int c = 0; c < NFEAT; ++c) wf[c] = (float)w1[c / 8][c % 8];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float a = bj1;
#pragma unroll
      for (int c = 0; c < NFEAT; ++c) a = fmaf(xs[rq + e][c], wf[c], a);
      a1[e] = a;
      hv[e] = gelu(a);
      HA[(rq + e) * LDH + j] = to_bf16(hv[e]);
    }
    store_t4(blk(g.H1t, WID), j, rq, hv);
  }
  __syncthreads();

  // hidden layers 2 and 3: a = h W^T + b, h' = BF16(GELU(a))
  auto hidden = [&](const f4& acc, bf16_t* dst, float bj, bf16_t* Ht, float (&av)[4]) {
    float hv[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      av[e] = acc[e] + bj;
      hv[e] = gelu(av[e]);
      dst[(rq + e) * LDH + j] = to_bf16(hv[e]);
    }
    store_t4(blk(Ht, WID), j, rq, hv);
    __syncthreads();
  };
  const float b2 = g.b2[j], b3 = g.b3[j];
  f4 acc = w2.times(HA, LDH, lane);
  const Weights<KH> w3(g.W3b, w, lane);
  hidden(acc, HB, b2, g.H2t, a2);
  acc = w3.times(HB, LDH, lane);
  Weights<KH> w4;
  if (w < NOUT / 16) w4.request(g.W4b, w, lane);
  const Weights<KO> w4t(g.W4t, w, lane);
  hidden(acc, HA, b3, g.H3t, a3);

  // output layer, loss and dL/dy = 2 (y - t) / (n NOUT) in normalised units;
  // waves 0-3 own outputs 16w .. 16w+15
  if (w < NOUT / 16) {
    acc = w4.times(HA, LDH, lane);
    const float bj = g.b4[j], sh = g.nm->out_shift[j], sc = g.nm->out_scale[j];
    double lsum = 0.0;
    float cs = 0.0f, dv[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float y = acc[e] + bj;
      float dy = 0.0f;
      if (r0 + rq + e < g.nvalid) {
        const float tn = (tv[e] - sh) * sc;
        const float res = y - tn;
        lsum += (double)res * (double)res;
        dy = res * g.dscale;
      }
      dv[e] = dy;
      DY[(rq + e) * LDY + j] = to_bf16(dy);
      cs += dy;
    }
    store_t4(blk(g.DYt, NOUT), j, rq, dv);
    cs = col_sum16(cs);
    if (lane < 16) g.bp4[(size_t)rb * NOUT + j] = cs;
    lsum = wave_sum(lsum);
    if (lane == 0) lred[w] = lsum;
  }
  static_assert(NOUT / 16 == 4, "loss partials of four waves");
  __syncthreads();
  if (t == 0) g.lpart[rb] = ((lred[0] + lred[1]) + lred[2]) + lred[3];

  // backward through layers 4 -> 3 -> 2 (da_l = (da_{l+1} W_{l+1}) GELU'(a_l)) and 2 -> 1
  float da[4];
  const Weights<KH> w3t(g.W3t, w, lane);
  auto back = [&](const float (&av)[4], float* bp) {
    float c0 = 0.0f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      da[e] = acc[e] * gelu_grad(av[e]);
      c0 += da[e];
    }
    c0 = col_sum16(c0);
    if (lane < 16) bp[(size_t)rb * WID + j] = c0;
  };
  auto hand_on = [&](bf16_t* dst, bf16_t* Dt) {
#pragma unroll
    for (int e = 0; e < 4; ++e) dst[(rq + e) * LDH + j] = to_bf16(da[e]);
    store_t4(blk(Dt, WID), j, rq, da);
    __syncthreads();
  };
  acc = w4t.times(DY, LDY, lane);
  back(a3, g.bp3);
  hand_on(HB, g.D3t);
  acc = w3t.times(HB, LDH, lane);
  const Weights<KH> w2t(g.W2t, w, lane);
  back(a2, g.bp2);
  hand_on(HA, g.D2t);
  acc = w2t.times(HA, LDH, lane);
  back(a1, g.bp1);
  // first layer's weight gradient, summed over the block's rows (rows e of this
  // lane, then across lanes); four features at a time, each quarter of the wave
  // stores one
  float* wp = g.w1p + (size_t)rb * NFEAT * WID + j;
#pragma unroll
  for (int c = 0; c < NFEAT; c += 4) {
    float cf[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      cf[q] = 0.0f;
#pragma unroll
      for (int e = 0; e < 4; ++e) cf[q] = fmaf(da[e], xs[rq + e][c + q], cf[q]);
      cf[q] = col_sum16(cf[q]);
    }
    const int q = lane >> 4;
    wp[(size_t)(c + q) * WID] = q == 0 ? cf[0] : q == 1 ? cf[1] : q == 2 ? cf[2] : cf[3];
  }
}

// ---------------------------------------------------------------------------
// gradient assembly (fixed-order sums of the partials) and Adam
// ---------------------------------------------------------------------------
struct WCopies {
  bf16_t *W1b, *W2b, *W2t, *W3b, *W3t, *W4b, *W4t;
};

__device__ __forceinline__ void store_copies(int p, float v, const WCopies& c) {
  const bf16_t b = to_bf16(v);
  if (p < OB1) {
    c.W1b[p] = b;
  } else if (p >= OW2 && p < OB2) {
    const int e = p - OW2, o = e / WID, i = e % WID;
    c.W2b[wpos(o, i, WID)] = b;
    c.W2t[wpos(i, o, WID)] = b;
  } else if (p >= OW3 && p < OB3) {
    const int e = p - OW3, o = e / WID, i = e % WID;
    c.W3b[wpos(o, i, WID)] = b;
    c.W3t[wpos(i, o, WID)] = b;
  } else if (p >= OW4 && p < OB4) {
    const int e = p - OW4, o = e / WID, i = e % WID;
    c.W4b[wpos(o, i, WID)] = b;
    c.W4t[wpos(i, o, NOUT)] = b;
  }
}

__global__ __launch_bounds__(256) void copies_kernel(const float* __restrict__ P, WCopies c) {
  const int p = blockIdx.x * 256 + threadIdx.x;
  if (p < NPAR) store_copies(p, P[p], c);
}

// Training control on the device, so that a captured epoch can be replayed:
// the learning rate of the epoch and the number of Adam steps taken before it.
struct TrainCtl {
  double t0;
  double lr;
};

struct WgradProduct {
  const bf16_t* A;   // [R][M][RB]
  const bf16_t* Bt;  // [R][WID][RB]
  int M, op;         // rows of the product, its place in the parameter vector
  bf16_t *W, *Wt;    // BF16 copies, M outputs of WID inputs and the transpose
};

struct GradArgs {
  WgradProduct p[3];
  int K, S, R;         // batch rows, splits of the weight products, RB-row blocks
  const float *w1p, *bp1, *bp2, *bp3, *bp4;
  const double* lpart;
  double inv_count;    // 1 / (nvalid * 64)
  double* loss;        // one FP64
  float* G;            // gradient out [NPAR] (without update)
  // Adam: step t = ctl->t0 + step + 1, bias corrections 1 - beta^t
  float *P, *Mo, *Ve;
  const TrainCtl* ctl;
  int step;
  double beta1, beta2;
  float eps;
  bf16_t* W1b;
};

__global__ void ctl_set_lr(TrainCtl* c, double lr) {
  if (threadIdx.x == 0) c->lr = lr;
}
__global__ void ctl_advance(TrainCtl* c, int nsteps) {
  if (threadIdx.x == 0) c->t0 += (double)nsteps;
}

// ---------------------------------------------------------------------------
// training step, part 2: the three weight-gradient products
//   gW_l[M][N] = sum over batch rows of da_l^T h_{l-1}  (A = da_l^T, Bt = h_{l-1}^T),
// every other sum over the batch, and Adam, in one launch.  A block takes one of
//   - a 32 x 32 tile of a product: wave s computes the splits s, s + 8, ... (KSPLIT
//     batch rows each, all operand fragments loaded first), the block adds the
//     splits in their order from LDS and updates the tile's weights and both
//     BF16 copies, the transposed one through LDS;
//   - 64 columns of the first layer's weight gradient or of a bias gradient: the
//     waves load 128 blocks' partials side by side, the first wave adds them in
//     order;
//   - the loss.
// At the training batch of 2048 rows that is one block per CU, 8.4 us; a product
// kernel with the splits' partials through memory and a kernel of one thread per
// parameter took 27.
// ---------------------------------------------------------------------------
constexpr int GT = 512, GW = GT / 64, TILE = 32, TP = TILE + 4;  // threads, waves, tile, its LDS pitch
constexpr int SUMR = 128;                                       // partials a block adds between barriers
constexpr int TILES4 = (NOUT / TILE) * (WID / TILE), TILES3 = (WID / TILE) * (WID / TILE);
constexpr int NTILES = TILES4 + 2 * TILES3, NW1B = WID * NFEAT / 64, NBIAS = (3 * WID + NOUT) / 64;
constexpr int GRAD_BLOCKS = NTILES + NW1B + NBIAS + 1;

struct AdamCoef {
  float bc1, bc2;
};
__device__ __forceinline__ AdamCoef adam_coef(const GradArgs& g) {
  const double t = g.ctl->t0 + (double)(g.step + 1);
  return AdamCoef{(float)(1.0 - pow(g.beta1, t)), (float)(1.0 - pow(g.beta2, t))};
}
__device__ __forceinline__ float adam(const GradArgs& g, const AdamCoef& c, int p, float gr, float m0, float v0,
                                      float w0) {
  const float lr = (float)g.ctl->lr, b1 = (float)g.beta1, b2 = (float)g.beta2;
  const float m = fmaf(1.0f - b1, gr, b1 * m0), v = fmaf(gr, (1.0f - b2) * gr, b2 * v0);
  g.Mo[p] = m;
  g.Ve[p] = v;
  const float w = w0 - lr * (m / c.bc1) / (sqrtf(v / c.bc2) + g.eps);
  g.P[p] = w;
  return w;
}

template <bool UPDATE>
__global__ __launch_bounds__(GT) void grad_kernel(GradArgs g) {
  __shared__ __align__(16) float part[GW * TILE * TP];
  __shared__ bf16_t tr[TILE][TILE + 2];
  __shared__ AdamCoef coef;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  int b = blockIdx.x;
  if (b < NTILES) {
    const int pi = b < TILES4 ? 0 : (b < TILES4 + TILES3 ? 1 : 2);
    const WgradProduct& P = g.p[pi];
    const int loc = pi == 0 ? b : (b - TILES4) % TILES3;
    const int row0 = loc / (WID / TILE) * TILE, col0 = loc % (WID / TILE) * TILE;
    const int r16 = lane & 15, kq = (lane >> 4) * 8, M = P.M;
    constexpr int EL = TILE * TILE / GT;  // elements per thread in the update
    float sum[EL];
    int pe[EL];
    float m0[EL], v0[EL], w0[EL];
#pragma unroll
    for (int q = 0; q < EL; ++q) {
      const int e = t + GT * q;
      sum[q] = 0.0f;
      pe[q] = P.op + (row0 + e / TILE) * WID + col0 + e % TILE;
    }
    for (int s0 = 0; s0 < g.S; s0 += GW) {
      const int kb = (s0 + w) * KSPLIT, nk = (min(g.K, kb + KSPLIT) - kb) >> 5;  // <= 0 past the last split
      f4 acc[2][2];
#pragma unroll
      for (int rt = 0; rt < 2; ++rt)
#pragma unroll
        for (int ct = 0; ct < 2; ++ct) acc[rt][ct] = f4{0.0f, 0.0f, 0.0f, 0.0f};
      bf16x8 fa[KSPLIT / 32][2], fb[KSPLIT / 32][2];
#pragma unroll
      for (int s = 0; s < KSPLIT / 32; ++s) {
        if (s < nk) {
          const int k = kb + 32 * s + kq;
          const bf16_t* pa = P.A + ((size_t)(k / RB) * M + row0 + r16) * RB + k % RB;
          const bf16_t* pb = P.Bt + ((size_t)(k / RB) * WID + col0 + r16) * RB + k % RB;
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            fa[s][q] = load8(pa + q * 16 * RB);
            fb[s][q] = load8(pb + q * 16 * RB);
          }
        }
      }
      if (s0 == 0 && UPDATE) {
#pragma unroll
        for (int q = 0; q < EL; ++q) {
          m0[q] = g.Mo[pe[q]];
          v0[q] = g.Ve[pe[q]];
          w0[q] = g.P[pe[q]];
        }
        if (w == GW - 1) {
          const AdamCoef c = adam_coef(g);
          if (lane == 0) coef = c;
        }
      }
#pragma unroll
      for (int s = 0; s < KSPLIT / 32; ++s) {
        if (s < nk) {
#pragma unroll
          for (int rt = 0; rt < 2; ++rt)
#pragma unroll
            for (int ct = 0; ct < 2; ++ct) acc[rt][ct] = mma(fa[s][rt], fb[s][ct], acc[rt][ct]);
        }
      }
      if (s0) __syncthreads();  // the sums below have read the previous splits
#pragma unroll
      for (int rt = 0; rt < 2; ++rt)
#pragma unroll
        for (int ct = 0; ct < 2; ++ct)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            part[(w * TILE + rt * 16 + (lane >> 4) * 4 + e) * TP + ct * 16 + r16] = acc[rt][ct][e];
      __syncthreads();
#pragma unroll
      for (int q = 0; q < EL; ++q) {
        const int e = t + GT * q;
#pragma unroll
        for (int s = 0; s < GW; ++s)
          if (s0 + s < g.S) sum[q] += part[(s * TILE + e / TILE) * TP + e % TILE];
      }
    }
    if constexpr (!UPDATE) {
#pragma unroll
      for (int q = 0; q < EL; ++q) g.G[pe[q]] = sum[q];
    } else {
      const AdamCoef c = coef;
#pragma unroll
      for (int q = 0; q < EL; ++q) {
        const int e = t + GT * q, i = e / TILE, j = e % TILE;
        tr[i][j] = to_bf16(adam(g, c, pe[q], sum[q], m0[q], v0[q], w0[q]));
      }
      __syncthreads();
      // a tile is two fragments of either copy
      static_assert(TILE == 32, "one 32-deep fragment");
#pragma unroll
      for (int q = 0; q < EL; ++q) {
        const int e = t + GT * q, f = e / FRAG, x = e % FRAG, o = 16 * f + x / 8 % 16, i = x / 128 * 8 + x % 8;
        P.W[((row0 / 16 + f) * (WID / 32) + col0 / 32) * FRAG + x] = tr[o][i];
        P.Wt[((col0 / 16 + f) * (M / 32) + row0 / 32) * FRAG + x] = tr[i][o];
      }
    }
    return;
  }
  b -= NTILES;
  if (b < NW1B + NBIAS) {
    // 64 columns: of w1p (feature-major, column c WID + j is parameter j NFEAT + c) or of a bias
    const float* src;
    int width, col, p;
    if (b < NW1B) {
      src = g.w1p;
      width = WID * NFEAT;
      col = 64 * b + lane;
      p = OW1 + (col % WID) * NFEAT + col / WID;
    } else {
      const int k = b - NW1B, l = min(k / (WID / 64), 3);
      src = l == 0 ? g.bp1 : l == 1 ? g.bp2 : l == 2 ? g.bp3 : g.bp4;
      width = l < 3 ? WID : NOUT;
      col = 64 * (k - l * (WID / 64)) + lane;
      p = (l == 0 ? OB1 : l == 1 ? OB2 : l == 2 ? OB3 : OB4) + col;
    }
    static_assert(SUMR * 64 <= GW * TILE * TP, "partials fit the LDS of a tile block");
    float sum = 0.0f;
    for (int r0 = 0; r0 < g.R; r0 += SUMR) {
      float v[SUMR / GW];
#pragma unroll
      for (int m = 0; m < SUMR / GW; ++m) {
        const int r = r0 + w + GW * m;
        v[m] = r < g.R ? src[(size_t)r * width + col] : 0.0f;
      }
      if (r0) __syncthreads();
#pragma unroll
      for (int m = 0; m < SUMR / GW; ++m) part[(w + GW * m) * 64 + lane] = v[m];
      __syncthreads();
      if (w == 0) {
        const int n = min(SUMR, g.R - r0);  // R is a multiple of 4
        for (int r = 0; r < n; r += 4) {
#pragma unroll
          for (int k = 0; k < 4; ++k) sum += part[(r + k) * 64 + lane];
        }
      }
    }
    if (w) return;
    if constexpr (!UPDATE) {
      g.G[p] = sum;
    } else {
      const float v = adam(g, adam_coef(g), p, sum, g.Mo[p], g.Ve[p], g.P[p]);
      if (b < NW1B) g.W1b[p - OW1] = to_bf16(v);
    }
    return;
  }
  // the loss
  double* lp = reinterpret_cast<double*>(part);
  static_assert(MAX_BATCH / RB * sizeof(double) <= sizeof(part), "loss partials fit");
  for (int r = t; r < g.R; r += GT) lp[r] = g.lpart[r];
  __syncthreads();
  if (t == 0) {
    double s = 0.0;
    for (int r = 0; r < g.R; r += 4) {
#pragma unroll
      for (int k = 0; k < 4; ++k) s += lp[r + k];
    }
    g.loss[0] = s * g.inv_count;
  }
}

// ---------------------------------------------------------------------------
// fused inference: 16 RT query rows per block of NW waves, activations stay in LDS
//
// Bound by vector instruction issue: a GELU is 22 instructions and two
// transcendentals, 768 of them a row, the first layer 6144 multiply-adds a row
// (47 of 61 us at 65536 rows; the matrix products alone would take 17).  With
// one thread of four forming all features of a row, one unit per thread in the
// first layer, lanes holding one unit of four rows and storing them as 16-bit
// words, integer rounding to BF16, row-major weights and two blocks a CU: 88 us.
// ---------------------------------------------------------------------------
template <int RT, int NW>
__global__ __launch_bounds__(64 * NW, NW == 16 ? 4 : 3) void predict_kernel(const float* __restrict__ X, int64_t n,
                                                               const Norm* __restrict__ nm, WCopies c,
                                                               const float* __restrict__ b1,
                                                               const float* __restrict__ b2,
                                                               const float* __restrict__ b3,
                                                               const float* __restrict__ b4, float* __restrict__ Y) {
  constexpr int NR = 16 * RT, NT = 64 * NW, CT = WID / 16 / NW;
  __shared__ __align__(16) bf16_t H[NR * LDH];
  __shared__ __align__(16) float xs[NR][NFEAT];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int r16 = lane & 15, kq = (lane >> 4) * 8, uq = (lane >> 4) * 4;
  const int64_t r0 = (int64_t)blockIdx.x * NR;
  // each wave's priority by the block's place on its CU: four blocks in step
  // share the vector units and then leave them idle for the matrix units (65536
  // rows 68 us without)
  if constexpr (NW == 4) {
    switch ((blockIdx.x >> 8) & 3) {
      case 1: __builtin_amdgcn_s_setprio(1); break;
      case 2: __builtin_amdgcn_s_setprio(2); break;
      case 3: __builtin_amdgcn_s_setprio(3); break;
    }
  }
  block_features<NR, NT>(X, nm, t, [&](int r) -> int64_t { return r0 + r < n ? r0 + r : -1; }, xs);
  __syncthreads();
  // layer 1 (K = NFEAT, plain FMA): a thread takes two neighbouring units of its
  // share of the rows, so that a row's features, the same for all lanes, are read
  // from LDS once for both and the result goes back as one 32-bit word
  constexpr int G = NT / (WID / 2), RG = NR / G;
  const int u = 2 * (t % (WID / 2)), g0 = (t / (WID / 2)) * RG;
  float wf[2][NFEAT], bu[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    bu[q] = b1[u + q];
#pragma unroll
    for (int k = 0; k < NFEAT; k += 8) {
      const bf16x8 v = load8(c.W1b + NFEAT * (u + q) + k);
#pragma unroll
      for (int m = 0; m < 8; ++m) wf[q][k + m] = (float)v[m];
    }
  }
#pragma unroll 2
  for (int r = g0; r < g0 + RG; ++r) {
    float a0 = bu[0], a1 = bu[1];
#pragma unroll
    for (int k = 0; k < NFEAT; ++k) {
      a0 = fmaf(xs[r][k], wf[0][k], a0);
      a1 = fmaf(xs[r][k], wf[1][k], a1);
    }
    *reinterpret_cast<uint32_t*>(H + r * LDH + u) = to_bf16x2(gelu(a0), gelu(a1));
  }
  __syncthreads();
  // hidden layers 2 and 3: wave w owns units 16 CT w .. 16 CT (w + 1) - 1 of all
  // rows.  The weights are the first operand, so a lane receives four
  // neighbouring units of one row.
#pragma unroll 1
  for (int layer = 0; layer < 2; ++layer) {
    const bf16_t* W = layer ? c.W3b : c.W2b;
    const float* bias = layer ? b3 : b2;
    f4 acc[RT][CT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) acc[rt][ct] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    const bf16_t* wb = W + (size_t)CT * w * (WID / 32) * FRAG + 8 * lane;
#pragma unroll CT == 1 ? 8 : 2
    for (int kk = 0; kk < WID; kk += 32) {
      bf16x8 a[RT], b[CT];
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) b[ct] = load8(wb + (ct * (WID / 32) + kk / 32) * FRAG);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) a[rt] = load8(&H[(rt * 16 + r16) * LDH + kk + kq]);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[rt][ct] = mma(b[ct], a[rt], acc[rt][ct]);
    }
    __syncthreads();
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const int j = 16 * (CT * w + ct) + uq;
      const f4 bj = *reinterpret_cast<const f4*>(bias + j);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = gelu(acc[rt][ct][e] + bj[e]);
        *reinterpret_cast<uint2*>(H + (rt * 16 + r16) * LDH + j) = uint2{to_bf16x2(v[0], v[1]), to_bf16x2(v[2], v[3])};
      }
    }
    __syncthreads();
  }
  // output layer: wave w owns outputs 16w .. 16w+15
  if (w >= NOUT / 16) return;
  f4 acc[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) acc[rt] = f4{0.0f, 0.0f, 0.0f, 0.0f};
  const bf16_t* wb = c.W4b + (size_t)w * (WID / 32) * FRAG + 8 * lane;
#pragma unroll CT == 1 ? 8 : 2
  for (int kk = 0; kk < WID; kk += 32) {
    const bf16x8 b = load8(wb + kk / 32 * FRAG);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) acc[rt] = mma(b, load8(&H[(rt * 16 + r16) * LDH + kk + kq]), acc[rt]);
  }
  const int j = 16 * w + uq;
  const f4 bj = *reinterpret_cast<const f4*>(b4 + j);
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int64_t i = r0 + rt * 16 + r16;
    if (i >= n) continue;
    f4 y;
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = (acc[rt][e] + bj[e]) / nm->out_scale[j + e] + nm->out_shift[j + e];
    *reinterpret_cast<f4_any*>(Y + i * NOUT + j) = y;
  }
}

}  // namespace

// per-column mean and 1/std of the targets (one block per column, FP64,
// fixed-order tree reduction)
__global__ __launch_bounds__(256) void column_stats(const float* __restrict__ T, int64_t n, Norm* nm,
                                                    double* out) {
  __shared__ double red[256];
  const int c = blockIdx.x, t = threadIdx.x;
  double s = 0.0;
  for (int64_t i = t; i < n; i += 256) s += (double)T[i * NOUT + c];
  red[t] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (t < o) red[t] += red[t + o];
    __syncthreads();
  }
  const double mean = red[0] / (double)n;
  __syncthreads();
  double q = 0.0;
  for (int64_t i = t; i < n; i += 256) {
    const double d = (double)T[i * NOUT + c] - mean;
    q += d * d;
  }
  red[t] = q;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (t < o) red[t] += red[t + o];
    __syncthreads();
  }
  if (t == 0) {
    const double sd = fmax(sqrt(red[0] / (double)n), 1e-6);
    out[c] = mean;
    out[NOUT + c] = 1.0 / sd;
    nm->out_shift[c] = (float)mean;
    nm->out_scale[c] = (float)(1.0 / sd);
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
struct surrogate_t {
  surrogate_params p;
  hipStream_t stream;
  int B;  // max_batch
  float *P, *Mo, *Ve;
  Norm* nm;
  WCopies wc;
  bf16_t *H1t, *H2t, *H3t, *DYt, *D3t, *D2t;
  float *bp1, *bp2, *bp3, *bp4, *w1p;
  double *lpart, *losses, *stats;
  TrainCtl* ctl;
  int64_t t;   // Adam steps taken
  bool loaded;
  // captured epoch, replayed while its inputs are the same buffers and sizes
  bool use_graph;
  hipGraphExec_t graph;
  const void* gkey[3];
  int64_t gn;
};

namespace {

// carve the workspace (base == nullptr: only measure)
size_t carve(int B, char* base, surrogate_t* s) {
  size_t off = 0;
  auto take = [&](size_t bytes) -> char* {
    off = (off + 255) & ~(size_t)255;
    char* q = base ? base + off : nullptr;
    off += bytes;
    return q;
  };
  const int R = B / RB;
  surrogate_t d{};
  surrogate_t& h = s ? *s : d;
  h.P = (float*)take(4ull * NPAR);
  h.Mo = (float*)take(4ull * NPAR);
  h.Ve = (float*)take(4ull * NPAR);
  h.nm = (Norm*)take(sizeof(Norm));
  h.wc.W1b = (bf16_t*)take(2ull * WID * NFEAT);
  h.wc.W2b = (bf16_t*)take(2ull * WID * WID);
  h.wc.W2t = (bf16_t*)take(2ull * WID * WID);
  h.wc.W3b = (bf16_t*)take(2ull * WID * WID);
  h.wc.W3t = (bf16_t*)take(2ull * WID * WID);
  h.wc.W4b = (bf16_t*)take(2ull * NOUT * WID);
  h.wc.W4t = (bf16_t*)take(2ull * NOUT * WID);
  bf16_t** act[] = {&h.H1t, &h.H2t, &h.H3t, &h.D3t, &h.D2t};
  for (bf16_t** a : act) *a = (bf16_t*)take(2ull * B * WID);
  h.DYt = (bf16_t*)take(2ull * B * NOUT);
  h.bp1 = (float*)take(4ull * R * WID);
  h.bp2 = (float*)take(4ull * R * WID);
  h.bp3 = (float*)take(4ull * R * WID);
  h.bp4 = (float*)take(4ull * R * NOUT);
  h.w1p = (float*)take(4ull * R * WID * NFEAT);
  h.lpart = (double*)take(8ull * R);
  h.losses = (double*)take(8ull * MAX_STEPS);
  h.stats = (double*)take(8ull * 2 * NOUT);
  h.ctl = (TrainCtl*)take(sizeof(TrainCtl));
  return off + 256;
}

int validate(const surrogate_params* p) {
  if (!p) { set_error("NULL params"); return LAT_EINVAL; }
  if (p->max_batch < 64 || p->max_batch > MAX_BATCH || p->max_batch % 64) {
    set_error("max_batch must be a multiple of 64 in [64, 16384]");
    return LAT_EINVAL;
  }
  if (!(p->beta1 >= 0.0 && p->beta1 < 1.0 && p->beta2 >= 0.0 && p->beta2 < 1.0 && p->eps > 0.0)) {
    set_error("Adam parameters: need 0 <= beta < 1 and eps > 0");
    return LAT_EINVAL;
  }
  for (int c = 0; c < NIN; ++c)
    if (!std::isfinite(p->in_shift[c]) || !std::isfinite(p->in_scale[c]) || p->in_scale[c] == 0.0f ||
        !std::isfinite(p->enc_freq[c])) {
      set_error("input normalisation must be finite with nonzero scale, and the encoding frequencies finite");
      return LAT_EINVAL;
    }
  for (int c = 0; c < NOUT; ++c)
    if (!std::isfinite(p->out_shift[c]) || !std::isfinite(p->out_scale[c]) || p->out_scale[c] == 0.0f) {
      set_error("output normalisation must be finite with nonzero scale");
      return LAT_EINVAL;
    }
  return LAT_OK;
}

void drop_graph(surrogate_t* h) {
  if (h->graph) hipGraphExecDestroy(h->graph);
  h->graph = nullptr;
  h->gkey[0] = h->gkey[1] = h->gkey[2] = nullptr;
  h->gn = 0;
}

// forward + backward of n rows (rows[] may be NULL) into G, loss into *loss_dev;
// with update, one Adam step on the master weights and their BF16 copies
int train_step(surrogate_t* h, const float* X, const float* T, const int32_t* rows, int n, float* G,
               double* loss_dev, bool update, int step) {
  hipStream_t st = h->stream;
  const int Bp = (n + 63) / 64 * 64, R = Bp / RB, S = (Bp + KSPLIT - 1) / KSPLIT;
  const WCopies& c = h->wc;
  // rows: forward, loss, backward to the input layer
  RowArgs ra{};
  ra.X = X; ra.T = T; ra.rows = rows; ra.nvalid = n;
  ra.dscale = (float)(2.0 / ((double)n * NOUT));
  ra.nm = h->nm;
  ra.W1b = c.W1b; ra.W2b = c.W2b; ra.W3b = c.W3b; ra.W4b = c.W4b;
  ra.W2t = c.W2t; ra.W3t = c.W3t; ra.W4t = c.W4t;
  ra.b1 = h->P + OB1; ra.b2 = h->P + OB2; ra.b3 = h->P + OB3; ra.b4 = h->P + OB4;
  ra.H1t = h->H1t; ra.H2t = h->H2t; ra.H3t = h->H3t;
  ra.DYt = h->DYt; ra.D3t = h->D3t; ra.D2t = h->D2t;
  ra.bp1 = h->bp1; ra.bp2 = h->bp2; ra.bp3 = h->bp3; ra.bp4 = h->bp4;
  ra.w1p = h->w1p; ra.lpart = h->lpart;
  hipLaunchKernelGGL(step_rows_kernel, dim3(R), dim3(64 * NWAVE), 0, st, ra);
  CL_HIP(hipGetLastError());
  GradArgs a{};
  a.p[0] = WgradProduct{h->DYt, h->H3t, NOUT, OW4, c.W4b, c.W4t};
  a.p[1] = WgradProduct{h->D3t, h->H2t, WID, OW3, c.W3b, c.W3t};
  a.p[2] = WgradProduct{h->D2t, h->H1t, WID, OW2, c.W2b, c.W2t};
  a.K = Bp; a.S = S; a.R = R;
  a.w1p = h->w1p; a.bp1 = h->bp1; a.bp2 = h->bp2; a.bp3 = h->bp3; a.bp4 = h->bp4;
  a.lpart = h->lpart;
  a.inv_count = 1.0 / ((double)n * NOUT);
  a.loss = loss_dev;
  a.G = G;
  a.P = h->P; a.Mo = h->Mo; a.Ve = h->Ve;
  a.W1b = c.W1b;
  if (update) {
    a.ctl = h->ctl;
    a.step = step;
    a.beta1 = h->p.beta1;
    a.beta2 = h->p.beta2;
    a.eps = (float)h->p.eps;
    hipLaunchKernelGGL(grad_kernel<true>, dim3(GRAD_BLOCKS), dim3(GT), 0, st, a);
  } else {
    hipLaunchKernelGGL(grad_kernel<false>, dim3(GRAD_BLOCKS), dim3(GT), 0, st, a);
  }
  CL_HIP(hipGetLastError());
  return LAT_OK;
}

}  // namespace

extern "C" int surrogate_workspace_size(const surrogate_params* p, size_t* bytes) {
  int rc = validate(p);
  if (rc) return rc;
  if (!bytes) { set_error("NULL argument"); return LAT_EINVAL; }
  *bytes = carve(p->max_batch, nullptr, nullptr);
  return LAT_OK;
}

extern "C" int surrogate_init(const surrogate_params* p, void* dev_ws, size_t ws_bytes, void* hip_stream,
                              surrogate_t** out) {
  int rc = validate(p);
  if (rc) return rc;
  if (!dev_ws || !out) { set_error("NULL argument"); return LAT_EINVAL; }
  const size_t need = carve(p->max_batch, nullptr, nullptr);
  if (ws_bytes < need) { set_error("workspace too small: need " + std::to_string(need)); return LAT_ENOMEM; }
  surrogate_t* h = new (std::nothrow) surrogate_t{};
  if (!h) { set_error("out of host memory"); return LAT_ENOMEM; }
  h->p = *p;
  h->stream = (hipStream_t)hip_stream;
  h->B = p->max_batch;
  h->use_graph = hip_stream != nullptr;
  char* base = (char*)(((uintptr_t)dev_ws + 255) & ~(uintptr_t)255);
  carve(h->B, base, h);
  Norm nm;
  std::memcpy(nm.in_shift, p->in_shift, sizeof nm.in_shift);
  std::memcpy(nm.in_scale, p->in_scale, sizeof nm.in_scale);
  std::memcpy(nm.out_shift, p->out_shift, sizeof nm.out_shift);
  std::memcpy(nm.out_scale, p->out_scale, sizeof nm.out_scale);
  std::memcpy(nm.enc_freq, p->enc_freq, sizeof nm.enc_freq);
  hipError_t e = hipMemcpyAsync(h->nm, &nm, sizeof(Norm), hipMemcpyHostToDevice, h->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
  if (e != hipSuccess) {
    set_error(std::string("surrogate_init: ") + hipGetErrorString(e));
    delete h;
    return LAT_EHIP;
  }
  *out = h;
  return LAT_OK;
}

extern "C" int surrogate_set_weights(surrogate_t* h, const float* host_w) {
  if (!h || !host_w) { set_error("NULL argument"); return LAT_EINVAL; }
  for (int i = 0; i < NPAR; ++i)
    if (!std::isfinite(host_w[i])) { set_error("non-finite weight"); return LAT_EINVAL; }
  CL_HIP(hipMemcpyAsync(h->P, host_w, 4ull * NPAR, hipMemcpyHostToDevice, h->stream));
  CL_HIP(hipMemsetAsync(h->Mo, 0, 4ull * NPAR, h->stream));
  CL_HIP(hipMemsetAsync(h->Ve, 0, 4ull * NPAR, h->stream));
  CL_HIP(hipMemsetAsync(h->ctl, 0, sizeof(TrainCtl), h->stream));
  hipLaunchKernelGGL(copies_kernel, dim3((NPAR + 255) / 256), dim3(256), 0, h->stream, h->P, h->wc);
  CL_HIP(hipGetLastError());
  CL_HIP(hipStreamSynchronize(h->stream));
  h->t = 0;
  h->loaded = true;
  return LAT_OK;
}

extern "C" int surrogate_get_weights(surrogate_t* h, float* host_w) {
  if (!h || !host_w) { set_error("NULL argument"); return LAT_EINVAL; }
  if (!h->loaded) { set_error("weights not set"); return LAT_ESTATE; }
  CL_HIP(hipMemcpyAsync(host_w, h->P, 4ull * NPAR, hipMemcpyDeviceToHost, h->stream));
  CL_HIP(hipStreamSynchronize(h->stream));
  return LAT_OK;
}

extern "C" int surrogate_fit_output_scale(surrogate_t* h, const float* dev_t, int64_t n, double* host_shift,
                                          double* host_scale) {
  if (!h || !dev_t) { set_error("NULL argument"); return LAT_EINVAL; }
  if (n < 2) { set_error("need at least 2 target rows"); return LAT_EINVAL; }
  hipLaunchKernelGGL(column_stats, dim3(NOUT), dim3(256), 0, h->stream, dev_t, n, h->nm, h->stats);
  CL_HIP(hipGetLastError());
  double st[2 * NOUT];
  CL_HIP(hipMemcpyAsync(st, h->stats, sizeof st, hipMemcpyDeviceToHost, h->stream));
  CL_HIP(hipStreamSynchronize(h->stream));
  for (int c = 0; c < 2 * NOUT; ++c)
    if (!std::isfinite(st[c])) { set_error("non-finite target statistics"); return LAT_ENONFINITE; }
  for (int c = 0; c < NOUT; ++c) {
    h->p.out_shift[c] = (float)st[c];
    h->p.out_scale[c] = (float)st[NOUT + c];
    if (host_shift) host_shift[c] = st[c];
    if (host_scale) host_scale[c] = st[NOUT + c];
  }
  return LAT_OK;
}

extern "C" int surrogate_loss_grad(surrogate_t* h, const float* dev_x, const float* dev_t, const int32_t* rows,
                                   int32_t n, float* dev_grad, double* loss) {
  if (!h || !dev_x || !dev_t || !dev_grad || !loss) { set_error("NULL argument"); return LAT_EINVAL; }
  if (!h->loaded) { set_error("weights not set"); return LAT_ESTATE; }
  if (n < 1 || n > h->B) { set_error("n must be in [1, max_batch]"); return LAT_EINVAL; }
  int rc = train_step(h, dev_x, dev_t, rows, n, dev_grad, h->losses, false, 0);
  if (rc) return rc;
  CL_HIP(hipMemcpyAsync(loss, h->losses, 8, hipMemcpyDeviceToHost, h->stream));
  CL_HIP(hipStreamSynchronize(h->stream));
  if (!std::isfinite(*loss)) { set_error("non-finite loss"); return LAT_ENONFINITE; }
  return LAT_OK;
}

extern "C" int surrogate_train_epoch(surrogate_t* h, const float* dev_x, const float* dev_t,
                                     const int32_t* dev_perm, int64_t n, double lr, double* mean_loss) {
  if (!h || !dev_x || !dev_t || !dev_perm || !mean_loss) { set_error("NULL argument"); return LAT_EINVAL; }
  if (!h->loaded) { set_error("weights not set"); return LAT_ESTATE; }
  if (n < 1) { set_error("n must be positive"); return LAT_EINVAL; }
  if (!(lr > 0.0) || !std::isfinite(lr)) { set_error("lr must be positive"); return LAT_EINVAL; }
  const int64_t steps = (n + h->B - 1) / h->B;
  if (steps > MAX_STEPS) { set_error("too many steps in one epoch (max 65536)"); return LAT_EINVAL; }
  hipLaunchKernelGGL(ctl_set_lr, dim3(1), dim3(64), 0, h->stream, h->ctl, lr);
  CL_HIP(hipGetLastError());
  auto record = [&]() -> int {
    for (int64_t s = 0; s < steps; ++s) {
      const int ns = (int)std::min<int64_t>(h->B, n - s * h->B);
      int rc = train_step(h, dev_x, dev_t, dev_perm + s * h->B, ns, nullptr, h->losses + s, true, (int)s);
      if (rc) return rc;
    }
    hipLaunchKernelGGL(ctl_advance, dim3(1), dim3(64), 0, h->stream, h->ctl, (int)steps);
    CL_HIP(hipGetLastError());
    return LAT_OK;
  };
  const bool same = h->graph && h->gkey[0] == dev_x && h->gkey[1] == dev_t && h->gkey[2] == dev_perm && h->gn == n;
  if (h->use_graph && !same) {
    drop_graph(h);
    CL_HIP(hipStreamBeginCapture(h->stream, hipStreamCaptureModeThreadLocal));
    const int rc = record();
    hipGraph_t g = nullptr;
    const hipError_t e = hipStreamEndCapture(h->stream, &g);
    if (rc) {
      if (g) hipGraphDestroy(g);
      return rc;
    }
    CL_HIP(e);
    const hipError_t ei = hipGraphInstantiate(&h->graph, g, nullptr, nullptr, 0);
    hipGraphDestroy(g);
    if (ei != hipSuccess) {
      h->graph = nullptr;
      set_error(std::string("hipGraphInstantiate: ") + hipGetErrorString(ei));
      return LAT_EHIP;
    }
    h->gkey[0] = dev_x;
    h->gkey[1] = dev_t;
    h->gkey[2] = dev_perm;
    h->gn = n;
  }
  if (h->use_graph) {
    CL_HIP(hipGraphLaunch(h->graph, h->stream));
  } else {
    const int rc = record();
    if (rc) return rc;
  }
  h->t += steps;
  std::vector<double> l((size_t)steps);
  CL_HIP(hipMemcpyAsync(l.data(), h->losses, 8 * steps, hipMemcpyDeviceToHost, h->stream));
  CL_HIP(hipStreamSynchronize(h->stream));
  double m = 0.0;
  for (double v : l) m += v;
  *mean_loss = m / (double)steps;
  if (!std::isfinite(*mean_loss)) { set_error("non-finite loss"); return LAT_ENONFINITE; }
  return LAT_OK;
}

extern "C" int surrogate_predict(surrogate_t* h, const float* dev_x, int64_t n, float* dev_y) {
  if (!h || !dev_x || !dev_y) { set_error("NULL argument"); return LAT_EINVAL; }
  if (!h->loaded) { set_error("weights not set"); return LAT_ESTATE; }
  if (n < 0 || n > ((int64_t)1 << 36)) { set_error("n out of range"); return LAT_EINVAL; }
  if (n == 0) return LAT_OK;
  const WCopies& c = h->wc;
  auto launch = [&](auto kernel, int rows, int threads) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)((n + rows - 1) / rows)), dim3(threads), 0, h->stream, dev_x, n, h->nm, c,
                       h->P + OB1, h->P + OB2, h->P + OB3, h->P + OB4, dev_y);
  };
  // Rows per block: 16 as long as every CU gets at most one block of sixteen
  // waves, whose wave has a single tile of units per layer (one row 8.1 us, 4096
  // rows 9.9; 32-row blocks 12.2, 64-row ones 22.9), then 32 (8192 rows 13.8 us,
  // 14.8 with 16 and 23.6 with 64; 16384 rows 24.5, 27.1 and 26.0).  Beyond that
  // four waves with four tiles each, which read a row's activations from LDS a
  // quarter as often and leave room for four blocks on a CU (32768 rows 37.7 us,
  // 32-row blocks 45.0; 65536 rows 61 us).
  constexpr int CUS = 256;
  if (n <= 16 * CUS) launch(predict_kernel<1, 16>, 16, 1024);
  else if (n <= 64 * CUS) launch(predict_kernel<2, 16>, 32, 1024);
  else launch(predict_kernel<4, 4>, 64, 256);
  CL_HIP(hipGetLastError());
  return LAT_OK;
}

extern "C" int surrogate_use_graph(surrogate_t* h, int on) {
  if (!h) { set_error("NULL handle"); return LAT_EINVAL; }
  if (on && !h->stream) { set_error("graph capture needs a created (non-default) stream"); return LAT_EINVAL; }
  CL_HIP(hipStreamSynchronize(h->stream));
  drop_graph(h);
  h->use_graph = on != 0;
  return LAT_OK;
}

extern "C" int surrogate_destroy(surrogate_t* h) {
  if (!h) return LAT_OK;
  hipError_t e = hipStreamSynchronize(h->stream);
  drop_graph(h);
  delete h;
  if (e != hipSuccess) { set_error(std::string("surrogate_destroy: ") + hipGetErrorString(e)); return LAT_EHIP; }
  return LAT_OK;
}
