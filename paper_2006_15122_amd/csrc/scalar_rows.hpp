// Full-row tile of the fused scalar pass: stepping passes and observations.
//
// A block holds whole z-rows of the lattice: N = W NL sites per row, W
// consecutive sites per lane moved as one 16-byte access (W = 4 in FP32
// storage, 2 in FP64).  It owns BY consecutive y-rows and marches along x
// over its share of planes like the general tile, with each site's drift and
// kick written term for term as there: from the same a and b, a pass gives every
// site the general tile's new field and momentum bit for bit.  Each site's
// energy terms join the FP64 totals one by one, as there (the four sites of a
// lane added in FP32 first round alike in a near-homogeneous state, 1e-8 of b's
// change, and saved next to nothing: 160^3 32.3 us a pass then, 31.6 now, 192^3
// 49.8 and 49.4, 320^3 204 and 203, 128^3 19.4 and 20.0), so the sums differ from
// the general tile's by the order of FP64 additions.  What
// changes is the memory side: the periodic z-neighbours of a row are in the row
// itself (no z halo loads at all), every global access is a whole 16-byte lane
// segment of a row, and one address serves W sites.  The only halo left is the
// two y-rows above and below the block, spread over all lanes.
//
// N is a run-time number (any multiple of 32), so the block size is too: with
// BY a multiple of 64 / W every block is whole waves.  Each row's place in LDS
// is an address formed once per lane, which costs nothing measurable against
// rows of a compiled length.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "common.hpp"
#include "internal.hpp"
#include "scalar_tile.hpp"

namespace cl {

// W consecutive sites of one row: the vector a lane loads and stores
template <typename T, int W>
struct RowVec {
  typedef T type __attribute__((ext_vector_type(W)));
};

__device__ __forceinline__ float fma_t(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double fma_t(double a, double b, double c) { return fma(a, b, c); }

// Per-lane accumulators of a block of whole waves into partials[pidx] (wave
// shuffles, then the waves in order).
constexpr int kRowsMaxThreads = 768;

template <int NACC>
__device__ __forceinline__ void rows_partials(double* partials, double (&acc)[NACC], int pidx) {
  __shared__ double red[kRowsMaxThreads / 64][NACC];
  const int tid = threadIdx.x, nw = blockDim.x >> 6;
#pragma unroll
  for (int k = 0; k < NACC; ++k) {
    const double s = wave_sum(acc[k]);
    if ((tid & 63) == 0) red[tid >> 6][k] = s;
  }
  __syncthreads();
  if (tid < NACC) {
    double s = 0.0;
    for (int w = 0; w < nw; ++w) s += red[w][tid];
    partials[(size_t)pidx * NACC + tid] = s;
  }
}

// As reduce_partials, for a block of any number of whole waves.
template <int NACC>
__device__ bool rows_reduce_partials(const double* partials, int first, int nb, double (&S)[NACC]) {
  __shared__ double red[kRowsMaxThreads / 64][NACC];
  const int tid = threadIdx.x, nw = blockDim.x >> 6;
  double tot[NACC];
#pragma unroll
  for (int k = 0; k < NACC; ++k) tot[k] = 0.0;
  for (int b = tid; b < nb; b += blockDim.x) {
#pragma unroll
    for (int k = 0; k < NACC; ++k) tot[k] += partials[(size_t)(first + b) * NACC + k];
  }
#pragma unroll
  for (int k = 0; k < NACC; ++k) {
    const double s = wave_sum(tot[k]);
    if ((tid & 63) == 0) red[tid >> 6][k] = s;
  }
  __syncthreads();
  if (tid != 0) return false;
  for (int k = 0; k < NACC; ++k) {
    double s = 0.0;
    for (int w = 0; w < nw; ++w) s += red[w][k];
    S[k] = s;
  }
  return true;
}

// LDS bytes of a block: two planes of NF fields, BY + 2 rows each
template <typename T>
__host__ __device__ constexpr size_t rows_lds_bytes(int nf, int N, int by) {
  return (size_t)2 * nf * (by + 2) * N * sizeof(T);
}

// KH: halo sites per lane, at least 2 NF W / BY.  IDLE: the block may have more
// lanes than the NL BY its rows take (batches of several N); the lanes beyond
// only join the barriers and sums.
// MODE kRowsObs: an observation pass, which neither drifts nor stores; its
// sums are the general tile's, each site's terms added in FP64.  kRowsObsSync:
// the same of a synchronised state, where no part of a kick enters E_K and the
// stencil is left out.
enum RowsMode { kRowsStep = 0, kRowsObs = 1, kRowsObsSync = 2 };
template <typename T, int W, int NF, int KH, bool IDLE, int MODE, typename GetAB>
__device__ __forceinline__ void scalar_rows(const ScalarArgs<T>& A, const int BY, int tile, int pidx, GetAB get_ab) {
  using VW = typename RowVec<T, W>::type;  // W consecutive sites
  constexpr bool FULL = MODE != kRowsStep;
  constexpr int NACC = Acc<NF, FULL>::N;
  // drifted planes in two buffers: plane x0 + i in buffer i & 1 (x0 - 1 in
  // buffer 1), rows y0-1 .. y0+BY, each a whole z-row; the x-1 neighbours of
  // the stencil are read from the other buffer
  extern __shared__ __align__(16) unsigned char rows_smem[];
  VW* const lds = reinterpret_cast<VW*>(rows_smem);

  const int N = A.N, NL = N / W, NT = NL * BY;
  const int tid = threadIdx.x;
  const int ty = tid / NL, tz = tid - ty * NL;
  const bool active = !IDLE || tid < NT;
  const int fst = (BY + 2) * NL, bst = NF * fst;  // field and buffer strides
  const int nyt = N / BY;
  const int yt = tile % nyt, xcI = tile / nyt;
  const int nx = A.nx ? A.nx : N / A.XC;
  const int y0 = yt * BY, x0 = x_first(N, xcI, nx), XC = x_first(N, xcI + 1, nx) - x0;
  const size_t NN = (size_t)N * N;
  const int own = (1 + ty) * NL + tz;  // this lane's place in a row buffer
  // its z-neighbours' places, in sites (periodic in the row)
  const int zl = ((1 + ty) * NL + (tz == 0 ? NL - 1 : tz - 1)) * W + W - 1;
  const int zh = ((1 + ty) * NL + (tz == NL - 1 ? 0 : tz + 1)) * W;

  const Coef<T> ckick = ucoef<T>((A.pd.wk1 + A.pd.wk2) * A.h);
  const Coef<T> cE = ucoef<T>((A.pd.mode == MODE_LF ? (A.pd.wk1 + A.pd.wk2) : A.pd.wk1) * A.h);
  const Coef<T> m2_0c = ucoef<T>(A.m2_0), m2_1c = ucoef<T>(A.m2_1), lamc = ucoef<T>(A.lam), qc_ = ucoef<T>(A.q);
  // potential-energy density V = p2 (m2_0/2 + lam p2/4) + c2 (m2_1/2 + q p2/2)
  const T hm2_0 = (T)(0.5 * A.m2_0), qlam = (T)(0.25 * A.lam), hm2_1 = (T)(0.5 * A.m2_1), hqq = (T)(0.5 * A.q);
  const bool lf = A.pd.mode == MODE_LF;

  double acc[NACC];
#pragma unroll
  for (int k = 0; k < NACC; ++k) acc[k] = 0.0;

  const int y = y0 + ty;
  // register planes (four sites each): pc = drifted x, qc = momentum at x,
  // (pn, qn) = raw x+1, (pf, qf) = raw x+2 in flight
  VW pc[NF], qc[NF], pn[NF], qn[NF], pf[NF], qf[NF];

  // halo rows y0-1 and y0+BY of plane x+1, loaded one plane ahead of their
  // use: 2 NF N single sites spread over all lanes, KH per lane
  const int NHI = 2 * NF * N;
  T hp[KH], hq[KH];
  // halo item k of this lane: row r (0: y0-1, 1: y0+BY), field f, site z; its
  // place in the fields and in a row buffer
  const T *hsrc[KH], *hsrq[KH];
  int hl[KH];
#pragma unroll
  for (int k = 0; k < KH; ++k) {
    const int it = tid + k * NT;
    const int rf = it / N, z = it - rf * N, r = rf / NF, f = rf - r * NF;
    const int yy = r == 0 ? (y0 - 1 + N) % N : (y0 + BY) % N;
    hsrc[k] = (f == 0 ? A.src[0] : A.src[NF - 1]) + (size_t)yy * N + z;
    hsrq[k] = (f == 0 ? A.src[2] : A.src[2 + NF - 1]) + (size_t)yy * N + z;
    hl[k] = active && it < NHI ? f * fst * W + (r == 0 ? 0 : BY + 1) * N + z : -1;
  }

  auto at = [&](const T* base, size_t o) {
    return *reinterpret_cast<const __attribute__((address_space(1))) VW*>(
        (const __attribute__((address_space(1))) T*)base + o);
  };
  auto store = [&](const VW& v, T* base, size_t o) {
    __builtin_nontemporal_store(v, reinterpret_cast<__attribute__((address_space(1))) VW*>(
                                       (__attribute__((address_space(1))) T*)base + o));
  };
  auto load_own = [&](int x, VW (&p)[NF], VW (&pq)[NF]) {
    if (!active) return;
    const size_t o = (size_t)x * NN + (size_t)y * N + W * tz;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      p[f] = at(A.src[f], o);
      pq[f] = at(A.src[2 + f], o);
    }
  };
  auto load_halo = [&](int x) {
#pragma unroll
    for (int k = 0; k < KH; ++k) {
      if (hl[k] >= 0) {
        hp[k] = load_g(hsrc[k], (size_t)x * NN);
        if constexpr (!FULL) hq[k] = load_g(hsrq[k], (size_t)x * NN);
      }
    }
  };

  // prologue: planes x0-1 (drifted, into buffer 1), x0 (drifted, into
  // buffer 0 with its halo), x0+1 (raw, in flight)
  const int xm = (x0 - 1 + N) % N;
  VW pm[NF];
  load_own(xm, pm, qf);  // qf: momentum of plane x0-1, only needed for its drift
  double a_in, b_in;
  get_ab(a_in, b_in);
  load_own(x0, pc, qc);
  load_halo(x0);
  load_own((x0 + 1) % N, pn, qn);
  const double anew = A.expand ? a_in + A.pd.wd * A.h * b_in : a_in;
  const double amid = 0.5 * (a_in + anew);
  const Coef<T> cdrift = ucoef<T>(A.pd.wd * A.h * apow(amid, -(3.0 - A.alpha)));
  const Coef<T> clap = ucoef<T>(apow(anew, 1.0 + A.alpha) / (A.dx * A.dx));
  const Coef<T> cpot = ucoef<T>(apow(anew, 3.0 + A.alpha));
  auto drift = [&](const VW& qv, const VW& pv) {
    if constexpr (FULL) return pv;
    VW r;
#pragma unroll
    for (int e = 0; e < W; ++e) r[e] = fma_c(cdrift, qv[e], pv[e]);
    return r;
  };
  // the drifted plane into LDS buffer b: own rows from registers, halo rows
  // drifted here
  auto store_lds = [&](int b) {
    if (!active) return;
#pragma unroll
    for (int f = 0; f < NF; ++f) lds[b * bst + f * fst + own] = pc[f];
    T* const row = reinterpret_cast<T*>(lds + b * bst);
#pragma unroll
    for (int k = 0; k < KH; ++k)
      if (hl[k] >= 0) row[hl[k]] = FULL ? hp[k] : fma_c(cdrift, hq[k], hp[k]);
  };
  if (active) {
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      lds[bst + f * fst + own] = drift(qf[f], pm[f]);
      pc[f] = drift(qc[f], pc[f]);
    }
  }
  store_lds(0);

  // One plane (x = x0 + i, in buffer B = i & 1); called twice per trip with
  // the register sets swapped (see the general tile): (pn, qn) hold raw plane
  // x+1, plane x+2 is loaded into (pf, qf), the halo rows of x+1 into (hp, hq).
  auto plane = [&](int i, auto bsel, VW (&pn)[NF], VW (&qn)[NF], VW (&pf)[NF], VW (&qf)[NF]) {
    constexpr int B = decltype(bsel)::value;
    const int x = x0 + i;
    if (i + 1 < XC) {
      load_own((x + 2) % N, pf, qf);
      load_halo((x + 1) % N);
    }
    __syncthreads();
    if (active) {
      const size_t o = (size_t)x * NN + (size_t)y * N + W * tz;
      // plane x+1 drifted, in place
#pragma unroll
      for (int f = 0; f < NF; ++f) pn[f] = drift(qn[f], pn[f]);
      if constexpr (FULL) {
        const T half = T(0.5), quarter = T(0.25);
        const T m2_0 = (T)A.m2_0, m2_1 = (T)A.m2_1, lam = (T)A.lam, q = (T)A.q;
#pragma unroll
        for (int e = 0; e < W; ++e) {
          const T p2 = pc[0][e] * pc[0][e];
          if constexpr (NF > 1) {
            const T c2 = pc[1][e] * pc[1][e];
            acc[5 * NF + 0] += (double)(half * (m2_0 * p2 + m2_1 * c2));
            acc[5 * NF + 2] += (double)(half * q * p2 * c2);
          } else {
            acc[5 * NF + 0] += (double)(half * m2_0 * p2);
          }
          acc[5 * NF + 1] += (double)(quarter * lam * p2 * p2);
        }
      } else {
#pragma unroll
        for (int e = 0; e < W; ++e) {
          const T p2 = pc[0][e] * pc[0][e];
          T v = p2 * fma_t(qlam, p2, hm2_0);
          if constexpr (NF > 1) {
            const T c2 = pc[1][e] * pc[1][e];
            v = fma_t(c2, fma_t(hqq, p2, hm2_1), v);
          }
          acc[3] += (double)v;
        }
      }
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        const VW* const pl = lds + B * bst + f * fst;
        const VW xm4 = lds[(1 - B) * bst + f * fst + own];
        const VW yp = pl[own + NL], ym = pl[own - NL];
        // the z-neighbours outside the lane's sites
        const T zlo = reinterpret_cast<const T*>(pl)[zl];
        const T zhi = reinterpret_cast<const T*>(pl)[zh];
        VW pout;
#pragma unroll
        for (int e = 0; e < W; ++e) {
          T cur[NF];
#pragma unroll
          for (int g = 0; g < NF; ++g) cur[g] = pc[g][e];
          const T c = cur[f];
          const T zp = e == W - 1 ? zhi : pc[f][e + 1];
          const T zm = e == 0 ? zlo : pc[f][e - 1];
          const T pin = qc[f][e];
          T pe = pin;
          if constexpr (MODE != kRowsObsSync) {
            // the general tile's Laplacian, term for term
            const T lap = ((xm4[e] - c) + (pn[f][e] - c)) + ((yp[e] - c) + (ym[e] - c)) + ((zp - c) + (zm - c));
            const T K = fma_c(clap, lap, -mul_c(cpot, dpot<T, NF>(f, cur, m2_0c, m2_1c, lamc, qc_)));
            pout[e] = fma_c(ckick, K, pin);
            pe = fma_c(cE, K, pin);
          }
          const T gx = pn[f][e] - c, gy = yp[e] - c, gz = zp - c;
          if constexpr (FULL) {
            acc[5 * f + 0] += (double)(pin * pin);
            acc[5 * f + 1] += (double)(pe * pe);
            acc[5 * f + 2] += (double)(gx * gx + gy * gy + gz * gz);
            acc[5 * f + 3] += (double)c;
            acc[5 * f + 4] += (double)(c * c);
          } else {
            acc[1] += (double)(pe * pe);
            acc[2] += (double)(gx * gx + gy * gy + gz * gz);
          }
        }
        if constexpr (!FULL) {
          if (lf) {
#pragma unroll
            for (int e = 0; e < W; ++e) acc[0] += (double)(qc[f][e] * qc[f][e]);
          }
          // streaming stores of the new state (read again only by the next pass)
          store(pc[f], A.dst[f], o);
          store(pout, A.dst[2 + f], o);
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      pc[f] = pn[f];
      qc[f] = qn[f];
    }
    // plane x+1 into the buffer of x-1, which no lane reads any more
    if (i + 1 < XC) store_lds(1 - B);
  };
  for (int i = 0; i < XC; i += 2) {
    plane(i, std::integral_constant<int, 0>{}, pn, qn, pf, qf);
    if (i + 1 < XC) plane(i + 1, std::integral_constant<int, 1>{}, pf, qf, pn, qn);
  }
  rows_partials<NACC>(A.partials, acc, pidx);
}

// Blocks of up to 768 lanes: at 168 VGPRs or fewer twelve waves share a CU.
template <typename T, int W, int NF, int BY, int MODE = kRowsStep>
__global__ __launch_bounds__(kRowsMaxThreads) void scalar_rows_kernel(ScalarArgs<T> A) {
  int bid = blockIdx.x;
  if (A.swizzle) bid = xcd_tile(bid, gridDim.x);
  auto get_ab = [&](double& a_in, double& b_in) {
    if (A.prev.partials) {
      constexpr int NP = Acc<NF, false>::N;
      __shared__ double ab[2];
      double S[NP];
      if (rows_reduce_partials<NP>(A.prev.partials, 0, A.prev.nblocks, S)) {
        double an, bn;
        finish_state<T, NF, false>(A, A.prev.pd, A.st, S, blockIdx.x == 0 ? A.prev.out : nullptr, an, bn);
        ab[0] = an;
        ab[1] = bn;
      }
      __syncthreads();
      a_in = ab[0];
      b_in = ab[1];
    } else {
      a_in = A.st->a;
      b_in = A.st->b;
    }
  };
  scalar_rows<T, W, NF, (2 * NF * W + BY - 1) / BY, false, MODE>(A, BY, bid, blockIdx.x, get_ab);
}

}  // namespace cl
