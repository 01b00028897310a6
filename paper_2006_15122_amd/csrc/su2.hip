// Doublet with SU(2) x U(1) gauge links on gfx950 (Sec. 6: staggered
// leapfrog, velocity Verlet and its Yoshida compositions; initial state
// Sec. 7.2).  Every pass of the shared schedule is one kernel, drift and kick
// in one sweep from one state buffer into the other with per-block FP64
// partial sums, whose finish (a and b) the next pass of a chain applies.
//
// Components (storage precision, N^3 each):
//   0..3   Phi = (Phi_0, Phi_1) as Re Phi_0, Im Phi_0, Re Phi_1, Im Phi_1
//          (Phi_c = (phi_2c + i phi_2c+1)/sqrt 2)
//   4..7   pi_Phi, same layout
//   8..10  phase th_i of the U(1) link V_i = exp(i th_i)
//   11..13 pi_A,i
//   14+4i+k  SU(2) link U_i = c0 + i c.sigma as (c0, c1, c2, c3)
//   26+3i+a  pi_B,i along T_a = sigma_a/2
// Kernels (forces of the lattice energies, the electric fields generating
// left multiplication of the links, U' = -i g dx pi_B U / a^{1-alpha}):
//   K_Phi   = a^{1+alpha} sum_i (W_i Phi_{+i} - 2 Phi + W_i(n-i)^dag Phi_{-i})/dx^2
//             - a^{3+alpha}(2 lambda |Phi|^2 + m2) Phi,   W_i = V_i U_i
//   K_A,i   = a^{1+alpha}(2e/dx)(f/w)^2 Im[Phi^dag W_i Phi_{+i}]
//             + a^{alpha-1}/(e dx^3) sum_{j!=i}(Im V_ij(n) - Im V_ij(n-j))
//   K_B,i^a = a^{1+alpha}(g/dx)(f/w)^2 Im[Phi^dag sigma_a W_i Phi_{+i}]
//             + a^{alpha-1} 2/(g dx^3) sum_{j!=i}(c_a[U_ij(n)] - c_a[U_j(n-j)^dag U_ij(n-j) U_j(n-j)])
// with c_a the vector part of an SU(2) element.  SU(2) elements are carried
// as quaternions (w, x, y, z) = w + i(x sigma_1 + y sigma_2 + z sigma_3).
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "common.hpp"
#include "internal.hpp"
#include "phase.hpp"

namespace cl {

constexpr int kSu2Comp = 35;
constexpr int kPH = 0, kPI = 4, kTH = 8, kPA = 11, kUL = 14, kPB = 26;
constexpr int kSu2Acc = 16;  // the workspace reserves 16 FP64 partials per 256-site block
constexpr int kSu2GaussAcc = 6;

// (aligned so that a quaternion moves as one 16-byte LDS access in FP32)
template <typename T>
struct alignas(16) Q4 {
  T w, x, y, z;
};
template <typename T>
struct Cx2 {
  T re, im;
};

template <typename T>
__device__ __forceinline__ Q4<T> qmul(const Q4<T>& a, const Q4<T>& b) {
  // (a0 + i a.s)(b0 + i b.s) = a0 b0 - a.b + i (a0 b + b0 a - a x b).s
  return Q4<T>{a.w * b.w - (a.x * b.x + a.y * b.y + a.z * b.z),
               a.w * b.x + b.w * a.x - (a.y * b.z - a.z * b.y),
               a.w * b.y + b.w * a.y - (a.z * b.x - a.x * b.z),
               a.w * b.z + b.w * a.z - (a.x * b.y - a.y * b.x)};
}
template <typename T>
__device__ __forceinline__ Q4<T> qdag(const Q4<T>& a) {
  return Q4<T>{a.w, -a.x, -a.y, -a.z};
}
template <typename T>
__device__ __forceinline__ Cx2<T> cmul2(Cx2<T> a, Cx2<T> b) {
  return Cx2<T>{a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
template <typename T>
__device__ __forceinline__ Cx2<T> cadd2(Cx2<T> a, Cx2<T> b) {
  return Cx2<T>{a.re + b.re, a.im + b.im};
}
template <typename T>
__device__ __forceinline__ Cx2<T> csub2(Cx2<T> a, Cx2<T> b) {
  return Cx2<T>{a.re - b.re, a.im - b.im};
}
// the 2x2 matrix of (w, x, y, z) minus w1 times the identity, applied to a
// doublet: [[w - w1 + i z, y + i x], [-y + i x, w - w1 - i z]] (w1 = 0: the
// element itself, w1 = 1: the element minus one)
template <typename T>
__device__ __forceinline__ void qapply(const Q4<T>& q, T wm, const Cx2<T> (&v)[2], Cx2<T> (&o)[2]) {
  o[0] = cadd2(cmul2(Cx2<T>{wm, q.z}, v[0]), cmul2(Cx2<T>{q.y, q.x}, v[1]));
  o[1] = cadd2(cmul2(Cx2<T>{-q.y, q.x}, v[0]), cmul2(Cx2<T>{wm, -q.z}, v[1]));
}
// w - 1 of a unit quaternion without cancellation: -|v|^2/(1 + w) for w > 0
template <typename T>
__device__ __forceinline__ T qw_m1(const Q4<T>& q) {
  const T v2 = q.x * q.x + q.y * q.y + q.z * q.z;
  return q.w > T(0) ? -quot_t(v2, T(1) + q.w) : q.w - T(1);
}
// Im(conj(a) b), Re(conj(a) b)
template <typename T>
__device__ __forceinline__ T cross_im(Cx2<T> a, Cx2<T> b) { return a.re * b.im - a.im * b.re; }
template <typename T>
__device__ __forceinline__ T dot_re(Cx2<T> a, Cx2<T> b) { return a.re * b.re + a.im * b.im; }

__device__ __forceinline__ float rsqrt_s(float x) { return rsqrtf(x); }
__device__ __forceinline__ double rsqrt_s(double x) { return 1.0 / sqrt(x); }

template <typename T>
__device__ __forceinline__ T wrap_turns(T t) {
  const T twopi = (T)6.283185307179586476925286766559;
  return t - twopi * rint(t * (T)0.15915494309189533576888376337251);
}

template <typename T>
struct Su2Args {
  const T* src[kSu2Comp];
  T* dst[kSu2Comp];
  int N;
  double dx, alpha, fmp2, lam, m2, e, g, wf2, h;
  int expand;
  PassDesc pd;
  double* partials;
  DevState* st;
};

// per-block sums of 256 threads' accumulators (waves in order) into the block's record
template <int NACC>
__device__ void su2_block_partials(double (&acc)[NACC], double* partials) {
  __shared__ double red[4][NACC];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
#pragma unroll
  for (int k = 0; k < NACC; ++k) {
    const double s = wave_sum(acc[k]);
    if (lane == 0) red[wv][k] = s;
  }
  __syncthreads();
  if (tid < NACC) partials[(size_t)blockIdx.x * NACC + tid] = ((red[0][tid] + red[1][tid]) + red[2][tid]) + red[3][tid];
}

// ---------------------------------------------------------------------------
// The pass kernel: drift and kick of one pass in one sweep.
//
// A block owns a TY x TZ tile of the (y, z) plane and marches along x over its
// share of planes.  Each plane enters LDS drifted (Phi, the U(1) phases and the SU(2)
// links of the tile and a one-site ring with corners); planes x and x+1 are
// held.
//
// Every site computes each of its three plaquettes once, P_ij(n) = U_i(n)
// U_j(n+i) U_i(n+j)^dag U_j(n)^dag, and hands the forces of the neighbours on:
// the backward plaquettes a link force needs are the same P seen from one site
// further, U_j(m)^dag P_ij(m) U_j(m) at n = m + j for link i and
// U_i(m)^dag P_ij(m) U_i(m) at n = m + i for link j, i.e. rotations of P's
// vector part.  The parallel-transported doublet W_d(m)^dag Phi(m) goes the same
// way, so each link's sine and cosine are formed once.  What goes to x+1 stays
// in registers, what goes to y+1 and z+1 passes through LDS; the
// row y0-1 and the column z0-1 are computed by the waves without ring sites.
//
// Bound by its instruction stream: about 1600 VALU instructions a wave and
// plane (46% of the issue slots at two waves per SIMD, which 247 VGPRs and
// 79 KB of LDS per block allow).  In FP32 a pass takes 209 us at 128^3, 34 us
// at 64^3 and 631 us at 192^3; a pointwise drift and a kick that read every
// neighbour's links from memory took 484, 67 and 1560 us.  Ring threads in
// waves of their own (six waves a block at 168 VGPRs) left one block on a CU
// and spilled: 395 us.  FP64 takes half the tile so that a block's planes fit
// (64^3: 122 us against 137, 96^3: 326 against 550).
// ---------------------------------------------------------------------------
template <typename T>
struct Su2PassArgs {
  const T* src;  // component c at src + c N^3
  T* dst;
  int N, nx;  // nx blocks along x
  double dx, alpha, fmp2, lam, m2, e, g, wf2, h;
  int expand;
  PassDesc pd;
  double* partials;
  DevState* st;
  PrevPass prev;  // finish of the previous pass of a chain (partials == nullptr: none)
};

// Sums of a stepping pass: pi_Phi^2, |W Phi_+ - Phi|^2, V, pi_A^2, 1 - cos Phi_ij,
// pi_B^2, 1 - Tr U_ij/2 (LF: in and out of the kick added).  Observation passes
// keep the kSu2Acc sums of the table above.
constexpr int kSu2StepAcc = 7;

// U^dag (i v.sigma) U as a vector: (w^2 - |q|^2) v + 2 (v.q) q - 2 w (v x q)
template <typename T>
struct V3 {
  T x, y, z;
};
template <typename T>
__device__ __forceinline__ V3<T> qrotate(const Q4<T>& u, const Q4<T>& p) {
  const T s = u.w * u.w - (u.x * u.x + u.y * u.y + u.z * u.z);
  const T d = T(2) * (p.x * u.x + p.y * u.y + p.z * u.z), w2 = T(2) * u.w;
  return V3<T>{s * p.x + d * u.x - w2 * (p.y * u.z - p.z * u.y), s * p.y + d * u.y - w2 * (p.z * u.x - p.x * u.z),
               s * p.z + d * u.z - w2 * (p.x * u.y - p.y * u.x)};
}

template <typename T, bool OBS>
__device__ void su2_finish_state(const Su2PassArgs<T>& A, const PassDesc& pd, const DevState* in, const double* S,
                                 DevState* out, double& a_next, double& b_next);
template <int NACC, int NT>
__device__ bool su2_reduce_records(const double* rec, int nb, double (&S)[NACC]);

// one site's raw components
template <typename T>
struct Su2Raw {
  T ph[4], pi[4], th[3], pa[3], pb[9];
  Q4<T> u[3];
};

template <int TZ, int TY>
struct Su2Tile {
  static constexpr int NT = TZ * TY, LY = TY + 2, LZ = TZ + 2;
  static constexpr int NR = 2 * LZ + 2 * TY;  // ring sites
};

template <typename T, int TZ, int TY, int WPE, int MODE>
__global__ __launch_bounds__(TZ* TY, WPE) void su2_pass_kernel(Su2PassArgs<T> A) {
  constexpr bool OBS = MODE == kPassObs;
  using Tile = Su2Tile<TZ, TY>;
  constexpr int LY = Tile::LY, LZ = Tile::LZ, NR = Tile::NR, NT = Tile::NT;
  constexpr int NACC = OBS ? kSu2Acc : kSu2StepAcc;
  static_assert(NR <= NT, "one ring site per thread");
  // first thread of the row y0-1 and of the column z0-1: waves that own no
  // ring site (where the block has four)
  constexpr int ROW0 = NT >= 256 ? 128 : 0, COL0 = NT >= 256 ? 192 : 64;
  static_assert(ROW0 + TZ <= COL0 && COL0 + TY <= NT, "row and column in different threads");
  __shared__ Q4<T> LU[2][3][LY][LZ];  // drifted SU(2) links
  __shared__ Q4<T> LP[2][LY][LZ];     // drifted Phi (re0, im0, re1, im1)
  __shared__ T Lt[2][3][LY][LZ];      // drifted U(1) phases
  // handed on to y+1 (0) and z+1 (1), at the receiver's place: (W^dag - 1) Phi,
  // two rotated plaquettes, two plaquette sines
  __shared__ Q4<T> Bh[2][TY][TZ];
  __shared__ T Bv[2][8][TY][TZ];
  __shared__ double red[NT / 64][NACC];

  const int N = A.N;
  const unsigned NN = (unsigned)N * N;
  const size_t V = (size_t)NN * N;
  const int tid = threadIdx.x;
  const int bid = xcd_tile(blockIdx.x, gridDim.x);
  const int nzt = N / TZ, nyt = N / TY;
  const int z0 = (bid % nzt) * TZ, y0 = ((bid / nzt) % nyt) * TY, xb = bid / (nzt * nyt),
            x0 = x_first(N, xb, A.nx), XC = x_first(N, xb + 1, A.nx) - x0;

  // places in the LDS tile of this thread's site and of its ring site
  const int tz = tid % TZ, ty = tid / TZ, ly = 1 + ty, lz = 1 + tz;
  const bool has_ring = tid < NR;
  int rly, rlz;
  if (tid < LZ) { rly = 0; rlz = tid; }
  else if (tid < 2 * LZ) { rly = TY + 1; rlz = tid - LZ; }
  else if (tid < 2 * LZ + TY) { rly = 1 + tid - 2 * LZ; rlz = TZ + 1; }
  else { rly = 1 + tid - 2 * LZ - TY; rlz = 0; }
  const unsigned plane = NN * (unsigned)sizeof(T);
  auto column = [&](int y, int z) -> unsigned {
    return ((unsigned)((y0 - 1 + y + N) % N) * N + (unsigned)((z0 - 1 + z + N) % N)) * (unsigned)sizeof(T);
  };
  const unsigned col = column(ly, lz), rcol = has_ring ? column(rly, rlz) : 0u;
  const bool low_row = tid >= ROW0 && tid < ROW0 + TZ, low_col = tid >= COL0 && tid < COL0 + TY;

  // Component c of the state through an address that steps from one component
  // to the next and is opaque to the compiler: 70 bases kept across the loop
  // overflow the scalar registers, and formed from the component number they
  // become 64-bit vector arithmetic, three instructions a load.  FP32 steps a
  // scalar base; FP64, whose constants fill the scalar registers, a vector one:
  // with 55 scalar registers spilled the compiler split live ranges where a
  // branch joins, ahead of the restored lane mask, and the lanes outside the
  // branch lost their LDS addresses (the build refuses such code).
  struct Walk {
    GlobalPtr<const char> p;
    size_t st;
    __device__ __forceinline__ Walk(const T* base, size_t V) : p((GlobalPtr<const char>)base), st(V * sizeof(T)) {
      hide();
    }
    __device__ __forceinline__ GlobalPtr<T> next(unsigned o) {
      const GlobalPtr<const char> q = p;
      p += st;
      hide();
      return at_offset<T>(q, o);
    }
    __device__ __forceinline__ void hide() {
      if constexpr (sizeof(T) == 4) asm volatile("" : "+s"(p));
      else asm volatile("" : "+v"(p));
    }
  };
  Su2Raw<T> raw, rraw;
  auto load_site = [&](Su2Raw<T>& w, unsigned o) {
    Walk c(A.src, V);
#pragma unroll
    for (int k = 0; k < 4; ++k) w.ph[k] = *c.next(o);
#pragma unroll
    for (int k = 0; k < 4; ++k) w.pi[k] = *c.next(o);
#pragma unroll
    for (int i = 0; i < 3; ++i) w.th[i] = *c.next(o);
#pragma unroll
    for (int i = 0; i < 3; ++i) w.pa[i] = *c.next(o);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      w.u[i].w = *c.next(o);
      w.u[i].x = *c.next(o);
      w.u[i].y = *c.next(o);
      w.u[i].z = *c.next(o);
    }
#pragma unroll
    for (int k = 0; k < 9; ++k) w.pb[k] = *c.next(o);
  };
  auto load_own = [&](int x) { load_site(raw, (unsigned)x * plane + col); };
  auto load_ring = [&](int x) {
    if (has_ring) load_site(rraw, (unsigned)x * plane + rcol);
  };
  // the first plane's loads need no coefficients: their latency overlaps the
  // previous pass's finish
  load_own((x0 - 1 + N) % N);

  double a_in, b_in;
  if (A.prev.partials) {
    __shared__ double ab[2];
    double S[kSu2StepAcc];
    if (su2_reduce_records<kSu2StepAcc, NT>(A.prev.partials, A.prev.nblocks, S)) {
      double an, bn;
      su2_finish_state<T, false>(A, A.prev.pd, A.st, S, blockIdx.x == 0 ? A.prev.out : nullptr, an, bn);
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
  const double hw = A.pd.wd * A.h;
  const double anew = A.expand ? a_in + hw * b_in : a_in;
  const double amid = 0.5 * (a_in + anew);
  // per-pass coefficients as hi + lo pairs (no coherent rounding of them)
  const double p1 = apow(amid, 1.0 - A.alpha), pl = apow(anew, 1.0 + A.alpha), pb = apow(anew, A.alpha - 1.0);
  const double dx3 = A.dx * A.dx * A.dx;
  // (FP64 keeps them in vector registers, of which one wave per SIMD has plenty:
  // in scalar ones they overflow that file)
  auto uc = [](double v) -> Coef<T> {
    if constexpr (sizeof(T) == 8) return coef<T>(v);
    else return ucoef<T>(v);
  };
  const Coef<T> cd = uc(hw * apow(amid, -(3.0 - A.alpha)));
  const Coef<T> cu = uc(A.e * hw * A.dx / (2.0 * p1));
  const Coef<T> cw = uc(A.g * hw * A.dx / (4.0 * p1));
  const Coef<T> cl = uc(pl / (A.dx * A.dx));
  const Coef<T> cp = uc(apow(anew, 3.0 + A.alpha));
  const Coef<T> cjA = uc(pl * 2.0 * A.e / A.dx / A.wf2);
  const Coef<T> cjB = uc(pl * A.g / A.dx / A.wf2);
  const Coef<T> cbA = uc(pb / (A.e * dx3));
  const Coef<T> cbB = uc(pb * 2.0 / (A.g * dx3));
  const Coef<T> ck = uc((A.pd.wk1 + A.pd.wk2) * A.h);
  const Coef<T> cE = uc((A.pd.mode == MODE_LF ? A.pd.wk1 + A.pd.wk2 : A.pd.wk1) * A.h);
  const T lam = (T)A.lam, m2 = (T)A.m2;
  const Coef<T> lam2c = uc(2.0 * A.lam), m2c = uc(A.m2);
  const bool lf = A.pd.mode == MODE_LF;

  // Drift of the raw site into LDS buffer b (Sec. 6.2.1 and 6.2.2):
  //   Phi += wd h pi / a_mid^{3-alpha};
  //   V   <- (1 - i u)/(1 + i u) V,  u = e wd h dx pi_A / (2 a_mid^{1-alpha}), as th -= 2 atan u;
  //   U   <- ((1 - |w|^2) - 2 i w.sigma)/(1 + |w|^2) U,  w = g wd h dx pi_B / (4 a_mid^{1-alpha}),
  // U renormalised to unit length after the product (rounding only).  A pass
  // without drift leaves the links as they are.
  auto drift_site = [&](const Su2Raw<T>& w, int b, int y, int z) {
    if constexpr (MODE != kPassStep) {
      LP[b][y][z] = Q4<T>{w.ph[0], w.ph[1], w.ph[2], w.ph[3]};
#pragma unroll
      for (int i = 0; i < 3; ++i) { Lt[b][i][y][z] = w.th[i]; LU[b][i][y][z] = w.u[i]; }
      return;
    }
    LP[b][y][z] = Q4<T>{fma_c(cd, w.pi[0], w.ph[0]), fma_c(cd, w.pi[1], w.ph[1]), fma_c(cd, w.pi[2], w.ph[2]),
                        fma_c(cd, w.pi[3], w.ph[3])};
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      Lt[b][i][y][z] = wrap_turns(w.th[i] - T(2) * atan_t(mul_c(cu, w.pa[i])));
      const T w0 = mul_c(cw, w.pb[3 * i]), w1 = mul_c(cw, w.pb[3 * i + 1]), w2 = mul_c(cw, w.pb[3 * i + 2]);
      const T ww = w0 * w0 + w1 * w1 + w2 * w2;
      // (1 + |w|^2) C U; the factor goes with the normalisation
      const Q4<T> n = qmul(Q4<T>{T(1) - ww, T(-2) * w0, T(-2) * w1, T(-2) * w2}, w.u[i]);
      const T r = rsqrt_s(n.w * n.w + n.x * n.x + n.y * n.y + n.z * n.z);
      LU[b][i][y][z] = Q4<T>{n.w * r, n.x * r, n.y * r, n.z * r};
    }
  };
  auto drift_into = [&](int b) {
    drift_site(raw, b, ly, lz);
    if (has_ring) drift_site(rraw, b, rly, rlz);
  };
  auto phi_at = [&](int b, int y, int z, Cx2<T> (&p)[2]) {
    const Q4<T> v = LP[b][y][z];
    p[0] = Cx2<T>{v.w, v.x};
    p[1] = Cx2<T>{v.y, v.z};
  };
  // (W^dag - 1) Phi = (U^dag - 1) y' + (conj V - 1) Phi, y' = conj(V) Phi, from (sin, cos - 1) of V's phase
  auto back = [&](const Q4<T>& u, T sn, T cm, const Cx2<T> (&p)[2]) -> Q4<T> {
    Cx2<T> vf[2], y[2], o[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      vf[k] = cmul2(Cx2<T>{cm, -sn}, p[k]);
      y[k] = cadd2(p[k], vf[k]);
    }
    const Q4<T> ud = qdag(u);
    qapply(ud, qw_m1(ud), y, o);
    const Cx2<T> a = cadd2(o[0], vf[0]), b = cadd2(o[1], vf[1]);
    return Q4<T>{a.re, a.im, b.re, b.im};
  };
  // (sin, cos - 1) of a link's or plaquette's phase: a drift wraps the links to
  // one turn; stored phases (a caller may write any) are any number
  auto sincos_link = [](T x, T* sn, T* cm) {
    if constexpr (MODE == kPassStep) sincos_m1_near(x, sn, cm);
    else sincos_m1_any(x, sn, cm);
  };
  // plaquettes of place (y, z) of plane buffer c (plane x+1 in buffer n)
  auto plB = [&](const Q4<T>& ua, const Q4<T>& ubf, const Q4<T>& ub, const Q4<T>& uaf) -> Q4<T> {
    return qmul(qmul(ua, ubf), qdag(qmul(ub, uaf)));
  };
  auto plA = [&](T ta, T tbf, T taf, T tb, T& om) -> T {
    T sn, cm;
    sincos_link((ta + tbf) - (taf + tb), &sn, &cm);
    om = -cm;  // 1 - cos Phi
    return sn;
  };

  double acc[NACC];
#pragma unroll
  for (int k = 0; k < NACC; ++k) acc[k] = 0.0;
  // handed on from plane x-1 of the own column
  Q4<T> hx{T(0), T(0), T(0), T(0)}, pxm = hx;
  V3<T> rx01{T(0), T(0), T(0)}, rx02 = rx01;
  T sx01 = T(0), sx02 = T(0);
  T qc[16], qn[16];
  auto momenta = [&](T (&q)[16]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) q[k] = raw.pi[k];
#pragma unroll
    for (int k = 0; k < 3; ++k) q[4 + k] = raw.pa[k];
#pragma unroll
    for (int k = 0; k < 9; ++k) q[7 + k] = raw.pb[k];
  };

  // prologue: plane x0-1 -> buffer 1, plane x0 -> buffer 0, what x0-1 hands on, plane x0+1 -> buffer 1
  load_ring((x0 - 1 + N) % N);
  drift_into(1);
  load_own(x0);
  load_ring(x0);
  drift_into(0);
  momenta(qc);
  __syncthreads();
  load_own((x0 + 1) % N);
  {
    T om;
    const Q4<T> u0 = LU[1][0][ly][lz];
    rx01 = qrotate(u0, plB(u0, LU[0][1][ly][lz], LU[1][1][ly][lz], LU[1][0][ly + 1][lz]));
    rx02 = qrotate(u0, plB(u0, LU[0][2][ly][lz], LU[1][2][ly][lz], LU[1][0][ly][lz + 1]));
    sx01 = plA(Lt[1][0][ly][lz], Lt[0][1][ly][lz], Lt[1][0][ly + 1][lz], Lt[1][1][ly][lz], om);
    sx02 = plA(Lt[1][0][ly][lz], Lt[0][2][ly][lz], Lt[1][0][ly][lz + 1], Lt[1][2][ly][lz], om);
    T sn, cm;
    sincos_link(Lt[1][0][ly][lz], &sn, &cm);
    Cx2<T> p[2];
    phi_at(1, ly, lz, p);
    hx = back(u0, sn, cm, p);
    pxm = LP[1][ly][lz];
  }
  load_ring((x0 + 1) % N);
  __syncthreads();
  drift_into(1);
  momenta(qn);
  __syncthreads();

  for (int i = 0; i < XC; ++i) {
    const int x = x0 + i, c = i & 1, n = c ^ 1;
    // ---- what every site of plane x computes once
    Cx2<T> lap[2];
    T eg = T(0), curA[3], curB[3][3], magA[3], magB[3][3], omA = T(0), omB = T(0);
    {
      Cx2<T> p[2];
      phi_at(c, ly, lz, p);
      const Q4<T> u0 = LU[c][0][ly][lz], u1 = LU[c][1][ly][lz], u2 = LU[c][2][ly][lz];
      const T t0 = Lt[c][0][ly][lz], t1 = Lt[c][1][ly][lz], t2 = Lt[c][2][ly][lz];
      // backward neighbour along x: W^dag Phi_- - Phi
      lap[0] = Cx2<T>{hx.w + (pxm.w - p[0].re), hx.x + (pxm.x - p[0].im)};
      lap[1] = Cx2<T>{hx.y + (pxm.y - p[1].re), hx.z + (pxm.z - p[1].im)};
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const Q4<T>& u = d == 0 ? u0 : d == 1 ? u1 : u2;
        T sn, cm;
        sincos_link(d == 0 ? t0 : d == 1 ? t1 : t2, &sn, &cm);
        Cx2<T> fp[2], um1f[2], g[2];
        phi_at(d == 0 ? n : c, ly + (d == 1), lz + (d == 2), fp);
        // W Phi_+ - Phi = (V - 1) y + (U - 1) Phi_+ + (Phi_+ - Phi),  y = U Phi_+
        qapply(u, qw_m1(u), fp, um1f);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const Cx2<T> y = cadd2(fp[k], um1f[k]);
          g[k] = cadd2(cadd2(cmul2(Cx2<T>{cm, sn}, y), um1f[k]), csub2(fp[k], p[k]));
          lap[k] = cadd2(lap[k], g[k]);
        }
        eg += g[0].re * g[0].re + g[0].im * g[0].im + g[1].re * g[1].re + g[1].im * g[1].im;
        // currents Im[Phi^dag g], Im[Phi^dag sigma_a g] (Im[Phi^dag sigma Phi] = 0)
        curA[d] = cross_im(p[0], g[0]) + cross_im(p[1], g[1]);
        curB[d][0] = cross_im(p[0], g[1]) + cross_im(p[1], g[0]);
        curB[d][1] = -dot_re(p[0], g[1]) + dot_re(p[1], g[0]);
        curB[d][2] = cross_im(p[0], g[0]) - cross_im(p[1], g[1]);
        const Q4<T> hb = back(u, sn, cm, p);
        if (d == 0) hx = hb;
        if (d == 1 && ty + 1 < TY) Bh[0][ty + 1][tz] = hb;
        if (d == 2 && tz + 1 < TZ) Bh[1][ty][tz + 1] = hb;
      }
      pxm = LP[c][ly][lz];
      auto to_y = [&](int k, T v) { if (ty + 1 < TY) Bv[0][k][ty + 1][tz] = v; };
      auto to_z = [&](int k, T v) { if (tz + 1 < TZ) Bv[1][k][ty][tz + 1] = v; };
      {
        T o01, o02, o12;
        const T S01 = plA(t0, Lt[n][1][ly][lz], Lt[c][0][ly + 1][lz], t1, o01);
        const T S02 = plA(t0, Lt[n][2][ly][lz], Lt[c][0][ly][lz + 1], t2, o02);
        const T S12 = plA(t1, Lt[c][2][ly + 1][lz], Lt[c][1][ly][lz + 1], t2, o12);
        omA = o01 + o02 + o12;
        magA[0] = S01 + S02;
        magA[1] = (sx01 - S01) + S12;
        magA[2] = (sx02 - S02) - S12;
        sx01 = S01;
        sx02 = S02;
        to_y(6, S01);
        to_y(7, S12);
        to_z(6, S02);
        to_z(7, S12);
      }
      {
        const Q4<T> P = plB(u0, LU[n][1][ly][lz], u1, LU[c][0][ly + 1][lz]);
        omB += -qw_m1(P);  // 1 - w = (2 - Tr)/2
        magB[0][0] = P.x; magB[0][1] = P.y; magB[0][2] = P.z;
        magB[1][0] = rx01.x - P.x; magB[1][1] = rx01.y - P.y; magB[1][2] = rx01.z - P.z;
        rx01 = qrotate(u0, P);
        const V3<T> t = qrotate(u1, P);
        to_y(0, t.x); to_y(1, t.y); to_y(2, t.z);
      }
      {
        const Q4<T> P = plB(u0, LU[n][2][ly][lz], u2, LU[c][0][ly][lz + 1]);
        omB += -qw_m1(P);
        magB[0][0] += P.x; magB[0][1] += P.y; magB[0][2] += P.z;
        magB[2][0] = rx02.x - P.x; magB[2][1] = rx02.y - P.y; magB[2][2] = rx02.z - P.z;
        rx02 = qrotate(u0, P);
        const V3<T> t = qrotate(u2, P);
        to_z(0, t.x); to_z(1, t.y); to_z(2, t.z);
      }
      {
        const Q4<T> P = plB(u1, LU[c][2][ly + 1][lz], u2, LU[c][1][ly][lz + 1]);
        omB += -qw_m1(P);
        magB[1][0] += P.x; magB[1][1] += P.y; magB[1][2] += P.z;
        magB[2][0] -= P.x; magB[2][1] -= P.y; magB[2][2] -= P.z;
        const V3<T> t = qrotate(u2, P), r = qrotate(u1, P);
        to_z(3, t.x); to_z(4, t.y); to_z(5, t.z);
        to_y(3, r.x); to_y(4, r.y); to_y(5, r.z);
      }
    }
    if (low_row) {
      // row y0-1, place (0, 1 + rid)
      const int rid = tid - ROW0, z = 1 + rid;
      const Q4<T> u0 = LU[c][0][0][z], u1 = LU[c][1][0][z], u2 = LU[c][2][0][z];
      const Q4<T> P01 = plB(u0, LU[n][1][0][z], u1, LU[c][0][1][z]);
      const Q4<T> P12 = plB(u1, LU[c][2][1][z], u2, LU[c][1][0][z + 1]);
      const V3<T> t = qrotate(u1, P01), r = qrotate(u1, P12);
      Bv[0][0][0][rid] = t.x; Bv[0][1][0][rid] = t.y; Bv[0][2][0][rid] = t.z;
      Bv[0][3][0][rid] = r.x; Bv[0][4][0][rid] = r.y; Bv[0][5][0][rid] = r.z;
      T om;
      Bv[0][6][0][rid] = plA(Lt[c][0][0][z], Lt[n][1][0][z], Lt[c][0][1][z], Lt[c][1][0][z], om);
      Bv[0][7][0][rid] = plA(Lt[c][1][0][z], Lt[c][2][1][z], Lt[c][1][0][z + 1], Lt[c][2][0][z], om);
      T sn, cm;
      sincos_link(Lt[c][1][0][z], &sn, &cm);
      Cx2<T> p[2];
      phi_at(c, 0, z, p);
      Bh[0][0][rid] = back(u1, sn, cm, p);
    }
    if (low_col) {
      // column z0-1, place (1 + q, 0)
      const int q = tid - COL0, y = 1 + q;
      const Q4<T> u0 = LU[c][0][y][0], u1 = LU[c][1][y][0], u2 = LU[c][2][y][0];
      const Q4<T> P02 = plB(u0, LU[n][2][y][0], u2, LU[c][0][y][1]);
      const Q4<T> P12 = plB(u1, LU[c][2][y + 1][0], u2, LU[c][1][y][1]);
      const V3<T> t = qrotate(u2, P02), r = qrotate(u2, P12);
      Bv[1][0][q][0] = t.x; Bv[1][1][q][0] = t.y; Bv[1][2][q][0] = t.z;
      Bv[1][3][q][0] = r.x; Bv[1][4][q][0] = r.y; Bv[1][5][q][0] = r.z;
      T om;
      Bv[1][6][q][0] = plA(Lt[c][0][y][0], Lt[n][2][y][0], Lt[c][0][y][1], Lt[c][2][y][0], om);
      Bv[1][7][q][0] = plA(Lt[c][1][y][0], Lt[c][2][y + 1][0], Lt[c][1][y][1], Lt[c][2][y][0], om);
      T sn, cm;
      sincos_link(Lt[c][2][y][0], &sn, &cm);
      Cx2<T> p[2];
      phi_at(c, y, 0, p);
      Bh[1][q][0] = back(u2, sn, cm, p);
    }
    // what the kick takes over is complete here: without these the compiler
    // sinks its computation past the barrier and keeps the inputs instead
    auto pin = [](T& v) { asm volatile("" : "+v"(v)); };
#pragma unroll
    for (int k = 0; k < 2; ++k) { pin(lap[k].re); pin(lap[k].im); }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      pin(curA[d]);
      pin(magA[d]);
#pragma unroll
      for (int a = 0; a < 3; ++a) { pin(curB[d][a]); pin(magB[d][a]); }
    }
    pin(eg);
    pin(omA);
    pin(omB);
    __syncthreads();
    // plane x+2 is in flight during the kick (its ring after the kick's
    // registers are free); the last iteration re-reads plane x+1 (unused) so
    // that the loads are unconditional
    const int xn = i + 1 < XC ? (x + 2) % N : (x + 1) % N;
    load_ring(xn);
    load_own(xn);
    __builtin_amdgcn_sched_barrier(0);
    // ---- kick of the own sites of plane x
    {
      const unsigned o = (unsigned)x * plane + col;
      const Q4<T> pq = LP[c][ly][lz], py = LP[c][ly - 1][lz], pz = LP[c][ly][lz - 1];
      const Q4<T> hy = Bh[0][ty][tz], hz = Bh[1][ty][tz];
      const T ph[4] = {pq.w, pq.x, pq.y, pq.z};
      const T lp[4] = {lap[0].re + ((hy.w + (py.w - pq.w)) + (hz.w + (pz.w - pq.w))),
                       lap[0].im + ((hy.x + (py.x - pq.x)) + (hz.x + (pz.x - pq.x))),
                       lap[1].re + ((hy.y + (py.y - pq.y)) + (hz.y + (pz.y - pq.y))),
                       lap[1].im + ((hy.z + (py.z - pq.z)) + (hz.z + (pz.z - pq.z)))};
      const T r2 = ph[0] * ph[0] + ph[1] * ph[1] + ph[2] * ph[2] + ph[3] * ph[3];
      T kin = T(0), kin0 = T(0), ka = T(0), ka0 = T(0), kb = T(0), kb0 = T(0);
      Walk w(A.dst, V);
      auto put = [&](T v) {
        if constexpr (!OBS) __builtin_nontemporal_store(v, w.next(o));
      };
#pragma unroll
      for (int k = 0; k < 4; ++k) put(ph[k]);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        // V'(Phi) = (2 lambda |Phi|^2 + m2) Phi
        const T K = mul_c(cl, lp[k]) - mul_c(cp, fma_c(lam2c, r2 * ph[k], mul_c(m2c, ph[k])));
        const T pe = fma_c(cE, K, qc[k]);
        kin0 += qc[k] * qc[k];
        kin += pe * pe;
        put(fma_c(ck, K, qc[k]));
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int d = 0; d < 3; ++d) put(Lt[c][d][ly][lz]);
      // magnetic forces: the neighbours' shares
      magA[0] -= Bv[0][6][ty][tz] + Bv[1][6][ty][tz];
      magA[1] -= Bv[1][7][ty][tz];
      magA[2] += Bv[0][7][ty][tz];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const T K = fma_c(cbA, magA[d], mul_c(cjA, curA[d]));
        const T ain = qc[4 + d], ae = fma_c(cE, K, ain);
        ka0 += ain * ain;
        ka += ae * ae;
        put(fma_c(ck, K, ain));
      }
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const Q4<T> u = LU[c][d][ly][lz];
        put(u.w);
        put(u.x);
        put(u.y);
        put(u.z);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        magB[0][a] -= Bv[0][a][ty][tz] + Bv[1][a][ty][tz];
        magB[1][a] -= Bv[1][3 + a][ty][tz];
        magB[2][a] += Bv[0][3 + a][ty][tz];
      }
#pragma unroll
      for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          const T KB = fma_c(cbB, magB[d][a], mul_c(cjB, curB[d][a]));
          const T bin = qc[7 + 3 * d + a], be = fma_c(cE, KB, bin);
          kb0 += bin * bin;
          kb += be * be;
          put(fma_c(ck, KB, bin));
        }
      if constexpr (OBS) {
        const T ts[kSu2Acc] = {kin0, kin, eg, lam * r2 * r2, m2 * r2, ka0, ka, omA, kb0, kb, omB,
                               ph[0], ph[1], ph[2], ph[3], r2};
#pragma unroll
        for (int k = 0; k < kSu2Acc; ++k) acc[k] += (double)ts[k];
      } else {
        // each term into its FP64 sum: two of them added in FP32 first would
        // round every site of a near-homogeneous state alike, and a and b with it
        const T ts[kSu2StepAcc] = {kin, eg, lam * r2 * r2, ka, omA, kb, omB};
#pragma unroll
        for (int k = 0; k < kSu2StepAcc; ++k) acc[k] += (double)ts[k];
        acc[2] += (double)(m2 * r2);
        if (lf) {
          acc[0] += (double)kin0;
          acc[3] += (double)ka0;
          acc[5] += (double)kb0;
        }
      }
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) qc[k] = qn[k];
    __syncthreads();
    if (i + 1 < XC) {
      drift_into(c);  // plane x+2 replaces plane x
      momenta(qn);
      __syncthreads();
    }
  }
  // the tile's sums: waves in order
#pragma unroll
  for (int k = 0; k < NACC; ++k) {
    const double s = wave_sum(acc[k]);
    if ((tid & 63) == 0) red[tid >> 6][k] = s;
  }
  __syncthreads();
  if (tid < NACC) {
    double s = red[0][tid];
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) s += red[w][tid];
    A.partials[(size_t)blockIdx.x * NACC + tid] = s;
  }
}

// Sums of nb records in a fixed order by one block of NT threads: thread t
// takes doubles t, t + NL, ... (NL a multiple of the record length, so the
// loads are coalesced and a thread's values belong to one accumulator), then
// the threads of each accumulator in order.  The first thread returns the
// sums in S.
template <int NACC, int NT>
__device__ bool su2_reduce_records(const double* rec, int nb, double (&S)[NACC]) {
  constexpr int NL = (NT / NACC) * NACC;
  static_assert(NT >= 64 && NACC <= 64, "the first wave finishes the sums");
  __shared__ double part[NL];
  const int tid = threadIdx.x;
  const int64_t nv = (int64_t)nb * NACC;
  if (tid < NL) {
    double s = 0.0;
#pragma unroll 8
    for (int64_t e = tid; e < nv; e += NL) s += rec[e];
    part[tid] = s;
  }
  __syncthreads();
  if (tid >= 64) return false;
  double v = 0.0;
  if (tid < NACC) {
#pragma unroll
    for (int l = 0; l < NL / NACC; ++l) v += part[l * NACC + tid];
  }
#pragma unroll
  for (int k = 0; k < NACC; ++k) S[k] = lane_value(v, k);
  return tid == 0;
}

// Energies (Sec. 5.4.1, Sec. 6.3.1) at a' from the lattice sums S of pass `pd`,
// which started from state `in`, and the scale-factor kernel with both gauge
// sectors, K_a = (1/3)(f/m_p)^2 a'^{1+2 alpha}[(alpha-2)E_K + alpha E_G + (alpha+1)E_V
// + (alpha-1)(E_K^A + E_G^A + E_K^B + E_G^B)]; b_out = b + (wk1 + wk2) h K_a.
// The state goes to `out` (may be `in`; nullptr: not stored); a and b after
// the pass are returned in a_next, b_next.
template <typename T, bool OBS>
__device__ void su2_finish_state(const Su2PassArgs<T>& A, const PassDesc& pd, const DevState* in, const double* S,
                                 DevState* out, double& a_next, double& b_next) {
  const double V = (double)A.N * A.N * A.N;
  const double a_in = in->a, b_in = in->b, al = A.alpha;
  const double a = A.expand ? a_in + pd.wd * A.h * b_in : a_in;
  const bool lf = pd.mode == MODE_LF;
  const double a2 = a * a, a4 = a2 * a2, a6 = a4 * a2, dx2 = A.dx * A.dx, dx4 = dx2 * dx2;
  // kinetic, gradient, potential, then electric and magnetic sums of U(1) and SU(2)
  double kin, grad, kA, mA, kB, mB;
  lattice_obs o = in->obs;
  bool bad = false;
  if constexpr (OBS) {
    kin = lf ? 0.5 * (S[0] + S[1]) : S[1];
    grad = S[2];
    o.EV_term[0] = S[4] / V;
    o.EV_term[1] = S[3] / V;
    o.EV_term[2] = 0.0;
    o.EV = o.EV_term[0] + o.EV_term[1];
    kA = lf ? 0.5 * (S[5] + S[6]) : S[6];
    mA = S[7];
    kB = lf ? 0.5 * (S[8] + S[9]) : S[9];
    mB = S[10];
    o.mean_f[0] = S[11] / V;
    o.mean_f[1] = S[12] / V;
    o.mean_lo[0] = S[13] / V;
    o.mean_lo[1] = S[14] / V;
    o.meansq_f[0] = S[15] / V;
    o.meansq_f[1] = 0.0;
  } else {
    const double f = lf ? 0.5 : 1.0;
    kin = f * S[0];
    grad = S[1];
    o.EV = S[2] / V;
    kA = f * S[3];
    mA = S[4];
    kB = f * S[5];
    mB = S[6];
    o.EV_term[0] = o.EV_term[1] = o.EV_term[2] = NAN;
    o.mean_f[0] = o.mean_f[1] = o.mean_lo[0] = o.mean_lo[1] = o.meansq_f[0] = o.meansq_f[1] = NAN;
  }
  for (int k = 0; k < (OBS ? kSu2Acc : kSu2StepAcc); ++k) bad = bad || !isfinite(S[k]);
  o.EK = kin / V / a6;
  o.EG = grad / V / (a2 * dx2);
  o.EK_A = A.wf2 * kA / V / (2.0 * a4);
  o.EG_A = A.wf2 * mA / V / (a4 * dx4 * A.e * A.e);
  o.EK_B = A.wf2 * kB / V / (2.0 * a4);
  o.EG_B = 2.0 * A.wf2 * (2.0 * mB) / V / (a4 * dx4 * A.g * A.g);
  o.EK_f[0] = o.EK;
  o.EK_f[1] = 0.0;
  o.EG_f[0] = o.EG;
  o.EG_f[1] = 0.0;
  const double gauge = o.EK_A + o.EG_A + o.EK_B + o.EG_B;
  const double rho = o.EK + o.EG + o.EV + gauge;
  double b_out = b_in, b_sync = b_in, hc = 0.0;
  if (A.expand) {
    const double Ka = A.fmp2 / 3.0 * apow(a, 1.0 + 2.0 * al) *
                      ((al - 2.0) * o.EK + al * o.EG + (al + 1.0) * o.EV + (al - 1.0) * gauge);
    b_out = b_in + (pd.wk1 + pd.wk2) * A.h * Ka;
    b_sync = lf ? 0.5 * (b_in + b_out) : b_in + pd.wk1 * A.h * Ka;
    const double rhs = A.fmp2 / 3.0 * apow(a, 2.0 * (al + 1.0)) * rho;
    hc = fabs(b_sync * b_sync - rhs) / (b_sync * b_sync);
  }
  const double eta_new = in->eta + pd.wd * A.h;
  o.eta = eta_new;
  o.a = a;
  o.b = b_sync;
  o.H = b_sync / a;
  o.rho = rho;
  o.p = o.EK - o.EG / 3.0 - o.EV + gauge / 3.0;
  o.w = rho != 0.0 ? o.p / rho : 0.0;
  o.hc = hc;
  o.step = 0;
  o.staggered = lf ? 1 : 0;
  o.reserved = 0;
  a_next = pd.update ? a : a_in;
  b_next = pd.update ? b_out : b_in;
  if (!out) return;
  if (out != in) *out = *in;
  out->obs = o;
  if (bad) out->nonfinite = 1;
  if (pd.update) {
    out->a = a;
    out->b = b_out;
    out->eta = eta_new;
  }
}

// The finish of the pass described by A, into `out`: one block of
// kSu2FinishThreads threads (four waves leave each thread the registers for
// its FP64 sums).
constexpr int kSu2FinishThreads = 256;

template <typename T, bool OBS>
__global__ __launch_bounds__(kSu2FinishThreads) void su2_finish_kernel(Su2PassArgs<T> A, int nblocks, DevState* out) {
  constexpr int NACC = OBS ? kSu2Acc : kSu2StepAcc;
  double S[NACC];
  if (!su2_reduce_records<NACC, kSu2FinishThreads>(A.partials, nblocks, S)) return;
  double an, bn;
  su2_finish_state<T, OBS>(A, A.pd, A.st, S, out, an, bn);
}

// Gauss residuals (Sec. 5.2 and Sec. 6.2, with the electric field at n - i
// transported to n):
//   G_A(n)   = sum_i (pi_A,i(n) - pi_A,i(n-i))/dx - 2e (f/w)^2 Im[Phi^dag pi]
//   G_B^a(n) = sum_i (pi_B,i(n) - U_i(n-i)^dag pi_B,i(n-i) U_i(n-i))^a/dx - g (f/w)^2 Im[Phi^dag sigma_a pi]
// in FP64 from the stored values.
template <typename T>
__global__ __launch_bounds__(256) void su2_gauss_kernel(Su2Args<T> A) {
  const int N = A.N;
  const size_t NN = (size_t)N * N, V = NN * N;
  const size_t s = (size_t)blockIdx.x * 256 + threadIdx.x;
  double acc[kSu2GaussAcc] = {0, 0, 0, 0, 0, 0};
  if (s < V) {
    const T* const* F = A.src;
    const int c[3] = {(int)(s / NN), (int)((s / N) % N), (int)(s % N)};
    const size_t str[3] = {NN, (size_t)N, 1};
    double divA = 0.0, divB[3] = {0.0, 0.0, 0.0};
    for (int i = 0; i < 3; ++i) {
      const size_t sm = c[i] > 0 ? s - str[i] : s + (size_t)(N - 1) * str[i];
      divA += ((double)F[kPA + i][s] - (double)F[kPA + i][sm]) / A.dx;
      const Q4<double> u{(double)F[kUL + 4 * i][sm], (double)F[kUL + 4 * i + 1][sm], (double)F[kUL + 4 * i + 2][sm],
                         (double)F[kUL + 4 * i + 3][sm]};
      // U^dag (x.sigma) U as the vector part of U^dag (0, x) U
      const Q4<double> xq{0.0, (double)F[kPB + 3 * i][sm], (double)F[kPB + 3 * i + 1][sm],
                          (double)F[kPB + 3 * i + 2][sm]};
      const Q4<double> t = qmul(qmul(qdag(u), xq), u);
      divB[0] += ((double)F[kPB + 3 * i][s] - t.x) / A.dx;
      divB[1] += ((double)F[kPB + 3 * i + 1][s] - t.y) / A.dx;
      divB[2] += ((double)F[kPB + 3 * i + 2][s] - t.z) / A.dx;
    }
    const Cx2<double> p0{(double)F[kPH][s], (double)F[kPH + 1][s]}, p1{(double)F[kPH + 2][s], (double)F[kPH + 3][s]};
    const Cx2<double> q0{(double)F[kPI][s], (double)F[kPI + 1][s]}, q1{(double)F[kPI + 2][s], (double)F[kPI + 3][s]};
    const double rhoA = 2.0 * A.e / A.wf2 * (cross_im(p0, q0) + cross_im(p1, q1));
    const double cB = A.g / A.wf2;
    const double rhoB[3] = {cB * (cross_im(p0, q1) + cross_im(p1, q0)), cB * (-dot_re(p0, q1) + dot_re(p1, q0)),
                            cB * (cross_im(p0, q0) - cross_im(p1, q1))};
    acc[0] = (divA - rhoA) * (divA - rhoA);
    acc[1] = divA * divA;
    acc[2] = rhoA * rhoA;
    for (int a = 0; a < 3; ++a) {
      acc[3] += (divB[a] - rhoB[a]) * (divB[a] - rhoB[a]);
      acc[4] += divB[a] * divB[a];
      acc[5] += rhoB[a] * rhoB[a];
    }
  }
  su2_block_partials<kSu2GaussAcc>(acc, A.partials);
}

__global__ __launch_bounds__(1024) void su2_gauss_finish_kernel(const double* partials, int nblocks, DevState* st) {
  __shared__ double red[16][kSu2GaussAcc];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  double tot[kSu2GaussAcc] = {0, 0, 0, 0, 0, 0};
  for (int b = tid; b < nblocks; b += 1024)
    for (int k = 0; k < kSu2GaussAcc; ++k) tot[k] += partials[(size_t)b * kSu2GaussAcc + k];
  for (int k = 0; k < kSu2GaussAcc; ++k) {
    const double v = wave_sum(tot[k]);
    if (lane == 0) red[wv][k] = v;
  }
  __syncthreads();
  if (tid != 0) return;
  double S[kSu2GaussAcc] = {0, 0, 0, 0, 0, 0};
  for (int k = 0; k < kSu2GaussAcc; ++k)
    for (int w = 0; w < 16; ++w) S[k] += red[w][k];
  const double dA = sqrt(S[1]) + sqrt(S[2]), dB = sqrt(S[4]) + sqrt(S[5]);
  st->obs.gauss = dA > 0.0 ? sqrt(S[0]) / dA : 0.0;
  st->obs.gauss_B = dB > 0.0 ? sqrt(S[3]) / dB : 0.0;
}

template <typename T>
static void su2_fill(lattice* h, Su2Args<T>& A, const PassDesc& pd) {
  for (int c = 0; c < kSu2Comp; ++c) {
    A.src[c] = static_cast<const T*>(h->buf[h->cur][c]);
    A.dst[c] = static_cast<T*>(h->buf[1 - h->cur][c]);
  }
  A.N = h->p.N;
  A.dx = h->dx;
  A.alpha = h->p.alpha;
  A.fmp2 = h->p.fstar_over_mp * h->p.fstar_over_mp;
  A.lam = h->p.lambda;
  A.m2 = h->p.m2[0];
  A.e = h->p.e;
  A.g = h->p.g;
  A.wf2 = h->p.omega_over_f * h->p.omega_over_f;
  A.h = h->p.dt;
  A.expand = h->p.expansion;
  A.pd = pd;
  A.partials = h->partials;
  A.st = h->st;
}

template <typename T>
static void su2_pass_args(lattice* h, Su2PassArgs<T>& A, const PassDesc& pd) {
  A = {};
  A.src = static_cast<const T*>(h->buf[h->cur][0]);
  A.dst = static_cast<T*>(h->buf[1 - h->cur][0]);
  A.N = h->p.N;
  A.dx = h->dx;
  A.alpha = h->p.alpha;
  A.fmp2 = h->p.fstar_over_mp * h->p.fstar_over_mp;
  A.lam = h->p.lambda;
  A.m2 = h->p.m2[0];
  A.e = h->p.e;
  A.g = h->p.g;
  A.wf2 = h->p.omega_over_f * h->p.omega_over_f;
  A.h = h->p.dt;
  A.expand = h->p.expansion;
  A.pd = pd;
  A.partials = h->partials;
  A.st = h->st;
}

// One pass of the shared schedule in one kernel; the buffers swap when it
// writes.  Within a chain the finish is the next pass's, else a kernel of its
// own follows.
template <typename T, int TZ, int TY, int WPE>
static int su2_pass_t(lattice* h, const PassDesc& pd, PassChain* chain) {
  Su2PassArgs<T> A;
  su2_pass_args(h, A, pd);
  const int N = h->p.N;
  constexpr int NT = Su2Tile<TZ, TY>::NT;
  const int tiles = (N / TZ) * (N / TY);
  // every block pays about three planes' work before its first (planes x0-1,
  // x0, x0+1 and what x0-1 hands on); at least 256 sites per block or one per CU,
  // the record regions' size
  A.nx = x_blocks(N, N, tiles, 256 * (4 * WPE / (NT / 64)), 3.0, (256 + NT - 1) / NT);
  const int nb = tiles * A.nx;
  if (nb > std::max<int64_t>((int64_t)N * N * N / 256, kCUs)) { set_error("SU(2) pass: records exceed their region"); return LAT_EINVAL; }
  DevState* slot[2] = {h->st, h->st2};
  if (chain) {
    A.st = slot[chain->rd];
    A.partials = (chain->k & 1) ? h->partials2 : h->partials;
    A.prev = chain->prev;
    if (A.prev.partials) A.prev.out = slot[1 - chain->rd];
  }
  if (!pd.write) {
    if (pd.wd != 0.0 || chain) { set_error("SU(2) pass: an observation neither drifts nor chains"); return LAT_EINVAL; }
    hipLaunchKernelGGL((su2_pass_kernel<T, TZ, TY, WPE, kPassObs>), dim3(nb), dim3(NT), 0, h->stream, A);
    CL_HIP(hipGetLastError());
    hipLaunchKernelGGL((su2_finish_kernel<T, true>), dim3(1), dim3(kSu2FinishThreads), 0, h->stream, A, nb, h->st);
    CL_HIP(hipGetLastError());
    return LAT_OK;
  }
  hipEvent_t ev0 = nullptr, ev1 = nullptr;
  if (2 * h->timer_used + 1 < h->timer.size()) {
    ev0 = h->timer[2 * h->timer_used];
    ev1 = h->timer[2 * h->timer_used + 1];
    ++h->timer_used;
  }
  auto* const kernel =
      pd.wd != 0.0 ? su2_pass_kernel<T, TZ, TY, WPE, kPassStep> : su2_pass_kernel<T, TZ, TY, WPE, kPassKick>;
  if (ev0)
    hipExtLaunchKernelGGL(kernel, dim3(nb), dim3(NT), 0, h->stream, ev0, ev1, 0, A);
  else
    hipLaunchKernelGGL(kernel, dim3(nb), dim3(NT), 0, h->stream, A);
  CL_HIP(hipGetLastError());
  if (chain) {
    if (A.prev.partials) chain->rd ^= 1;
    chain->prev = PrevPass{A.partials, nb, pd, nullptr};
    ++chain->k;
  } else {
    hipLaunchKernelGGL((su2_finish_kernel<T, false>), dim3(1), dim3(kSu2FinishThreads), 0, h->stream, A, nb, h->st);
    CL_HIP(hipGetLastError());
  }
  h->cur ^= 1;
  return LAT_OK;
}

// Trailing finish of a chain: the last pass's records, from the slot that
// pass started from, into h->st.
template <typename T>
static int su2_chain_finish(lattice* h, const PassChain& c) {
  Su2PassArgs<T> A;
  su2_pass_args(h, A, c.prev.pd);
  A.partials = const_cast<double*>(c.prev.partials);
  A.st = c.rd ? h->st2 : h->st;
  hipLaunchKernelGGL((su2_finish_kernel<T, false>), dim3(1), dim3(kSu2FinishThreads), 0, h->stream, A,
                     c.prev.nblocks, h->st);
  CL_HIP(hipGetLastError());
  return LAT_OK;
}

template <typename T>
static int su2_gauss_t(lattice* h) {
  Su2Args<T> A;
  su2_fill(h, A, pass(0.0, 0.0, 0.0, MODE_VV, 0, 0));
  const int64_t V = (int64_t)h->p.N * h->p.N * h->p.N;
  const int nb = (int)((V + 255) / 256);
  hipLaunchKernelGGL(su2_gauss_kernel<T>, dim3(nb), dim3(256), 0, h->stream, A);
  CL_HIP(hipGetLastError());
  hipLaunchKernelGGL(su2_gauss_finish_kernel, dim3(1), dim3(1024), 0, h->stream, h->partials, nb, h->st);
  CL_HIP(hipGetLastError());
  return LAT_OK;
}

static int su2_pass(lattice* h, const PassDesc& pd, PassChain* chain = nullptr) {
  return h->p.precision == LAT_FP32 ? su2_pass_t<float, 32, 8, 2>(h, pd, chain)
                                    : su2_pass_t<double, 32, 4, 1>(h, pd, chain);
}

int su2_step(lattice* h, int64_t n) {
  const std::vector<PassDesc> sched = pass_schedule(h->p.integrator, h->weights, &h->staggered, n);
  PassChain chain;
  for (const PassDesc& pd : sched) {
    const int rc = su2_pass(h, pd, &chain);
    if (rc) return rc;
  }
  if (chain.k) {
    const int rc = h->p.precision == LAT_FP32 ? su2_chain_finish<float>(h, chain) : su2_chain_finish<double>(h, chain);
    if (rc) return rc;
  }
  h->step += n;
  return LAT_OK;
}

int su2_energies(lattice* h) {
  int rc = h->p.precision == LAT_FP32 ? su2_gauss_t<float>(h) : su2_gauss_t<double>(h);
  if (rc) return rc;
  if (h->staggered) return su2_pass(h, pass(0.0, 0.0, 1.0, MODE_LF, 0, 0));
  return su2_pass(h, pass(0.0, 0.0, 0.0, MODE_VV, 0, 0));
}

// ---------------------------------------------------------------------------
// initial state (Sec. 7.2)
// ---------------------------------------------------------------------------
// Phi = (phi_0 + i phi_1, phi_2 + i phi_3)/sqrt 2 and pi = a^{3-alpha} Phi' from
// the FP64 real components; the charge densities rho_A, rho_B^a (Sec. 6.2 Gauss
// laws) as the real parts of four complex arrays.
template <typename T>
__global__ void su2_store_kernel(const double* f, const double* d, Su2Args<T> A, double2* rho, int64_t V,
                                 double cpi) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= V) return;
  const double is2 = 0.70710678118654752440084436210485;
  double ph[4], pq[4];
  for (int k = 0; k < 4; ++k) {
    ph[k] = f[(size_t)k * V + i] * is2;
    pq[k] = cpi * d[(size_t)k * V + i] * is2;
    A.dst[kPH + k][i] = (T)ph[k];
    A.dst[kPI + k][i] = (T)pq[k];
  }
  const Cx2<double> p0{ph[0], ph[1]}, p1{ph[2], ph[3]}, q0{pq[0], pq[1]}, q1{pq[2], pq[3]};
  const double cB = A.g / A.wf2;
  rho[i] = make_double2(2.0 * A.e / A.wf2 * (cross_im(p0, q0) + cross_im(p1, q1)), 0.0);
  rho[V + i] = make_double2(cB * (cross_im(p0, q1) + cross_im(p1, q0)), 0.0);
  rho[2 * V + i] = make_double2(cB * (-dot_re(p0, q1) + dot_re(p1, q0)), 0.0);
  rho[3 * V + i] = make_double2(cB * (cross_im(p0, q0) - cross_im(p1, q1)), 0.0);
}

template <typename T>
__global__ void su2_unit_links_kernel(Su2Args<T> A, int64_t V) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= V) return;
  for (int i = 0; i < 3; ++i) {
    A.dst[kTH + i][s] = T(0);
    A.dst[kUL + 4 * i][s] = T(1);
    A.dst[kUL + 4 * i + 1][s] = T(0);
    A.dst[kUL + 4 * i + 2][s] = T(0);
    A.dst[kUL + 4 * i + 3][s] = T(0);
  }
}

template <typename T>
static int su2_init_state_t(lattice* h) {
  const lattice_params& p = h->p;
  const int N = p.N;
  const int64_t V = (int64_t)N * N * N;
  const double a = p.a0, al = p.alpha, fmp2 = p.fstar_over_mp * p.fstar_over_mp;
  // every real component starts at phi0[0] (and dphi0[0]), as Sec. 7.2 does
  const double pb = p.phi0[0], db = p.dphi0[0];
  const double s = 4.0 * pb * pb, r2 = 0.5 * s;
  const double rho_hom = 4.0 * db * db / (2.0 * std::pow(a, 2.0 * al)) + p.lambda * r2 * r2 + p.m2[0] * r2;
  const double Hhom = p.expansion ? std::sqrt(fmp2 / 3.0 * std::pow(a, 2.0 * (al + 1.0)) * rho_hom) / a : 0.0;
  const double m2eff = p.lambda * (s + 2.0 * pb * pb) + p.m2[0];
  // scratch in the other state buffer: 8 V doubles of fields, then 4 V complex charges
  char* base = static_cast<char*>(h->buf[1 - h->cur][0]);
  double* fld = reinterpret_cast<double*>(base);
  double2* rho = reinterpret_cast<double2*>(base + (size_t)8 * V * sizeof(double));
  for (int n = 0; n < 4; ++n)
    for (int deriv = 0; deriv < 2; ++deriv) {
      int rc = charged_mode_field(h, n, deriv, m2eff, Hhom, deriv ? db : pb, fld + (size_t)(deriv * 4 + n) * V);
      if (rc) return rc;
    }
  Su2Args<T> A;
  su2_fill(h, A, pass(0.0, 0.0, 0.0, MODE_VV, 0, 0));
  for (int c = 0; c < kSu2Comp; ++c) A.dst[c] = static_cast<T*>(h->buf[h->cur][c]);
  const int thr = 256;
  const int blk = (int)((V + thr - 1) / thr);
  hipLaunchKernelGGL(su2_store_kernel<T>, dim3(blk), dim3(thr), 0, h->stream, fld, fld + 4 * V, A, rho, V,
                     std::pow(a, 3.0 - al));
  CL_HIP(hipGetLastError());
  hipLaunchKernelGGL(su2_unit_links_kernel<T>, dim3(blk), dim3(thr), 0, h->stream, A, V);
  CL_HIP(hipGetLastError());
  // each charge: forward DFT into its own slot, then the three minimum-norm solutions
  double2* F = reinterpret_cast<double2*>(h->fft);
  for (int q = 0; q < 4; ++q) {
    CL_HIP(hipMemcpyAsync(F, rho + (size_t)q * V, (size_t)V * sizeof(double2), hipMemcpyDeviceToDevice, h->stream));
    int rc = run_fft3d(h, +1, 1.0);
    if (rc) return rc;
    CL_HIP(hipMemcpyAsync(rho + (size_t)q * V, F, (size_t)V * sizeof(double2), hipMemcpyDeviceToDevice, h->stream));
  }
  for (int q = 0; q < 4; ++q) {
    void* out[3];
    for (int i = 0; i < 3; ++i) out[i] = q == 0 ? h->buf[h->cur][kPA + i] : h->buf[h->cur][kPB + 3 * i + (q - 1)];
    int rc = gauss_solve_fields(h, rho + (size_t)q * V, out, p.precision == LAT_FP32);
    if (rc) return rc;
  }
  int rc = upload_scalars(h, a, 0.0, 0.0);
  if (rc) return rc;
  h->staggered = 0;
  h->step = 0;
  if (p.expansion) {
    rc = su2_energies(h);
    if (rc) return rc;
    DevState d;
    CL_HIP(hipMemcpyAsync(&d, h->st, sizeof(DevState), hipMemcpyDeviceToHost, h->stream));
    CL_HIP(hipStreamSynchronize(h->stream));
    const double b0 = std::sqrt(fmp2 / 3.0 * std::pow(a, 2.0 * (al + 1.0)) * d.obs.rho);
    rc = upload_scalars(h, a, b0, 0.0);
    if (rc) return rc;
  }
  return LAT_OK;
}

int su2_init_state(lattice* h) {
  return h->p.precision == LAT_FP32 ? su2_init_state_t<float>(h) : su2_init_state_t<double>(h);
}

}  // namespace cl
