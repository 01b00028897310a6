// Fused scalar-field pass for gfx950: drift, 7-point stencil kick, FP64
// volume averages and the scale-factor update, in one sweep over the lattice.
//
// Method (arXiv:2006.15122): Hamiltonian form of the scalar EOM (Sec. 4.2.3)
//   phi' = a^{-(3-alpha)} pi,  pi' = a^{1+alpha} lap phi - a^{3+alpha} V_{,phi},
//   b'   = (1/3)(f*/m_p)^2 a^{1+2 alpha}[(alpha-2) E_K + alpha E_G + (alpha+1) E_V],
// integrated by velocity Verlet / Yoshida (Sec. 4.2.3, 4.3.2) or staggered leapfrog
// scheme III (Sec. 4.2.1).  Consecutive kicks of the Verlet chain are merged
// (Sec. 3.3.2: velocity Verlet is leapfrog plus a synchronising half kick), so
// one pass = drift of sub-step p followed by the kick that closes p and opens
// p+1.  The drift needs the global energies of the previous pass: a one-block
// finish kernel reduces the per-tile FP64 partials in a fixed order and
// advances a and b in FP64 before the next pass starts.
//
// Tiling: a block owns a TY x TZ tile of the (y, z) plane and marches along x
// over XC planes.  z is the fastest index, so each wavefront loads contiguous
// rows.  The drifted plane x (with a one-site y/z halo) sits in LDS; the x-1,
// x+1 neighbours stay in registers.  Halo sites are drifted redundantly by the
// neighbouring tiles, which removes a separate drift pass over HBM.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "common.hpp"
#include "internal.hpp"
#include "scalar_rows.hpp"
#include "scalar_tile.hpp"

namespace cl {

// ---------------------------------------------------------------------------
// Host-side launch table
// ---------------------------------------------------------------------------
struct Shape {
  int tz, by, ry;
};

// With ev0/ev1 the dispatch itself carries the device's start and stop
// timestamps of the pass kernel (hipExtLaunchKernel), nothing else changes.
// fin: where the finish kernel after the pass stores the state (nullptr: no
// finish kernel; the next pass of the chain carries it).
template <typename T, int NF, bool FULL, int TZ, int BY, int RY>
hipError_t launch_shape(const ScalarArgs<T>& A, int nblocks, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1,
                        DevState* fin) {
  if (ev0)
    hipExtLaunchKernelGGL((scalar_pass_kernel<T, NF, FULL, TZ, BY, RY>), dim3(nblocks), dim3(TZ * BY), 0, s, ev0,
                          ev1, 0, A);
  else
    hipLaunchKernelGGL((scalar_pass_kernel<T, NF, FULL, TZ, BY, RY>), dim3(nblocks), dim3(TZ * BY), 0, s, A);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !fin) return e;
  hipLaunchKernelGGL((scalar_finish_kernel<T, NF, FULL>), dim3(1), dim3(kFinishThreads), 0, s, A, nblocks, fin);
  return hipGetLastError();
}

// Full-row tiles (stepping passes): tz = N, ry = 1, by y-rows per block.
template <typename T, int W, int NF, int BY, int MODE = kRowsStep>
hipError_t launch_rows(const ScalarArgs<T>& A, int nblocks, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1,
                       DevState* fin) {
  const dim3 blk(A.N / W * BY);
  const size_t shm = rows_lds_bytes<T>(NF, A.N, BY);
  if (ev0)
    hipExtLaunchKernelGGL((scalar_rows_kernel<T, W, NF, BY, MODE>), dim3(nblocks), blk, shm, s, ev0, ev1, 0, A);
  else
    hipLaunchKernelGGL((scalar_rows_kernel<T, W, NF, BY, MODE>), dim3(nblocks), blk, shm, s, A);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !fin) return e;
  hipLaunchKernelGGL((scalar_finish_kernel<T, NF, MODE != kRowsStep>), dim3(1), dim3(kFinishThreads), 0, s, A, nblocks,
                     fin);
  return hipGetLastError();
}

// Stepping passes: every compiled tile shape (FP32 two-field is the
// production case; the other storage/field combinations get a subset).
// (the four- and eight-row shapes exceed 128 VGPRs with the coefficient pairs
// and spill the prefetched plane; they are not built for this case)
#define CL_SHAPES_MAIN(X, T, NF) \
  X(T, NF, 64, 4, 2)             \
  X(T, NF, 64, 8, 2)             \
  X(T, NF, 32, 8, 2)             \
  X(T, NF, 128, 8, 2)            \
  X(T, NF, 256, 4, 2)            \
  X(T, NF, 128, 4, 2)
#define CL_SHAPES_SMALL(X, T, NF) \
  X(T, NF, 64, 4, 2)              \
  X(T, NF, 32, 8, 2)              \
  X(T, NF, 32, 4, 4)

// full-row shapes (tz = N sites, by rows, ry = 1) in blocks of at most
// kRowsMaxThreads lanes and 96 KB of LDS: four sites per lane in FP32 storage,
// two in FP64 (two FP32 sites per lane fit two blocks per CU but are slower:
// 113.9 against 109.7 us per pass at 256^3)
#define CL_ROWS_F32(X, T, NF) \
  X(T, NF, 4, 4)              \
  X(T, NF, 4, 8)              \
  X(T, NF, 4, 16)
#define CL_ROWS_F64(X, T, NF) \
  X(T, NF, 2, 2)              \
  X(T, NF, 2, 4)              \
  X(T, NF, 2, 8)

// general shapes, then full-row ones (tz = 0 stands for N)
static const Shape kShapesMain[] = {{64, 4, 2},  {64, 8, 2}, {32, 8, 2}, {128, 8, 2}, {256, 4, 2},
                                    {128, 4, 2}, {0, 4, 1},  {0, 8, 1},  {0, 16, 1}};
static const Shape kShapesSmall[] = {{64, 4, 2}, {32, 8, 2}, {32, 4, 4}, {0, 4, 1}, {0, 8, 1}, {0, 16, 1}};
static const Shape kShapesF64[] = {{64, 4, 2}, {32, 8, 2}, {32, 4, 4}, {0, 2, 1}, {0, 4, 1}, {0, 8, 1}};

// Observation passes: the 32 x 16 general tile with 8 planes, which divides
// every supported N, where no full-row block fits; else full rows, as many
// planes as leave 512 blocks.
static const int kObsTz = 32, kObsBy = 8, kObsRy = 2, kObsXc = 8;

static Tiling obs_tiling(int fp32, int nf, int N) {
  const int ns = num_shapes(fp32, nf);
  for (int by : {8, 4, 2})
    for (int i = 0; i < ns; ++i) {
      Tiling t{};
      if (!get_shape(fp32, nf, N, i, &t.tz, &t.by, &t.ry) || t.ry != 1 || t.by != by || t.tz != N) continue;
      // (at most 2048 records at 512^3: lattice_energies_noalloc's scratch
      // takes them wherever it takes the general tile's)
      for (int xc : {32, 16, 8, 4, 2}) {
        t.xc = xc;
        if ((int64_t)(N / by) * (N / xc) >= 512) return t;
      }
      return t;
    }
  return Tiling{kObsTz, kObsBy, kObsRy, kObsXc};
}

// Blocks of a pass on tile t.  Full rows share the planes among at least N / xc
// of them (*nx along x): 168 VGPRs let twelve waves share a CU; a block reads
// two planes beyond its own.
static int64_t pass_blocks(int fp32, int N, const Tiling& t, int* nx) {
  const int tiles = (N / t.tz) * (N / (t.by * t.ry));
  *nx = 0;
  if (t.ry == 1) {
    const int waves = N / (fp32 ? 4 : 2) * t.by / 64;
    *nx = x_blocks(N, t.xc, tiles, 256 * std::max(1, 12 / waves), 2.0, 8);
  }
  return (int64_t)tiles * (*nx ? *nx : N / t.xc);
}

int64_t scalar_obs_blocks(int fp32, int nf, int N) {
  int nx;
  return pass_blocks(fp32, N, obs_tiling(fp32, nf, N), &nx);
}

template <typename T, int NF>
hipError_t launch_scalar_pass_t(const ScalarArgs<T>& A, const Shape& sh, int nblocks, hipStream_t s, bool full,
                                hipEvent_t ev0, hipEvent_t ev1, DevState* fin) {
  if (full) {
    if (sh.ry > 1) return launch_shape<T, NF, true, 32, 8, 2>(A, nblocks, s, ev0, ev1, fin);
    const bool sync = A.pd.mode == MODE_VV && A.pd.wk1 == 0.0;  // no kick in E_K
#define XF(TT, NFF, w, b) \
  if (sh.by == b)            \
    return sync ? launch_rows<TT, w, NFF, b, kRowsObsSync>(A, nblocks, s, ev0, ev1, fin) \
                : launch_rows<TT, w, NFF, b, kRowsObs>(A, nblocks, s, ev0, ev1, fin);
    if constexpr (std::is_same<T, float>::value) {
      CL_ROWS_F32(XF, T, NF)
    } else {
      CL_ROWS_F64(XF, T, NF)
    }
#undef XF
    return hipErrorInvalidValue;
  }
#define X(TT, NFF, a, b, c) \
  if (sh.tz == a && sh.by == b && sh.ry == c)  \
    return launch_shape<TT, NFF, false, a, b, c>(A, nblocks, s, ev0, ev1, fin);
#define XR(TT, NFF, w, b) \
  if (sh.ry == 1 && sh.by == b) return launch_rows<TT, w, NFF, b>(A, nblocks, s, ev0, ev1, fin);
  if constexpr (std::is_same<T, float>::value && NF == 2) {
    CL_SHAPES_MAIN(X, T, NF)
  } else {
    CL_SHAPES_SMALL(X, T, NF)
  }
  if constexpr (std::is_same<T, float>::value) {
    CL_ROWS_F32(XR, T, NF)
  } else {
    CL_ROWS_F64(XR, T, NF)
  }
#undef XR
#undef X
  return hipErrorInvalidValue;
}

int num_shapes(int fp32, int nf) {
  if (fp32) return nf == 2 ? (int)(sizeof(kShapesMain) / sizeof(Shape)) : (int)(sizeof(kShapesSmall) / sizeof(Shape));
  return (int)(sizeof(kShapesF64) / sizeof(Shape));
}
// Shape i at size N; false where a full-row block would hold a part of a
// wave, too many lanes or too much LDS.
bool get_shape(int fp32, int nf, int N, int i, int* tz, int* by, int* ry) {
  const Shape& sh = fp32 ? (nf == 2 ? kShapesMain[i] : kShapesSmall[i]) : kShapesF64[i];
  *tz = sh.tz ? sh.tz : N;
  *by = sh.by;
  *ry = sh.ry;
  if (sh.ry > 1) return true;
  const int nt = N / (fp32 ? 4 : 2) * sh.by;
  const size_t lds = fp32 ? rows_lds_bytes<float>(nf, N, sh.by) : rows_lds_bytes<double>(nf, N, sh.by);
  return nt % 64 == 0 && nt <= kRowsMaxThreads && lds <= 98304;
}


// Launch one pass.  buffers: src/dst arrays [4] in storage precision.
hipError_t launch_scalar_pass(int fp32, int nf, const void* const* src, void* const* dst, int N, int tz,
                              int by, int ry, int xc, int swizzle, const double* phys, int expand,
                              const PassDesc& pd, double* partials, int64_t max_records, DevState* st,
                              hipStream_t s, int* nblocks_out, int full, hipEvent_t ev0, hipEvent_t ev1,
                              const PrevPass& prev, DevState* fin) {
  if (full && (prev.partials || !fin)) return hipErrorInvalidValue;  // observation passes finish themselves
  if ((pd.write != 0) == (full != 0)) return hipErrorInvalidValue;    // stepping passes store, observations do not
  const Tiling t = full ? obs_tiling(fp32, nf, N) : Tiling{tz, by, ry, xc};
  const Shape sh{t.tz, t.by, t.ry};
  int nx = 0;
  const int64_t records = pass_blocks(fp32, N, t, &nx);
  if (records > max_records) return hipErrorInvalidValue;  // they would leave their region
  const int nblocks = (int)records;
  if (nblocks_out) *nblocks_out = nblocks;
  auto fill = [&](auto& A, auto* tag) {
    using TT = std::remove_pointer_t<decltype(tag)>;
    for (int i = 0; i < 4; ++i) {
      A.src[i] = static_cast<const TT*>(src[i]);
      A.dst[i] = static_cast<TT*>(dst[i]);
    }
    A.N = N;
    A.XC = t.xc;
    A.nx = nx;
    A.swizzle = swizzle;
    A.dx = phys[0];
    A.alpha = phys[1];
    A.fmp2 = phys[2];
    A.m2_0 = phys[3];
    A.m2_1 = phys[4];
    A.lam = phys[5];
    A.q = phys[6];
    A.h = phys[7];
    A.expand = expand;
    A.pd = pd;
    A.partials = partials;
    A.st = st;
    A.prev = prev;
  };
  if (fp32) {
    ScalarArgs<float> A;
    fill(A, (float*)nullptr);
    return nf == 1 ? launch_scalar_pass_t<float, 1>(A, sh, nblocks, s, full, ev0, ev1, fin)
                   : launch_scalar_pass_t<float, 2>(A, sh, nblocks, s, full, ev0, ev1, fin);
  } else {
    ScalarArgs<double> A;
    fill(A, (double*)nullptr);
    return nf == 1 ? launch_scalar_pass_t<double, 1>(A, sh, nblocks, s, full, ev0, ev1, fin)
                   : launch_scalar_pass_t<double, 2>(A, sh, nblocks, s, full, ev0, ev1, fin);
  }
}

// Finish kernel alone: the pass `pd` that wrote `nblocks` partial records
// started from state `in`; the result goes to `out` (the trailing finish of a
// chain of passes).
hipError_t launch_scalar_finish(int fp32, int nf, int N, const double* phys, int expand, const PassDesc& pd,
                                double* partials, int nblocks, DevState* in, DevState* out, hipStream_t s) {
  auto go = [&](auto* tag) -> hipError_t {
    using TT = std::remove_pointer_t<decltype(tag)>;
    ScalarArgs<TT> A = {};
    A.N = N;
    A.dx = phys[0];
    A.alpha = phys[1];
    A.fmp2 = phys[2];
    A.m2_0 = phys[3];
    A.m2_1 = phys[4];
    A.lam = phys[5];
    A.q = phys[6];
    A.h = phys[7];
    A.expand = expand;
    A.pd = pd;
    A.partials = partials;
    A.st = in;
    if (nf == 1)
      hipLaunchKernelGGL((scalar_finish_kernel<TT, 1, false>), dim3(1), dim3(kFinishThreads), 0, s, A, nblocks, out);
    else
      hipLaunchKernelGGL((scalar_finish_kernel<TT, 2, false>), dim3(1), dim3(kFinishThreads), 0, s, A, nblocks, out);
    return hipGetLastError();
  };
  return fp32 ? go((float*)nullptr) : go((double*)nullptr);
}

}  // namespace cl
