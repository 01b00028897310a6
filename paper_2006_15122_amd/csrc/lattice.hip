// Host side of the C ABI declared in include/cosmolat.h: parameter checks,
// workspace carving, the sequence of fused passes for each integrator, state
// transfer, observables and the tile autotuner.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <initializer_list>
#include <map>
#include <mutex>
#include <tuple>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "common.hpp"
#include "internal.hpp"

namespace cl {

static thread_local std::string g_err;
void set_error(const std::string& msg) { g_err = msg; }

static size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Yoshida weights of VVn (Sec. 3.4.1, appendix table).  VV4 is the symmetric
// triple jump w1 = w3 = 1/(2 - 2^{1/3}), w2 = -2^{1/3}/(2 - 2^{1/3}), which
// sums to one.
// VV6, VV8 and VV10 use the printed rows of that table: the first half of the
// weights and the middle one; the second half mirrors the first.
static std::vector<double> mirrored(std::initializer_list<double> half, double mid) {
  std::vector<double> w(half);
  w.push_back(mid);
  for (auto it = half.end(); it != half.begin();) w.push_back(*--it);
  return w;
}

std::vector<double> vv_weights(int integrator) {
  switch (integrator) {
    case LAT_VV4: {
      const double c = std::cbrt(2.0);
      const double w1 = 1.0 / (2.0 - c), w2 = -c / (2.0 - c);
      return {w1, w2, w1};
    }
    case LAT_VV6:
      return mirrored({0.78451361047755726382, 0.23557321335935813368, -1.1776799841788710069},
                      1.3151863206839112189);
    case LAT_VV8:
      return mirrored({0.74167036435061295345, -0.40910082580003159400, 0.19075471029623837995,
                       -0.57386247111608226666, 0.29906418130365592384, 0.33462491824529818378,
                       0.31529309239676659663},
                      -0.79688793935291635402);
    case LAT_VV10:
      return mirrored({-0.48159895600253002870, 0.0036303931544595926879, 0.50180317558723140279,
                       0.28298402624506254868, 0.80702967895372223806, -0.026090580538592205447,
                       -0.87286590146318071547, -0.52373568062510581643, 0.44521844299952789252,
                       0.18612289547097907887, 0.23137327866438360633, -0.52191036590418628905,
                       0.74866113714499296793, 0.066736511890604057532, -0.80360324375670830316},
                      0.91249037635867994571);
    default:
      return {1.0};
  }
}

int validate(const lattice_params* p) {
  if (!p) { set_error("params is NULL"); return LAT_EINVAL; }
  if (p->model != LAT_MODEL_SCALAR && !is_u1(*p) && !is_su2(*p)) { set_error("unknown model"); return LAT_EINVAL; }
  if (is_su2(*p) && p->nf != 4) { set_error("SU(2) x U(1) model needs nf = 4"); return LAT_EINVAL; }
  if (is_su2(*p) && !(p->e > 0.0 && p->g > 0.0)) { set_error("SU(2) x U(1) model needs e > 0 and g > 0"); return LAT_EINVAL; }
  if (p->model == LAT_MODEL_SCALAR && (p->nf < 1 || p->nf > 2)) { set_error("scalar model needs nf = 1 or 2"); return LAT_EINVAL; }
  if (is_u1(*p) && p->nf != 2) { set_error("U1 model needs nf = 2"); return LAT_EINVAL; }
  if (p->N < 32 || p->N > 1024 || p->N % 32 != 0) { set_error("N must be a multiple of 32 in [32, 1024]"); return LAT_EINVAL; }
  if (p->integrator < LAT_LF2 || p->integrator > LAT_VV10) { set_error("unknown integrator"); return LAT_EINVAL; }
  if (p->precision != LAT_FP32 && p->precision != LAT_FP64) { set_error("unknown precision"); return LAT_EINVAL; }
  if (!(p->kIR > 0.0) || !(p->dt > 0.0)) { set_error("kIR and dt must be positive"); return LAT_EINVAL; }
  const double dx = 2.0 * M_PI / (p->kIR * p->N);
  if (p->dt > dx / std::sqrt(3.0)) { set_error("time step above the Courant bound dx/sqrt(3)"); return LAT_EINVAL; }
  if (p->ic != LAT_IC_VACUUM && p->ic != LAT_IC_HOMOGENEOUS) { set_error("unknown ic"); return LAT_EINVAL; }
  if (p->expansion && !(p->fstar_over_mp > 0.0)) { set_error("expansion needs fstar_over_mp > 0"); return LAT_EINVAL; }
  if (!(p->a0 > 0.0)) { set_error("a0 must be positive"); return LAT_EINVAL; }
  return LAT_OK;
}

// Workspace layout (each region 256-byte aligned):
//   2 DevState | pass partials | chain partials | spectrum partials | state buffer 0 | state buffer 1 |
//   FFT scratch | FFT roots
static int spec_bins(int N) { return (int)std::floor(std::sqrt(3.0) * N / 2.0) + 1; }

static void layout(const lattice_params* p, size_t* off_part, size_t* off_part2, size_t* off_spec, size_t* off_buf0,
                   size_t* off_buf1, size_t* off_fft, size_t* total, size_t* comp_bytes, int* ncomp,
                   int64_t* max_blocks) {
  const int64_t N = p->N;
  const int64_t V = N * N * N;
  const size_t elem = p->precision == LAT_FP32 ? 4 : 8;
  const int nc = ncomponents(p);
  const int64_t mb = (N / 32) * (N / 8) * (N / 4);
  // per-block FP64 partials: a scalar pass writes at most 13 per block, of
  // which there are one per CU or per 32 x 8 x 4 sites; the U(1) site kernels
  // write up to 16 per block of 256 sites
  const size_t part_doubles = std::max((size_t)std::max<int64_t>(mb, kCUs) * 32, (size_t)(V / 256) * 16);
  size_t o = align_up(2 * sizeof(DevState), 256);
  *off_part = o;
  o = align_up(o + part_doubles * sizeof(double), 256);
  // every other pass of a chain writes its records here: at most mb blocks
  // (of 1024 sites or more) or one per CU, of 4 scalar or 5 U(1) sums; SU(2) x U(1)
  // blocks take 256 sites or more, or are one per CU, and write 7
  *off_part2 = o;
  o = align_up(o + (size_t)std::max<int64_t>(is_su2(*p) ? V / 256 : mb, kCUs) * 16 * sizeof(double), 256);
  *off_spec = o;
  o = align_up(o + (size_t)(spec_blocks((int)N) + 2) * spec_bins((int)N) * 24, 256);
  *off_buf0 = o;
  *comp_bytes = align_up((size_t)V * elem, 256);
  o += (size_t)nc * (*comp_bytes);
  *off_buf1 = o;
  o += (size_t)nc * (*comp_bytes);
  *off_fft = o;
  o = align_up(o + (size_t)V * 16, 256);
  o = align_up(o + (size_t)N * 16, 256);  // FFT twiddle table, right after the scratch
  *total = o;
  *ncomp = nc;
  *max_blocks = mb;
}

int ncomponents(const lattice_params* p) {
  if (is_u1(*p)) return 10;  // phi (2), pi (2), link phases or A_i (3), piA (3)
  if (is_su2(*p)) return 35;  // Phi (4), pi (4), U(1) phases (3), piA (3), SU(2) links (12), piB (9)
  return 2 * p->nf;
}

}  // namespace cl

using namespace cl;

static int su2_set_state(lattice_t* h, const double* fields, const double* momenta, const double* links,
                         const double* link_momenta, const lattice_scalars* s);
static int su2_get_state(lattice_t* h, double* fields, double* momenta, double* links, double* link_momenta,
                         lattice_scalars* s);

extern "C" {

const char* lattice_last_error(void) { return g_err.c_str(); }

int lattice_workspace_size(const lattice_params* p, size_t* bytes) {
  const int rc = cl::validate(p);
  if (rc) return rc;
  if (!bytes) { set_error("bytes is NULL"); return LAT_EINVAL; }
  size_t a, a2, b, c, d, e, t, cb;
  int nc;
  int64_t mb;
  layout(p, &a, &a2, &e, &b, &c, &d, &t, &cb, &nc, &mb);
  *bytes = t;
  return LAT_OK;
}

int lattice_init(const lattice_params* p, void* dev_ws, size_t ws_bytes, void* hip_stream, lattice_t** out) {
  int rc = validate(p);
  if (rc) return rc;
  if (!out || !dev_ws) { set_error("out or dev_ws is NULL"); return LAT_EINVAL; }
  size_t off_part, off_part2, off_spec, off_b0, off_b1, off_fft, total, cb;
  int nc;
  int64_t mb;
  layout(p, &off_part, &off_part2, &off_spec, &off_b0, &off_b1, &off_fft, &total, &cb, &nc, &mb);
  if (ws_bytes < total) {
    set_error("workspace too small: need " + std::to_string(total) + " bytes");
    return LAT_ENOMEM;
  }
  if (((uintptr_t)dev_ws) % 256 != 0) { set_error("workspace must be 256-byte aligned"); return LAT_EINVAL; }
  rc = noalloc_setup();
  if (rc) return rc;
  lattice* L = new lattice();
  L->p = *p;
  L->stream = (hipStream_t)hip_stream;
  char* ws = (char*)dev_ws;
  L->ws = ws;
  L->st = (DevState*)ws;
  L->st2 = L->st + 1;
  L->partials = (double*)(ws + off_part);
  L->partials2 = (double*)(ws + off_part2);
  L->spec = ws + off_spec;
  L->max_blocks = mb;
  L->ncomp = nc;
  L->comp_bytes = cb;
  for (int c = 0; c < nc; ++c) {
    L->buf[0][c] = ws + off_b0 + (size_t)c * cb;
    L->buf[1][c] = ws + off_b1 + (size_t)c * cb;
  }
  L->fft = ws + off_fft;
  L->twiddle = ws + off_fft + align_up((size_t)p->N * p->N * p->N * 16, 256);
  L->cur = 0;
  L->dx = 2.0 * M_PI / (p->kIR * p->N);
  L->weights = vv_weights(p->integrator);
  L->staggered = 0;
  L->step = 0;
  default_tiling(L);
  // Tune first, on zeroed buffers, so that the timed passes can ping-pong
  // between the two state copies exactly as lattice_step does; the initial
  // state is built afterwards.
  if (p->N >= 128 && !is_su2(*p)) {
    // The tile fixes the order of the FP64 partial sums, so the first pick for
    // a configuration is kept for the process: later lattices of the same
    // model, size, precision and integrator reproduce its results bitwise.
    using Key = std::tuple<int, int, int, int, int, int, int>;
    static std::map<Key, Tiling> picks;
    static std::mutex picks_mu;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) dev = 0;
    const Key key{dev, p->model, p->nf, p->N, p->precision, p->integrator, p->expansion};
    bool known = false;
    {
      std::lock_guard<std::mutex> lock(picks_mu);
      auto it = picks.find(key);
      if (it != picks.end()) { L->tile = it->second; known = true; }
    }
    if (!known) {
      rc = autotune(L);
      if (rc) { delete L; return rc; }
      std::lock_guard<std::mutex> lock(picks_mu);
      picks.emplace(key, L->tile);
    }
  }
  rc = init_state(L);
  if (rc) { delete L; return rc; }
  *out = L;
  return LAT_OK;
}

static void drop_timer(lattice_t* h) {
  for (hipEvent_t e : h->timer) hipEventDestroy(e);
  h->timer.clear();
  h->timer_used = 0;
}

int lattice_destroy(lattice_t* h) {
  if (!h) return LAT_OK;
  hipStreamSynchronize(h->stream);
  drop_timer(h);
  delete h;
  return LAT_OK;
}

int lattice_pass_timer(lattice_t* h, int32_t max_launches) {
  if (!h) { set_error("NULL handle"); return LAT_EINVAL; }
  if (max_launches < 0 || max_launches > (1 << 20)) { set_error("max_launches must be in [0, 2^20]"); return LAT_EINVAL; }
  CL_HIP(hipStreamSynchronize(h->stream));
  drop_timer(h);
  h->timer.reserve(2 * (size_t)max_launches);
  for (int i = 0; i < 2 * max_launches; ++i) {
    hipEvent_t e;
    hipError_t r = hipEventCreate(&e);
    if (r != hipSuccess) {
      drop_timer(h);
      set_error(std::string("hipEventCreate: ") + hipGetErrorString(r));
      return LAT_EHIP;
    }
    h->timer.push_back(e);
  }
  return LAT_OK;
}

int lattice_pass_timer_read(lattice_t* h, double* total_ms, int64_t* launches) {
  if (!h || !total_ms || !launches) { set_error("NULL argument"); return LAT_EINVAL; }
  CL_HIP(hipStreamSynchronize(h->stream));
  double t = 0.0;
  for (size_t i = 0; i < h->timer_used; ++i) {
    float ms = 0.0f;
    CL_HIP(hipEventElapsedTime(&ms, h->timer[2 * i], h->timer[2 * i + 1]));
    t += ms;
  }
  *total_ms = t;
  *launches = (int64_t)h->timer_used;
  h->timer_used = 0;
  return LAT_OK;
}

int lattice_get_tiling(lattice_t* h, int32_t* tz, int32_t* by, int32_t* ry, int32_t* xc) {
  if (!h) { set_error("NULL handle"); return LAT_EINVAL; }
  if (tz) *tz = h->tile.tz;
  if (by) *by = h->tile.by;
  if (ry) *ry = h->tile.ry;
  if (xc) *xc = h->tile.xc;
  return LAT_OK;
}

int lattice_set_tiling(lattice_t* h, int32_t tz, int32_t by, int32_t ry, int32_t xc) {
  if (!h) { set_error("NULL handle"); return LAT_EINVAL; }
  Tiling t{tz, by, ry, xc};
  if (!tiling_ok(h, t)) { set_error("tile shape not compiled or does not divide N"); return LAT_EINVAL; }
  h->tile = t;
  return LAT_OK;
}

int lattice_field_device_ptr(lattice_t* h, int c, void** ptr, int32_t* elem_bytes) {
  if (!h || !ptr) { set_error("NULL argument"); return LAT_EINVAL; }
  if (c < 0 || c >= h->ncomp) { set_error("component out of range"); return LAT_EINVAL; }
  *ptr = h->buf[h->cur][c];
  if (elem_bytes) *elem_bytes = h->p.precision == LAT_FP32 ? 4 : 8;
  return LAT_OK;
}

int lattice_set_state(lattice_t* h, const double* fields, const double* momenta, const double* links,
                      const double* link_momenta, const lattice_scalars* s) {
  if (!h || !fields || !momenta || !s) { set_error("NULL argument"); return LAT_EINVAL; }
  if (is_su2(h->p)) return su2_set_state(h, fields, momenta, links, link_momenta, s);
  const bool u1 = is_u1(h->p), nc = h->p.model == LAT_MODEL_U1_NC;
  if (u1 && (!links || !link_momenta)) { set_error("U1 state needs links and link momenta"); return LAT_EINVAL; }
  if (!u1 && (links || link_momenta)) { set_error("scalar state takes no links"); return LAT_EINVAL; }
  const int64_t V = (int64_t)h->p.N * h->p.N * h->p.N;
  const int nf = h->p.nf;
  std::vector<const double*> comps;
  for (int f = 0; f < nf; ++f) comps.push_back(fields + f * V);
  for (int f = 0; f < nf; ++f) comps.push_back(momenta + f * V);
  std::vector<double> phases;
  if (nc) {
    // the gauge field A_i is stored as given
    for (int i = 0; i < 3; ++i) comps.push_back(links + i * V);
    for (int c = 0; c < 3; ++c) comps.push_back(link_momenta + c * V);
  } else if (u1) {
    // a unit link (Re, Im) is stored by its phase
    phases.resize((size_t)3 * V);
    for (int i = 0; i < 3; ++i)
      for (int64_t k = 0; k < V; ++k) {
        const double re = links[(2 * i) * V + k], im = links[(2 * i + 1) * V + k];
        if (!std::isfinite(re) || !std::isfinite(im)) { set_error("non-finite link"); return LAT_ENONFINITE; }
        phases[(size_t)i * V + k] = std::atan2(im, re);
      }
    for (int i = 0; i < 3; ++i) comps.push_back(phases.data() + (size_t)i * V);
    for (int c = 0; c < 3; ++c) comps.push_back(link_momenta + c * V);
  }
  for (size_t c = 0; c < comps.size(); ++c)
    for (int64_t i = 0; i < V; ++i)
      if (!std::isfinite(comps[c][i])) { set_error("non-finite value in state"); return LAT_ENONFINITE; }
  int rc = upload_components(h, comps.data(), (int)comps.size());
  if (rc) return rc;
  rc = upload_scalars(h, s->a, s->b, s->eta);
  if (rc) return rc;
  h->staggered = s->staggered ? 1 : 0;
  h->step = s->step;
  return LAT_OK;
}

int lattice_get_state(lattice_t* h, double* fields, double* momenta, double* links, double* link_momenta,
                      lattice_scalars* s) {
  if (!h) { set_error("NULL handle"); return LAT_EINVAL; }
  if (is_su2(h->p)) return su2_get_state(h, fields, momenta, links, link_momenta, s);
  const int64_t V = (int64_t)h->p.N * h->p.N * h->p.N;
  const int nf = h->p.nf;
  const bool u1 = is_u1(h->p), nc = h->p.model == LAT_MODEL_U1_NC;
  std::vector<double*> comps((size_t)h->ncomp, nullptr);
  for (int f = 0; f < nf; ++f) {
    if (fields) comps[f] = fields + f * V;
    if (momenta) comps[nf + f] = momenta + f * V;
  }
  std::vector<double> phases;
  if (nc) {
    for (int i = 0; i < 3; ++i) if (links) comps[4 + i] = links + i * V;
    for (int c = 0; c < 3; ++c) if (link_momenta) comps[7 + c] = link_momenta + c * V;
  } else if (u1) {
    if (links) {
      phases.resize((size_t)3 * V);
      for (int i = 0; i < 3; ++i) comps[4 + i] = phases.data() + (size_t)i * V;
    }
    for (int c = 0; c < 3; ++c) if (link_momenta) comps[7 + c] = link_momenta + c * V;
  }
  int rc = download_components(h, comps.data(), (int)comps.size());
  if (rc) return rc;
  if (u1 && !nc && links) {
    for (int i = 0; i < 3; ++i)
      for (int64_t k = 0; k < V; ++k) {
        const double t = phases[(size_t)i * V + k];
        links[(2 * i) * V + k] = std::cos(t);
        links[(2 * i + 1) * V + k] = std::sin(t);
      }
  }
  if (s) {
    DevState d;
    CL_HIP(hipMemcpyAsync(&d, h->st, sizeof(DevState), hipMemcpyDeviceToHost, h->stream));
    CL_HIP(hipStreamSynchronize(h->stream));
    s->a = d.a;
    s->b = d.b;
    s->eta = d.eta;
    s->step = h->step;
    s->staggered = h->staggered;
    s->reserved = 0;
  }
  return LAT_OK;
}

// SU(2) x U(1): fields, momenta 4 N^3 each; links = the U(1) links (Re, Im),
// 3*2*N^3, then the SU(2) links (c0, c1, c2, c3), 3*4*N^3; link momenta =
// pi_A (3*N^3) then pi_B (direction i, component a: 9*N^3).  U(1) links are
// stored by phase.
static int su2_set_state(lattice_t* h, const double* fields, const double* momenta, const double* links,
                         const double* link_momenta, const lattice_scalars* s) {
  if (!links || !link_momenta) { set_error("SU(2) x U(1) state needs links and link momenta"); return LAT_EINVAL; }
  const int64_t V = (int64_t)h->p.N * h->p.N * h->p.N;
  std::vector<const double*> comps;
  for (int k = 0; k < 4; ++k) comps.push_back(fields + k * V);
  for (int k = 0; k < 4; ++k) comps.push_back(momenta + k * V);
  std::vector<double> phases((size_t)3 * V);
  for (int i = 0; i < 3; ++i)
    for (int64_t k = 0; k < V; ++k) {
      const double re = links[(2 * i) * V + k], im = links[(2 * i + 1) * V + k];
      if (!std::isfinite(re) || !std::isfinite(im)) { set_error("non-finite link"); return LAT_ENONFINITE; }
      phases[(size_t)i * V + k] = std::atan2(im, re);
    }
  for (int i = 0; i < 3; ++i) comps.push_back(phases.data() + (size_t)i * V);
  for (int i = 0; i < 3; ++i) comps.push_back(link_momenta + i * V);
  for (int k = 0; k < 12; ++k) comps.push_back(links + (6 + k) * V);
  for (int k = 0; k < 9; ++k) comps.push_back(link_momenta + (3 + k) * V);
  for (size_t c = 0; c < comps.size(); ++c)
    for (int64_t i = 0; i < V; ++i)
      if (!std::isfinite(comps[c][i])) { set_error("non-finite value in state"); return LAT_ENONFINITE; }
  int rc = upload_components(h, comps.data(), (int)comps.size());
  if (rc) return rc;
  rc = upload_scalars(h, s->a, s->b, s->eta);
  if (rc) return rc;
  h->staggered = s->staggered ? 1 : 0;
  h->step = s->step;
  return LAT_OK;
}

static int su2_get_state(lattice_t* h, double* fields, double* momenta, double* links, double* link_momenta,
                         lattice_scalars* s) {
  const int64_t V = (int64_t)h->p.N * h->p.N * h->p.N;
  std::vector<double*> comps((size_t)h->ncomp, nullptr);
  for (int k = 0; k < 4; ++k) {
    if (fields) comps[k] = fields + k * V;
    if (momenta) comps[4 + k] = momenta + k * V;
  }
  std::vector<double> phases;
  if (links) {
    phases.resize((size_t)3 * V);
    for (int i = 0; i < 3; ++i) comps[8 + i] = phases.data() + (size_t)i * V;
    for (int k = 0; k < 12; ++k) comps[14 + k] = links + (6 + k) * V;
  }
  if (link_momenta) {
    for (int i = 0; i < 3; ++i) comps[11 + i] = link_momenta + i * V;
    for (int k = 0; k < 9; ++k) comps[26 + k] = link_momenta + (3 + k) * V;
  }
  int rc = download_components(h, comps.data(), (int)comps.size());
  if (rc) return rc;
  if (links) {
    for (int i = 0; i < 3; ++i)
      for (int64_t k = 0; k < V; ++k) {
        const double t = phases[(size_t)i * V + k];
        links[(2 * i) * V + k] = std::cos(t);
        links[(2 * i + 1) * V + k] = std::sin(t);
      }
  }
  if (s) {
    DevState d;
    CL_HIP(hipMemcpyAsync(&d, h->st, sizeof(DevState), hipMemcpyDeviceToHost, h->stream));
    CL_HIP(hipStreamSynchronize(h->stream));
    s->a = d.a;
    s->b = d.b;
    s->eta = d.eta;
    s->step = h->step;
    s->staggered = h->staggered;
    s->reserved = 0;
  }
  return LAT_OK;
}

int lattice_step(lattice_t* h, int64_t nsteps) {
  if (!h) { set_error("NULL handle"); return LAT_EINVAL; }
  if (nsteps < 0) { set_error("nsteps < 0"); return LAT_EINVAL; }
  if (is_u1(h->p)) return u1_step(h, nsteps);
  if (is_su2(h->p)) return su2_step(h, nsteps);
  return scalar_step(h, nsteps);
}

int lattice_energies(lattice_t* h, lattice_obs* out) {
  if (!h || !out) { set_error("NULL argument"); return LAT_EINVAL; }
  int rc = is_u1(h->p) ? u1_energies(h) : is_su2(h->p) ? su2_energies(h) : scalar_energies(h);
  if (rc) return rc;
  DevState d;
  CL_HIP(hipMemcpyAsync(&d, h->st, sizeof(DevState), hipMemcpyDeviceToHost, h->stream));
  CL_HIP(hipStreamSynchronize(h->stream));
  *out = d.obs;
  out->step = h->step;
  out->staggered = h->staggered;
  if (d.nonfinite) { set_error("non-finite volume average"); return LAT_ENONFINITE; }
  return LAT_OK;
}

}  // extern "C"

namespace cl {

// ---------------------------------------------------------------------------
// state transfer
// ---------------------------------------------------------------------------
int upload_components(lattice* h, const double* const* comps, int n) {
  const int64_t V = (int64_t)h->p.N * h->p.N * h->p.N;
  const bool f32 = h->p.precision == LAT_FP32;
  std::vector<float> tmp32;
  for (int c = 0; c < n; ++c) {
    void* d = h->buf[h->cur][c];
    if (f32) {
      tmp32.resize((size_t)V);
      for (int64_t i = 0; i < V; ++i) tmp32[(size_t)i] = (float)comps[c][i];
      CL_HIP(hipMemcpyAsync(d, tmp32.data(), (size_t)V * 4, hipMemcpyHostToDevice, h->stream));
      CL_HIP(hipStreamSynchronize(h->stream));
    } else {
      CL_HIP(hipMemcpyAsync(d, comps[c], (size_t)V * 8, hipMemcpyHostToDevice, h->stream));
      CL_HIP(hipStreamSynchronize(h->stream));
    }
  }
  return LAT_OK;
}

int download_components(lattice* h, double* const* comps, int n) {
  const int64_t V = (int64_t)h->p.N * h->p.N * h->p.N;
  const bool f32 = h->p.precision == LAT_FP32;
  std::vector<float> tmp32;
  for (int c = 0; c < n; ++c) {
    if (!comps[c]) continue;
    const void* d = h->buf[h->cur][c];
    if (f32) {
      tmp32.resize((size_t)V);
      CL_HIP(hipMemcpyAsync(tmp32.data(), d, (size_t)V * 4, hipMemcpyDeviceToHost, h->stream));
      CL_HIP(hipStreamSynchronize(h->stream));
      for (int64_t i = 0; i < V; ++i) comps[c][i] = (double)tmp32[(size_t)i];
    } else {
      CL_HIP(hipMemcpyAsync(comps[c], d, (size_t)V * 8, hipMemcpyDeviceToHost, h->stream));
      CL_HIP(hipStreamSynchronize(h->stream));
    }
  }
  return LAT_OK;
}

int upload_scalars(lattice* h, double a, double b, double eta) {
  DevState d;
  std::memset(&d, 0, sizeof(d));
  d.a = a;
  d.b = b;
  d.eta = eta;
  d.obs.gauss = NAN;
  CL_HIP(hipMemcpyAsync(h->st, &d, sizeof(DevState), hipMemcpyHostToDevice, h->stream));
  CL_HIP(hipStreamSynchronize(h->stream));
  return LAT_OK;
}

// ---------------------------------------------------------------------------
// scalar passes
// ---------------------------------------------------------------------------
void phys_of(const lattice* h, double* phys) {
  phys[0] = h->dx;
  phys[1] = h->p.alpha;
  phys[2] = h->p.fstar_over_mp * h->p.fstar_over_mp;
  phys[3] = h->p.m2[0];
  phys[4] = h->p.m2[1];
  phys[5] = h->p.lambda;
  phys[6] = h->p.q;
  phys[7] = h->p.dt;
}

int scalar_pass(lattice* h, const PassDesc& pd, bool full, PassChain* chain) {
  double phys[8];
  phys_of(h, phys);
  const int nf = h->p.nf;
  const void* src[4] = {nullptr, nullptr, nullptr, nullptr};
  void* dst[4] = {nullptr, nullptr, nullptr, nullptr};
  // component order in buffers: phi_0..phi_{nf-1}, pi_0..pi_{nf-1};
  // kernel slots: phi_0, phi_1, pi_0, pi_1
  for (int f = 0; f < nf; ++f) {
    src[f] = h->buf[h->cur][f];
    src[2 + f] = h->buf[h->cur][nf + f];
    dst[f] = h->buf[1 - h->cur][f];
    dst[2 + f] = h->buf[1 - h->cur][nf + f];
  }
  int nb = 0;
  hipEvent_t ev0 = nullptr, ev1 = nullptr;
  if (!full && 2 * h->timer_used + 1 < h->timer.size()) {
    ev0 = h->timer[2 * h->timer_used];
    ev1 = h->timer[2 * h->timer_used + 1];
    ++h->timer_used;
  }
  DevState* slot[2] = {h->st, h->st2};
  DevState* st = h->st;
  DevState* fin = h->st;
  double* part = h->partials;
  PrevPass prev{};
  if (chain) {
    if (full) { set_error("observation passes do not chain"); return LAT_EINVAL; }
    st = slot[chain->rd];
    part = (chain->k & 1) ? h->partials2 : h->partials;
    prev = chain->prev;
    if (prev.partials) prev.out = slot[1 - chain->rd];
    fin = nullptr;
  }
  hipError_t e = launch_scalar_pass(h->p.precision == LAT_FP32, nf, src, dst, h->p.N, h->tile.tz, h->tile.by,
                                    h->tile.ry, h->tile.xc, 1, phys, h->p.expansion, pd, part,
                                    std::max<int64_t>(h->max_blocks, kCUs), st, h->stream, &nb, full ? 1 : 0, ev0, ev1,
                                    prev, fin);
  if (e != hipSuccess) {
    set_error(std::string("scalar pass launch: ") + hipGetErrorString(e));
    return LAT_EHIP;
  }
  if (pd.write) h->cur ^= 1;
  if (chain) {
    if (prev.partials) chain->rd ^= 1;
    chain->prev = PrevPass{part, nb, pd, nullptr};
    ++chain->k;
  }
  return LAT_OK;
}

PassDesc pass(double wd, double wk1, double wk2, int mode, int write, int update) {
  PassDesc p;
  p.wd = wd;
  p.wk1 = wk1;
  p.wk2 = wk2;
  p.mode = mode;
  p.write = write;
  p.update = update;
  return p;
}

// Passes of one lattice_step(n) call (Sec. 3.3.2/4.3.2 with merged kicks; Sec.
// 4.2.1).  staggered is updated for leapfrog.
std::vector<PassDesc> pass_schedule(int integrator, const std::vector<double>& w, int* staggered, int64_t n) {
  std::vector<PassDesc> out;
  if (integrator == LAT_LF2) {
    if (!*staggered) {
      // pi_{-1/2} = pi_0 - (h/2) K, b_{-1/2} = b_0 - (h/2) K_a
      out.push_back(pass(0.0, 0.0, -0.5, MODE_VV, 1, 1));
      *staggered = 1;
    }
    if (n == 0) return out;
    out.push_back(pass(0.0, 0.0, 1.0, MODE_LF, 1, 1));                       // kick at phi_n
    for (int64_t j = 1; j < n; ++j) out.push_back(pass(1.0, 0.0, 1.0, MODE_LF, 1, 1));  // drift, kick
    out.push_back(pass(1.0, 0.0, 0.0, MODE_LF, 1, 1));                       // closing drift
    return out;
  }
  if (n == 0) return out;
  const int s = (int)w.size();
  out.push_back(pass(0.0, 0.0, 0.5 * w[0], MODE_VV, 1, 1));  // opening half kick
  for (int64_t it = 0; it < n; ++it)
    for (int p = 0; p < s; ++p) {
      const bool last = (it == n - 1) && (p == s - 1);
      const double nxt = last ? 0.0 : w[(p + 1) % s];
      out.push_back(pass(w[p], 0.5 * w[p], 0.5 * nxt, MODE_VV, 1, 1));
    }
  return out;
}

int scalar_step(lattice* h, int64_t n) {
  const std::vector<PassDesc> sched = pass_schedule(h->p.integrator, h->weights, &h->staggered, n);
  PassChain chain;
  for (const PassDesc& pd : sched) {
    const int rc = scalar_pass(h, pd, false, &chain);
    if (rc) return rc;
  }
  const int rc = scalar_chain_end(h, chain);
  if (rc) return rc;
  h->step += n;
  return LAT_OK;
}

// The last pass's finish, from the slot it started from into h->st.
int scalar_chain_end(lattice* h, const PassChain& chain) {
  if (chain.k == 0) return LAT_OK;
  double phys[8];
  phys_of(h, phys);
  DevState* slot[2] = {h->st, h->st2};
  const hipError_t e = launch_scalar_finish(h->p.precision == LAT_FP32, h->p.nf, h->p.N, phys, h->p.expansion,
                                            chain.prev.pd, const_cast<double*>(chain.prev.partials),
                                            chain.prev.nblocks, slot[chain.rd], h->st, h->stream);
  if (e != hipSuccess) {
    set_error(std::string("finish launch: ") + hipGetErrorString(e));
    return LAT_EHIP;
  }
  return LAT_OK;
}

int scalar_energies(lattice* h) {
  if (h->p.integrator == LAT_LF2 && h->staggered) return scalar_pass(h, pass(0.0, 0.0, 1.0, MODE_LF, 0, 0), true);
  return scalar_pass(h, pass(0.0, 0.0, 0.0, MODE_VV, 0, 0), true);
}

// ---------------------------------------------------------------------------
// tiling
// ---------------------------------------------------------------------------
bool tiling_ok(const lattice* h, const Tiling& t) {
  if (is_su2(h->p)) return false;  // its passes have one tile
  bool compiled = false;
  const int fp32 = h->p.precision == LAT_FP32;
  const bool u1 = is_u1(h->p);
  const int ns = u1 ? u1_num_shapes(fp32) : num_shapes(fp32, h->p.nf);
  for (int i = 0; i < ns; ++i) {
    int tz, by, ry;
    if (u1) u1_get_shape(fp32, i, &tz, &by, &ry);
    else if (!get_shape(fp32, h->p.nf, h->p.N, i, &tz, &by, &ry)) continue;
    if (tz == t.tz && by == t.by && ry == t.ry) compiled = true;
  }
  if (!compiled) return false;
  const int N = h->p.N;
  if (!u1 && t.ry == 1 && t.tz != N) return false;  // full-row tiles hold whole z-rows
  const int ty = t.by * t.ry;
  if (N % t.tz || N % ty || t.xc < 1 || N % t.xc) return false;
  const int64_t nb = (int64_t)(N / t.tz) * (N / ty) * (N / t.xc);
  return nb <= h->max_blocks;
}

void default_tiling(lattice* h) {
  const int N = h->p.N;
  if (is_su2(h->p)) {
    h->tile = Tiling{0, 0, 0, 0};
    return;
  }
  // FP64 two-field lattices take full rows, eight to a block, whose pass shares
  // the planes by itself (two and four rows a block: 32^3 7.9 us a pass with
  // four, 7.1 with eight; 64^3 14.2, 10.2 and 8.7; 96^3 17.5 to 21.4 with four,
  // 17.5 with eight; the best general tile 11.8 at 64^3).
  h->tile = Tiling{N, 8, 1, 8};
  if (!is_u1(h->p) && h->p.precision == LAT_FP64 && h->p.nf == 2 && tiling_ok(h, h->tile)) return;
  // Else, below 128^3 (where no tuner runs) a pass is latency: many blocks that
  // march few planes, down to 1024 sites a block, up to 512 blocks (scalar FP32
  // 64^3: 8.0 us a pass with two planes a block, 9.6 with four; 96^3: 11.6 with
  // four, 12.8 with two; U(1) 64^3: 20.7 with two, 27.2 with four; 96^3: 34.3
  // with eight, 42.5 with four).
  Tiling t = is_u1(h->p) ? Tiling{32, 8, 1, 1} : Tiling{32, 8, 2, 1};
  if (N % 64 == 0 && !(is_u1(h->p) && h->p.precision == LAT_FP64)) t = Tiling{64, 4, 2, 1};
  const int64_t plane = (int64_t)t.tz * t.by * t.ry, tiles = (int64_t)N * N / plane;
  for (int c = 1; c <= N; ++c) {
    if (N % c) continue;
    t.xc = c;
    if (plane * c >= 1024 && tiles * (N / c) <= 512 && tiling_ok(h, t)) break;
  }
  h->tile = tiling_ok(h, t) ? t : is_u1(h->p) ? Tiling{32, 8, 1, 8} : Tiling{32, 8, 2, 8};
}

// Time every compiled tile shape and x-chunk on zeroed state buffers with
// chains of full passes (a, b left untouched) that ping-pong between the two
// buffers as lattice_step does; keep the fastest.  One sweep over every
// candidate, then two over those within a tenth of the quickest, each
// keeping its quicker time, so that one slow sample (a clock ramp, a
// neighbour's traffic) cannot hand the choice to a tile 5-10% slower.  The
// caller builds the initial state afterwards.
int autotune(lattice* h) {
  // zero state (finite arithmetic), a = 1, b = 0; the caller builds the real
  // state after tuning
  for (int c = 0; c < h->ncomp; ++c) {
    CL_HIP(hipMemsetAsync(h->buf[0][c], 0, h->comp_bytes, h->stream));
    CL_HIP(hipMemsetAsync(h->buf[1][c], 0, h->comp_bytes, h->stream));
  }
  int rc = upload_scalars(h, 1.0, 0.0, 0.0);
  if (rc) return rc;
  hipEvent_t e0, e1;
  CL_HIP(hipEventCreate(&e0));
  CL_HIP(hipEventCreate(&e1));
  const bool u1 = is_u1(h->p);
  // planes per block: few enough to fill the chip, many enough for the two
  // planes every block reads beyond its own
  std::vector<int> xcs = {8, 12, 16, 24, 32, 48, 64};
  if (u1 || h->p.N < 256) xcs.insert(xcs.begin(), {4, 6});
  Tiling bt = h->tile;
  const int fp32 = h->p.precision == LAT_FP32;
  const PassDesc pd = pass(1.0, 0.5, 0.5, MODE_VV, 1, 0);
  // k passes chained as lattice_step chains them, and the closing finish
  auto run = [&](int k) {
    PassChain c;
    int r = LAT_OK;
    for (int j = 0; j < k && !r; ++j) r = u1 ? u1_pass(h, pd, &c) : scalar_pass(h, pd, false, &c);
    if (!r) r = u1 ? u1_chain_end(h, c) : scalar_chain_end(h, c);
    return r;
  };
  std::vector<Tiling> cand;
  const int ns = u1 ? u1_num_shapes(fp32) : num_shapes(fp32, h->p.nf);
  for (int i = 0; i < ns; ++i) {
    int tz, by, ry;
    if (u1) u1_get_shape(fp32, i, &tz, &by, &ry);
    else if (!get_shape(fp32, h->p.nf, h->p.N, i, &tz, &by, &ry)) continue;
    for (int xc : xcs) {
      const Tiling t{tz, by, ry, xc};
      if (tiling_ok(h, t)) cand.push_back(t);
    }
  }
  std::vector<float> tbest(cand.size(), 1e30f);
  float least = 1e30f;
  for (int sweep = 0; sweep < 3 && !rc; ++sweep) {
    for (size_t i = 0; i < cand.size() && !rc; ++i) {
      if (sweep && tbest[i] > 1.1f * least) continue;
      h->tile = cand[i];
      rc = run(2);  // warm-up, ping-pong
      if (rc) break;
      hipError_t e = hipEventRecord(e0, h->stream);
      if (e == hipSuccess) rc = run(h->p.N < 256 ? 12 : 6);
      if (!rc && e == hipSuccess) e = hipEventRecord(e1, h->stream);
      if (!rc && e == hipSuccess) e = hipEventSynchronize(e1);
      float ms = 0.f;
      if (!rc && e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
      if (e != hipSuccess) {
        set_error(std::string("autotune timing: ") + hipGetErrorString(e));
        rc = LAT_EHIP;
        break;
      }
      tbest[i] = std::min(tbest[i], ms);
      least = std::min(least, ms);
    }
  }
  float best = 1e30f;
  for (size_t i = 0; i < cand.size(); ++i)
    if (tbest[i] < best) { best = tbest[i]; bt = cand[i]; }
  hipEventDestroy(e0);
  hipEventDestroy(e1);
  h->cur = 0;
  h->tile = bt;
  return rc;
}

}  // namespace cl
