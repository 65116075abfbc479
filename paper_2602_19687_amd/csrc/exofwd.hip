// Host side of the C ABI: configuration checks, table encoding and upload,
// workspace, kernel launches and per-kernel event timing.
#include "../../include/exofwd.h"
#include "kernels.h"
#include "adjoint.h"
#include "emission.h"
#include "ck.h"

#include <algorithm>
#include <array>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <fstream>
#include <mutex>
#include <sstream>
#include <string>
#include <vector>

using namespace exofwd;

struct exofwd_ctx {
  Model m{};
  Work w{};
  Tables tb{};
  AdjWork aw{};
  int precision = 0;
  int device = 0;
  int batch_max = 0;
  std::vector<void*> allocs;
  int64_t bytes = 0;
  int32_t* d_lo = nullptr;
  int32_t* d_hi = nullptr;
  double* d_y = nullptr;
  double* d_yerr = nullptr;
  uint8_t* d_mask = nullptr;
  std::string err;
  bool profiling = false;
  struct Ev {
    std::string name;
    hipEvent_t a, b;
  };
  std::vector<Ev> events;
  // captured launch sequences, keyed by call kind, batch, pointers and stream
  struct Graph {
    int kind, B;
    std::array<const void*, 7> ptr;
    hipStream_t st;
    hipGraphExec_t exec;
    uint64_t used;
  };
  std::vector<Graph> graphs;
  bool use_graphs = false;
  bool capturing = false;
  uint64_t tick = 0;
};

namespace {

exofwd_status fail(exofwd_ctx* c, exofwd_status s, const std::string& msg) {
  if (c) c->err = msg;
  return s;
}

template <typename T>
T* dalloc(exofwd_ctx* c, size_t count) {
  if (count == 0) count = 1;
  void* p = nullptr;
  if (hipMalloc(&p, count * sizeof(T)) != hipSuccess) return nullptr;
  c->allocs.push_back(p);
  c->bytes += (int64_t)(count * sizeof(T));
  return static_cast<T*>(p);
}

template <typename T>
bool upload(T* dst, const T* src, size_t count) {
  return hipMemcpy(dst, src, count * sizeof(T), hipMemcpyHostToDevice) == hipSuccess;
}

// a row of an FP64 table: entries below kAbsentLog (the lowest double, say) would overflow
// on the way to log2
void copy_log_row(double* dst, const double* src, int n) {
  for (int i = 0; i < n; ++i) dst[i] = std::max(src[i], kAbsentLog);
}

bool ascending(const double* v, int n) {
  for (int i = 0; i + 1 < n; ++i)
    if (!(v[i + 1] > v[i])) return false;
  return true;
}

// Gauss-Legendre nodes/weights on [-1, 1] by Newton iteration on P_n.
void gauss_legendre(int n, double* x, double* wgt) {
  for (int i = 0; i < n; ++i) {
    double z = std::cos(M_PI * (i + 0.75) / (n + 0.5));
    double dp = 0.0;
    for (int it = 0; it < 100; ++it) {
      double p0 = 1.0, p1 = z;
      for (int k = 2; k <= n; ++k) {
        double p2 = ((2.0 * k - 1.0) * z * p1 - (k - 1.0) * p0) / k;
        p0 = p1;
        p1 = p2;
      }
      if (n == 1) { p1 = z; p0 = 1.0; }
      dp = n * (z * p1 - p0) / (z * z - 1.0);
      double dz = p1 / dp;
      z -= dz;
      if (std::fabs(dz) < 1e-16) break;
    }
    x[i] = z;
    wgt[i] = 2.0 / ((1.0 - z * z) * dp * dp);
  }
}

// Reduced-precision table storage: per (source, nu) offset c = float((min+max)/2)
// of log2 sigma over the interpolation axes, entries float16(log2 sigma - c);
// with `wide` each entry is float32(log2 sigma - c) in the space of two halves
// (emission, whose flux is sensitive to opacity error).
void encode_tables(const double* log10_tab, int n_src, int n_rows, int n_nu, int n_nu_pad, std::vector<_Float16>& h,
                   std::vector<float>& c, bool wide = false) {
  const int k = wide ? 2 : 1;
  h.assign((size_t)n_src * n_rows * n_nu_pad * k, (_Float16)0.0f);
  c.assign((size_t)n_src * n_nu_pad, -1000.0f);
  for (int s = 0; s < n_src; ++s) {
    const double* t = log10_tab + (size_t)s * n_rows * n_nu;
    for (int i = 0; i < n_nu; ++i) {
      double mn = INFINITY, mx = -INFINITY;
      for (int r = 0; r < n_rows; ++r) {
        double v = t[(size_t)r * n_nu + i] * kLog2_10;
        mn = v < mn ? v : mn;
        mx = v > mx ? v : mx;
      }
      const float cf = (float)(0.5 * (mn + mx));
      c[(size_t)s * n_nu_pad + i] = cf;
      for (int r = 0; r < n_rows; ++r) {
        double v = t[(size_t)r * n_nu + i] * kLog2_10 - (double)cf;
        const size_t e = ((size_t)s * n_rows + r) * n_nu_pad + i;
        if (wide) {
          const float f = (float)v;
          std::memcpy(&h[2 * e], &f, sizeof f);
          continue;
        }
        h[e] = (_Float16)v;
      }
    }
  }
}

exofwd_status check_hip(exofwd_ctx* c, hipError_t e, const char* what) {
  if (e == hipSuccess) return EXOFWD_OK;
  return fail(c, EXOFWD_ERR_DEVICE, std::string(what) + ": " + hipGetErrorString(e));
}

// ---- scratch of the allocation-free forward call (exofwd_forward_noalloc)
// Every device the library runs on holds one copy of this array until the process
// ends.  Host code never passes the array's name to a kernel (on the host it is only
// a stand-in for the symbol): it uses the device address looked up below.
static __device__ __align__(256) unsigned char scratch[EXOFWD_NOALLOC_SCRATCH_BYTES];
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_addr[kMaxDevices];      // device address of `scratch` on each device, once looked up
bool g_scratch_tried[kMaxDevices];

// Looks up the array's address on `dev`, which must be the current device
// (once per device; later calls return the stored address, nullptr if the lookup failed).
void* scratch_address(int dev) {
  if (dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_tried[dev]) {
    g_scratch_tried[dev] = true;
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) == hipSuccess) g_scratch_addr[dev] = p;
  }
  return g_scratch_addr[dev];
}

}  // namespace

// ---------------------------------------------------------------------------
// kernel timing helpers (used by every launch site)
namespace exofwd {
void prof_begin(exofwd_ctx* c, const char* name, hipStream_t st) {
  if (!c->profiling || c->capturing) return;
  exofwd_ctx::Ev e;
  e.name = name;
  hipEventCreate(&e.a);
  hipEventCreate(&e.b);
  hipEventRecord(e.a, st);
  c->events.push_back(e);
}
void prof_end(exofwd_ctx* c, hipStream_t st) {
  if (!c->profiling || c->capturing || c->events.empty()) return;
  hipEventRecord(c->events.back().b, st);
}
}  // namespace exofwd

// Text of the last exofwd_create failure on this thread (exofwd_last_error(NULL)).
static thread_local std::string g_create_err;

extern "C" {

const char* exofwd_strerror(exofwd_status s) {
  switch (s) {
    case EXOFWD_OK: return "ok";
    case EXOFWD_ERR_ARG: return "invalid argument";
    case EXOFWD_ERR_SHAPE: return "shape mismatch";
    case EXOFWD_ERR_CONFIG: return "invalid configuration";
    case EXOFWD_ERR_NOMEM: return "device allocation failed";
    case EXOFWD_ERR_DEVICE: return "HIP runtime error";
    case EXOFWD_ERR_UNSUPPORTED: return "unsupported request";
  }
  return "unknown status";
}

const char* exofwd_last_error(const exofwd_ctx* c) {
  if (c) return c->err.c_str();
  return g_create_err.empty() ? "null context" : g_create_err.c_str();
}
int32_t exofwd_num_params(const exofwd_ctx* c) { return c ? c->m.P : -1; }
int32_t exofwd_num_nu(const exofwd_ctx* c) { return c ? c->m.n_nu : -1; }
int32_t exofwd_num_bins(const exofwd_ctx* c) { return c ? c->m.K : -1; }
int32_t exofwd_precision(const exofwd_ctx* c) { return c ? c->precision : -1; }
int32_t exofwd_grad_supported(const exofwd_ctx* c) {
  return c ? (adjoint_supported(c->m, c->precision == EXOFWD_PREC_FP64) ? 1 : 0) : -1;
}
int64_t exofwd_device_bytes(const exofwd_ctx* c) { return c ? c->bytes : -1; }

static void drop_graphs(exofwd_ctx* c) {
  for (auto& g : c->graphs) hipGraphExecDestroy(g.exec);
  c->graphs.clear();
}

exofwd_status exofwd_destroy(exofwd_ctx* c) {
  if (!c) return EXOFWD_OK;
  hipSetDevice(c->device);
  hipDeviceSynchronize();
  drop_graphs(c);
  for (auto& e : c->events) {
    hipEventDestroy(e.a);
    hipEventDestroy(e.b);
  }
  for (void* p : c->allocs) hipFree(p);
  delete c;
  return EXOFWD_OK;
}

static exofwd_status create_fail(exofwd_status s, const std::string& msg) {
  g_create_err = "exofwd_create: " + msg;
  return s;
}

static bool all_finite(const double* v, size_t n) {
  for (size_t i = 0; i < n; ++i)
    if (!std::isfinite(v[i])) return false;
  return true;
}

exofwd_status exofwd_create(const exofwd_config* cfg, exofwd_ctx** out) {
  if (!out) return create_fail(EXOFWD_ERR_ARG, "out is NULL");
  *out = nullptr;
  if (!cfg) return create_fail(EXOFWD_ERR_ARG, "cfg is NULL");
  g_create_err.clear();
  // ---- validation (nothing touches the device before this passes)
  const auto& g = *cfg;
  const exofwd_status E = EXOFWD_ERR_CONFIG;
  if (g.mode != EXOFWD_TRANSMISSION && g.mode != EXOFWD_EMISSION) return create_fail(E, "unknown mode");
  if (g.precision != EXOFWD_PREC_FP64 && g.precision != EXOFWD_PREC_MIXED) return create_fail(E, "unknown precision");
  if (g.tp_kind < EXOFWD_TP_ISOTHERMAL || g.tp_kind > EXOFWD_TP_GUILLOT7) return create_fail(E, "unknown T-p profile");
  if (g.tp_kind == EXOFWD_TP_PCHIP && (g.n_knots < 2 || g.n_knots > kMaxKnots))
    return create_fail(E, "n_knots outside [2, 8]");
  if (g.n_species < 1 || g.n_species > kMaxSpecies) return create_fail(E, "n_species outside [1, 8]");
  if (g.n_layers_max < 1 || g.n_layers_max > kMaxLayers) return create_fail(E, "n_layers_max outside [1, 160]");
  if (g.batch_max < 1) return create_fail(E, "batch_max < 1");
  if (g.n_nu < 1 || !g.nu || !ascending(g.nu, g.n_nu) || !(g.nu[0] > 0.0))
    return create_fail(E, "nu must hold n_nu >= 1 positive ascending wavenumbers");
  if (g.n_t < 2 || g.n_t > kMaxAxis || g.n_p < 2 || g.n_p > kMaxAxis || !g.t_grid || !g.logp_grid || !g.log10_xsec)
    return create_fail(E, "table axes need 2..255 points each and the table pointers");
  if (!ascending(g.t_grid, g.n_t) || !ascending(g.logp_grid, g.n_p)) return create_fail(E, "table axes not ascending");
  if (g.has_cia && (g.n_tc < 2 || g.n_tc > kMaxAxis || !g.tc_grid || !g.log10_cia || !ascending(g.tc_grid, g.n_tc)))
    return create_fail(E, "CIA axis needs 2..255 ascending temperatures and the CIA table");
  if (!(g.mu_fixed > 0.0) && !g.species_mass) return create_fail(E, "species_mass is NULL and mu_fixed <= 0");
  if (g.n_bins < 1 || !g.bin_lo || !g.bin_hi || !g.y_obs || !g.y_err) return create_fail(E, "bins or data missing");
  for (int k = 0; k < g.n_bins; ++k) {
    if (g.bin_lo[k] < 0 || g.bin_hi[k] > g.n_nu || g.bin_lo[k] >= g.bin_hi[k] || !(g.y_err[k] > 0.0))
      return create_fail(E, "bin " + std::to_string(k) + " empty, outside [0, n_nu) or with y_err <= 0");
    // bins are ordered and disjoint, so every wavenumber feeds at most one bin
    if (k > 0 && g.bin_lo[k] < g.bin_hi[k - 1]) return create_fail(E, "bins not ordered and disjoint");
  }
  if (!(g.p_bot_bar > g.p_top_bar) || !(g.p_top_bar > 0.0) || !(g.p_ref_bar > 0.0))
    return create_fail(E, "pressures need p_bot > p_top > 0 and p_ref > 0");
  if (!(g.r_p > 0.0) || !(g.r_s > 0.0) || !(g.g_ref > 0.0)) return create_fail(E, "r_p, r_s and g_ref must be > 0");
  if (g.mode == EXOFWD_EMISSION && (g.n_mu < 1 || g.n_mu > kMaxMu || !(g.t_star > 0.0)))
    return create_fail(E, "emission needs n_mu in [1, 8] and t_star > 0");
  if (g.has_cloud) {
    if (g.cloud_model != EXOFWD_CLOUD_GREY_DECK && g.cloud_model != EXOFWD_CLOUD_NONGREY)
      return create_fail(E, "unknown cloud model");
    if (g.cloud_model == EXOFWD_CLOUD_NONGREY &&
        (g.mode != EXOFWD_TRANSMISSION || g.cloud_profile < EXOFWD_QPROF_UNIFORM || g.cloud_profile > EXOFWD_QPROF_POWER ||
         g.cloud_qext < EXOFWD_QEXT_FIT || g.cloud_qext > EXOFWD_QEXT_GREY))
      return create_fail(E, "the non-grey cloud is a transmission model with a known profile and Q_ext form");
  }
  if (g.has_fcld && (!g.has_cloud || g.mode != EXOFWD_TRANSMISSION))
    return create_fail(E, "cloudy/clear mixing needs a transmission model with a cloud");
  if (g.has_bd && (g.mode != EXOFWD_EMISSION || g.has_scale || !(g.bd_distance > 0.0)))
    return create_fail(E, "an isolated object is an emission model without R_p scaling and with a distance > 0");
  // correlated-k tables: kCkG g-points per bin, reduced precision, forward model only
  if (g.ck_g != 0) {
    if (g.ck_g != kCkG) return create_fail(EXOFWD_ERR_UNSUPPORTED, "correlated-k tables need exactly 8 g-points");
    if (g.precision != EXOFWD_PREC_MIXED)
      return create_fail(EXOFWD_ERR_UNSUPPORTED, "correlated-k tables run in reduced precision only");
    if (g.ck_mix != EXOFWD_CK_RORR && g.ck_mix != EXOFWD_CK_PRODUCT) return create_fail(E, "unknown ck_mix");
    if (g.ck_mix == EXOFWD_CK_PRODUCT && g.mode != EXOFWD_TRANSMISSION)
      return create_fail(E, "the product of the absorbers' transmission functions is a transmission mixing");
    if (g.has_fcld || g.has_bd || (g.has_cloud && g.cloud_model != EXOFWD_CLOUD_GREY_DECK))
      return create_fail(EXOFWD_ERR_UNSUPPORTED,
                         "correlated-k tables take no cloudy/clear mixing, isolated object or non-grey cloud");
    if (!g.ck_weights) return create_fail(E, "ck_weights is NULL");
    double sw = 0.0;
    for (int i = 0; i < g.ck_g; ++i) {
      if (!(g.ck_weights[i] > 0.0)) return create_fail(E, "ck_weights must be > 0");
      sw += g.ck_weights[i];
    }
    if (std::fabs(sw - 1.0) > 1e-9) return create_fail(E, "ck_weights must sum to 1");
  } else if (g.ck_mix != 0 || g.ck_weights) {
    return create_fail(E, "ck_mix and ck_weights need ck_g > 0");
  }
  const int gk = g.ck_g ? g.ck_g : 1;   // table columns per spectral point
  // The reduced-precision kernels read the encoded tables, and the gradient's stored
  // optical depths of a sample, through buffer resources whose range and offsets are
  // 32-bit: each of these buffers must stay below 2^31 bytes (checked before any
  // table is read).
  if (g.precision == EXOFWD_PREC_MIXED) {
    const uint64_t lim = 0x7fffffffull;
    const uint64_t npad = ((uint64_t)g.n_nu + kTileNu - 1) / kTileNu * kTileNu;
    const uint64_t eb = (g.mode == EXOFWD_EMISSION || g.ck_g) ? 4 : 2;
    const uint64_t lpad = ((uint64_t)g.n_layers_max + 31) / 32 * 32;
    const uint64_t tab = (uint64_t)g.n_species * g.n_t * g.n_p * npad * gk * eb;
    const uint64_t cia = g.has_cia ? 2ull * g.n_tc * npad * eb : 0;
    if (tab > lim || cia > lim || lpad * npad * gk * 4 > lim)
      return create_fail(EXOFWD_ERR_UNSUPPORTED,
                         "reduced precision addresses each table, and a sample's stored optical depths, with "
                         "32-bit offsets: line table " + std::to_string(tab) + " B, CIA table " +
                             std::to_string(cia) + " B, optical depths " + std::to_string(lpad * npad * gk * 4) +
                             " B; each must be below 2^31 B");
  }
  // log10 tables must be finite: a zero cross-section is given as a finite floor
  // (the reduced-precision encoding keeps each wavenumber's range over the grid)
  if (!all_finite(g.log10_xsec, (size_t)g.n_species * g.n_t * g.n_p * g.n_nu * gk))
    return create_fail(E, "log10_xsec holds a non-finite entry");
  if (g.has_cia && !all_finite(g.log10_cia, (size_t)2 * g.n_tc * g.n_nu))
    return create_fail(E, "log10_cia holds a non-finite entry");
  // a k-table row is a cumulative distribution's inverse: non-decreasing in g (the
  // mixing kernel merges the rows as sorted runs)
  if (g.ck_g) {
    const size_t rows = (size_t)g.n_species * g.n_t * g.n_p * g.n_nu;
    for (size_t r = 0; r < rows; ++r)
      for (int q = 1; q < g.ck_g; ++q)
        if (g.log10_xsec[r * g.ck_g + q] < g.log10_xsec[r * g.ck_g + q - 1])
          return create_fail(E, "log10_xsec: a k-table row decreases in g");
  }
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || g.device < 0 || g.device >= ndev)
    return create_fail(EXOFWD_ERR_DEVICE, "no HIP device with ordinal " + std::to_string(g.device));

  auto* c = new exofwd_ctx();
  c->precision = g.precision;
  c->device = g.device;
  c->batch_max = g.batch_max;
  if (hipSetDevice(g.device) != hipSuccess) {
    delete c;
    return create_fail(EXOFWD_ERR_DEVICE, "hipSetDevice failed");
  }
  // the allocation-free call's scratch address on this device (its failure only
  // disables that call, which then reports it)
  scratch_address(g.device);
  Model& m = c->m;
  m.mode = g.mode;
  m.tp_kind = g.tp_kind;
  m.n_knots = g.tp_kind == EXOFWD_TP_PCHIP ? g.n_knots : 0;
  m.S = g.n_species;
  m.L_max = g.n_layers_max;
  m.L_pad = (g.n_layers_max + 31) / 32 * 32;
  m.has_cia = g.has_cia ? 1 : 0;
  m.has_ray = g.has_rayleigh ? 1 : 0;
  m.has_cloud = g.has_cloud ? 1 : 0;
  m.cloud_ng = (g.has_cloud && g.cloud_model == EXOFWD_CLOUD_NONGREY) ? 1 : 0;
  m.cloud_profile = m.cloud_ng ? g.cloud_profile : 0;
  m.cloud_qext = m.cloud_ng ? g.cloud_qext : 0;
  // non-grey: [log10 r] + [a, log10 Q0] (fitted Q) + profile (1 or 3) + feature (4)
  m.n_cloud = !m.has_cloud ? 0
              : !m.cloud_ng ? 1
                            : (m.cloud_qext == kQextGrey ? 1 : 3) + (m.cloud_profile == kQprofUniform ? 1 : 3) +
                                  (m.cloud_qext == kQextFeature ? 4 : 0);
  m.has_scale = g.has_scale ? 1 : 0;
  m.has_offset = g.has_offset ? 1 : 0;
  m.n_mu = g.mode == EXOFWD_EMISSION ? g.n_mu : 0;
  m.n_nu = g.n_nu;
  m.n_nu_pad = (g.n_nu + kTileNu - 1) / kTileNu * kTileNu;
  m.n_tiles = m.n_nu_pad / kTileNu;
  m.n_tiles64 = m.n_nu_pad / kTile64;
  m.n_t = g.n_t;
  m.n_p = g.n_p;
  m.n_tc = g.has_cia ? g.n_tc : 2;
  m.K = g.n_bins;
  {
    // lanes per bin in the likelihood sums: about one wavenumber per lane or more
    const double mean = (double)(g.bin_hi[g.n_bins - 1] - g.bin_lo[0]) / g.n_bins;
    m.ll_lanes = mean >= 64 ? 64 : mean >= 32 ? 32 : mean >= 16 ? 16 : 8;
  }
  switch (g.tp_kind) {
    case EXOFWD_TP_ISOTHERMAL: m.n_tp = 1; break;
    case EXOFWD_TP_GUILLOT3: m.n_tp = 3; break;
    case EXOFWD_TP_PCHIP: m.n_tp = g.n_knots; break;
    case EXOFWD_TP_BARSTOW: m.n_tp = 1; break;
    case EXOFWD_TP_MILNE: m.n_tp = 5; break;
    default: m.n_tp = 7; break;   // EXOFWD_TP_GUILLOT7
  }
  int k = m.n_tp + m.S;
  m.idx_cloud = m.has_cloud ? k : -1;
  k += m.n_cloud;
  m.has_fcld = g.has_fcld ? 1 : 0;
  m.idx_fcld = m.has_fcld ? k++ : -1;
  m.has_bd = g.has_bd ? 1 : 0;
  m.idx_bd = m.has_bd ? k : -1;
  k += 2 * m.has_bd;
  m.bd_dist = g.has_bd ? g.bd_distance : 0.0;
  m.ck = g.ck_g ? 1 : 0;
  m.ck_mix = g.ck_mix;
  m.idx_scale = m.has_scale ? k++ : -1;
  m.idx_offset = m.has_offset ? k++ : -1;
  m.P = k;
  m.mu_fixed = g.mu_fixed;
  m.log10_pbot = std::log10(g.p_bot_bar);
  m.log10_ptop = std::log10(g.p_top_bar);
  m.p_ref = g.p_ref_bar * kBar;
  m.log10_pref = std::log10(m.p_ref / kBar);
  m.r_p = g.r_p;
  m.r_s = g.r_s;
  m.g_ref = g.g_ref;
  m.kappa_ir = g.kappa_ir;
  m.f_hem = g.f_hem;
  m.kappa_cloud = g.kappa_cloud;
  m.t_star = g.t_star;
  m.dilution = g.dilution;
  m.err_c = g.err_c;
  // zero without Rayleigh scattering: the gradient's composition terms use them as they are
  m.ray_h2 = m.has_ray ? g.ray_h2 : 0.0;
  m.ray_he = m.has_ray ? g.ray_he : 0.0;
  for (int s = 0; s < m.S; ++s) m.mass[s] = g.species_mass ? g.species_mass[s] : 0.0;
  if (m.n_mu > 0) {
    double x[kMaxMu], wg[kMaxMu];
    gauss_legendre(m.n_mu, x, wg);
    for (int i = 0; i < m.n_mu; ++i) {
      m.mu_nodes[i] = 0.5 * (x[i] + 1.0);
      m.mu_weights[i] = 0.5 * wg[i];
    }
  }

  const bool fp64 = g.precision == EXOFWD_PREC_FP64;
  // per-sample buffers hold the virtual samples (two per sample with the cloudy/clear mixing)
  const int Lp = m.L_pad, B = g.batch_max * (m.has_fcld ? 2 : 1), RL = rec_stride(m, fp64);
  const size_t np = (size_t)m.n_nu_pad;
  bool ok = true;
  auto A = [&](auto* p) { ok = ok && p != nullptr; return p; };

  // ---- grids and spectral axis
  double* d_t = A(dalloc<double>(c, m.n_t));
  double* d_p = A(dalloc<double>(c, m.n_p));
  double* d_tc = A(dalloc<double>(c, m.n_tc));
  double* d_nu = A(dalloc<double>(c, np));
  if (!ok) { exofwd_destroy(c); return create_fail(EXOFWD_ERR_NOMEM, "device allocation failed"); }
  std::vector<double> nu_pad(np, g.nu[g.n_nu - 1]);
  std::memcpy(nu_pad.data(), g.nu, sizeof(double) * g.n_nu);
  std::vector<double> tc(m.n_tc, 0.0);
  if (m.has_cia) std::memcpy(tc.data(), g.tc_grid, sizeof(double) * m.n_tc);
  else { tc[0] = 0.0; tc[1] = 1.0; }
  ok = upload(d_t, g.t_grid, m.n_t) && upload(d_p, g.logp_grid, m.n_p) && upload(d_tc, tc.data(), m.n_tc) &&
       upload(d_nu, nu_pad.data(), np);
  m.t_grid = d_t;
  m.logp_grid = d_p;
  m.tc_grid = d_tc;
  m.nu = d_nu;

  // ---- tables
  std::vector<double> nu4(np);
  for (size_t i = 0; i < np; ++i) nu4[i] = std::pow(nu_pad[i] / 1.0e4, 4);
  const int rows = m.n_t * m.n_p;
  if (fp64) {
    std::vector<double> t64((size_t)m.S * rows * np, -1000.0);
    for (int s = 0; s < m.S; ++s)
      for (int r = 0; r < rows; ++r)
        copy_log_row(&t64[((size_t)s * rows + r) * np], g.log10_xsec + ((size_t)s * rows + r) * g.n_nu, g.n_nu);
    double* d64 = A(dalloc<double>(c, t64.size()));
    double* dn4 = A(dalloc<double>(c, np));
    if (ok) ok = upload(d64, t64.data(), t64.size()) && upload(dn4, nu4.data(), np);
    c->tb.t64 = d64;
    c->tb.nu4d = dn4;
    if (m.has_cia) {
      std::vector<double> c64((size_t)2 * m.n_tc * np, -1000.0);
      for (int r = 0; r < 2 * m.n_tc; ++r)
        copy_log_row(&c64[(size_t)r * np], g.log10_cia + (size_t)r * g.n_nu, g.n_nu);
      double* dc = A(dalloc<double>(c, c64.size()));
      if (ok) ok = upload(dc, c64.data(), c64.size());
      c->tb.tc64 = dc;
    }
  } else {
    std::vector<_Float16> h;
    std::vector<float> off;
    const bool wide = m.mode == kEmission || m.ck;
    // correlated-k: one column per (bin, g-point), [bin][g] with the bins padded like wavenumbers
    encode_tables(g.log10_xsec, m.S, rows, g.n_nu * gk, (int)np * gk, h, off, wide);
    uint16_t* dh = A(dalloc<uint16_t>(c, h.size()));
    float* dc = A(dalloc<float>(c, off.size()));
    float* dn4 = A(dalloc<float>(c, np));
    std::vector<float> nu4f(np);
    for (size_t i = 0; i < np; ++i) nu4f[i] = (float)nu4[i];
    if (ok)
      ok = upload(dh, reinterpret_cast<const uint16_t*>(h.data()), h.size()) && upload(dc, off.data(), off.size()) &&
           upload(dn4, nu4f.data(), np);
    c->tb.h = dh;
    c->tb.c = dc;
    c->tb.nu4f = dn4;
    if (m.ck) {
      float wv[kCkG];
      double wd[kCkG], ev[kCkG];
      double run = 0.0;
      for (int i = 0; i < kCkG; ++i) {
        wv[i] = (float)g.ck_weights[i];
        wd[i] = g.ck_weights[i];
        for (int k2 = 0; k2 < kCkG; ++k2) run += ck_pair_weight(g.ck_weights[i], g.ck_weights[k2]);
        ev[i] = run;
      }
      float* dw = A(dalloc<float>(c, kCkG));
      double* dwd = A(dalloc<double>(c, kCkG));
      double* de = A(dalloc<double>(c, kCkG));
      if (ok) ok = upload(dw, wv, kCkG) && upload(dwd, wd, kCkG) && upload(de, ev, kCkG);
      c->tb.ckw = dw;
      c->tb.ckwd = dwd;
      c->tb.cke = de;
    }
    if (m.has_cia) {
      encode_tables(g.log10_cia, 2, m.n_tc, g.n_nu, (int)np, h, off, wide);
      uint16_t* dhc = A(dalloc<uint16_t>(c, h.size()));
      float* dcc = A(dalloc<float>(c, off.size()));
      if (ok) ok = upload(dhc, reinterpret_cast<const uint16_t*>(h.data()), h.size()) && upload(dcc, off.data(), off.size());
      c->tb.hc = dhc;
      c->tb.cc = dcc;
    }
  }

  // ---- bins and data
  c->d_lo = A(dalloc<int32_t>(c, m.K));
  c->d_hi = A(dalloc<int32_t>(c, m.K));
  c->d_y = A(dalloc<double>(c, m.K));
  c->d_yerr = A(dalloc<double>(c, m.K));
  c->d_mask = A(dalloc<uint8_t>(c, m.K));
  if (ok) {
    std::vector<uint8_t> mask(m.K, 0);
    if (g.offset_mask) std::memcpy(mask.data(), g.offset_mask, m.K);
    ok = upload(c->d_lo, g.bin_lo, m.K) && upload(c->d_hi, g.bin_hi, m.K) && upload(c->d_y, g.y_obs, m.K) &&
         upload(c->d_yerr, g.y_err, m.K) && upload(c->d_mask, mask.data(), m.K);
  }

  // ---- workspace
  Work& w = c->w;
  const size_t rs = fp64 ? 8 : 4;
  w.status = A(dalloc<int32_t>(c, B));
  w.nlay = A(dalloc<int32_t>(c, B));
  if (layer_classes_used(m) && !fp64) w.cls = A(dalloc<int32_t>(c, 2 + 2 * (size_t)B));
  w.t_lay = A(dalloc<double>(c, (size_t)B * Lp));
  w.t_lev = A(dalloc<double>(c, (size_t)B * (Lp + 1)));
  if (m.mode == kEmission && !fp64) w.inv_tlev = A(dalloc<double>(c, (size_t)B * (Lp + 1)));
  w.r_lev = A(dalloc<double>(c, (size_t)B * (Lp + 1)));
  w.core = A(dalloc<double>(c, B));
  w.cloud = A(dalloc<double>(c, (size_t)B * kCloudSpec));
  if (m.cloud_ng && g.precision == EXOFWD_PREC_MIXED)
    w.cloud_q = A(dalloc<float>(c, (size_t)B * (1 + kCloudSpec) * m.n_nu_pad));
  w.cells = A(dalloc<int32_t>(c, (size_t)B * Lp));
  if (!fp64 || m.mode == kEmission) w.lsg = A(dalloc<int32_t>(c, (size_t)B * (Lp + 1)));
  if (m.mode == kTransmission && !fp64) w.front = A(dalloc<int32_t>(c, (size_t)B * m.n_tiles));
  w.rec = A(dalloc<unsigned char>(c, (size_t)B * Lp * RL * rs));
  w.area = A(dalloc<unsigned char>(c, (size_t)B * Lp * rs));
  if (m.mode == kTransmission) {
    if (fp64) {
      w.pm64 = A(dalloc<double>(c, (size_t)B * Lp * Lp));
    } else {
      const size_t plane = (size_t)(Lp / 32) * (Lp / 16) * 512;
      w.pfrag = A(dalloc<uint16_t>(c, (size_t)B * 2 * plane));
      w.ptfrag = A(dalloc<uint16_t>(c, (size_t)B * 2 * plane));
    }
  }
  w.spec = A(dalloc<unsigned char>(c, (size_t)B * m.n_nu * rs));
  if (m.ck && m.ck_mix == kCkRorr) w.ckmix = A(dalloc<float>(c, (size_t)B * Lp * np * kCkG));
  w.dm = A(dalloc<double>(c, (size_t)B * m.K));
  w.lnl_tmp = A(dalloc<double>(c, B));
  w.mdot = A(dalloc<double>(c, B));
  if (m.has_fcld) {
    w.gv = A(dalloc<double>(c, (size_t)B * m.P));
    w.fbar = A(dalloc<double>(c, B));
  }
  {
    int32_t* d_bin = A(dalloc<int32_t>(c, np));
    double* d_inv = A(dalloc<double>(c, m.K));
    std::vector<int32_t> bin_of(np, -1);
    std::vector<double> inv(m.K);
    for (int k2 = 0; k2 < m.K; ++k2) {
      for (int i = g.bin_lo[k2]; i < g.bin_hi[k2]; ++i) bin_of[i] = k2;
      inv[k2] = 1.0 / (double)(g.bin_hi[k2] - g.bin_lo[k2]);
    }
    if (ok) ok = upload(d_bin, bin_of.data(), np) && upload(d_inv, inv.data(), m.K);
    w.bin_of = d_bin;
    w.inv_cnt = d_inv;
  }
  if (ok) ok = adjoint_alloc(c->aw, m, B, fp64, [&](size_t bytes) {
    return (void*)dalloc<unsigned char>(c, bytes);
  });
  if (!ok) {
    exofwd_destroy(c);
    return create_fail(EXOFWD_ERR_NOMEM, "device allocation or upload failed");
  }
  hipError_t e = m.ck ? ck_configure(m) : m.mode == kTransmission ? trans_fwd_configure(m, fp64)
                                                                   : emission_configure(m, fp64);
  if (e == hipSuccess) e = profile_configure(m, fp64);
  if (e == hipSuccess) e = adjoint_configure(m, fp64);
  if (e != hipSuccess) {
    exofwd_destroy(c);
    return create_fail(EXOFWD_ERR_DEVICE, std::string("kernel attributes: ") + hipGetErrorString(e));
  }
  if (hipDeviceSynchronize() != hipSuccess) {
    exofwd_destroy(c);
    return create_fail(EXOFWD_ERR_DEVICE, "device synchronisation failed");
  }
  *out = c;
  return EXOFWD_OK;
}

static exofwd_status check_call(exofwd_ctx* c, int32_t B, const double* params) {
  if (!c) return EXOFWD_ERR_ARG;
  if (B < 1 || B > c->batch_max) return fail(c, EXOFWD_ERR_SHAPE, "B outside [1, batch_max]");
  if (!params) return fail(c, EXOFWD_ERR_ARG, "params is NULL");
  if (hipSetDevice(c->device) != hipSuccess) return fail(c, EXOFWD_ERR_DEVICE, "hipSetDevice failed");
  c->err.clear();
  return EXOFWD_OK;
}

static exofwd_status run_forward(exofwd_ctx* c, const Work& w, int32_t B, const double* params,
                                 const int32_t* n_layers, void* spectra, double* lnL, int32_t* status,
                                 void* hip_stream, void* dtau_out);
static exofwd_status run_grad(exofwd_ctx* c, int32_t B, const double* params, const int32_t* n_layers,
                              void* spectra, double* lnL, double* grad, int32_t* status, void* hip_stream);

extern "C++" {
static constexpr size_t kMaxGraphs = 16;

// Replays the launch sequence of a call whose (kind, B, pointers, stream) was seen
// before; otherwise captures it on the stream first.  A caller that is itself
// capturing gets the kernels enqueued into its own graph.
template <typename F>
static exofwd_status graph_call(exofwd_ctx* c, int kind, int B, const std::array<const void*, 7>& ptr,
                                hipStream_t st, F&& enqueue) {
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &cs) != hipSuccess) return fail(c, EXOFWD_ERR_DEVICE, "stream query failed");
  if (cs != hipStreamCaptureStatusNone) return enqueue();
  auto launch = [&](exofwd_ctx::Graph& g) {
    g.used = ++c->tick;
    prof_begin(c, "graph", st);
    const hipError_t e = hipGraphLaunch(g.exec, st);
    prof_end(c, st);
    return e == hipSuccess ? EXOFWD_OK : fail(c, EXOFWD_ERR_DEVICE, "hipGraphLaunch failed");
  };
  for (auto& g : c->graphs)
    if (g.kind == kind && g.B == B && g.ptr == ptr && g.st == st) return launch(g);
  if (st == nullptr) return fail(c, EXOFWD_ERR_ARG, "graph replay needs a stream other than the null stream");
  c->capturing = true;
  if (hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal) != hipSuccess) {
    c->capturing = false;
    return fail(c, EXOFWD_ERR_DEVICE, "hipStreamBeginCapture failed");
  }
  const exofwd_status s = enqueue();
  hipGraph_t graph = nullptr;
  const hipError_t e = hipStreamEndCapture(st, &graph);
  c->capturing = false;
  if (s != EXOFWD_OK || e != hipSuccess || !graph) {
    if (graph) hipGraphDestroy(graph);
    return s != EXOFWD_OK ? s : fail(c, EXOFWD_ERR_DEVICE, "hipStreamEndCapture failed");
  }
  hipGraphExec_t exec = nullptr;
  const hipError_t ei = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
  hipGraphDestroy(graph);
  if (ei != hipSuccess) return fail(c, EXOFWD_ERR_DEVICE, "hipGraphInstantiate failed");
  if (c->graphs.size() >= kMaxGraphs) {
    auto lru = std::min_element(c->graphs.begin(), c->graphs.end(),
                                [](const auto& a, const auto& b) { return a.used < b.used; });
    hipGraphExecDestroy(lru->exec);
    c->graphs.erase(lru);
  }
  c->graphs.push_back({kind, B, ptr, st, exec, 0});
  return launch(c->graphs.back());
}
}  // extern "C++"

exofwd_status exofwd_forward(exofwd_ctx* c, int32_t B, const double* params, const int32_t* n_layers, void* spectra,
                             double* lnL, int32_t* status, void* hip_stream) {
  exofwd_status s = check_call(c, B, params);
  if (s) return s;
  auto enqueue = [&]() { return run_forward(c, c->w, B, params, n_layers, spectra, lnL, status, hip_stream, nullptr); };
  if (!c->use_graphs) return enqueue();
  return graph_call(c, 0, B, {params, n_layers, spectra, lnL, status, nullptr, nullptr}, (hipStream_t)hip_stream,
                    enqueue);
}

static exofwd_status run_forward(exofwd_ctx* c, const Work& w, int32_t B, const double* params,
                                 const int32_t* n_layers, void* spectra, double* lnL, int32_t* status,
                                 void* hip_stream, void* dtau_out) {
  exofwd_status s = EXOFWD_OK;
  hipStream_t st = (hipStream_t)hip_stream;
  const bool fp64 = c->precision == EXOFWD_PREC_FP64;
  // with the cloudy/clear mixing the kernels run 2B virtual samples into the internal
  // spectra; the likelihood kernel mixes each pair into the caller's spectrum
  const int Bv = c->m.has_fcld ? 2 * B : B;
  void* spec = (spectra && !c->m.has_fcld) ? spectra : w.spec;
  prof_begin(c, "profile", st);
  launch_profile(c->m, w, Bv, params, n_layers, fp64, st);
  prof_end(c, st);
  if ((s = check_hip(c, hipGetLastError(), "profile launch"))) return s;
  if (c->m.ck) {
    if (c->m.ck_mix == kCkRorr) {
      prof_begin(c, "ck_mix", st);
      launch_ck_mix(c->m, w, c->tb, Bv, st);
      prof_end(c, st);
      if ((s = check_hip(c, hipGetLastError(), "k-distribution mixing launch"))) return s;
    }
    prof_begin(c, "ck_spectrum", st);
    launch_ck_spectrum(c->m, w, c->tb, Bv, spec, st);
  } else if (c->m.mode == kTransmission) {
    prof_begin(c, "trans_fwd", st);
    launch_trans_fwd(c->m, w, c->tb, Bv, spec, fp64, st, (float*)dtau_out);
  } else {
    prof_begin(c, "emis_fwd", st);
    launch_emission(c->m, w, c->tb, Bv, spec, fp64, st, dtau_out);
  }
  prof_end(c, st);
  if ((s = check_hip(c, hipGetLastError(), "spectrum launch"))) return s;
  prof_begin(c, "loglike", st);
  launch_loglike(c->m, w, B, params, spec, c->m.has_fcld ? spectra : nullptr, fp64, c->d_lo, c->d_hi, c->d_y,
                 c->d_yerr, c->m.has_offset ? c->d_mask : nullptr, lnL, status, st);
  prof_end(c, st);
  return check_hip(c, hipGetLastError(), "loglike launch");
}

extern "C++" {
// Per-call workspace of a forward call for B samples laid out from `base` in
// 256-byte aligned pieces; returns its size in bytes.  With base == nullptr it only
// sizes the layout.  The tables and the bin map stay the context's own.
static size_t carve_forward_work(const exofwd_ctx* c, int B, bool internal_spec, unsigned char* base, Work& w) {
  const Model& m = c->m;
  const bool fp64 = c->precision == EXOFWD_PREC_FP64, trans = m.mode == kTransmission;
  const size_t Bv = (size_t)(m.has_fcld ? 2 * B : B), Lp = (size_t)m.L_pad, rs = fp64 ? 8 : 4;
  size_t off = 0;
  auto take = [&](size_t bytes) -> unsigned char* {
    unsigned char* p = base ? base + off : nullptr;
    off += (bytes + 255) / 256 * 256;
    return p;
  };
  w = Work{};
  w.status = (int32_t*)take(4 * Bv);
  w.nlay = (int32_t*)take(4 * Bv);
  if (layer_classes_used(m) && !fp64) w.cls = (int32_t*)take(4 * (2 + 2 * Bv));
  w.t_lay = (double*)take(8 * Bv * Lp);
  w.t_lev = (double*)take(8 * Bv * (Lp + 1));
  if (!trans && !fp64) w.inv_tlev = (double*)take(8 * Bv * (Lp + 1));
  w.r_lev = (double*)take(8 * Bv * (Lp + 1));
  w.core = (double*)take(8 * Bv);
  w.cloud = (double*)take(8 * Bv * kCloudSpec);
  if (m.cloud_ng && !fp64) w.cloud_q = (float*)take(4 * Bv * (1 + kCloudSpec) * (size_t)m.n_nu_pad);
  w.cells = (int32_t*)take(4 * Bv * Lp);
  if (!fp64) w.lsg = (int32_t*)take(4 * Bv * (Lp + 1));
  if (trans && !fp64) w.front = (int32_t*)take(4 * Bv * (size_t)m.n_tiles);
  w.rec = take(rs * Bv * Lp * (size_t)rec_stride(m, fp64));
  w.area = take(rs * Bv * Lp);
  if (trans && fp64) w.pm64 = (double*)take(8 * Bv * Lp * Lp);
  if (trans && !fp64) w.pfrag = (uint16_t*)take(2 * Bv * 2 * (Lp / 32) * (Lp / 16) * 512);
  if (internal_spec) w.spec = take(rs * Bv * (size_t)m.n_nu);
  if (m.ck && m.ck_mix == kCkRorr) w.ckmix = (float*)take(4 * Bv * Lp * (size_t)m.n_nu_pad * kCkG);
  w.dm = (double*)take(8 * Bv * (size_t)m.K);
  w.lnl_tmp = (double*)take(8 * Bv);
  w.mdot = (double*)take(8 * Bv);
  if (m.has_fcld) w.fbar = (double*)take(8 * Bv);
  w.bin_of = c->w.bin_of;
  w.inv_cnt = c->w.inv_cnt;
  return off;
}
}  // extern "C++"

exofwd_status exofwd_forward_noalloc(exofwd_ctx* c, int32_t B, const double* params, const int32_t* n_layers,
                                     void* spectra, double* lnL, int32_t* status, void* hip_stream) {
  exofwd_status s = check_call(c, B, params);
  if (s) return s;
  unsigned char* base = static_cast<unsigned char*>(scratch_address(c->device));
  if (!base) return fail(c, EXOFWD_ERR_DEVICE, "the static scratch array has no device address on this device");
  const bool internal_spec = !spectra || c->m.has_fcld;
  Work w;
  const size_t need = carve_forward_work(c, B, internal_spec, nullptr, w);
  if (need > (size_t)EXOFWD_NOALLOC_SCRATCH_BYTES)
    return fail(c, EXOFWD_ERR_SHAPE, "exofwd_forward_noalloc: " + std::to_string(B) + " samples need " +
                                         std::to_string(need) + " bytes of scratch, more than the static array's " +
                                         std::to_string((size_t)EXOFWD_NOALLOC_SCRATCH_BYTES));
  carve_forward_work(c, B, internal_spec, base, w);
  // no timing events either (creating them may allocate)
  const bool prof = c->profiling;
  c->profiling = false;
  s = run_forward(c, w, B, params, n_layers, spectra, lnL, status, hip_stream, nullptr);
  c->profiling = prof;
  return s;
}

exofwd_status exofwd_grad(exofwd_ctx* c, int32_t B, const double* params, const int32_t* n_layers, void* spectra,
                          double* lnL, double* grad, int32_t* status, void* hip_stream) {
  exofwd_status s = check_call(c, B, params);
  if (s) return s;
  if (!lnL || !grad) return fail(c, EXOFWD_ERR_ARG, "lnL and grad are required");
  if (!adjoint_supported(c->m, c->precision == EXOFWD_PREC_FP64))
    return fail(c, EXOFWD_ERR_UNSUPPORTED,
                "the adjoint needs at most 160 padded layers");
  auto enqueue = [&]() { return run_grad(c, B, params, n_layers, spectra, lnL, grad, status, hip_stream); };
  if (!c->use_graphs) return enqueue();
  return graph_call(c, 1, B, {params, n_layers, spectra, lnL, grad, status, nullptr}, (hipStream_t)hip_stream,
                    enqueue);
}

static exofwd_status run_grad(exofwd_ctx* c, int32_t B, const double* params, const int32_t* n_layers,
                              void* spectra, double* lnL, double* grad, int32_t* status, void* hip_stream) {
  exofwd_status s;
  // the reverse passes read the forward's layer optical depths (not the FP64 transmission one)
  void* dtau_out = c->precision == EXOFWD_PREC_MIXED ? (void*)c->aw.dtau
                                                     : (c->m.mode == kEmission ? (void*)c->aw.dtau64 : nullptr);
  if ((s = run_forward(c, c->w, B, params, n_layers, spectra, lnL, status, hip_stream, dtau_out))) return s;
  hipStream_t st = (hipStream_t)hip_stream;
  const bool fp64 = c->precision == EXOFWD_PREC_FP64;
  const int Bv = c->m.has_fcld ? 2 * B : B;
  if (c->m.mode == kTransmission) {
    prof_begin(c, "trans_adj", st);
    launch_trans_adjoint(c->m, c->w, c->tb, c->aw, Bv, fp64, st);
  } else {
    prof_begin(c, "emis_adj", st);
    launch_emis_adjoint(c->m, c->w, c->aw, Bv, fp64, st);
  }
  prof_end(c, st);
  if ((s = check_hip(c, hipGetLastError(), "adjoint launch"))) return s;
  if (!fp64 || c->m.mode == kEmission) {
    prof_begin(c, "layer_sums", st);
    launch_layer_sums(c->m, c->w, c->tb, c->aw, Bv, fp64, st);
    prof_end(c, st);
    if ((s = check_hip(c, hipGetLastError(), "layer-sum launch"))) return s;
  }
  prof_begin(c, "chain", st);
  launch_chain(c->m, c->w, c->aw, Bv, params, c->d_mask, c->m.has_fcld ? c->w.gv : grad, fp64, st);
  if (c->m.has_fcld) launch_mix_grad(c->m, c->w, B, grad, st);
  prof_end(c, st);
  return check_hip(c, hipGetLastError(), "chain launch");
}

exofwd_status exofwd_set_profiling(exofwd_ctx* c, int32_t enable) {
  if (!c) return EXOFWD_ERR_ARG;
  hipSetDevice(c->device);
  for (auto& e : c->events) {
    hipEventSynchronize(e.b);
    hipEventDestroy(e.a);
    hipEventDestroy(e.b);
  }
  c->events.clear();
  c->profiling = enable != 0;
  return EXOFWD_OK;
}

exofwd_status exofwd_kernel_time(exofwd_ctx* c, const char* name, double* total_ms, int32_t* launches) {
  if (!c || !name || !total_ms || !launches) return EXOFWD_ERR_ARG;
  double tot = 0.0;
  int n = 0;
  for (auto& e : c->events) {
    if (e.name != name) continue;
    if (hipEventSynchronize(e.b) != hipSuccess) return fail(c, EXOFWD_ERR_DEVICE, "event sync failed");
    float ms = 0.0f;
    if (hipEventElapsedTime(&ms, e.a, e.b) != hipSuccess) return fail(c, EXOFWD_ERR_DEVICE, "elapsed time failed");
    tot += ms;
    ++n;
  }
  *total_ms = tot;
  *launches = n;
  return EXOFWD_OK;
}

exofwd_status exofwd_set_graphs(exofwd_ctx* c, int32_t enable) {
  if (!c) return EXOFWD_ERR_ARG;
  hipSetDevice(c->device);
  if (!c->graphs.empty()) hipDeviceSynchronize();
  drop_graphs(c);
  c->use_graphs = enable != 0;
  return EXOFWD_OK;
}

exofwd_status exofwd_set_tuning(exofwd_ctx* c, const int32_t* t) {
  if (!c || !t) return EXOFWD_ERR_ARG;
  if (t[0] != 0 && t[0] != 1) return fail(c, EXOFWD_ERR_ARG, "forward order must be 0 or 1");
  const bool tunable_adj = c->precision == EXOFWD_PREC_MIXED && c->m.mode == kTransmission &&
                           adjoint_supported(c->m, false);
  AdjWork aw = c->aw;
  if (tunable_adj && !adjoint_set_tuning(aw, c->m, t[1], t[2], t[3]))
    return fail(c, EXOFWD_ERR_ARG, "reverse shape, chunk target or layer-sum tiles not valid for this context");
  hipSetDevice(c->device);
  hipDeviceSynchronize();
  drop_graphs(c);
  c->m.fwd_tile_major = t[0];
  c->aw = aw;
  return EXOFWD_OK;
}

exofwd_status exofwd_get_tuning(const exofwd_ctx* c, int32_t* t) {
  if (!c || !t) return EXOFWD_ERR_ARG;
  t[0] = c->m.fwd_tile_major;
  t[1] = c->aw.variant;
  t[2] = c->aw.chunk_target;
  t[3] = c->aw.ls_tiles;
  return EXOFWD_OK;
}

extern "C++" {
namespace {

// parameters of a valid, cloud-free mid-range atmosphere for timing runs
std::vector<double> neutral_params(const Model& m) {
  std::vector<double> th(m.P, 0.0);
  if (m.tp_kind == kTpIso) th[0] = 1200.0;
  else if (m.tp_kind == kTpGuillot3) { th[0] = 500.0; th[1] = 1200.0; th[2] = 0.0; }
  else if (m.tp_kind == kTpBarstow) th[0] = 1000.0;
  else if (m.tp_kind == kTpMilne) { th[0] = 1000.0; th[1] = -2.0; th[2] = 0.6; th[3] = -1.0; th[4] = 1.0; }
  else if (m.tp_kind == kTpGuillot7) {
    th[0] = 300.0; th[1] = 1200.0; th[2] = -2.0; th[3] = 0.0; th[4] = 0.4; th[5] = -2.0; th[6] = 1.0;
  } else for (int k = 0; k < m.n_tp; ++k) th[k] = 1200.0;
  for (int s2 = 0; s2 < m.S; ++s2) th[m.n_tp + s2] = -6.0;
  if (m.has_cloud && !m.cloud_ng) th[m.idx_cloud] = m.log10_pbot + 1.0;
  if (m.cloud_ng) {
    // thin haze of 1 um particles over the whole column (every cloud term still evaluated)
    int k = m.idx_cloud;
    th[k++] = 0.0;
    if (m.cloud_qext != kQextGrey) { th[k++] = 4.0; th[k++] = 1.0; }
    th[k++] = -8.0;
    if (m.cloud_profile == kQprofSlab) { th[k++] = m.log10_ptop; th[k++] = m.log10_pbot; }
    else if (m.cloud_profile == kQprofPower) { th[k++] = m.log10_pbot; th[k++] = 1.0; }
    if (m.cloud_qext == kQextFeature) { th[k++] = 0.5; th[k++] = 10.0; th[k++] = 0.0; th[k++] = 0.0; }
  }
  if (m.has_fcld) th[m.idx_fcld] = 0.5;
  if (m.has_bd) { th[m.idx_bd] = 5.0; th[m.idx_bd + 1] = 50.0; }
  if (m.has_scale) th[m.idx_scale] = 1.0;
  if (m.has_offset) th[m.idx_offset] = 0.0;
  return th;
}

std::string tuning_key(const exofwd_ctx* c, int B) {
  hipDeviceProp_t prop{};
  hipGetDeviceProperties(&prop, c->device);
  std::ostringstream k;
  k << prop.gcnArchName << "/cu" << prop.multiProcessorCount << " mode" << c->m.mode << " prec" << c->precision
    << " S" << c->m.S << " cia" << c->m.has_cia << " ng" << c->m.cloud_ng << " fcld" << c->m.has_fcld << " Lpad" << c->m.L_pad << " Lmax" << c->m.L_max << " nu"
    << c->m.n_nu_pad << " tab" << c->m.n_t << "x" << c->m.n_p << " B" << B;
  std::string key = k.str();
  for (char& ch : key)
    if (ch == ' ' || ch == '=') ch = '_';
  return key;
}

}  // namespace
}  // extern "C++"

exofwd_status exofwd_autotune(exofwd_ctx* c, int32_t B, const double* params, const int32_t* n_layers,
                              const char* cache_path) {
  if (!c) return EXOFWD_ERR_ARG;
  if (B < 1 || B > c->batch_max) return fail(c, EXOFWD_ERR_SHAPE, "B outside [1, batch_max]");
  if (hipSetDevice(c->device) != hipSuccess) return fail(c, EXOFWD_ERR_DEVICE, "hipSetDevice failed");
  const bool mixed_trans = c->precision == EXOFWD_PREC_MIXED && c->m.mode == kTransmission && !c->m.ck;
  if (!mixed_trans) return EXOFWD_OK;   // the FP64 and emission launches have no tunable shape
  const bool grad = adjoint_supported(c->m, false);
  const std::string key = tuning_key(c, B);

  // ---- cached result
  std::vector<std::string> lines;
  if (cache_path) {
    std::ifstream in(cache_path);
    std::string line;
    while (std::getline(in, line)) {
      if (line.empty()) continue;
      std::istringstream ls(line);
      std::string k;
      int32_t t[4];
      const bool parsed = static_cast<bool>(ls >> k >> t[0] >> t[1] >> t[2] >> t[3]);
      if (parsed && k == key) {
        if (exofwd_set_tuning(c, t) == EXOFWD_OK) return EXOFWD_OK;
        continue;   // a stale entry for this key is timed again and replaced
      }
      lines.push_back(line);
    }
  }

  // ---- timing runs on a private stream
  const size_t P = (size_t)c->m.P;
  double* d_th = nullptr;
  double *d_lnl = nullptr, *d_g = nullptr;
  int32_t* d_st = nullptr;
  hipStream_t st = nullptr;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  bool ok = hipMalloc(&d_lnl, B * sizeof(double)) == hipSuccess && hipMalloc(&d_g, B * P * sizeof(double)) == hipSuccess &&
            hipMalloc(&d_st, B * sizeof(int32_t)) == hipSuccess && hipStreamCreate(&st) == hipSuccess &&
            hipEventCreate(&e0) == hipSuccess && hipEventCreate(&e1) == hipSuccess;
  if (ok && !params) {
    const std::vector<double> one = neutral_params(c->m);
    std::vector<double> all(B * P);
    for (int b = 0; b < B; ++b) std::copy(one.begin(), one.end(), all.begin() + b * P);
    ok = hipMalloc(&d_th, B * P * sizeof(double)) == hipSuccess &&
         hipMemcpy(d_th, all.data(), B * P * sizeof(double), hipMemcpyHostToDevice) == hipSuccess;
  }
  const double* th = params ? params : d_th;
  const bool prof = c->profiling, graphs = c->use_graphs;
  c->profiling = false;
  c->use_graphs = false;
  auto step = [&]() {
    return grad ? run_grad(c, B, th, n_layers, nullptr, d_lnl, d_g, d_st, st)
                : run_forward(c, c->w, B, th, n_layers, nullptr, d_lnl, d_st, st, nullptr);
  };
  auto time_once = [&](const int32_t* t) -> double {
    if (exofwd_set_tuning(c, t) != EXOFWD_OK) return 1e30;
    if (step() != EXOFWD_OK) return 1e30;
    float best = 1e30f;
    for (int rep = 0; rep < 5; ++rep) {
      hipEventRecord(e0, st);
      if (step() != EXOFWD_OK) return 1e30;
      hipEventRecord(e1, st);
      if (hipEventSynchronize(e1) != hipSuccess) return 1e30;
      float ms = 0.0f;
      hipEventElapsedTime(&ms, e0, e1);
      best = std::min(best, ms);
    }
    return best;
  };
  int32_t cur[4], best_t[4];
  exofwd_get_tuning(c, cur);
  std::copy(cur, cur + 4, best_t);
  double best = ok ? time_once(cur) : 1e30;
  auto consider = [&](const int32_t* t) {
    const double ms = time_once(t);
    if (ms < best) {
      best = ms;
      std::copy(t, t + 4, best_t);
    }
  };
  if (ok && best < 1e30) {
    // coordinate descent: forward grid order, then reverse shape x chunk target, then layer-sum tiles
    for (int o = 0; o < 2; ++o) {
      int32_t t[4] = {o, best_t[1], best_t[2], best_t[3]};
      consider(t);
    }
    if (grad) {
      for (int v = 0; v < kAdjVariants; ++v)
        for (int tg : kChunkTargets) {
          int32_t t[4] = {best_t[0], v, tg, best_t[3]};
          consider(t);
        }
      for (int lt : kLsTileChoices) {
        int32_t t[4] = {best_t[0], best_t[1], best_t[2], lt};
        consider(t);
      }
      // the forward grid order once more, now beside the tuned reverse pass (the two
      // orders are within a few per cent of each other)
      for (int o = 0; o < 2; ++o) {
        int32_t t[4] = {o, best_t[1], best_t[2], best_t[3]};
        consider(t);
      }
    }
  }
  const exofwd_status applied = exofwd_set_tuning(c, best_t);
  c->profiling = prof;
  c->use_graphs = graphs;
  if (e0) hipEventDestroy(e0);
  if (e1) hipEventDestroy(e1);
  if (st) hipStreamDestroy(st);
  hipFree(d_th);
  hipFree(d_lnl);
  hipFree(d_g);
  hipFree(d_st);
  if (!ok || best >= 1e30) return fail(c, EXOFWD_ERR_DEVICE, "autotune timing runs failed");
  if (applied != EXOFWD_OK) return applied;
  if (cache_path) {
    std::ofstream out(cache_path, std::ios::trunc);
    for (const auto& line : lines) out << line << "\n";
    out << key << " " << best_t[0] << " " << best_t[1] << " " << best_t[2] << " " << best_t[3] << "\n";
    if (!out) return fail(c, EXOFWD_ERR_ARG, "cannot write the autotune cache file");
  }
  return EXOFWD_OK;
}

}  // extern "C"
