// Per-sample atmospheric profile in FP64: T-p profile, free chemistry,
// hydrostatic altitudes, per-layer opacity records, path matrix and annulus
// areas.  One workgroup of 512 threads per sample.
#include "cloud.h"
#include "kernels.h"
#include "opacity.h"
#include "tp.h"

namespace exofwd {

// Largest i with grid[i] <= x, capped at n-2, and the linear weight; x is
// clamped to the grid first (a clamped x gets w = 0 or 1).  NaN maps to cell 0.
__device__ inline void cell_index(const double* grid, int n, double x, int& i, double& w) {
  if (!(x > grid[0])) { i = 0; w = 0.0; return; }
  if (x >= grid[n - 1]) { i = n - 2; w = 1.0; return; }
  int lo = 0, hi = n - 1;
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (grid[mid] <= x) lo = mid; else hi = mid;
  }
  i = lo;
  w = (x - grid[lo]) / (grid[lo + 1] - grid[lo]);
}

// Monotone cubic Hermite slopes (Fritsch-Carlson with the Fritsch-Butland
// weighted harmonic mean inside, three-point shape-preserving ends).
__device__ void pchip_slopes(const double* xk, const double* yk, int n, double* d) {
  double h[kMaxKnots], del[kMaxKnots];
  for (int k = 0; k < n - 1; ++k) { h[k] = xk[k + 1] - xk[k]; del[k] = (yk[k + 1] - yk[k]) / h[k]; }
  if (n == 2) { d[0] = d[1] = del[0]; return; }
  for (int k = 1; k < n - 1; ++k) {
    double a = del[k - 1], b = del[k];
    if (a == 0.0 || b == 0.0 || (a > 0.0) != (b > 0.0)) {
      d[k] = 0.0;
    } else {
      double w1 = 2.0 * h[k] + h[k - 1], w2 = h[k] + 2.0 * h[k - 1];
      d[k] = (w1 + w2) / (w1 / a + w2 / b);
    }
  }
  auto end = [](double h0, double h1, double m0, double m1) {
    double dd = ((2.0 * h0 + h1) * m0 - h0 * m1) / (h0 + h1);
    auto sgn = [](double v) { return (v > 0.0) - (v < 0.0); };
    if (sgn(dd) != sgn(m0)) return 0.0;
    if (sgn(m0) != sgn(m1) && fabs(dd) > fabs(3.0 * m0)) return 3.0 * m0;
    return dd;
  };
  d[0] = end(h[0], h[1], del[0], del[1]);
  d[n - 1] = end(h[n - 2], h[n - 3], del[n - 2], del[n - 3]);
}

__device__ double pchip_eval(const double* xk, const double* yk, const double* d, int n, double x) {
  int k = 0;
  while (k < n - 2 && xk[k + 1] <= x) ++k;
  double hk = xk[k + 1] - xk[k];
  double t = (x - xk[k]) / hk;
  double omt = 1.0 - t;
  return (1.0 + 2.0 * t) * omt * omt * yk[k] + t * omt * omt * hk * d[k] + t * t * (3.0 - 2.0 * t) * yk[k + 1] +
         t * t * (t - 1.0) * hk * d[k + 1];
}

// Reduced modified Guillot profile (Eq. 16 with q_int = q_irr = 2/3, mu_* = 1/sqrt 3).
__device__ inline double guillot3(double t_int, double t_eq, double gam, double tau, double f_hem) {
  const double s3 = 1.7320508075688772935274463415059;
  const double q = 2.0 / 3.0;
  double ti2 = t_int * t_int, te2 = t_eq * t_eq;
  double t4 = 0.75 * ti2 * ti2 * (q + tau) +
              0.75 * te2 * te2 * 4.0 * f_hem * (q + 1.0 / (gam * s3) + (gam / s3 - 1.0 / (gam * s3)) * exp(-gam * tau * s3));
  return sqrt(sqrt(t4));
}

// Round to nearest even bf16 (finite inputs).
__device__ inline uint16_t bf16_rn(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ inline float bf16_to_f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// log2 of a prefactor, finite in FP64 also for zero (in FP32 the constant is -inf, whose
// power the hardware's exponential takes as zero)
__device__ inline double log2_or_absent(double v) { return v == 0.0 ? kAbsentLog : log2(v); }

// Path matrix entries P_1D[i][l] (Eq. 43), l in [l0, l1), l0 >= i, with b_i the mid radius
// of layer i: put(l, value).  The l > i case uses
// sqrt(r_up^2-b^2) - sqrt(r_lo^2-b^2) = dr (r_up+r_lo)/(s_up+s_lo), which has no
// cancellation; square roots are taken of (r-b)(r+b), each level's once.
template <typename Put>
__device__ inline void path_entries(const double* r, const double* dr, int i, int l0, int l1, Put put) {
  const double b = 0.5 * (r[i] + r[i + 1]);
  // sqrt(r^2 - b^2)
  auto leg = [&](double rl) {
    double half;
    return sqrt_d((rl - b) * (rl + b), half);
  };
  int l = l0;
  if (l == i) {
    double sup = sqrt(0.5 * dr[i] * (r[i + 1] + b));
    put(l, 2.0 * sup / dr[i]);
    ++l;
  }
  if (l >= l1) return;
  double rlo = r[l], slo = leg(rlo);
#pragma unroll 1
  for (; l < l1; ++l) {
    const double rup = r[l + 1], sup = leg(rup);
    const double den = sup + slo;
    put(l, div_d(2.0 * (rup + rlo), den, rcp_d(den)));
    rlo = rup;
    slo = sup;
  }
}
constexpr int kPathSeg = 8;      // entries of one work item of the path matrix
constexpr int kBlockP = 512;     // threads of the profile kernel

// row length (words) of the reduced-precision path matrix in LDS: odd, so rows and columns
// are both read without bank conflicts
__host__ __device__ constexpr int path_ld(int Lp) { return Lp + 1; }

// Bound by latency (one workgroup per sample): every phase is spread over the threads, the
// serial recursion reads ahead, and each path-matrix entry is formed once, its transposed
// copy coming from LDS.  100 layers: one sample 75 -> 21 us, 1024 samples 164 -> 56 us.
template <typename Real>
__global__ __launch_bounds__(kBlockP) void k_profile(Model m, Work w, const double* __restrict__ params,
                                                    const int32_t* __restrict__ n_layers) {
  const int b = blockIdx.x;
  const int tid = threadIdx.x;
  const int Lp = m.L_pad;
  __shared__ double s_t[kMaxLayers + 1];      // layer T
  __shared__ double s_tl[kMaxLayers + 1];     // level T (emission)
  __shared__ double s_u[kMaxLayers + 1];      // 1/r at levels
  __shared__ double s_r[kMaxLayers + 1];
  __shared__ double s_dr[kMaxLayers];
  __shared__ double s_inc[kMaxLayers];
  __shared__ double s_knot_x[kMaxKnots], s_knot_y[kMaxKnots], s_knot_d[kMaxKnots];
  __shared__ int s_badt;
  __shared__ int s_cell[kMaxLayers];
  __shared__ double s_n[kMaxLayers], s_x[kMaxSpecies], s_th[kMaxParams];
  __shared__ int s_finite, s_above, s_unbound;
  __shared__ unsigned long long s_runs[3], s_heads[3];   // layer-sum groups: bits of run starts, of group heads
  extern __shared__ double s_dyn[];
  double *s_tg = s_dyn, *s_pg = s_tg + m.n_t, *s_cg = s_pg + m.n_p;   // table axes
  // reduced precision, transmission: path matrix as bf16 hi | lo << 16
  uint32_t* s_pm = reinterpret_cast<uint32_t*>(s_cg + m.n_tc);

  // virtual sample b of real sample bs; a clear one (cloudy/clear mixing) has no cloud
  const int bs = real_sample(m, b);
  const bool cloudy = m.has_cloud && !clear_sample(m, b);
  const double* th = s_th;
  int L = n_layers ? n_layers[bs] : m.L_max;
  int status = 0;
  if (L < 1 || L > m.L_max) {
    status = kBadLayers;
    L = m.L_max;
  }
  if (tid < m.P) s_th[tid] = params[(size_t)bs * m.P + tid];
  if (tid < m.n_t) s_tg[tid] = m.t_grid[tid];
  if (tid < m.n_tc) s_cg[tid] = m.tc_grid[tid];
  if (tid >= 256 && tid < 256 + m.n_p) s_pg[tid - 256] = m.logp_grid[tid - 256];
  if (tid == 0) {
    s_finite = 1;
    s_above = 0;
    s_unbound = 0;
  }
  __syncthreads();
  if (tid < m.P && !isfinite(th[tid])) s_finite = 0;
  // chemistry (Eq. 35-36)
  if (tid < m.S) s_x[tid] = exp10(th[m.n_tp + tid]);
  __syncthreads();
  if (!status && !s_finite) status = kNonfinite;
  double sx = 0.0;
  for (int s = 0; s < m.S; ++s) sx += s_x[s];
  const double xh2 = (1.0 - sx) / (1.0 + kHeH2);
  const double xhe = kHeH2 * xh2;
  double mu = m.mu_fixed;
  if (!(mu > 0.0)) {
    mu = xh2 * kMH2 + xhe * kMHe;
    for (int s = 0; s < m.S; ++s) mu += s_x[s] * m.mass[s];
  }
  const double scale = m.has_scale ? th[m.idx_scale] : 1.0;
  // an isolated object retrieves its gravity; its radius at p_ref is sqrt(G M / g) (Eq. 47)
  const double g_ref = m.has_bd ? exp10(th[m.idx_bd]) : m.g_ref;
  const double r_ref = m.has_bd ? sqrt(kGrav * th[m.idx_bd + 1] * kMJup / g_ref) : m.r_p * scale;

  const double step = (m.log10_ptop - m.log10_pbot) / L;   // log10 p per layer (negative)
  const double dlnp = -step * 2.302585092994045684017991454684;  // ln(p_l / p_{l+1})
  auto logp_lev = [&](int j) { return j == L ? m.log10_ptop : m.log10_pbot + j * step; };

  if (tid == 0) {
    s_badt = 0;
    if (m.tp_kind == kTpPchip) {
      for (int k = 0; k < m.n_knots; ++k) {
        s_knot_x[k] = m.n_knots == 1 ? m.log10_ptop
                                     : m.log10_ptop + k * ((m.log10_pbot - m.log10_ptop) / (m.n_knots - 1));
        s_knot_y[k] = th[k];
      }
      s_knot_x[m.n_knots - 1] = m.log10_pbot;
      pchip_slopes(s_knot_x, s_knot_y, m.n_knots, s_knot_d);
    }
  }
  __syncthreads();

  auto temperature = [&](double log10p_bar) {
    if (m.tp_kind == kTpIso) return th[0];
    if (m.tp_kind == kTpGuillot3) {
      double tau = m.kappa_ir * exp10(log10p_bar) * kBar / g_ref;
      return guillot3(th[0], th[1], exp10(th[2]), tau, m.f_hem);
    }
    if (m.tp_kind == kTpBarstow) return th[0] * barstow_factor(log10p_bar);
    if (m.tp_kind == kTpMilne) return sqrt(sqrt(milne_t4(th, log10p_bar, g_ref)));
    if (m.tp_kind == kTpGuillot7) return sqrt(sqrt(guillot7_t4(th, log10p_bar, g_ref, m.f_hem)));
    return pchip_eval(s_knot_x, s_knot_y, s_knot_d, m.n_knots, log10p_bar);
  };

  // layer temperatures, and the levels' in emission (one copy of the profiles' code: a
  // kernel that runs each of its lines once is held up by fetching them)
  int badt = 0;
  for (int q = tid; q < L + (m.mode == kEmission ? L + 1 : 0); q += kBlockP) {
    const bool lev = q >= L;
    const double t = temperature(lev ? logp_lev(q - L) : 0.5 * (logp_lev(q) + logp_lev(q + 1)));
    (lev ? s_tl[q - L] : s_t[q]) = t;
    badt |= !(t > 0.0) || !isfinite(t);
  }
  if (badt) atomicOr(&s_badt, 1);
  __syncthreads();
  if (!status) {
    if (s_badt) status |= kBadT;
    if (!(sx < 1.0)) status |= kBadVmr;
  }

  // hydrostatics (1/r linear in ln p inside each isothermal layer)
  const double kk = kB / (mu * kMu * g_ref * r_ref * r_ref);
  const double lpref = m.log10_pref;
  for (int l = tid; l < L; l += kBlockP) s_inc[l] = kk * s_t[l] * dlnp;
  for (int j = tid; j <= L; j += kBlockP)
    if (logp_lev(j) > lpref) atomicAdd(&s_above, 1);
  __syncthreads();
  if (tid < 64 && !status) {
    // one wave, every lane the same: the loops then run on scalar registers
    const int lref = __builtin_amdgcn_readfirstlane(min(max(s_above - 1, 0), L - 1));
    const int Lu = __builtin_amdgcn_readfirstlane(L);
    const double ln10 = 2.302585092994045684017991454684;
    const double u_ref = 1.0 / r_ref;
    double u = u_ref + kk * s_t[lref] * (logp_lev(lref) - lpref) * ln10;
    s_u[lref] = u;
    // the increments eight at a time: one LDS round trip for eight dependent sums
    constexpr int kAhead = 8;
    int j = lref - 1;
#pragma unroll 1
    for (; j >= kAhead - 1; j -= kAhead) {
      double v[kAhead];
#pragma unroll
      for (int k = 0; k < kAhead; ++k) v[k] = s_inc[j - k];
#pragma unroll
      for (int k = 0; k < kAhead; ++k) s_u[j - k] = u = u + v[k];
    }
#pragma unroll 1
    for (; j >= 0; --j) s_u[j] = u = u + s_inc[j];
    u = u_ref - kk * s_t[lref] * (lpref - logp_lev(lref + 1)) * ln10;
    s_u[lref + 1] = u;
    j = lref + 1;
#pragma unroll 1
    for (; j + kAhead <= Lu; j += kAhead) {
      double v[kAhead];
#pragma unroll
      for (int k = 0; k < kAhead; ++k) v[k] = s_inc[j + k];
#pragma unroll
      for (int k = 0; k < kAhead; ++k) s_u[j + k + 1] = u = u - v[k];
    }
#pragma unroll 1
    for (; j < Lu; ++j) s_u[j + 1] = u = u - s_inc[j];
  }
  __syncthreads();
  if (!status)
    for (int j = tid; j <= L; j += kBlockP)
      if (!(s_u[j] > 0.0)) s_unbound = 1;
  __syncthreads();
  if (!status && s_unbound) status = kUnbound;

  if (tid == 0) {
    w.status[b] = status;
    w.nlay[b] = L;
  }
  if (status) return;   // uniform across the workgroup

  for (int j = tid; j <= L; j += kBlockP) s_r[j] = 1.0 / s_u[j];
  __syncthreads();
  // dr_l = r_{l+1} - r_l = (u_l - u_{l+1}) r_l r_{l+1}, and u_l - u_{l+1} = inc_l
  for (int l = tid; l < L; l += kBlockP) s_dr[l] = s_inc[l] * s_r[l] * s_r[l + 1];
  __syncthreads();

  double* t_lay = w.t_lay + (size_t)b * Lp;
  double* t_lev = w.t_lev + (size_t)b * (Lp + 1);
  double* r_lev = w.r_lev + (size_t)b * (Lp + 1);
  for (int l = tid; l < Lp; l += kBlockP) t_lay[l] = l < L ? s_t[l] : 0.0;
  for (int j = tid; j <= Lp; j += kBlockP) {
    r_lev[j] = j <= L ? s_r[j] : 0.0;
    t_lev[j] = (m.mode == kEmission && j <= L) ? s_tl[j] : 0.0;
    if (w.inv_tlev) w.inv_tlev[(size_t)b * (Lp + 1) + j] = j <= L ? 1.0 / s_tl[j] : 0.0;
  }
  // transmission: opaque-core depth (r_0/R_s)^2; emission: (R_ref/R_s)^2 of Eq. 45
  if (tid == 0)
    w.core[b] = m.mode == kTransmission ? s_r[0] * s_r[0] / (m.r_s * m.r_s)
                                        : r_ref * r_ref / (m.has_bd ? m.bd_dist * m.bd_dist : m.r_s * m.r_s);

  // per-layer opacity records
  const bool wide = rec_wide(m, sizeof(Real) == 8);
  const int RL = rec_stride(m, sizeof(Real) == 8);
  Real* rec = reinterpret_cast<Real*>(w.rec) + (size_t)b * Lp * RL;
  Real* area = reinterpret_cast<Real*>(w.area) + (size_t)b * Lp;
  const double log10_pc = m.has_cloud ? th[m.idx_cloud] : 0.0;
  // non-grey cloud: per-sample constants of Q_ext and where the profile's parameters start
  const int q_first = m.idx_cloud + (m.cloud_qext == kQextGrey ? 1 : 3);
  const double r_eff = m.cloud_ng ? 1.0e-4 * exp10(th[m.idx_cloud]) : 1.0;
  if (m.cloud_ng && tid == 0) {
    double* cl = w.cloud + (size_t)b * kCloudSpec;
    const bool fit = m.cloud_qext != kQextGrey, feat = m.cloud_qext == kQextFeature;
    const int f0 = q_first + (m.cloud_profile == kQprofUniform ? 1 : 3);
    cl[0] = r_eff;
    cl[1] = fit ? th[m.idx_cloud + 1] : 0.0;
    cl[2] = fit ? exp10(th[m.idx_cloud + 2]) : 0.0;
    cl[3] = feat ? th[f0] : 0.0;
    cl[4] = feat ? th[f0 + 1] : 1.0;
    cl[5] = feat ? exp10(th[f0 + 2]) : 1.0;
    cl[6] = feat ? th[f0 + 3] : 0.0;
  }
  for (int l = tid; l < Lp; l += kBlockP) {
    Real* rl = rec + (size_t)l * RL;
    if (l >= L) {
      w.cells[(size_t)b * Lp + l] = 0;
      for (int k = 0; k < kRecFixed; ++k) rl[k] = Real(0);
      rl[5] = rl[6] = Real(-1000);
      area[l] = Real(0);
      continue;
    }
    const double t = s_t[l];
    const double lp_bar = 0.5 * (logp_lev(l) + logp_lev(l + 1));
    const double n = exp10(lp_bar) * kBar / (kB * t);
    const double dr = s_dr[l];
    int it, ip, itc = 0;
    double wt, wp, wtc = 0.0;
    cell_index(s_tg, m.n_t, t, it, wt);
    cell_index(s_pg, m.n_p, lp_bar, ip, wp);
    if (m.has_cia) cell_index(s_cg, m.n_tc, t, itc, wtc);
    w.cells[(size_t)b * Lp + l] = pack_cells(it, ip, itc);
    s_cell[l] = pack_cells(it, ip, itc);
    rl[0] = Real(wt);
    rl[1] = Real(wp);
    rl[2] = Real(wtc);
    const bool trans = m.mode == kTransmission;
    rl[3] = Real((trans && m.has_ray) ? n * (xh2 * m.ray_h2 + xhe * m.ray_he) * dr : 0.0);
    double dcl = 0.0;
    if (m.cloud_ng && cloudy) {
      // column q_l rho_l dr_l 3 / (4 r_eff); the kernels multiply it by Q_ext(nu) (Eq. 23)
      dcl = condensate_q(m.cloud_profile, th + q_first, logp_lev(l), logp_lev(l + 1), lp_bar, nullptr) * mu * kMu *
            n * dr * 0.75 / r_eff;
    } else if (trans && cloudy && !m.cloud_ng) {
      double f = (logp_lev(l) - log10_pc) * 2.302585092994045684017991454684 / dlnp;
      f = f < 0.0 ? 0.0 : (f > 1.0 ? 1.0 : f);
      dcl = m.kappa_cloud * mu * kMu * n * f * dr;
    }
    rl[4] = Real(dcl);
    rl[5] = Real(m.has_cia ? log2_or_absent(n * n * xh2 * xh2 * dr) : -1000.0);
    rl[6] = Real(m.has_cia ? log2_or_absent(n * n * xh2 * xhe * dr) : -1000.0);
    s_n[l] = n;
    area[l] = Real(dr * (s_r[l] + s_r[l + 1]) / (m.r_s * m.r_s));
  }
  __syncthreads();
  // the line sources' prefactors, a thread per (layer, source)
  for (int e = tid; e < Lp * m.S; e += kBlockP) {
    const int l = e / m.S, s = e - l * m.S;
    Real* rl = rec + (size_t)l * RL;
    const double pre = l < L ? s_n[l] * s_x[s] * s_dr[l] : 0.0;
    rl[kRecFixed + s] = l < L ? Real(log2_or_absent(pre)) : Real(-1000);
    if (wide) rl[kRecFixed + m.S + s] = Real(pre);
  }
  if (w.lsg) {
    // layer-sum groups: a run of layers in one table cell reads one set of table rows, so
    // the layer sums fetch them once per tile for the whole group.  The runs' starts (and
    // the end) as bits, then the group heads, every kLsGroup-th layer of a run.
    static_assert(kMaxLayers < 192, "three words of 64 layers");
    const int wq = tid >> 6, bit = tid & 63;
    if (wq < 3) {
      const bool start = tid == L || (tid < L && (tid == 0 || s_cell[tid] != s_cell[tid - 1]));
      const unsigned long long mask = __builtin_amdgcn_ballot_w64(start);
      if (bit == 0) s_runs[wq] = mask;
    }
    __syncthreads();
    bool head = false;
    int cnt = 0;
    if (wq < 3) {
      if (tid < L) {
        int q = wq;
        unsigned long long below = s_runs[q] & (~0ull >> (63 - bit));
        while (!below) below = s_runs[--q];   // bit 0 of word 0 is a start
        const int first = 64 * q + 63 - __builtin_clzll(below);
        q = wq;
        unsigned long long after = s_runs[q] & ~(~0ull >> (63 - bit));
        while (!after) after = s_runs[++q];   // bit L is set
        const int next = 64 * q + __builtin_ctzll(after);
        head = (tid - first) % kLsGroup == 0;
        cnt = min(kLsGroup, next - tid);
      }
      const unsigned long long mask = __builtin_amdgcn_ballot_w64(head);
      if (bit == 0) s_heads[wq] = mask;
    }
    __syncthreads();
    int32_t* grp = w.lsg + (size_t)b * (Lp + 1);
    if (head) {
      int n = __builtin_popcountll(s_heads[wq] & ((1ull << bit) - 1));
      for (int q = 0; q < wq; ++q) n += __builtin_popcountll(s_heads[q]);
      grp[1 + n] = tid | (cnt << 16);
    }
    if (tid == 0)
      grp[0] = __builtin_popcountll(s_heads[0]) + __builtin_popcountll(s_heads[1]) + __builtin_popcountll(s_heads[2]);
  }

  if (m.mode != kTransmission) return;
  // the upper triangle, in row segments of kPathSeg entries
  const int nseg = (L + kPathSeg - 1) / kPathSeg;
  if constexpr (sizeof(Real) == 8) {
    double* pm = w.pm64 + (size_t)b * Lp * Lp;
    for (int e = tid; e < Lp * Lp; e += kBlockP) {
      const int i = e / Lp, l = e % Lp;
      if (l < i || l >= L) pm[e] = 0.0;
    }
    for (int e = tid; e < nseg * L; e += kBlockP) {
      const int i = e % L, l0 = i + kPathSeg * (e / L);
      if (l0 < L) path_entries(s_r, s_dr, i, l0, min(l0 + kPathSeg, L), [&](int l, double v) { pm[(size_t)i * Lp + l] = v; });
    }
  } else {
    const int ldp = path_ld(Lp);
    for (int e = tid; e < nseg * L; e += kBlockP) {
      const int i = e % L, l0 = i + kPathSeg * (e / L);
      if (l0 < L)
        path_entries(s_r, s_dr, i, l0, min(l0 + kPathSeg, L), [&](int l, double v) {
          const uint16_t hv = bf16_rn((float)v);
          s_pm[i * ldp + l] = hv | ((uint32_t)bf16_rn((float)(v - (double)bf16_to_f(hv))) << 16);
        });
    }
    __syncthreads();
    // bf16 hi/lo A-operand fragments of v_mfma_f32_32x32x16_bf16:
    // lane holds row 32*mi + lane%32, columns 16*kb + 8*(lane/32) + j, j = 0..7
    const int MB = Lp / 32, KB = Lp / 16;
    const size_t plane = (size_t)MB * KB * 512;
    uint16_t* fh = w.pfrag + (size_t)b * 2 * plane;
    // the transposed fragments serve only the adjoint; a forward-only workspace has none
    uint16_t* fth = w.ptfrag ? w.ptfrag + (size_t)b * 2 * plane : nullptr;
    for (int e = tid; e < MB * KB * 64; e += kBlockP) {
      const int lane = e & 63, kb = (e >> 6) % KB, mi = (e >> 6) / KB;
      const int row = 32 * mi + (lane & 31);
      const int col0 = 16 * kb + 8 * (lane >> 5);
      // P[row][col] for the forward product, P[col][row] (transpose) for the adjoint
      uint32_t v[8], vt[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int col = col0 + j;
        v[j] = (row <= col && col < L) ? s_pm[row * ldp + col] : 0u;
        vt[j] = (col <= row && row < L) ? s_pm[col * ldp + row] : 0u;
      }
      auto put = [&](uint16_t* dst, const uint32_t (&x)[8], uint32_t sel) {   // the low or high halves
        uint32_t d[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) d[j] = __builtin_amdgcn_perm(x[2 * j + 1], x[2 * j], sel);
        *reinterpret_cast<uint4*>(dst + (size_t)e * 8) = make_uint4(d[0], d[1], d[2], d[3]);
      };
      put(fh, v, 0x05040100u);
      put(fh + plane, v, 0x07060302u);
      if (fth) {
        put(fth, vt, 0x05040100u);
        put(fth + plane, vt, 0x07060302u);
      }
    }
  }
}

// Non-grey cloud, reduced precision: Q_ext and its derivatives once per (sample,
// wavenumber), read by the forward kernel (Q_ext) and the layer sums (both).
// One thread per wavenumber; grid (n_nu_pad / kBlock, B).
__global__ __launch_bounds__(kBlock) void k_cloud_q(Model m, Work w) {
  const int b = blockIdx.y;
  const int nu = blockIdx.x * kBlock + threadIdx.x;
  if (nu >= m.n_nu_pad || w.status[b]) return;
  float dq[kCloudSpec];
  const float q = cloud_q<float>(m.cloud_qext, load_cloud<float>(w.cloud + (size_t)b * kCloudSpec), (float)m.nu[nu], dq);
  float* out = w.cloud_q + (size_t)b * (1 + kCloudSpec) * m.n_nu_pad + nu;
  out[0] = q;
#pragma unroll
  for (int k = 0; k < kCloudSpec; ++k) out[(size_t)(1 + k) * m.n_nu_pad] = dq[k];
}

constexpr int kBlockClasses = 256;

// Layer-count classes of the call: class 0 holds the samples of at most kShortLayers
// layers (and invalid samples, which the kernels skip), class 1 the rest; each list is
// ordered longest first (ties by sample index), so the most expensive work items start
// first.  One workgroup; a sample's rank counts the samples ahead of it in its class.
__global__ __launch_bounds__(kBlockClasses) void k_layer_classes(Work w, int B) {
  __shared__ int s_l[kBlockClasses];   // layer counts of a run of samples (0: invalid)
  auto layers = [&](int q) { return w.status[q] ? 0 : w.nlay[q]; };
  int n_long = 0;
  for (int b0 = 0; b0 < B; b0 += kBlockClasses) {
    const int b = b0 + threadIdx.x;
    const int lb = b < B ? layers(b) : 0;
    const bool cb = lb > kShortLayers;
    int rank = 0;
    n_long = 0;
    for (int q0 = 0; q0 < B; q0 += kBlockClasses) {
      __syncthreads();   // the last run's readers are done
      if (q0 + (int)threadIdx.x < B) s_l[threadIdx.x] = layers(q0 + threadIdx.x);
      __syncthreads();
      const int n = min(kBlockClasses, B - q0);
      for (int q = 0; q < n; ++q) {
        const int lq = s_l[q];
        const bool cq = lq > kShortLayers;
        n_long += cq;
        rank += cq == cb && (lq > lb || (lq == lb && q0 + q < b));
      }
    }
    if (b < B) w.cls[2 + (cb ? B : 0) + rank] = b;
  }
  if (threadIdx.x == 0) {
    w.cls[0] = B - n_long;
    w.cls[1] = n_long;
  }
}

void launch_layer_classes(const Model& m, const Work& w, int B, hipStream_t st) {
  (void)m;
  hipLaunchKernelGGL(k_layer_classes, dim3(1), dim3(kBlockClasses), 0, st, w, B);
}

// dynamic LDS of the profile kernel: the table axes and, in reduced precision, the path matrix
static size_t profile_lds_bytes(const Model& m, bool fp64) {
  return (size_t)(m.n_t + m.n_p + m.n_tc) * 8 +
         (m.mode == kTransmission && !fp64 ? (size_t)m.L_pad * path_ld(m.L_pad) * 4 : 0);
}

hipError_t profile_configure(const Model& m, bool fp64) {
  if (fp64) return hipSuccess;
  return hipFuncSetAttribute((const void*)k_profile<float>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)((size_t)kMaxLayers * path_ld(kMaxLayers) * 4 + 3 * kMaxAxis * 8));
}

void launch_profile(const Model& m, const Work& w, int B, const double* params, const int32_t* n_layers,
                    bool fp64, hipStream_t st) {
  if (fp64) {
    hipLaunchKernelGGL(k_profile<double>, dim3(B), dim3(kBlockP), profile_lds_bytes(m, true), st, m, w, params, n_layers);
  } else {
    hipLaunchKernelGGL(k_profile<float>, dim3(B), dim3(kBlockP), profile_lds_bytes(m, false), st, m, w, params, n_layers);
    if (m.cloud_ng)
      hipLaunchKernelGGL(k_cloud_q, dim3((unsigned)((m.n_nu_pad + kBlock - 1) / kBlock), (unsigned)B), dim3(kBlock), 0,
                         st, m, w);
  }
}

}  // namespace exofwd
