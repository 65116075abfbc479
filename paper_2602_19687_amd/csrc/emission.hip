// Emission forward kernels: per (sample, 64-wavenumber tile) the vertical
// optical depth of every layer (pure absorption: line tables and CIA), the
// Planck intensity at every level, the upward linear-in-tau intensity sweep
// for each Gauss-Legendre angle and the planet/star flux ratio (Eq. 45).
// One thread owns one (wavenumber, angle) pair during the sweep.
//
// Reduced precision: the tables store log2 sigma - c as FP32, one 4-byte word
// per entry (24 significant bits, against 11 for the FP16 transmission tables):
// emitted flux is far more sensitive to opacity errors than the transit depth.
#include "emission.h"
#include "kernels.h"
#include "opacity.h"

namespace exofwd {

// plain FP64 path: 256 threads per 64-wavenumber tile, the column in chunks of kChunk64
// layers.  Each wave forms the optical depths of a contiguous quarter of the chunk (the
// table entries of a cell kept while the cell is unchanged) and Planck rows, into LDS; each
// wave then carries its angles up through the chunk.  Chunks keep the LDS at 35 KB, so four
// workgroups share a CU (one, when whole columns were staged).  24 samples x 20000
// wavenumbers x 100 layers x 8 absorbers: 3.06 -> 0.86 ms; bound by the FP64 vector rate.
constexpr int kChunk64 = 32;

template <int S, bool CIA>
__global__ __launch_bounds__(kBlock) void k_emission_fp64(Model m, Work w, Tables tb, int B, double* __restrict__ spec,
                                                          double* __restrict__ dtau_out) {
  __shared__ double s_dt[kChunk64][kTile64], s_b[kChunk64 + 1][kTile64], s_f[kBlock / 64][kTile64];
  constexpr int kWaves = kBlock / 64, kAngles = kMaxMu / kWaves;
  const int logical = xcd_logical_block(blockIdx.x, gridDim.x);
  const int b = logical % B, tile = logical / B;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int Lp = m.L_pad;
  const int nu0 = tile * kTile64;
  double* out = spec + (size_t)b * m.n_nu;
  if (w.status[b]) {
    if (tid < kTile64 && nu0 + tid < m.n_nu) out[nu0 + tid] = __builtin_nan("");
    return;
  }
  const int L = w.nlay[b];
  const auto rec = const_ptr(reinterpret_cast<const double*>(w.rec)) + (size_t)b * Lp * rec_len(S);
  const auto cells = const_ptr(w.cells) + (size_t)b * Lp;
  const auto t_lev = const_ptr(w.t_lev) + (size_t)b * (Lp + 1);
  const int nu = nu0 + lane;
  const double nud = m.nu[nu];
  const double c1n3 = 2.0 * kHpl * kC * kC * nud * nud * nud;
  const double c2n = kHpl * kC / kB * nud;
  double inv_mu[kAngles], inten[kAngles], bb = 0.0;
#pragma unroll
  for (int q = 0; q < kAngles; ++q) {
    const int k = wv + kWaves * q;
    inv_mu[q] = k < m.n_mu ? 1.0 / m.mu_nodes[k] : 0.0;
    inten[q] = 0.0;
  }
  for (int c0 = 0; c0 < L; c0 += kChunk64) {
    const int n = min(kChunk64, L - c0);
    LayerRows64<S, CIA> rows;
    int cell_prev = -1;
    for (int l = c0 + n * wv / kWaves; l < c0 + n * (wv + 1) / kWaves; ++l) {
      const int cl = cells[l];
      if (cl != cell_prev) {
        fetch_rows64<S, CIA>(m, tb, cl, nu, rows);
        cell_prev = cl;
      }
      double d = eval_rows64<S, CIA>(rec + (size_t)l * rec_len(S), rows, 0.0, 0.0);
      d = d > 1.0e300 ? 1.0e300 : d;
      s_dt[l - c0][lane] = d;
      // the reverse pass reads the layer optical depths back
      if (dtau_out) __builtin_nontemporal_store(d, &dtau_out[((size_t)b * Lp + l) * m.n_nu_pad + nu]);
    }
    for (int j = wv; j <= n; j += kWaves) {
      double em1, ie;
      s_b[j][lane] = planck_d(c1n3, c2n / t_lev[c0 + j], em1, ie);
    }
    __syncthreads();
    if (c0 == 0) {
      bb = s_b[0][lane];
#pragma unroll
      for (int q = 0; q < kAngles; ++q) inten[q] = bb;
    }
    if (wv < m.n_mu) {
      for (int l = 0; l < n; ++l) {
        const double d = s_dt[l][lane], bt = s_b[l + 1][lane];
#pragma unroll
        for (int q = 0; q < kAngles; ++q) {
          if (wv + kWaves * q >= m.n_mu) break;
          double e, om, src, r;
          slab_d(d * inv_mu[q], e, om, src, r);
          // I e^-x + B_top (1 - e^-x) + (B_bot - B_top) src, as an increment of I
          inten[q] = fma(om, bt - inten[q], fma(bb - bt, src, inten[q]));
        }
        bb = bt;
      }
    }
    __syncthreads();   // the next chunk overwrites the rows
  }
  double flux = 0.0;
#pragma unroll
  for (int q = 0; q < kAngles; ++q) {
    const int k = wv + kWaves * q;
    if (k < m.n_mu) flux = fma(2.0 * M_PI * m.mu_weights[k] * m.mu_nodes[k], inten[q], flux);
  }
  s_f[wv][lane] = flux;
  __syncthreads();
  if (tid < kTile64 && nu0 + tid < m.n_nu) {
    const double f = (s_f[0][tid] + s_f[1][tid]) + (s_f[2][tid] + s_f[3][tid]);
    const double fstar =
        m.has_bd ? 1.0 : M_PI * 2.0 * kHpl * kC * kC * nud * nud * nud / expm1(kHpl * kC * nud / (kB * m.t_star));
    out[nu0 + tid] = m.dilution * f / fstar * w.core[b];
  }
}

// reduced precision: one wave per (sample, 64-wavenumber tile), one wavenumber per
// lane, streaming up the layers: each layer's optical depth and its upper level's
// Planck intensity are formed where the angle sweeps need them, so nothing is
// staged in LDS and waves never wait for each other.  A workgroup holds four
// neighbouring tiles of one sample.
template <int S, bool CIA>
__global__ __launch_bounds__(kBlock) void k_emission_mixed(Model m, Work w, Tables tb, int B, float* __restrict__ spec,
                                                           float* __restrict__ dtau_out) {
  const int logical = xcd_logical_block(blockIdx.x, gridDim.x);
  const int b = logical % B;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tile = (logical / B) * 4 + wv;
  if (tile >= m.n_tiles64) return;
  const int nu0 = tile * kTile64, nu = nu0 + lane;
  float* out = spec + (size_t)b * m.n_nu;
  if (w.status[b]) {
    if (nu < m.n_nu) out[nu] = __builtin_nanf("");
    return;
  }
  const int L = w.nlay[b], Lp = m.L_pad;
  constexpr int RL = rec_len(S);
  const float* rec = reinterpret_cast<const float*>(w.rec) + (size_t)b * Lp * RL;
  const int32_t* cells = w.cells + (size_t)b * Lp;
  const double* t_lev = w.t_lev + (size_t)b * (Lp + 1);
  const double* inv_t = w.inv_tlev + (size_t)b * (Lp + 1);
  const size_t npad = (size_t)m.n_nu_pad;
  // FP32 tables: 4 bytes per (row, wavenumber)
  const uint32_t row_bytes = (uint32_t)npad * 4u, tstep = (uint32_t)m.n_p * row_bytes;
  const __amdgpu_buffer_rsrc_t rh = make_rsrc(tb.h, (size_t)S * m.n_t * m.n_p * npad * 4);
  const __amdgpu_buffer_rsrc_t rhc = make_rsrc(CIA ? (const void*)tb.hc : (const void*)tb.h,
                                               CIA ? (size_t)2 * m.n_tc * npad * 4 : 0);
  const uint32_t voff = (uint32_t)lane * 4u, nu0_bytes = (uint32_t)nu0 * 4u;
  float cs[S], ccs[2];
#pragma unroll
  for (int s2 = 0; s2 < S; ++s2) cs[s2] = tb.c[(size_t)s2 * npad + nu];
#pragma unroll
  for (int p = 0; p < 2; ++p) ccs[p] = CIA ? tb.cc[(size_t)p * npad + nu] : 0.0f;

  const double nud = m.nu[nu];
  const float c1n3 = (float)(2.0 * kHpl * kC * kC * nud * nud * nud);
  const double c2n_log2e = kHpl * kC / kB * 1.4426950408889634074 * nud;
  auto planck_at = [&](int j) {
    float y, em1;
    return planck_split(c1n3, c2n_log2e, inv_t[j], y, em1);
  };
  const int n_mu = m.n_mu;
  // the intensities accumulate in FP64: a hundred FP32 updates would leave ~1e-6 of
  // rounding in the flux, which the likelihood residuals near the best fit amplify
  float inv_mu[kMaxMu];
  double inten[kMaxMu];
  float b_bot = planck_at(0);
#pragma unroll
  for (int k = 0; k < kMaxMu; ++k) {
    inv_mu[k] = k < n_mu ? (float)(1.0 / m.mu_nodes[k]) : 0.0f;
    inten[k] = b_bot;
  }

  // table entries of the current cell: a layer in the same cell as the one below reuses them
  float tp[4 * S + 4];
  int cell_prev = -1;
  for (int l = 0; l < L; ++l) {
    // ---- optical depth of layer l
    const int cl = cells[l];
    const float* rl = rec + (size_t)l * RL;
    if (cl != cell_prev) {
      const int it = cl & 255, ip = (cl >> 8) & 255, itc = cl >> 16;
#pragma unroll
      for (int s2 = 0; s2 < S; ++s2) {
        const uint32_t row = (uint32_t)((s2 * m.n_t + it) * m.n_p + ip) * row_bytes + nu0_bytes;
        tp[4 * s2] = load_f32(rh, voff, row);
        tp[4 * s2 + 1] = load_f32(rh, voff, row + tstep);
        tp[4 * s2 + 2] = load_f32(rh, voff, row + row_bytes);
        tp[4 * s2 + 3] = load_f32(rh, voff, row + tstep + row_bytes);
      }
      if (CIA) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          const uint32_t row = (uint32_t)(p * m.n_tc + itc) * row_bytes + nu0_bytes;
          tp[4 * S + 2 * p] = load_f32(rhc, voff, row);
          tp[4 * S + 2 * p + 1] = load_f32(rhc, voff, row + row_bytes);
        }
      }
      cell_prev = cl;
    }
    const float wt = rl[0], wp = rl[1];
    const float w11 = wt * wp, w10 = wt - w11, w01 = wp - w11, w00 = 1.0f - wt - wp + w11;
    float d = 0.0f;
#pragma unroll
    for (int s2 = 0; s2 < S; ++s2) {
      const float p00 = tp[4 * s2], p10 = tp[4 * s2 + 1], p01 = tp[4 * s2 + 2], p11 = tp[4 * s2 + 3];
      float v = cs[s2] + rl[kRecFixed + s2];
      v = fmaf(w00, p00, v);
      v = fmaf(w10, p10, v);
      v = fmaf(w01, p01, v);
      v = fmaf(w11, p11, v);
      d += exp2_fast(v);
    }
    if (CIA) {
      const float wtc = rl[2];
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const float a = tp[4 * S + 2 * p], c2 = tp[4 * S + 2 * p + 1];
        float v = ccs[p] + rl[5 + p];
        v = fmaf(1.0f - wtc, a, v);
        v = fmaf(wtc, c2, v);
        d += exp2_fast(v);
      }
    }
    // the reverse pass reads the layer optical depths back
    if (dtau_out) __builtin_nontemporal_store(d, &dtau_out[((size_t)b * Lp + l) * npad + nu]);
    // ---- the sweep through layer l for every angle
    const float b_top = planck_at(l + 1);
    const float db = b_bot - b_top;
#pragma unroll
    for (int k = 0; k < kMaxMu; ++k) {
      if (k >= n_mu) break;
      const float x = d * inv_mu[k];
      const float e = exp2_fast(-1.4426950408889634f * x);
      float om, src;
      slab_terms(x, e, om, src);
      // I e^-x + B_top (1 - e^-x) + (B_bot - B_top) src, as an increment of I
      inten[k] = fma((double)om, (double)b_top - inten[k], fma((double)db, (double)src, inten[k]));
    }
    b_bot = b_top;
  }
  double flux = 0.0;
#pragma unroll
  for (int k = 0; k < kMaxMu; ++k)
    if (k < n_mu) flux = fma(2.0 * M_PI * m.mu_weights[k] * m.mu_nodes[k], inten[k], flux);
  if (nu < m.n_nu) {
    const double fstar =
        m.has_bd ? 1.0 : M_PI * 2.0 * kHpl * kC * kC * nud * nud * nud / expm1(kHpl * kC * nud / (kB * m.t_star));
    out[nu] = (float)(m.dilution * flux / fstar * w.core[b]);
  }
}

template <int S, bool CIA>
const void* emis_kernel(bool fp64) {
  return fp64 ? (const void*)k_emission_fp64<S, CIA> : (const void*)k_emission_mixed<S, CIA>;
}

const void* emis_kernel_for(int S, bool cia, bool fp64) {
#define EXOFWD_CASE(n) \
  case n: return cia ? emis_kernel<n, true>(fp64) : emis_kernel<n, false>(fp64);
  switch (S) {
    EXOFWD_CASE(1) EXOFWD_CASE(2) EXOFWD_CASE(3) EXOFWD_CASE(4)
    EXOFWD_CASE(5) EXOFWD_CASE(6) EXOFWD_CASE(7) EXOFWD_CASE(8)
  }
#undef EXOFWD_CASE
  return nullptr;
}

hipError_t emission_configure(const Model& m, bool fp64) {
  return emis_kernel_for(m.S, m.has_cia, fp64) ? hipSuccess : hipErrorInvalidValue;
}

void launch_emission(const Model& m, const Work& w, const Tables& tb, int B, void* spec, bool fp64, hipStream_t st,
                     void* dtau_out) {
  // FP64: a tile per workgroup; reduced precision: four 64-wavenumber tiles (one per wave)
  // of one sample
  const dim3 grid((unsigned)((fp64 ? m.n_tiles64 : (m.n_tiles64 + 3) / 4) * B));
  void* args[] = {(void*)&m, (void*)&w, (void*)&tb, (void*)&B, (void*)&spec, (void*)&dtau_out};
  hipLaunchKernel(emis_kernel_for(m.S, m.has_cia, fp64), grid, dim3(kBlock), args, 0, st);
}

}  // namespace exofwd
