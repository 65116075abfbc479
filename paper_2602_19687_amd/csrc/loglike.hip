// Binned Gaussian log-likelihood in FP64 (Eq. 1-3): box-car bin means of the
// spectrum, the instrument offset on masked bins, lnL and d lnL / d m_k; with
// the cloudy/clear mixing (Eq. 26) also the mixed spectrum and d lnL / d f_cld.
// A group of lanes (8 to 64, after the mean bin width) sums one bin: its lanes stride
// through the bin's wavenumbers (coalesced) and their partial sums meet in a fixed
// butterfly.  Then a workgroup per sample forms the bins' terms, a thread each, and adds
// them in a fixed order.  The bin sums run in a kernel of their own, over many workgroups,
// from kSplitLL wavenumbers on (they pass through the d lnL / d m_k buffer); below, in the
// sample's workgroup, where another launch would cost more than it gives.  Measured, both
// kernels against one: 1 sample x 30000 wavenumbers 11 us (26), 64 x 400000 59 (222), 1024 x
// 30000 91 (120); 1 x 2000 in one kernel 5.7.  About the line, whole calls on 2 layers, split
// against not (1, 256 and 1024 samples): 2000 wavenumbers 23.2 us (20.8), 40.9 (37.7), 110.5
// (109.0); 4096 23.3 (23.4), 55.8 (54.7), 182 (182); 8192 23.7 (27.5), 86.8 (88.3), 332 (333).
#include "kernels.h"

#include <type_traits>

namespace exofwd {

constexpr int kBlockLL = 512;    // threads per sample of the likelihood kernel
constexpr int kBinsLL = 4;       // bins of a group of lanes in flight
constexpr int kSplitLL = 4096;   // wavenumbers from which the bin sums have a kernel of their own

// Sums of kBinsLL bins k, k + step, ... (those below K) by the group of gl lanes holding
// lane glane of it: the bins' loads are in flight together
template <typename SpecT>
__device__ inline void bin_sums(const SpecT* __restrict__ sp, const int32_t* __restrict__ lo,
                                const int32_t* __restrict__ hi, int k, int step, int K, int gl, int glane, double* out) {
  double sum[kBinsLL];
  int i0[kBinsLL], i1[kBinsLL], most = 0;
#pragma unroll
  for (int u = 0; u < kBinsLL; ++u) {
    const int q = k + u * step;
    i0[u] = q < K ? lo[q] + glane : 0;
    i1[u] = q < K ? hi[q] : 0;
    most = max(most, i1[u] - i0[u]);
    sum[u] = 0.0;
  }
  for (int off = 0; off < most; off += gl) {
    SpecT v[kBinsLL];
#pragma unroll
    for (int u = 0; u < kBinsLL; ++u) v[u] = i0[u] + off < i1[u] ? sp[i0[u] + off] : SpecT(0);
#pragma unroll
    for (int u = 0; u < kBinsLL; ++u) sum[u] += (double)v[u];
  }
#pragma unroll
  for (int u = 0; u < kBinsLL; ++u) sum[u] = group_sum_all(sum[u], gl);
  if (glane == 0) {
#pragma unroll
    for (int u = 0; u < kBinsLL; ++u)
      if (k + u * step < K) out[k + u * step] = sum[u];
  }
}

// workgroups per sample of k_bin_sums
__host__ __device__ inline int bin_sum_blocks(const Model& m) {
  const int per = kBlock / m.ll_lanes * kBinsLL;
  return (m.K + per - 1) / per;
}

// bin sums of every (virtual) sample; one workgroup per kBinsLL bins of each of its groups
template <typename SpecT>
__global__ __launch_bounds__(kBlock) void k_bin_sums(Model m, Work w, const SpecT* __restrict__ spec,
                                                     const int32_t* __restrict__ lo, const int32_t* __restrict__ hi) {
  const int gl = m.ll_lanes, ngrp = kBlock / gl, nblk = bin_sum_blocks(m);
  const int v = blockIdx.x / nblk, blk = blockIdx.x - v * nblk;
  if (w.status[v]) return;
  bin_sums(spec + (size_t)v * m.n_nu, lo, hi, blk * ngrp * kBinsLL + (int)threadIdx.x / gl, ngrp, m.K, gl,
           threadIdx.x & (gl - 1), w.dm + (size_t)v * m.K);
}

// SUMS: the bin sums are formed here; else they are in w.dm
template <typename SpecT, bool SUMS>
__global__ __launch_bounds__(kBlockLL) void k_loglike(Model m, Work w, const double* __restrict__ params,
                                                    const SpecT* __restrict__ spec, SpecT* __restrict__ spec_out,
                                                    const int32_t* __restrict__ lo, const int32_t* __restrict__ hi,
                                                    const double* __restrict__ y, const double* __restrict__ yerr,
                                                    const uint8_t* __restrict__ mask, double* __restrict__ lnl,
                                                    int32_t* __restrict__ status_out) {
  const int b = blockIdx.x, tid = threadIdx.x;
  __shared__ double s_part[kBlockLL / 64], s_fpart[kBlockLL / 64], s_mpart[kBlockLL / 64];
  // cloudy/clear mixing (Eq. 26): virtual samples 2b (cloudy) and 2b+1 (clear) give
  // the spectrum f Phi_cld + (1 - f) Phi_cf; their dm carry the factors f and 1 - f
  const bool mix = m.has_fcld;
  const int bc = mix ? 2 * b : b;
  int status = mix ? (w.status[bc] | w.status[bc + 1]) : w.status[b];
  double* dm = w.dm + (size_t)bc * m.K;
  double* dm_cf = mix ? dm + m.K : nullptr;
  if (status) {
    for (int k = tid; k < m.K; k += kBlockLL) {
      dm[k] = 0.0;
      if (mix) dm_cf[k] = 0.0;
    }
    if (mix && spec_out)
      for (int i = tid; i < m.n_nu; i += kBlockLL) spec_out[(size_t)b * m.n_nu + i] = (SpecT)__builtin_nan("");
    if (tid == 0) {
      if (lnl) lnl[b] = kInvalidLnL;
      if (status_out) status_out[b] = status;
      if (mix) w.fbar[b] = 0.0;
      w.mdot[b] = 0.0;
    }
    return;
  }
  const double* th = params + (size_t)b * m.P;
  const double offset = m.has_offset ? th[m.idx_offset] * 1.0e-6 : 0.0;
  const double f = mix ? th[m.idx_fcld] : 1.0;
  const double infl = exp10(2.0 * m.err_c);
  const double half_ln2pi = 0.91893853320467274178032973640562;
  const SpecT* sp = spec + (size_t)bc * m.n_nu;
  const SpecT* sp_cf = mix ? sp + m.n_nu : nullptr;
  if (mix && spec_out)
    for (int i = tid; i < m.n_nu; i += kBlockLL)
      spec_out[(size_t)b * m.n_nu + i] = (SpecT)(f * (double)sp[i] + (1.0 - f) * (double)sp_cf[i]);
  double part = 0.0, fpart = 0.0, mpart = 0.0;
  if constexpr (SUMS) {
    const int gl = m.ll_lanes, ngrp = kBlockLL / gl;
    for (int k = tid / gl; k < m.K; k += kBinsLL * ngrp) {
      bin_sums(sp, lo, hi, k, ngrp, m.K, gl, tid & (gl - 1), dm);
      if (mix) bin_sums(sp_cf, lo, hi, k, ngrp, m.K, gl, tid & (gl - 1), dm_cf);
    }
    __syncthreads();
  }
  // the bins' terms, a thread per bin; a bin's sum gives way to its d lnL / d m_k
  for (int k = tid; k < m.K; k += kBlockLL) {
    const double cnt = (double)(hi[k] - lo[k]);
    const double m_cld = dm[k] / cnt, m_cf = mix ? dm_cf[k] / cnt : 0.0;
    const double mk = (mix ? f * m_cld + (1.0 - f) * m_cf : m_cld) + (mask && mask[k] ? offset : 0.0);
    const double s2 = yerr[k] * yerr[k] + infl;
    const double r = y[k] - mk;
    part += -0.5 * log(s2) - half_ln2pi - 0.5 * r * r / s2;
    if (mix) {
      dm[k] = f * r / s2;
      dm_cf[k] = (1.0 - f) * r / s2;
      fpart += r / s2 * (m_cld - m_cf);
    } else {
      dm[k] = r / s2;
    }
    mpart += r / s2 * (mix ? f * m_cld + (1.0 - f) * m_cf : m_cld);
  }
  // sums over the block in a fixed order: each wave's butterfly, then the waves
  part = wave_sum_all(part);
  fpart = wave_sum_all(fpart);
  mpart = wave_sum_all(mpart);
  if ((tid & 63) == 0) {
    s_part[tid >> 6] = part;
    s_fpart[tid >> 6] = fpart;
    s_mpart[tid >> 6] = mpart;
  }
  __syncthreads();
  if (tid == 0) {
    for (int k = 1; k < kBlockLL / 64; ++k) {
      s_part[0] += s_part[k];
      s_fpart[0] += s_fpart[k];
      s_mpart[0] += s_mpart[k];
    }
  }
  if (tid == 0) {
    double v = s_part[0];
    if (!isfinite(v)) {
      v = kInvalidLnL;
      status = kNonfinite;
      w.status[bc] = status;
      if (mix) w.status[bc + 1] = status;
    }
    if (lnl) lnl[b] = v;
    w.lnl_tmp[b] = v;
    if (mix) w.fbar[b] = status ? 0.0 : s_fpart[0];
    w.mdot[b] = status ? 0.0 : s_mpart[0];
    if (status_out) status_out[b] = status;
  }
}

__global__ __launch_bounds__(kBlock) void k_mix_grad(Model m, Work w, int B, double* __restrict__ grad) {
  const long i = (long)blockIdx.x * kBlock + threadIdx.x;
  if (i >= (long)B * m.P) return;
  const int b = (int)(i / m.P), j = (int)(i % m.P);
  grad[i] = j == m.idx_fcld ? w.fbar[b] : w.gv[(size_t)(2 * b) * m.P + j] + w.gv[(size_t)(2 * b + 1) * m.P + j];
}

void launch_loglike(const Model& m, const Work& w, int B, const double* params, const void* spec, void* spec_out,
                    bool spec_f64, const int32_t* bin_lo, const int32_t* bin_hi, const double* y, const double* yerr,
                    const uint8_t* mask, double* lnl, int32_t* status_out, hipStream_t st) {
  auto run = [&](auto* sp, auto* sp_out) {
    using SpecT = std::remove_const_t<std::remove_pointer_t<decltype(sp)>>;
    if (m.n_nu < kSplitLL) {
      hipLaunchKernelGGL((k_loglike<SpecT, true>), dim3(B), dim3(kBlockLL), 0, st, m, w, params, sp, sp_out, bin_lo,
                         bin_hi, y, yerr, mask, lnl, status_out);
      return;
    }
    hipLaunchKernelGGL(k_bin_sums<SpecT>, dim3((unsigned)(bin_sum_blocks(m) * (m.has_fcld ? 2 * B : B))), dim3(kBlock), 0,
                       st, m, w, sp, bin_lo, bin_hi);
    hipLaunchKernelGGL((k_loglike<SpecT, false>), dim3(B), dim3(kBlockLL), 0, st, m, w, params, sp, sp_out, bin_lo,
                       bin_hi, y, yerr, mask, lnl, status_out);
  };
  if (spec_f64) run((const double*)spec, (double*)spec_out);
  else run((const float*)spec, (float*)spec_out);
}

void launch_mix_grad(const Model& m, const Work& w, int B, double* grad, hipStream_t st) {
  const long n = (long)B * m.P;
  hipLaunchKernelGGL(k_mix_grad, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, m, w, B, grad);
}

}  // namespace exofwd
