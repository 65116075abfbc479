// Per-layer opacity evaluation shared by the transmission forward and adjoint
// kernels.  A wave evaluates one layer at a time (all per-layer data are
// wave-uniform and live in SGPRs); lanes run along wavenumber.
//
// Reduced-precision form, two adjacent wavenumbers per lane:
//   dtau = D + R nu4 + sum_s 2^(c_s + bilinear(h_s) + lam_s) + sum_pairs 2^(c_p + lerp_T(h_p) + lam_p)
// with FP16 table entries h = log2 sigma - c (c per source and wavenumber),
// bilinear weights in (T, log p), lam = log2 of the layer prefactor
// (n X dr for lines, n^2 X X dr for CIA), R the Rayleigh and D the cloud term
// (the non-grey cloud's D is a column that multiplies Q_ext(nu)).
#pragma once
#include "common.h"

namespace exofwd {

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

__device__ inline float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

// 1 - e^-tau given e = e^-tau: below tau = 1/64, where 1 - e keeps too few digits
// of a thin chord's absorption in FP32, the series tau (1 - tau/2 + tau^2/6)
// (truncation tau^3/24 relative, under 2e-7)
__device__ inline float one_minus_exp(float tau, float e) {
  return tau < 0.015625f ? tau * (1.0f - tau * (0.5f - tau * (1.0f / 6.0f))) : 1.0f - e;
}

// Wave-uniform data of one (sample, layer).
template <int S>
struct LayerCoef {
  uint32_t row[S];      // byte offset of the (s, iT, iP) table row at the tile start
  uint32_t rowc[2];     // byte offset of the (pair, iTc) CIA row at the tile start
  float w00, w10, w01, w11, wtc, R, D;
  float lam[S], lamc[2];
  float col[S];        // line prefactors n X_s dr (2^lam)
  float wt, wp, omp;   // T and log p weights, 1 - wP (derivative form of the bilinear)
  int cell;            // packed (iT, iP, iTc): equal cells read equal table pairs
};

struct TableGeom {
  uint32_t row_bytes;   // n_nu_pad * 2
  uint32_t tstep;       // bytes from iT to iT+1
  uint32_t pstep;       // bytes from iP to iP+1
};

template <int S>
__device__ inline LayerCoef<S> load_layer(const Model& m, const int32_t* __restrict__ cells,
                                          const float* __restrict__ rec, int l, uint32_t nu0_bytes,
                                          const TableGeom& g) {
  LayerCoef<S> c;
  const int cl = cells[l];
  const int it = cl & 255, ip = (cl >> 8) & 255, itc = cl >> 16;
  c.cell = cl;
  const float* rl = rec + (size_t)l * rec_len_wide(S);
  const float wt = rl[0], wp = rl[1];
  c.wt = wt;
  c.wp = wp;
  c.omp = 1.0f - wp;
  c.w11 = wt * wp;
  c.w10 = wt - c.w11;
  c.w01 = wp - c.w11;
  c.w00 = 1.0f - wt - wp + c.w11;
  c.wtc = rl[2];
  c.R = rl[3];
  c.D = rl[4];
  c.lamc[0] = rl[5];
  c.lamc[1] = rl[6];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    c.lam[s] = rl[kRecFixed + s];
    c.col[s] = rl[kRecFixed + S + s];
    c.row[s] = (uint32_t)(((s * m.n_t + it) * m.n_p + ip)) * g.row_bytes + nu0_bytes;
  }
#pragma unroll
  for (int p = 0; p < 2; ++p) c.rowc[p] = (uint32_t)(p * m.n_tc + itc) * g.row_bytes + nu0_bytes;
  return c;
}

// Per-lane constants for two adjacent wavenumbers.
template <int S>
struct LaneConst {
  float c0[S], c1[S], cc0[2], cc1[2], nu4_0, nu4_1;
};

template <int S, bool CIA>
__device__ inline LaneConst<S> load_lane(const Model& m, const Tables& tb, int nu) {
  LaneConst<S> k;
  const size_t np = (size_t)m.n_nu_pad;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const float2 c = *reinterpret_cast<const float2*>(tb.c + s * np + nu);
    k.c0[s] = c.x;
    k.c1[s] = c.y;
  }
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    if (CIA) {
      const float2 c = *reinterpret_cast<const float2*>(tb.cc + p * np + nu);
      k.cc0[p] = c.x;
      k.cc1[p] = c.y;
    } else {
      k.cc0[p] = k.cc1[p] = 0.0f;
    }
  }
  const float2 n4 = *reinterpret_cast<const float2*>(tb.nu4f + nu);
  k.nu4_0 = n4.x;
  k.nu4_1 = n4.y;
  return k;
}

__device__ inline float load_f32(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(float, (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}
__device__ inline half2_t load_h2(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(half2_t, (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}

// Raw FP16 table pairs of one layer: four bilinear corners per line source,
// two T rows per CIA pair.
template <int S, bool CIA>
struct LayerRaw {
  half2_t h[4 * S + (CIA ? 4 : 0)];
};

template <int S, bool CIA>
__device__ inline void fetch_terms(const LayerCoef<S>& c, const TableGeom& g, __amdgpu_buffer_rsrc_t rh,
                                   __amdgpu_buffer_rsrc_t rhc, uint32_t voff, LayerRaw<S, CIA>& r) {
#pragma unroll
  for (int s = 0; s < S; ++s) {
    r.h[4 * s + 0] = load_h2(rh, voff, c.row[s]);
    r.h[4 * s + 1] = load_h2(rh, voff, c.row[s] + g.tstep);
    r.h[4 * s + 2] = load_h2(rh, voff, c.row[s] + g.pstep);
    r.h[4 * s + 3] = load_h2(rh, voff, c.row[s] + g.tstep + g.pstep);
  }
  if constexpr (CIA) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      r.h[4 * S + 2 * p] = load_h2(rhc, voff, c.rowc[p]);
      r.h[4 * S + 2 * p + 1] = load_h2(rhc, voff, c.rowc[p] + g.row_bytes);
    }
  }
}

// Optical depth of one layer at two wavenumbers from its fetched table pairs:
// Rayleigh + cloud, the VMR-weighted line terms (bilinear in T and log p of the
// log2 tables) and the CIA pair terms (linear in T).
// With the non-grey cloud (NGC) D is the layer's cloud column and q0, q1 the
// extinction efficiency Q_ext at the two wavenumbers.
template <int S, bool CIA, bool NGC = false>
__device__ inline void eval_terms(const LayerCoef<S>& c, const LaneConst<S>& k, const LayerRaw<S, CIA>& r, float& d0,
                                  float& d1, float q0 = 1.0f, float q1 = 1.0f) {
  if constexpr (NGC) {
    d0 = fmaf(c.D, q0, c.R * k.nu4_0);
    d1 = fmaf(c.D, q1, c.R * k.nu4_1);
  } else {
    d0 = fmaf(c.R, k.nu4_0, c.D);
    d1 = fmaf(c.R, k.nu4_1, c.D);
  }
  // line terms: the cross-section (log2 sigma = c + the interpolated entry) times the
  // layer's prefactor, which then costs no add to the exponent
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const half2_t h00 = r.h[4 * s], h10 = r.h[4 * s + 1], h01 = r.h[4 * s + 2], h11 = r.h[4 * s + 3];
    float v0 = fmaf(c.w00, (float)h00.x, k.c0[s]);
    float v1 = fmaf(c.w00, (float)h00.y, k.c1[s]);
    v0 = fmaf(c.w10, (float)h10.x, v0);
    v1 = fmaf(c.w10, (float)h10.y, v1);
    v0 = fmaf(c.w01, (float)h01.x, v0);
    v1 = fmaf(c.w01, (float)h01.y, v1);
    v0 = fmaf(c.w11, (float)h11.x, v0);
    v1 = fmaf(c.w11, (float)h11.y, v1);
    d0 = fmaf(c.col[s], exp2_fast(v0), d0);
    d1 = fmaf(c.col[s], exp2_fast(v1), d1);
  }
  if constexpr (CIA) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const half2_t a = r.h[4 * S + 2 * p], b = r.h[4 * S + 2 * p + 1];
      float v0 = k.cc0[p] + c.lamc[p];
      float v1 = k.cc1[p] + c.lamc[p];
      v0 = fmaf(1.0f - c.wtc, (float)a.x, v0);
      v1 = fmaf(1.0f - c.wtc, (float)a.y, v1);
      v0 = fmaf(c.wtc, (float)b.x, v0);
      v1 = fmaf(c.wtc, (float)b.y, v1);
      d0 += exp2_fast(v0);
      d1 += exp2_fast(v1);
    }
  }
}

__device__ inline __amdgpu_buffer_rsrc_t make_rsrc(const void* p, size_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)(bytes > 0x7fffffffu ? 0x7fffffff : bytes),
                                           0x00020000);
}

typedef __attribute__((ext_vector_type(2))) float float2v;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

// A float as a packed (bf16 hi | bf16 lo << 16) pair, hi + lo ~ 16 significant
// bits; both roundings are the hardware's round-to-nearest-even conversion.
__device__ inline uint32_t pack_hl(float v) {
  const float hf = (float)(__bf16)v;
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((float2v){v, v - hf}, bf16x2));
}

// bf16 hi pair (a, b) and lo pair of two floats, each as one dword (a in the low half).
__device__ inline void split_pair(float a, float b, uint32_t& hp, uint32_t& lp) {
  hp = __builtin_bit_cast(uint32_t, __builtin_convertvector((float2v){a, b}, bf16x2));
  const float ha = __uint_as_float(hp << 16), hb = __uint_as_float(hp & 0xffff0000u);
  lp = __builtin_bit_cast(uint32_t, __builtin_convertvector((float2v){a - ha, b - hb}, bf16x2));
}

// hi and lo bf16x8 fragments from eight packed pairs
__device__ inline void frag_hl(const uint32_t* x, bf16x8& hi, bf16x8& lo) {
  uint32_t h[4], l[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    h[i] = __builtin_amdgcn_perm(x[2 * i + 1], x[2 * i], 0x05040100u);
    l[i] = __builtin_amdgcn_perm(x[2 * i + 1], x[2 * i], 0x07060302u);
  }
  hi = __builtin_bit_cast(bf16x8, make_uint4(h[0], h[1], h[2], h[3]));
  lo = __builtin_bit_cast(bf16x8, make_uint4(l[0], l[1], l[2], l[3]));
}

// ---------------------------------------------------------------------------
// Plain FP64 form: log10 sigma tables read as they are, one wavenumber per lane.

// (2^f - 1) / f on [-1/2, 1/2], interpolated at the Chebyshev points of the interval: then
// 1 + f q(f) is 2^f to 2e-17 relative
__device__ inline double exp2_q(double f) {
  double q = 4.4549605981865186e-10;
  q = fma(q, f, 7.072585949269223e-09);
  q = fma(q, f, 1.0178062445845774e-07);
  q = fma(q, f, 1.321544258792169e-06);
  q = fma(q, f, 1.525273382983612e-05);
  q = fma(q, f, 0.0001540353044173605);
  q = fma(q, f, 0.0013333558146416936);
  q = fma(q, f, 0.009618129107606888);
  q = fma(q, f, 0.0555041086648216);
  q = fma(q, f, 0.24022650695910097);
  return fma(q, f, 0.6931471805599453);
}
// sqrt(x), correctly rounded but for the rarest ties, and half = 1 / (2 sqrt(x)) to 1e-13 (x
// > 0 normal): one coupled Newton step, then the root's own residual
__device__ inline double sqrt_d(double x, double& half) {
  const double r = __builtin_amdgcn_rsq(x);
  double g = x * r, h = 0.5 * r;
  const double d = fma(-h, g, 0.5);
  g = fma(g, d, g);
  half = h = fma(h, d, h);
  return fma(fma(-g, g, x), h, g);
}
// 1 / s from half = 1 / (2 s) to 1e-13 (0.5 ulp)
__device__ inline double rcp_of_root_d(double s, double half) {
  const double r = half + half;
  return fma(fma(-s, r, 1.0), r, r);
}
// 2^x for finite x (0 or infinity past the exponent range).  At x = -inf, x - rint(x) would
// be a NaN: the exponents are kept finite where they come from (kAbsentLog).
__device__ inline double exp2_d(double x) {
  const double n = __builtin_rint(x), f = x - n;
  return __builtin_ldexp(fma(exp2_q(f), f, 1.0), (int)n);
}
// 1 / x (x and 1 / x normal): two Newton steps, the last of which rounds once (0.5 ulp)
__device__ inline double rcp_d(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  return fma(fma(-x, r, 1.0), r, r);
}
// a / b given r = 1 / b, with the quotient's own residual added (0.5 ulp; a r alone 1.4)
__device__ inline double div_d(double a, double b, double r) {
  const double q = a * r;
  return fma(fma(-b, q, a), r, q);
}
// e = e^y and em1 = e^y - 1, which keeps its digits where y is small, for -760 <= y <= 709:
// y = n ln 2 + r with ln 2 in two parts (the first product's difference is exact, Cody and
// Waite), em1 = 2^n (r + r^2 h(r)) + (2^n - 1) with h = (e^r - 1 - r) / r^2 interpolated at
// the Chebyshev points of [-ln 2 / 2, ln 2 / 2] (to 2e-18).  Both within an ulp (em1 two for
// y in [0.35, 1.04]), as the library's.  As 2^(y log2 e) they would carry the rounding of
// the product: e^-30 to 25 ulp.
__device__ inline void exp_d(double y, double& em1, double& e) {
  const double n = __builtin_rint(y * 1.4426950408889634074);
  double r = fma(n, -0.6931471805599453, y);
  r = fma(n, -2.3190468138462996e-17, r);
  double h = 2.0914679376583935e-09;
  h = fma(h, r, 2.510520637395701e-08);
  h = fma(h, r, 2.7557273661348637e-07);
  h = fma(h, r, 2.7557255425746435e-06);
  h = fma(h, r, 2.4801587325533363e-05);
  h = fma(h, r, 0.00019841269874800493);
  h = fma(h, r, 0.0013888888888883752);
  h = fma(h, r, 0.008333333333326141);
  h = fma(h, r, 0.04166666666666667);
  h = fma(h, r, 0.1666666666666667);
  h = fma(h, r, 0.5);
  const double t = fma(r * r, h, r), s = __builtin_ldexp(1.0, (int)n);
  em1 = fma(s, t, s - 1.0);
  e = fma(s, t, s);
}
// e = e^-tau (0 past 745) and om = 1 - e^-tau for tau >= 0 (infinite included; a NaN stays one)
__device__ inline void absorb_d(double tau, double& om, double& e) {
  double em1;
  exp_d(tau > 760.0 ? -760.0 : -tau, em1, e);
  om = -em1;
}
// e^-tau alone
__device__ inline double exp_neg_d(double tau) {
  double om, e;
  absorb_d(tau, om, e);
  return e;
}

// Table entries of one layer at this lane's wavenumber: four bilinear corners (T and log p
// steps: 00, 10, 01, 11) per line source, two T rows per CIA pair.
template <int S, bool CIA>
struct LayerRows64 {
  double t[4 * S + (CIA ? 4 : 0)];
};

template <int S, bool CIA>
__device__ inline void fetch_rows64(const Model& m, const Tables& tb, int cl, int nu, LayerRows64<S, CIA>& r) {
  const int it = cl & 255, ip = (cl >> 8) & 255, itc = cl >> 16;
  const size_t npad = (size_t)m.n_nu_pad, tstep = (size_t)m.n_p * npad;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const double* p = tb.t64 + (((size_t)s * m.n_t + it) * m.n_p + ip) * npad;
    r.t[4 * s] = p[nu];
    r.t[4 * s + 1] = (p + tstep)[nu];
    r.t[4 * s + 2] = (p + npad)[nu];
    r.t[4 * s + 3] = (p + tstep + npad)[nu];
  }
  if constexpr (CIA) {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const double* p = tb.tc64 + ((size_t)c * m.n_tc + itc) * npad;
      r.t[4 * S + 2 * c] = p[nu];
      r.t[4 * S + 2 * c + 1] = (p + npad)[nu];
    }
  }
}

// Optical depth of one layer (record rl) from its table entries; qext multiplies the cloud
// column (1 for the grey deck).  The bilinear weights carry the factor log2(10).
template <int S, bool CIA, typename Rec>
__device__ inline double eval_rows64(Rec rl, const LayerRows64<S, CIA>& r, double nu4,
                                     double qext) {
  const double wt = rl[0], wp = rl[1];
  const double a = (1.0 - wp) * kLog2_10, b = wp * kLog2_10;
  const double w00 = (1.0 - wt) * a, w10 = wt * a, w01 = (1.0 - wt) * b, w11 = wt * b;
  double acc = fma(rl[3], nu4, rl[4] * qext);
#pragma unroll
  for (int s = 0; s < S; ++s) {
    double x = fma(w00, r.t[4 * s], rl[kRecFixed + s]);
    x = fma(w10, r.t[4 * s + 1], x);
    x = fma(w01, r.t[4 * s + 2], x);
    acc += exp2_d(fma(w11, r.t[4 * s + 3], x));
  }
  if constexpr (CIA) {
    const double wc = rl[2] * kLog2_10, wc0 = (1.0 - rl[2]) * kLog2_10;
#pragma unroll
    for (int c = 0; c < 2; ++c)
      acc += exp2_d(fma(wc, r.t[4 * S + 2 * c + 1], fma(wc0, r.t[4 * S + 2 * c], rl[5 + c])));
  }
  return acc;
}

// Line and CIA terms t of one layer with the derivative dw of each exponent with respect
// to its T weight (log2 units), formed from the differences of the table entries.
template <int S, bool CIA, typename Rec>
__device__ inline void eval_rows64_deriv(Rec rl, const LayerRows64<S, CIA>& r, double* t,
                                         double* dw) {
  const double wt = rl[0], a = (1.0 - rl[1]) * kLog2_10, b = rl[1] * kLog2_10;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const double t00 = r.t[4 * s], t10 = r.t[4 * s + 1], t01 = r.t[4 * s + 2], t11 = r.t[4 * s + 3];
    dw[s] = fma(b, t11 - t01, a * (t10 - t00));
    t[s] = exp2_d(fma(wt, dw[s], fma(b, t01, fma(a, t00, rl[kRecFixed + s]))));
  }
  if constexpr (CIA) {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const double t0 = r.t[4 * S + 2 * c], t1 = r.t[4 * S + 2 * c + 1];
      dw[S + c] = (t1 - t0) * kLog2_10;
      t[S + c] = exp2_d(fma(rl[2], dw[S + c], fma(kLog2_10, t0, rl[5 + c])));
    }
  }
}

// ---- FP64 chord products on v_mfma_f64_16x16x4f64 (a matrix product of the same rate as
// the vector FMAs, issued beside them): 16 x 16 tiles, k in blocks of 16 split over the
// lane quarters h = lane / 16 as k = 16 K + 4 h + step, so a lane's four entries of a row
// are contiguous.  A: row lane % 16; B: column lane % 16; D: row h + 4 e in element e.
typedef __attribute__((ext_vector_type(4))) double f64x4;

constexpr int kMaxBlocks16 = kMaxLayers / 16;
// layers rounded up to a whole 16-row block: the rows of the FP64 kernels' LDS tiles
__host__ __device__ constexpr int rows16(int layers) { return (layers + 15) / 16 * 16; }

// 16-row blocks of `part` of `parts` (2 or 4): each block in turn, the costliest first,
// goes to the part with the least cost so far; block i of nb costs nb - i, or i + 1 with `rev`
__device__ inline unsigned split_blocks16(int part, int parts, int nb, bool rev) {
  unsigned mine = 0;
  int c[4] = {0, 0, 0, 0};
  for (int q = 0; q < nb; ++q) {
    int best = 0;
    for (int p = 1; p < parts; ++p)
      if (c[p] < c[best]) best = p;
    if (best == part) mine |= 1u << (rev ? nb - 1 - q : q);
    c[best] += nb - q;
  }
  return mine;
}

}  // namespace exofwd
