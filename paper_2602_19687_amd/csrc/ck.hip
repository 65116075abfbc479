// Correlated-k path (Section "Gas phase opacities"): per spectral bin, each
// absorber's k-table holds the cross section at kCkG g-points of the bin's
// cumulative distribution with quadrature weights w_g (sum 1).  The species are
// mixed layer by layer by random overlap with resorting and rebinning (RORR,
// Amundsen et al. 2017): two k-distributions, as layer optical depths, combine on
// all g-point pairs (sum of the depths, product of the weights); the pairs are
// sorted and the sorted distribution is averaged over each original g-interval
// [E_{n-1}, E_n], E_n = w_1 + ... + w_n.  The next absorber is then mixed into the
// result, in table order.  The grey continuum (CIA, Rayleigh, grey deck at the bin
// centre) is added to every g-point.  Each g-point's column then goes through the
// transmission chord (Eq. 44) or the emission sweep (Eq. 45), and the bin's
// spectrum is the g-weighted sum.
//
// k_ck_mix: one wave per (sample, layer, 16 bins), a quad of lanes per bin.  Lane q of a
//   quad holds g-points 2q and 2q + 1: it interpolates every absorber there (FP32
//   table entries relative to per-(absorber, column) offsets, bilinear in (T, log p),
//   exp2 with the layer prefactor) and, in a merge, holds rows 2q and 2q + 1 of the
//   8 x 8 pair matrix, each mixture point with every absorber point, which ascend
//   because both distributions do.  The 64 pair sums are sorted by three merge levels:
//   the lane's two rows (an odd-even merge of registers), then two lanes, then the quad
//   (bitonic, quad_perm moves between lanes); keys = the value's bits above the low
//   six, a code of the pair in the low six.  The exact sums and weights are looked up by
//   code, their running sums (weights U, weights x values I, FP64) go to LDS in sorted
//   order, and each lane finds its two g-interval edges there by bisection: the integral
//   of the sorted distribution up to an edge E inside element r is I_r + v_r (E - U_r).
//   Output: the mixed layer optical depths [B][L_pad][n_bins_pad x 8] (FP32), read by
//   k_ck_trans (bf16x3 MFMA chord, as the cross-section path) or k_ck_emis (one lane per
//   (bin, g-point) column sweeping up the layers).
#include "ck.h"
#include "emission.h"
#include "kernels.h"
#include "opacity.h"

namespace exofwd {

// two adjacent FP32 table entries (8 bytes) through a buffer resource
__device__ inline float2 load_f32x2(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0);
  return make_float2(__uint_as_float(v[0]), __uint_as_float(v[1]));
}

// DPP lane moves inside a quad (gfx9 quad_perm encodings)
constexpr int kDppXor1 = 0xB1;         // [1,0,3,2]
constexpr int kDppQuadMirror = 0x1B;   // [3,2,1,0]
constexpr int kDppQuadPrev = 0x90;     // [0,0,1,2]
constexpr int dpp_quad_lane(int j) { return j * 0x55; }   // lane j of the quad to all four

// the smaller of a and b for z = 0, the larger for z = ~0 (one v_med3_u32)
__device__ inline uint32_t pick(uint32_t a, uint32_t b, uint32_t z) { return max(min(a, b), min(max(a, b), z)); }

// One cross-lane step of the sorting network: register r meets the partner lane's
// register r (or 15 - r with REV); the lane with z = 0 keeps the smaller key.
template <int CTRL, bool REV>
__device__ inline void net_cross(uint32_t (&k)[16], uint32_t z) {
  uint32_t o[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) o[r] = dpp_mov<CTRL>(k[REV ? 15 - r : r]);
#pragma unroll
  for (int r = 0; r < 16; ++r) k[r] = pick(k[r], o[r], z);
}
__device__ inline void order2(uint32_t& a, uint32_t& b) {
  const uint32_t lo = min(a, b), hi = max(a, b);
  a = lo;
  b = hi;
}
// half-cleaner inside a lane
template <int J>
__device__ inline void net_half(uint32_t (&k)[16]) {
#pragma unroll
  for (int r = 0; r < 16; ++r)
    if (!(r & J)) order2(k[r], k[r + J]);
}
// a lane's bitonic sequence of 16 sorted ascending
__device__ inline void net_local16(uint32_t (&k)[16]) {
  net_half<8>(k); net_half<4>(k); net_half<2>(k); net_half<1>(k);
}
// step of the odd-even merge of registers 0-7 with registers 8-15
template <int J>
__device__ inline void net_odd_even(uint32_t (&k)[16]) {
#pragma unroll
  for (int r = 0; r < 16; ++r)
    if ((r & J) && r + J < 16) order2(k[r], k[r + J]);
}

// Sort the 64 keys of a quad, element 16 q + r on lane q, register r, when registers
// 0-7 and registers 8-15 of every lane already ascend.  z1 / z2: ~0 where bit 0 / bit 1
// of q is set, else 0.
__device__ inline void sort_quad64(uint32_t (&k)[16], uint32_t z1, uint32_t z2) {
  // runs of 16: the lane's two rows (odd-even merge, 25 exchanges)
  net_half<8>(k); net_odd_even<4>(k); net_odd_even<2>(k); net_odd_even<1>(k);
  // runs of 32: lanes q, q ^ 1, mirrored
  net_cross<kDppXor1, true>(k, z1);
  net_local16(k);
  // runs of 64: the quad mirrored, then q ^ 1
  net_cross<kDppQuadMirror, true>(k, z2);
  net_cross<kDppXor1, false>(k, z1);
  net_local16(k);
}

// orders this wave's LDS accesses (its other lanes' data): LDS serves a wave in order,
// so only the compiler has to keep the order
__device__ inline void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Bound by the vector unit and the LDS together (88 % and 84 % of their cycles busy at
// 256 samples x 100 layers x 2485 bins x 8 absorbers, 29.4 ms; eight lanes per bin with
// every element's overlap with every interval took 50.8 ms: 670 vector instructions per
// merge of eight bins, now 270).  Four waves per SIMD: 116 registers, 36 KB per block.
//
// LDS of one wave, used in turn for the pair sums, the running weights, the running
// integrals and the sorted values of its 16 bins.  The kernel keeps the LDS as busy as
// the vector unit, so each layout keeps a lane off its neighbours' banks:
//   pair sums: the pair of code c of bin g at float 8 c + g % 8 (+ 512 for the upper
//     eight bins), so a bin's lookups, at four random codes at a time, stay in its own
//     eight banks; the code of register r on lane q is r ^ 18 q (row c / 8, and the
//     column xor 2 q), so the four lanes of a quad store to different banks;
//   running sums: slot n of bin g at double kCkInter n + g % kCkInter (the bins in groups
//     of kCkInter); sorted element 16 q + r in slot 4 r + q, so the stores fill the
//     banks; slots 64-67 hold the sums in front of each lane.
// The pair weights are kept in kCkInter copies, bin g reading copy g % kCkInter.
constexpr int kCkSlots = 68;
constexpr int kCkInter = 4;

template <int S, bool CIA>
__global__ __launch_bounds__(kBlock) void k_ck_mix(Model m, Work w, Tables tb, int B) {
  __shared__ double s_bin[kBlock / 64][kCkBinsPerWave * kCkSlots];
  __shared__ double s_wpair[64 * kCkInter];   // the pair weights by code
  for (int i = threadIdx.x; i < 64 * kCkInter; i += kBlock) {
    const int c = i / kCkInter, row = c >> 3;
    s_wpair[i] = ck_pair_weight(tb.ckwd[row], tb.ckwd[(c & 7) ^ (row & 6)]);
  }
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int b = blockIdx.z, l = blockIdx.y;
  const int j0 = (blockIdx.x * (kBlock / 64) + wv) * kCkBinsPerWave;
  if (j0 >= m.n_nu || w.status[b] || l >= w.nlay[b]) return;
  const int Lp = m.L_pad;
  constexpr int RL = rec_len(S);
  const float* rl = reinterpret_cast<const float*>(w.rec) + ((size_t)b * Lp + l) * RL;
  const int cl = w.cells[(size_t)b * Lp + l];
  const int it = cl & 255, ip = (cl >> 8) & 255, itc = cl >> 16;
  const float wt = rl[0], wp = rl[1], wtc = rl[2], ray = rl[3], deck = rl[4];
  const float w11 = wt * wp, w10 = wt - w11, w01 = wp - w11, w00 = 1.0f - wt - wp + w11;
  const size_t npad = (size_t)m.n_nu_pad, ncol = npad * kCkG;
  const uint32_t row_bytes = (uint32_t)ncol * 4u, tstep = (uint32_t)m.n_p * row_bytes;
  const __amdgpu_buffer_rsrc_t rh = make_rsrc(tb.h, (size_t)S * m.n_t * m.n_p * ncol * 4);
  const __amdgpu_buffer_rsrc_t rhc = make_rsrc(CIA ? (const void*)tb.hc : (const void*)tb.h,
                                               CIA ? (size_t)2 * m.n_tc * npad * 4 : 0);
  // lane q of quad grp: g-points 2q, 2q + 1 of bin j0 + grp
  const int grp = lane >> 2, q = lane & 3;
  const bool real = j0 + grp < m.n_nu;
  const int j = real ? j0 + grp : m.n_nu - 1;   // a quad past the last bin repeats it and stores nothing
  const uint32_t col = (uint32_t)(j * kCkG + 2 * q), voff = col * 4u;
  float sp0[S], sp1[S];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const uint32_t row = (uint32_t)((s * m.n_t + it) * m.n_p + ip) * row_bytes;
    const float2 c = *reinterpret_cast<const float2*>(tb.c + (size_t)s * ncol + col);
    const float lam = rl[kRecFixed + s];
    const float2 t00 = load_f32x2(rh, voff, row), t10 = load_f32x2(rh, voff, row + tstep);
    const float2 t01 = load_f32x2(rh, voff, row + row_bytes), t11 = load_f32x2(rh, voff, row + tstep + row_bytes);
    float v0 = c.x + lam, v1 = c.y + lam;
    v0 = fmaf(w00, t00.x, v0);
    v1 = fmaf(w00, t00.y, v1);
    v0 = fmaf(w10, t10.x, v0);
    v1 = fmaf(w10, t10.y, v1);
    v0 = fmaf(w01, t01.x, v0);
    v1 = fmaf(w01, t01.y, v1);
    v0 = fmaf(w11, t11.x, v0);
    v1 = fmaf(w11, t11.y, v1);
    sp0[s] = exp2_fast(v0);
    sp1[s] = exp2_fast(v1);
  }
  const uint32_t z1 = (q & 1) ? ~0u : 0u, z2 = (q & 2) ? ~0u : 0u;
  const double g1 = q > 0 ? 1.0 : 0.0, g2 = q > 1 ? 1.0 : 0.0, g3 = q > 2 ? 1.0 : 0.0;
  const double e0 = tb.cke[2 * q], e1 = tb.cke[2 * q + 1];
  const double inv0 = 1.0 / tb.ckwd[2 * q], inv1 = 1.0 / tb.ckwd[2 * q + 1];
  float* pairs = reinterpret_cast<float*>(s_bin[wv]) + (grp & 7) + 512 * (grp >> 3);
  double* sums = s_bin[wv] + (grp % kCkInter) + kCkInter * kCkSlots * (grp / kCkInter);
  float* vals = reinterpret_cast<float*>(sums);   // the sorted values, in the low half of each slot
  const double* wpair = s_wpair + (grp & (kCkInter - 1));
  constexpr uint32_t kSlotB = 8 * kCkInter, kLaneB = kSlotB, kRegB = 4 * kSlotB, kTopB = 64 * kSlotB;
  auto sum_at = [&](uint32_t byte) { return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(sums) + byte); };
  auto val_at = [&](uint32_t byte) { return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(vals) + byte); };
  // codes of the registers: pair_code[j] + 8 i + k for register 8 i + 2 j + k
  uint32_t pair_code[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) pair_code[k] = (uint32_t)(16 * q + 2 * (k ^ q));
  // sum over the quad's lanes below this one
  auto quad_excl = [&](double t) {
    return fma(dpp_mov<dpp_quad_lane(0)>(t), g1, fma(dpp_mov<dpp_quad_lane(1)>(t), g2, dpp_mov<dpp_quad_lane(2)>(t) * g3));
  };

  float mix0 = sp0[0], mix1 = sp1[0];   // the running mixture: absorber 0 to start
#pragma unroll
  for (int s = 1; s < S; ++s) {
    // rows 2q and 2q + 1 of the pair matrix
    float v[16];
    {
      const float b0 = dpp_mov<dpp_quad_lane(0)>(sp0[s]), b1 = dpp_mov<dpp_quad_lane(0)>(sp1[s]);
      const float b2 = dpp_mov<dpp_quad_lane(1)>(sp0[s]), b3 = dpp_mov<dpp_quad_lane(1)>(sp1[s]);
      const float b4 = dpp_mov<dpp_quad_lane(2)>(sp0[s]), b5 = dpp_mov<dpp_quad_lane(2)>(sp1[s]);
      const float b6 = dpp_mov<dpp_quad_lane(3)>(sp0[s]), b7 = dpp_mov<dpp_quad_lane(3)>(sp1[s]);
      const float br[8] = {b0, b1, b2, b3, b4, b5, b6, b7};
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        v[r] = mix0 + br[r];
        v[8 + r] = mix1 + br[r];
      }
    }
    wave_lds_fence();   // the previous merge's lookups are done before the tables are rewritten
    uint32_t key[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const uint32_t c0 = pair_code[(r >> 1) & 3], ik = (uint32_t)((r & 8) | (r & 1));
      pairs[8 * c0 + 8 * ik] = v[r];
      // optical depths are >= 0, so the bit patterns order like the values; the low
      // six bits carry the pair's code (pairs within 64 ulp may swap: < 4e-6 relative)
      key[r] = ((__float_as_uint(v[r]) & ~63u) | c0) | ik;
    }
    wave_lds_fence();
    sort_quad64(key, z1, z2);
    // The running weight U in front of each sorted element (from the lane's first one),
    // in FP64: an interval edge often falls exactly on an element boundary (a negligible
    // absorber leaves the pairs in blocks of one mixture point, whose weights sum to the
    // edge), and there a rounding of the running weight would move a sliver of the next,
    // possibly far larger, value into the interval.  The pair weights are whole multiples
    // of 2^-52 and so are the edges, so every such sum and difference is exact.
    float vs[16];
    double ie[16], i_lane;   // the integral in front of each element, from the lane's first one
    {
      double wr[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const uint32_t code = key[r] & 63u;
        vs[r] = pairs[8 * code];
        wr[r] = wpair[kCkInter * code];
      }
      wave_lds_fence();
      double u = 0.0, isum = 0.0;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        sums[kCkInter * (4 * r + q)] = u;
        ie[r] = isum;
        u += wr[r];
        isum = fma((double)vs[r], wr[r], isum);
      }
      sums[kCkInter * (64 + q)] = quad_excl(u);
      i_lane = quad_excl(isum);
    }
    wave_lds_fence();
    // the element holding each edge, the last one whose U is at most the edge (U_0 = 0):
    // its lane, then its register (slots 4 r + lane)
    const uint32_t h0 = sum_at(kTopB + 2 * kLaneB) <= e0 ? 2 * kLaneB : 0u;
    const uint32_t h1 = sum_at(kTopB + 2 * kLaneB) <= e1 ? 2 * kLaneB : 0u;
    uint32_t a0 = h0 + (sum_at(kTopB + kLaneB + h0) <= e0 ? kLaneB : 0u);
    uint32_t a1 = h1 + (sum_at(kTopB + kLaneB + h1) <= e1 ? kLaneB : 0u);
    const uint32_t l0 = kTopB + a0, l1 = kTopB + a1;
    double x0 = e0 - sum_at(l0), x1 = e1 - sum_at(l1);
    auto probe = [&](uint32_t step) {
      const double u0 = sum_at(a0 + step), u1 = sum_at(a1 + step);
      a0 += u0 <= x0 ? step : 0u;
      a1 += u1 <= x1 ? step : 0u;
    };
    probe(8 * kRegB);
    probe(4 * kRegB);
    probe(2 * kRegB);
    probe(kRegB);
    x0 -= sum_at(a0);
    x1 -= sum_at(a1);
    wave_lds_fence();
#pragma unroll
    for (int r = 0; r < 16; ++r) sums[kCkInter * (4 * r + q)] = ie[r];
    sums[kCkInter * (64 + q)] = i_lane;
    wave_lds_fence();
    double f0 = sum_at(l0) + sum_at(a0), f1 = sum_at(l1) + sum_at(a1);
    wave_lds_fence();
#pragma unroll
    for (int r = 0; r < 16; ++r) vals[2 * kCkInter * (4 * r + q)] = vs[r];
    wave_lds_fence();
    f0 = fma((double)val_at(a0), x0, f0);
    f1 = fma((double)val_at(a1), x1, f1);
    // interval 2q starts at the previous lane's second edge
    const double fp = dpp_mov<kDppQuadPrev>(f1);
    mix0 = (float)((f0 - (q > 0 ? fp : 0.0)) * inv0);
    mix1 = (float)((f1 - f0) * inv1);
  }
  // grey continuum at the bin centre: deck, Rayleigh and the two CIA pairs
  float dc = fmaf(ray, tb.nu4f[j], deck);
  if (CIA) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const uint32_t rowc = (uint32_t)(p * m.n_tc + itc) * (uint32_t)npad * 4u;
      const uint32_t vo = (uint32_t)j * 4u;
      float v = tb.cc[(size_t)p * npad + j] + rl[5 + p];
      v = fmaf(1.0f - wtc, load_f32(rhc, vo, rowc), v);
      v = fmaf(wtc, load_f32(rhc, vo, rowc + (uint32_t)npad * 4u), v);
      dc += exp2_fast(v);
    }
  }
  if (real)   // read once, by the spectrum kernel
    __builtin_nontemporal_store((float2v){mix0 + dc, mix1 + dc},
                                reinterpret_cast<float2v*>(w.ckmix + ((size_t)b * Lp + l) * ncol + col));
}

// Transmission: per (sample, 128-column tile) the chord tau = P dtau on MFMA
// (bf16 hi/lo split of both operands, as the cross-section kernel), the transit
// depth of every (bin, g-point) column and the g-weighted sum per bin.
__global__ __launch_bounds__(kBlockT) void k_ck_trans(Model m, Work w, Tables tb, int B, float* __restrict__ spec) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int n_ct = m.n_tiles * kCkG;   // 128-column tiles per sample
  const int logical = xcd_logical_block(blockIdx.x, gridDim.x);
  const int b = logical / n_ct, tile = logical % n_ct;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int Lp = m.L_pad;
  const int c0 = tile * kTileNu;          // first column; bins c0/8 .. c0/8 + 15
  const int j0 = c0 / kCkG;
  float* out = spec + (size_t)b * m.n_nu;
  if (w.status[b]) {
    if (tid < kTileNu / kCkG && j0 + tid < m.n_nu) out[j0 + tid] = __builtin_nanf("");
    return;
  }
  const int L = w.nlay[b];
  const size_t ncol = (size_t)m.n_nu_pad * kCkG;
  const int stride = Lp + 8;
  uint16_t* s_bhi = reinterpret_cast<uint16_t*>(lds);
  uint16_t* s_blo = s_bhi + kTileNu * stride;
  float* s_area = reinterpret_cast<float*>(s_blo + kTileNu * stride);
  float* s_red = s_area + Lp;   // [8][32]
  const float* area = reinterpret_cast<const float*>(w.area) + (size_t)b * Lp;
  for (int i = tid; i < Lp; i += kBlockT) s_area[i] = area[i];

  // phase A: the mixed layer optical depths of the tile -> bf16 hi/lo B operand in LDS
  const float* src = w.ckmix + (size_t)b * Lp * ncol + c0 + 2 * lane;
  const bool real = (c0 + 2 * lane) / kCkG < m.n_nu;   // columns of padding bins hold nothing
  const int KBe = (L + 15) >> 4;
  for (int o = wv; o < 2 * KBe; o += kBlockT / 64) {
    float e0[8], e1[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int l = 8 * o + q;
      float2 d = make_float2(0.0f, 0.0f);
      if (l < L && real) {
        const float2v v = __builtin_nontemporal_load(reinterpret_cast<const float2v*>(src + (size_t)l * ncol));
        d = make_float2(v.x, v.y);
      }
      e0[q] = fminf(d.x, 16384.0f);
      e1[q] = fminf(d.y, 16384.0f);
    }
    uint32_t h0[4], l0[4], h1[4], l1[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      split_pair(e0[2 * q], e0[2 * q + 1], h0[q], l0[q]);
      split_pair(e1[2 * q], e1[2 * q + 1], h1[q], l1[q]);
    }
    const int r0 = (2 * lane) * stride + 8 * o, r1 = r0 + stride;
    *reinterpret_cast<uint4*>(s_bhi + r0) = make_uint4(h0[0], h0[1], h0[2], h0[3]);
    *reinterpret_cast<uint4*>(s_blo + r0) = make_uint4(l0[0], l0[1], l0[2], l0[3]);
    *reinterpret_cast<uint4*>(s_bhi + r1) = make_uint4(h1[0], h1[1], h1[2], h1[3]);
    *reinterpret_cast<uint4*>(s_blo + r1) = make_uint4(l1[0], l1[1], l1[2], l1[3]);
  }
  __syncthreads();

  // phase B: tau = P dtau; wave wv owns 32-column block (wv & 3) and half (wv >> 2) of the row blocks
  const int MBe = (L + 31) >> 5;
  const int KB = Lp >> 4;
  const int nb = wv & 3;
  const size_t plane = (size_t)(Lp >> 5) * KB * 512;
  const uint16_t* fh = w.pfrag + (size_t)b * 2 * plane;
  const uint16_t* fl = fh + plane;
  const int col = 32 * nb + (lane & 31);
  const int khalf = 8 * (lane >> 5);
  float dsum = 0.0f;
  for (int mi = (wv >> 2); mi < MBe; mi += 2) {
    f32x16 acc = {};
    for (int kb = 2 * mi; kb < KBe; ++kb) {
      const size_t fo = ((size_t)(mi * KB + kb) * 64 + lane) * 8;
      const bf16x8 ah = *reinterpret_cast<const bf16x8*>(fh + fo);
      const bf16x8 al = *reinterpret_cast<const bf16x8*>(fl + fo);
      const bf16x8 bh = *reinterpret_cast<const bf16x8*>(s_bhi + col * stride + 16 * kb + khalf);
      const bf16x8 bl = *reinterpret_cast<const bf16x8*>(s_blo + col * stride + 16 * kb + khalf);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh, acc, 0, 0, 0);
    }
    // phase C: annulus-weighted absorption of each column's chords
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int r = 32 * mi + 8 * (q >> 2) + 4 * (lane >> 5) + (q & 3);
      dsum = fmaf(s_area[r], one_minus_exp(acc[q], exp2_fast(-1.4426950408889634f * acc[q])), dsum);
    }
  }
  dsum += __shfl_xor(dsum, 32);
  if (lane < 32) s_red[wv * 32 + lane] = dsum;
  __syncthreads();
  if (tid < kTileNu) {
    // column tid = bin tid/8, g-point tid%8: weighted, then summed over the bin's eight columns
    const int h = tid >> 5, c = tid & 31;
    float v = (float)w.core[b] + s_red[h * 32 + c] + s_red[(h + 4) * 32 + c];
    v *= tb.ckw[tid & (kCkG - 1)];
    v += __shfl_xor(v, 1);
    v += __shfl_xor(v, 2);
    v += __shfl_xor(v, 4);
    const int j = j0 + (tid >> 3);
    if ((tid & (kCkG - 1)) == 0 && j < m.n_nu) out[j] = v;
  }
}

// Transmission with random overlap along each chord (the product of the absorbers'
// transmission functions): a tile of 16 bins x 8 g-points (128 columns) runs one
// pass per absorber; absorber 0's columns also carry the grey continuum (exact: the
// chord is linear, so its factor e^-tau_c multiplies absorber 0's g-sum).  Per chord
// row the absorption of absorber s is A_s = sum_g w_g (1 - e^-tau_s,g), and the
// passes combine it as A (+) A_s = A + A_s - A A_s (= 1 - (1 - A)(1 - A_s), without
// the cancellation of a thin chord's 1 - product of transmissions), kept in the
// registers of the lanes that own the rows.  One absorber per pass keeps a wave's table
// loads on 16 contiguous bins of one table row.  Bound by vector work and the latency of
// its barrier-separated phases at two workgroups per CU (LDS).  256 samples x 2179 bins x
// 6 absorbers x 100 layers: 8.5 -> 4.1 ms (every layer fetched its entries again, 48 LDS
// permutes and 16 read-modify-writes per 32-row block formed and kept the g-sums, and the
// layer records came by vector loads).
constexpr int kProdBins = kTileNu / kCkG;   // bins per tile

template <int S, bool CIA>
__global__ __launch_bounds__(kBlockT) void k_ck_trans_prod(Model m, Work w, Tables tb, int B,
                                                           float* __restrict__ spec) {
  constexpr int kSlots = 3;   // row blocks of a wave: five row blocks in two halves
  extern __shared__ __align__(16) unsigned char lds[];
  const int n_bt = (m.n_nu + kProdBins - 1) / kProdBins;   // bin tiles per sample
  const int logical = xcd_logical_block(blockIdx.x, gridDim.x);
  const int b = logical / n_bt, tile = logical % n_bt;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int Lp = m.L_pad;
  const int j0 = kProdBins * tile;
  float* out = spec + (size_t)b * m.n_nu;
  if (w.status[b]) {
    if (tid < kProdBins && j0 + tid < m.n_nu) out[j0 + tid] = __builtin_nanf("");
    return;
  }
  const int L = w.nlay[b];
  const int stride = Lp + 8;
  uint16_t* s_bhi = reinterpret_cast<uint16_t*>(lds);
  uint16_t* s_blo = s_bhi + kTileNu * stride;
  float* s_area = reinterpret_cast<float*>(s_blo + kTileNu * stride);
  float* s_abs = s_area + Lp;   // [kProdBins][Lp]: combined absorption per bin and chord row, after the last pass
  const float* area = reinterpret_cast<const float*>(w.area) + (size_t)b * Lp;
  for (int i = tid; i < Lp; i += kBlockT) s_area[i] = area[i];

  // this lane's two columns: bin jj of the tile, g-points g and g + 1
  const int c2 = 2 * lane, jj = c2 >> 3, g = c2 & 7;
  const bool real = j0 + jj < m.n_nu;   // columns of bins past the last hold nothing
  const int j = real ? j0 + jj : m.n_nu - 1;
  const size_t npad = (size_t)m.n_nu_pad, ncol = npad * kCkG;
  const uint32_t row_bytes = (uint32_t)ncol * 4u, tstep = (uint32_t)m.n_p * row_bytes;
  const __amdgpu_buffer_rsrc_t rh = make_rsrc(tb.h, (size_t)S * m.n_t * m.n_p * ncol * 4);
  const __amdgpu_buffer_rsrc_t rhc = make_rsrc(CIA ? (const void*)tb.hc : (const void*)tb.h,
                                               CIA ? (size_t)2 * m.n_tc * npad * 4 : 0);
  const uint32_t col = (uint32_t)(j * kCkG + g), vo = col * 4u;
  const float nu4 = tb.nu4f[j];
  float cc[2] = {0.0f, 0.0f};
  if (CIA) {
    cc[0] = tb.cc[j];
    cc[1] = tb.cc[npad + j];
  }
  constexpr int RL = rec_len(S);
  const auto rec = const_ptr(reinterpret_cast<const float*>(w.rec)) + (size_t)b * Lp * RL;
  const auto cells = const_ptr(w.cells) + (size_t)b * Lp;
  const int KBe = (L + 15) >> 4, MBe = (L + 31) >> 5, KB = Lp >> 4;
  const int nb = wv & 3;
  const size_t plane = (size_t)(Lp >> 5) * KB * 512;
  // this sample's P fragments (hi plane, then lo plane), as in the cross-section kernel
  const __amdgpu_buffer_rsrc_t rs_f = make_rsrc(w.pfrag + (size_t)b * 2 * plane, 2 * plane * 2);
  const uint32_t lo_plane = (uint32_t)plane * 2u, voff_f = (uint32_t)lane * 16u;
  const int ccol = 32 * nb + (lane & 31);
  const int khalf = 8 * (lane >> 5);
  const float wg_even = tb.ckw[lane & 6], wg_odd = (lane & 1) ? tb.ckw[lane & 7] : 1.0f;
  const int bin_c = 4 * nb + ((lane & 31) >> 3);   // the tile bin of this lane's MFMA column
  // row blocks of this wave, cost-balanced between the two waves of a column block
  int slot_mi[kSlots];
  {
    const unsigned mine = split_blocks32(wv >> 2, MBe, KBe);
    int n = 0;
    for (int mi = 0; mi < MBe; ++mi)
      if ((mine & (1u << mi)) && n < kSlots) slot_mi[n++] = mi;
    for (; n < kSlots; ++n) slot_mi[n] = -1;
  }
  // combined absorption of the passes so far, of two rows of each block per lane: rows
  // q = 2 k + {0, 1} of the 16 MFMA rows, k from the lane's place among its bin's eight
  float comb[kSlots][2];
  const bool k1 = lane & 1, k2 = lane & 2, k4 = lane & 4;

#pragma unroll 1
  for (int s = 0; s < S; ++s) {
    // phase A: absorber s's optical depth of every layer at the tile's columns -> bf16
    // hi/lo B operand in LDS
    const float2 cof = *reinterpret_cast<const float2*>(tb.c + (size_t)s * ncol + col);
    // a contiguous run of layer octets per wave; a layer in the cell of the one before it
    // reuses its table entries
    float2 t00, t10, t01, t11;
    float ca[2], cb[2];
    int cell_prev = -1;
    for (int o = 2 * KBe * wv / (kBlockT / 64); o < 2 * KBe * (wv + 1) / (kBlockT / 64); ++o) {
      float e0[8], e1[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int l = 8 * o + q;
        float d0 = 0.0f, d1 = 0.0f;
        if (l < L) {
          const auto rl = rec + (size_t)l * RL;
          const int cl = cells[l];
          if (cl != cell_prev) {
            const int it = cl & 255, ip = (cl >> 8) & 255, itc = cl >> 16;
            const uint32_t row = (uint32_t)((s * m.n_t + it) * m.n_p + ip) * row_bytes;
            t00 = load_f32x2(rh, vo, row);
            t10 = load_f32x2(rh, vo, row + tstep);
            t01 = load_f32x2(rh, vo, row + row_bytes);
            t11 = load_f32x2(rh, vo, row + tstep + row_bytes);
            if (CIA && s == 0) {
#pragma unroll
              for (int p = 0; p < 2; ++p) {
                const uint32_t rowc = (uint32_t)(p * m.n_tc + itc) * (uint32_t)npad * 4u;
                ca[p] = load_f32(rhc, (uint32_t)j * 4u, rowc);
                cb[p] = load_f32(rhc, (uint32_t)j * 4u, rowc + (uint32_t)npad * 4u);
              }
            }
            cell_prev = cl;
          }
          const float wt = rl[0], wp = rl[1];
          const float w11 = wt * wp, w10 = wt - w11, w01 = wp - w11, w00 = 1.0f - wt - wp + w11;
          const float lam = rl[kRecFixed + s];
          float v0 = cof.x + lam, v1 = cof.y + lam;
          v0 = fmaf(w00, t00.x, v0);
          v1 = fmaf(w00, t00.y, v1);
          v0 = fmaf(w10, t10.x, v0);
          v1 = fmaf(w10, t10.y, v1);
          v0 = fmaf(w01, t01.x, v0);
          v1 = fmaf(w01, t01.y, v1);
          v0 = fmaf(w11, t11.x, v0);
          v1 = fmaf(w11, t11.y, v1);
          d0 = exp2_fast(v0);
          d1 = exp2_fast(v1);
          if (s == 0) {
            // the grey continuum at the bin centre rides on absorber 0
            float dc = fmaf(rl[3], nu4, rl[4]);
            if (CIA) {
              const float wtc = rl[2];
#pragma unroll
              for (int p = 0; p < 2; ++p) {
                float v = cc[p] + rl[5 + p];
                v = fmaf(1.0f - wtc, ca[p], v);
                v = fmaf(wtc, cb[p], v);
                dc += exp2_fast(v);
              }
            }
            d0 += dc;
            d1 += dc;
          }
          if (!real) d0 = d1 = 0.0f;
        }
        e0[q] = fminf(d0, 16384.0f);
        e1[q] = fminf(d1, 16384.0f);
      }
      uint32_t h0[4], l0[4], h1[4], l1[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        split_pair(e0[2 * q], e0[2 * q + 1], h0[q], l0[q]);
        split_pair(e1[2 * q], e1[2 * q + 1], h1[q], l1[q]);
      }
      const int r0 = c2 * stride + 8 * o, r1 = r0 + stride;
      *reinterpret_cast<uint4*>(s_bhi + r0) = make_uint4(h0[0], h0[1], h0[2], h0[3]);
      *reinterpret_cast<uint4*>(s_blo + r0) = make_uint4(l0[0], l0[1], l0[2], l0[3]);
      *reinterpret_cast<uint4*>(s_bhi + r1) = make_uint4(h1[0], h1[1], h1[2], h1[3]);
      *reinterpret_cast<uint4*>(s_blo + r1) = make_uint4(l1[0], l1[1], l1[2], l1[3]);
    }
    __syncthreads();

    // phase B: tau = P dtau over this wave's row blocks
#pragma unroll
    for (int q2 = 0; q2 < kSlots; ++q2) {
      const int mi = slot_mi[q2];
      if (mi < 0) continue;
      f32x16 acc = {};
      // fragments in two groups of two K blocks, one group in flight (blocks past KBe read
      // the next row block's, or zeros past the range, and are never used)
      bf16x8 ga[2][2], gb[2][2];
      auto load = [&](bf16x8 (&gr)[2][2], int k) {
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int y = 0; y < 2; ++y)
            gr[x][y] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(
                                                      rs_f, voff_f, (uint32_t)(mi * KB + k + x) * 1024u + (y ? lo_plane : 0u), 0));
      };
      auto product = [&](const bf16x8 (&gr)[2][2], int k0) {
#pragma unroll
        for (int x = 0; x < 2; ++x) {
          const int kb = k0 + x;
          if (kb >= KBe) break;
          const bf16x8 bh = *reinterpret_cast<const bf16x8*>(s_bhi + ccol * stride + 16 * kb + khalf);
          const bf16x8 bl = *reinterpret_cast<const bf16x8*>(s_blo + ccol * stride + 16 * kb + khalf);
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(gr[x][1], bh, acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(gr[x][0], bl, acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(gr[x][0], bh, acc, 0, 0, 0);
        }
      };
      load(ga, 2 * mi);
#pragma unroll 1
      for (int kb = 2 * mi; kb < KBe; kb += 4) {
        load(gb, kb + 2);
        product(ga, kb);
        if (kb + 2 >= KBe) break;
        load(ga, kb + 4);
        product(gb, kb + 2);
      }
      // phase C: per row, absorber s's g-weighted absorption in its bin: the 16 rows summed
      // over the bin's eight lanes by halving exchanges (lane ^ 1, 2, 4), so each lane ends
      // with two rows, which it combines into the bin's running absorption
      // (a pair of lanes adds w x of the even g-point, fused, to the rounded w x of the odd)
      float a[16], h8[8], h4[4];
#pragma unroll
      for (int q = 0; q < 16; ++q) a[q] = wg_odd * one_minus_exp(acc[q], exp2_fast(-1.4426950408889634f * acc[q]));
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const float keep = k1 ? a[q + 8] : a[q], recv = lane_xor<1>(k1 ? a[q] : a[q + 8]);
        h8[q] = fmaf(wg_even, k1 ? recv : keep, k1 ? keep : recv);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) h4[q] = (k2 ? h8[q + 4] : h8[q]) + lane_xor<2>(k2 ? h8[q] : h8[q + 4]);
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const float av = (k4 ? h4[q + 2] : h4[q]) + lane_xor<4>(k4 ? h4[q] : h4[q + 2]);
        const float prev = s == 0 ? 0.0f : comb[q2][q];
        comb[q2][q] = fmaf(-prev, av, prev + av);
      }
    }
    __syncthreads();   // the next pass overwrites the B operand
  }
  // MFMA row q of block mi is row 32 mi + 8 (q / 4) + 4 (lane / 32) + q % 4
  {
    const int q0 = (k1 ? 8 : 0) + (k2 ? 4 : 0) + (k4 ? 2 : 0);
#pragma unroll
    for (int q2 = 0; q2 < kSlots; ++q2) {
      if (slot_mi[q2] < 0) continue;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int r = 32 * slot_mi[q2] + 8 * (q0 >> 2) + 4 * (lane >> 5) + ((q0 & 3) + q);
        s_abs[bin_c * Lp + r] = comb[q2][q];
      }
    }
  }
  __syncthreads();
  // the bins' combined absorption, annulus-weighted and summed over the rows: 32
  // threads per bin
  const int bj = tid >> 5;
  float v = 0.0f;
  for (int i = tid & 31; i < 32 * MBe; i += 32) v = fmaf(s_area[i], s_abs[bj * Lp + i], v);
#pragma unroll
  for (int off = 16; off > 0; off >>= 1) v += __shfl_xor(v, off);
  if ((tid & 31) == 0 && j0 + bj < m.n_nu) out[j0 + bj] = (float)w.core[b] + v;
}

// Emission: one lane per (bin, g-point) column, sweeping up the layers with the
// linear-in-tau source at the bin centre's Planck intensity (FP64 intensities, as
// the cross-section kernel), then the g-weighted flux per bin and F_p / F_*.
__global__ __launch_bounds__(kBlock) void k_ck_emis(Model m, Work w, Tables tb, int B, float* __restrict__ spec) {
  const int n_ct = m.n_tiles64 * kCkG;   // 64-column tiles per sample
  const int logical = xcd_logical_block(blockIdx.x, gridDim.x);
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int gw = logical * (kBlock / 64) + wv;
  const int b = gw / n_ct, tile = gw % n_ct;
  if (b >= B) return;
  const int colx = tile * kTile64 + lane, j = colx / kCkG;
  float* out = spec + (size_t)b * m.n_nu;
  if (w.status[b]) {
    if ((lane & (kCkG - 1)) == 0 && j < m.n_nu) out[j] = __builtin_nanf("");
    return;
  }
  const int L = w.nlay[b], Lp = m.L_pad;
  const size_t ncol = (size_t)m.n_nu_pad * kCkG;
  const float* dt = w.ckmix + (size_t)b * Lp * ncol + colx;
  const double* t_lev = w.t_lev + (size_t)b * (Lp + 1);
  const double* inv_t = w.inv_tlev + (size_t)b * (Lp + 1);
  const double nud = m.nu[j];
  const float c1n3 = (float)(2.0 * kHpl * kC * kC * nud * nud * nud);
  const double c2n_log2e = kHpl * kC / kB * 1.4426950408889634074 * nud;
  auto planck_at = [&](int lv) {
    float y, em1;
    return planck_split(c1n3, c2n_log2e, inv_t[lv], y, em1);
  };
  const int n_mu = m.n_mu;
  float inv_mu[kMaxMu];
  double inten[kMaxMu];
  float b_bot = planck_at(0);
#pragma unroll
  for (int k = 0; k < kMaxMu; ++k) {
    inv_mu[k] = k < n_mu ? (float)(1.0 / m.mu_nodes[k]) : 0.0f;
    inten[k] = b_bot;
  }
  const bool real = j < m.n_nu;   // columns of padding bins hold nothing
  for (int l = 0; l < L; ++l) {
    const float d = real ? __builtin_nontemporal_load(&dt[(size_t)l * ncol]) : 0.0f;
    const float b_top = planck_at(l + 1);
    const float db = b_bot - b_top;
#pragma unroll
    for (int k = 0; k < kMaxMu; ++k) {
      if (k >= n_mu) break;
      const float x = d * inv_mu[k];
      const float e = exp2_fast(-1.4426950408889634f * x);
      float om, src;
      slab_terms(x, e, om, src);
      inten[k] = fma((double)om, (double)b_top - inten[k], fma((double)db, (double)src, inten[k]));
    }
    b_bot = b_top;
  }
  double flux = 0.0;
#pragma unroll
  for (int k = 0; k < kMaxMu; ++k)
    if (k < n_mu) flux = fma(2.0 * M_PI * m.mu_weights[k] * m.mu_nodes[k], inten[k], flux);
  flux *= (double)tb.ckw[lane & (kCkG - 1)];
  flux += __shfl_xor(flux, 1);
  flux += __shfl_xor(flux, 2);
  flux += __shfl_xor(flux, 4);
  if ((lane & (kCkG - 1)) == 0 && j < m.n_nu) {
    const double fstar = M_PI * 2.0 * kHpl * kC * kC * nud * nud * nud / expm1(kHpl * kC * nud / (kB * m.t_star));
    out[j] = (float)(m.dilution * flux / fstar * w.core[b]);
  }
}

// ---------------------------------------------------------------------------
template <int S, bool CIA>
const void* ck_mix_kernel() { return (const void*)k_ck_mix<S, CIA>; }

static const void* ck_mix_kernel_for(int S, bool cia) {
#define EXOFWD_CASE(n) \
  case n: return cia ? ck_mix_kernel<n, true>() : ck_mix_kernel<n, false>();
  switch (S) {
    EXOFWD_CASE(1) EXOFWD_CASE(2) EXOFWD_CASE(3) EXOFWD_CASE(4)
    EXOFWD_CASE(5) EXOFWD_CASE(6) EXOFWD_CASE(7) EXOFWD_CASE(8)
  }
#undef EXOFWD_CASE
  return nullptr;
}

template <int S, bool CIA>
const void* ck_prod_kernel() { return (const void*)k_ck_trans_prod<S, CIA>; }

static const void* ck_prod_kernel_for(int S, bool cia) {
#define EXOFWD_CASE(n) \
  case n: return cia ? ck_prod_kernel<n, true>() : ck_prod_kernel<n, false>();
  switch (S) {
    EXOFWD_CASE(1) EXOFWD_CASE(2) EXOFWD_CASE(3) EXOFWD_CASE(4)
    EXOFWD_CASE(5) EXOFWD_CASE(6) EXOFWD_CASE(7) EXOFWD_CASE(8)
  }
#undef EXOFWD_CASE
  return nullptr;
}

static size_t ck_trans_lds_bytes(const Model& m) {
  return (size_t)2 * kTileNu * (m.L_pad + 8) * 2 + (size_t)m.L_pad * 4 + 8 * 32 * 4;
}
static size_t ck_prod_lds_bytes(const Model& m) {
  return (size_t)2 * kTileNu * (m.L_pad + 8) * 2 + (size_t)m.L_pad * 4 * (1 + kProdBins);
}

hipError_t ck_configure(const Model& m) {
  if (m.mode != kTransmission) return ck_mix_kernel_for(m.S, m.has_cia) ? hipSuccess : hipErrorInvalidValue;
  if (m.ck_mix == kCkProduct) {
    const void* k = ck_prod_kernel_for(m.S, m.has_cia);
    if (!k) return hipErrorInvalidValue;
    return hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)ck_prod_lds_bytes(m));
  }
  if (!ck_mix_kernel_for(m.S, m.has_cia)) return hipErrorInvalidValue;
  return hipFuncSetAttribute((const void*)k_ck_trans, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)ck_trans_lds_bytes(m));
}

void launch_ck_mix(const Model& m, const Work& w, const Tables& tb, int B, hipStream_t st) {
  if (m.ck_mix != kCkRorr) return;   // the product of transmissions mixes inside its chord kernel
  const unsigned gx = (unsigned)((m.n_nu + kCkBinsPerWave * (kBlock / 64) - 1) / (kCkBinsPerWave * (kBlock / 64)));
  void* args[] = {(void*)&m, (void*)&w, (void*)&tb, (void*)&B};
  hipLaunchKernel(ck_mix_kernel_for(m.S, m.has_cia), dim3(gx, (unsigned)m.L_max, (unsigned)B), dim3(kBlock), args, 0,
                  st);
}

void launch_ck_spectrum(const Model& m, const Work& w, const Tables& tb, int B, void* spec, hipStream_t st) {
  if (m.ck_mix == kCkProduct) {
    void* args[] = {(void*)&m, (void*)&w, (void*)&tb, (void*)&B, (void*)&spec};
    hipLaunchKernel(ck_prod_kernel_for(m.S, m.has_cia),
                    dim3((unsigned)(B * ((m.n_nu + kProdBins - 1) / kProdBins))), dim3(kBlockT), args,
                    ck_prod_lds_bytes(m), st);
    return;
  }
  if (m.mode == kTransmission) {
    hipLaunchKernelGGL(k_ck_trans, dim3((unsigned)(B * m.n_tiles * kCkG)), dim3(kBlockT), ck_trans_lds_bytes(m), st, m,
                       w, tb, B, (float*)spec);
  } else {
    const int waves = B * m.n_tiles64 * kCkG;
    hipLaunchKernelGGL(k_ck_emis, dim3((unsigned)((waves + kBlock / 64 - 1) / (kBlock / 64))), dim3(kBlock), 0, st, m,
                       w, tb, B, (float*)spec);
  }
}

}  // namespace exofwd
