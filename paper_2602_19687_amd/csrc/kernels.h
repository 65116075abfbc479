// Launch entry points of the gfx950 kernels (host side of each .hip file).
#pragma once
#include "common.h"

namespace exofwd {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;

// block id -> logical id such that consecutive logical ids share an XCD
// (the dispatcher deals workgroups round-robin over the 8 XCDs)
__device__ inline int xcd_logical_block(int bid, int nblk) {
  if ((nblk & 7) != 0) return bid;
  return (bid & 7) * (nblk >> 3) + (bid >> 3);
}

// Position in a layer-count class's sample list of sample slot s of a launch whose
// logical blocks (xcd_logical_block over n_slots * per_slot blocks) give each XCD a
// contiguous run of n_slots / 8 slots: the positions are dealt round the XCDs
// (slot s of XCD k holds position 8 (s - k n_slots / 8) + k), so a class that fills
// only part of the grid still spreads over every XCD, longest samples first on each.
__device__ inline int class_position(int s, int n_slots, int per_slot) {
  if ((n_slots & 7) != 0 || (((long)n_slots * per_slot) & 7) != 0) return s;
  const int spx = n_slots >> 3;
  return (s % spx) * 8 + s / spx;
}

// 32-row blocks of the path matrix of one of two waves that share a column block: each block
// in turn goes to the wave with the least cost so far; block mi costs its K extent KBe - 2 mi
__device__ inline unsigned split_blocks32(int part, int MBe, int KBe) {
  unsigned mine = 0;
  int c0 = 0, c1 = 0;
  for (int mi = 0; mi < MBe; ++mi) {
    const int cost = KBe - 2 * mi;
    if (c0 <= c1) {
      if (part == 0) mine |= 1u << mi;
      c0 += cost;
    } else {
      if (part == 1) mine |= 1u << mi;
      c1 += cost;
    }
  }
  return mine;
}

// ---- sums over a wave of 16 values per lane at once: the lanes of quad n (n = lane / 4) get
// the sum of v[n].  Halving exchanges: each step a lane passes on the half of its values
// that its partner keeps, so the 16 sums take about 40 instructions (FP32) where a
// butterfly takes 12 and six LDS accesses for each.  The sums have the butterfly's tree
// (lanes l ^ 32, then 16, 8, 4, 2, 1), bit for bit.
template <int CTRL>
__device__ inline uint32_t dpp_mov(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
__device__ inline float dpp_mov(float v) { return __uint_as_float(dpp_mov<CTRL>(__float_as_uint(v))); }
template <int CTRL>
__device__ inline double dpp_mov(double v) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint64_t lo = dpp_mov<CTRL>((uint32_t)u), hi = dpp_mov<CTRL>((uint32_t)(u >> 32));
  return __longlong_as_double((long long)(lo | (hi << 32)));
}
// the value of lane l ^ BIT (1, 2, 4 or 8)
template <int BIT>
__device__ inline uint32_t lane_xor(uint32_t v) {
  if constexpr (BIT == 1) return dpp_mov<0xB1>(v);         // quad_perm [1,0,3,2]
  else if constexpr (BIT == 2) return dpp_mov<0x4E>(v);    // quad_perm [2,3,0,1]
  else if constexpr (BIT == 8) return dpp_mov<0x128>(v);   // row_ror:8
  else {
    const int up = __builtin_amdgcn_update_dpp(0, (int)v, 0x104, 0xF, 0x5, true);      // row_shl:4, quads 0 and 2
    return (uint32_t)__builtin_amdgcn_update_dpp(up, (int)v, 0x114, 0xF, 0xA, true);   // row_shr:4, quads 1 and 3
  }
}
template <int BIT>
__device__ inline float lane_xor(float v) { return __uint_as_float(lane_xor<BIT>(__float_as_uint(v))); }
template <int BIT>
__device__ inline double lane_xor(double v) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint64_t lo = lane_xor<BIT>((uint32_t)u), hi = lane_xor<BIT>((uint32_t)(u >> 32));
  return __longlong_as_double((long long)(lo | (hi << 32)));
}
// x and y after the upper half of x and the lower half of y (BIT 32; BIT 16: the odd rows
// of x and the even rows of y) changed places
template <int BIT>
__device__ inline void lane_swap(uint32_t& x, uint32_t& y) {
  if constexpr (BIT == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
    x = r[0];
    y = r[1];
  } else {
    const auto r = __builtin_amdgcn_permlane16_swap(x, y, false, false);
    x = r[0];
    y = r[1];
  }
}
// lanes with bit BIT of the lane clear: a + a of lane ^ BIT; set: the same for b
template <int BIT>
__device__ inline float halve_add(float a, float b) {
  uint32_t x = __float_as_uint(a), y = __float_as_uint(b);
  lane_swap<BIT>(x, y);
  return __uint_as_float(x) + __uint_as_float(y);
}
template <int BIT>
__device__ inline double halve_add(double a, double b) {
  const uint64_t ua = (uint64_t)__double_as_longlong(a), ub = (uint64_t)__double_as_longlong(b);
  uint32_t xl = (uint32_t)ua, xh = (uint32_t)(ua >> 32), yl = (uint32_t)ub, yh = (uint32_t)(ub >> 32);
  lane_swap<BIT>(xl, yl);
  lane_swap<BIT>(xh, yh);
  return __longlong_as_double((long long)((uint64_t)xl | ((uint64_t)xh << 32))) +
         __longlong_as_double((long long)((uint64_t)yl | ((uint64_t)yh << 32)));
}
template <typename T>
__device__ inline T wave_sums16(const T (&v)[16], int lane) {
  T a[8], b[4], c[2];
#pragma unroll
  for (int i = 0; i < 8; ++i) a[i] = halve_add<32>(v[i], v[i + 8]);
#pragma unroll
  for (int i = 0; i < 4; ++i) b[i] = halve_add<16>(a[i], a[i + 4]);
  const bool k8 = lane & 8, k4 = lane & 4;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const T keep = k8 ? b[i + 2] : b[i], send = k8 ? b[i] : b[i + 2];
    c[i] = keep + lane_xor<8>(send);
  }
  const T keep = k4 ? c[1] : c[0], send = k4 ? c[0] : c[1];
  T r = keep + lane_xor<4>(send);
  r += lane_xor<2>(r);
  r += lane_xor<1>(r);
  return r;
}
// sum over the aligned groups of g = 8, 16, 32 or 64 lanes, every lane gets it (the same
// tree), by lane moves alone
template <typename T>
__device__ inline T group_sum_all(T v, int g) {
  if (g >= 64) v = halve_add<32>(v, v);
  if (g >= 32) v = halve_add<16>(v, v);
  if (g >= 16) v += lane_xor<8>(v);
  v += lane_xor<4>(v);
  v += lane_xor<2>(v);
  v += lane_xor<1>(v);
  return v;
}
template <typename T>
__device__ inline T wave_sum_all(T v) { return group_sum_all(v, 64); }

void launch_profile(const Model& m, const Work& w, int B, const double* params, const int32_t* n_layers,
                    bool fp64, hipStream_t st);
hipError_t profile_configure(const Model& m, bool fp64);
// dtau_out (reduced precision only, may be null): layer optical depths [B][L_pad][n_nu_pad] for the reverse pass
void launch_trans_fwd(const Model& m, const Work& w, const Tables& tb, int B, void* spec, bool fp64,
                      hipStream_t st, float* dtau_out = nullptr);
// B real samples; with the cloudy/clear mixing spec holds the 2B virtual spectra and the
// mixed spectrum goes to spec_out (may be null)
void launch_loglike(const Model& m, const Work& w, int B, const double* params, const void* spec, void* spec_out,
                    bool spec_f64, const int32_t* bin_lo, const int32_t* bin_hi, const double* y, const double* yerr,
                    const uint8_t* mask, double* lnl, int32_t* status_out, hipStream_t st);
// cloudy/clear mixing: grad[b] = gv[2b] + gv[2b+1], with d lnL / d f_cld from the likelihood kernel
void launch_mix_grad(const Model& m, const Work& w, int B, double* grad, hipStream_t st);
size_t trans_fwd_lds_bytes(const Model& m, bool fp64);
// Layer-count classes of a reduced-precision transmission call whose padded layer count
// exceeds kShortLayers: w.cls = [count0, count1, samples of class 0 (at most kShortLayers
// layers, and invalid ones) longest first, then class 1 longest first, each list B long]
inline bool layer_classes_used(const Model& m) { return m.mode == kTransmission && !m.ck && m.L_pad > kShortLayers; }
void launch_layer_classes(const Model& m, const Work& w, int B, hipStream_t st);
hipError_t trans_fwd_configure(const Model& m, bool fp64);

}  // namespace exofwd
