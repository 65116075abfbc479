// Reverse pass of the transmission path.
//
// For every (sample, wavenumber chunk) a fused kernel takes the layer optical
// depths (stored by the forward kernel in the reduced-precision path,
// recomputed in FP64), forms the slant optical depth and the seeds
//   delta_bar(nu) = (d lnL / d m_k) / N_k          (nu in bin k)
//   tau_bar_i(nu) = delta_bar(nu) a_i e^{-tau_i(nu)}
// and accumulates, over its wavenumbers,
//   abar_i   = sum_nu delta_bar (1 - e^{-tau_i})                      (annulus areas)
//   Pbar_il  = sum_nu tau_bar_i dtau_l                                (path matrix)
//   dtau_bar = P^T tau_bar                                            (opacity)
// The per-layer sums of adjoint.h over dtau_bar are formed in the same kernel
// (FP64) or by a separate high-occupancy kernel from the stored dtau_bar
// (reduced precision). The FP64 chain kernel then walks back through the
// path-matrix geometry, the hydrostatic recursion, n = p/kT, chemistry, the
// cloud deck and the T-p profile to d lnL / d params.
#include "adjoint.h"
#include "kernels.h"
#include "cloud.h"
#include "opacity.h"
#include "tp.h"

#include <climits>

namespace exofwd {

// a float pair read once (stored dtau_bar): a non-temporal load
__device__ inline float2 ld_stream2(const float* p) {
  const float2v v = __builtin_nontemporal_load(reinterpret_cast<const float2v*>(p));
  return make_float2(v.x, v.y);
}

// cost-balanced split of 32-row blocks between `parts` (2 or 4) waves: each block in
// turn goes to the part with the least cost so far (the lowest such part on a tie);
// `rev` costs rows by their K extent in the transposed product (grows with the
// block index)
__host__ __device__ inline unsigned split_blocks(int part, int parts, int MBe, int KBe, bool rev) {
  unsigned mine = 0;
  int c[4] = {0, 0, 0, 0};
  for (int q = 0; q < MBe; ++q) {
    const int mi = rev ? MBe - 1 - q : q;
    const int cost = rev ? (2 * mi + 2 < KBe ? 2 * mi + 2 : KBe) : KBe - 2 * mi;
    int best = 0;
    for (int p = 1; p < parts; ++p)
      if (c[p] < c[best]) best = p;
    if (best == part) mine |= 1u << mi;
    c[best] += cost;
  }
  return mine;
}

// index of the q-th set bit of mask (or -1)
__device__ inline int nth_bit(unsigned mask, int q) {
  for (int i = 0; i < 32; ++i)
    if (mask & (1u << i)) {
      if (q == 0) return i;
      --q;
    }
  return -1;
}

// ============================================================================
// reduced-precision reverse kernel over TILE-wavenumber tiles for up to MB
// 32-row blocks (L_pad <= 32 MB); each wave owns one 32-wavenumber column block
// and one of PARTS cost-balanced parts of the row blocks, so every path-matrix
// fragment it loads feeds the products of its whole column block
template <int TILE, int MB, int PARTS>
struct AdjShape {
  static constexpr int kTile = TILE;
  static constexpr int kNb = TILE / 32;                           // column blocks per tile
  static constexpr int kWaves = PARTS * kNb;                      // PARTS row-block parts per column block
  static constexpr int kThreads = 64 * kWaves;
  static constexpr int kHalves = TILE / 64;                       // 64-wavenumber halves (phase A items)
  static constexpr int kSlots = PARTS == 2 ? (MB + 1) / 2 : (MB <= 4 ? 1 : 2);   // row blocks per wave (checked on the host)
  static constexpr int kPSlots = (MB * (MB + 1) / 2 + kWaves - 1) / kWaves;   // 32x32 Pbar tiles per wave
  static constexpr int kItems = (4 * kHalves * MB + kWaves - 1) / kWaves;     // (layer octet, half) items per wave
};

// `cls` (may be null): the layer-count classes of the call (layer_classes), whose class
// `cl` this launch serves (its samples have at most 32 MB layers)
template <int S, bool CIA, int TILE, int MB, int PARTS>
__global__ __launch_bounds__(2 * PARTS * TILE) void k_trans_adj_mixed(Model m, Work w, Tables tb, AdjWork aw, int B,
                                                                      int C, const int32_t* __restrict__ cls, int cl) {
  using Sh = AdjShape<TILE, MB, PARTS>;
  static_assert(Sh::kThreads == 2 * PARTS * TILE, "launch bound");
  static_assert(Sh::kItems * Sh::kWaves >= 4 * Sh::kHalves * MB, "phase A items cover 4 MB octets per half");
  constexpr int kTileA = Sh::kTile, kBlockA = Sh::kThreads, kNbA = Sh::kNb, kWavesA = Sh::kWaves;
  constexpr int kSlots = Sh::kSlots, kPSlotsA = Sh::kPSlots, kItemsA = Sh::kItems, kHalves = Sh::kHalves;
  extern __shared__ __align__(16) unsigned char lds[];
  const int logical = xcd_logical_block(blockIdx.x, gridDim.x);
  // a sample's chunks on neighbouring workgroups of one XCD: its path-matrix fragments,
  // re-read for every tile, stay in that XCD's L2 while its chunks run
  const int chunk = logical % C;
  int b = logical / C;
  if (cls) {
    // the class's samples, longest first, dealt round the XCDs; the grid covers the whole batch
    b = class_position(b, B, C);
    if (b >= cls[cl]) return;
    b = cls[2 + cl * B + b];
  }
  if (w.status[b]) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int Lp = m.L_pad, L = w.nlay[b];
  const int rows = Lp < 32 * MB ? Lp : 32 * MB;        // LDS rows: the layers this shape can hold
  // dwords per wavenumber row (b128-conflict-free), fixed by the shape rather than by
  // L_pad: the gathers of phase E then address eight rows from one register with
  // immediate offsets
  constexpr int ld = 32 * MB + 4;
  uint32_t* s_dt = reinterpret_cast<uint32_t*>(lds);   // dtau    [nu][ld] as packed bf16 hi/lo
  uint32_t* s_tt = s_dt + kTileA * ld;                 // tau_bar [nu][ld] as packed bf16 hi/lo
  float* s_area = reinterpret_cast<float*>(s_tt + kTileA * ld);   // [Lp]

  const float* area = reinterpret_cast<const float*>(w.area) + (size_t)b * Lp;
  for (int i = tid; i < rows; i += kBlockA) s_area[i] = area[i];

  const size_t npad = (size_t)m.n_nu_pad;
  const int KBe = (L + 15) >> 4, MBe = (L + 31) >> 5, KB = Lp >> 4;
  const int nb = wv % kNbA, part = wv / kNbA;
  // row blocks of this wave (slot q -> block index or -1), fixed for the whole call;
  // readfirstlane keeps them in scalar registers
  int t_mi[kSlots], d_ml[kSlots];
  {
    const unsigned mine_t = split_blocks(part, PARTS, MBe, KBe, false);   // rows i of tau
    const unsigned mine_d = split_blocks(part, PARTS, MBe, KBe, true);    // rows l of dtau_bar
#pragma unroll
    for (int q = 0; q < kSlots; ++q) {
      t_mi[q] = __builtin_amdgcn_readfirstlane(nth_bit(mine_t, q));
      d_ml[q] = __builtin_amdgcn_readfirstlane(nth_bit(mine_d, q));
    }
  }
  const size_t plane = (size_t)(Lp >> 5) * KB * 512;
  // this sample's P and P^T fragments (hi plane, then lo plane); lanes address
  // their 16 bytes with the vector offset, blocks with the scalar offset
  const __amdgpu_buffer_rsrc_t rs_p = make_rsrc(w.pfrag + (size_t)b * 2 * plane, 2 * plane * 2);
  const __amdgpu_buffer_rsrc_t rs_pt = make_rsrc(w.ptfrag + (size_t)b * 2 * plane, 2 * plane * 2);
  const uint32_t lo_plane = (uint32_t)plane * 2u, voff_f = (uint32_t)lane * 16u;
  auto frag = [&](__amdgpu_buffer_rsrc_t rs, int blk, uint32_t pl) {
    return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rs, voff_f, (uint32_t)blk * 1024u + pl, 0));
  };
  const int col = 32 * nb + (lane & 31);
  const int h = lane >> 5;
  const double* dm = w.dm + (size_t)b * m.K;
  // 32x32 product over k-steps [k_lo, k_hi): A = path-matrix fragments (rs) of blocks
  // row0 + k, B = the packed hi/lo rows 16k.. of the LDS array src at this wave's
  // column.  The fragments go in two groups of two steps: one group's loads are in
  // flight while the other group's products run.  Every iteration issues the same
  // loads (steps past k_hi read the next row block's fragments, or zeros past the
  // buffer's range, and are never used), so the waits count only the older group.
  auto kloop = [&](__amdgpu_buffer_rsrc_t rs, int row0, int k_lo, int k_hi, const uint32_t* src) {
    f32x16 acc = {};
    bf16x8 ga[2][2], gb[2][2];   // [step][hi, lo]
    auto load = [&](bf16x8 (&g)[2][2], int k) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        g[u][0] = frag(rs, row0 + k + u, 0);
        g[u][1] = frag(rs, row0 + k + u, lo_plane);
      }
    };
    auto product = [&](const bf16x8 (&g)[2][2], int k0) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int k = k0 + u;
        if (k >= k_hi) break;
        bf16x8 bh, bl;
        {
          const uint4 x0 = *reinterpret_cast<const uint4*>(src + col * ld + 16 * k + 8 * h);
          const uint4 x1 = *reinterpret_cast<const uint4*>(src + col * ld + 16 * k + 8 * h + 4);
          const uint32_t x[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
          frag_hl(x, bh, bl);
        }
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(g[u][1], bh, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(g[u][0], bl, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(g[u][0], bh, acc, 0, 0, 0);
      }
    };
    load(ga, k_lo);
#pragma unroll 1
    for (int kb = k_lo; kb < k_hi; kb += 4) {
      load(gb, kb + 2);
      product(ga, kb);
      if (kb + 2 >= k_hi) break;
      load(ga, kb + 4);
      product(gb, kb + 2);
    }
    return acc;
  };

  // Pbar tiles (32x32, column block >= row block), round-robin over the waves
  int pt_mi[kPSlotsA], pt_nl[kPSlotsA];
  {
    int t = 0;
    for (int q = 0; q < kPSlotsA; ++q) pt_mi[q] = pt_nl[q] = -1;
    for (int mi = 0; mi < MBe; ++mi)
      for (int nl = mi; nl < MBe; ++nl, ++t)
        if (t % kWavesA == wv && t / kWavesA < kPSlotsA) {
          pt_mi[t / kWavesA] = mi;
          pt_nl[t / kWavesA] = nl;
        }
#pragma unroll
    for (int q = 0; q < kPSlotsA; ++q) {
      pt_mi[q] = __builtin_amdgcn_readfirstlane(pt_mi[q]);
      pt_nl[q] = __builtin_amdgcn_readfirstlane(pt_nl[q]);
    }
  }
  f32x16 abar_acc[kSlots], pbar_acc[kPSlotsA];
#pragma unroll
  for (int q = 0; q < kSlots; ++q) abar_acc[q] = f32x16{};
#pragma unroll
  for (int q = 0; q < kPSlotsA; ++q) pbar_acc[q] = f32x16{};

  // this sample's stored optical depths and dtau_bar ([L_pad][n_nu_pad], rebased per tile)
  const float* dtau_b = aw.dtau + (size_t)b * Lp * npad;
  float* dtb_b = aw.dtb + (size_t)b * Lp * npad;
  const int ntiles = m.n_nu_pad / kTileA;
  const int t0 = chunk * ntiles / C, t1 = (chunk + 1) * ntiles / C;

  // the stored optical depths of a tile are fetched into registers while the
  // previous tile's Pbar product runs, then written to LDS as packed hi/lo:
  // items (layer octet o, half of the tile), a lane takes one wavenumber of the half
  uint32_t pf[kItemsA][8];   // packed bf16 hi | lo << 16, as the forward stored them
  // row offsets go in the scalar offset (wave-uniform, recomputed per tile); rows
  // [L, 32 MBe) lie inside the sample's L_pad rows and are replaced by zero when staged
  const __amdgpu_buffer_rsrc_t rs_dt = make_rsrc(dtau_b, (size_t)Lp * npad * 4);
  const uint32_t rowb = (uint32_t)npad * 4u;
  // layers below the tile's opaque frontier feed only chords whose seeds are zero
  // (nothing below reads them): they are neither fetched nor staged
  auto front_of = [&](int tile) { return w.front[(size_t)b * m.n_tiles + min(tile, t1 - 1) * kTileA / kTileNu]; };
  auto fetch = [&](int tile, int lo_row) {
#pragma unroll
    for (int q = 0; q < kItemsA; ++q) {
      const int it = wv + kWavesA * q;
      if (it >= 4 * kHalves * MBe) continue;   // 4 MBe layer octets per half
      const int o = it / kHalves;
      if (8 * o + 8 <= lo_row) {
#pragma unroll
        for (int j = 0; j < 8; ++j) pf[q][j] = 0u;
        continue;
      }
      const uint32_t voff = (uint32_t)(64 * (it % kHalves) + lane) * 4u;
      const uint32_t soff = (uint32_t)((8 * o * npad + (size_t)tile * kTileA) * 4);
#pragma unroll
      for (int j = 0; j < 8; ++j)
        pf[q][j] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rs_dt, voff, soff + j * rowb, kCpolStream);
    }
  };
  auto stage = [&](int lo_row) {
    // L passed through an empty asm: the row tests below are then formed where
    // they are used, instead of being hoisted out of the tile loop as 32 masks
    int Lq = L;
    asm volatile("" : "+s"(Lq));
#pragma unroll
    for (int q = 0; q < kItemsA; ++q) {
      const int it = wv + kWavesA * q;
      if (it >= 4 * kHalves * MBe) continue;   // 4 MBe layer octets per half
      const int o = it / kHalves, nu = 64 * (it % kHalves) + lane;
      uint32_t d[8];
      if (8 * o >= lo_row && 8 * o + 8 <= Lq) {   // the whole octet (the frontier is a multiple of 32 rows)
#pragma unroll
        for (int j = 0; j < 8; ++j) d[j] = pf[q][j];
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) d[j] = (8 * o + j < Lq && 8 * o + j >= lo_row) ? pf[q][j] : 0u;
      }
      uint32_t* dst = s_dt + nu * ld + 8 * o;
      *reinterpret_cast<uint4*>(dst) = make_uint4(d[0], d[1], d[2], d[3]);
      *reinterpret_cast<uint4*>(dst + 4) = make_uint4(d[4], d[5], d[6], d[7]);
    }
  };
  // ---- phase A of the first tile
  // What a tile starts from comes before it starts: the frontier and the bin two
  // barriers ahead (during the Pbar product of the tile before), the bin's seed from
  // behind the next barrier on. Read at the tile's start the two chained gathers stood
  // in front of its first product, and the frontier in front of the fetch: headline
  // batch 25.8 -> 25.3 ms for the call, 64 fine-grid gradients 21.4 -> 20.8.
  int mi0 = 0, f_next = 0, bin = -1;
  double dmv = 0.0, icv = 0.0;
  auto bin_at = [&](int tile) { return w.bin_of[min(tile, t1 - 1) * kTileA + col]; };
  if (t0 < t1) {
    mi0 = __builtin_amdgcn_readfirstlane(front_of(t0));
    fetch(t0, 32 * mi0);
    f_next = front_of(t0 + 1);
    bin = bin_at(t0);
    dmv = dm[max(bin, 0)];
    icv = w.inv_cnt[max(bin, 0)];
    stage(32 * mi0);
  }
  __syncthreads();

  for (int tile = t0; tile < t1; ++tile) {
    const int nu0 = tile * kTileA;
    // row blocks below mi0 hold only opaque chords (tau > kOpaqueTau across the
    // forward pass's 128-wavenumber tile): their seeds are exactly zero, so their
    // products are skipped and the results are those of the full computation
    const int mi0_next = __builtin_amdgcn_readfirstlane(f_next);

    // ---- phases B, C: tau = P dtau; seeds; tau_bar -> LDS [nu][i]; abar accumulation
    {
      const float dbar = bin >= 0 ? (float)(dmv * icv) : 0.0f;
#pragma unroll
      for (int q = 0; q < kSlots; ++q) {
        const int mi = t_mi[q];
        if (mi < 0) continue;
        if (mi < mi0) {
          // e^-tau = 0: abar takes dbar (1 - 0), tau_bar is 0
#pragma unroll
          for (int j = 0; j < 16; ++j) abar_acc[q][j] += dbar;
#pragma unroll
          for (int qd = 0; qd < 4; ++qd)
            *reinterpret_cast<uint4*>(s_tt + col * ld + 32 * mi + 8 * qd + 4 * h) = make_uint4(0u, 0u, 0u, 0u);
          continue;
        }
        const f32x16 acc = kloop(rs_p, mi * KB, 2 * mi, KBe, s_dt);
#pragma unroll
        for (int qd = 0; qd < 4; ++qd) {
          float tv[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int j = 4 * qd + r;
            const int row = 32 * mi + 8 * qd + 4 * h + r;
            const float e = exp2_fast(-1.4426950408889634f * acc[j]);
            abar_acc[q][j] = fmaf(dbar, one_minus_exp(acc[j], e), abar_acc[q][j]);
            tv[r] = dbar * s_area[row] * e;
          }
          *reinterpret_cast<uint4*>(s_tt + col * ld + 32 * mi + 8 * qd + 4 * h) =
              make_uint4(pack_hl(tv[0]), pack_hl(tv[1]), pack_hl(tv[2]), pack_hl(tv[3]));
        }
      }
    }
    __syncthreads();
    // ---- phase A of the next tile, part 1: its optical depths are in flight
    // while phase E (LDS and MFMA only) runs
    const bool more = tile + 1 < t1;
    if (more) fetch(tile + 1, 32 * mi0_next);
    f_next = front_of(tile + 2);
    bin = bin_at(tile + 1);

    // ---- phase E: Pbar += tau_bar dtau^T over the tile's wavenumbers (bf16x3 MFMA, k = wavenumber);
    // operands gathered from eight wavenumber rows of the packed hi/lo LDS arrays
#pragma unroll
    for (int q = 0; q < kPSlotsA; ++q) {
      const int mi = pt_mi[q], nl = pt_nl[q];
      if (mi < mi0) continue;   // also the empty slots (mi = -1): zero seeds add nothing
      const uint32_t* pa = s_tt + 8 * h * ld + 32 * mi + (lane & 31);
      const uint32_t* pbp = s_dt + 8 * h * ld + 32 * nl + (lane & 31);
#pragma unroll 1
      for (int ks = 0; ks < kTileA / 16; ++ks) {
        // the step's row offset kept opaque in a scalar register: each operand's eight
        // rows are then one address plus immediate offsets (the arrays lie past 64 KB)
        int off = 16 * ks * ld;
        asm volatile("" : "+s"(off));
        uint32_t va[8], vb[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          va[e] = pa[off + e * ld];
          vb[e] = pbp[off + e * ld];
        }
        bf16x8 ah, al, bh, bl;
        frag_hl(va, ah, al);
        frag_hl(vb, bh, bl);
        pbar_acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh, pbar_acc[q], 0, 0, 0);
        pbar_acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl, pbar_acc[q], 0, 0, 0);
        pbar_acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh, pbar_acc[q], 0, 0, 0);
      }
    }
    // ---- phase A of the next tile, part 2: every wave is past phase E, the last
    // reader of this tile's dtau
    __syncthreads();
    if (more) stage(32 * mi0_next);
    dmv = dm[max(bin, 0)];
    icv = w.inv_cnt[max(bin, 0)];
    // ---- phase D: dtau_bar = P^T tau_bar (rows l, this wave's column block) -> HBM
    {
      const __amdgpu_buffer_rsrc_t rs_db = make_rsrc(dtb_b + nu0, ((size_t)Lp * npad - nu0) * 4);
#pragma unroll
      for (int q = 0; q < kSlots; ++q) {
        const int ml = d_ml[q];
        // rows below the opaque frontier would be exact zeros: the readers of
        // dtau_bar consult the frontier instead, so they are not stored
        if (ml < mi0) continue;
        const int kend = min(2 * ml + 2, KBe);
        // the seed rows of blocks below mi0 are zero: the sum starts at row 32 mi0
        const int kbeg = min(2 * mi0, kend);
        const f32x16 acc = kloop(rs_pt, ml * KB, kbeg, kend, s_tt);
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const int row = 32 * ml + 8 * (j >> 2) + 4 * h + (j & 3);
          // rows [L, 32 MBe) land in this sample's padding rows, which nothing reads
          // element copied to a scalar first: a bit_cast of a vector element lowers to element 0
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint((float)acc[j]), rs_db,
                                                (uint32_t)((row * npad + col) * 4), 0, kCpolStream);
        }
      }
    }
    mi0 = mi0_next;
    __syncthreads();   // the next tile reads the staged dtau and overwrites tau_bar
  }

  // ---- write this chunk's partials
  const size_t pair = (size_t)b * C + chunk;
  float* pb = reinterpret_cast<float*>(aw.pbar) + pair * Lp * Lp;
#pragma unroll
  for (int q = 0; q < kPSlotsA; ++q) {
    const int mi = pt_mi[q], nl = pt_nl[q];
    if (mi < 0) continue;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int row = 32 * mi + 8 * (j >> 2) + 4 * h + (j & 3);
      pb[(size_t)row * Lp + 32 * nl + (lane & 31)] = pbar_acc[q][j];
    }
  }
  // abar: reduce over the 32 columns of each lane half, then over the column blocks
#pragma unroll
  for (int q = 0; q < kSlots; ++q) {
    const int mi = t_mi[q];
    if (mi < 0) continue;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      float v = abar_acc[q][j];
      for (int off = 16; off > 0; off >>= 1) v += __shfl_xor(v, off);
      abar_acc[q][j] = v;
    }
  }
  double* s_ab = reinterpret_cast<double*>(lds);   // [kNbA][Lp], all waves are past the loop
#pragma unroll
  for (int q = 0; q < kSlots; ++q) {
    const int mi = t_mi[q];
    if (mi < 0) continue;
    if ((lane & 31) == 0) {
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int row = 32 * mi + 8 * (j >> 2) + 4 * h + (j & 3);
        s_ab[nb * Lp + row] = (double)abar_acc[q][j];
      }
    }
  }
  __syncthreads();
  double* ab = aw.abar + pair * Lp;
  for (int i = tid; i < Lp; i += kBlockA) {
    double v = 0.0;
    if (i < 32 * MBe)
#pragma unroll
      for (int n = 0; n < kNbA; ++n) v += s_ab[n * Lp + i];
    ab[i] = v;
  }
}

// a * h.x + c and a * h.y + c with the FP16 half taken as an operand of the FMA
// (v_fma_mix_f32): the same single rounding as converting it first, without a
// converted copy of the table pairs held in registers across a group's layers
__device__ inline float fma_f16lo(float a, half2_t h, float c) {
  float d;
  asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel_hi:[0,1,0]" : "=v"(d) : "v"(a), "v"(h), "v"(c));
  return d;
}
__device__ inline float fma_f16hi(float a, half2_t h, float c) {
  float d;
  asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[0,1,0] op_sel_hi:[0,1,0]" : "=v"(d) : "v"(a), "v"(h), "v"(c));
  return d;
}

// Line and CIA terms of one layer for two wavenumbers together with the derivative of each
// exponent with respect to the T weight, from the two log p-interpolated rows u0 (at iT) and
// u1 (at iT+1), both offset by c + lam:
//   exponent = u0 + wT (u1 - u0),  d exponent / d wT = u1 - u0.
// The line pairs enter their FMAs as FP16 operands.
template <int S, bool CIA>
__device__ inline void eval_terms_deriv_f16(const LayerCoef<S>& c, const LaneConst<S>& k, const LayerRaw<S, CIA>& r,
                                            float* t0, float* t1, float* dw0, float* dw1) {
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const half2_t h00 = r.h[4 * s], h10 = r.h[4 * s + 1], h01 = r.h[4 * s + 2], h11 = r.h[4 * s + 3];
    const float cl0 = k.c0[s] + c.lam[s], cl1 = k.c1[s] + c.lam[s];
    const float u00 = fma_f16lo(c.omp, h00, fma_f16lo(c.wp, h01, cl0));
    const float u10 = fma_f16lo(c.omp, h10, fma_f16lo(c.wp, h11, cl0));
    const float u01 = fma_f16hi(c.omp, h00, fma_f16hi(c.wp, h01, cl1));
    const float u11 = fma_f16hi(c.omp, h10, fma_f16hi(c.wp, h11, cl1));
    dw0[s] = u10 - u00;
    dw1[s] = u11 - u01;
    t0[s] = exp2_fast(fmaf(c.wt, dw0[s], u00));
    t1[s] = exp2_fast(fmaf(c.wt, dw1[s], u01));
  }
  if constexpr (CIA) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const half2_t a = r.h[4 * S + 2 * p], b = r.h[4 * S + 2 * p + 1];
      const float u0 = (float)a.x + (k.cc0[p] + c.lamc[p]);
      const float u1 = (float)a.y + (k.cc1[p] + c.lamc[p]);
      dw0[S + p] = (float)b.x - (float)a.x;
      dw1[S + p] = (float)b.y - (float)a.y;
      t0[S + p] = exp2_fast(fmaf(c.wtc, dw0[S + p], u0));
      t1[S + p] = exp2_fast(fmaf(c.wtc, dw1[S + p], u1));
    }
  }
}

// ============================================================================
// reduced-precision per-layer sums: one wave per (sample, layer group, ls_tiles tiles),
// a layer group being a run of up to kLsGroup consecutive layers in one table cell
// (listed by the profile kernel), whose table pairs are fetched once per tile,
// together with the tile's dtau_bar; lanes hold two wavenumbers, partial sums stay
// in registers across the tiles and are reduced over the wave once, 16 sums at a time by
// halving lane exchanges (one store per layer; 14 butterflies of six LDS permutes each
// before: 1024 samples x 30000 wavenumbers x 100 layers, the gradient call 27.8 -> 26.35 ms)

template <int S, bool CIA, bool NGC>
__global__ __launch_bounds__(kBlock) void k_layer_sums_mixed(Model m, Work w, Tables tb, AdjWork aw, int B) {
  constexpr int NS = n_sums(S);
  constexpr int kLs = kLsGroup;
  const int lane = threadIdx.x & 63;
  // consecutive waves (one wavenumber chunk) on one XCD: its L2 holds that chunk's table columns
  const int gw = xcd_logical_block(blockIdx.x, gridDim.x) * (kBlock / 64) +
                 __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int NG = m.L_max;   // groups per sample: at most one per layer
  const int per_chunk = B * NG;
  const int chunk = gw / per_chunk;
  if (chunk >= aw.lsum_chunks) return;
  const int rem = gw - chunk * per_chunk;
  const int b = rem / NG, lg = rem - b * NG;
  if (w.status[b]) return;
  const int Lp = m.L_pad;
  const int32_t* grp = w.lsg + (size_t)b * (Lp + 1);
  if (lg >= grp[0]) return;
  const int l0 = grp[1 + lg] & 0xffff, cnt = grp[1 + lg] >> 16;
  const size_t npad = (size_t)m.n_nu_pad;
  TableGeom g;
  g.row_bytes = (uint32_t)npad * 2u;
  g.tstep = (uint32_t)m.n_p * g.row_bytes;
  g.pstep = g.row_bytes;
  const __amdgpu_buffer_rsrc_t rh = make_rsrc(tb.h, (size_t)S * m.n_t * m.n_p * npad * 2);
  const __amdgpu_buffer_rsrc_t rhc = make_rsrc(CIA ? (const void*)tb.hc : (const void*)tb.h,
                                               CIA ? (size_t)2 * m.n_tc * npad * 2 : 0);
  const uint32_t voff = (uint32_t)lane * 4u;
  const float* rec = reinterpret_cast<const float*>(w.rec) + (size_t)b * Lp * rec_len_wide(S);
  const int32_t* cells = w.cells + (size_t)b * Lp;
  const float* dtb = aw.dtb + (size_t)b * Lp * npad;

  float acc[kLs][NS];
#pragma unroll
  for (int q = 0; q < kLs; ++q)
#pragma unroll
    for (int k = 0; k < NS; ++k) acc[q][k] = 0.0f;
  // non-grey cloud: Q_ext at the lane's two wavenumbers weights the cloud sum (its
  // spectral parameters are summed by k_cloud_spectral: more live registers here
  // would cost this kernel its load pipelining)
  const float* cq = NGC ? w.cloud_q + (size_t)b * (1 + kCloudSpec) * npad : nullptr;

  const int t0 = chunk * aw.ls_tiles, t1 = min(t0 + aw.ls_tiles, m.n_tiles);
  for (int tile = t0; tile < t1; ++tile) {
    const int nu0 = tile * kTileNu;
    // every chord through the group's layers opaque across the tile: dtau_bar is
    // exactly zero there and the tile adds nothing (the deep layers of most
    // atmospheres).  Rows below the reverse pass's opaque frontier are not stored.
    const int lo_row = 32 * w.front[(size_t)b * m.n_tiles + tile];
    if (l0 + cnt <= lo_row) continue;
    float2 dbq[kLs];
#pragma unroll
    for (int q = 0; q < kLs; ++q)
      dbq[q] = (q < cnt && l0 + q >= lo_row) ? ld_stream2(dtb + (size_t)(l0 + q) * npad + nu0 + 2 * lane)
                                             : make_float2(0.0f, 0.0f);
    // the group's table pairs, fetched with dtau_bar (one memory round trip per tile)
    // before the test that skips a tile whose dtau_bar is zero
    const LayerCoef<S> c0 = load_layer<S>(m, cells, rec, l0, (uint32_t)nu0 * 2u, g);
    LayerRaw<S, CIA> raw;
    fetch_terms<S, CIA>(c0, g, rh, rhc, voff, raw);
    const LaneConst<S> kc = load_lane<S, CIA>(m, tb, nu0 + 2 * lane);
    bool live = false;
#pragma unroll
    for (int q = 0; q < kLs; ++q) live |= dbq[q].x != 0.0f || dbq[q].y != 0.0f;
    if (__builtin_amdgcn_ballot_w64(live) == 0) continue;
    float q0 = 1.0f, q1 = 1.0f;
    if constexpr (NGC) {
      const float2 q = *reinterpret_cast<const float2*>(cq + nu0 + 2 * lane);
      q0 = q.x;
      q1 = q.y;
    }
#pragma unroll
    for (int q = 0; q < kLs; ++q) {
      if (q >= cnt) continue;
      const float2 db = dbq[q];
      const LayerCoef<S> c = q == 0 ? c0 : load_layer<S>(m, cells, rec, l0 + q, (uint32_t)nu0 * 2u, g);
      float t0_[S + 2], t1_[S + 2], dw0[S + 2], dw1[S + 2];
      eval_terms_deriv_f16<S, CIA>(c, kc, raw, t0_, t1_, dw0, dw1);
      // G_s += db t_s per wavenumber; the T-weight sums take db once per wavenumber
      // times z = sum_s t_s dw_s
      float z0 = 0.0f, z1 = 0.0f;
#pragma unroll
      for (int s = 0; s < S; ++s) {
        acc[q][s] = fmaf(db.x, t0_[s], fmaf(db.y, t1_[s], acc[q][s]));
        z0 = fmaf(t0_[s], dw0[s], z0);
        z1 = fmaf(t1_[s], dw1[s], z1);
      }
      acc[q][S] = fmaf(db.x, z0, fmaf(db.y, z1, acc[q][S]));
      if (CIA) {
        float y0 = 0.0f, y1 = 0.0f;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          acc[q][S + 1 + p] = fmaf(db.x, t0_[S + p], fmaf(db.y, t1_[S + p], acc[q][S + 1 + p]));
          y0 = fmaf(t0_[S + p], dw0[S + p], y0);
          y1 = fmaf(t1_[S + p], dw1[S + p], y1);
        }
        acc[q][S + 3] = fmaf(db.x, y0, fmaf(db.y, y1, acc[q][S + 3]));
      }
      acc[q][S + 4] = fmaf(db.x, kc.nu4_0, fmaf(db.y, kc.nu4_1, acc[q][S + 4]));
      if constexpr (NGC) {
        acc[q][S + 5] = fmaf(db.x, q0, fmaf(db.y, q1, acc[q][S + 5]));
      } else {
        acc[q][S + 5] += db.x + db.y;
      }
    }
  }
  float* out = aw.lsum + ((size_t)b * aw.lsum_stride + chunk) * Lp * NS;
#pragma unroll
  for (int q = 0; q < kLs; ++q) {
    if (q >= cnt) continue;
    float v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = k < NS ? acc[q][k < NS ? k : 0] : 0.0f;
    const float tot = wave_sums16(v, lane);
    if ((lane & 3) == 0 && (lane >> 2) < NS) out[(size_t)(l0 + q) * NS + (lane >> 2)] = tot;
  }
}

// Non-grey cloud: sums over wavenumber of G(nu) dQ_ext/dp_k with
// G(nu) = sum_l D_l dtau_bar_l(nu), the derivative of lnL along the cloud's
// spectral shape; one wave per (sample, layer-sum chunk), two wavenumbers per lane.
__global__ __launch_bounds__(kBlock) void k_cloud_spectral(Model m, Work w, AdjWork aw, int B) {
  const int lane = threadIdx.x & 63;
  const int gw = blockIdx.x * (kBlock / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int b = gw / aw.lsum_chunks, chunk = gw - b * aw.lsum_chunks;
  if (b >= B || w.status[b]) return;
  const int L = w.nlay[b], Lp = m.L_pad;
  const size_t npad = (size_t)m.n_nu_pad;
  const float* rec = reinterpret_cast<const float*>(w.rec) + (size_t)b * Lp * rec_len_wide(m.S);
  const float* dtb = aw.dtb + (size_t)b * Lp * npad;
  const float* cq = w.cloud_q + (size_t)b * (1 + kCloudSpec) * npad;
  float hq[kCloudSpec] = {};
  const int t0 = chunk * aw.ls_tiles, t1 = min(t0 + aw.ls_tiles, m.n_tiles);
  for (int tile = t0; tile < t1; ++tile) {
    const int nu = tile * kTileNu + 2 * lane;
    float g0 = 0.0f, g1 = 0.0f;
    // rows below the opaque frontier are zero (and not stored); kFly rows in flight
    constexpr int kFly = 8;
    int l = 32 * w.front[(size_t)b * m.n_tiles + tile];
    for (; l + kFly <= L; l += kFly) {
      float2 d[kFly];
#pragma unroll
      for (int u = 0; u < kFly; ++u) d[u] = *reinterpret_cast<const float2*>(dtb + (size_t)(l + u) * npad + nu);
#pragma unroll
      for (int u = 0; u < kFly; ++u) {
        const float dl = rec[(size_t)(l + u) * rec_len_wide(m.S) + 4];
        g0 = fmaf(dl, d[u].x, g0);
        g1 = fmaf(dl, d[u].y, g1);
      }
    }
    for (; l < L; ++l) {
      const float dl = rec[(size_t)l * rec_len_wide(m.S) + 4];
      const float2 d = *reinterpret_cast<const float2*>(dtb + (size_t)l * npad + nu);
      g0 = fmaf(dl, d.x, g0);
      g1 = fmaf(dl, d.y, g1);
    }
#pragma unroll
    for (int k = 0; k < kCloudSpec; ++k) {
      const float2 d = *reinterpret_cast<const float2*>(cq + (size_t)(1 + k) * npad + nu);
      hq[k] = fmaf(g0, d.x, fmaf(g1, d.y, hq[k]));
    }
  }
#pragma unroll
  for (int k = 0; k < kCloudSpec; ++k) {
    const float tot = wave_sum_all(hq[k]);
    if (lane == 0) aw.hq[((size_t)b * aw.lsum_stride + chunk) * kCloudSpec + k] = tot;
  }
}

// ============================================================================
// FP64 reverse kernel: 512 threads, one sample and wavenumber chunk per workgroup, every
// product on v_mfma_f64_16x16x4f64

// Per tile: the layer optical depths (each wave a contiguous run of layers) -> LDS; the
// chords, seeds and tau_bar -> LDS; the path-matrix adjoint (accumulated in registers over
// the chunk's tiles) and dtau_bar, which replaces the optical depths in LDS; the per-layer
// sums, the layers above the tile's opaque frontier split evenly over the waves.  The
// terms of the sums are formed again from the tables: recomputing costs less than the
// registers or the memory traffic of keeping them.  A tile's tau_bar is zero (as exact
// zeros) in the 16-row blocks below the frontier, whose products and sums are skipped.
// Samples run fastest over the workgroups, so an XCD's workgroups read the same table
// columns.  24 samples x 30000 wavenumbers x 100 layers x 6 absorbers: the whole FP64
// gradient call 14.0 -> 3.5 ms (vector products with one LDS and one memory read per FMA,
// 14 wave butterflies per layer and tile, and table columns no neighbour shared).  What is
// left: the accumulators of Pbar and abar stay live beside a cell's table entries and terms
// in the sums, so the kernel takes all 256 registers (two waves per SIMD) and spills 140 to
// 648 bytes per lane (456 at six absorbers with CIA); vector instructions issue in 32 % of
// its cycles.
//
// TILE = 64 wavenumbers up to 128 padded layers; 32 (lanes 32-63 hold no wavenumber and add
// zeros) up to 160, where two 64-wavenumber arrays no longer fit in LDS.
template <int S, bool CIA, int TILE>
__global__ __launch_bounds__(kBlockT) void k_trans_adj_fp64(Model m, Work w, Tables tb, AdjWork aw, int B, int C) {
  constexpr int kWaves = kBlockT / 64, kNb = TILE / 16, kParts = kWaves / kNb, ld = TILE + 2;
  constexpr int kMB = TILE == 64 ? 8 : 10;         // most 16-row blocks
  constexpr int kSlots = TILE == 64 ? 4 : 3;       // row blocks of a wave (split_blocks16 of up to kMB blocks)
  constexpr int kPSlots = (kMB * (kMB + 1) / 2 + kWaves - 1) / kWaves;   // 16x16 Pbar tiles of a wave
  constexpr int NS = n_sums(S);
  static_assert(NS <= 16, "wave_sums16");
  extern __shared__ __align__(16) unsigned char lds[];
  const int logical = xcd_logical_block(blockIdx.x, gridDim.x);
  const int b = logical % B, chunk = logical / B;
  if (w.status[b]) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int Lp = m.L_pad, L = w.nlay[b], MB = (L + 15) >> 4, R = rows16(m.L_max);
  double* s_dt = reinterpret_cast<double*>(lds);   // dtau, later dtau_bar [l][ld]
  double* s_tb = s_dt + R * ld;                    // tau_bar [i][ld]
  double* s_sums = s_tb + R * ld;                  // [R][16]
  double* s_g = s_sums + R * 16;                   // [kWaves][64] non-grey cloud: sum_l D_l dtau_bar_l of a wave's layers
  double* s_hq = s_g + kWaves * 64;                // [kCloudSpec][64] its sums over nu of G(nu) dQ/dp_k, G summed over the layers
  double* s_area = s_hq + kCloudSpec * 64;         // [R]
  int* s_live = reinterpret_cast<int*>(s_area + R);   // row blocks with a chord that is not opaque
  const bool act = lane < TILE;                    // this lane holds a wavenumber of the tile
  for (int i = tid; i < R * 16; i += kBlockT) s_sums[i] = 0.0;

  const auto rec = const_ptr(reinterpret_cast<const double*>(w.rec)) + (size_t)b * Lp * rec_len(S);
  const auto cells = const_ptr(w.cells) + (size_t)b * Lp;
  const double* pm = w.pm64 + (size_t)b * Lp * Lp;
  const double* area = reinterpret_cast<const double*>(w.area) + (size_t)b * Lp;
  for (int i = tid; i < R; i += kBlockT) s_area[i] = area[i];
  const double* dm = w.dm + (size_t)b * m.K;

  // row blocks of the chord (t) and dtau_bar (d) products of this wave's column block, and
  // its Pbar tiles (column block >= row block, round-robin over the waves)
  const int h = lane >> 4, n16 = lane & 15, nb = wv % kNb, part = wv / kNb;
  int t_mi[kSlots], d_ml[kSlots], pt_mi[kPSlots], pt_nl[kPSlots];
  {
    const unsigned mine_t = split_blocks16(part, kParts, MB, false), mine_d = split_blocks16(part, kParts, MB, true);
#pragma unroll
    for (int q = 0; q < kSlots; ++q) {
      t_mi[q] = __builtin_amdgcn_readfirstlane(nth_bit(mine_t, q));
      d_ml[q] = __builtin_amdgcn_readfirstlane(nth_bit(mine_d, q));
    }
    int t = 0;
    for (int q = 0; q < kPSlots; ++q) pt_mi[q] = pt_nl[q] = -1;
    for (int mi = 0; mi < MB; ++mi)
      for (int nl = mi; nl < MB; ++nl, ++t)
        if (t % kWaves == wv && t / kWaves < kPSlots) {
          pt_mi[t / kWaves] = mi;
          pt_nl[t / kWaves] = nl;
        }
#pragma unroll
    for (int q = 0; q < kPSlots; ++q) {
      pt_mi[q] = __builtin_amdgcn_readfirstlane(pt_mi[q]);
      pt_nl[q] = __builtin_amdgcn_readfirstlane(pt_nl[q]);
    }
  }
  f64x4 abar_acc[kSlots], pacc[kPSlots];
#pragma unroll
  for (int q = 0; q < kSlots; ++q) abar_acc[q] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int q = 0; q < kPSlots; ++q) pacc[q] = f64x4{0.0, 0.0, 0.0, 0.0};

  if (m.cloud_ng && wv == 0)
    for (int k = 0; k < kCloudSpec; ++k) s_hq[k * 64 + lane] = 0.0;
  auto q_ext = [&](int nu, double* dq) {
    return cloud_q<double>(m.cloud_qext, load_cloud<double>(w.cloud + (size_t)b * kCloudSpec), m.nu[nu], dq);
  };
  const int ntiles = m.n_nu_pad / TILE;
  const int t0 = chunk * ntiles / C, t1 = (chunk + 1) * ntiles / C;
  for (int tile = t0; tile < t1; ++tile) {
    const int nu = tile * TILE + (act ? lane : 0);
    const double nu4 = tb.nu4d[nu];
    const double qx = m.cloud_ng ? q_ext(nu, nullptr) : 1.0;
    // ---- optical depths
    if (tid < kMaxBlocks16) s_live[tid] = 0;
    {
      LayerRows64<S, CIA> rows;
      int cell_prev = -1;
      for (int l = L * wv / kWaves; l < L * (wv + 1) / kWaves; ++l) {
        const int cl = cells[l];
        if (cl != cell_prev) {
          fetch_rows64<S, CIA>(m, tb, cl, nu, rows);
          cell_prev = cl;
        }
        const double d = eval_rows64<S, CIA>(rec + (size_t)l * rec_len(S), rows, nu4, qx);
        if (act) s_dt[l * ld + lane] = d > 1.0e300 ? 1.0e300 : d;   // finite, as in the forward kernel
      }
    }
    for (int l = L + wv; l < 16 * MB; l += kWaves)
      if (act) s_dt[l * ld + lane] = 0.0;
    __syncthreads();
    // ---- chords, seeds, tau_bar
    {
      const int nu_c = tile * TILE + 16 * nb + n16;
      const int bin = w.bin_of[nu_c];
      const double dbar = bin >= 0 ? dm[bin] * w.inv_cnt[bin] : 0.0;
      const double* pb = s_dt + 4 * h * ld + 16 * nb + n16;
#pragma unroll
      for (int q = 0; q < kSlots; ++q) {
        const int mi = t_mi[q];
        if (mi < 0) continue;
        const double* pa = pm + (size_t)(16 * mi + n16) * Lp + 4 * h;
        f64x4 acc = {0.0, 0.0, 0.0, 0.0};
        f64x4 a = *reinterpret_cast<const f64x4*>(pa + 16 * mi);
#pragma unroll 1
        for (int K = mi; K < MB; ++K) {
          const f64x4 cur = a;
          if (K + 1 < MB) a = *reinterpret_cast<const f64x4*>(pa + 16 * (K + 1));
#pragma unroll
          for (int j = 0; j < 4; ++j)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(cur[j], pb[(16 * K + j) * ld], acc, 0, 0, 0);
        }
        bool live = false;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int i = 16 * mi + h + 4 * e;
          double om, ex;
          absorb_d(acc[e], om, ex);   // a thin chord's om to its last digits: abar sums nothing larger
          abar_acc[q][e] = fma(dbar, om, abar_acc[q][e]);
          s_tb[i * ld + 16 * nb + n16] = dbar * s_area[i] * ex;
          live |= !(ex == 0.0);
        }
        if (__builtin_amdgcn_ballot_w64(live) != 0 && lane == 0) s_live[mi] = 1;
      }
    }
    __syncthreads();
    int mi0 = 0;
    while (mi0 < MB && !s_live[mi0]) ++mi0;
    mi0 = __builtin_amdgcn_readfirstlane(mi0);
    // ---- Pbar += tau_bar dtau^T (k = wavenumber)
#pragma unroll
    for (int q = 0; q < kPSlots; ++q) {
      const int mi = pt_mi[q], nl = pt_nl[q];
      if (mi < mi0) continue;   // also the empty slots (mi = -1)
      const double* pa = s_tb + (16 * mi + n16) * ld + h;
      const double* pb = s_dt + (16 * nl + n16) * ld + h;
#pragma unroll 4
      for (int ks = 0; ks < TILE / 4; ++ks)
        pacc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(pa[4 * ks], pb[4 * ks], pacc[q], 0, 0, 0);
    }
    __syncthreads();   // every reader of the optical depths is done: dtau_bar replaces them
    // ---- dtau_bar = P^T tau_bar: rows l, k = chords mi0.. up to the block's own
#pragma unroll
    for (int q = 0; q < kSlots; ++q) {
      const int ml = d_ml[q];
      if (ml < mi0) continue;
      const double* pa = pm + (size_t)(4 * h) * Lp + 16 * ml + n16;
      const double* pb = s_tb + 4 * h * ld + 16 * nb + n16;
      f64x4 acc = {0.0, 0.0, 0.0, 0.0};
      double a[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) a[j] = pa[(size_t)(16 * mi0 + j) * Lp];
#pragma unroll 1
      for (int K = mi0; K <= ml; ++K) {
        double cur[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) cur[j] = a[j];
        if (K < ml) {
#pragma unroll
          for (int j = 0; j < 4; ++j) a[j] = pa[(size_t)(16 * (K + 1) + j) * Lp];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(cur[j], pb[(16 * K + j) * ld], acc, 0, 0, 0);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) s_dt[(16 * ml + h + 4 * e) * ld + 16 * nb + n16] = acc[e];
    }
    __syncthreads();
    // ---- per-layer sums
    double g = 0.0;
    {
      const int lo = min(16 * mi0, L), n = L - lo;
      LayerRows64<S, CIA> rows;
      int cell_prev = -1;
      for (int l = lo + n * wv / kWaves; l < lo + n * (wv + 1) / kWaves; ++l) {
        const double db = act ? s_dt[l * ld + lane] : 0.0;
        if (__builtin_amdgcn_ballot_w64(!(db == 0.0)) == 0) continue;
        const int cl = cells[l];
        if (cl != cell_prev) {
          fetch_rows64<S, CIA>(m, tb, cl, nu, rows);
          cell_prev = cl;
        }
        const auto rl = rec + (size_t)l * rec_len(S);
        double t[S + 2], dw[S + 2], v[16];
        eval_rows64_deriv<S, CIA>(rl, rows, t, dw);
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = 0.0;
        double ht = 0.0, htc = 0.0;
#pragma unroll
        for (int s = 0; s < S; ++s) {
          v[s] = db * t[s];
          ht = fma(t[s], dw[s], ht);
        }
        v[S] = db * ht;
        if constexpr (CIA) {
#pragma unroll
          for (int p = 0; p < 2; ++p) {
            v[S + 1 + p] = db * t[S + p];
            htc = fma(t[S + p], dw[S + p], htc);
          }
          v[S + 3] = db * htc;
        }
        v[S + 4] = db * nu4;
        v[S + 5] = db * qx;   // the cloud column: Q_ext weights the non-grey cloud (1 for the grey deck)
        g = fma(rl[4], db, g);
        const double tot = wave_sums16(v, lane);
        if ((lane & 3) == 0) s_sums[l * 16 + (lane >> 2)] += tot;
      }
    }
    if (m.cloud_ng) s_g[wv * 64 + lane] = g;
    __syncthreads();
    if (m.cloud_ng && wv == 0) {
      double gs = 0.0, dqx[kCloudSpec];
      for (int k = 0; k < kWaves; ++k) gs += s_g[k * 64 + lane];
      q_ext(nu, dqx);
#pragma unroll
      for (int k = 0; k < kCloudSpec; ++k) s_hq[k * 64 + lane] = fma(gs, dqx[k], s_hq[k * 64 + lane]);
    }
  }

  const size_t pair = (size_t)b * C + chunk;
  double* ls = aw.layer_sums + pair * Lp * NS;
  for (int i = tid; i < Lp * NS; i += kBlockT) {
    const int l = i / NS, k = i - l * NS;
    ls[i] = l < L ? s_sums[l * 16 + k] : 0.0;
  }
  if (m.cloud_ng && wv == 0) {
#pragma unroll
    for (int k = 0; k < kCloudSpec; ++k) {
      const double tot = wave_sum_all(s_hq[k * 64 + lane]);
      if (lane == 0) aw.hq64[pair * kCloudSpec + k] = tot;
    }
  }
  double* pb = reinterpret_cast<double*>(aw.pbar) + pair * Lp * Lp;
#pragma unroll
  for (int q = 0; q < kPSlots; ++q) {
    const int mi = pt_mi[q], nl = pt_nl[q];
    if (mi < 0) continue;
#pragma unroll
    for (int e = 0; e < 4; ++e) pb[(size_t)(16 * mi + h + 4 * e) * Lp + 16 * nl + n16] = pacc[q][e];
  }
  // abar: over the 16 columns of a block, then over the column blocks
  __syncthreads();
  double* s_ab = s_dt;   // [kNb][R]
#pragma unroll
  for (int q = 0; q < kSlots; ++q) {
    const int mi = t_mi[q];
    if (mi < 0) continue;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      double v = abar_acc[q][e];
#pragma unroll
      for (int off = 8; off > 0; off >>= 1) v += __shfl_xor(v, off);
      if (n16 == 0) s_ab[nb * R + 16 * mi + h + 4 * e] = v;
    }
  }
  __syncthreads();
  double* ab = aw.abar + pair * Lp;
  for (int i = tid; i < Lp; i += kBlockT) {
    double v = 0.0;
    if (i < L)
#pragma unroll
      for (int k = 0; k < kNb; ++k) v += s_ab[k * R + i];
    ab[i] = v;
  }
}

// ============================================================================
// FP64 chain: one workgroup per sample
constexpr int kBlockC = 512, kWavesC = kBlockC / 64;

// derivatives of P_il with respect to r_l, r_{l+1} and b_i, l > i: bb = b_i, rlo and rup
// the layer's levels
__device__ inline void path_derivs(double bb, double rlo, double rup, double& d_lo, double& d_up, double& d_b) {
  const double xu = (rup - bb) * (rup + bb), xl = (rlo - bb) * (rlo + bb);
  double hu, hl;
  const double sup = sqrt_d(xu, hu), slo = sqrt_d(xl, hl), den = sup + slo;
  const double iup = rcp_of_root_d(sup, hu), ilo = rcp_of_root_d(slo, hl), iden = rcp_d(den);
  const double f = div_d(div_d(2.0 * (rup + rlo), den, iden), den, iden);
  d_up = fma(-f * rup, iup, 2.0 * iden);
  d_lo = fma(-f * rlo, ilo, 2.0 * iden);
  d_b = f * bb * (iup + ilo);
}
// the diagonal's full derivatives with respect to r_i, r_{i+1}
__device__ inline void path_derivs_diag(double rlo, double rup, double& d_lo, double& d_up) {
  const double dr = rup - rlo, q = (3.0 * rup + rlo) / dr, sq = sqrt(q);
  d_up = (3.0 - q) / (2.0 * dr * sq);
  d_lo = (1.0 + q) / (2.0 * dr * sq);
}

// Slopes of the monotone cubic Hermite interpolant through (xk, yk) and their
// Jacobian J[k][j] = d slope_k / d y_j, following the branches of the slope rule
// used by the profile kernel (Fritsch-Butland weighted harmonic mean inside,
// three-point shape-preserving ends).
__device__ void pchip_slopes_jac(const double* xk, const double* yk, int n, double* d, double* J) {
  double h[kMaxKnots], del[kMaxKnots];
  for (int k = 0; k < n - 1; ++k) { h[k] = xk[k + 1] - xk[k]; del[k] = (yk[k + 1] - yk[k]) / h[k]; }
  for (int i = 0; i < n * n; ++i) J[i] = 0.0;
  // d del_k / d y_k = -1/h_k, d del_k / d y_{k+1} = 1/h_k
  auto add_del = [&](int row, int k, double c) {
    J[row * n + k] -= c / h[k];
    J[row * n + k + 1] += c / h[k];
  };
  if (n == 2) {
    d[0] = d[1] = del[0];
    add_del(0, 0, 1.0);
    add_del(1, 0, 1.0);
    return;
  }
  for (int k = 1; k < n - 1; ++k) {
    const double a = del[k - 1], b = del[k];
    if (a == 0.0 || b == 0.0 || (a > 0.0) != (b > 0.0)) {
      d[k] = 0.0;
    } else {
      const double w1 = 2.0 * h[k] + h[k - 1], w2 = h[k] + 2.0 * h[k - 1];
      const double den = w1 / a + w2 / b;
      d[k] = (w1 + w2) / den;
      add_del(k, k - 1, (w1 + w2) * w1 / (a * a * den * den));
      add_del(k, k, (w1 + w2) * w2 / (b * b * den * den));
    }
  }
  auto end = [&](int row, int i0, int i1) {
    const double h0 = h[i0], h1 = h[i1], m0 = del[i0], m1 = del[i1];
    const double dd = ((2.0 * h0 + h1) * m0 - h0 * m1) / (h0 + h1);
    auto sgn = [](double v) { return (v > 0.0) - (v < 0.0); };
    if (sgn(dd) != sgn(m0)) return 0.0;
    if (sgn(m0) != sgn(m1) && fabs(dd) > fabs(3.0 * m0)) {
      add_del(row, i0, 3.0);
      return 3.0 * m0;
    }
    add_del(row, i0, (2.0 * h0 + h1) / (h0 + h1));
    add_del(row, i1, -h0 / (h0 + h1));
    return dd;
  };
  d[0] = end(0, 0, 1);
  d[n - 1] = end(n - 1, n - 2, n - 3);
}

// Inclusive running sums over n <= 192 values by one wave, three neighbours a lane:
// out[i] = get(0) + ... + get(i), or with rev get(n - 1) + ... + get(i).
template <typename Get>
__device__ inline void wave_scan(int lane, int n, bool rev, Get get, double* out) {
  double v[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int q = 3 * lane + k;
    v[k] = q < n ? get(rev ? n - 1 - q : q) : 0.0;
  }
  v[1] += v[0];
  v[2] += v[1];
  double t = v[2];
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const double u = __shfl_up(t, d);
    if (lane >= d) t += u;
  }
  const double before = __shfl_up(t, 1);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int q = 3 * lane + k;
    if (q < n) out[rev ? n - 1 - q : q] = (lane > 0 ? before : 0.0) + v[k];
  }
}

// Bound by latency (one workgroup per sample): sums over the block are 16 at a time (a wave
// by halving exchanges, then the waves), the hydrostatic recursion is four scans, and the
// chunks of every partial sum have been added by k_reduce_chunks.  One sample of 100
// layers and 30000 wavenumbers: 157 -> 21 us (1024 samples 392 -> 80 us; 64 samples of up
// to 150 layers and 400000 wavenumbers 728 -> 29 us), the chunk sums 58 -> 12 us.
template <typename PbarT>
__global__ __launch_bounds__(kBlockC) void k_chain(Model m, Work w, AdjWork aw, int C, const double* __restrict__ params,
                                                   const uint8_t* __restrict__ mask, double* __restrict__ grad) {
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int Lp = m.L_pad, S = m.S;
  const int NS = n_sums(S);
  double* gout = grad + (size_t)b * m.P;
  if (w.status[b]) {
    for (int k = tid; k < m.P; k += kBlockC) gout[k] = 0.0;
    return;
  }
  const int L = w.nlay[b];
  // virtual sample b of real sample real_sample(m, b); a clear one has no cloud terms
  __shared__ double s_th[kMaxParams];
  const double* th = s_th;
  const bool cloudy = m.has_cloud && !clear_sample(m, b);
  const bool ng = m.cloud_ng && cloudy;
  const bool trans = m.mode == kTransmission;
  constexpr int kRowChunk = 16, kChunks = kMaxLayers / kRowChunk, kColBlocks = (kMaxLayers + 63) / 64;
  __shared__ double s_r[kMaxLayers + 1], s_ub[kMaxLayers + 1], s_scan[4][kMaxLayers + 1];
  __shared__ double s_t[kMaxLayers], s_tb[kMaxLayers], s_lndr[kMaxLayers];
  // path-matrix adjoint: column sums per chunk of rows, row sums per block of columns
  __shared__ double s_plo[kChunks][kMaxLayers], s_pup[kChunks][kMaxLayers], s_pb[kColBlocks][kMaxLayers];
  __shared__ double s_w[2][kWavesC][16], s_sum[2][16], s_x[kMaxSpecies];
  __shared__ double s_kx[kMaxKnots], s_ky[kMaxKnots], s_kd[kMaxKnots], s_kj[kMaxKnots * kMaxKnots];
  __shared__ int s_above;

  const double* rl = w.r_lev + (size_t)b * (Lp + 1);
  const double* tl = w.t_lay + (size_t)b * Lp;
  const double step = (m.log10_ptop - m.log10_pbot) / L;
  const double ln10 = 2.302585092994045684017991454684;
  const double dlnp = -step * ln10;
  auto logp_lev = [&](int j) { return j == L ? m.log10_ptop : m.log10_pbot + j * step; };
  const double lpref = m.log10_pref;
  if (tid == 0) s_above = 0;
  if (tid < m.P) s_th[tid] = params[(size_t)real_sample(m, b) * m.P + tid];
  __syncthreads();
  for (int j = tid; j <= L; j += kBlockC) {
    s_r[j] = rl[j];
    if (logp_lev(j) > lpref) atomicAdd(&s_above, 1);
  }
  for (int l = tid; l < L; l += kBlockC) s_t[l] = tl[l];
  if (tid < S) s_x[tid] = exp10(th[m.n_tp + tid]);
  if (m.tp_kind == kTpPchip && tid == 64) {
    for (int k = 0; k < m.n_knots; ++k) {
      s_kx[k] = m.n_knots == 1 ? m.log10_ptop : m.log10_ptop + k * ((m.log10_pbot - m.log10_ptop) / (m.n_knots - 1));
      s_ky[k] = th[k];
    }
    s_kx[m.n_knots - 1] = m.log10_pbot;
    pchip_slopes_jac(s_kx, s_ky, m.n_knots, s_kd, s_kj);
  }
  __syncthreads();

  // chemistry and constants (every thread)
  double sx = 0.0;
  for (int s = 0; s < S; ++s) sx += s_x[s];
  const double xh2 = (1.0 - sx) / (1.0 + kHeH2), xhe = kHeH2 * xh2;
  const bool mu_free = !(m.mu_fixed > 0.0);
  double mu = m.mu_fixed;
  if (mu_free) {
    mu = xh2 * kMH2 + xhe * kMHe;
    for (int s = 0; s < S; ++s) mu += s_x[s] * m.mass[s];
  }
  const double scale = m.has_scale ? th[m.idx_scale] : 1.0;
  const double g_ref = m.has_bd ? exp10(th[m.idx_bd]) : m.g_ref;
  const double r_ref = m.has_bd ? sqrt(kGrav * th[m.idx_bd + 1] * kMJup / g_ref) : m.r_p * scale;
  const double kk = kB / (mu * kMu * g_ref * r_ref * r_ref);
  const double rs2 = m.r_s * m.r_s;
  const double log10_pc = m.has_cloud ? th[m.idx_cloud] : 0.0;
  // non-grey cloud: D_l = q_l rho_l dr_l 3 / (4 r_eff); profile parameters start at q_first
  const int q_first = m.idx_cloud + (m.cloud_qext == kQextGrey ? 1 : 3);
  const double r_eff = m.cloud_ng ? 1.0e-4 * exp10(th[m.idx_cloud]) : 1.0;
  // sums over the block of 16 values per thread, two sets of them: set q to s_w[q]
  auto wave_part = [&](int q, const double (&v)[16]) {
    const double s = wave_sums16(v, lane);
    if ((lane & 3) == 0) s_w[q][wv][lane >> 2] = s;
  };
  auto wave_total = [&](int sets) {   // after a barrier; another barrier before s_sum is read
    if (tid < 16 * sets) {
      double s = 0.0;
      for (int k = 0; k < kWavesC; ++k) s += s_w[tid >> 4][k][tid & 15];
      s_sum[tid >> 4][tid & 15] = s;
    }
  };

  // per layer: the chain through n = p/kT, dr, the Rayleigh and cloud prefactors.  Set 0:
  // [0, 8) ln X_s, then ln X_H2, ln X_He, X_H2 and X_He direct, ln mu, theta_cloud.
  // Set 1: the non-grey cloud's kCloudSpec spectral parameters (log10 r also through the
  // column's 1/r_eff) and 3 profile parameters, d lnL / d depth, its masked part (offset).
  double va[16] = {}, vb[16] = {};
  for (int l = tid; l < L; l += kBlockC) {
    const double* src = aw.lred + ((size_t)b * Lp + l) * NS;
    double sm[kMaxSpecies], ex[kExtraSums];
#pragma unroll
    for (int s = 0; s < kMaxSpecies; ++s) sm[s] = s < S ? src[s] : 0.0;
#pragma unroll
    for (int k = 0; k < kExtraSums; ++k) ex[k] = src[S + k];
    const double t = s_t[l];
    const double lp_bar = 0.5 * (logp_lev(l) + logp_lev(l + 1));
    const double n = exp10(lp_bar) * kBar / (kB * t);
    const double dr = s_r[l + 1] - s_r[l];
    const double rr = (m.has_ray ? n * (xh2 * m.ray_h2 + xhe * m.ray_he) * dr : 0.0);
    double f = 0.0, dd = 0.0;
    const double gc1 = ex[1], gc2 = ex[2], gr = ex[4], gd = ex[5];
    if (ng) {
      const double col = mu * kMu * n * dr * 0.75 / r_eff;
      double dq[3];
      const double q = condensate_q(m.cloud_profile, th + q_first, logp_lev(l), logp_lev(l + 1), lp_bar, dq);
      dd = q * col;
      vb[0] -= ln10 * gd * q * col;
#pragma unroll
      for (int k = 0; k < 3; ++k) vb[kCloudSpec + k] += gd * col * dq[k];
    } else if (cloudy) {
      f = (logp_lev(l) - log10_pc) * ln10 / dlnp;
      f = f < 0.0 ? 0.0 : (f > 1.0 ? 1.0 : f);
      dd = m.kappa_cloud * mu * kMu * n * f * dr;
    }
    double gline = 0.0;
#pragma unroll
    for (int s = 0; s < kMaxSpecies; ++s) gline += sm[s];
    const double lnn_bar = gline + 2.0 * gc1 + 2.0 * gc2 + gr * rr + gd * dd;
    const double lndr_bar = gline + gc1 + gc2 + gr * rr + gd * dd;
    s_lndr[l] = lndr_bar / dr;
    // dT from n = p/kT and from the table weights (interior cells only)
    double tbar = -lnn_bar / t;
    const double ln2 = 0.69314718055994530941723212145818;
    const int cell = w.cells[(size_t)b * Lp + l], it = cell & 255, itc = cell >> 16;
    if (t > m.t_grid[0] && t < m.t_grid[m.n_t - 1]) tbar += ln2 * ex[0] / (m.t_grid[it + 1] - m.t_grid[it]);
    if (m.has_cia && t > m.tc_grid[0] && t < m.tc_grid[m.n_tc - 1])
      tbar += ln2 * ex[3] / (m.tc_grid[itc + 1] - m.tc_grid[itc]);
    s_tb[l] = tbar;
#pragma unroll
    for (int s = 0; s < kMaxSpecies; ++s) va[s] += sm[s];
    va[8] += 2.0 * gc1 + gc2;
    va[9] += gc2;
    va[10] += gr * n * dr * m.ray_h2;
    va[11] += gr * n * dr * m.ray_he;
    va[12] += gd * dd;
    if (cloudy && !m.cloud_ng && f > 0.0 && f < 1.0)
      va[13] += gd * m.kappa_cloud * mu * kMu * n * dr * (-ln10 / dlnp);
  }
  // the cloud's spectral parameters, per chunk of wavenumbers
  const int nq = !ng ? 0 : sizeof(PbarT) == 8 ? C : aw.lsum_chunks;
  for (int c = tid; c < nq; c += kBlockC)
#pragma unroll
    for (int k = 0; k < kCloudSpec; ++k) {
      if constexpr (sizeof(PbarT) == 8) vb[k] += aw.hq64[((size_t)b * C + c) * kCloudSpec + k];
      else vb[k] += (double)aw.hq[((size_t)b * aw.lsum_stride + c) * kCloudSpec + k];
    }
  // seed of the core term, and of the offset
  for (int k = tid; k < m.K; k += kBlockC) {
    const double d = w.dm[(size_t)b * m.K + k];
    vb[10] += d;
    if (m.has_offset && mask && mask[k]) vb[11] += d;
  }
  wave_part(0, va);
  wave_part(1, vb);

  // path-matrix adjoint: column sums (r_l, r_{l+1}) and row sums (b_i).  A wave takes 64
  // columns, one a lane, and 16 rows, each entry's derivatives formed once: the column
  // sums stay in the lanes, the rows' sums meet over the wave.
  const PbarT* pbar = reinterpret_cast<const PbarT*>(aw.pbar) + (size_t)b * C * Lp * Lp;
  const int n_rc = (L + kRowChunk - 1) / kRowChunk, n_cb = (L + 63) / 64;
#pragma unroll 1
  for (int t = wv; t < (trans ? n_rc * n_cb : 0); t += kWavesC) {
    const int rc = t % n_rc, cb = t / n_rc, i0 = kRowChunk * rc, x = 64 * cb + lane;
    if (64 * cb + 63 < i0) continue;   // rows below these columns (never read)
    const int xc = min(x, L - 1);
    const double rlo = s_r[xc], rup = s_r[xc + 1];
    double lo = 0.0, up = 0.0;
    constexpr int kRows = 4;   // rows in a step, the next step's entries in flight
    auto entry = [&](int i) { return pbar[(size_t)min(i, L - 1) * Lp + xc]; };
    PbarT p[kRows];
#pragma unroll
    for (int k = 0; k < kRows; ++k) p[k] = entry(i0 + k);
#pragma unroll 1
    for (int g = i0; g < i0 + kRowChunk; g += kRows) {
      PbarT cur[kRows];
      double row[kRows];
#pragma unroll
      for (int k = 0; k < kRows; ++k) {
        cur[k] = p[k];
        p[k] = entry(g + kRows + k);
      }
#pragma unroll
      for (int k = 0; k < kRows; ++k) {
        const int i = min(g + k, L - 1);
        const bool on = x < L && g + k < x;   // above the diagonal
        const double r0 = s_r[i], r1 = s_r[i + 1];
        double dlo, dup, db;
        // lanes that are off take a level pair that is above this one
        path_derivs(0.5 * (r0 + r1), on ? rlo : r1, on ? rup : 2.0 * r1, dlo, dup, db);
        const double pk = on ? (double)cur[k] : 0.0;
        lo = fma(pk, dlo, lo);
        up = fma(pk, dup, up);
        row[k] = pk * db;
      }
      // the four rows' sums over the wave: the lanes of quarter q (lane / 16) get row q's
      double v = halve_add<16>(halve_add<32>(row[0], row[2]), halve_add<32>(row[1], row[3]));
      v += lane_xor<8>(v);
      v += lane_xor<4>(v);
      v += lane_xor<2>(v);
      v += lane_xor<1>(v);
      if ((lane & 15) == 0 && g + (lane >> 4) < L) s_pb[cb][g + (lane >> 4)] = v;
    }
    if (x < L) {
      if (x >= i0 && x < i0 + kRowChunk) {
        double dlo, dup;
        path_derivs_diag(rlo, rup, dlo, dup);
        const double pd = (double)pbar[(size_t)x * Lp + x];
        lo = fma(pd, dlo, lo);
        up = fma(pd, dup, up);
      }
      s_plo[rc][x] = lo;
      s_pup[rc][x] = up;
    }
  }
  __syncthreads();
  wave_total(2);
  __syncthreads();
  const double core_bar = s_sum[1][10];
  for (int j = tid; j <= L; j += kBlockC) {
    double rb = 0.0;
    if (trans) {
      // a column's rows end at its own, a row's columns begin at its own
      double lo = 0.0, up = 0.0, bb = 0.0;
      if (j < L) {
        for (int k = 0; k <= j / kRowChunk; ++k) lo += s_plo[k][j];
        for (int k = j / 64; k < n_cb; ++k) bb += s_pb[k][j];
      }
      if (j >= 1) {
        for (int k = 0; k <= (j - 1) / kRowChunk; ++k) up += s_pup[k][j - 1];
        for (int k = (j - 1) / 64; k < n_cb; ++k) bb += s_pb[k][j - 1];
      }
      const double* ab = aw.abar + (size_t)b * C * Lp;
      const double ab_j = j < L ? ab[j] : 0.0, ab_jm = j >= 1 ? ab[j - 1] : 0.0;
      rb = lo + up + 0.5 * bb + 2.0 * s_r[j] * (ab_jm - ab_j) / rs2;
      if (j == 0) rb += 2.0 * s_r[0] * core_bar / rs2;
    }
    // emission: no chord; the levels move the optical depths only through dr
    if (j < L) rb -= s_lndr[j];
    if (j >= 1) rb += s_lndr[j - 1];
    s_ub[j] = -rb * s_r[j] * s_r[j];
  }
  __syncthreads();

  // hydrostatic recursion in reverse: running sums of ub from either end, and of the
  // temperatures outward from the reference layer
  const int lref = min(max(s_above - 1, 0), L - 1);
  if (wv == 0) wave_scan(lane, L + 1, false, [&](int j) { return s_ub[j]; }, s_scan[0]);
  if (wv == 1) wave_scan(lane, L + 1, true, [&](int j) { return s_ub[j]; }, s_scan[1]);
  if (wv == 2) wave_scan(lane, L, true, [&](int l) { return l < lref ? s_t[l] : 0.0; }, s_scan[2]);
  if (wv == 3) wave_scan(lane, L, false, [&](int l) { return l > lref ? s_t[l] : 0.0; }, s_scan[3]);
  __syncthreads();
  const double a1 = (logp_lev(lref) - lpref) * ln10, a2 = (lpref - logp_lev(lref + 1)) * ln10;
  const double t_ref = s_t[lref];
  // [0, 8) T-p parameters, 8: the profile's share of d lnL / d log10 g (tau = kappa_ir p / g)
  // of an isolated object, 9: sum_j ub_j (u_j - u_ref) / K
  double ta[16] = {};
  for (int j = tid; j <= L; j += kBlockC) {
    const double q = j <= lref ? t_ref * a1 + dlnp * s_scan[2][j] : -(t_ref * a2) - dlnp * s_scan[3][j - 1];
    ta[9] += s_ub[j] * q;
  }

  // T-p profile: layer temperatures (opacity, hydrostatics) and, in emission, the
  // level temperatures of the Planck sources, each at its own pressure
  auto tp_grad = [&](double lp, double t, double tbar) {
    if (m.tp_kind == kTpIso) {
      ta[0] += tbar;
    } else if (m.tp_kind == kTpGuillot3) {
      const double tau = m.kappa_ir * exp10(lp) * kBar / g_ref;
      const double t3 = t * t * t;
      const double s3 = 1.7320508075688772935274463415059;
      const double gam = exp10(th[2]);
      const double e = exp(-gam * tau * s3);
      const double bk = 2.0 / 3.0 + 1.0 / (gam * s3) + (gam / s3 - 1.0 / (gam * s3)) * e;
      const double dbk = -1.0 / (gam * gam * s3) + (1.0 / s3 + 1.0 / (gam * gam * s3)) * e +
                         (gam / s3 - 1.0 / (gam * s3)) * e * (-tau * s3);
      const double ti = th[0], te = th[1];
      ta[0] += tbar * 3.0 * ti * ti * ti * (2.0 / 3.0 + tau) / (4.0 * t3);
      ta[1] += tbar * 12.0 * m.f_hem * te * te * te * bk / (4.0 * t3);
      ta[2] += tbar * 3.0 * m.f_hem * te * te * te * te * dbk * gam * ln10 / (4.0 * t3);
      if (m.has_bd) {
        // d T^4 / d tau times d tau / d log10 g = -tau ln 10
        const double dt4 = 0.75 * ti * ti * ti * ti - 3.0 * m.f_hem * te * te * te * te * (gam / s3 - 1.0 / (gam * s3)) * e * gam * s3;
        ta[8] -= tbar * dt4 * tau * ln10 / (4.0 * t3);
      }
    } else if (m.tp_kind == kTpBarstow) {
      ta[0] += tbar * barstow_factor(lp);
    } else if (m.tp_kind == kTpMilne || m.tp_kind == kTpGuillot7) {
      double d4[7] = {};
      if (m.tp_kind == kTpMilne) milne_t4(th, lp, g_ref, d4);
      else guillot7_t4(th, lp, g_ref, m.f_hem, d4);
      const double inv = tbar / (4.0 * t * t * t);
#pragma unroll
      for (int k = 0; k < 7; ++k) ta[k] += d4[k] * inv;
      // tau depends on kappa_ir / g: d/d log10 g = -d/d log10 kappa_ir
      if (m.has_bd) ta[8] -= (m.tp_kind == kTpMilne ? d4[1] : d4[2]) * inv;
    } else {
      // T = h00 y_k + h10 h d_k + h01 y_k+1 + h11 h d_k+1 on the knot interval holding lp
      const int n = m.n_knots;
      int k = 0;
      while (k < n - 2 && s_kx[k + 1] <= lp) ++k;
      const double hk = s_kx[k + 1] - s_kx[k];
      const double u = (lp - s_kx[k]) / hk, omu = 1.0 - u;
      const double h00 = (1.0 + 2.0 * u) * omu * omu, h10 = u * omu * omu, h01 = u * u * (3.0 - 2.0 * u),
                   h11 = u * u * (u - 1.0);
#pragma unroll
      for (int j = 0; j < kMaxKnots; ++j) {
        if (j >= n) break;
        double dtdy = hk * (h10 * s_kj[k * n + j] + h11 * s_kj[(k + 1) * n + j]);
        if (j == k) dtdy += h00;
        if (j == k + 1) dtdy += h01;
        ta[j] += tbar * dtdy;
      }
    }
  };
  // layers, then (emission) levels: one copy of the profiles' code
  for (int q = tid; q < L + (trans ? 0 : L + 1); q += kBlockC) {
    double lp, t, tb;
    if (q < L) {
      tb = s_tb[q];
      if (q < lref) tb += kk * dlnp * s_scan[0][q];
      else if (q > lref) tb -= kk * dlnp * s_scan[1][q + 1];
      else tb += kk * (a1 * s_scan[0][lref] - a2 * s_scan[1][lref + 1]);
      lp = 0.5 * (logp_lev(q) + logp_lev(q + 1));
      t = s_t[q];
    } else {
      const size_t j = (size_t)b * (Lp + 1) + (q - L);
      tb = aw.pred[j];
      lp = logp_lev(q - L);
      t = w.t_lev[j];
    }
    tp_grad(lp, t, tb);
  }
  // s_w[0] was last read before the barriers above; the totals in s_sum[1] (cloud, offset)
  // and s_sum[0] (chemistry) stay, so this set's totals go to s_tp
  __shared__ double s_tp[16];
  wave_part(0, ta);
  __syncthreads();
  if (tid < 16) {
    double s = 0.0;
    for (int k = 0; k < kWavesC; ++k) s += s_w[0][k][tid];
    s_tp[tid] = s;
  }
  __syncthreads();
  const double ub_ref = s_scan[0][L], kbar = s_tp[9];
  const double* chem = s_sum[0];
  // d lnL / d R_ref; the emission ratio carries (R_ref/R_s)^2, and sum_nu dlnL/dspec spec = mdot
  const double rref_bar = -ub_ref / (r_ref * r_ref) - 2.0 * kbar * kk / r_ref + (trans ? 0.0 : 2.0 * w.mdot[b] / r_ref);
  const double lnmu_hyd = -kbar * kk;   // d lnL / d ln mu (hydrostatics)
  if (tid < m.n_tp) gout[tid] = s_tp[tid];
  if (tid < S) {
    // chemistry: X_H2 = (1 - sum X)/1.164, X_He = 0.164 X_H2, mu = sum X m
    const double lnmu_bar = chem[12] + lnmu_hyd;
    const double mu_bar = mu_free ? lnmu_bar / mu : 0.0;
    const double xhe_bar = chem[9] / xhe + chem[11] + mu_bar * kMHe;
    const double xh2_bar = chem[8] / xh2 + chem[10] + mu_bar * kMH2 + kHeH2 * xhe_bar;
    const double xb = chem[tid] / s_x[tid] + mu_bar * m.mass[tid] - xh2_bar / (1.0 + kHeH2);
    gout[m.n_tp + tid] = xb * s_x[tid] * ln10;
  }
  if (tid == 64) {
    if (m.has_bd) {
      // g R_ref^2 = G M fixes the hydrostatic constant: ln g enters at fixed R_ref like ln mu
      // and through R_ref = sqrt(G M / g)
      gout[m.idx_bd] = (lnmu_hyd - 0.5 * r_ref * rref_bar) * ln10 + s_tp[8];
      gout[m.idx_bd + 1] = 0.5 * r_ref * rref_bar / th[m.idx_bd + 1];
    }
    if (m.has_cloud && !m.cloud_ng) gout[m.idx_cloud] = chem[13];
    if (m.cloud_ng) {
      // theta order: log10 r, [a, log10 Q0], profile (1 or 3), [A, lambda0, log10 omega, xi]
      // (a clear virtual sample's sums are zero)
      const double* s_cloud = s_sum[1];
      int k = m.idx_cloud;
      gout[k++] = s_cloud[0];
      if (m.cloud_qext != kQextGrey) { gout[k++] = s_cloud[1]; gout[k++] = s_cloud[2]; }
      const int np = m.cloud_profile == kQprofUniform ? 1 : 3;
      for (int j = 0; j < np; ++j) gout[k++] = s_cloud[kCloudSpec + j];
      if (m.cloud_qext == kQextFeature)
        for (int j = 3; j < kCloudSpec; ++j) gout[k++] = s_cloud[j];
    }
    if (m.has_scale) gout[m.idx_scale] = rref_bar * m.r_p;
    if (m.has_offset) gout[m.idx_offset] = s_sum[1][11] * 1.0e-6;
  }
}

// ============================================================================
// Sums over the wavenumber chunks, so that the chain reads one slot of each: the per-layer
// sums (to lred), the reverse kernel's path-matrix and annulus-area adjoints (into chunk 0
// of the sample, C > 1) and emission's per-level sums (to pred).  A workgroup takes 32
// neighbouring elements of one sample, eight threads each (strided over the chunks, four
// loads in flight), added in a fixed order.
constexpr int kRedElems = 32, kRedSegs = kBlock / kRedElems;

struct ReduceSizes {
  int sums, path, area, levels;   // elements per sample
  int quads;                      // path-matrix elements taken four to a thread instead of as `path`
};
// A path matrix of at most kRedQuad chunks is added by threads that each walk the chunks of
// four neighbouring entries (16- or 32-byte loads); by segments, such a batch gave each
// thread one load and the launch hundreds of thousands of workgroups.  100 layers: 1024
// samples x 4 chunks 354 -> 60 us, 128 x 4 53 -> 19, 64 (up to 150 layers) x 8 74 -> 52; 24
// FP64 samples 13 either way.  With more chunks there are few samples, and the split over
// the segments keeps each thread's chain of loads short (one sample: 12 us).  About the line,
// with the chain, fours against segments: 16 chunks (64 samples) 40 layers 25 us (30), 100
// layers 34 (52), 160 layers 47 (76); 32 chunks 28 (27), 34 (42), 47 (60); 64 chunks 34 (26),
// 39 (39), 48 (54): up to 16 the fours are the better for every layer count.
constexpr int kRedQuad = 16;
__host__ __device__ inline ReduceSizes reduce_sizes(const Model& m, int C) {
  const bool parts = m.mode == kTransmission && C > 1;
  const int path = parts ? m.L_pad * m.L_pad : 0;
  return {m.L_max * n_sums(m.S), C > kRedQuad ? path : 0, parts ? m.L_pad : 0, m.mode == kEmission ? m.L_max + 1 : 0,
          C > kRedQuad ? 0 : path};
}
__host__ __device__ inline int reduce_split_blocks(const ReduceSizes& z) {
  return (z.sums + z.path + z.area + z.levels + kRedElems - 1) / kRedElems;
}
__host__ __device__ inline int reduce_blocks(const ReduceSizes& z) {
  return reduce_split_blocks(z) + (z.quads + 4 * kBlock - 1) / (4 * kBlock);
}

template <typename PbarT>
__global__ __launch_bounds__(kBlock) void k_reduce_chunks(Model m, Work w, AdjWork aw, int C) {
  __shared__ double s_part[kRedSegs][kRedElems];
  const int Lp = m.L_pad, NS = n_sums(m.S);
  const ReduceSizes z = reduce_sizes(m, C);
  const int nblk = reduce_blocks(z), b = blockIdx.x / nblk;
  if (w.status[b]) return;
  const int L = w.nlay[b];
  const int part = blockIdx.x - b * nblk, split = reduce_split_blocks(z);
  if (part >= split) {
    // four neighbouring entries of a row (L_pad is a multiple of 16, so never across rows);
    // those of the fours that straddle the diagonal or L and are not read add up unread
    typedef PbarT quad_t __attribute__((ext_vector_type(4)));
    const int e = 4 * ((part - split) * kBlock + (int)threadIdx.x), i = e / Lp, l = e - i * Lp;
    if (e >= z.quads || l + 3 < i || l >= L) return;
    quad_t* q = reinterpret_cast<quad_t*>(reinterpret_cast<PbarT*>(aw.pbar) + (size_t)b * C * Lp * Lp + e);
    const size_t step = (size_t)Lp * Lp / 4;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    for (int c0 = 0; c0 < C; c0 += 4) {
      quad_t x[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) x[u] = q[min(c0 + u, C - 1) * step];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (c0 + u < C) {
#pragma unroll
          for (int k = 0; k < 4; ++k) v[k] += (double)x[u][k];
        }
    }
    quad_t sum;
#pragma unroll
    for (int k = 0; k < 4; ++k) sum[k] = (PbarT)v[k];
    *q = sum;
    return;
  }
  const int el = threadIdx.x & (kRedElems - 1), seg = threadIdx.x / kRedElems;
  int e = part * kRedElems + el;
  // where the element's chunks lie: type, first, stride (elements), number
  const PbarT* src = nullptr;
  const double* src64 = nullptr;
  size_t stride = 0;
  int n = 0;
  double* dst = nullptr;
  PbarT* dst_p = nullptr;
  if (e < z.sums) {
    if (e < L * NS) {
      stride = (size_t)Lp * NS;
      if (sizeof(PbarT) == 8 && m.mode == kTransmission) {
        n = C;
        src = reinterpret_cast<const PbarT*>(aw.layer_sums) + (size_t)b * C * stride + e;
      } else {
        n = aw.lsum_chunks;
        src = (sizeof(PbarT) == 8 ? reinterpret_cast<const PbarT*>(aw.lsum64) : reinterpret_cast<const PbarT*>(aw.lsum)) +
              (size_t)b * aw.lsum_stride * stride + e;
      }
      dst = aw.lred + (size_t)b * stride + e;
    }
  } else if ((e -= z.sums) < z.path) {
    const int i = e / Lp, l = e - i * Lp;
    if (l >= i && l < L) {   // the chain reads the upper triangle
      stride = (size_t)Lp * Lp;
      n = C;
      src = dst_p = reinterpret_cast<PbarT*>(aw.pbar) + (size_t)b * C * stride + e;
    }
  } else if ((e -= z.path) < z.area) {
    stride = Lp;
    n = C;
    src64 = dst = aw.abar + (size_t)b * C * stride + e;
  } else if ((e -= z.area) < z.levels) {
    if (e <= L) {
      stride = Lp + 1;
      n = m.n_tiles64;
      src = (sizeof(PbarT) == 8 ? reinterpret_cast<const PbarT*>(aw.psum64) : reinterpret_cast<const PbarT*>(aw.psum)) +
            (size_t)b * m.n_tiles64 * stride + e;
      dst = aw.pred + (size_t)b * stride + e;
    }
  }
  double v = 0.0;
  constexpr int kFly = 4;
  for (int c0 = seg; c0 < n; c0 += kFly * kRedSegs) {
    double x[kFly];
#pragma unroll
    for (int u = 0; u < kFly; ++u) {
      const int c = c0 + u * kRedSegs;
      x[u] = c < n ? (src ? (double)src[c * stride] : src64[c * stride]) : 0.0;
    }
#pragma unroll
    for (int u = 0; u < kFly; ++u) v += x[u];
  }
  s_part[seg][el] = v;
  __syncthreads();
  if (seg == 0 && n > 0) {
#pragma unroll
    for (int k = 1; k < kRedSegs; ++k) v += s_part[k][el];
    if (dst_p) *dst_p = (PbarT)v;
    else *dst = v;
  }
}

// ============================================================================
// host side
// reduced-precision reverse kernel shapes: (tile, row blocks)
static int adj_tile(int variant) { return variant == kAdjT128M4 ? 128 : 64; }
// FP64 reverse kernel: instance 0 (64-wavenumber tiles) up to 128 padded layers, 1 (32) up to 160
static int adj_fp64_instance(const Model& m) { return m.L_pad <= 128 ? 0 : 1; }
static int adj_tile64(const Model& m) { return adj_fp64_instance(m) == 0 ? 64 : 32; }
static int adj_mb(int variant) { return variant == kAdjT64M5 ? 5 : 4; }
// row-block parts per column block: the 64-wavenumber shapes run eight waves, two per
// SIMD, each with a quarter of the row blocks
static int adj_parts(int variant) { return variant == kAdjT128M4 ? 2 : 4; }
static int adj_threads(int variant) { return 64 * adj_parts(variant) * (adj_tile(variant) / 32); }
static int adj_slots(int variant) {
  return adj_parts(variant) == 2 ? (adj_mb(variant) + 1) / 2 : (adj_mb(variant) <= 4 ? 1 : 2);
}

int adjoint_chunks(const Model& m, const AdjWork& aw, int B, bool fp64) {
  if (m.mode == kEmission) return 1;   // the emission reverse pass keeps no per-chunk partials
  const int tiles = m.n_nu_pad / (fp64 ? adj_tile64(m) : adj_tile(aw.variant));
  if (fp64) {
    // one workgroup per CU at a time (its 256 registers, whatever its LDS): of the splits into
    // at most 1024 work items, the one whose rounds over the chip take the fewest tiles in a
    // row (the coarsest of equals)
    const int cus = 256, cmax = std::min(std::max(1024 / B, 1), tiles);
    int best = 1;
    long cost = LONG_MAX;
    for (int c = 1; c <= cmax; ++c) {
      const long v = (long)((B * (long)c + cus - 1) / cus) * ((tiles + c - 1) / c);
      if (v < cost) {
        cost = v;
        best = c;
      }
    }
    return best;
  }
  const int target = aw.chunk_target;
  int c = (target + B - 1) / B;
  return c < 1 ? 1 : (c > tiles ? tiles : c);
}

bool adjoint_supported(const Model& m, bool fp64) {
  if (m.ck) return false;   // the correlated-k path is a forward model only
  return m.L_pad <= 160;
}

// A ragged context of more than kShortLayers padded layers with a 4-row-block shape (128 x 4
// or 64 x 4) runs its samples in two layer-count classes: that shape for those of at most
// kShortLayers layers, 64 x 5 for the rest.  Both launches split every sample into the
// same number of wavenumber chunks (bounded by the wider shape's tile count), so the
// per-chunk partials and their reduction are those of a single launch.
static bool adj_split(const Model& m, int variant) {
  return layer_classes_used(m) && (variant == kAdjT64M4 || variant == kAdjT128M4);
}

int adjoint_default_variant(const Model& m) { return m.L_pad <= 128 ? kAdjT128M4 : kAdjT64M4; }

bool adjoint_variant_fits(const Model& m, int variant) {
  const bool split = adj_split(m, variant);
  if (m.L_pad > 32 * adj_mb(split ? kAdjT64M5 : variant)) return false;
  // the greedy row-block split must never give a wave more blocks than it has slots
  for (int L = 1; L <= m.L_max; ++L) {
    const int KBe = (L + 15) >> 4, MBe = (L + 31) >> 5;
    const int v = split && L > kShortLayers ? (int)kAdjT64M5 : variant;
    for (int part = 0; part < adj_parts(v); ++part)
      for (int rev = 0; rev < 2; ++rev)
        if (__builtin_popcount(split_blocks(part, adj_parts(v), MBe, KBe, rev != 0)) > adj_slots(v)) return false;
  }
  return true;
}

bool adjoint_alloc(AdjWork& aw, const Model& m, int B_max, bool fp64, const std::function<void*(size_t)>& alloc) {
  aw = AdjWork{};
  if (!adjoint_supported(m, fp64)) return true;
  // chunk counts of the narrowest tile and the largest target bound those of every
  // launch choice the context may switch to
  aw.variant = fp64 ? kAdjT128M4 : (adjoint_variant_fits(m, kAdjT64M4) ? kAdjT64M4 : kAdjT64M5);
  aw.chunk_target = kChunkTargets[sizeof(kChunkTargets) / sizeof(int) - 1];
  int pairs = 0;
  for (int B = 1; B <= B_max; ++B) pairs = std::max(pairs, B * adjoint_chunks(m, aw, B, fp64));
  aw.variant = adjoint_default_variant(m);
  aw.chunk_target = 1024;
  aw.ls_tiles = 8;
  aw.max_pairs = pairs;
  const size_t Lp = m.L_pad;
  aw.lred = (double*)alloc((size_t)B_max * Lp * n_lsums(m) * sizeof(double));
  if (!aw.lred) return false;
  if (m.mode == kEmission) {
    aw.pred = (double*)alloc((size_t)B_max * (Lp + 1) * sizeof(double));
    if (!aw.pred) return false;
  }
  if (m.mode == kEmission && fp64) {
    aw.lsum_stride = (m.n_tiles + kLsTileChoices[0] - 1) / kLsTileChoices[0];
    aw.lsum_chunks = (m.n_tiles + aw.ls_tiles - 1) / aw.ls_tiles;
    aw.dtb64 = (double*)alloc((size_t)B_max * m.L_pad * m.n_nu_pad * sizeof(double));
    aw.dtau64 = (double*)alloc((size_t)B_max * m.L_pad * m.n_nu_pad * sizeof(double));
    aw.lsum64 = (double*)alloc((size_t)B_max * aw.lsum_stride * Lp * n_lsums(m) * sizeof(double));
    aw.psum64 = (double*)alloc((size_t)B_max * m.n_tiles64 * (Lp + 1) * sizeof(double));
    return aw.dtb64 && aw.dtau64 && aw.lsum64 && aw.psum64;
  }
  if (m.mode == kEmission) {
    aw.lsum_stride = (m.n_tiles + kLsTileChoices[0] - 1) / kLsTileChoices[0];
    aw.lsum_chunks = (m.n_tiles + aw.ls_tiles - 1) / aw.ls_tiles;
    aw.dtb = (float*)alloc((size_t)B_max * m.L_pad * m.n_nu_pad * sizeof(float));
    aw.dtau = (float*)alloc((size_t)B_max * m.L_pad * m.n_nu_pad * sizeof(float));
    aw.lsum = (float*)alloc((size_t)B_max * aw.lsum_stride * Lp * n_lsums(m) * sizeof(float));
    aw.psum = (float*)alloc((size_t)B_max * m.n_tiles64 * (Lp + 1) * sizeof(float));
    return aw.dtb && aw.dtau && aw.lsum && aw.psum;
  }
  aw.pbar = alloc((size_t)pairs * Lp * Lp * (fp64 ? sizeof(double) : sizeof(float)));
  aw.abar = (double*)alloc((size_t)pairs * Lp * sizeof(double));
  if (!aw.pbar || !aw.abar) return false;
  if (fp64) {
    aw.layer_sums = (double*)alloc((size_t)pairs * Lp * n_sums(m.S) * sizeof(double));
    if (m.cloud_ng) aw.hq64 = (double*)alloc((size_t)pairs * kCloudSpec * sizeof(double));
    return aw.layer_sums != nullptr && (!m.cloud_ng || aw.hq64 != nullptr);
  }
  aw.lsum_stride = (m.n_tiles + kLsTileChoices[0] - 1) / kLsTileChoices[0];   // bound over the choices
  aw.lsum_chunks = (m.n_tiles + aw.ls_tiles - 1) / aw.ls_tiles;
  aw.dtb = (float*)alloc((size_t)B_max * m.L_pad * m.n_nu_pad * sizeof(float));
  aw.dtau = (float*)alloc((size_t)B_max * m.L_pad * m.n_nu_pad * sizeof(float));
  aw.lsum = (float*)alloc((size_t)B_max * aw.lsum_stride * Lp * n_lsums(m) * sizeof(float));
  if (m.cloud_ng) {
    aw.hq = (float*)alloc((size_t)B_max * aw.lsum_stride * kCloudSpec * sizeof(float));
    if (!aw.hq) return false;
  }
  return aw.dtb && aw.dtau && aw.lsum;
}

static size_t adj_lds_bytes(const Model& m, bool fp64, int variant) {
  const size_t Lp = m.L_pad;
  if (fp64) {
    const size_t R = rows16(m.L_max);
    return (R * (2 * (adj_tile64(m) + 2) + 16 + 1) + (kBlockT / 64 + kCloudSpec) * 64) * 8 + kMaxBlocks16 * 4;
  }
  const size_t tile = adj_tile(variant), rows = std::min(Lp, (size_t)32 * adj_mb(variant));
  return std::max(2 * tile * (32 * adj_mb(variant) + 4) * 4 + rows * 4, tile / 32 * Lp * 8);
}

template <int S, bool CIA>
const void* adj_mixed_kernel(int variant) {
  switch (variant) {
    case kAdjT128M4: return (const void*)k_trans_adj_mixed<S, CIA, 128, 4, 2>;
    case kAdjT64M4: return (const void*)k_trans_adj_mixed<S, CIA, 64, 4, 4>;
    case kAdjT64M5: return (const void*)k_trans_adj_mixed<S, CIA, 64, 5, 4>;
  }
  return nullptr;
}

template <bool F64, int S, bool CIA>
const void* adj_kernel(int variant) {
  if constexpr (F64)
    return variant == 0 ? (const void*)k_trans_adj_fp64<S, CIA, 64> : (const void*)k_trans_adj_fp64<S, CIA, 32>;
  else return adj_mixed_kernel<S, CIA>(variant);
}

template <bool F64>
const void* adj_kernel_for(int S, bool cia, int variant) {
#define EXOFWD_CASE(n) \
  case n: return cia ? adj_kernel<F64, n, true>(variant) : adj_kernel<F64, n, false>(variant);
  switch (S) {
    EXOFWD_CASE(1) EXOFWD_CASE(2) EXOFWD_CASE(3) EXOFWD_CASE(4)
    EXOFWD_CASE(5) EXOFWD_CASE(6) EXOFWD_CASE(7) EXOFWD_CASE(8)
  }
#undef EXOFWD_CASE
  return nullptr;
}

const void* ls_kernel_for(int S, bool cia, bool ng) {
#define EXOFWD_CASE(n) \
  case n:                                                                                          \
    return ng ? (cia ? (const void*)k_layer_sums_mixed<n, true, true> : (const void*)k_layer_sums_mixed<n, false, true>) \
              : (cia ? (const void*)k_layer_sums_mixed<n, true, false> : (const void*)k_layer_sums_mixed<n, false, false>);
  switch (S) {
    EXOFWD_CASE(1) EXOFWD_CASE(2) EXOFWD_CASE(3) EXOFWD_CASE(4)
    EXOFWD_CASE(5) EXOFWD_CASE(6) EXOFWD_CASE(7) EXOFWD_CASE(8)
  }
#undef EXOFWD_CASE
  return nullptr;
}

hipError_t adjoint_configure(const Model& m, bool fp64) {
  if (!adjoint_supported(m, fp64) || m.mode == kEmission) return hipSuccess;
  if (fp64) {
    const void* k = adj_kernel_for<true>(m.S, m.has_cia, adj_fp64_instance(m));
    const size_t bytes = adj_lds_bytes(m, true, 0);
    if (!k || bytes > 160 * 1024) return hipErrorInvalidValue;
    return hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  }
  bool any = false;
  for (int v = 0; v < kAdjVariants; ++v) {
    if (!adjoint_variant_fits(m, v)) continue;
    // a split shape also launches 64 x 5 for the long class
    for (int u : {v, adj_split(m, v) ? (int)kAdjT64M5 : v}) {
      const size_t bytes = adj_lds_bytes(m, false, u);
      if (bytes > 160 * 1024) continue;
      const void* k = adj_kernel_for<false>(m.S, m.has_cia, u);
      if (!k) return hipErrorInvalidValue;
      const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
      if (e != hipSuccess) return e;
      any = true;
    }
  }
  return any ? hipSuccess : hipErrorInvalidValue;
}

bool adjoint_set_tuning(AdjWork& aw, const Model& m, int variant, int chunk_target, int ls_tiles) {
  if (variant < 0 || variant >= kAdjVariants || !adjoint_variant_fits(m, variant) ||
      adj_lds_bytes(m, false, variant) > 160 * 1024)
    return false;
  bool ok_t = false, ok_l = false;
  for (int t : kChunkTargets) ok_t |= t == chunk_target;
  for (int t : kLsTileChoices) ok_l |= t == ls_tiles;
  if (!ok_t || !ok_l) return false;
  aw.variant = variant;
  aw.chunk_target = chunk_target;
  aw.ls_tiles = ls_tiles;
  aw.lsum_chunks = (m.n_tiles + ls_tiles - 1) / ls_tiles;
  return true;
}

void launch_trans_adjoint(const Model& m, const Work& w, const Tables& tb, const AdjWork& aw, int B, bool fp64,
                          hipStream_t st) {
  int C = adjoint_chunks(m, aw, B, fp64);
  if (fp64) {
    void* args[] = {(void*)&m, (void*)&w, (void*)&tb, (void*)&aw, (void*)&B, (void*)&C};
    hipLaunchKernel(adj_kernel_for<true>(m.S, m.has_cia, adj_fp64_instance(m)), dim3((unsigned)(B * C)), dim3(kBlockT),
                    args, adj_lds_bytes(m, true, 0), st);
    return;
  }
  const int32_t* cls = adj_split(m, aw.variant) ? w.cls : nullptr;   // the forward built the classes
  for (int cl = 0; cl < (cls ? 2 : 1); ++cl) {
    const int v = cl == 1 ? (int)kAdjT64M5 : aw.variant;
    void* args[] = {(void*)&m, (void*)&w, (void*)&tb, (void*)&aw, (void*)&B, (void*)&C, (void*)&cls, (void*)&cl};
    hipLaunchKernel(adj_kernel_for<false>(m.S, m.has_cia, v), dim3((unsigned)(B * C)), dim3(adj_threads(v)), args,
                    adj_lds_bytes(m, false, v), st);
  }
}

void launch_layer_sums(const Model& m, const Work& w, const Tables& tb, const AdjWork& aw, int B, bool fp64,
                       hipStream_t st) {
  if (m.mode == kEmission) {
    launch_layer_sums_emis(m, w, tb, aw, B, fp64, st);
    return;
  }
  const int NG = m.L_max;   // layer groups per sample: at most one per layer
  const long waves = (long)aw.lsum_chunks * B * NG;
  void* args2[] = {(void*)&m, (void*)&w, (void*)&tb, (void*)&aw, (void*)&B};
  // a whole number of blocks per XCD; the waves past the last chunk return at once
  const long blocks = ((waves + 3) / 4 + 7) / 8 * 8;
  hipLaunchKernel(ls_kernel_for(m.S, m.has_cia, m.cloud_ng), dim3((unsigned)blocks), dim3(kBlock), args2, 0, st);
  if (m.cloud_ng) {
    const long cw = (long)B * aw.lsum_chunks;
    hipLaunchKernelGGL(k_cloud_spectral, dim3((unsigned)((cw + 3) / 4)), dim3(kBlock), 0, st, m, w, aw, B);
  }
}

void launch_chain(const Model& m, const Work& w, const AdjWork& aw, int B, const double* params, const uint8_t* mask,
                  double* grad, bool fp64, hipStream_t st) {
  const int C = adjoint_chunks(m, aw, B, fp64);
  const unsigned grid = (unsigned)(reduce_blocks(reduce_sizes(m, C)) * B);
  if (fp64) {
    hipLaunchKernelGGL(k_reduce_chunks<double>, dim3(grid), dim3(kBlock), 0, st, m, w, aw, C);
    hipLaunchKernelGGL(k_chain<double>, dim3(B), dim3(kBlockC), 0, st, m, w, aw, C, params, mask, grad);
  } else {
    hipLaunchKernelGGL(k_reduce_chunks<float>, dim3(grid), dim3(kBlock), 0, st, m, w, aw, C);
    hipLaunchKernelGGL(k_chain<float>, dim3(B), dim3(kBlockC), 0, st, m, w, aw, C, params, mask, grad);
  }
}

}  // namespace exofwd
