// The general vijp's sweep over the anti-diagonals of the output grid (see EpiDiagAccum) for whole images: one workgroup
// takes an image through all its diagonals. An image's diagonals depend on each other but not on other images, so
// what one launch per diagonal passes through memory and the launch itself stays in the workgroup: the taps in registers,
// the last two diagonals in LDS, a barrier in place of a launch. Only kernels that reach one position back (three earlier
// neighbours), which is what k <= p + 2 s gives.
//
//   h'[i, j] = G[i, j] - h'[i-1, j-1] A_0 - h'[i-1, j] A_1 - h'[i, j-1] A_2
//
// A diagonal is a product of (its positions) x 3C by 3C x C, in tiles of 32 positions. Wavefront (n, q) owns 32 of the C
// columns and every KG-th step of 16 k, adds them up and hands the sums over in LDS. Products are formed from three bf16 parts
// as in gemm_split.h (there: accuracy, sign, range): the taps' parts stay in registers for the whole sweep, those of an h' are made once
// when it is finished. What bounds it: for one tile the chain barrier, fragment reads, products (C = 64: 18 matrix
// instructions a wavefront, two wavefronts to a SIMD), exchange, barrier.
#pragma once

#include "gemm_split.h"

namespace mw {

template <int C>
struct SweepCfg {
  static constexpr int NT32 = C / 32;
  // groups of K: as many wavefronts as have a step of K each and whose taps leave room in the registers
  static constexpr int KG = C == 32 ? 6 : (C == 64 ? 4 : 2);
  static constexpr int WAVES = NT32 * KG;
  static constexpr int NT = 64 * WAVES;
  static constexpr int STEPS = 3 * C / 16 / KG;   // steps of 16 k of a wavefront
  static_assert(STEPS * KG * 16 == 3 * C, "K divides over the groups");
  static constexpr int PITCH = 2 * C + 16;        // bytes of one position in one plane (the pad spreads rows over the banks)
  static constexpr int PARK = 32 * 36 * 4;        // bytes of a wavefront's 32 x 32 sums
  static constexpr int QUADS = (8 * C + NT - 1) / NT;  // groups of four values a thread finishes per tile
  static constexpr int row_bytes() { return 3 * 3 * PITCH; }   // three diagonals, three planes
  static constexpr int fixed_bytes() { return WAVES * PARK + 16; }
};

struct SweepImages {
  int Ho, Wo;
  float* CT;            // [n_img][Ho][Wo][C]: G in, h' out
  const float* A;       // [C][3C], slots (i-1, j-1), (i-1, j), (i, j-1)
};

// Magnitudes up to which neither a part nor a sum of the three products of parts can overflow; see the repeat below.
constexpr float SWEEP_BIG_H = 0x1p40f, SWEEP_BIG_A = 0x1p20f;

template <int C>
__global__ void __launch_bounds__(SweepCfg<C>::NT) sweep_images_kernel(SweepImages p) {
  using Cfg = SweepCfg<C>;
  extern __shared__ __align__(16) char smem[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int nt = wave % Cfg::NT32, kg = wave / Cfg::NT32, r = lane & 31, g = lane >> 5;
  const bool by_row = p.Ho <= p.Wo;               // positions of a diagonal are counted along the shorter side
  const int D = by_row ? p.Ho : p.Wo;
  const int rows = D + 1;                         // row 0 of a diagonal stands for positions outside the grid: zeros
  const int plane = rows * Cfg::PITCH, diag = 3 * plane;
  float* const park = reinterpret_cast<float*>(smem);
  uint32_t* const big = reinterpret_cast<uint32_t*>(smem + Cfg::WAVES * Cfg::PARK);
  char* const hist = smem + Cfg::fixed_bytes();
  float* const ct = p.CT + (int64_t)blockIdx.x * p.Ho * p.Wo * C;

  // positions a diagonal does not have are read as zeros (i - 1 < 0: row 0; j - 1 < 0: rows not written yet)
  for (int i = threadIdx.x; i < 3 * diag / 16; i += Cfg::NT) reinterpret_cast<u32x4*>(hist)[i] = u32x4{0, 0, 0, 0};
  if (threadIdx.x == 0) *big = 0;
  __syncthreads();

  // this wavefront's taps: column nt * 32 + r of the result, steps kg, kg + KG, ...; odd groups with the other sign
  bf16x8 fb[Cfg::STEPS][3];
  {
    float top = 0.f;
    const float up = split_up(kg & 1);
#pragma unroll
    for (int s = 0; s < Cfg::STEPS; ++s) {
      const float4* q = reinterpret_cast<const float4*>(p.A + (int64_t)(nt * 32 + r) * 3 * C + (s * Cfg::KG + kg) * 16 + 8 * g);
      const float4 a = q[0], b = q[1];
      const SplitPair v[4] = {split_pair(a.x, a.y, up, top), split_pair(a.z, a.w, up, top), split_pair(b.x, b.y, up, top),
                              split_pair(b.z, b.w, up, top)};
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const u32x4 w{v[0].part[i], v[1].part[i], v[2].part[i], v[3].part[i]};
        fb[s][i] = __builtin_bit_cast(bf16x8, w);
      }
    }
    if (top >= SWEEP_BIG_A * split_up(false)) *big = 1;
  }

  const int other = (by_row ? p.Wo : p.Ho) - 1, last = p.Ho + p.Wo - 2;
  // positions [lo, hi] of diagonal d
  auto lo_of = [&](int d) { return d > other ? d - other : 0; };
  auto hi_of = [&](int d) { return d < D - 1 ? d : D - 1; };
  // The values this thread finishes in the tile of positions from `first` on, four channels of a position each. They are
  // requested one tile ahead, so that memory is not part of the chain.
  float4 next[Cfg::QUADS];
  int next_at[Cfg::QUADS];
  auto request = [&](int d, int first) {
#pragma unroll
    for (int u = 0; u < Cfg::QUADS; ++u) {
      const int q = (int)threadIdx.x + u * Cfg::NT, pos = first + q / (C / 4);
      const bool in = q < 8 * C && d <= last && pos <= hi_of(d);
      const int i = by_row ? pos : d - pos, j = by_row ? d - pos : pos;
      next_at[u] = in ? (i * p.Wo + j) * C + 4 * (q % (C / 4)) : -1;
      next[u] = in ? *reinterpret_cast<const float4*>(ct + next_at[u]) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  };
  request(0, 0);
  for (int d = 0; d <= last; ++d) {
    const int lo = lo_of(d), hi = hi_of(d);
    char* const now = hist + (d % 3) * diag;
    const char* const d1 = hist + ((d + 2) % 3) * diag;   // diagonal d - 1
    const char* const d2 = hist + ((d + 1) % 3) * diag;   // diagonal d - 2
    for (int first = lo; first <= hi; first += 32) {
      float4 G[Cfg::QUADS];
      int at[Cfg::QUADS];
#pragma unroll
      for (int u = 0; u < Cfg::QUADS; ++u) {
        G[u] = next[u];
        at[u] = next_at[u];
      }
      if (first + 32 <= hi) request(d, first + 32);
      else request(d + 1, lo_of(d + 1));
      f32x16 acc;
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[i] = 0.f;
      const int pos = first + r < D ? first + r : D - 1;   // (rows past the diagonal: any, not stored)
#pragma unroll
      for (int s = 0; s < Cfg::STEPS; ++s) {
        const int k = (s * Cfg::KG + kg) * 16, slot = k / C;
        // slot 0: (i-1, j-1); 1: (i-1, j); 2: (i, j-1): one position back where the counted coordinate goes back
        const int back = slot == 0 || (slot == 1) == by_row ? 1 : 0;
        const char* src = (slot == 0 ? d2 : d1) + (pos + 1 - back) * Cfg::PITCH + (k % C + 8 * g) * 2;
        bf16x8 fa[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) fa[i] = *reinterpret_cast<const bf16x8*>(src + i * plane);
#pragma unroll
        for (int q = 0; q < 6; ++q) {   // from the smallest to the largest, as in SplitProduct::multiply
          constexpr int PA[6] = {0, 2, 1, 0, 1, 0}, PB[6] = {2, 0, 1, 1, 0, 0};
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[PA[q]], fb[s][PB[q]], acc, 0, 0, 0);
        }
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) park[wave * (Cfg::PARK / 4) + acc_row(i, g) * 36 + r] = acc[i];
      // (what the repeat reads from memory was stored by this workgroup before an earlier barrier; *big is up to date here)
      __syncthreads();
      float top = 0.f;
#pragma unroll
      for (int u = 0; u < Cfg::QUADS; ++u) {
        const int q = (int)threadIdx.x + u * Cfg::NT, row = q / (C / 4), c = 4 * (q % (C / 4));
        if (at[u] >= 0) {
          float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int w = 0; w < Cfg::KG; ++w) {
            const float4 t = *reinterpret_cast<const float4*>(park + (w * Cfg::NT32 + c / 32) * (Cfg::PARK / 4) + row * 36 + c % 32);
            const float sign = (w & 1) ? -1.f : 1.f;
            v[0] += sign * t.x;
            v[1] += sign * t.y;
            v[2] += sign * t.z;
            v[3] += sign * t.w;
          }
          bool finite = true;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            finite &= fabsf(v[e]) < __builtin_inff();
            v[e] *= 0x1p-24f * 0x1p-24f;
          }
          // Large operands: parts or sums may have left fp32's range. Those values again from the earlier positions as
          // they are (rare, so one by one).
          if (!finite && *big) {
            const int ps = first + row, i = by_row ? ps : d - ps, j = by_row ? d - ps : ps;
            for (int e = 0; e < 4; ++e) {
              if (fabsf(v[e]) < __builtin_inff()) continue;
              float sum = 0.f;
              for (int k = 0; k < 3 * C; ++k) {
                const int slot = k / C, y = i - (slot < 2 ? 1 : 0), x = j - (slot != 1 ? 1 : 0);
                if (y >= 0 && x >= 0) sum += ct[((int64_t)y * p.Wo + x) * C + k % C] * p.A[(int64_t)(c + e) * 3 * C + k];
              }
              v[e] = sum;
            }
          }
          const float4 h = make_float4(G[u].x - v[0], G[u].y - v[1], G[u].z - v[2], G[u].w - v[3]);
          *reinterpret_cast<float4*>(ct + at[u]) = h;
          const SplitPair a = split_pair(h.x, h.y, split_up(false), top), b = split_pair(h.z, h.w, split_up(false), top);
          char* dst = now + (first + row + 1) * Cfg::PITCH + c * 2;
#pragma unroll
          for (int i = 0; i < 3; ++i) *reinterpret_cast<u32x2*>(dst + i * plane) = u32x2{a.part[i], b.part[i]};
        }
      }
      if (top >= SWEEP_BIG_H * split_up(false)) *big = 1;
      __syncthreads();   // the sums are read, the diagonal is written
    }
  }
}

constexpr int SWEEP_LDS_MAX = 160 * 1024;
// bytes of LDS for images of Ho x Wo
template <int C>
inline int sweep_lds_bytes(int Ho, int Wo) {
  return SweepCfg<C>::fixed_bytes() + ((Ho < Wo ? Ho : Wo) + 1) * SweepCfg<C>::row_bytes();
}

}  // namespace mw
