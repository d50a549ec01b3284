// fp32 products on the half-precision matrix unit (gfx950): every fp32 operand value is split into the sum of two
// fp16 values while its tile is staged, and a product a b is formed as a_hi b_hi + a_hi b_lo + a_lo b_hi in
// v_mfma_f32_32x32x16_f16, sums in fp32.
//
// What it is for. v_mfma_f32_32x32x2_f32 does 64 flop per clock and SIMD; the fp16 instruction does 1024, so three
// of them take 3/16 of the time. Measured (MI355X): 1024 x 4096 x 4096 in 115 us (299 TFLOP/s) against 247 us with
// fp32 instructions, 512 x 2048 x 2048 in 26 us against 43 us, 256 x 1024 x 1024 in 7.3 us against 10.0 us. What
// bounds it then: the fp16 unit at the clock its own power draw allows (about 1.75 PFLOP/s on dense random data, 580
// TFLOP/s of these products), LDS traffic (4 bytes an element, as for fp32) and, for small outputs, operand bytes
// per CU.
//
// Accuracy. A scaled value is hi + lo with hi = fp16(v), lo = fp16(v - hi): hi takes 11 bits, lo the next 11 and the
// sign of lo one more, so |v - hi - lo| <= 2^-23 |v| as long as lo does not fall below fp16's subnormal spacing
// 2^-24, i.e. for |v| >= 2^-2 after scaling; below, the error is at most 2^-25 absolute. The dropped a_lo b_lo is at
// most 2^-22 |a b|. Both are random in sign and enter a sum of K products as 7e-8 of its norm, whatever K is, while
// the rounding of the running fp32 sum grows like sqrt(number of additions): there the fp16 instruction, which adds
// sixteen products at a time, makes fewer of them. Normwise error against fp64 for N(0, 1) operands, K = 128 / 512 /
// 2048: 1.2e-7 / 1.9e-7 / 3.6e-7, with the fp32 instruction 2.0e-7 / 4.1e-7 / 8.1e-7.
//
// Range. fp16 holds 2^-24 .. 65504, fp32 far more, so every row of an operand tile (a row of A, a row of B^T) has
// a power-of-two scale of its own, chosen from the largest of its first SPLIT_SAMPLE values so that this one lies in
// [2^5, 2^6) (split_choose, which also looks at the rows beside it); the result is scaled back by an exact exponent
// shift. While a tile is staged the largest magnitude of every row is tracked: if a later value does not fit under
// 65504 (infinities among them), or a row whose sample was all zero turns out to be tiny beside its neighbours, the
// workgroup computes its tile again with fp32 instructions and takes those results for the rows and columns concerned
// (about the time of an fp32 product once more: 87 us instead of 29 for 2048 x 2048 x 512). A result thus depends on
// its row and column and their aligned groups of 32, not on what else is in the tile or on the tile's shape. NaN
// passes through both halves by itself. (A scale is at most 2^126: with it every value below 2^-115, subnormals
// included, is held exactly.)
#pragma once

#include "gemm_f32.h"

namespace mw {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// One workgroup = WM x WN x WK wavefronts, each with WTM x WTN accumulator tiles of 32 x 32 and, per K tile, KS
// steps of 16 k of its own (BK = 16 KS WK).
template <int WTM_, int WTN_, int WM_, int WN_, int WK_, int KS_>
struct SplitCfg {
  static constexpr int WTM = WTM_, WTN = WTN_, WM = WM_, WN = WN_, WK = WK_, KS = KS_;
  static constexpr int PREC = 2;
  static constexpr int ST = 2;   // LDS stages; as many further K tiles are in flight in registers
  static constexpr int BM = 32 * WTM * WM;
  static constexpr int BN = 32 * WTN * WN;
  static constexpr int BK = 16 * KS * WK;
  static constexpr int NT = 64 * WM * WN * WK;
  static constexpr int NACC = WTM * WTN;
  static constexpr int CNT = 16 / WK;            // finished accumulator registers per wavefront and 32 x 32 tile
  static constexpr int PLANE = (BM + BN) * BK * 2;  // bytes of one half (hi or lo) of a staged K tile
  static constexpr int STAGE = 2 * PLANE;
  static constexpr int PARKED = NT * NACC * (16 - CNT) * 4;
  static constexpr int MAIN = 2 * STAGE > PARKED ? 2 * STAGE : PARKED;
  static constexpr int PARTS = 4;   // wavefronts that may hold a share of a row's sample
  static constexpr int LDS_BYTES = MAIN + (BM + BN) * 4 * (PARTS + 1) + 16;   // + maxima and a scale exponent per operand row, a flag
  static_assert((BM + BN) * (BK + 4) * 4 <= 2 * STAGE, "the fp32 repeat stages its tile in the same memory");
};
// Shapes that were fastest over the layer sizes in use (us at M x N x K; 512 threads each):
//   Split256  8192 x 1024 x 1024: 69 (128 x 128: 81),  131072 x 128 x 1152: 170 (218)
//   Split128  1024 x 4096 x 4096: 115 (256 x 128: 161), 2048 x 2048 x 512: 21 (64 x 64: 30)
//   Split64   512 x 2048 x 2048: 26 (128 x 128: 48)
using Split256 = SplitCfg<2, 2, 4, 2, 1, 2>;  // 256 x 128, K tile 32
using Split128 = SplitCfg<2, 2, 2, 2, 2, 1>;  // 128 x 128, K tile 32, K split over two groups of four wavefronts
using Split64 = SplitCfg<1, 1, 2, 2, 2, 2>;   //  64 x  64, K tile 64, likewise

using Split64Q = SplitCfg<1, 1, 2, 2, 1, 2>;  // 64 x 64, K tile 32, four wavefronts: gathers of 32 channels and odd multiples

template <class Cfg>
constexpr bool is_split() { return Cfg::PREC == 2; }

// Byte address of the 8-k chunk c of a row inside a plane of rows of BK halves. The xor (and for 64-byte rows the
// exchange of neighbouring rows) spreads the rows that a wavefront reads (32 rows, one chunk) or writes (eight
// rows four apart, all chunks) over all banks.
template <int BK>
__device__ __forceinline__ int split_addr(int row, int c) {
  constexpr int CH = BK / 8;
  static_assert(CH == 4 || CH == 8 || CH == 16, "rows of 32, 64 or 128 halves");
  if (CH == 4) return (row ^ ((row >> 2) & 1)) * 64 + ((c ^ (((row >> 1) ^ (row >> 3)) & 3)) << 4);
  if (CH == 8) return row * 128 + ((c ^ (((row >> 1) & 7) ^ ((row & 1) << 2))) << 4);
  return row * 256 + ((c ^ (row & 15)) << 4);
}

// (fp16(x s), fp16(y s)) and (fp16(x s - hi.x), fp16(y s - hi.y)), each rounded once
__device__ __forceinline__ uint32_t split_hi(float x, float sx, float y, float sy) {
  uint32_t d;
  asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(d) : "v"(x), "v"(sx));
  asm("v_fma_mixhi_f16 %0, %1, %2, 0" : "+v"(d) : "v"(y), "v"(sy));
  return d;
}
__device__ __forceinline__ uint32_t split_lo(float x, float sx, float y, float sy, uint32_t hi) {
  uint32_t d;
  asm("v_fma_mixlo_f16 %0, %1, %2, -%3 op_sel:[0,0,0] op_sel_hi:[0,0,1]" : "=v"(d) : "v"(x), "v"(sx), "v"(hi));
  asm("v_fma_mixhi_f16 %0, %1, %2, -%3 op_sel:[0,0,1] op_sel_hi:[0,0,1]" : "+v"(d) : "v"(y), "v"(sy), "v"(hi));
  return d;
}
__device__ __forceinline__ float max3_abs(float x, float y, float m) { return fmaxf(fmaxf(fabsf(x), fabsf(y)), m); }
// combine over the eight lanes of an aligned group of eight
__device__ __forceinline__ float dpp_f32(float v, int quad_or_mirror) {
  const int i = __float_as_int(v);
  int r;
  switch (quad_or_mirror) {
    case 0: r = __builtin_amdgcn_update_dpp(i, i, 0xB1, 0xF, 0xF, false); break;   // lane ^ 1
    case 1: r = __builtin_amdgcn_update_dpp(i, i, 0x4E, 0xF, 0xF, false); break;   // lane ^ 2
    case 2: r = __builtin_amdgcn_update_dpp(i, i, 0x141, 0xF, 0xF, false); break;  // the other half of eight (mirrored)
    default: r = __builtin_amdgcn_update_dpp(i, i, 0x140, 0xF, 0xF, false); break; // the other half of sixteen (mirrored)
  }
  return __int_as_float(r);
}
__device__ __forceinline__ float max_over_8(float v) {
#pragma unroll
  for (int k = 0; k < 3; ++k) v = fmaxf(v, dpp_f32(v, k));
  return v;
}
__device__ __forceinline__ float sum_over_8(float v) {
#pragma unroll
  for (int k = 0; k < 3; ++k) v += dpp_f32(v, k);
  return v;
}
__device__ __forceinline__ float pow2(int e) { return __int_as_float((e + 127) << 23); }  // -126 <= e <= 127

constexpr int SPLIT_SAMPLE = 64;       // leading k of a row that choose its scale
constexpr int SPLIT_TOP = 5;           // a sampled maximum is scaled to 2^5 .. 2^6, see `Range` above
constexpr int SPLIT_DEFAULT_EXP = 8;    // rows without any sample to go by: 2^-12 .. 2^7 are at home with it
constexpr float SPLIT_LEAST = 0x1p-4f;  // a scaled row maximum below this has lost precision
// Scale exponent e of a row whose sampled maximum is m: m 2^e in [2^TOP, 2^(TOP + 1)), clamped to what a float holds.
__device__ __forceinline__ int split_exponent(float m) {
  const int e = SPLIT_TOP + 127 - (int)(__float_as_uint(m) >> 23);
  return e > 126 ? 126 : e;
}

// One operand tile, R rows x BK k, in registers, with the scales of the rows this thread stages.
template <int LAYOUT, int R, int BK, int NT, bool VEC, class XfDev>
struct SplitLoader {
  static constexpr int NV = R * BK / 4 / NT;                        // 4-element chunks per thread
  static constexpr int KP = LAYOUT == KCONTIG ? 1 : (NV >= 4 ? 4 : 2);  // rows fast in memory: consecutive k in one thread
  static constexpr int NTASK = NV / KP;
  static constexpr int NS = LAYOUT == KCONTIG ? NV : 4 * NTASK;     // rows per thread
  static_assert(NV * 4 * NT == R * BK && NV % KP == 0, "tile must divide evenly over the workgroup");
  using Map = ChunkMap<LAYOUT, R, BK, NT, KP>;
  // shares of a row's sample, each complete within one wavefront
  static constexpr int PARTS = LAYOUT == KCONTIG ? 1 : (BK < SPLIT_SAMPLE ? BK : SPLIT_SAMPLE) / (8 * KP);

  float4 v[NV];
  typename XfDev::Aux aux[NV];

  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, int64_t ld, int row0, int k0, int n_rows, int n_k,
                                       const XfDev& xf) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int r = row0 + Map::row(i), k = k0 + Map::k(i);
      const Chunk c = LAYOUT == KCONTIG ? xf.template chunk<LAYOUT>(i, r, k, n_rows, n_k, ld)
                                        : xf.template chunk<LAYOUT>(i, k, r, n_k, n_rows, ld);
      if (VEC) {
        v[i] = buf_load_f32x4(rs, c.nvalid ? c.e * 4u : OOB);
      } else {
        v[i].x = buf_load_f32(rs, c.nvalid > 0 ? c.e * 4u : OOB);
        v[i].y = buf_load_f32(rs, c.nvalid > 1 ? c.e * 4u + 4u : OOB);
        v[i].z = buf_load_f32(rs, c.nvalid > 2 ? c.e * 4u + 8u : OOB);
        v[i].w = buf_load_f32(rs, c.nvalid > 3 ? c.e * 4u + 12u : OOB);
      }
      xf.template fetch<VEC>(aux[i], c);
    }
  }

  // Largest sampled magnitude of every row of the tile into m[PARTS][R] (LDS): the first SPLIT_SAMPLE k, which
  // take this K tile and with a K tile of 32 the next one (`second`, else NULL) too.
  __device__ __forceinline__ void sample(const SplitLoader* second, float* __restrict__ m, const XfDev& xf) const {
    if (LAYOUT == KCONTIG) {
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const float4 w = xf.apply(v[i], aux[i]);
        float x = max3_abs(w.x, w.y, max3_abs(w.z, w.w, 0.f));
        if (second) {
          const float4 u = xf.apply(second->v[i], second->aux[i]);
          x = max3_abs(u.x, u.y, max3_abs(u.z, u.w, x));
        }
        x = max_over_8(x);
        if (BK > 32) x = fmaxf(x, dpp_f32(x, 3));   // sixteen lanes hold 64 k
        if (Map::k(i) == 0) m[Map::row(i)] = x;
      }
    } else {
#pragma unroll
      for (int j = 0; j < NTASK; ++j) {
        float x[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < KP; ++kk) {
          const int i = j * KP + kk;
          const float4 w = xf.apply(v[i], aux[i]);
          x[0] = fmaxf(x[0], fabsf(w.x));
          x[1] = fmaxf(x[1], fabsf(w.y));
          x[2] = fmaxf(x[2], fabsf(w.z));
          x[3] = fmaxf(x[3], fabsf(w.w));
          if (second) {
            const float4 u = xf.apply(second->v[i], second->aux[i]);
            x[0] = fmaxf(x[0], fabsf(u.x));
            x[1] = fmaxf(x[1], fabsf(u.y));
            x[2] = fmaxf(x[2], fabsf(u.z));
            x[3] = fmaxf(x[3], fabsf(u.w));
          }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) x[q] = max_over_8(x[q]);
        const int kg = Map::k(j * KP) / KP;
        if ((kg & 7) == 0 && Map::k(j * KP) < SPLIT_SAMPLE)
          *reinterpret_cast<float4*>(m + (kg >> 3) * R + Map::row(j * KP)) = make_float4(x[0], x[1], x[2], x[3]);
      }
    }
  }
  static __device__ __forceinline__ int row_of(int j) { return LAYOUT == KCONTIG ? Map::row(j) : Map::row((j / 4) * KP) + (j & 3); }
};

// The scale exponent of every operand row of the tile, by one thread per row: from the sampled maxima m[PARTS][..] of
// the A rows and, after Cfg::PARTS * BM floats, of the B rows, into ex as 2 e + (1: the row's sample was all zero).
// The sample of a row may be far below its later values: all zero or next to it (a unit that is off in nearly all of
// them, the padding of an image). So a sampled maximum counts as no less than 2^-7 of the largest one in the row's
// aligned group of 32, which every tile shape holds whole: eight times that one still fits, and 2^-16 of it is
// precise. Sampled values below 2^-13 of it are taken as they are (the rows differ in scale, then).
template <class Cfg, int PARTS_A, int PARTS_B>
__device__ __forceinline__ void split_choose(const float* __restrict__ m, int* __restrict__ ex) {
  const int i = threadIdx.x;
  static_assert(Cfg::BM + Cfg::BN <= Cfg::NT && Cfg::BM % 64 == 0 || Cfg::BM + Cfg::BN <= 64, "a thread per row, whole wavefronts");
  if (i < Cfg::BM + Cfg::BN) {
    const bool is_b = i >= Cfg::BM;
    const float* q = is_b ? m + Cfg::PARTS * Cfg::BM + (i - Cfg::BM) : m + i;
    float x = q[0];
#pragma unroll
    for (int p = 1; p < (PARTS_A > PARTS_B ? PARTS_A : PARTS_B); ++p)
      if (p < (is_b ? PARTS_B : PARTS_A)) x = fmaxf(x, q[p * (is_b ? Cfg::BN : Cfg::BM)]);
    float top = max_over_8(x);
    top = fmaxf(top, dpp_f32(top, 3));
    top = fmaxf(top, __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(top), 0x401F)));  // lane ^ 16
    const bool own = x >= 0x1p-7f * top || (x > 0.f && x < 0x1p-13f * top);
    const int e = top > 0.f ? split_exponent(own ? x : 0x1p-7f * top) : SPLIT_DEFAULT_EXP;
    ex[i] = 2 * e + (x == 0.f ? 1 : 0);
  }
}

// Scales and running maxima of the rows a thread stages.
template <class Ld>
struct SplitRows {
  float s[Ld::NS], mx[Ld::NS];
  uint32_t defaulted;   // bit j: row j's sample was all zero

  __device__ __forceinline__ void take(const int* __restrict__ ex) {
    defaulted = 0;
#pragma unroll
    for (int j = 0; j < Ld::NS; ++j) {
      const int x = ex[Ld::row_of(j)];
      s[j] = pow2(x >> 1);
      defaulted |= (uint32_t)(x & 1) << j;
      mx[j] = 0.f;
    }
  }
  // whether a row's scale may not have suited the values this thread saw (its share of the row's)
  __device__ __forceinline__ bool bad() const {
    bool b = false;
#pragma unroll
    for (int j = 0; j < Ld::NS; ++j) {
      const float x = mx[j] * s[j];
      b |= !(x <= 65504.f) || (((defaulted >> j) & 1u) && mx[j] > 0.f && x < SPLIT_LEAST);
    }
    return b;
  }
  // the same for a whole row: m its true maximum, x its entry of the exponent table
  static __device__ __forceinline__ bool row_bad(float m, int x) {
    const float y = m * pow2(x >> 1);
    return !(y <= 65504.f) || ((x & 1) && m > 0.f && y < SPLIT_LEAST);
  }
};

// Split the staged values of `ld` into both planes of an LDS stage (`base`: this operand's rows of the hi plane).
template <int PLANE, bool COLSUM, int NT, int BK, class Ld, class XfDev>
__device__ __forceinline__ void split_store(const Ld& ld, SplitRows<Ld>& rows, const XfDev& xf, char* __restrict__ base,
                                            float* __restrict__ csum) {
  using Map = typename Ld::Map;
  if constexpr (Ld::KP == 1) {
#pragma unroll
    for (int i = 0; i < Ld::NV; ++i) {
      const float4 w = xf.apply(ld.v[i], ld.aux[i]);
      const float s = rows.s[i];
      rows.mx[i] = max3_abs(w.z, w.w, max3_abs(w.x, w.y, rows.mx[i]));
      u32x2 hi, lo;
      hi.x = split_hi(w.x, s, w.y, s);
      hi.y = split_hi(w.z, s, w.w, s);
      lo.x = split_lo(w.x, s, w.y, s, hi.x);
      lo.y = split_lo(w.z, s, w.w, s, hi.y);
      // a thread's chunks are the same k of rows so far apart that they have the same pattern of chunks
      static_assert(NT * 4 / BK % (BK == 32 ? 32 : 16) == 0, "see split_addr");
      char* p = base + split_addr<BK>(Map::row(0), Map::k(0) >> 3) + (Map::k(0) & 4) * 2 + i * (NT * 4 / BK) * BK * 2;
      *reinterpret_cast<u32x2*>(p) = hi;
      *reinterpret_cast<u32x2*>(p + PLANE) = lo;
    }
  } else {
#pragma unroll
    for (int j = 0; j < Ld::NTASK; ++j) {
      float e[4][Ld::KP];
#pragma unroll
      for (int kk = 0; kk < Ld::KP; ++kk) {
        const float4 w = xf.apply(ld.v[j * Ld::KP + kk], ld.aux[j * Ld::KP + kk]);
        e[0][kk] = w.x;
        e[1][kk] = w.y;
        e[2][kk] = w.z;
        e[3][kk] = w.w;
      }
      const int k = Map::k(j * Ld::KP), row = Map::row(j * Ld::KP);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float s = rows.s[4 * j + q];
        uint32_t hi[Ld::KP / 2], lo[Ld::KP / 2];
#pragma unroll
        for (int h = 0; h < Ld::KP / 2; ++h) {
          const float x = e[q][2 * h], y = e[q][2 * h + 1];
          rows.mx[4 * j + q] = max3_abs(x, y, rows.mx[4 * j + q]);
          if (COLSUM) csum[4 * j + q] += x + y;
          hi[h] = split_hi(x, s, y, s);
          lo[h] = split_lo(x, s, y, s, hi[h]);
        }
        char* p = base + split_addr<BK>(row + q, k >> 3) + (k & 7) * 2;
        if constexpr (Ld::KP == 4) {
          u32x2 a, b;
          a.x = hi[0]; a.y = hi[1];
          b.x = lo[0]; b.y = lo[1];
          *reinterpret_cast<u32x2*>(p) = a;
          *reinterpret_cast<u32x2*>(p + PLANE) = b;
        } else {
          *reinterpret_cast<uint32_t*>(p) = hi[0];
          *reinterpret_cast<uint32_t*>(p + PLANE) = lo[0];
        }
      }
    }
  }
}

// The staged values as they are, [row][BK + 4] fp32, for the repeat with fp32 instructions.
template <int BK, class Ld, class XfDev>
__device__ __forceinline__ void plain_store(const Ld& ld, const XfDev& xf, float* __restrict__ base) {
  using Map = typename Ld::Map;
#pragma unroll
  for (int i = 0; i < Ld::NV; ++i) {
    const float4 w = xf.apply(ld.v[i], ld.aux[i]);
    float* p = base + Map::row(i) * (BK + 4) + Map::k(i);
    if (Ld::KP == 1) {
      *reinterpret_cast<float4*>(p) = w;
    } else {
      p[0] = w.x;
      p[BK + 4] = w.y;
      p[2 * (BK + 4)] = w.z;
      p[3 * (BK + 4)] = w.w;
    }
  }
}

// One product of a workgroup tile over the whole K range.
template <class Cfg, int LA, int LB, bool VEC, class XfDev>
struct SplitProduct {
  static constexpr int BM = Cfg::BM, BN = Cfg::BN, BK = Cfg::BK, NT = Cfg::NT;
  using LdA = SplitLoader<LA, BM, BK, NT, VEC, XfDev>;
  using LdB = SplitLoader<LB, BN, BK, NT, VEC, ANone::Dev>;
  LdA a[2];
  LdB b[2];

  // out[tile][j]: finished values of accumulator registers wk * CNT + j (acc_row) of the wavefront's tiles, the K
  // groups added in the order 0, 1, 2, ...
  // csum (COLSUM): this thread's share of the sums over k of the A rows it stages.
  // LDS may be reused after the caller's next barrier (run starts with one before it writes the stages).
  template <bool COLSUM>
  __device__ __forceinline__ void run(const float* __restrict__ A, int64_t lda, const float* __restrict__ B, int64_t ldb, int M,
                                      int N, int K, int m0, int n0, float* __restrict__ lds_f, XfDev& xf,
                                      float (&out)[Cfg::NACC][Cfg::CNT], float* __restrict__ csum) {
    char* const lds = reinterpret_cast<char*>(lds_f);
    float* const rmax = reinterpret_cast<float*>(lds + Cfg::MAIN);  // maxima of the A rows, then of the B rows
    int* const rexp = reinterpret_cast<int*>(rmax + Cfg::PARTS * (BM + BN));  // their scale exponents
    int* const flag = rexp + BM + BN;
    static_assert(LdA::PARTS <= Cfg::PARTS && LdB::PARTS <= Cfg::PARTS, "room for the shares");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wk = wave % Cfg::WK, wn = (wave / Cfg::WK) % Cfg::WN, wm = wave / (Cfg::WK * Cfg::WN);
    const int r = lane & 31, g = lane >> 5;

    const uint32_t bytes_a = LA == KCONTIG ? xf.extent(M, K, lda) : xf.extent(K, M, lda);
    const uint32_t bytes_b = LB == KCONTIG ? extent_bytes(N, K, ldb) : extent_bytes(K, N, ldb);
    const __amdgpu_buffer_rsrc_t ra = make_rsrc(A, bytes_a), rb = make_rsrc(B, bytes_b);
    const ANone::Dev none;
    const int nkt = (K + BK - 1) / BK;
    constexpr bool GATHERED = XfDev::GATHERED;

    SplitRows<LdA> rows_a;
    SplitRows<LdB> rows_b;
    f32x16 acc[Cfg::NACC];
#pragma unroll
    for (int i = 0; i < Cfg::NACC; ++i)
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[i][j] = 0.f;
    if (COLSUM) {
#pragma unroll
      for (int j = 0; j < LdA::NS; ++j) csum[j] = 0.f;
    }
#define MW_REQUEST(slot, idx)                       \
  do {                                              \
    a[slot].load(ra, lda, m0, (idx) * BK, M, K, xf); \
    b[slot].load(rb, ldb, n0, (idx) * BK, N, K, none); \
    xf.template advance<LA, BK>();                  \
  } while (0)
    xf.template prepare<LA, BM, BK, NT, LdA::KP>(m0, M, K);
    if constexpr (GATHERED) {
      // the sample of a gathered operand comes from a tile that is not in the padding
      xf.template seek_sample<LA, BK>();
      a[1].load(ra, lda, m0, 0, M, K, xf);
      xf.template unseek<LA>();
    }
    MW_REQUEST(0, 0);
    if (!GATHERED) MW_REQUEST(1, 1);
    a[0].sample(GATHERED || BK < SPLIT_SAMPLE ? &a[1] : nullptr, rmax, xf);
    if (GATHERED) MW_REQUEST(1, 1);
    b[0].sample(BK < SPLIT_SAMPLE ? &b[1] : nullptr, rmax + Cfg::PARTS * BM, none);
    if (threadIdx.x == 0) *flag = 0;
    __syncthreads();
    split_choose<Cfg, LdA::PARTS, LdB::PARTS>(rmax, rexp);
    __syncthreads();
    rows_a.take(rexp);
    rows_b.take(rexp + BM);

#define MW_TO_LDS(slot, stage)                                                                                            \
  do {                                                                                                                    \
    split_store<Cfg::PLANE, COLSUM, NT, BK>(a[slot], rows_a, xf, lds + (stage) * Cfg::STAGE, csum);                       \
    split_store<Cfg::PLANE, false, NT, BK>(b[slot], rows_b, none, lds + (stage) * Cfg::STAGE + BM * BK * 2, (float*)nullptr); \
  } while (0)
#define MW_MULTIPLY(stage) multiply(lds + (stage) * Cfg::STAGE, wm, wn, wk, r, g, acc)
    MW_TO_LDS(0, 0);
    MW_REQUEST(0, 2);
    __syncthreads();
    // tile t is in LDS stage t % 2, the registers hold tiles t + 1 and t + 2. The last tile is peeled off: after it
    // nothing is staged.
#define MW_STEP(u)                        \
  do {                                    \
    MW_MULTIPLY(u);                       \
    MW_TO_LDS(1 - (u), 1 - (u));          \
    MW_REQUEST(1 - (u), t + (u) + 3);     \
    __syncthreads();                      \
  } while (0)
    int t = 0;
    for (; t + 2 < nkt; t += 2) {
      MW_STEP(0);
      MW_STEP(1);
    }
    if (t + 1 < nkt) {   // two tiles are left, or one
      MW_STEP(0);
      MW_MULTIPLY(1);
    } else {
      MW_MULTIPLY(0);
    }
#undef MW_STEP
#undef MW_TO_LDS
#undef MW_MULTIPLY
#undef MW_REQUEST
    // Add the K groups and undo the scales (an exact exponent shift). A wavefront keeps CNT registers of every
    // tile and hands the others over through LDS.
    if (rows_a.bad() || rows_b.bad()) *flag = 1;
    __syncthreads();   // (also: the stages are free)
    bool again = __builtin_amdgcn_readfirstlane(*flag) != 0;
    if (again) {  // by the rows' true maxima
      uint32_t* um = reinterpret_cast<uint32_t*>(rmax);
      for (int i = threadIdx.x; i < BM + BN; i += NT) um[i] = 0u;
      __syncthreads();
#pragma unroll
      for (int j = 0; j < LdA::NS; ++j) atomicMax(um + LdA::row_of(j), __float_as_uint(rows_a.mx[j]));
#pragma unroll
      for (int j = 0; j < LdB::NS; ++j) atomicMax(um + BM + LdB::row_of(j), __float_as_uint(rows_b.mx[j]));
      __syncthreads();
      bool bad = false;
      for (int i = threadIdx.x; i < BM + BN; i += NT) bad |= SplitRows<LdA>::row_bad(rmax[i], rexp[i]);
      again = __syncthreads_or(bad);
    }
    finish(lds_f, rexp, true, acc, out, wm, wn, wk, r, g, lane);
    if (again) {
      repeat_f32(ra, lda, rb, ldb, M, N, K, m0, n0, lds_f, rmax, rexp, xf, out, nkt, wm, wn, wk, r, g, lane);
    }
  }

  __device__ __forceinline__ void multiply(const char* __restrict__ st, int wm, int wn, int wk, int r, int g,
                                           f32x16 (&acc)[Cfg::NACC]) const {
#pragma unroll
    for (int ks = 0; ks < Cfg::KS; ++ks) {
      const int c = (ks * Cfg::WK + wk) * 2 + g;   // the groups take the 16-k steps in turn
      // rows 32 apart have the same pattern of chunks (split_addr)
      const char* sa = st + split_addr<BK>(r, c) + wm * Cfg::WTM * 32 * BK * 2;
      const char* sb = st + split_addr<BK>(r, c) + (BM + wn * Cfg::WTN * 32) * BK * 2;
      f16x8 fa[2][Cfg::WTM], fb[2][Cfg::WTN];
#pragma unroll
      for (int p = 0; p < 2; ++p) {
#pragma unroll
        for (int i = 0; i < Cfg::WTM; ++i)
          fa[p][i] = *reinterpret_cast<const f16x8*>(sa + p * Cfg::PLANE + i * 32 * BK * 2);
#pragma unroll
        for (int i = 0; i < Cfg::WTN; ++i)
          fb[p][i] = *reinterpret_cast<const f16x8*>(sb + p * Cfg::PLANE + i * 32 * BK * 2);
      }
      // a_hi b_lo, a_lo b_hi, a_hi b_hi
#pragma unroll
      for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int i = 0; i < Cfg::WTM; ++i)
#pragma unroll
          for (int j = 0; j < Cfg::WTN; ++j)
            acc[i * Cfg::WTN + j] =
                __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[q == 1][i], fb[q == 0][j], acc[i * Cfg::WTN + j], 0, 0, 0);
    }
  }

  // The product again with fp32 instructions, one K tile at a time through registers and LDS, for the rows and columns
  // whose scale did not suit. Rare, so simple.
  __device__ __forceinline__ void repeat_f32(__amdgpu_buffer_rsrc_t ra, int64_t lda, __amdgpu_buffer_rsrc_t rb, int64_t ldb, int M, int N,
                                             int K, int m0, int n0, float* __restrict__ lds, const float* __restrict__ rmax,
                                             int* __restrict__ rexp, XfDev& xf, float (&out)[Cfg::NACC][Cfg::CNT], int nkt, int wm,
                                             int wn, int wk, int r, int g, int lane) {
    const ANone::Dev none;
    f32x16 acc[Cfg::NACC];
#pragma unroll
    for (int i = 0; i < Cfg::NACC; ++i)
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[i][j] = 0.f;
    float* const sb = lds + BM * (BK + 4);
    xf.template prepare<LA, BM, BK, NT, LdA::KP>(m0, M, K);
#pragma clang loop unroll(disable)
    for (int t = 0; t < nkt; ++t) {
      a[0].load(ra, lda, m0, t * BK, M, K, xf);
      b[0].load(rb, ldb, n0, t * BK, N, K, none);
      xf.template advance<LA, BK>();
      __syncthreads();
      plain_store<BK>(a[0], xf, lds);
      plain_store<BK>(b[0], none, sb);
      __syncthreads();
#pragma clang loop unroll(disable)
      for (int j = 0; j < Cfg::KS * 8; ++j) {
        const int k = ((j >> 3) * Cfg::WK + wk) * 16 + 8 * g + (j & 7);
        float fa[Cfg::WTM], fb[Cfg::WTN];
#pragma unroll
        for (int i = 0; i < Cfg::WTM; ++i) fa[i] = lds[((wm * Cfg::WTM + i) * 32 + r) * (BK + 4) + k];
#pragma unroll
        for (int n = 0; n < Cfg::WTN; ++n) fb[n] = sb[((wn * Cfg::WTN + n) * 32 + r) * (BK + 4) + k];
#pragma unroll
        for (int i = 0; i < Cfg::WTM; ++i)
#pragma unroll
          for (int n = 0; n < Cfg::WTN; ++n)
            acc[i * Cfg::WTN + n] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i], fb[n], acc[i * Cfg::WTN + n], 0, 0, 0);
      }
    }
    __syncthreads();
    float again[Cfg::NACC][Cfg::CNT];
    finish(lds, rexp, false, acc, again, wm, wn, wk, r, g, lane);
#pragma unroll
    for (int tm = 0; tm < Cfg::WTM; ++tm)
#pragma unroll
      for (int tn = 0; tn < Cfg::WTN; ++tn) {
        const int col = BM + (wn * Cfg::WTN + tn) * 32 + r;
        const bool bad_col = SplitRows<LdB>::row_bad(rmax[col], rexp[col]);
#pragma unroll
        for (int j = 0; j < Cfg::CNT; ++j) {
          const int row = (wm * Cfg::WTM + tm) * 32 + acc_row(wk * Cfg::CNT + j, g);
          if (bad_col || SplitRows<LdA>::row_bad(rmax[row], rexp[row])) out[tm * Cfg::WTN + tn][j] = again[tm * Cfg::WTN + tn][j];
        }
      }
  }

  // Sums of one accumulator register over the K groups, in the order of the groups, and the exponent shift
  // back. Entered with the LDS stages free; the caller's next use of LDS follows a barrier of its own.
  __device__ __forceinline__ void finish(float* __restrict__ lds, const int* __restrict__ rexp, bool scaled,
                                         const f32x16 (&acc)[Cfg::NACC], float (&out)[Cfg::NACC][Cfg::CNT], int wm, int wn,
                                         int wk, int r, int g, int lane) const {
    constexpr int CNT = Cfg::CNT, WK = Cfg::WK, NACC = Cfg::NACC;
    if constexpr (WK > 1) {
      float* const base = lds + (size_t)((wm * Cfg::WN + wn) * WK) * (WK - 1) * NACC * CNT * 64;
      // slot of register j of tile t, from group `from`, kept for group `to`
      auto slot = [&](int to, int from, int t, int j) {
        const int f = from < to ? from : (from > to ? from - 1 : 0);   // (from == to: any slot, the value is not used)
        return (((to * (WK - 1) + f) * NACC + t) * CNT + j) * 64 + lane;
      };
#pragma unroll
      for (int w = 0; w < WK; ++w)
        if (w != wk) {
#pragma unroll
          for (int t = 0; t < NACC; ++t)
#pragma unroll
            for (int j = 0; j < CNT; ++j) base[slot(w, wk, t, j)] = acc[t][w * CNT + j];
        }
      __syncthreads();
#pragma unroll
      for (int t = 0; t < NACC; ++t)
#pragma unroll
        for (int j = 0; j < CNT; ++j) {
          float own = acc[t][j];
#pragma unroll
          for (int q = 1; q < WK; ++q) own = wk == q ? acc[t][q * CNT + j] : own;
          float sum = 0.f;
#pragma unroll
          for (int w = 0; w < WK; ++w) {
            const float other = base[slot(wk, w, t, j)];
            const float part = w == wk ? own : other;
            sum = w == 0 ? part : sum + part;
          }
          out[t][j] = sum;
        }
    } else {
#pragma unroll
      for (int t = 0; t < NACC; ++t)
#pragma unroll
        for (int j = 0; j < CNT; ++j) out[t][j] = acc[t][j];
    }
    if (!scaled) return;
#pragma unroll
    for (int tm = 0; tm < Cfg::WTM; ++tm)
#pragma unroll
      for (int tn = 0; tn < Cfg::WTN; ++tn) {
        const int ec = rexp[BM + (wn * Cfg::WTN + tn) * 32 + r] >> 1;
#pragma unroll
        for (int j = 0; j < CNT; ++j) {
          const int er = rexp[(wm * Cfg::WTM + tm) * 32 + acc_row(wk * CNT + j, g)] >> 1;
          out[tm * Cfg::WTN + tn][j] = __builtin_ldexpf(out[tm * Cfg::WTN + tn][j], -(er + ec));
        }
      }
  }

  // Column sums of A: the threads' shares (run's csum) added over the threads of a row, scale * sum + beta * old into
  // dst[row]. LDS must be free (the caller's barrier); whole workgroup.
  __device__ __forceinline__ void column_sums(const float* __restrict__ csum, float* __restrict__ lds, float* __restrict__ dst, int m0,
                                              int M, float scale, float beta) const {
    static_assert(LA == RCONTIG, "rows fast in memory");
    using Map = typename LdA::Map;
    constexpr int PARTS = BK / LdA::KP / 8;   // groups of eight lanes that share a row
#pragma unroll
    for (int j = 0; j < LdA::NS; ++j) {
      const float v = sum_over_8(csum[j]);
      const int k = Map::k((j / 4) * LdA::KP) / LdA::KP;   // which k group
      if ((k & 7) == 0) lds[(k >> 3) * BM + LdA::row_of(j)] = v;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < BM && m0 + i < M; i += NT) {
      float v = lds[i];
      for (int q = 1; q < PARTS; ++q) v += lds[q * BM + i];
      v *= scale;
      if (beta != 0.f) v += beta * dst[m0 + i];
      dst[m0 + i] = v;
    }
  }
};

// out[set][tile][j] of the wavefront to the epilogue, one 32 x 32 tile (CNT registers of it) at a time
template <class Cfg, int NSETS, class EpiDev>
__device__ __forceinline__ void split_epilogue(int M, int N, int m0, int n0, const float (*out)[Cfg::NACC][Cfg::CNT], EpiDev& epi) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wk = wave % Cfg::WK, wn = (wave / Cfg::WK) % Cfg::WN, wm = wave / (Cfg::WK * Cfg::WN);
#pragma unroll
  for (int tm = 0; tm < Cfg::WTM; ++tm)
#pragma unroll
    for (int tn = 0; tn < Cfg::WTN; ++tn) {
      float v[NSETS][Cfg::CNT];
#pragma unroll
      for (int s = 0; s < NSETS; ++s)
#pragma unroll
        for (int j = 0; j < Cfg::CNT; ++j) v[s][j] = out[s][tm * Cfg::WTN + tn][j];
      epi.template part<Cfg::CNT>(M, N, m0 + (wm * Cfg::WTM + tm) * 32, n0 + (wn * Cfg::WTN + tn) * 32 + (lane & 31), lane >> 5,
                                  wk * Cfg::CNT, v);
    }
}

// One product for a workgroup tile, handed to the epilogue (all 64 lanes of a wavefront together, see
// reduce_and_finish). colsum_dst (COLSUM; NULL: none) is written by the workgroups with n0 == 0.
template <class Cfg, int LA, int LB, bool VEC, bool COLSUM, class XfDev, class EpiDev>
__device__ __forceinline__ void split_product(const float* __restrict__ A, int64_t lda, const float* __restrict__ B, int64_t ldb, int M,
                                              int N, int K, int m0, int n0, float* __restrict__ lds, XfDev& xf, EpiDev& epi,
                                              float* __restrict__ colsum_dst, float colsum_scale, float colsum_beta) {
  SplitProduct<Cfg, LA, LB, VEC, XfDev> p;
  float out[Cfg::NACC][Cfg::CNT];
  float csum[COLSUM ? decltype(p)::LdA::NS : 1];
  p.template run<COLSUM>(A, lda, B, ldb, M, N, K, m0, n0, lds, xf, out, csum);
  split_epilogue<Cfg, 1>(M, N, m0, n0, &out, epi);
  if constexpr (COLSUM) {
    if (n0 == 0 && colsum_dst) {
      __syncthreads();
      p.column_sums(csum, lds, colsum_dst, m0, M, colsum_scale, colsum_beta);
    }
  }
}

}  // namespace mw
