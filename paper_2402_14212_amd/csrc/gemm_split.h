// fp32 products on the bf16 matrix unit (gfx950): every fp32 operand value is split into the sum of three bf16 values
// while its tile is staged, and a product a b is formed from the six largest of the nine products of parts in
// v_mfma_f32_32x32x16_bf16, sums in fp32.
//
// What it is for. v_mfma_f32_32x32x2_f32 does 64 flop per clock and SIMD; the bf16 instruction does 1024, so six of
// them take 3/8 of the time. Measured (MI355X): 1024 x 4096 x 4096 in 177 us (194 TFLOP/s)
// against 250 us with fp32 instructions, 2048 x 2048 x 2048 in 94 us against 137 us, 1408 x 1536 x 1024 in 41 us against 57 us.
// What bounds it then: the bf16 unit at the clock that its own power draw allows (1.2 PFLOP/s of bf16 at the first
// size), LDS traffic (6 bytes an element) and, for small outputs, one workgroup on a CU. Two fp16 halves with a scale
// for each row are three products (127 us), but hold a value only relative to its row's largest: with reciprocal
// scales along K of 2^-12 .. 2^12 their error was 3e-3 of sum |a b|.
//
// Accuracy. v = hi + mid + lo exactly, each part the bf16 next to what is left: a part takes eight bits of the 24, its
// sign one more. Left out are a_mid b_lo, a_lo b_mid and a_lo b_lo, together at most 2^-24 |a b| (|mid| <= 2^-8 |v|,
// |lo| <= 2^-17 |v|): about one rounding of one product, whatever the other terms of the sum are. A term by itself is exact:
// its products of parts are added from the smallest to the largest, so that the partial sums are the low ends of v.
// The rounding of the running fp32 sum is less than with fp32 instructions, because an instruction adds sixteen
// products at a time. Normwise error against fp64 for N(0, 1) operands, K = 128 / 512 / 2048:
// 1.1e-7 / 2.4e-7 / 4.9e-7, with the fp32 instruction 2.0e-7 / 4.1e-7 / 8.1e-7 (5.7e-7 with K split in two).
//
// Sign. The bf16 unit brings the products of an instruction and the running sum to one exponent and rounds what falls
// off downwards, whatever its sign (measured: the error has the same mean for A B and -A B). Products of lower parts
// have bits there, so that every result came out low by 1.5e-7 of the results' rms (K = 4096), a fifth of its rounding
// error. A weight gradient, a sum over samples, averages rounding errors but not that: 2.2e-4 off, four layers after a
// re-seed at width 4096 (fp32 instructions 1.4e-4). So one half of K is summed with A negated: the running sum changes
// its sign every SPLIT_TURN K tiles, and the K groups have opposite ones. The means of the two halves cancel (3e-10
// is left, and the gradient is 1.3e-4 off); it costs 1 % of the time.
//
// Range. bf16 has fp32's exponents, but the lower parts of values below 2^-110 would fall under its subnormals. So both
// operands are multiplied by 2^SPLIT_UP on their way (exact; the least part of the least subnormal is then a normal
// bf16) and the result is scaled back. Values from 2^(127 - SPLIT_UP) on, infinities, NaN and sums beyond
// 2^(127 - 2 SPLIT_UP) then do not give a finite result: a workgroup that sees one, from operands large enough for
// it, computes its tile again with fp32 instructions and takes those results for the elements concerned. The time depends on the
// data otherwise only where the result is a pre-activation (see NearZero).
#pragma once

#include <type_traits>

#include "gemm_f32.h"

namespace mw {

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
  static constexpr int PLANE = (BM + BN) * BK * 2;  // bytes of one part of a staged K tile
  static constexpr int STAGE = 3 * PLANE;
  static constexpr int PARKED = NT * NACC * (16 - CNT) * 4;
  static constexpr int MAIN = 2 * STAGE > PARKED ? 2 * STAGE : PARKED;
  static constexpr int LDS_BYTES = MAIN + 16;   // + flags
  static_assert((BM + BN) * (BK + 4) * 4 <= 2 * STAGE, "the fp32 repeat stages its tile in the same memory");
};
// Shapes that were fastest over the layer sizes in use (us at M x N x K; 512 threads each, one workgroup to a CU):
//   Split256  4096 x 4096 x 1024 (TN): 188 (128 x 128: 200)
//   Split128  2048 x 2048 x 2048: 94 (64 x 64: 150), 2048 x 2048 x 512 (TN): 30 (64 x 64: 51)
//   Split64   1024 x 1024 x 1024: 22.5 (128 x 128: 38.6)
using Split256 = SplitCfg<2, 2, 4, 2, 1, 2>;  // 256 x 128, K tile 32
using Split128 = SplitCfg<2, 2, 2, 2, 2, 1>;  // 128 x 128, K tile 32, K split over two groups of four wavefronts
using Split64 = SplitCfg<1, 1, 2, 2, 2, 2>;   //  64 x  64, K tile 64, likewise

using Split64Q = SplitCfg<1, 1, 2, 2, 1, 2>;  // 64 x 64, K tile 32, four wavefronts, three to a CU: gathers, see gather_tile

template <class Cfg>
constexpr bool is_split() { return Cfg::PREC == 2; }

constexpr int SPLIT_UP = 24;   // see `Range` above
constexpr int SPLIT_TURN = 4;  // see `Sign` above: K tiles in a row of one sign (even)
__device__ __forceinline__ float split_up(bool negative) { return negative ? -(float)(1 << SPLIT_UP) : (float)(1 << SPLIT_UP); }

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

// The three parts of x and y, two bf16 to a word (x in the lower half); top (TOP): the largest magnitude seen, NaN aside
struct SplitPair { uint32_t part[3]; };
__device__ __forceinline__ uint32_t bf16_pair(float x, float y) {
  uint32_t d;
  asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(d) : "v"(x), "v"(y));
  return d;
}
template <bool TOP = true>
__device__ __forceinline__ SplitPair split_pair(float x, float y, float up, float& top) {
  SplitPair p;
  x *= up;
  y *= up;
  if (TOP) top = fmaxf(fmaxf(fabsf(x), fabsf(y)), top);
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    p.part[i] = bf16_pair(x, y);
    if (i < 2) {   // (exact: what is left of a value that was rounded to nearest)
      x -= __uint_as_float(p.part[i] << 16);
      y -= __uint_as_float(p.part[i] & 0xFFFF0000u);
    }
  }
  return p;
}
// sum + the squares of two bf16 (the shifted values are those that split_pair takes away; with v_dot2_f32_bf16 1024 x 4096 x 4096
// takes 3 us more)
__device__ __forceinline__ float add_squares(uint32_t pair, float sum) {
  const float x = __uint_as_float(pair << 16), y = __uint_as_float(pair & 0xFFFF0000u);
  return fmaf(x, x, fmaf(y, y, sum));
}
// combine over the eight lanes of an aligned group of eight
__device__ __forceinline__ float dpp_f32(float v, int quad_or_mirror) {
  const int i = __float_as_int(v);
  int r;
  switch (quad_or_mirror) {
    case 0: r = __builtin_amdgcn_update_dpp(i, i, 0xB1, 0xF, 0xF, false); break;   // lane ^ 1
    case 1: r = __builtin_amdgcn_update_dpp(i, i, 0x4E, 0xF, 0xF, false); break;   // lane ^ 2
    default: r = __builtin_amdgcn_update_dpp(i, i, 0x141, 0xF, 0xF, false); break; // the other half of eight (mirrored)
  }
  return __int_as_float(r);
}
__device__ __forceinline__ float sum_over_8(float v) {
#pragma unroll
  for (int k = 0; k < 3; ++k) v += dpp_f32(v, k);
  return v;
}

// One operand tile, R rows x BK k, in registers.
template <int LAYOUT, int R, int BK, int NT, bool VEC, class XfDev>
struct SplitLoader {
  static constexpr int NV = R * BK / 4 / NT;                        // 4-element chunks per thread
  static constexpr int KP = LAYOUT == KCONTIG ? 1 : (NV >= 4 ? 4 : 2);  // rows fast in memory: consecutive k in one thread
  static constexpr int NTASK = NV / KP;
  static constexpr int NS = LAYOUT == KCONTIG ? NV : 4 * NTASK;     // rows per thread
  static_assert(NV * 4 * NT == R * BK && NV % KP == 0, "tile must divide evenly over the workgroup");
  using Map = ChunkMap<LAYOUT, R, BK, NT, KP>;

  float4 v[NV];
  typename XfDev::Aux aux[NV];
  uint32_t code[VEC ? 1 : NV];

  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, int64_t ld, int row0, int k0, int n_rows, int n_k,
                                       const XfDev& xf) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int r = row0 + Map::row(i), k = k0 + Map::k(i);
      const Chunk c = LAYOUT == KCONTIG ? xf.template chunk<LAYOUT>(i, r, k, n_rows, n_k, ld)
                                        : xf.template chunk<LAYOUT>(i, k, r, n_k, n_rows, ld);
      const uint32_t total = VEC ? 0u : extent_bytes(LAYOUT == KCONTIG ? n_rows : n_k, LAYOUT == KCONTIG ? n_k : n_rows, ld) / 4u;
      if (VEC) v[i] = buf_load_f32x4(rs, c.nvalid ? c.e * 4u : OOB);
      else v[i] = load_chunk<false>(rs, c, total, code[i]);
      xf.template fetch<VEC, false>(aux[i], c, total);
    }
  }

  // chunk i as it is staged
  __device__ __forceinline__ float4 value(int i, const XfDev& xf) const {
    const float4 w = xf.apply(v[i], aux[i]);
    return VEC ? w : mend_chunk(w, code[VEC ? 0 : i]);
  }

  static __device__ __forceinline__ int row_of(int j) { return LAYOUT == KCONTIG ? Map::row(j) : Map::row((j / 4) * KP) + (j & 3); }
};

// Split the staged values of `ld` into the planes of an LDS stage (`base`: this operand's rows of the first plane). SIGNED:
// operand A, negated if `negative` and, once more, where the second K group reads it. COLSUM, SQUARES: csum gets the sums of the values
// or of the squares of their first parts, by row; the latter stand in for the largest magnitude. scale: a power of two.
template <class Cfg, bool SIGNED, bool COLSUM, bool SQUARES, class Ld, class XfDev>
__device__ __forceinline__ void split_store(const Ld& ld, const XfDev& xf, char* __restrict__ base, float* __restrict__ csum,
                                            float& top, bool negative, float scale = (float)(1 << SPLIT_UP)) {
  static_assert(!(COLSUM && SQUARES), "one or the other");
  using Map = typename Ld::Map;
  constexpr int BK = Cfg::BK, NT = Cfg::NT, PLANE = Cfg::PLANE;
  // (k: the same 16-k step for all of a chunk)
  auto up = [&](int k) { return SIGNED && (negative != (Cfg::WK == 2 && ((k >> 4) & 1))) ? -scale : scale; };
  if constexpr (Ld::KP == 1) {
#pragma unroll
    for (int i = 0; i < Ld::NV; ++i) {
      const float4 w = ld.value(i, xf);
      const SplitPair a = split_pair<!SQUARES>(w.x, w.y, up(Map::k(0)), top), b = split_pair<!SQUARES>(w.z, w.w, up(Map::k(0)), top);
      if (SQUARES) csum[i] = add_squares(b.part[0], add_squares(a.part[0], csum[i]));
      // a thread's chunks are the same k of rows so far apart that they have the same pattern of chunks
      static_assert(NT * 4 / BK % (BK == 32 ? 32 : 16) == 0, "see split_addr");
      char* p = base + split_addr<BK>(Map::row(0), Map::k(0) >> 3) + (Map::k(0) & 4) * 2 + i * (NT * 4 / BK) * BK * 2;
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        u32x2 d;
        d.x = a.part[q];
        d.y = b.part[q];
        *reinterpret_cast<u32x2*>(p + q * PLANE) = d;
      }
    }
  } else {
#pragma unroll
    for (int j = 0; j < Ld::NTASK; ++j) {
      float e[4][Ld::KP];
#pragma unroll
      for (int kk = 0; kk < Ld::KP; ++kk) {
        const float4 w = ld.value(j * Ld::KP + kk, xf);
        e[0][kk] = w.x;
        e[1][kk] = w.y;
        e[2][kk] = w.z;
        e[3][kk] = w.w;
      }
      const int k = Map::k(j * Ld::KP), row = Map::row(j * Ld::KP);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        SplitPair s[Ld::KP / 2];
#pragma unroll
        for (int h = 0; h < Ld::KP / 2; ++h) {
          const float x = e[q][2 * h], y = e[q][2 * h + 1];
          if (COLSUM) csum[4 * j + q] += x + y;
          s[h] = split_pair<!SQUARES>(x, y, up(k), top);
          if (SQUARES) csum[4 * j + q] = add_squares(s[h].part[0], csum[4 * j + q]);
        }
        char* p = base + split_addr<BK>(row + q, k >> 3) + (k & 7) * 2;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          if constexpr (Ld::KP == 4) {
            u32x2 d;
            d.x = s[0].part[i];
            d.y = s[1].part[i];
            *reinterpret_cast<u32x2*>(p + i * PLANE) = d;
          } else {
            *reinterpret_cast<uint32_t*>(p + i * PLANE) = s[0].part[i];
          }
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
    const float4 w = ld.value(i, xf);
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

// Pre-activations next to zero (an epilogue with NEAR_ZERO). The sign of a pre-activation selects a linear piece of the network,
// so that one which rounding takes over zero changes gradients by a finite step, however small the error. A value that
// lies, with its bias, within NEAR_ERROR sqrt(K) |a| |b| of zero, a and b its row of A and its column of B, is therefore formed again
// in 64 bits by the whole wavefront. The line stands on the operands themselves (the squares of their first parts are added up while
// they are staged), so that it holds at the edges of the matrix, next to rows of any size and where sums cancel. The largest errors
// seen over sqrt(K) |a| |b|, among two million values each, K = 1024 .. 8192: 1e-9 .. 3e-9 for N(0, 1) operands, 1.4e-8 where the terms
// of one half of K have one sign and those of the other half the other, 1.2e-8 where two terms of 1000 times the others' size
// cancel, 1.9e-8 where the two groups of K have sums of opposite sign.
// Of N(0, 1) values 3.2e-8 K are that near: 0.3 of a wavefront's 2048 at K = 4096. What it costs: 1024 x
// 4096 x 4096 206 us instead of 194, about half of it the squares, half the sums; 131072 x 128 x 1152 283 instead of 275.
// More than NEAR_MOST in one wavefront (sums that cancel all over; a column that is near zero in all rows, as in deep networks whose
// rows have become alike, is 32), or rows so small or large that their squares leave
// fp32: the workgroup's tile is formed again with fp32 instructions, as the pre-activations of smaller layers are. Rows and
// columns of zeros are exact and not concerned; nor are values that are exactly zero where a wavefront has more than NEAR_MOST of them,
// since that is not rounding but operands whose products are zeros (identities, masks, blocks). Apart from that a value depends on its row, its column and the tile alone, and a
// product that is formed again elsewhere with the same tile has the same bits.
// Signs that differ from the 64-bit network's, twelve inputs each, with fp32 products and here: five layers of 2500 .. 2301 on 1500
// rows 58 and 43, six of 2048 on 1024 43 and 37, of 3000 on 700 63 and 42, of 4096 on 1024 (eleven) 146 and 94; none in the first layer here.
// What is left comes from the rounding of the layers' inputs, as it does with fp32 products.
constexpr float NEAR_ERROR = 4e-8f;
constexpr int NEAR_MOST = 64;
constexpr float NEAR_SQUARES_MIN = 0x1p-100f, NEAR_SQUARES_MAX = 0x1p120f;   // (of the values as they are staged, times a power of two)

template <class EpiDev, class = void>
struct near_zero : std::false_type {};
template <class EpiDev>
struct near_zero<EpiDev, std::enable_if_t<EpiDev::NEAR_ZERO>> : std::true_type {};

// the float next to v in the direction of the sign
__device__ __forceinline__ float next_float(float v, bool upwards) {
  if (v == 0.f) return upwards ? 0x1p-149f : -0x1p-149f;
  const uint32_t u = __float_as_uint(v);
  return __uint_as_float((v > 0.f) == upwards ? u + 1 : u - 1);
}

template <class Cfg>
struct NearZero {
  static constexpr int PARTS = 2;                           // of a column of B, at most
  static constexpr int FLOATS = Cfg::BM + PARTS * Cfg::BN;  // for A's rows and B's columns, in LDS behind what is parked
  static_assert(Cfg::WK == 2 && Cfg::BK == 32 && Cfg::NACC * Cfg::CNT <= 64 && Cfg::PARKED + FLOATS * 4 <= Cfg::MAIN,
                "a barrier between the squares and their use, eight lanes to a row, one flag a value");
  static __device__ __forceinline__ float* place(float* lds) { return lds + Cfg::PARKED / 4; }

  // One operand's squares from the threads' shares: the norms of KCONTIG rows, squares in parts R apart of others.
  template <class Ld, int LAYOUT, int R>
  static __device__ __forceinline__ void gather(const float* __restrict__ share, float* __restrict__ dst) {
    static_assert(LAYOUT == KCONTIG || Cfg::BK / Ld::KP / 8 == PARTS, "see column_sums");
#pragma unroll
    for (int j = 0; j < Ld::NS; ++j) {
      const float v = sum_over_8(share[j]);
      const int k = LAYOUT == KCONTIG ? 0 : Ld::Map::k((j / 4) * Ld::KP) / Ld::KP;
      if (((int)threadIdx.x & 7) == 0) dst[(k >> 3) * R + Ld::row_of(j)] = LAYOUT == KCONTIG ? norm(v) : v;
    }
  }
  // |.| of the values as staged; what is too small or too large is infinite, for find() below
  static __device__ __forceinline__ float norm(float squares) {
    const float n = __builtin_amdgcn_sqrtf(squares);
    return squares > NEAR_SQUARES_MAX || (squares > 0.f && squares < NEAR_SQUARES_MIN) ? __builtin_inff() : n;
  }

  // out and bias (epi's, of this lane's columns): times the powers of two of both operands. The values of a wavefront that are formed again (bit i * CNT + j: out[i][j]); all: its
  // tile is to be. (Rows and columns outside the matrix are zeros, and so are their results.)
  template <int LB>
  static __device__ __forceinline__ unsigned long long find(int K, const float (&bias)[Cfg::WTN], const float* __restrict__ norms,
                                                            const float (&out)[Cfg::NACC][Cfg::CNT], bool& all) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 31, g = lane >> 5;
    const int wk = wave % Cfg::WK, wn = (wave / Cfg::WK) % Cfg::WN, wm = wave / (Cfg::WK * Cfg::WN);
    const float c = NEAR_ERROR * __builtin_amdgcn_sqrtf((float)K);
    float line[Cfg::WTN];
#pragma unroll
    for (int tn = 0; tn < Cfg::WTN; ++tn) {
      const float* p = norms + Cfg::BM + (wn * Cfg::WTN + tn) * 32 + r;
      line[tn] = c * (LB == RCONTIG ? norm(p[0] + p[Cfg::BN]) : p[0]);
    }
    uint32_t flags[2] = {0, 0}, zeros[2] = {0, 0};
    bool outside = false;
#pragma unroll
    for (int tm = 0; tm < Cfg::WTM; ++tm)
#pragma unroll
      for (int j = 0; j < Cfg::CNT; ++j) {
        const float a = norms[(wm * Cfg::WTM + tm) * 32 + acc_row(wk * Cfg::CNT + j, g)];
#pragma unroll
        for (int tn = 0; tn < Cfg::WTN; ++tn) {
          const int bit = (tm * Cfg::WTN + tn) * Cfg::CNT + j;
          const float v = out[tm * Cfg::WTN + tn][j], near = line[tn] * a;
          // (infinite, or zero because of an underflow; 0 times infinity is a row of zeros beside one that is too large: NaN)
          outside |= near == __builtin_inff() || (near == 0.f && v != 0.f);
          flags[bit >> 5] |= fabsf(v + bias[tn]) < near ? 1u << (bit & 31) : 0u;
          zeros[bit >> 5] |= v == 0.f ? 1u << (bit & 31) : 0u;
        }
      }
    unsigned long long found = flags[0] | (unsigned long long)flags[1] << 32;
    int count = 0;
    if (__ballot(found != 0)) {
      const unsigned long long zero = found & (zeros[0] | (unsigned long long)zeros[1] << 32);
      int none = __popcll(zero);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) none += __shfl_xor(none, o);
      if (none > NEAR_MOST) found &= ~zero;
      count = __popcll(found);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) count += __shfl_xor(count, o);
    }
    all = outside || count > NEAR_MOST;
    return found;
  }

  template <int Q>
  static __device__ __forceinline__ void load(float (&v)[Q], __amdgpu_buffer_rsrc_t rs, uint32_t off) {
    if constexpr (Q == 4) {
      const float4 w = buf_load_f32x4(rs, off);
      v[0] = w.x;
      v[1] = w.y;
      v[2] = w.z;
      v[3] = w.w;
    } else {
      v[0] = buf_load_f32(rs, off);
    }
  }

  // whole wavefronts; VEC: K is a multiple of four
  template <int LB, bool VEC, class XfDev>
  static __device__ __forceinline__ void form_again(unsigned long long flags, __amdgpu_buffer_rsrc_t ra, int64_t lda, __amdgpu_buffer_rsrc_t rb,
                                                    int64_t ldb, int K, int m0, int n0, const XfDev& xf, const float (&bias)[Cfg::WTN],
                                                    float (&out)[Cfg::NACC][Cfg::CNT]) {
    constexpr int AT_ONCE = LB == KCONTIG ? 8 : 5;   // in flight: 2048 k, or 1280
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wk = wave % Cfg::WK, wn = (wave / Cfg::WK) % Cfg::WN, wm = wave / (Cfg::WK * Cfg::WN);
    unsigned long long some = __ballot(flags != 0);
    while (some) {
      const int from = __builtin_amdgcn_readfirstlane((int)__builtin_ctzll(some));
      const uint32_t lower = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)flags, from);
      const uint32_t upper = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(flags >> 32), from);
      const int which = lower ? __builtin_ctz(lower) : 32 + __builtin_ctz(upper);
      const int i = which / Cfg::CNT, j = which % Cfg::CNT;
      const int row = m0 + (wm * Cfg::WTM + i / Cfg::WTN) * 32 + acc_row(wk * Cfg::CNT + j, from >> 5);
      const int col = n0 + (wn * Cfg::WTN + i % Cfg::WTN) * 32 + (from & 31);
      // four k a lane; where rows end inside such four, one
      constexpr int Q = VEC ? 4 : 1, STEP = 64 * Q;
      double sum = 0.0;
#pragma clang loop unroll(disable)
      for (int k0 = Q * lane; k0 - Q * lane < K; k0 += STEP * AT_ONCE) {
        float va[AT_ONCE][Q], vb[AT_ONCE][Q];
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u) {
          const int k = k0 + STEP * u;
          load<Q>(va[u], ra, k < K ? xf.place(row, k, lda) : OOB);
          if (LB == KCONTIG) {
            load<Q>(vb[u], rb, k < K ? ((uint32_t)col * (uint32_t)ldb + (uint32_t)k) * 4u : OOB);
          } else {
#pragma unroll
            for (int q = 0; q < Q; ++q) vb[u][q] = buf_load_f32(rb, k < K ? ((uint32_t)(k + q) * (uint32_t)ldb + (uint32_t)col) * 4u : OOB);
          }
        }
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u)
#pragma unroll
          for (int q = 0; q < Q; ++q) sum += (double)va[u][q] * (double)vb[u][q];
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
      // the epilogue adds the bias in fp32, exactly where the two are next to each other: the float beside the sum where
      // the sum's own rounding would change the sign
      float b = bias[0];
#pragma unroll
      for (int tn = 1; tn < Cfg::WTN; ++tn) b = i % Cfg::WTN == tn ? bias[tn] : b;
      float v = (float)sum;
      const bool positive = sum + (double)b > 0.0;
      if ((v + b > 0.f) != positive) v = next_float(v, positive);   // (lane `from` has that column's bias)
#pragma unroll
      for (int w = 0; w < Cfg::NACC * Cfg::CNT; ++w)
        if (w == which && lane == from) out[w / Cfg::CNT][w % Cfg::CNT] = v;
      if (lane == from) flags &= ~(1ull << which);
      some = __ballot(flags != 0);
    }
  }
};

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
  // epi: where the results are pre-activations, those next to zero are formed again (NearZero).
  // A workgroup's first use of LDS; it may be reused after the caller's next barrier.
  template <bool COLSUM, class EpiDev>
  __device__ __forceinline__ void run(const float* __restrict__ A, int64_t lda, const float* __restrict__ B, int64_t ldb, int M,
                                      int N, int K, int m0, int n0, float* __restrict__ lds_f, XfDev& xf,
                                      float (&out)[Cfg::NACC][Cfg::CNT], float* __restrict__ csum, const EpiDev& epi) {
    constexpr bool NEAR = near_zero<EpiDev>::value;
    char* const lds = reinterpret_cast<char*>(lds_f);
    uint32_t* const flag = reinterpret_cast<uint32_t*>(lds + Cfg::MAIN);  // not finite, largest magnitudes of A and B, all again
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wk = wave % Cfg::WK, wn = (wave / Cfg::WK) % Cfg::WN, wm = wave / (Cfg::WK * Cfg::WN);
    const int r = lane & 31, g = lane >> 5;

    const uint32_t bytes_a = LA == KCONTIG ? xf.extent(M, K, lda) : xf.extent(K, M, lda);
    const uint32_t bytes_b = LB == KCONTIG ? extent_bytes(N, K, ldb) : extent_bytes(K, N, ldb);
    const __amdgpu_buffer_rsrc_t ra = make_rsrc(A, bytes_a), rb = make_rsrc(B, bytes_b);
    const ANone::Dev none;
    const int nkt = (K + BK - 1) / BK;
    float top_a = 0.f, top_b = 0.f;
    f32x16 acc[Cfg::NACC];
#pragma unroll
    for (int i = 0; i < Cfg::NACC; ++i)
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[i][j] = 0.f;
    if (COLSUM) {
#pragma unroll
      for (int j = 0; j < LdA::NS; ++j) csum[j] = 0.f;
    }
    float sq_a[NEAR ? LdA::NS : 1], sq_b[NEAR ? LdB::NS : 1];   // squares of the rows this thread stages
    if constexpr (NEAR) {
#pragma unroll
      for (int j = 0; j < LdA::NS; ++j) sq_a[j] = 0.f;
#pragma unroll
      for (int j = 0; j < LdB::NS; ++j) sq_b[j] = 0.f;
    }
#define MW_REQUEST(slot, idx)                       \
  do {                                              \
    a[slot].load(ra, lda, m0, (idx) * BK, M, K, xf); \
    b[slot].load(rb, ldb, n0, (idx) * BK, N, K, none); \
    xf.template advance<LA, BK>();                  \
  } while (0)
    xf.template prepare<LA, BM, BK, NT, LdA::KP>(m0, M, K);
    MW_REQUEST(0, 0);
    MW_REQUEST(1, 1);
    if (threadIdx.x < (NEAR ? 4 : 3)) flag[threadIdx.x] = 0;
    const float up_a = NEAR ? near_scale(flag + 1, xf, lane) : (float)(1 << SPLIT_UP);

    // idx: the K tile
#define MW_TO_LDS(slot, stage, idx)                                                                                          \
  do {                                                                                                                       \
    split_store<Cfg, true, COLSUM, NEAR>(a[slot], xf, lds + (stage) * Cfg::STAGE, NEAR ? sq_a : csum, top_a, ((idx) / SPLIT_TURN) & 1, up_a); \
    split_store<Cfg, false, false, NEAR>(b[slot], none, lds + (stage) * Cfg::STAGE + BM * BK * 2, NEAR ? sq_b : (float*)nullptr, top_b, false); \
  } while (0)
#define MW_MULTIPLY(stage) multiply(lds + (stage) * Cfg::STAGE, wm, wn, wk, r, g, acc)
    MW_TO_LDS(0, 0, 0);
    MW_REQUEST(0, 2);
    __syncthreads();
    // tile t is in LDS stage t % 2, the registers hold tiles t + 1 and t + 2. The last tile is peeled off: after it
    // nothing is staged.
#define MW_STEP(u)                                   \
  do {                                               \
    MW_MULTIPLY(u);                                  \
    MW_TO_LDS(1 - (u), 1 - (u), t + (u) + 1);        \
    MW_REQUEST(1 - (u), t + (u) + 3);                \
    __syncthreads();                                 \
  } while (0)
    int t = 0;
    for (; t + 2 < nkt; t += 2) {
      turn(t, acc);
      MW_STEP(0);
      MW_STEP(1);
    }
    turn(t, acc);
    if (t + 1 < nkt) {   // two tiles are left, or one
      MW_STEP(0);
      MW_MULTIPLY(1);
    } else {
      MW_MULTIPLY(0);
    }
    if ((t / SPLIT_TURN) & 1) negate(acc);
#undef MW_STEP
#undef MW_TO_LDS
#undef MW_MULTIPLY
#undef MW_REQUEST
    // Add the K groups. A wavefront keeps CNT registers of every tile and hands the others over through LDS.
    __syncthreads();   // the stages are free
    using Near = NearZero<Cfg>;
    float bias[NEAR ? Cfg::WTN : 1];
    if constexpr (NEAR) {
#pragma unroll
      for (int tn = 0; tn < Cfg::WTN; ++tn) bias[tn] = epi.bias_of(n0 + (wn * Cfg::WTN + tn) * 32 + r, N);
      Near::template gather<LdA, LA, BM>(sq_a, Near::place(lds_f));
      Near::template gather<LdB, LB, BN>(sq_b, Near::place(lds_f) + BM);
    }
    finish<true>(lds_f, acc, out, wm, wn, wk, lane);
    static_assert(SPLIT_UP == 24, "both operands");
    if constexpr (NEAR) {
      bool all = false;
      float scaled[Cfg::WTN];
#pragma unroll
      for (int tn = 0; tn < Cfg::WTN; ++tn) scaled[tn] = bias[tn] * up_a * 0x1p24f;   // (infinite: far from any sum)
      const unsigned long long near = Near::template find<LB>(K, scaled, Near::place(lds_f), out, all);
      if (all) flag[3] = 1;
      __syncthreads();
      if (__builtin_amdgcn_readfirstlane(flag[3]) != 0) {
        repeat_f32<true>(ra, lda, rb, ldb, M, N, K, m0, n0, lds_f, xf, out, nkt, wm, wn, wk, r, g, lane);
        return;
      }
      const float down = 1.f / up_a;
#pragma unroll
      for (int i = 0; i < Cfg::NACC; ++i)
#pragma unroll
        for (int j = 0; j < Cfg::CNT; ++j) out[i][j] = out[i][j] * 0x1p-24f * down;
      Near::template form_again<LB, VEC>(near, ra, lda, rb, ldb, K, m0, n0, xf, bias, out);
      return;   // (no part and no sum can have overflowed: what is not finite has met a NaN)
    }
    bool finite = true;
#pragma unroll
    for (int i = 0; i < Cfg::NACC; ++i)
#pragma unroll
      for (int j = 0; j < Cfg::CNT; ++j) {
        finite &= fabsf(out[i][j]) < __builtin_inff();
        out[i][j] *= 0x1p-24f * 0x1p-24f;
      }
    if (!finite) *flag = 1;
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(flag[0]) == 0) return;
    // Operands so small that neither a part nor a sum can have overflowed: what is not finite has met a NaN, and fp32
    // instructions would say the same (a network whose training has diverged takes no longer than another)
    atomicMax(flag + 1, __float_as_uint(top_a));
    atomicMax(flag + 2, __float_as_uint(top_b));
    __syncthreads();
    top_a = __uint_as_float(flag[1]);
    top_b = __uint_as_float(flag[2]);
    if (top_a < 0x1p126f && top_b < 0x1p126f && top_a * top_b * (float)K < 0x1p126f) return;
    repeat_f32<false>(ra, lda, rb, ldb, M, N, K, m0, n0, lds_f, xf, out, nkt, wm, wn, wk, r, g, lane);
  }

  // The power of two that brings the first K tile of A next to one (activations of deep networks shrink layer by layer to where
  // their squares would be zero). Rows may then be 2^50 smaller and values 2^50 larger. peak: a word of LDS that holds zero after the next barrier.
  __device__ __forceinline__ float near_scale(uint32_t* __restrict__ peak, const XfDev& xf, int lane) const {
    float m = 0.f;
#pragma unroll
    for (int i = 0; i < LdA::NV; ++i) {
      const float4 w = a[0].value(i, xf);
      m = fmaxf(fmaxf(fmaxf(fabsf(w.x), fabsf(w.y)), fmaxf(fabsf(w.z), fabsf(w.w))), m);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    __syncthreads();
    if (lane == 0) atomicMax(peak, __float_as_uint(m));
    __syncthreads();
    const uint32_t u = (uint32_t)__builtin_amdgcn_readfirstlane((int)*peak);
    int e = 127 - (int)(u >> 23);
    e = u == 0 || u >= 0x7F800000u ? 0 : (e < -100 ? -100 : (e > 120 ? 120 : e));
    return __uint_as_float((uint32_t)(127 + e) << 23);
  }

  static __device__ __forceinline__ void negate(f32x16 (&acc)[Cfg::NACC]) {
#pragma unroll
    for (int i = 0; i < Cfg::NACC; ++i)
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[i][j] = -acc[i][j];
  }
  // before K tile t (even) is multiplied
  static __device__ __forceinline__ void turn(int t, f32x16 (&acc)[Cfg::NACC]) {
    static_assert(Cfg::WK <= 2 && SPLIT_TURN % 2 == 0, "one sign or two");
    if (t > 0 && t % SPLIT_TURN == 0) negate(acc);
  }

  __device__ __forceinline__ void multiply(const char* __restrict__ st, int wm, int wn, int wk, int r, int g,
                                           f32x16 (&acc)[Cfg::NACC]) const {
#pragma unroll
    for (int ks = 0; ks < Cfg::KS; ++ks) {
      const int c = (ks * Cfg::WK + wk) * 2 + g;   // the groups take the 16-k steps in turn
      // rows 32 apart have the same pattern of chunks (split_addr)
      const char* sa = st + split_addr<BK>(r, c) + wm * Cfg::WTM * 32 * BK * 2;
      const char* sb = st + split_addr<BK>(r, c) + (BM + wn * Cfg::WTN * 32) * BK * 2;
      bf16x8 fa[3][Cfg::WTM], fb[3][Cfg::WTN];
#pragma unroll
      for (int p = 0; p < 3; ++p) {
#pragma unroll
        for (int i = 0; i < Cfg::WTM; ++i)
          fa[p][i] = *reinterpret_cast<const bf16x8*>(sa + p * Cfg::PLANE + i * 32 * BK * 2);
#pragma unroll
        for (int i = 0; i < Cfg::WTN; ++i)
          fb[p][i] = *reinterpret_cast<const bf16x8*>(sb + p * Cfg::PLANE + i * 32 * BK * 2);
      }
      // from the smallest to the largest: parts (a, b) = (0, 2), (2, 0), (1, 1), (0, 1), (1, 0), (0, 0)
#pragma unroll
      for (int q = 0; q < 6; ++q) {
        constexpr int PA[6] = {0, 2, 1, 0, 1, 0}, PB[6] = {2, 0, 1, 1, 0, 0};
#pragma unroll
        for (int i = 0; i < Cfg::WTM; ++i)
#pragma unroll
          for (int j = 0; j < Cfg::WTN; ++j)
            acc[i * Cfg::WTN + j] =
                __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[PA[q]][i], fb[PB[q]][j], acc[i * Cfg::WTN + j], 0, 0, 0);
      }
    }
  }

  // The product again with fp32 instructions, one K tile at a time through registers and LDS, for the elements that are
  // not finite or for all. Rare, so simple.
  template <bool ALL>
  __device__ __forceinline__ void repeat_f32(__amdgpu_buffer_rsrc_t ra, int64_t lda, __amdgpu_buffer_rsrc_t rb, int64_t ldb, int M, int N,
                                             int K, int m0, int n0, float* __restrict__ lds, XfDev& xf,
                                             float (&out)[Cfg::NACC][Cfg::CNT], int nkt, int wm, int wn, int wk, int r, int g,
                                             int lane) {
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
    finish<false>(lds, acc, again, wm, wn, wk, lane);
#pragma unroll
    for (int i = 0; i < Cfg::NACC; ++i)
#pragma unroll
      for (int j = 0; j < Cfg::CNT; ++j)
        if (ALL || !(fabsf(out[i][j]) < __builtin_inff())) out[i][j] = again[i][j];
  }

  // Sums of one accumulator register over the K groups, in the order of the groups (SIGNED: the second group's taken away,
  // see `Sign` above). Entered with the LDS stages free;
  // the caller's next use of LDS follows a barrier of its own.
  template <bool SIGNED>
  __device__ __forceinline__ void finish(float* __restrict__ lds, const f32x16 (&acc)[Cfg::NACC],
                                         float (&out)[Cfg::NACC][Cfg::CNT], int wm, int wn, int wk, int lane) const {
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
            sum = w == 0 ? part : (SIGNED ? sum - part : sum + part);
          }
          out[t][j] = sum;
        }
    } else {
#pragma unroll
      for (int t = 0; t < NACC; ++t)
#pragma unroll
        for (int j = 0; j < CNT; ++j) out[t][j] = acc[t][j];
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
  p.template run<COLSUM>(A, lda, B, ldb, M, N, K, m0, n0, lds, xf, out, csum, epi);
  split_epilogue<Cfg, 1>(M, N, m0, n0, &out, epi);
  if constexpr (COLSUM) {
    if (n0 == 0 && colsum_dst) {
      __syncthreads();
      p.column_sums(csum, lds, colsum_dst, m0, M, colsum_scale, colsum_beta);
    }
  }
}

}  // namespace mw
