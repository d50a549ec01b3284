// Tile dispatch shared by the gemm_*.hip translation units.
#pragma once
#include "gemm_kernels.h"
#include "mw_internal.h"

namespace mw {

// Which tiles a launcher can be asked for (each one is a kernel): every tile (the kernel-level entry point takes fp32
// tiles by name), those of pick_tile_z, those of pick_tile_f32 and pick_tile, those of weight gradients.
enum TileSet { TILES_ALL, TILES_Z, TILES_LAYER, TILES_DW };

template <int LA, int LB, bool COLSUM, TileSet SET, class Xf, class Epi>
inline hipError_t dispatch_gemm(int tile, int M, int N, int K, const float* A, int64_t lda, const float* B,
                                int64_t ldb, const Xf& xf, const Epi& epi, float* colsum_out,
                                float colsum_scale, hipStream_t stream, float colsum_beta = 0.f) {
#define MW_LAUNCH_TILE(CFG)                                                                                            \
  return launch_gemm<CFG, LA, LB, Xf, Epi, COLSUM>(M, N, K, A, lda, B, ldb, xf, epi, colsum_out, colsum_scale, \
                                                   stream, colsum_beta)
  if (tile == TILE_AUTO) tile = LA == RCONTIG ? pick_tile_tn(M, N, K) : pick_tile(M, N, K);
  switch (tile) {
    case TILE_64: MW_LAUNCH_TILE(Tile64);
    case TILE_128W8: MW_LAUNCH_TILE(Tile128W8);
    case TILE_64X128: MW_LAUNCH_TILE(Tile64x128);
    default: break;
  }
  if constexpr (!COLSUM && SET != TILES_DW) {
    if (tile == TILE_FINE) MW_LAUNCH_TILE(FineCfg);
    if (tile == TILE_FINE_K4) MW_LAUNCH_TILE(FineK4Cfg);
  }
  if (tile == TILE_S128) MW_LAUNCH_TILE(Split128);
  if constexpr (SET != TILES_Z)
    if (tile == TILE_S64) MW_LAUNCH_TILE(Split64);
  if constexpr (SET != TILES_DW) {
    if (tile == TILE_32K4) MW_LAUNCH_TILE(Tile32K4);
    if (tile == TILE_64K2) MW_LAUNCH_TILE(Tile64K2);
  }
  if constexpr (SET == TILES_ALL || SET == TILES_DW)
    if (tile == TILE_128) MW_LAUNCH_TILE(Tile128);
  if constexpr (LA == RCONTIG)
    if (tile == TILE_S256) MW_LAUNCH_TILE(Split256);
  if constexpr (SET == TILES_ALL)
    if (tile == TILE_32K8) MW_LAUNCH_TILE(Tile32K8);
#undef MW_LAUNCH_TILE
  return hipErrorInvalidValue;
}

}  // namespace mw
