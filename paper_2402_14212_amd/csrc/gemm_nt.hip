// NT products: C[M][N] = A[M][K] B[N][K]^T (forward pre-activations, affine vijp, Gram matrix).
#include "gemm_dispatch.h"

namespace mw {

hipError_t gemm_plain_nt(int tile, int M, int N, int K, float alpha, const float* A, int64_t lda, const float* B,
                         int64_t ldb, float beta, float* C, int64_t ldc, const float* bias, hipStream_t stream) {
  EpiStore epi{C, ldc, alpha, beta, bias};
  return dispatch_gemm<KCONTIG, KCONTIG, false, TILES_ALL>(tile, M, N, K, A, lda, B, ldb, ANone{}, epi, nullptr, 0.f, stream);
}

hipError_t gemm_fwd_act(int tile, int M, int N, int K, const float* X, const float* W, const float* bias,
                        float alpha, float* Xout, uint64_t* mask, hipStream_t stream, float* Zkeep) {
  if (mask) {
    if (N % 32 != 0) return hipErrorInvalidValue;
    EpiFwdAct<true> epi{Xout, bias, alpha, reinterpret_cast<uint32_t*>(mask), Zkeep};
    return dispatch_gemm<KCONTIG, KCONTIG, false, TILES_Z>(tile, M, N, K, X, K, W, K, ANone{}, epi, nullptr, 0.f, stream);
  }
  EpiFwdAct<false> epi{Xout, bias, alpha, nullptr, Zkeep};
  return dispatch_gemm<KCONTIG, KCONTIG, false, TILES_Z>(tile, M, N, K, X, K, W, K, ANone{}, epi, nullptr, 0.f, stream);
}

namespace {
template <class Cfg, bool VEC>
hipError_t fwd_and_mask_t(int M, int N, int K, const float* X, const float* W, const EpiFwdAct<false>& epi, const MaskTask<Cfg::NT>& m,
                          hipStream_t stream) {
  auto t = make_gemm_task<Cfg, KCONTIG, KCONTIG, VEC, ANone, EpiFwdAct<false>, false>(M, N, K, X, K, W, K, ANone{}, epi, nullptr, 0.f);
  return launch_task_pair<Cfg::NT>(t, m, stream);
}
template <class Cfg>
hipError_t fwd_and_mask(int M, int N, int K, const float* X, const float* W, const EpiFwdAct<false>& epi, const float* mask_of, int64_t n_of,
                        uint64_t* mask, hipStream_t stream) {
  const MaskTask<Cfg::NT> m{mask_of, n_of, mask};
  return operand_vec_ok(K) ? fwd_and_mask_t<Cfg, true>(M, N, K, X, W, epi, m, stream)
                           : fwd_and_mask_t<Cfg, false>(M, N, K, X, W, epi, m, stream);
}
}  // namespace

hipError_t gemm_fwd_act_and_mask(int tile, int M, int N, int K, const float* X, const float* W, const float* bias, float alpha, float* Xout,
                                 const float* mask_of, int64_t n_of, uint64_t* mask, hipStream_t stream, uint64_t* more) {
  const EpiFwdAct<false> epi{Xout, bias, alpha, nullptr, nullptr};
  if (extent_ok(M, K, K) && extent_ok(N, K, K) && extent_ok(M, N, N) && (int64_t)(M < N ? M : N) * K >= 4 && n_of > 0) switch (tile) {
    case TILE_FINE: return fwd_and_mask<FineCfg>(M, N, K, X, W, epi, mask_of, n_of, mask, stream);
    case TILE_FINE_K4: return fwd_and_mask<FineK4Cfg>(M, N, K, X, W, epi, mask_of, n_of, mask, stream);
    case TILE_32K4: return fwd_and_mask<Tile32K4>(M, N, K, X, W, epi, mask_of, n_of, mask, stream);
    case TILE_64: return fwd_and_mask<Tile64>(M, N, K, X, W, epi, mask_of, n_of, mask, stream);
    default: break;
  }
  *more += 1;
  hipError_t e = ew_mask_from_act(mask_of, n_of, mask, stream);
  return e != hipSuccess ? e : gemm_fwd_act(tile, M, N, K, X, W, bias, alpha, Xout, nullptr, stream);
}

hipError_t gemm_fwd_again(int tile, int M, int N, int K, const float* X, const float* W, const float* bias, float alpha, float* Xout,
                          const uint64_t* mask, unsigned long long* mismatches, hipStream_t stream) {
  EpiFwdAgain epi{Xout, bias, alpha, reinterpret_cast<const uint32_t*>(mask), mismatches};
  return dispatch_gemm<KCONTIG, KCONTIG, false, TILES_Z>(tile, M, N, K, X, K, W, K, ANone{}, epi, nullptr, 0.f, stream);
}

}  // namespace mw
