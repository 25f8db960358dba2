// The 64x32 phased tile of nt_gemm_phased.h for fp32, and 64x64 (a unit of its own, to build in
// parallel).
#include "nt_gemm_phased.h"

namespace nt {

hipError_t gemm_slim_f32(const void* A, int lda, const void* Bt, int M, int N, int K, const GemmEpi& epi,
                         hipStream_t s, int role, int bn) {
  if (role == 1) {
    if (epi.lnf_colsum) return launch_slim<float, 2, 6, 1, true>(A, lda, Bt, M, N, K, epi, s);
    return launch_slim<float, 2, 6, 1, false>(A, lda, Bt, M, N, K, epi, s);
  }
  if (role != 0 || epi.lnf_colsum) return hipErrorInvalidValue;
  return bn == 64 ? launch_slim<float, 4, 4, 0, false>(A, lda, Bt, M, N, K, epi, s)
                  : launch_slim<float, 2, 6, 0, false>(A, lda, Bt, M, N, K, epi, s);
}

}  // namespace nt
