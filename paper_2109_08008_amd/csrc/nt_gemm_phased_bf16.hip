// The phased tiles of nt_gemm_phased.h for one element type (a unit each, to build in parallel).
#include "nt_gemm_phased.h"

namespace nt {

hipError_t gemm_phased_bf16(const void* A, int lda, const void* Bt, int M, int N, int K, const GemmEpi& epi,
                       hipStream_t s, int role, int bm) {
  return launch_roles<bf16>(A, lda, Bt, M, N, K, epi, s, role, bm);
}

}  // namespace nt
