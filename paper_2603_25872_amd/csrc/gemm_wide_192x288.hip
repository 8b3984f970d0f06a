// The GEMM's tile of 192 rows x 288 columns: rounds of tiles that 256 x 256 leaves part-filled (see kTiles in gemm.hip).
#include "gemm_wide.h"

namespace drf {

drf_status launch_gemm_wide_192x288(const bf16_t* A, const bf16_t* W, int M, int N, int K, const Epilogue& e, hipStream_t st, int m_first)
{
    return launch_wide_mode<192, 288, false>(A, W, M, N, K, e, st, m_first);
}

}  // namespace drf
