// The 192-column form of the GEMM's 256-row tiles: rounds of tiles that 256 columns leave part-filled (see kTiles in gemm.hip).
#include "gemm_wide.h"

namespace drf {

drf_status launch_gemm_wide_192(const bf16_t* A, const bf16_t* W, int M, int N, int K, const Epilogue& e, hipStream_t st, int m_first)
{
    return launch_wide_mode<256, 192, false>(A, W, M, N, K, e, st, m_first);
}

}  // namespace drf
