// The 288-column form of the GEMM's 256-row tiles (a file each: they are the longest to compile).
#include "gemm_wide.h"

namespace drf {

drf_status launch_gemm_wide_288(const bf16_t* A, const bf16_t* W, int M, int N, int K, const Epilogue& e, hipStream_t st, int m_first)
{
    return launch_wide_mode<256, 288>(A, W, M, N, K, e, st, m_first);
}

}  // namespace drf
