// The tiles of the two-pair GEMM (numbers: kTiles in gemm.hip).
#include "gemm_pair.h"

namespace drf {

drf_status launch_gemm_pair(int tile, const bf16_t* A, const bf16_t* W, int M, int N, int K, const Epilogue& e, hipStream_t st, int m_first)
{
    switch (tile) {
    case 13: return launch_pair<256, 144, 3>(A, W, M, N, K, e, st, m_first);
    case 17: return launch_pair<64, 144, 4>(A, W, M, N, K, e, st, m_first);
    default: return launch_pair<128, 144, 4>(A, W, M, N, K, e, st, m_first);      // 8, 16
    }
}

}  // namespace drf
