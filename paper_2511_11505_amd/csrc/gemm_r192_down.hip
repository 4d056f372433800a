// The bf16 down pass of gemm_r192.hpp (a file of its own, so that the two
// compile side by side: 21 s each).
#include "gemm_r192.hpp"

namespace fs {

void launch_r192_down(const void* A, const int32_t* rows, const int32_t* goff, int G,
                    int64_t m_total, const void* B, int K, int NOUT, void* C, int ldc, int cus,
                    int hmax, hipStream_t s) {
  run_r192<MODE_DOWN, false>(A, rows, goff, G, m_total, B, K, NOUT, C, ldc, cus, hmax, nullptr, nullptr, s);
}

}  // namespace fs
