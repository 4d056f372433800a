// The FP8 passes of gemm_r192.hpp.
#include "gemm_r192.hpp"

namespace fs {

void launch_r192_fp8(bool gateup, const uint8_t* A, const int32_t* rows, const int32_t* goff, int G,
                     int64_t m_total, const uint8_t* B, int K, int NOUT, void* C, int ldc, int cus,
                     int hmax, const float* sA, const float* sB, hipStream_t s) {
  if (gateup)
    run_r192<MODE_GATEUP, true>(A, rows, goff, G, m_total, B, K, NOUT, C, ldc, cus, hmax, sA, sB, s);
  else
    run_r192<MODE_DOWN, true>(A, rows, goff, G, m_total, B, K, NOUT, C, ldc, cus, hmax, sA, sB, s);
}

}  // namespace fs
