// Launch of ffn_any.hip's grouped GEMM.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace locmoe {

// C[rows, N] = epilogue(A[rows, K] . W[N, K]^T) per segment; rows_max: rows per segment at most, T: tokens (rows in all)
template <bool A_F32, bool PACKED, int EPI, bool OUT_F32>
int any_gemm(const void* A, const void* W, void* C, void* aux, const int32_t* seg_off, const int32_t* buf_expert, int E,
             int rows_max, int T, int Kdim, int Ndim, hipStream_t st);

// the largest of three times that overlap, a little more where they are alike
inline double soft_max(double a, double b, double c = 0.0) {
  return sqrt(sqrt(a * a * a * a + b * b * b * b + c * c * c * c));
}

// its expected time in us for bf16 activations, `rows` rows in every segment
double any_gemm_time(int E, int rows, int Kdim, int Ndim);

}  // namespace locmoe
