// Launch of ffn_any.hip's grouped GEMM.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "locmoe.h"

namespace locmoe {

// C[rows, N] = epilogue(A[rows, K] . W[N, K]^T) per segment; rows_max: rows per segment at most, T: tokens (rows in all)
template <bool A_F32, bool PACKED, int EPI, bool OUT_F32>
int any_gemm(const void* A, const void* W, void* C, void* aux, const int32_t* seg_off, const int32_t* buf_expert, int E,
             int rows_max, int T, int Kdim, int Ndim, hipStream_t st);

// the largest of three times that overlap, a little more where they are alike
inline double soft_max(double a, double b, double c = 0.0) {
  return sqrt(sqrt(a * a * a * a + b * b * b * b + c * c * c * c));
}

// the tiles that it takes for a GEMM: at most bm rows x bn columns; weight tiles dealt to the XCDs, or in runs; 64-bit
// offsets inside a tile
struct AnyTiles {
  int bm, bn;
  bool dealt, far;
};
AnyTiles any_tiles(bool a_f32, bool packed, int E, int rows_max, int T, int Kdim, int Ndim);

// its expected time in us for bf16 activations, `rows` rows in every segment
double any_gemm_time(int E, int rows, int Kdim, int Ndim);

}  // namespace locmoe

// The kernel that takes a GEMM of desc (0: the first of the FFN and of the data gradients, the second with `keeps_z`;
// 1: the second), for example "ffn_gemm_any<192, 128, dealt>"; "" for a descriptor that is refused.  Not part of the
// interface: the tests and the bench ask by it which kernel a shape reaches, on a machine without a GPU as for 256 units.
extern "C" const char* locmoe_internal_ffn_kernel(const locmoe_desc* desc, int second, int keeps_z);
