// fp32 products of the library (gemm_split.hip, gemm_pair.hip): operands of any alignment and row distance, any M, N, K > 0.
#pragma once

#include <hip/hip_runtime.h>

#include "gemm_f32_plan.h"

namespace grass {

hipError_t gemm_f32(bool a_kn, bool b_kn, const float* A, const float* B, float* C, uint64_t M, uint64_t N, uint64_t K,
                    uint64_t lda, uint64_t ldb, uint64_t ldc, int accumulate, int lower_only, const GemmPlan& plan,
                    float* partials, hipStream_t st);

}  // namespace grass
