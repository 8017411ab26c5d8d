// fp32 products of the library (gemm_split.hip, gemm_pair.hip): operands of any alignment and row distance, any M, N, K > 0.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace grass {

// 256 x 256, 128 x 128, 64 x 512, 128 x 256 (only with two fp16 pieces, A row-major)
enum : int { kTile256 = 0, kTile128 = 1, kTile64 = 2, kTile128x256 = 3 };
struct GemmPlan {
    int tile;
    uint32_t splits;
    bool pair;                   // two fp16 pieces (gemm_pair.hip) instead of three bf16 ones
    double us = 0.0;             // estimated time
};
// A product cut after `head_n` columns of C: `head` covers the columns before (none if head_n == 0), `tail` the others.
struct GemmCut {
    uint64_t head_n;
    GemmPlan head, tail;
};

// 16 rows so far apart that their byte offsets need more than 32 bits: 15 ld and at most 256 columns, 4 bytes each, stay
// below 2^32 for every ld < 2^26
inline bool gemm_f32_wide(uint64_t ld) { return ld >= (1ull << 26); }

constexpr uint64_t kPairMinK = 256;      // k per workgroup from which on two fp16 pieces are used

GemmPlan gemm_f32_plan(bool a_kn, bool b_kn, uint64_t M, uint64_t N, uint64_t K, uint64_t ld_max, bool lower_only,
                       uint32_t max_splits);
// Columns of C that fill one round of the chip with the tile of `plan`.
uint64_t gemm_f32_round_columns(const GemmPlan& plan, uint64_t M);
GemmCut gemm_f32_cut(uint64_t M, uint64_t N, uint64_t K, uint64_t ld_max, uint32_t max_splits);
hipError_t gemm_f32(bool a_kn, bool b_kn, const float* A, const float* B, float* C, uint64_t M, uint64_t N, uint64_t K,
                    uint64_t lda, uint64_t ldb, uint64_t ldc, int accumulate, int lower_only, const GemmPlan& plan,
                    float* partials, hipStream_t st);

}  // namespace grass
