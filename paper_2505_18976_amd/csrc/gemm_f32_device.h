// What the fp32 product kernels (gemm_split.hip, gemm_pair.hip) share: arguments, numbering of the tiles, barrier.
#pragma once

#include "gemm_f32.h"
#include "grass_device.h"

namespace grass {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));    // a 16-byte load needs only 4-byte alignment here
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

struct GemmF32Args {
    const float* A;       // M x K, or K x M (AKN)
    const float* B;       // N x K, or K x N (BKN)
    float* C;             // M x N
    uint64_t M, N, K, lda, ldb, ldc;
    uint32_t tiles_m, tiles_n;
    int accumulate;              // C += instead of C =
    int lower_only;              // symmetric product: tiles strictly above the diagonal are skipped
    uint32_t splits;             // split-K: workgroup (split, tile) contracts one of `splits` contiguous ranges of K
    uint64_t split_stride_c;     //          into C + split*split_stride_c
    const float* weight = nullptr;      // gemm_f32_pair_weighted: K rounded up to 32 factors of the columns of A, 16-byte aligned
};

__device__ __forceinline__ void f32_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

__device__ __forceinline__ void wait_lds() { __builtin_amdgcn_s_waitcnt(0xC07F); }   // lgkmcnt == 0, others free

// Tile and K range of this workgroup.
struct GemmTile { uint32_t tm, tn, split; };
__device__ __forceinline__ GemmTile gemm_f32_tile(const GemmF32Args& a) {
    const uint32_t total = a.lower_only ? a.tiles_m * (a.tiles_m + 1) / 2 : a.tiles_m * a.tiles_n;
    uint32_t split = blockIdx.x / total;
    uint32_t bid = blockIdx.x - split * total;
    uint32_t logical = bid;
    if (a.splits % 8 == 0) {                                              // a K range stays on one XCD: operands are read
        const uint32_t w = blockIdx.x / 8;                                // into one L2 only
        split = (w / total) * 8 + blockIdx.x % 8;
        logical = w % total;
    } else if (total % 8 == 0) {
        logical = (bid % 8) * (total / 8) + bid / 8;                      // consecutive tiles stay on one XCD
    }
    uint32_t tn, tm;
    if (a.lower_only) {                                                   // tiles on or below the diagonal, row by row
        tm = (uint32_t)((sqrtf(8.0f * (float)logical + 1.0f) - 1.0f) * 0.5f);
        while (tm * (tm + 1) / 2 > logical) --tm;
        while ((tm + 1) * (tm + 2) / 2 <= logical) ++tm;
        tn = logical - tm * (tm + 1) / 2;
    } else if (total % 256 == 0 && a.tiles_m % 8 == 0 && a.tiles_n % 4 == 0 && a.tiles_m >= 16) {
        const uint32_t block = logical >> 5, within = logical & 31, blocks_m = a.tiles_m / 8;   // 8 x 4 tiles per XCD
        tm = (block % blocks_m) * 8 + (within & 7);
        tn = (block / blocks_m) * 4 + (within >> 3);
    } else {
        tn = logical / a.tiles_m;
        tm = logical % a.tiles_m;
    }
    return GemmTile{tm, tn, split};
}

// What the backward product R = C G of a Selective-Mask step is for: the gradient of its columns,
// grad[c] = 2 sigma sigma' sum_t Gt[t][c] R[t][c] - lambda sigma' with sigma = sigmoid(S[c] inv_temp).
struct GradTail {
    const float* Gt;
    uint64_t ldgt;
    const float* S;
    float inv_temp, lambda;
    float* grad;
};
// (A * weight) B^T for at most 128 rows of A, K ranges as in GemmPlan.
hipError_t gemm_f32_pair_weighted(const GemmF32Args& a, hipStream_t st);
// The product A B (B K-major, at most 128 rows of A, not accumulated) straight to the gradient; C is scratch for tiles that
// have to be computed again.
hipError_t gemm_f32_pair_grad(const GemmF32Args& a, const GradTail& g, hipStream_t st);

// gemm_pair.hip: tile as in GemmPlan, row distances for which gemm_f32_wide is false.
hipError_t gemm_f32_pair(bool a_kn, bool b_kn, int tile, const GemmF32Args& a, hipStream_t st);

}  // namespace grass
