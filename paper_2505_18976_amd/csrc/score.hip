// Dense contractions on the matrix cores: the attribute-stage score GEMM
// (Sec. 2.1: all-pair inner products of compressed gradients) and the dense
// Gaussian projection baseline (Sec. 2.2: g_hat = P g, P_ij ~ N(0, 1/k)).
//
// Both are C[M x N] (+)= A[M x K] * B[N x K]^T with A and B row-major and K
// contiguous ("NT" GEMM).  mode 0 (fp32) runs on gemm_split.hip; mode 1 (operands
// rounded to bf16) on the direct-to-LDS kernel of gemm_bf16.hip when there is a
// workspace for the rounded copies.  Without one the kernel below rounds while it
// stages: a workgroup of 4 wavefronts (2 x 2) computes a 128 x 128 tile of C; each
// wavefront owns 64 x 64 = 2 x 2 MFMA tiles of 32 x 32 (v_mfma_f32_32x32x16_bf16).
// K is consumed in slices of 32 staged through LDS, with the next slice
// prefetched into registers while the current one feeds the MFMAs.
// Workgroup ids are remapped so that each XCD (ids are dealt round-robin to the
// 8 XCDs) walks a contiguous range of tiles and re-uses its operands in its L2.
#include "gemm_f32.h"
#include "grass_device.h"

namespace grass {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int BM = 128, BN = 128, BK = 32;
constexpr int kGemmThreads = 256;
constexpr int kLdBf16 = BK + 8;    // bf16 per m-row (80 bytes)

struct GemmArgs {
    const float* A;   // M x K
    const float* B;   // N x K
    float* C;         // M x N
    uint64_t M, N, K, lda, ldb, ldc;
    uint32_t tiles_m, tiles_n;
    int accumulate;   // C += instead of C =
};

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (uint16_t)((u >> 16) | 0x40u);   // NaN stays NaN
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// Loads 4 consecutive k of one row with the widest access the alignment allows;
// out-of-range rows and k read as zero.
template <int V>
__device__ __forceinline__ float4 load4(const float* base, uint64_t ld, uint64_t row, uint64_t rows, uint64_t k0,
                                        uint64_t K) {
    float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
    if (row >= rows) return r;
    const float* p = base + row * ld + k0;
    if (k0 + 4 <= K) {
        if constexpr (V == 4) {
            r = *reinterpret_cast<const float4*>(p);
        } else if constexpr (V == 2) {
            const float2 a = *reinterpret_cast<const float2*>(p);
            const float2 b = *reinterpret_cast<const float2*>(p + 2);
            r = make_float4(a.x, a.y, b.x, b.y);
        } else {
            r = make_float4(p[0], p[1], p[2], p[3]);
        }
    } else {
        if (k0 + 0 < K) r.x = p[0];
        if (k0 + 1 < K) r.y = p[1];
        if (k0 + 2 < K) r.z = p[2];
        if (k0 + 3 < K) r.w = p[3];
    }
    return r;
}

template <int V>
__global__ void __launch_bounds__(kGemmThreads) __attribute__((amdgpu_waves_per_eu(3, 3))) gemm_nt_kernel(GemmArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;

    // XCD-aware tile order: consecutive logical tiles share the same B (train) tile.
    const uint32_t total = a.tiles_m * a.tiles_n;
    const uint32_t bid = blockIdx.x;
    const uint32_t per_xcd = (total + 7) / 8;
    uint32_t logical = (bid % 8) * per_xcd + bid / 8;
    if (total % 8 != 0) logical = bid;              // ragged grids keep the plain order
    if (logical >= total) return;
    const uint32_t tn = logical / a.tiles_m, tm = logical % a.tiles_m;
    const uint64_t m0 = (uint64_t)tm * BM, n0 = (uint64_t)tn * BN;

    // staging map: 8 lanes cover the 32 k of one row (coalesced 128-byte rows)
    const int kq = tid & 7;            // which group of 4 k
    const int r0 = tid >> 3;           // row 0..31, +32 per step

    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    float4 ra[4], rb[4];
    auto fetch = [&](uint64_t k0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            ra[i] = load4<V>(a.A, a.lda, m0 + r0 + 32 * i, a.M, k0 + kq * 4, a.K);
            rb[i] = load4<V>(a.B, a.ldb, n0 + r0 + 32 * i, a.N, k0 + kq * 4, a.K);
        }
    };

    const uint64_t nkt = (a.K + BK - 1) / BK;
    fetch(0);
    for (uint64_t kt = 0; kt < nkt; ++kt) {
        __syncthreads();    // everyone is done reading the previous slice
        uint16_t* As = reinterpret_cast<uint16_t*>(smem);      // [BM][kLdBf16]
        uint16_t* Bs = As + BM * kLdBf16;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = r0 + 32 * i;
            ushort4 pa, pb;
            pa.x = f32_to_bf16_rne(ra[i].x); pa.y = f32_to_bf16_rne(ra[i].y);
            pa.z = f32_to_bf16_rne(ra[i].z); pa.w = f32_to_bf16_rne(ra[i].w);
            pb.x = f32_to_bf16_rne(rb[i].x); pb.y = f32_to_bf16_rne(rb[i].y);
            pb.z = f32_to_bf16_rne(rb[i].z); pb.w = f32_to_bf16_rne(rb[i].w);
            *reinterpret_cast<ushort4*>(As + row * kLdBf16 + kq * 4) = pa;
            *reinterpret_cast<ushort4*>(Bs + row * kLdBf16 + kq * 4) = pb;
        }
        __syncthreads();
        if (kt + 1 < nkt) fetch((kt + 1) * BK);

#pragma unroll
        for (int kk = 0; kk < BK; kk += 16) {
            bf16x8 fa[2], fb[2];
#pragma unroll
            for (int i = 0; i < 2; ++i)
                fa[i] = *reinterpret_cast<const bf16x8*>(As + (wm * 64 + i * 32 + (lane & 31)) * kLdBf16 + kk +
                                                         (lane >> 5) * 8);
#pragma unroll
            for (int j = 0; j < 2; ++j)
                fb[j] = *reinterpret_cast<const bf16x8*>(Bs + (wn * 64 + j * 32 + (lane & 31)) * kLdBf16 + kk +
                                                         (lane >> 5) * 8);
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
        }
    }

    // accumulator element e of a lane: row 8*(e/4) + 4*(lane/32) + e%4, column lane%32
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const uint64_t col = n0 + wn * 64 + j * 32 + (lane & 31);
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const uint64_t row = m0 + wm * 64 + i * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
                if (row < a.M && col < a.N) {
                    float* c = a.C + row * a.ldc + col;
                    *c = a.accumulate ? *c + acc[i][j][e] : acc[i][j][e];
                }
            }
        }
}

static int vec_width(const float* p, uint64_t ld) {
    if (aligned(p, 16) && ld % 4 == 0) return 4;
    if (aligned(p, 8) && ld % 2 == 0) return 2;
    return 1;
}

// defined in gemm_bf16.hip: 256 x 256 tiles fed by direct-to-LDS loads
bool launch_gemm_dma(const void* A, const void* B, float* C, uint64_t M, uint64_t N, uint64_t K, uint64_t lda, uint64_t ldb,
                     uint64_t ldc, int accumulate, hipStream_t st, hipError_t* err, uint32_t splits, float* partials);
uint32_t gemm_dma_splits(uint64_t M, uint64_t N, uint64_t K, uint32_t max_splits);
hipError_t convert_to_bf16(const float* src, uint64_t rows, uint64_t cols, uint64_t cols_pad, uint64_t ld_src, uint16_t* dst,
                           uint64_t ld_dst, hipStream_t st);

static hipError_t launch_gemm_bf16_staged(const GemmArgs& a, hipStream_t st) {
    GemmArgs g = a;
    g.tiles_m = (uint32_t)ceil_div(a.M, BM);
    g.tiles_n = (uint32_t)ceil_div(a.N, BN);
    const uint64_t total = (uint64_t)g.tiles_m * g.tiles_n;
    if (total == 0 || total > 0x7FFFFFFFull) return hipErrorInvalidValue;
    int v = vec_width(a.A, a.lda);
    const int vb = vec_width(a.B, a.ldb);
    if (vb < v) v = vb;
    const size_t lds = (size_t)2 * BM * kLdBf16 * sizeof(uint16_t);
    dim3 grid((uint32_t)total), block(kGemmThreads);
    if (v == 4) hipLaunchKernelGGL(gemm_nt_kernel<4>, grid, block, lds, st, g);
    else if (v == 2) hipLaunchKernelGGL(gemm_nt_kernel<2>, grid, block, lds, st, g);
    else hipLaunchKernelGGL(gemm_nt_kernel<1>, grid, block, lds, st, g);
    return hipGetLastError();
}

// P[a, b] for b in [p0, p0+pc): one Box-Muller normal per hash, scaled to variance 1/k.
// blockIdx.x: a run of 256 columns, blockIdx.y (+ stride): rows.
// BF16: the value is rounded to bf16 (nearest even) and columns pc..pc_pad are zero-filled (whole K slices for the
// bf16 GEMM); otherwise pc_pad == pc.
template <bool BF16>
__global__ void __launch_bounds__(256) gauss_matrix_kernel(uint64_t sub, uint64_t p, uint32_t k, uint64_t p0,
                                                           uint64_t pc, uint64_t pc_pad, void* Pv, uint64_t ldP,
                                                           float inv_sqrt_k) {
    const uint64_t col = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (col >= pc_pad) return;
    for (uint32_t row = blockIdx.y; row < k; row += gridDim.y) {
        float v = 0.0f;
        if (col < pc) {
            const uint64_t h = sm(sub, (uint64_t)row * p + p0 + col);
            const float u1 = ((float)(uint32_t)(h >> 41) + 0.5f) * (1.0f / 8388608.0f);           // (0, 1), exact
            const float u2 = (float)(uint32_t)((h >> 16) & 0xFFFFFFu) * (1.0f / 16777216.0f);      // [0, 1)
            // hardware transcendentals: v_log_f32 is log2, v_cos_f32 takes its argument in revolutions (cos(2 pi u2))
            v = __builtin_amdgcn_sqrtf(-1.3862943611198906f * __builtin_amdgcn_logf(u1)) * __builtin_amdgcn_cosf(u2) * inv_sqrt_k;
        }
        if constexpr (BF16) static_cast<uint16_t*>(Pv)[(uint64_t)row * ldP + col] = f32_to_bf16_rne(v);
        else static_cast<float*>(Pv)[(uint64_t)row * ldP + col] = v;
    }
}

static void launch_gauss_matrix(uint64_t sub, uint64_t p, uint32_t k, uint64_t p0, uint64_t pc, uint64_t pc_pad, bool bf16,
                                void* P, uint64_t ldP, hipStream_t hs) {
    const uint32_t gx = (uint32_t)ceil_div(pc_pad, 256);
    uint32_t gy = k;                                   // about 16K workgroups keep every CU busy
    if ((uint64_t)gx * gy > 16384) gy = (uint32_t)(16384 / gx > 0 ? 16384 / gx : 1);
    if (gy > 65535) gy = 65535;
    const float scale = 1.0f / sqrtf((float)k);
    if (bf16)
        hipLaunchKernelGGL(gauss_matrix_kernel<true>, dim3(gx, gy), dim3(256), 0, hs, sub, p, k, p0, pc, pc_pad, P, ldP, scale);
    else
        hipLaunchKernelGGL(gauss_matrix_kernel<false>, dim3(gx, gy), dim3(256), 0, hs, sub, p, k, p0, pc, pc_pad, P, ldP, scale);
}

}  // namespace grass

using namespace grass;

// Workspace plan of grass_score: bf16 copies of both operands (mode 1) and K-range partial sums when the M x N
// output has too few tiles to fill the chip.
constexpr uint32_t kScoreMaxSplits = 64;      // K ranges of a score product with few output tiles: 8 tiles of 128 x 128 are
                                              // then two workgroups on each of 256 CUs
constexpr uint32_t kScoreMaxSplitsBf16 = 32;
struct ScorePlan {
    uint64_t kp;               // K rounded up to whole 64-byte bf16 slices
    size_t off_test, off_train, off_part, total;
    GemmCut f32;               // mode 0
    uint32_t splits;           // either mode (mode 0: of the columns behind f32.head_n)
};
static size_t up256s(size_t x) { return (x + 255) / 256 * 256; }
static ScorePlan score_plan(uint64_t N, uint64_t M, uint64_t K, int mode) {
    ScorePlan P;
    P.kp = (K + 31) / 32 * 32;
    size_t o = 0;
    P.off_test = o;  if (mode == 1) o += up256s((size_t)M * P.kp * 2);
    P.off_train = o; if (mode == 1) o += up256s((size_t)N * P.kp * 2);
    P.f32 = GemmCut{};
    if (mode == 0) { P.f32 = gemm_f32_cut(M, N, K, 0, kScoreMaxSplits); P.splits = P.f32.tail.splits; }
    else P.splits = ceil_div(M, 128) * ceil_div(N, 128) < 1024 && K >= 4096 ? gemm_dma_splits(M, N, P.kp, kScoreMaxSplitsBf16) : 1;
    P.off_part = o;  if (P.splits > 1) o += up256s((size_t)P.splits * M * (N - P.f32.head_n) * 4);
    P.total = o;
    return P;
}

extern "C" grass_status grass_score_workspace_bytes(uint64_t N, uint64_t M, uint64_t K, int compute_mode,
                                                    size_t* host_bytes) {
    if (!host_bytes || K == 0 || (compute_mode != 0 && compute_mode != 1)) return GRASS_EINVAL;
    *host_bytes = (N == 0 || M == 0) ? 0 : score_plan(N, M, K, compute_mode).total;
    return GRASS_OK;
}

extern "C" grass_status grass_score(const float* train, const float* test, int compute_mode, uint64_t N, uint64_t M,
                                    uint64_t K, uint64_t ld_train, uint64_t ld_test, float* scores,
                                    uint64_t ld_scores, void* ws, size_t ws_bytes, grass_stream stream) {
    if (K == 0 || (compute_mode != 0 && compute_mode != 1)) return GRASS_EINVAL;
    if (N == 0 || M == 0) return GRASS_OK;
    if (!train || !test || !scores || ld_train < K || ld_test < K || ld_scores < N) return GRASS_EINVAL;
    hipStream_t hs = as_stream(stream);
    const ScorePlan P = score_plan(N, M, K, compute_mode);
    const bool have_ws = ws != nullptr && ws_bytes >= P.total && P.total > 0;
    if (ws != nullptr && P.total > 0 && (ws_bytes < P.total || !aligned(ws, 256))) return GRASS_EWORKSPACE;
    unsigned char* base = static_cast<unsigned char*>(ws);
    float* partials = have_ws && P.splits > 1 ? reinterpret_cast<float*>(base + P.off_part) : nullptr;
    if (compute_mode == 0) {
        GemmCut cut = P.f32;
        if (!partials && P.splits > 1) cut = gemm_f32_cut(M, N, K, 0, 1);
        if (cut.head_n != 0) {
            if (gemm_f32(false, false, test, train, scores, M, cut.head_n, K, ld_test, ld_train, ld_scores, 0, 0, cut.head, nullptr,
                         hs) != hipSuccess)
                return GRASS_EHIP;
            train += cut.head_n * ld_train;
            scores += cut.head_n;
            N -= cut.head_n;
        }
        if (gemm_f32(false, false, test, train, scores, M, N, K, ld_test, ld_train, ld_scores, 0, 0, cut.tail, partials, hs) !=
            hipSuccess)
            return GRASS_EHIP;
    } else if (have_ws) {
        // round both operands once, then the bf16 direct-to-LDS kernel (zero-padded to whole K slices)
        uint16_t* te = reinterpret_cast<uint16_t*>(base + P.off_test);
        uint16_t* tr = reinterpret_cast<uint16_t*>(base + P.off_train);
        if (convert_to_bf16(test, M, K, P.kp, ld_test, te, P.kp, hs) != hipSuccess) return GRASS_EHIP;
        if (convert_to_bf16(train, N, K, P.kp, ld_train, tr, P.kp, hs) != hipSuccess) return GRASS_EHIP;
        hipError_t derr = hipSuccess;
        if (!launch_gemm_dma(te, tr, scores, M, N, P.kp, P.kp, P.kp, ld_scores, 0, hs, &derr, P.splits, partials) ||
            derr != hipSuccess)
            return GRASS_EHIP;
    } else {
        GemmArgs a;
        a.A = test; a.B = train; a.C = scores;
        a.M = M; a.N = N; a.K = K; a.lda = ld_test; a.ldb = ld_train; a.ldc = ld_scores;
        a.accumulate = 0;
        return launch_gemm_bf16_staged(a, hs) == hipSuccess ? GRASS_OK : GRASS_EHIP;
    }
    if (partials)
        hipLaunchKernelGGL(reduce_partials_kernel, dim3((uint32_t)ceil_div(M * N, 256)), dim3(256), 0, hs, partials, M,
                           (uint32_t)N, P.splits, 1.0f, scores, ld_scores);
    return launch_status();
}

extern "C" grass_status grass_gauss_matrix(uint64_t seed, uint64_t stream_id, uint64_t p, uint32_t k, uint64_t p0,
                                           uint64_t pc, float* P, uint64_t ldP, grass_stream stream) {
    if (p == 0 || k == 0 || pc == 0 || p0 + pc > p || !P || ldP < pc) return GRASS_EINVAL;
    if (ceil_div(pc, 256) > 0x7FFFFFFFull) return GRASS_EUNSUPPORTED;
    launch_gauss_matrix(substream(seed, stream_id), p, k, p0, pc, pc, false, P, ldP, as_stream(stream));
    return launch_status();
}

static uint64_t gauss_chunk(uint64_t p, uint64_t p_chunk) {
    uint64_t pc = p_chunk == 0 ? 8192 : p_chunk;
    pc = (pc + 31) / 32 * 32;              // whole 64-byte K slices of fp32 and of bf16
    return pc > p ? (p + 31) / 32 * 32 : pc;
}

// Workspace plan of grass_gauss_project.  mode 0: the fp32 chunk of P.  mode 1 (n, k >= 128): bf16 chunks of P and
// of g.  Both: K-range partial sums when the n x k output has too few tiles to fill the chip.
struct GaussPlan {
    uint64_t pc;
    uint32_t splits;           // K ranges of the first (largest) chunk's product; later chunks never use more
    GemmPlan f32;              // mode 0
    bool bf16_path;
    size_t off_p, off_g, off_part, total;
};
static GaussPlan gauss_plan(uint64_t n, uint64_t p, uint32_t k, uint64_t p_chunk, int mode) {
    GaussPlan G;
    G.pc = gauss_chunk(p, p_chunk);
    G.bf16_path = mode == 1 && n >= 128 && k >= 128;
    const uint64_t first = G.pc < p ? G.pc : p;
    G.splits = 1;
    G.f32 = GemmPlan{kTile128, 1, false};
    if (mode == 0) { G.f32 = gemm_f32_plan(false, false, n, k, first, 0, false, 8); G.splits = G.f32.splits; }
    else if (G.bf16_path && first % 32 == 0) G.splits = gemm_dma_splits(n, k, first, 8);
    size_t o = 0;
    G.off_p = o; o += up256s((size_t)k * G.pc * (G.bf16_path ? 2 : 4));
    G.off_g = o; if (G.bf16_path) o += up256s((size_t)n * G.pc * 2);       // a chunk of g rounded to bf16
    G.off_part = o; if (G.splits > 1) o += up256s((size_t)G.splits * n * k * 4);
    G.total = o;
    return G;
}

extern "C" grass_status grass_gauss_project_workspace_bytes(uint64_t n, uint64_t p, uint32_t k, uint64_t p_chunk,
                                                            size_t* host_bytes) {
    if (!host_bytes || p == 0 || k == 0) return GRASS_EINVAL;
    const size_t a = gauss_plan(n, p, k, p_chunk, 0).total, b = gauss_plan(n, p, k, p_chunk, 1).total;
    *host_bytes = a > b ? a : b;           // the mode is not an argument of the query: enough for either
    return GRASS_OK;
}

extern "C" grass_status grass_gauss_project(const float* g, uint64_t n, uint64_t p, uint64_t ldg, uint32_t k,
                                            uint64_t seed, uint64_t stream_id, uint64_t p_chunk, int compute_mode,
                                            float* out, uint64_t ldo, void* ws, size_t ws_bytes,
                                            grass_stream stream) {
    if (p == 0 || k == 0 || (compute_mode != 0 && compute_mode != 1)) return GRASS_EINVAL;
    if (n == 0) return GRASS_OK;
    if (!g || !out || ldg < p || ldo < k) return GRASS_EINVAL;
    GaussPlan G = gauss_plan(n, p, k, p_chunk, compute_mode);
    const uint64_t pc = G.pc;
    if (ceil_div(pc, 256) > 0x7FFFFFFFull) return GRASS_EUNSUPPORTED;
    if (!ws || ws_bytes < G.total || !aligned(ws, 256)) return GRASS_EWORKSPACE;
    unsigned char* base = static_cast<unsigned char*>(ws);
    float* partials = G.splits > 1 ? reinterpret_cast<float*>(base + G.off_part) : nullptr;
    hipStream_t hs = as_stream(stream);
    const uint64_t sub = substream(seed, stream_id);
    for (uint64_t p0 = 0; p0 < p; p0 += pc) {
        const uint64_t cur = p0 + pc <= p ? pc : p - p0;
        const int accumulate = p0 != 0;
        if (G.bf16_path) {
            // P and g chunks rounded to bf16 once (zero-padded to whole K slices), bf16 matrix cores, fp32 accumulation
            const uint64_t cur_pad = (cur + 31) / 32 * 32;
            uint16_t* Pb = reinterpret_cast<uint16_t*>(base + G.off_p);
            uint16_t* gb = reinterpret_cast<uint16_t*>(base + G.off_g);
            launch_gauss_matrix(sub, p, k, p0, cur, cur_pad, true, Pb, pc, hs);
            if (convert_to_bf16(g + p0, n, cur, cur_pad, ldg, gb, pc, hs) != hipSuccess) return GRASS_EHIP;
            uint32_t s_cur = G.splits > 1 ? gemm_dma_splits(n, k, cur_pad, G.splits) : 1;
            if (s_cur > G.splits) s_cur = G.splits;
            float* C = G.splits > 1 ? partials : out;
            const uint64_t ldc = G.splits > 1 ? k : ldo;
            hipError_t derr = hipSuccess;
            if (!launch_gemm_dma(gb, Pb, C, n, k, cur_pad, pc, pc, ldc, accumulate, hs, &derr, s_cur,
                                 s_cur > 1 ? partials : nullptr) || derr != hipSuccess)
                return GRASS_EHIP;
            continue;
        }
        float* P = reinterpret_cast<float*>(base + G.off_p);
        launch_gauss_matrix(sub, p, k, p0, cur, cur, false, P, pc, hs);
        if (compute_mode == 0) {
            GemmPlan plan = G.f32;
            if (p0 != 0 && cur != pc) plan = gemm_f32_plan(false, false, n, k, cur, 0, false, G.splits);     // a short tail
            float* C = G.splits > 1 ? partials : out;          // one range left: into partial sum 0
            if (gemm_f32(false, false, g + p0, P, C, n, k, cur, ldg, pc, G.splits > 1 ? k : ldo, accumulate, 0, plan, partials,
                         hs) != hipSuccess)
                return GRASS_EHIP;
        } else {
            GemmArgs a;
            a.A = g + p0; a.B = P; a.C = out;
            a.M = n; a.N = k; a.K = cur; a.lda = ldg; a.ldb = pc; a.ldc = ldo;
            a.accumulate = accumulate;
            if (launch_gemm_bf16_staged(a, hs) != hipSuccess) return GRASS_EHIP;
        }
    }
    if (G.splits > 1) {
        const uint64_t total = n * (uint64_t)k;
        if (ceil_div(total, 256) > 0x7FFFFFFFull) return GRASS_EUNSUPPORTED;
        hipLaunchKernelGGL(reduce_partials_kernel, dim3((uint32_t)ceil_div(total, 256)), dim3(256), 0, hs, partials, n, k,
                           G.splits, 1.0f, out, ldo);
    }
    return launch_status();
}
