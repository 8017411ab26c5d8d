// LoGra baseline: factorised dense projection Gauss_{k_in (x) k_out} for one
// linear layer (Sec. 3.3.2 "Recap on LoGra", Eq. (3)):
//     out_i = sum_t (P_in x_t) (x) (P_out g_t),   flat index a*k_out + b,
// with P_in (k_in x d_in) and P_out (k_out x d_out) dense (Gaussian) matrices
// supplied by the caller in bf16.  This is the method FactGraSS is compared with;
// it has to read every column of x and g, where FactGraSS reads k' of them.
//
// Bound: HBM (every byte of x and g once).  Two launches:
//   logra_project_kernel  a = X P_in^T and b = G P_out^T for all n T tokens at once: sample
//            borders do not matter here, so a workgroup takes 128 tokens of one factor and a
//            range of its columns, and the ranges are cut so that every CU is busy for about
//            the same time whatever the shape (few tokens, d_in != d_out).
//   logra_outer_kernel    out_i = sum_t a_t (x) b_t from the fp32 partial sums of the ranges
//            (out of the caches), on the fp32 matrix cores.
// A single kernel (logra_short.hip) gives each workgroup 64 tokens of one sample and all columns of both factors; it remains
// for calls whose two launches cost more than that, see short_logra.  7 x 1,000 tokens were 112 such workgroups, all as long
// as the wider factor.  Measured against it, kernels together (calls back to back):
//   7 x 1,000 tokens, 2,048 -> 8,192            82 -> 41 us (78 -> 40)
//   32 x 512 tokens, 4,096 -> 4,096             57 -> 53 us (54 -> 51); the projection reads at 5.7 TB/s
//   9 x 21 tokens, 2,224 -> 7,008               (53 -> 17, launches included)
#include "grass_device.h"

namespace grass {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// logra_short.hip
hipError_t launch_logra_short(const uint16_t* x, const uint16_t* g, uint64_t n, uint64_t T, uint32_t d_in, uint32_t d_out,
                              const uint16_t* pin, uint32_t k_in, const uint16_t* pout, uint32_t k_out, float* out, uint64_t ldo,
                              hipStream_t st);

constexpr int LP = 64;                 // projected width handled (k_in, k_out <= 64)
constexpr int kProjTokens = 128;       // tokens per workgroup of the projection
constexpr int kProjThreads = 512;
constexpr int kProjStages = 6;
constexpr int kProjStageBytes = (kProjTokens + LP) * 128;      // 64 columns of the token rows, then of the projection rows

__device__ __align__(16) const uint32_t g_logra_zeros[4] = {0u, 0u, 0u, 0u};

struct LograFactor {
    const uint16_t* src;               // tokens x d
    const uint16_t* proj;              // k x d
    uint32_t d, k;
    uint32_t groups, per_range;        // groups of 64 columns; groups per workgroup
    float* part;                       // [range][token][64]
};
struct LograProjectArgs {
    LograFactor f[2];                  // x, g
    uint64_t tokens;
    uint32_t tiles, ranges_x;
    uint32_t* counters;                // 16 per sample, cleared for the second kernel (none: 0 of them)
    uint32_t n_counters;
};

// 128 tokens x 64 projected columns.  Operands go memory -> LDS directly, 64 columns (128 bytes of a row) at a time through
// six stages: five groups (120 KB) stay in flight behind the one being multiplied.  Of the eight wavefronts, four per 64
// tokens, each multiplies its 16 of the 64 columns (token rows are read once from LDS, projection rows twice) and they add
// up at the end.  The 16-byte chunk c of row r sits at position c ^ ((r >> 1) & 7), so fragment reads are free of bank
// conflicts.  The token rows are read once from memory (non-temporal); the projection rows come out of L2.  Workgroups of a
// range start at different groups of it, or they would all ask the same L2 channels for the same projection columns at
// the same time.
__global__ void __launch_bounds__(kProjThreads) logra_project_kernel(LograProjectArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (blockIdx.x == 0)
        for (uint32_t i = threadIdx.x; i < a.n_counters; i += kProjThreads) a.counters[i] = 0;
    const uint32_t tile = blockIdx.x % a.tiles, all_ranges = blockIdx.x / a.tiles;
    const bool is_g = all_ranges >= a.ranges_x;                // uniform
    const uint32_t range = is_g ? all_ranges - a.ranges_x : all_ranges;
    const LograFactor f = is_g ? a.f[1] : a.f[0];
    const uint64_t t0 = (uint64_t)tile * kProjTokens;
    const uint32_t g_begin = range * f.per_range;
    const uint32_t len = g_begin + f.per_range < f.groups ? f.per_range : f.groups - g_begin;      // >= 1
    const uint32_t rot = tile * 5 % len;
    auto group_of = [&](uint32_t i) { const uint32_t q = i + rot; return g_begin + (q >= len ? q - len : q); };

    // load map: 24 instructions of 8 rows per stage, three per wavefront: two of token rows, one of projection rows.
    // Lane l moves the chunk at position l % 8 of row l / 8.
    const unsigned char* src[3];
    uint32_t cofs[3];                                          // byte offset of the lane's chunk inside the group
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const bool tok = j < 2;
        const int r = (tok ? wave * 16 + j * 8 : wave * 8) + (lane >> 3);      // row of the operand's tile
        const int kc = (lane & 7) ^ ((r >> 1) & 7);
        const uint64_t lim = tok ? a.tokens : f.k;             // rows past the end re-read the last one; never used
        uint64_t row = tok ? t0 + r : (uint64_t)r;
        row = row < lim ? row : lim - 1;
        src[j] = reinterpret_cast<const unsigned char*>(tok ? f.src : f.proj) + row * f.d * 2;
        cofs[j] = kc * 16;
    }
    const uint32_t row_bytes = f.d * 2;
    auto load = [&](uint32_t i, int stage) {
        const uint32_t gb = group_of(i) * 128;
        unsigned char* base = smem + stage * kProjStageBytes;
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const uint32_t b = gb + cofs[j];                   // columns past d count as zero
            const unsigned char* p = b < row_bytes ? src[j] + b : reinterpret_cast<const unsigned char*>(g_logra_zeros);
            unsigned char* l = base + (j < 2 ? wave * 2048 + j * 1024 : kProjTokens * 128 + wave * 1024);
            if (j < 2) __builtin_amdgcn_global_load_lds(reinterpret_cast<const uint32_t*>(p), reinterpret_cast<uint32_t*>(l), 16, 0, 2);
            else __builtin_amdgcn_global_load_lds(reinterpret_cast<const uint32_t*>(p), reinterpret_cast<uint32_t*>(l), 16, 0, 0);
        }
    };
    auto barrier = [] {                                        // no fence: later groups stay in flight across it
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
    const int half = wave >> 2, kstep = wave & 3;              // which 64 tokens, which 16 of a group's columns
    const int pos = ((2 * kstep + (lane >> 5)) ^ ((lane >> 1) & 7)) * 16;
    const int a_row = (half * 64 + (lane & 31)) * 128 + pos, b_row = (kProjTokens + (lane & 31)) * 128 + pos;

#pragma unroll
    for (uint32_t i = 0; i < kProjStages - 1; ++i)
        if (i < len) load(i, i);
    int stage = 0;
    for (uint32_t i = 0; i < len; ++i) {
        // the wavefront's part of group i has landed (three loads of each younger group may be in flight); behind the
        // barrier everybody's has, and everybody has finished reading the stage of group i - 1
        const uint32_t younger = len - 1 - i;
        if (younger >= 4) __builtin_amdgcn_s_waitcnt(0x0F7C);
        else if (younger == 3) __builtin_amdgcn_s_waitcnt(0x0F79);
        else if (younger == 2) __builtin_amdgcn_s_waitcnt(0x0F76);
        else if (younger == 1) __builtin_amdgcn_s_waitcnt(0x0F73);
        else __builtin_amdgcn_s_waitcnt(0x0F70);
        barrier();
        if (i + kProjStages - 1 < len) load(i + kProjStages - 1, stage == 0 ? kProjStages - 1 : stage - 1);
        const unsigned char* st = smem + stage * kProjStageBytes;
        bf16x8 tf[2], pf[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            tf[q] = *reinterpret_cast<const bf16x8*>(st + a_row + q * 32 * 128);
            pf[q] = *reinterpret_cast<const bf16x8*>(st + b_row + q * 32 * 128);
        }
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[q][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tf[q], pf[j], acc[q][j], 0, 0, 0);
        stage = stage == kProjStages - 1 ? 0 : stage + 1;
    }
    // sum of the four wavefronts of each half: [kstep][token][64] in the staging area
    __syncthreads();
    float* sums = reinterpret_cast<float*>(smem);
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e)
                sums[(kstep * kProjTokens + half * 64 + q * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3)) * LP + j * 32 + (lane & 31)] = acc[q][j][e];
    __syncthreads();
    float* out = f.part + ((uint64_t)range * a.tokens + t0) * LP;
#pragma unroll
    for (int i = 0; i < kProjTokens * LP / 4 / kProjThreads; ++i) {
        const int o = (i * kProjThreads + (int)threadIdx.x) * 4;               // element of the tokens x 64 block
        f32x4 v = *reinterpret_cast<const f32x4*>(sums + o);
#pragma unroll
        for (int w = 1; w < 4; ++w) {
            const f32x4 u = *reinterpret_cast<const f32x4*>(sums + w * kProjTokens * LP + o);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] += u[e];
        }
        if (t0 + o / LP < a.tokens) *reinterpret_cast<f32x4*>(out + o) = v;
    }
}

struct LograOuterArgs {
    const float *pa, *pb;              // [range][token][64]
    uint32_t ranges_a, ranges_b;
    uint64_t tokens, T, n;
    uint64_t tokens_per_block;
    uint32_t chunks;
    uint32_t k_in, k_out;
    float* partial;                    // [sample][chunk][block][16 x 16]
    uint32_t* counters;
    float* out;
    uint64_t ldo;
};

// The token loop of one wavefront of WAVES: U ranges and 4 / U runs of 16 tokens of both factors in flight at a time.  With
// twice as many the tokens of a sample are dealt to half as many wavefronts (100 x 128 tokens, 2,048 -> 1,024: the call takes
// 32.3 us, 27.3 with 4 / U; 7 x 1,000, 2,048 -> 8,192: 39.7 and 38.8; 27 shapes 4 % in the geometric mean, none slower).
template <int U, int WAVES>
__device__ __forceinline__ void logra_outer_tokens(const LograOuterArgs& a, uint64_t sample, uint32_t ab, uint32_t bb, uint64_t c0,
                                                   uint64_t c1, int wave, int lane, float (*st)[16][16], f32x4& acc) {
    constexpr int RUNS = 4 / U;
    const uint32_t ranges = a.ranges_a > a.ranges_b ? a.ranges_a : a.ranges_b;
    const int tr = lane >> 2, c4 = (lane & 3) * 4;
    for (uint64_t t0 = c0 + 16 * RUNS * wave; t0 < c1; t0 += 16 * RUNS * WAVES) {
        uint64_t ofs[RUNS];
        f32x4 va[RUNS], vb[RUNS];
#pragma unroll
        for (int i = 0; i < RUNS; ++i) {
            const uint64_t t = t0 + tr + 16 * i, tc = t < c1 ? t : c1 - 1;
            ofs[i] = (sample * a.T + tc) * LP + c4;
            va[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            vb[i] = va[i];
        }
        for (uint32_t r = 0; r < ranges; r += U) {             // ranges are added in order
            f32x4 qa[U][RUNS], qb[U][RUNS];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                const uint32_t ru = r + u;
                const float* ra = a.pa + (uint64_t)(ru < a.ranges_a ? ru : a.ranges_a - 1) * a.tokens * LP + ab * 16;
                const float* rb = a.pb + (uint64_t)(ru < a.ranges_b ? ru : a.ranges_b - 1) * a.tokens * LP + bb * 16;
#pragma unroll
                for (int i = 0; i < RUNS; ++i) {
                    qa[u][i] = *reinterpret_cast<const f32x4*>(ra + ofs[i]);
                    qb[u][i] = *reinterpret_cast<const f32x4*>(rb + ofs[i]);
                }
            }
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                const bool ua = r + u < a.ranges_a, ub = r + u < a.ranges_b;           // uniform
#pragma unroll
                for (int i = 0; i < RUNS; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        va[i][e] += ua ? qa[u][i][e] : 0.0f;
                        vb[i][e] += ub ? qb[u][i][e] : 0.0f;
                    }
            }
        }
#pragma unroll
        for (int i = 0; i < RUNS; ++i) {                       // 16 tokens at a time through LDS
            if (t0 + 16 * i >= c1) break;                      // uniform
            const bool live = t0 + tr + 16 * i < c1;           // rows past the chunk count as zero
#pragma unroll
            for (int e = 0; e < 4; ++e) { va[i][e] = live ? va[i][e] : 0.0f; vb[i][e] = live ? vb[i][e] : 0.0f; }
            *reinterpret_cast<f32x4*>(&st[0][tr][c4]) = va[i];
            *reinterpret_cast<f32x4*>(&st[1][tr][c4]) = vb[i];
            // the wavefront's own LDS writes and reads stay in order
#pragma unroll
            for (int k = 0; k < 16; k += 4)
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(st[0][k + (lane >> 4)][lane & 15], st[1][k + (lane >> 4)][lane & 15], acc,
                                                           0, 0, 0);
        }
    }
}

// A workgroup owns a 16 x 16 block of one sample's output and (usually) all of its tokens; its wavefronts take runs of
// tokens in turn, each for itself (sum of the ranges, a copy in its own part of LDS in the layout of
// v_mfma_f32_16x16x4_f32), and add up at the end.  The 16 blocks of a sample run on one XCD, so the partial sums come out
// of its L2 after the first of them.  Only when few samples have so many tokens that a workgroup would read megabytes are
// the tokens cut into chunks; the workgroup of a block that arrives last then adds the chunks in their order.
template <int WAVES>
__global__ void __launch_bounds__(64 * WAVES) logra_outer_kernel(LograOuterArgs a) {
    __shared__ __align__(16) float stage[WAVES][2][16][16];
    __shared__ float red[WAVES][256];
    __shared__ uint32_t arrived;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t chunk = blockIdx.y;
    const uint64_t sample = (uint64_t)(blockIdx.x / 128) * 8 + blockIdx.x % 8;
    const uint32_t block = blockIdx.x / 8 % 16, ab = block / 4, bb = block % 4;
    if (sample >= a.n || ab * 16 >= a.k_in || bb * 16 >= a.k_out) return;      // uniform
    const uint64_t c0 = chunk * a.tokens_per_block;
    const uint64_t c1 = c0 + a.tokens_per_block < a.T ? c0 + a.tokens_per_block : a.T;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    const uint32_t ranges = a.ranges_a > a.ranges_b ? a.ranges_a : a.ranges_b;
    if (ranges > 2) logra_outer_tokens<4, WAVES>(a, sample, ab, bb, c0, c1, wave, lane, stage[wave], acc);
    else if (ranges == 2) logra_outer_tokens<2, WAVES>(a, sample, ab, bb, c0, c1, wave, lane, stage[wave], acc);
    else logra_outer_tokens<1, WAVES>(a, sample, ab, bb, c0, c1, wave, lane, stage[wave], acc);
    // element e of a lane: row (a) 4(lane/16) + e, column (b) lane%16
#pragma unroll
    for (int e = 0; e < 4; ++e) red[wave][(4 * (lane >> 4) + e) * 16 + (lane & 15)] = acc[e];
    __syncthreads();
    float v = 0.0f;
    if (tid < 256) {
#pragma unroll
        for (int w = 0; w < WAVES; ++w) v += red[w][tid];
    }
    const uint32_t ai = ab * 16 + (tid >> 4), bi = bb * 16 + (tid & 15);
    float* o = a.out + sample * a.ldo + (uint64_t)ai * a.k_out + bi;
    const bool mine_out = tid < 256 && ai < a.k_in && bi < a.k_out;
    if (a.chunks == 1) {                                       // uniform
        if (mine_out) *o = v;
        return;
    }
    // The chunk's sums and their reads are agent-scope atomics: they go past the L2 caches of the eight XCDs, so no fence
    // has to write back and invalidate those (measured with __threadfence() here: 10 us more).  The stores have arrived
    // (vmcnt 0) in every wavefront before the barrier, and the counter is only raised behind it.
    float* mine = a.partial + (sample * a.chunks * 16 + block) * 256 + tid;    // chunks are 16 blocks apart
    if (tid < 256)
        __hip_atomic_store(mine + (uint64_t)chunk * (LP * LP), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) arrived = __hip_atomic_fetch_add(a.counters + sample * 16 + block, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (arrived + 1 != a.chunks || !mine_out) return;
    v = 0.0f;
#pragma unroll 8
    for (uint32_t c = 0; c < a.chunks; ++c)
        v += __hip_atomic_load(mine + (uint64_t)c * (LP * LP), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *o = v;
}

struct LograPlan {
    uint64_t tokens;
    uint32_t tiles, max_ranges;        // ranges of both factors together
    uint64_t tokens_per_block;         // of the outer products
    uint32_t chunks;
    size_t off_counters, off_partial, ws_bytes;
};

static size_t up256l(size_t x) { return (x + 255) / 256 * 256; }

static void plan_logra(uint64_t n, uint64_t T, LograPlan* pl) {
    pl->tokens = n * T;
    pl->tiles = (uint32_t)ceil_div(pl->tokens, kProjTokens);
    // at most three rounds of workgroups of the projection; at least one range per factor
    const uint32_t fit = 3u * kNumCU / pl->tiles;
    pl->max_ranges = fit > 2 ? fit : 2;
    // Outer products: cutting the tokens of a sample costs about 4 us (partial sums past the caches, the counter, their
    // sum), as much as a workgroup takes for 1,024 tokens.
    const uint64_t room = kNumCU / (16 * n) + 1;               // more workgroups than this only queue up
    uint64_t chunks = ceil_div(T, 2048);
    if (chunks > room) chunks = room;
    pl->tokens_per_block = ceil_div(ceil_div(T, chunks), 256) * 256;
    pl->chunks = (uint32_t)ceil_div(T, pl->tokens_per_block);
    size_t o = up256l((size_t)pl->max_ranges * pl->tokens * LP * sizeof(float));
    pl->off_counters = o; o += up256l((size_t)n * 16 * sizeof(uint32_t));
    pl->off_partial = o; if (pl->chunks > 1) o += (size_t)n * pl->chunks * LP * LP * sizeof(float);
    pl->ws_bytes = o;
}

// Cuts the columns of the two factors (gx and gg groups of 64) into ranges of at most `len` groups.  One workgroup runs on
// a CU at a time, so a cut costs (rounds of 256 workgroups) x (len + 3): about three groups' worth of time (0.76 us each
// at 5.5 TB/s) go to filling the pipeline and to the partial sum.  Every range adds a partial sum that the second kernel
// reads (0.17 us per 1,000 tokens).  Ranges of fewer than 4 groups are not tried.  16,384 tokens, 8,192 -> 2,048: 75 us in
// one range each, 64 in three and one.  Returns the estimated time of the projection: between that of whole rounds and
// that of the same work spread evenly (the ranges of the shorter factor end early).
static double cut_logra(const LograPlan& pl, uint32_t gx, uint32_t gg, uint32_t* len_x, uint32_t* len_g) {
    const uint32_t longest = gx > gg ? gx : gg;
    double best = 0.0, us = 0.0;
    for (uint32_t ranges = 1; ranges <= pl.max_ranges; ++ranges) {             // of the longer factor
        uint32_t len = (longest + ranges - 1) / ranges;
        if (ranges > 1 && len < 4) break;
        const uint32_t rx = (gx + len - 1) / len, rg = (gg + len - 1) / len;
        if (rx + rg > pl.max_ranges) break;
        const double rounds = (double)(((uint64_t)pl.tiles * (rx + rg) + kNumCU - 1) / kNumCU);
        const double sums = (rx + rg) * (double)pl.tokens * 2.2e-4, cost = rounds * (len + 3.0) + sums;
        if (best == 0.0 || cost < best) {
            best = cost; *len_x = (gx + rx - 1) / rx; *len_g = (gg + rg - 1) / rg;
            us = 0.38 * (cost + (double)pl.tiles * (gx + gg + 3.0 * (rx + rg)) / kNumCU + sums);
        }
    }
    return us;
}

// One launch of logra_short_kernel instead of the two: rounds of one sample per CU, 64 tokens at a time, 5 us and 1 us per
// 128 columns of the longer factor, against the projection and the outer products (16 workgroups per sample, four on a CU);
// neither takes less than the host needs for it.  Of 418 drawn shapes (1 to 2,048 samples of 1 to 4,096 tokens) the choice
// was within 5 % of the better one on 416 and 9 % at most; with two launches throughout 116 were slower than with one, up
// to twice: 345 x 24 tokens, 112 -> 48 columns 26.8 us (12.5 in one launch), 256 x 64, 768 -> 768 22.4 (14.3), 3 x 40, 512 ->
// 512 13.2 (12.2).
static bool short_logra(uint64_t n, uint64_t T, uint32_t d_in, uint32_t d_out, uint32_t k_in, double project_us) {
    if (T > 256) return false;
    const uint32_t longest = d_in > d_out ? d_in : d_out;
    double one = (double)(ceil_div(n, kNumCU) * ceil_div(T, 64)) * (5.0 + (double)ceil_div(longest, 128));
    double two = project_us + (double)ceil_div(n * 16, 4 * kNumCU) * (0.8 + 0.65 * (double)ceil_div(k_in, 16)) + 2.0;
    one = one > 8.7 ? one : 8.7;
    two = two > 12.5 ? two : 12.5;
    return one < two;
}

// Without a workspace one launch is the only way.  Calls that never needed one keep running without: the tokens of a sample
// are one chunk of at most 64, or of at most 256 where the samples alone fill the chip.
static bool logra_needs_no_workspace(uint64_t n, uint64_t T) { return T <= 64 || (T <= 256 && n >= (uint64_t)kNumCU); }

}  // namespace grass

using namespace grass;

static grass_status check_logra(uint64_t n, uint64_t T, uint32_t k_in, uint32_t k_out) {
    if (T == 0 || k_in == 0 || k_out == 0) return GRASS_EINVAL;
    if (n > 65535 || k_in > LP || k_out > LP) return GRASS_EUNSUPPORTED;
    if (n != 0 && T > (1ull << 37) / n) return GRASS_EUNSUPPORTED;             // token tiles are numbered in 32 bits
    return GRASS_OK;
}

extern "C" grass_status logra_linear_workspace_bytes(uint64_t n, uint64_t T, uint32_t k_in, uint32_t k_out,
                                                     size_t* host_bytes) {
    if (!host_bytes) return GRASS_EINVAL;
    grass_status st = check_logra(n, T, k_in, k_out);
    if (st != GRASS_OK) return st;
    if (n == 0) { *host_bytes = 0; return GRASS_OK; }
    LograPlan pl;
    plan_logra(n, T, &pl);
    *host_bytes = pl.ws_bytes;
    return GRASS_OK;
}

extern "C" grass_status logra_linear(const void* x, const void* gout, uint64_t n, uint64_t T, uint32_t d_in,
                                     uint32_t d_out, const void* P_in, uint32_t k_in, const void* P_out,
                                     uint32_t k_out, float* out, uint64_t ldo, void* ws, size_t ws_bytes,
                                     grass_stream stream) {
    grass_status st = check_logra(n, T, k_in, k_out);
    if (st != GRASS_OK) return st;
    if (d_in == 0 || d_out == 0) return GRASS_EINVAL;
    if (n == 0) return GRASS_OK;
    const uint64_t kk = (uint64_t)k_in * k_out;
    if (!x || !gout || !P_in || !P_out || !out || ldo < kk) return GRASS_EINVAL;
    // 16-byte chunks along the feature dimension
    if (d_in % 8 != 0 || d_out % 8 != 0 || !aligned(x, 16) || !aligned(gout, 16) || !aligned(P_in, 16) ||
        !aligned(P_out, 16))
        return GRASS_EUNSUPPORTED;
    if (d_in > (1u << 24) || d_out > (1u << 24)) return GRASS_EUNSUPPORTED;   // 32-bit byte offsets inside a row
    LograPlan pl;
    plan_logra(n, T, &pl);
    const bool have_ws = ws && ws_bytes >= pl.ws_bytes && aligned(ws, 256);
    if (!have_ws && !logra_needs_no_workspace(n, T)) return GRASS_EWORKSPACE;
    LograProjectArgs p;
    uint32_t len_x, len_g;
    const uint32_t gx = (d_in + 63) / 64, gg = (d_out + 63) / 64;
    const double project_us = cut_logra(pl, gx, gg, &len_x, &len_g);
    if (!have_ws || short_logra(n, T, d_in, d_out, k_in, project_us))
        return launch_logra_short(static_cast<const uint16_t*>(x), static_cast<const uint16_t*>(gout), n, T, d_in, d_out,
                                  static_cast<const uint16_t*>(P_in), k_in, static_cast<const uint16_t*>(P_out), k_out, out, ldo,
                                  as_stream(stream)) == hipSuccess ? GRASS_OK : GRASS_EHIP;
    unsigned char* base = static_cast<unsigned char*>(ws);
    const uint32_t rx = (gx + len_x - 1) / len_x, rg = (gg + len_g - 1) / len_g;
    float* part = reinterpret_cast<float*>(base);
    float* part_g = part + (uint64_t)rx * pl.tokens * LP;
    p.f[0] = LograFactor{static_cast<const uint16_t*>(x), static_cast<const uint16_t*>(P_in), d_in, k_in, gx, len_x, part};
    p.f[1] = LograFactor{static_cast<const uint16_t*>(gout), static_cast<const uint16_t*>(P_out), d_out, k_out, gg, len_g, part_g};
    p.tokens = pl.tokens; p.tiles = pl.tiles; p.ranges_x = rx;
    p.counters = reinterpret_cast<uint32_t*>(base + pl.off_counters);
    p.n_counters = pl.chunks > 1 ? (uint32_t)n * 16 : 0;
    const uint64_t blocks = (uint64_t)pl.tiles * (rx + rg);
    if (rx + rg > pl.max_ranges || blocks > 0x7FFFFFFFull) return GRASS_EUNSUPPORTED;

    LograOuterArgs o;
    o.pa = part; o.pb = part_g; o.ranges_a = rx; o.ranges_b = rg;
    o.tokens = pl.tokens; o.T = T; o.n = n; o.tokens_per_block = pl.tokens_per_block; o.chunks = pl.chunks;
    o.k_in = k_in; o.k_out = k_out;
    o.partial = reinterpret_cast<float*>(base + pl.off_partial);
    o.counters = p.counters; o.out = out; o.ldo = ldo;

    hipStream_t hs = as_stream(stream);
    static LdsOptIn opt_in;
    if (allow_large_lds(opt_in, reinterpret_cast<const void*>(logra_project_kernel)) != hipSuccess) return GRASS_EHIP;
    hipLaunchKernelGGL(logra_project_kernel, dim3((uint32_t)blocks), dim3(kProjThreads), kProjStages * kProjStageBytes, hs, p);
    const dim3 grid((uint32_t)ceil_div(n, 8) * 128, pl.chunks);
    // 16 wavefronts where the blocks of all samples leave CUs idle and there are tokens for them (10 x 130 tokens 16.3 -> 15.2 us;
    // 64 x 256 tokens 20.7 with 8, 22.6 with 16)
    if (T > 128 && n <= 16) hipLaunchKernelGGL(logra_outer_kernel<16>, grid, dim3(1024), 0, hs, o);
    else hipLaunchKernelGGL(logra_outer_kernel<8>, grid, dim3(512), 0, hs, o);
    return launch_status();
}
