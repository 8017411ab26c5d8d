// fp32 products on the fp16 matrix cores: C[M x N] = or += A * B^T with fp32 operands and fp32 accumulation, for workgroups that
// contract at least 256 k.  Sums are within the bound of the products of three bf16 pieces (gemm_split.hip), |error| <= 2^-23 (6
// ceil(k / 16) + 65) sum |a b|, and on ordinary data closer than those.
//
// Every row of an operand ("slot") is scaled by a power of two and split into two fp16 numbers, a = a0 + a1 with a0 = fp16(a)
// and a1 = fp16(a - a0), both rounded to nearest: 23 of the 24 significant bits, the last one with an error of one unit at
// most (Markidis, Der Chien, Laure, Peng and Vetter, "NVIDIA tensor core programmability, performance & precision", 2018, split
// fp32 operands so).  Three of the four products of two such sums are accumulated by v_mfma_f32_16x16x32_f16; a1 b1 is below
// 2^-22 |a b|, 2^-24.8 in the root mean square.  The sums take half as many roundings as six products of bf16 pieces do, which
// more than makes up for the bit.  Error against fp64, 2-norm, one K range, normal data (three bf16 pieces in brackets): K = 64
// 1.1e-7 (1.1e-7), 256 1.9e-7 (2.4e-7), 1,024 3.6e-7 (4.9e-7), 4,096 7.1e-7 (1.0e-6); 100 x 1,000 x 1,863,690 in 64 ranges 5.9e-6
// (1.1e-5); FIM of 65,536 x 4,096 rows 4.0e-7 (2.8e-6); largest deviations likewise.  Below 256 k there is next to nothing to
// gain (launches start 8 us later, the bit shows), so shorter ranges stay with gemm_split.hip.
//
// Scales.  fp16 reaches from 2^-24 to 2^16.  A workgroup takes the largest |x| of a sample of every slot, 64 values or more, and scales it
// to 2^9..2^10: values up to 2^6 times the sample's largest fit, smaller ones lose nothing above 2^-11 of it and are off by 2^-34
// of it below.  What that takes from a sum is judged by the sample and by the size of the sum alone, once the sums are there.
// The few that do not pass are summed again one by one in fp64; where they are more, the tile is computed again with three
// bf16 pieces.  Tiles of scattered values go there at once.  The diagonal of a matrix whose rows are its columns (an inverse) is
// known to be large: it is scaled to 2^14..2^15 at most and the rest of the row as if it was not there.
//
// Bound: the power that the matrix cores and the data on the way to them draw.  1,024 x 65,536 x 4,096 takes 1.45 ms = 1,140
// TFLOP/s of fp16 products at 1.4 to 1.7 GHz, matrix cores 65 to 69 % busy; without loads and splitting it would be 1.15 ms, a loop of
// matrix instructions alone 0.95.  What counts is therefore work beside the matrix instructions: 16 x 16 x 32 instructions
// (1,806 TFLOP/s alone on random data; 32 x 32 x 16: 1,611), whole lines of 32 k per load, one exclusive or against bank
// conflicts (26 % of the cycles before), no arithmetic on addresses, five vector operations per pair of values.
//   three bf16 pieces -> two fp16 pieces
//   1,024 x 65,536 x 4,096, A B^T                     2.25 -> 1.45 ms
//   65,536 x 4,096 x 4,096, A B^T                     9.5  -> 5.1
//   65,536 x 4,096, lower tiles of A^T A              5.3  -> 2.9
//   100 x 1,000 x 1,863,690, A B^T, unaligned rows    3.3  -> 1.85
//   100 x 327,680 x 1,000, A B                        0.50 -> 0.38
// Two groups on their way instead of one (150 us for 64 x 65,536 x 2,048 either way) and vector instructions that are not
// spread over the matrix instructions (1 to 2 % slower) did not pay.
#include <type_traits>

#include "gemm_split_device.h"

namespace grass {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef const float __attribute__((address_space(1)))* gfloat;             // global loads, whatever the compiler can tell
typedef const unsigned char __attribute__((address_space(1)))* gbyte;
typedef const f32x4u __attribute__((address_space(1)))* gvec;

// Exponent of the leading bit of a positive fp32 number given by its bits; 128 for infinity.
__device__ __forceinline__ int lead_exponent(uint32_t bits) {
    return bits >= 0x800000u ? (int)(bits >> 23) - 127 : -118 - (int)__builtin_clz(bits);
}
__device__ __forceinline__ int clamp_exponent(int e) { return e < -126 ? -126 : e > 127 ? 127 : e; }

template <int CTRL, class T>
__device__ __forceinline__ T swap_lanes(T x) {
    return __builtin_bit_cast(T, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}
// `f` over 8 neighbouring lanes, in all of them: quad_perm 1 0 3 2, quad_perm 2 3 0 1, row_half_mirror.
template <class T, class F>
__device__ __forceinline__ T over_8_lanes(T x, F f) {
    x = f(x, swap_lanes<0xB1>(x));
    x = f(x, swap_lanes<0x4E>(x));
    return f(x, swap_lanes<0x141>(x));
}

constexpr uint32_t kDone = 0, kExact = ~0u;
constexpr int kSampleTop = 9, kDiagonalTop = 14;   // exponents to which the largest value of a sample is scaled, a diagonal at most

typedef unsigned char __attribute__((address_space(3)))* lds_byte;

// The gradient of the columns of a tile from its R = `get(i, j, e)` (element e of block (i, j)), all rows of which it holds: a
// lane multiplies its 4 columns with Gt and sums its rows in fp64, lanes and wavefronts are added in a fixed order.
// CHECK: where the sum over the rows of |Gt R| is not finite or, for kSize, not above that of |Gt| <lost(i, e), col(j)>, below which
// the scales may have taken bits from an R, false is returned and nothing stored.
enum : int { kNothing = 0, kFinite = 1, kSize = 2 };
template <int RB, int NB, int WR, int WC, int CHECK, class Get, class Lost, class Col>
__device__ __forceinline__ bool grad_tail(const GemmF32Args& a, const GradTail& t, double* part, uint64_t n0, Get get, Lost lost, Col col) {
    constexpr int TN = 16 * NB * WC;
    const int lane = threadIdx.x & 63, lq = lane >> 4, lc = lane & 15, wave = threadIdx.x >> 6, wm = wave / WC, wn = wave % WC;
    const uint64_t c0 = n0 + wn * NB * 16 + 4 * lc;
    const bool all = c0 + 4 <= a.N;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    float size[4] = {0.0f, 0.0f, 0.0f, 0.0f}, lx[4] = {0.0f, 0.0f, 0.0f, 0.0f}, ly[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint64_t row = (wm * RB + i) * 16 + 4 * lq + e;
            if (row >= a.M || c0 >= a.N) continue;
            const float* gt = t.Gt + row * t.ldgt + c0;
            f32x4 x{0.0f, 0.0f, 0.0f, 0.0f};
            if (all) {
                x = *reinterpret_cast<const f32x4u*>(gt);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (c0 + j < a.N) x[j] = gt[j];
            }
            f32x2 l;
            if constexpr (CHECK == kSize) l = lost(i, e);
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (all || c0 + j < a.N) {
                    const float r = get(i, j, e);
                    s[j] += (double)x[j] * (double)r;
                    if constexpr (CHECK != kNothing) size[j] = __builtin_fmaf(__builtin_fabsf(x[j]), __builtin_fabsf(r), size[j]);
                    if constexpr (CHECK == kSize) {
                        lx[j] = __builtin_fmaf(__builtin_fabsf(x[j]), l[0], lx[j]);
                        ly[j] = __builtin_fmaf(__builtin_fabsf(x[j]), l[1], ly[j]);
                    }
                }
        }
    float* const check = reinterpret_cast<float*>(part + WR * TN);
    int* const vote = reinterpret_cast<int*>(check + WR * TN);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        s[j] += __shfl_xor(s[j], 16);
        s[j] += __shfl_xor(s[j], 32);
        if constexpr (CHECK == kSize) {
            const f32x2 c = col(j);
            size[j] -= lx[j] * c[0] + ly[j] * c[1];
        }
        if constexpr (CHECK != kNothing) {
            size[j] += __shfl_xor(size[j], 16);
            size[j] += __shfl_xor(size[j], 32);
        }
    }
    __syncthreads();                                           // the memory of `part` is free
    if (CHECK != kNothing && threadIdx.x == 0) *vote = 0;
    if (lq == 0) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            part[wm * TN + wn * NB * 16 + 4 * lc + j] = s[j];
            if constexpr (CHECK != kNothing) check[wm * TN + wn * NB * 16 + 4 * lc + j] = size[j];
        }
    }
    __syncthreads();
    if constexpr (CHECK != kNothing) {
        for (int c = threadIdx.x; c < TN && n0 + c < a.N; c += 64 * WR * WC) {
            float sum = check[c];
#pragma unroll
            for (int w = 1; w < WR; ++w) sum += check[w * TN + c];
            if (!(sum >= 0.0f && sum < __builtin_inff())) *vote = 1;
        }
        __syncthreads();
        if (*vote != 0) return false;                          // uniform
    }
    for (int c = threadIdx.x; c < TN && n0 + c < a.N; c += 64 * WR * WC) {
        double sum = part[c];
#pragma unroll
        for (int w = 1; w < WR; ++w) sum += part[w * TN + c];
        const uint64_t j = n0 + c;
        const float sig = sigmoidf(t.S[j] * t.inv_temp), dsig = sig * (1.0f - sig) * t.inv_temp;
        t.grad[j] = (float)(2.0 * (double)sig * (double)dsig * sum - (double)t.lambda * (double)dsig);
    }
    return true;
}

// What a function that is not inlined is handed arrives in vector registers; this puts it back.
template <class T>
__device__ __forceinline__ T uniform(T x) {
    uint32_t w[sizeof(T) / 4];
    __builtin_memcpy(w, &x, sizeof(T));
#pragma unroll
    for (uint32_t i = 0; i < sizeof(T) / 4; ++i) w[i] = __builtin_amdgcn_readfirstlane(w[i]);
    __builtin_memcpy(&x, w, sizeof(T));
    return x;
}
__device__ __forceinline__ unsigned char* uniform_lds(lds_byte p) { return (unsigned char*)(lds_byte)(uintptr_t)uniform((uint32_t)(uintptr_t)p); }

// The sums of a tile that did not pass, in fp64 straight from memory.  The rare ends of a tile are functions of their own: in one
// function they cost the main loop registers that it has to spill.
template <int RB, int NB, int WR, int WC, bool AKN, bool BKN, bool WEIGHT>
__device__ __attribute__((noinline)) void sum_again(GemmF32Args a, lds_byte lds, uint32_t total) {
    constexpr uint32_t NW = WR * WC, THREADS = 64 * NW;
    static_assert((NW == 4 || NW == 8) && 128 * NW * (4 + 8 * NW) <= 2 * 8 * 16 * 16 * (RB * WR + NB * WC), "LDS of the stages");
    a = uniform(a);
    total = uniform(total);
    unsigned char* const smem = uniform_lds(lds);
    const uint32_t* const list = reinterpret_cast<const uint32_t*>(smem);        // [128 NW]
    double* const parts = reinterpret_cast<double*>(smem + 128 * NW * 4);
    const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const auto [tm, tn, split] = gemm_f32_tile(a);
    a.C += split * a.split_stride_c;
    const uint64_t m0 = (uint64_t)tm * (16 * RB * WR), n0 = (uint64_t)tn * (16 * NB * WC);
    const uint64_t ng_all = (a.K + 31) / 32, k_begin = split * ng_all / a.splits * 32, k_last = (split + 1) * ng_all / a.splits * 32;
    const uint64_t k_end = k_last < a.K ? k_last : a.K;
    const float kr = (float)(k_end - k_begin);
    // of long ranges by several wavefronts, whose parts are added in their order
    const uint32_t share = total >= NW || kr < 4096.0f ? 1 : kr < 8192.0f ? 2 : kr < 16384.0f || NW == 4 ? 4 : 8, part = wave % share;
#pragma unroll 1
    for (uint32_t t = wave / share; t < total; t += NW / share) {
        const uint32_t at = __builtin_amdgcn_readfirstlane(list[t]);
        const uint64_t row = m0 + (at >> 16), col = n0 + (at & 0xFFFFu);
        const gfloat pa = (gfloat)(AKN ? a.A + row : a.A + row * a.lda), pb = (gfloat)(BKN ? a.B + col : a.B + col * a.ldb);
        double sum = 0.0;
        uint64_t k0 = k_begin + 2048 * part;
        auto dot = [&](auto full, auto n) {                    // 256 n of k, 4 in a row for a lane, requested together
            constexpr bool FULL = decltype(full)::value;
            constexpr int U = decltype(n)::value;
            f32x4 ya[U], yb[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint64_t k = k0 + 256 * u + 4 * lane;
                if constexpr (FULL && !AKN) ya[u] = *(gvec)(pa + k);
                if constexpr (FULL && !BKN) yb[u] = *(gvec)(pb + k);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const bool ok = FULL || k + q < k_end;
                    if constexpr (!FULL || AKN) ya[u][q] = ok ? pa[AKN ? (k + q) * a.lda : k + q] : 0.0f;
                    if constexpr (!FULL || BKN) yb[u][q] = ok ? pb[BKN ? (k + q) * a.ldb : k + q] : 0.0f;
                    if constexpr (WEIGHT) ya[u][q] *= ok ? a.weight[k + q] : 0.0f;
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) sum = __builtin_fma((double)ya[u][q], (double)yb[u][q], sum);
        };
        const std::true_type full;
        const std::false_type rest;
#pragma unroll 1
        for (; k0 + 2048 <= k_end; k0 += 2048 * share) dot(full, std::integral_constant<int, 8>{});
        if (k0 < k_end) {                                      // uniform; of one part at most
            if (k0 + 1024 <= k_end) { dot(full, std::integral_constant<int, 4>{}); k0 += 1024; }
            if (k0 + 512 <= k_end) { dot(full, std::integral_constant<int, 2>{}); k0 += 512; }
            dot(rest, std::integral_constant<int, 2>{});
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
        if (lane == 0) parts[t * share + part] = sum;
    }
    __syncthreads();
    for (uint32_t t = threadIdx.x; t < total; t += THREADS) {
        double sum = parts[t * share];
        for (uint32_t q = 1; q < share; ++q) sum += parts[t * share + q];
        float* const c = a.C + (m0 + (list[t] >> 16)) * a.ldc + n0 + (list[t] & 0xFFFFu);
        *c = a.accumulate ? *c + (float)sum : (float)sum;
    }
}

// One workgroup owns a TM x TN tile of C; its WR x WC wavefronts own RB x NB blocks of 16 x 16 each.  K is consumed in groups
// of 32 through two LDS stages.  A group travels from memory into registers one group before it is split and stored, which
// is spread over the multiplication of the group before it.  A row-major B is loaded again register by register as they are stored,
// A in one bunch behind its last store: one by one it takes longer (1,024 x 65,536 x 65,536 19.1 -> 20.1 ms, 1,000 x 50,001 x 4,096
// 0.990 -> 0.998, 65,536 x 4,096 cached 11.59 -> 11.66, mask training 9.64 -> 9.65).  The barrier of a group sits before its last row
// of blocks: by then every wavefront has the fragments of this group in registers and its part of the next group in LDS.
// AKN / BKN: the operand is stored K-major (K x M resp. K x N).
// Returns kDone, kExact (the tile's data do not suit two fp16 pieces; nothing has been stored) or how many sums are left for
// sum_again.
template <int RB, int NB, int WR, int WC, bool AKN, bool BKN, bool WEIGHT = false, bool GRAD = false>
__device__ __forceinline__ uint32_t pair_tile(GemmF32Args a, lds_byte lds, const GradTail* tail = nullptr) {
    unsigned char* const smem = (unsigned char*)lds;
    constexpr int NW = WR * WC, THREADS = 64 * NW;
    constexpr int TM = 16 * RB * WR, TN = 16 * NB * WC, SLOTS = TM + TN;
    constexpr int CA = TM / (8 * NW), CB = TN / (8 * NW), NC = CA + CB;      // chunks of 4 fp32 per thread and group
    static_assert(TM % (8 * NW) == 0 && TN % (8 * NW) == 0 && (!AKN || CA == 4) && (!BKN || CB == 4) && NB == 4, "loading map");
    constexpr int kReg = SLOTS * 16, kPlane = 4 * kReg, kStage = 2 * kPlane;
    uint32_t* const mx = reinterpret_cast<uint32_t*>(smem + 2 * kStage);      // [SLOTS] largest |x| of a slot's sample (bits), then
    float* const nrm = reinterpret_cast<float*>(mx);                          //         its squares, then the slot's 2-norm (scaled)
    int* const ex = reinterpret_cast<int*>(mx + SLOTS);                       // [SLOTS] exponent of a slot's scale
    uint32_t* const few = mx + 2 * SLOTS;                                     // [SLOTS] values of the sample that the scale leaves few bits,
    float* const gam = reinterpret_cast<float*>(few);                         //         then what that means for the slot
    uint32_t* const mx2 = mx + 3 * SLOTS;                                     // [SLOTS] largest |x| but for the diagonal, then
    int* const bias = reinterpret_cast<int*>(mx2);                            //         sum of what those values lose, away from zero, in 2^-33,
    float* const odd = reinterpret_cast<float*>(bias);                        //         then the share of gam against an ordinary row, < 0: odd row
    uint32_t* const mt = mx + 4 * SLOTS;                                      // rows, list, columns of the tile; the largest weight; odd rows
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave / WC, wn = wave % WC;
    const auto [tm, tn, split] = gemm_f32_tile(a);
    const uint64_t m0 = (uint64_t)tm * TM, n0 = (uint64_t)tn * TN;
    a.C += split * a.split_stride_c;
    const uint64_t ng_all = (a.K + 31) / 32;
    const uint64_t g0 = split * ng_all / a.splits;
    const uint32_t ng = (uint32_t)((split + 1) * ng_all / a.splits - g0);     // >= 1: splits <= ng_all

    // ---- loading.  What depends on the lane is worked out where it is needed (`ln` hides the lane from the compiler, which
    // would keep all of it in registers through the main loop).
    struct Side {
        gfloat mat;
        uint64_t ld, rows, first, r0;      // first: first row of the tile; K-major: r0 = first column that is loaded
        uint64_t k0, step;                 // first k of the range; elements from a group to the next
        int T, slot0;                      // rows of the tile, slot of the first one
        bool narrow;
    };
    auto make = [&](bool kmajor, const float* src, uint64_t ld, uint64_t rows, uint64_t first, int T, int slot0) {
        Side o{(gfloat)src, ld, rows, first, first, g0 * 32, kmajor ? 32 * ld : 32, T, slot0, false};
        if (kmajor) {
            o.narrow = rows < 4;                               // too narrow for 16-byte loads
            o.r0 = first + 4 <= rows ? first : o.narrow ? 0 : rows - 4;
        }
        return o;
    };
    const Side sa = make(AKN, a.A, a.lda, a.M, m0, TM, 0), sb = make(BKN, a.B, a.ldb, a.N, n0, TN, TM);
    const std::integral_constant<bool, AKN> km_a;
    const std::integral_constant<bool, BKN> km_b;
    auto hide = [](int x) {
        asm volatile("" : "+v"(x));
        return x;
    };
    // Row-major: chunk i of a wavefront is 8 rows, 8 lanes take the 32 k of one.  Lanes past the edge repeat the last row, chunks
    // past the edge the tile's first.  K-major: a thread takes 4 columns of 4 k, chunk i is its row i on loading and its column
    // i on storing; columns that reach past the edge are moved back to the last 4.
    auto column = [&](const Side& o, int ln) { return 4 * (ln >> 1) + 128 * (wave % (o.T / 128)); };
    auto column_at = [&](const Side& o, int ln) {              // inside the tile, may be negative
        const int c = column(o, ln);
        return o.first + c + 4 > o.rows && !o.narrow ? (int)((int64_t)o.rows - 4 - (int64_t)o.first) : c;
    };
    auto first_k = [&](auto km, const Side& o, int ln) {       // k of a group: first_k..+3
        return decltype(km)::value ? 4 * ((ln & 1) + 2 * (wave / (o.T / 128))) : 4 * (ln & 7);
    };
    auto chunk_row = [&](const Side& o, int i) { return (uint32_t)(wave * (o.T / NW) + 8 * i); };     // inside the tile
    auto past = [&](const Side& o, int i) { return o.first + chunk_row(o, i) >= o.rows; };
    auto cut = [&](const Side& o, int i) {                     // the chunk, or the first if this one is past the edge, crosses it
        return past(o, i) ? o.rows - o.first < 8 : o.rows - o.first - chunk_row(o, i) < 8;
    };
    auto lane_load = [&](auto km, const Side& o, int ln) -> uint32_t {        // byte offset of the lane from a chunk's base
        if constexpr (decltype(km)::value) {
            return (4 * (ln & 1) * (uint32_t)o.ld + (uint32_t)(column_at(o, ln) + (int)(o.first - o.r0))) * 4;
        } else {
            return ((uint32_t)(ln >> 3) * (uint32_t)o.ld + 4 * (ln & 7)) * 4;
        }
    };
    auto lane_load_cut = [&](auto km, const Side& o, int ln) -> uint32_t {    // the same in a row-major chunk that crosses the edge
        if (decltype(km)::value || o.rows - o.first >= (uint64_t)o.T) return 0;
        const uint32_t left = (uint32_t)(o.rows - o.first), last = (left < 8 ? left : left & 7) - 1, r = (uint32_t)(ln >> 3);
        return ((r < last ? r : last) * (uint32_t)o.ld + 4 * (ln & 7)) * 4;
    };
    // Slot of chunk (row-major) or column (K-major) i.  Column c of 64 lies in slot 16 (c % 4) + c / 4, which spreads the
    // stores over the banks and gives a lane 4 consecutive columns of a result.  Columns before the tile (it has fewer than 4)
    // go to its last slot, which is past the edge.
    auto slot_of = [&](auto km, const Side& o, int ln, int i) {
        if constexpr (decltype(km)::value) {
            int c = column_at(o, ln) + i;
            c = c < 0 ? o.T - 1 : c;
            return o.slot0 + (c & ~63) + (c & 3) * 16 + ((c >> 2) & 15);
        } else {
            return o.slot0 + (int)chunk_row(o, i) + (ln >> 3);
        }
    };
    // LDS: [piece][k / 8][slot][8 k].  A quarter of the k's slots change places by an exclusive or, so that neither the
    // stores (4 slots of all k, or 16 slots of 4 k, in 32 lanes) nor the 16-byte reads of fragments (16 slots of two quarters
    // in 32 lanes) meet in a bank.
    auto turn = [](int quarter) { return (quarter & 1) * 12 ^ (quarter >> 1) * 4; };
    auto in_plane = [&](auto km, const Side& o, int ln, int slot) {           // byte offset of the thread's 4 k of a slot
        const int kq = first_k(km, o, ln) / 4;
        return (uint32_t)((kq >> 1) * kReg + (slot ^ turn(kq >> 1)) * 16 + (kq & 1) * 8);
    };
    auto base_of = [&](auto km, const Side& o, int i) {        // of chunk i in the first group
        if constexpr (decltype(km)::value) return o.mat + (o.k0 + 8 * (wave / (o.T / 128)) + i) * o.ld + o.r0;
        else return o.mat + (o.first + (past(o, i) ? 0 : chunk_row(o, i))) * o.ld + o.k0;
    };
    // Groups whose 32 k all exist are loaded unconditionally, so that the compiler's wait counts leave the newer loads in
    // flight; the last group of a range goes through guarded loads.
    uint32_t nf;
    {
        const uint64_t k_full = a.K / 32;
        nf = (uint32_t)(k_full <= g0 ? 0 : k_full - g0 < ng ? k_full - g0 : ng);
        if ((AKN && a.M < 4) || (BKN && a.N < 4)) nf = 0;
    }
    auto load_full = [&](gfloat p, uint64_t step, uint32_t gofs, uint32_t g) {
        p += g * step;
        asm volatile("" : "+s"(p));                            // stays a scalar base: no 64-bit lane addresses
        return *(gvec)((gbyte)p + gofs);
    };
    auto load_part = [&](auto km, gfloat p, const Side& o, uint32_t gofs, int i, uint32_t g, int ln) {
        constexpr bool KM = decltype(km)::value;
        const gfloat q = (gfloat)((gbyte)(p + g * o.step) + gofs);
        const uint64_t k = o.k0 + (uint64_t)g * 32 + first_k(km, o, ln);
        f32x4 x;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            bool ok = k + (KM ? i : e) < a.K;
            if (KM && o.narrow) ok = ok && column(o, ln) + e < (int)o.rows;
            x[e] = ok ? q[e] : 0.0f;
        }
        return x;
    };
    static_assert(!WEIGHT || !AKN, "weights");
    f32x4 xa[CA], xb[CB], za[CA], zb[CB];                      // a group on its way, the first group
    f32x4 xw, zw;                                              // the weights of the thread's k of these
    auto weight_at = [&](uint32_t g) -> f32x4 {
        if constexpr (WEIGHT) return *(gvec)((gfloat)a.weight + g0 * 32 + (uint64_t)g * 32 + 4 * (lane & 7));
        else return f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    };
    auto weigh = [&](f32x4& v, const f32x4& w) {               // rounded once, as a matrix of products would be
        if constexpr (WEIGHT) v *= w;
    };
    // 4 k of one slot: chunk i of a row-major operand, column i of a K-major one
    auto values = [&](auto km, const auto& x, int i) {
        if constexpr (decltype(km)::value) return f32x4{x[0][i], x[1][i], x[2][i], x[3][i]};
        else return x[i];
    };
    auto largest = [](const f32x4& v) {
        const float m = __builtin_fmaxf(__builtin_fabsf(v[0]), __builtin_fabsf(v[1]));
        return __builtin_fmaxf(m, __builtin_fmaxf(__builtin_fabsf(v[2]), __builtin_fabsf(v[3])));
    };

    if ((AKN && m0 + TM > a.M) || (BKN && n0 + TN > a.N)) {    // slots past the edge that nothing is stored in
        for (int t = threadIdx.x; t < 2 * kStage / 16; t += THREADS) reinterpret_cast<f32x4*>(smem)[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    // What the scales may take from a sum.  The pieces are off by 2^-23 of a value, and of values below 2^-2 (scaled) by up to 2^-25.
    // Products of three bf16 pieces are within 2^-23 (6 ceil(k / 16) + 65) sum |a b|, those of two fp16 pieces, but for values below
    // 2^-2, within 2^-23 (3 ceil(k / 32) + 64) + 2^-21.  In between there is room for an error of 2^-25 / unit times sum |a b|.  Values
    // from 8 unit on take a quarter of it at most.  n smaller ones in a row a take at most 2^-25 sqrt(n) |b|_2, and likewise for b;
    // the rest has room for that if the sum, which is at most sum |a b|, is not below 4/3 unit (gam_a |b|_2 + gam_b |a|_2), gam =
    // sqrt(n).  That much is lost if all errors have one sign.  Otherwise they add up to 2^-25 sqrt(f / 3) |b|_2 in the root mean
    // square, f = n / k, whatever n is, and seven times that is gam = 4 sqrt(f).  f is twice what the sample says.  The mean of the
    // errors in the sample, as far as it is more than chance makes it (1.2 / sqrt(c) for c of them), is the part that has one sign,
    // as equal values have; a quarter where the sample has too few to tell.  gam is 2 at least, for up to four such values that the sample
    // does not show.  |a|_2 is sqrt(2) times what the sample says, and a value of 2^11 that it does not show.
    // A row is ordinary if 24 of 32 values in the sample are 1 and more.  Two of them meet at enough k for sum |a b| to be above that
    // whatever the sum is (0.5 of their sums per tile of 1,000 x 50,001 x 4,096 would not pass, and cost 5 us at the end of a
    // launch).  What the n small values of an odd row meet in an ordinary one is rather n / k of it: min(1, 2 sqrt(f)), at least
    // 1/4, of gam counts.
    // Values too large for their scale, infinities and NaNs leave sums that are not finite.
    const uint64_t k_begin = g0 * 32, k_end = (g0 + ng) * 32 < a.K ? (g0 + ng) * 32 : a.K;
    const float kr = (float)(k_end - k_begin), unit = 0.25f / (0.28125f * kr - 3.0f);
    f32x4 acc[RB][NB];
    {
        const int ln = hide(threadIdx.x & 63);
        const uint32_t ga = lane_load(km_a, sa, ln), gb = lane_load(km_b, sb, ln);
        gfloat pa[CA];
        gfloat pb[CB];
        const uint32_t ga_cut = lane_load_cut(km_a, sa, ln), gb_cut = lane_load_cut(km_b, sb, ln);
        bool ca[CA], cb[CB];
#pragma unroll
        for (int i = 0; i < CA; ++i) { pa[i] = base_of(km_a, sa, i); ca[i] = !AKN && cut(sa, i); }
#pragma unroll
        for (int i = 0; i < CB; ++i) { pb[i] = base_of(km_b, sb, i); cb[i] = !BKN && cut(sb, i); }
        auto load_a = [&](int i, uint32_t g) { return load_full(pa[i], sa.step, ca[i] ? ga_cut : ga, g); };
        auto load_b = [&](int i, uint32_t g) { return load_full(pb[i], sb.step, cb[i] ? gb_cut : gb, g); };
        auto fetch = [&](auto& ya, auto& yb, f32x4& yw, uint32_t g) {
            if (WEIGHT && g < ng) yw = weight_at(g);           // uniform
            if (g < nf) {                                      // uniform; in the order in which the main loop waits for them
#pragma unroll
                for (int i = 0; i < CA; ++i) {
                    ya[i] = load_a(i, g);
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int i = 0; i < CB; ++i) {
                    yb[i] = load_b(i, g);
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else if (g < ng) {
                const int lp = hide(threadIdx.x & 63);
#pragma unroll
                for (int i = 0; i < CA; ++i) ya[i] = load_part(km_a, pa[i], sa, ca[i] ? ga_cut : ga, i, g, lp);
#pragma unroll
                for (int i = 0; i < CB; ++i) yb[i] = load_part(km_b, pb[i], sb, cb[i] ? gb_cut : gb, i, g, lp);
            }
        };
        // ---- scales, from a sample of the range: the first group of 32 k and one to three more, those of a K-major operand from 32 or 96
        // places.
        {
            constexpr int QS = 4;
            fetch(za, zb, zw, 0);
            for (int t = threadIdx.x; t < SLOTS; t += THREADS) mx[t] = few[t] = bias[t] = 0;
            if (threadIdx.x < 5) mt[threadIdx.x] = 0;
            auto place = [&](int at, float of) { return (uint32_t)(((float)at + 0.5f) * ((float)nf * of)); };       // below nf
            const bool more = ng >= 64;                        // uniform: short ranges are sampled in two groups
            // The last group of a row holds the diagonal, if the range does: that of a nearly diagonal matrix (an inverse) towers above
            // the rest of the row, which is scaled as if it was not there as far as fp16 reaches.
            auto diagonal = [&](const Side& o, int i) {        // its group, ng outside of the range
                const uint64_t d = (o.first + chunk_row(o, i)) / 32 - g0;             // wraps below the range
                return nf != 0 && d < ng && !past(o, i) ? (uint32_t)d : ng;
            };
            const uint32_t group[QS] = {0, (uint32_t)__builtin_amdgcn_readfirstlane(place(0, more ? 1.0f / 3.0f : 1.0f)),
                                        (uint32_t)__builtin_amdgcn_readfirstlane(place(1, 1.0f / 3.0f)),
                                        (uint32_t)__builtin_amdgcn_readfirstlane(place(2, 1.0f / 3.0f))};             // of a row's parts
            auto look = [&](auto km, const Side& o, gfloat p, uint32_t gofs, int t, int i) {
                uint32_t g;
                if constexpr (decltype(km)::value) {
                    g = place(((t - 1) * 4 + i) * 8 + first_k(km, o, ln) / 4, more ? 1.0f / 96.0f : 1.0f / 32.0f);
                    if (nf == 0 || (t != 1 && !more)) return f32x4{0.0f, 0.0f, 0.0f, 0.0f};                           // uniform
                } else {
                    const uint32_t d = t == QS - 1 ? diagonal(o, i) : ng;
                    if (d < ng && d >= nf) return load_part(km, p, o, gofs, i, d, ln);                                // uniform
                    g = d < nf ? d : group[t];
                    if (nf == 0 || (t != 1 && !more && d >= nf)) return f32x4{0.0f, 0.0f, 0.0f, 0.0f};                // uniform
                }
                return f32x4(*(gvec)((gbyte)p + gofs + (uint64_t)g * (4 * o.step)));
            };
            f32x4 ya[QS][CA], yb[QS][CB], yw;                  // weights of the second part of the sample
#pragma unroll
            for (int t = 1; t < QS; ++t) {
#pragma unroll
                for (int i = 0; i < CA; ++i) ya[t][i] = look(km_a, sa, pa[i], ca[i] ? ga_cut : ga, t, i);
#pragma unroll
                for (int i = 0; i < CB; ++i) yb[t][i] = look(km_b, sb, pb[i], cb[i] ? gb_cut : gb, t, i);
            }
            // Weights are at most one, and in a trained mask a few are one and the others next to nothing, which a sample would miss:
            // rows are scaled by their own largest value and the largest weight of the range.
            float wm = 0.0f;
            if constexpr (WEIGHT) {
                yw = *(gvec)((gfloat)a.weight + g0 * 32 + (uint64_t)place(0, more ? 1.0f / 3.0f : 1.0f) * 32 + 4 * (ln & 7));
                for (uint64_t j = 4 * threadIdx.x; j < (uint64_t)ng * 32; j += 4 * THREADS) wm = __builtin_fmaxf(wm, largest(f32x4(*(gvec)((gfloat)a.weight + g0 * 32 + j))));
            }
            fetch(xa, xb, xw, 1);
#pragma unroll
            for (int i = 0; i < CA; ++i) ya[0][i] = za[i];
#pragma unroll
            for (int i = 0; i < CB; ++i) yb[0][i] = zb[i];
            // Columns past the edge are loaded from the last ones again, which count once.
            auto counts = [&](auto km, const Side& o, int i) { return !decltype(km)::value || column_at(o, ln) + i >= column(o, ln); };
            // The 8 lanes that hold a row agree on what is in it; a column is spread over wavefronts.
            auto top = [](float x, float y) { return __builtin_fmaxf(x, y); };
            auto add = [](auto x, auto y) { return x + y; };
            auto post = [&](auto km, const Side& o, const auto& y, const gfloat* p, const bool* c, uint32_t gofs, uint32_t gofs_cut, auto n) {
                constexpr int N = decltype(n)::value;
                float m[N], diag[N];
                bool uneven = false;
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    uint32_t quads = 0;                        // that are not zero
                    float l[QS];
                    diag[i] = 0.0f;
                    const uint32_t d = decltype(km)::value ? ng : diagonal(o, i);
#pragma unroll
                    for (int t = QS - 1; t >= 0; --t) {
                        f32x4 v = values(km, y[t], i);
                        quads += largest(v) != 0.0f;
                        if (!decltype(km)::value && t == QS - 1 && d < ng) {          // uniform
                            const int row = (int)((o.first + chunk_row(o, i)) & 31) + (ln >> 3);
                            const bool mine = row >> 2 == (ln & 7);
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                if (mine && (row & 3) == e) { diag[i] = __builtin_fabsf(v[e]); v[e] = 0.0f; }
                        }
                        l[t] = largest(v);
                        if constexpr (!decltype(km)::value) {
                            l[t] = over_8_lanes(l[t], top);
                            if (t < QS - 1 && d == group[t]) l[t] = l[QS - 1];        // the same group, without the diagonal
                        }
                    }
                    m[i] = top(top(l[0], l[1]), l[2]);
                    uneven |= __builtin_fminf(__builtin_fminf(l[0], l[1]), more ? l[2] : l[1]) * 64.0f <= m[i];
                    m[i] = top(m[i], l[3]);
                    if constexpr (decltype(km)::value) {
                        if (quads != 0 && counts(km, o, i)) atomicAdd(&few[slot_of(km, o, ln, i)], quads);
                    } else {
                        few[slot_of(km, o, ln, i)] = over_8_lanes(quads, add);
                    }
                }
                if constexpr (!decltype(km)::value) {
                    // Rows whose groups are of different sizes or zero (half of the neurons dead) are looked at in 24 more places, one
                    // per lane.  For all rows that would be eight times the lines (64 x 65,536 x 2,048: 140 -> 156 us).
                    if (nf != 0 && __any(uneven)) {            // uniform
#pragma unroll 1
                        for (int t = 0; t < 3; ++t) {
                            const uint64_t g = place(t * 8 + (ln & 7), 1.0f / 24.0f);
                            f32x4 z[N];
#pragma unroll
                            for (int i = 0; i < N; ++i) z[i] = *(gvec)((gbyte)p[i] + (c[i] ? gofs_cut : gofs) + g * (4 * o.step));
#pragma unroll
                            for (int i = 0; i < N; ++i) m[i] = __builtin_fmaxf(m[i], largest(z[i]));
                        }
#pragma unroll
                        for (int i = 0; i < N; ++i) m[i] = over_8_lanes(m[i], top);
                    }
                }
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    const int slot = slot_of(km, o, ln, i);
                    if constexpr (decltype(km)::value) {
                        atomicMax(&mx[slot], __float_as_uint(m[i]));
                    } else {
                        mx[slot] = __float_as_uint(top(m[i], over_8_lanes(diag[i], top)));
                        mx2[slot] = __float_as_uint(m[i]);
                    }
                }
            };
            __syncthreads();
            post(km_a, sa, ya, pa, ca, ga, ga_cut, std::integral_constant<int, CA>{});
            post(km_b, sb, yb, pb, cb, gb, gb_cut, std::integral_constant<int, CB>{});
            if (WEIGHT) atomicMax(&mt[3], __float_as_uint(wm));
            __syncthreads();
            auto inside = [&](auto km, const Side& o, int t) { // a slot in front of the edge
                const int s = t - o.slot0;
                return o.first + (decltype(km)::value ? (s & ~63) + 4 * (s & 15) + ((s >> 4) & 3) : s) < o.rows;
            };
            // Slots without a value other than zero get the largest scale: a value that the sample does not show is too large for it,
            // or one of very few bits.  Where more than an eighth of the others have values in 1 to 5 of 32 quads of the sample (scattered
            // ones, not runs), too many samples are empty by chance, and sums of nothing (which do not pass) are frequent.
            for (int t = threadIdx.x; t < SLOTS; t += THREADS) {
                const bool side = t >= TM;                     // uniform
                uint32_t u = mx[t], u2 = (side ? BKN : AKN) ? u : mx2[t];
                if (WEIGHT && !side) {
                    u = __float_as_uint(__uint_as_float(u) * __uint_as_float(mt[3]));
                    u2 = __float_as_uint(__uint_as_float(u2) * __uint_as_float(mt[3]));
                }
                int e = 127;
                if (u != 0) e = kSampleTop - lead_exponent(u2 != 0 ? u2 : u);
                if (u2 != 0 && e > kDiagonalTop - lead_exponent(u)) e = kDiagonalTop - lead_exponent(u);
                ex[t] = clamp_exponent(e);
                const bool live = u != 0 && (side ? inside(km_b, sb, t) : inside(km_a, sa, t));
                const uint32_t n = __builtin_popcountll(__ballot(live)), rare = __builtin_popcountll(__ballot(live && few[t] - 1 < 5));
                if ((t & 63) == 0) atomicAdd(&mt[side ? 2 : 0], n << 16 | rare);
                mx[t] = 0;
                bias[t] = 0;
                few[t] = live ? 0 : ~0u;
            }
            __syncthreads();
            const uint32_t va = mt[0], vb = mt[2];
            if (nf != 0 && ((va & 0xFFFFu) * 8 > va >> 16 || (vb & 0xFFFFu) * 8 > vb >> 16)) return kExact;          // uniform
            if constexpr (WEIGHT) {
#pragma unroll
                for (int i = 0; i < CA; ++i) weigh(ya[1][i], yw);
            }
            // What the second part of the sample, 32 values of a slot, says about the range
            auto count = [&](auto km, const Side& o, const auto& y, int n) {
                const uint32_t small = (__float_as_uint(8.0f * unit) << 1) - 1;
#pragma unroll
                for (int i = 0; i < n; ++i) {
                    const int slot = slot_of(km, o, ln, i);
                    const bool use = counts(km, o, i) && few[slot] != ~0u;
                    const f32x4 v = values(km, y, i) * __builtin_ldexpf(1.0f, ex[slot]);
                    float q = 0.0f;
                    uint32_t least = ~0u, c = 0;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const uint32_t u = (__float_as_uint(v[e]) << 1) - 1;          // order of |v|, zero above all
                        q = __builtin_fmaf(v[e], v[e], q);
                        least = u < least ? u : least;
                        c += __builtin_fabsf(v[e]) >= 1.0f;
                    }
                    c <<= 16;
                    if (least < small) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) c += (__float_as_uint(v[e]) << 1) - 1 < small;
                    }
                    if constexpr (decltype(km)::value) {
                        if (use) {
                            atomicAdd(&mx[slot], (uint32_t)q); // at most 2^25 in all
                            atomicAdd(&few[slot], c);
                        }
                    } else {
                        q = over_8_lanes(q, add);
                        c = over_8_lanes(c, add);
                        if (use) { mx[slot] = (uint32_t)q; few[slot] = c; }
                    }
                }
            };
            count(km_a, sa, ya[1], CA);
            count(km_b, sb, yb[1], CB);
            __syncthreads();
            auto lose = [&](auto km, const Side& o, const auto& y, int n) {
#pragma unroll
                for (int i = 0; i < n; ++i) {
                    const int slot = slot_of(km, o, ln, i);
                    if (!counts(km, o, i) || few[slot] == ~0u || (few[slot] & 0xFFFFu) < 4) continue;
                    const f32x4 v = values(km, y, i) * __builtin_ldexpf(1.0f, ex[slot]);
                    int r = 0;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float x = __builtin_fabsf(v[e]), h = (float)(_Float16)x;
                        if (x < 8.0f * unit) r += (int)(((x - h) - (float)(_Float16)(x - h)) * 8589934592.0f);
                    }
                    if (r) atomicAdd(&bias[slot], r);
                }
            };
            lose(km_a, sa, ya[1], CA);
            lose(km_b, sb, yb[1], CB);
            __syncthreads();
            for (int t = threadIdx.x; t < SLOTS; t += THREADS) {
                const bool in = few[t] != ~0u;
                const float c = (float)(few[t] & 0xFFFFu), f = (2.0f * c + (c > 0.0f)) * (1.0f / 32.0f);
                const float lean = c < 4.0f ? 0.25f : __builtin_fabsf((float)bias[t]) / (256.0f * c) - 1.2f * __builtin_amdgcn_rsqf(c);
                const float share = __builtin_fmaxf(0.25f, __builtin_fminf(1.0f, 2.0f * __builtin_sqrtf(f)));
                odd[t] = few[t] >> 16 < 24 ? -share : share;
                if (in && odd[t] < 0.0f) mt[4] = 1;
                nrm[t] = in ? __builtin_sqrtf((float)mx[t] * (kr / 16.0f) + 4194304.0f) : 0.0f;
                gam[t] = in ? __builtin_fmaxf(2.0f, __builtin_sqrtf(f) * __builtin_fmaxf(4.0f, lean * __builtin_sqrtf(kr))) : 0.0f;
            }
        }
        float fsa[CA], fsb[CB];                                // scales of the thread's slots
        // Rows past the edge are scaled by zero: products with zero take less of the power that limits the clock.
        auto scale_of = [&](auto km, const Side& o, int i) {
            const uint64_t row = decltype(km)::value ? o.first + (int64_t)(column_at(o, ln) + i) : o.first + chunk_row(o, i) + (ln >> 3);
            return row < o.rows ? __builtin_ldexpf(1.0f, ex[slot_of(km, o, ln, i)]) : 0.0f;
        };
#pragma unroll
        for (int i = 0; i < CA; ++i) fsa[i] = scale_of(km_a, sa, i);
#pragma unroll
        for (int i = 0; i < CB; ++i) fsb[i] = scale_of(km_b, sb, i);
        // LDS byte offset of the thread's columns; of its first row: the others are 8 slots apart, which the exclusive or may turn
        // into 8 back (bit 7 of the offset).
        uint32_t wa[AKN ? CA : 1], wb[BKN ? CB : 1];
#pragma unroll
        for (int i = 0; i < (AKN ? CA : 1); ++i) wa[i] = in_plane(km_a, sa, ln, slot_of(km_a, sa, ln, i));
#pragma unroll
        for (int i = 0; i < (BKN ? CB : 1); ++i) wb[i] = in_plane(km_b, sb, ln, slot_of(km_b, sb, ln, i));

        // Two fp16 pieces of 4 values.
        auto stash = [&](auto km, const auto& x, const f32x4* wt, const uint32_t* w, float scale, int i, uint32_t stage) {
            f32x4 v = values(km, x, i);
            if (wt) weigh(v, *wt);
            u32x2 p0, p1;
#pragma unroll
            for (int e = 0; e < 4; e += 2) {
                const f16x2 h = __builtin_convertvector((f32x2{v[e] * scale, v[e + 1] * scale}), f16x2);
                p0[e / 2] = __builtin_bit_cast(uint32_t, h);
                p1[e / 2] = __builtin_bit_cast(uint32_t, (f16x2{(_Float16)__builtin_fmaf(v[e], scale, -(float)h[0]),
                                                                (_Float16)__builtin_fmaf(v[e + 1], scale, -(float)h[1])}));
            }
            unsigned char* st = smem + (decltype(km)::value ? w[i] + stage : ((w[0] + stage) ^ ((i & 1) * 128)) + (i >> 1) * 256);
            *reinterpret_cast<u32x2*>(st) = p0;
            *reinterpret_cast<u32x2*>(st + kPlane) = p1;
        };

        // ---- fragments: lane l holds k 8 (l / 16)..+7 of slot l % 16 of a block of 16
        const uint32_t fofs = (ln >> 4) * kReg + ((ln & 15) ^ turn(ln >> 4)) * 16;
        const uint32_t a_ofs = fofs + wm * RB * 256, b_ofs = fofs + (TM + wn * NB * 16) * 16;
        struct Frag { f16x8 p[2]; };
        auto load = [&](Frag& f, uint32_t at, int block) {
#pragma unroll
            for (int q = 0; q < 2; ++q) f.p[q] = *reinterpret_cast<const f16x8*>(smem + at + (q * kPlane + block * 256));
        };
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

        // ---- pipeline
        const std::true_type yes;
        const std::false_type no;
#pragma unroll
        for (int i = 0; i < CA; ++i) stash(km_a, za, &zw, wa, fsa[i], i, 0);
#pragma unroll
        for (int i = 0; i < CB; ++i) stash(km_b, zb, nullptr, wb, fsb[i], i, 0);
        Frag fa[2], fb[NB];
        uint32_t cur = 0, g = 0;
        auto group = [&](auto full, uint32_t gi) {
            constexpr bool FULL = decltype(full)::value;
            const uint32_t nxt = kStage - cur;
            const uint32_t a_cur = a_ofs + cur;
#pragma unroll
            for (int i = 0; i < RB; ++i) {
                if (i + 1 < RB) {
                    load(fa[(i + 1) & 1], a_cur, i + 1);
#pragma unroll
                    for (int q = 0; q < NC; ++q) {
                        if (q * (RB - 1) / NC != i) continue;
                        if (q < CA) {
                            stash(km_a, xa, &xw, wa, fsa[q], q, nxt);
                            if constexpr (FULL) {
                                if (q == CA - 1) {
                                    if (WEIGHT) xw = weight_at(gi + 2);
#pragma unroll
                                    for (int r = 0; r < CA; ++r) xa[r] = load_a(r, gi + 2);
                                }
                            }
                        } else {
                            const int r = q - CA;
                            stash(km_b, xb, nullptr, wb, fsb[r], r, nxt);
                            if constexpr (FULL) {
                                if (!BKN) xb[r] = load_b(r, gi + 2);
                                else if (r == CB - 1) {
#pragma unroll
                                    for (int r2 = 0; r2 < CB; ++r2) xb[r2] = load_b(r2, gi + 2);
                                }
                            }
                        }
                    }
                } else {
                    if constexpr (!FULL) fetch(xa, xb, xw, gi + 2);
                    wait_lds();
                    f32_barrier();
                    load(fa[0], a_ofs + nxt, 0);
                }
                // products of pieces, small terms first.  The last block of rows goes column by column: the fragments of B
                // are replaced as they fall free, so that one set of them is enough.
                constexpr int ka[3] = {1, 0, 0}, kb[3] = {0, 1, 0};
                auto mma = [&](int j, int t) {
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fa[i & 1].p[ka[t]], fb[j].p[kb[t]], acc[i][j], 0, 0, 0);
                };
                if (i + 1 < RB) {
#pragma unroll
                    for (int t = 0; t < 3; ++t)
#pragma unroll
                        for (int j = 0; j < NB; ++j) mma(j, t);
                } else {
#pragma unroll
                    for (int j = 0; j < NB; j += 2) {
#pragma unroll
                        for (int t = 0; t < 3; ++t) { mma(j, t); mma(j + 1, t); }
                        load(fb[j], b_ofs + nxt, j);
                        load(fb[j + 1], b_ofs + nxt, j + 1);
                    }
                }
#pragma unroll
                for (int q = 0; q < 3 * NB / 2; ++q) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);               // two matrix instructions
                    __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);               // vector arithmetic
                    __builtin_amdgcn_sched_group_barrier(0x300, 1, 0);               // one LDS read or write
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            cur = nxt;
        };
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0x0F70);                    // vmcnt == 0, or the loop's waits would also be for loads before it
        __builtin_amdgcn_sched_barrier(0);
        wait_lds();
        f32_barrier();
#pragma unroll
        for (int j = 0; j < NB; ++j) load(fb[j], b_ofs, j);
        load(fa[0], a_ofs, 0);
        for (; g + 2 < nf; ++g) group(yes, g);
        for (; g < ng; ++g) group(no, g);

    }

    // ---- check of the sums; the stages are no longer read
    uint32_t* const list = reinterpret_cast<uint32_t*>(smem);
    const int ln = hide(threadIdx.x & 63), lq = ln >> 4, lc = ln & 15;
    __syncthreads();
    auto a_row = [&](int i, int r) {                           // row of A in slot r of the wavefront's block i of 16
        const int s = wm * RB * 16 + i * 16 + r;
        return m0 + (AKN ? (s & ~63) + 4 * (s & 15) + ((s >> 4) & 3) : s);
    };
    auto b_col = [&](int j) {                                  // column of C in block j of the lane
        const int s = wn * NB * 16 + j * 16 + lc;
        return n0 + (BKN ? (s & ~63) + 4 * (s & 15) + ((s >> 4) & 3) : s);
    };
    const int* const ea = ex + wm * RB * 16 + 4 * lq;
    const int* const eb = ex + TM + wn * NB * 16 + lc;
    const float* const na = nrm + wm * RB * 16 + 4 * lq;
    const float* const nb = nrm + TM + wn * NB * 16 + lc;
    const float* const ga = gam + wm * RB * 16 + 4 * lq;
    const float* const gb = gam + TM + wn * NB * 16 + lc;
    const float* const oa = odd + wm * RB * 16 + 4 * lq;
    const float* const ob = odd + TM + wn * NB * 16 + lc;
    const bool any_odd = mt[4] != 0;                           // uniform
    if constexpr (GRAD) {
        auto r = [&](int i, int j, int e) { return __builtin_ldexpf(acc[i][j][e], -(ea[i * 16 + e] + eb[j * 16])); };
        auto lost = [&](int i, int e) {
            const float x = __builtin_ldexpf(4.0f / 3.0f * unit, -ea[i * 16 + e]);
            return f32x2{x * na[i * 16 + e], x * ga[i * 16 + e]};
        };
        auto col = [&](int j) { return f32x2{__builtin_ldexpf(gb[j * 16], -eb[j * 16]), __builtin_ldexpf(nb[j * 16], -eb[j * 16])}; };
        double* const part = reinterpret_cast<double*>(smem);
        if (any_odd) return grad_tail<RB, NB, WR, WC, kSize>(a, *tail, part, n0, r, lost, col) ? kDone : kExact;          // uniform
        return grad_tail<RB, NB, WR, WC, kFinite>(a, *tail, part, n0, r, lost, col) ? kDone : kExact;
    } else {
        // Sums that do not pass, 4 bits each (e) of the 4 blocks of a row of blocks.  Slots without a value other than zero have
        // nothing to lose.
        const bool interior = m0 + TM <= a.M && n0 + TN <= a.N;                       // uniform
        uint32_t todo[(RB + 1) / 2], n = 0;
#pragma unroll
        for (int i = 0; i < (RB + 1) / 2; ++i) todo[i] = 0;
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            float worst = 0.0f, sum = 0.0f;                    // cheaply first: 128 sums a lane
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int j = 0; j < NB; ++j) sum = __builtin_fmaf(acc[i][j][e], 0.0f, sum);
            if (any_odd) {                                     // uniform
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float x = 4.0f / 3.0f * unit * na[i * 16 + e], g = 4.0f / 3.0f * unit * ga[i * 16 + e];
#pragma unroll
                    for (int j = 0; j < NB; ++j)
                        worst = __builtin_fmaxf(worst, __builtin_fmaf(x, gb[j * 16], __builtin_fmaf(g, nb[j * 16], -__builtin_fabsf(acc[i][j][e]))));
                }
            }
            if (!__any(!(worst <= 0.0f && sum == 0.0f))) continue;                    // uniform
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float x = 4.0f / 3.0f * unit * na[i * 16 + e], g = 4.0f / 3.0f * unit * ga[i * 16 + e];
                const bool in = interior || a_row(i, 4 * lq + e) < a.M;
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    const float p = oa[i * 16 + e], q = ob[j * 16];
                    const float low = p > 0.0f && q > 0.0f ? 0.0f : x * gb[j * 16] * (p < 0.0f ? 1.0f : __builtin_fabsf(q)) +
                                                                    g * nb[j * 16] * (q < 0.0f ? 1.0f : __builtin_fabsf(p));
                    const float v = __builtin_fabsf(acc[i][j][e]);
                    if (!(v >= low && v < __builtin_inff()) && in && (interior || b_col(j) < a.N)) todo[i / 2] |= 1u << ((i & 1) * 16 + j * 4 + e);
                }
            }
        }
#pragma unroll
        for (int i = 0; i < (RB + 1) / 2; ++i) n += __builtin_popcount(todo[i]);
        // As many of them as can be summed one by one in less time than the tile takes with three bf16 pieces (1,000 + 100 rows of
        // 1,863,690 in 64 ranges: 13 us each, 1.9 ms).  A column of a K-major operand is a line of 128 bytes per value (50 us for 9,362 of them).
        const uint32_t limit = AKN ? 2 * NW : BKN ? 4 * NW : kr < 4.0f * SLOTS / NW ? NW * (uint32_t)kr / 16 : SLOTS / 4;
        if (n != 0) {
            uint32_t at = atomicAdd(&mt[1], n);
#pragma unroll
            for (int q = 0; q < (RB + 1) / 2; ++q)
                for (uint32_t w = todo[q]; w != 0; w &= w - 1, ++at) {
                    const int bit = __builtin_ctz(w), i = 2 * q + (bit >> 4), j = bit >> 2 & 3, e = bit & 3;
                    if (at < limit) list[at] = (uint32_t)(a_row(i, 4 * lq + e) - m0) << 16 | (uint32_t)(b_col(j) - n0);
                }
        }
        __syncthreads();
        const uint32_t total = mt[1];
        if (total > limit) return kExact;                      // uniform

        // ---- results
        const bool quads = BKN && interior && !a.accumulate && a.ldc % 4 == 0 && (reinterpret_cast<uintptr_t>(a.C) & 15) == 0;
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint64_t row = a_row(i, 4 * lq + e);
                const int er = ea[i * 16 + e];
                float v[NB];
#pragma unroll
                for (int j = 0; j < NB; ++j) v[j] = __builtin_ldexpf(acc[i][j][e], -(er + eb[j * 16]));
                float* const c = a.C + row * a.ldc;
                if (quads) {
                    *reinterpret_cast<f32x4*>(c + b_col(0)) = f32x4{v[0], v[1], v[2], v[3]};
                } else {
#pragma unroll
                    for (int j = 0; j < NB; ++j) {
                        const uint64_t col = b_col(j);
                        if (interior && !a.accumulate) c[col] = v[j];
                        else if (row < a.M && col < a.N && !(a.accumulate && (todo[i / 2] >> ((i & 1) * 16 + j * 4 + e) & 1)))
                            c[col] = a.accumulate ? c[col] + v[j] : v[j];
                    }
                }
            }
        return total;
    }
}

// A tile that pair_tile gives up, on three bf16 pieces.
template <int RB, int NB, int WR, int WC, bool AKN, bool BKN, bool WEIGHT>
__device__ __attribute__((noinline)) void exact_tile(GemmF32Args a, lds_byte lds) {
    constexpr int TM = 16 * RB * WR, TN = 16 * NB * WC;
    a = uniform(a);
    unsigned char* const smem = uniform_lds(lds);
    const auto [tm, tn, split] = gemm_f32_tile(a);
    a.C += split * a.split_stride_c;
    const uint64_t ng_all = (a.K + 31) / 32, g0 = split * ng_all / a.splits, ng = (split + 1) * ng_all / a.splits - g0;
    const uint64_t m0 = (uint64_t)tm * TM, n0 = (uint64_t)tn * TN;
    constexpr uint32_t lds_bytes = 2 * 8 * (TM + TN) * 16;     // the stages of pair_tile
    if constexpr (RB == 8) {
        static_assert(split_lds<4, 2, 2, 4>() <= lds_bytes && TM == 256 && TN == 256, "256 x 256");
        split_tile<4, 2, 2, 4, AKN, BKN, false, WEIGHT>(a, smem, threadIdx.x, m0, n0, g0, ng);
    } else {                                                   // halves of 128 x 128, 4 wavefronts each; TM == 64 has no rows 64..127
        constexpr uint32_t half = split_lds<2, 2, 2, 2>();
        static_assert(half * (TN / 128) <= lds_bytes && TM <= 128 && TN / 128 * 4 == WR * WC, "128 x 128");
        const uint32_t h = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
        split_tile<2, 2, 2, 2, AKN, BKN, false, WEIGHT>(a, smem + h * half, threadIdx.x & 255, m0, n0 + h * 128, g0, ng);
    }
}

template <int RB, int NB, int WR, int WC, bool AKN, bool BKN, bool WEIGHT = false>
__global__ void __launch_bounds__(64 * WR * WC, 2) gemm_pair_kernel(GemmF32Args a) {
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t left = pair_tile<RB, NB, WR, WC, AKN, BKN, WEIGHT>(a, (lds_byte)smem);
    if (left == kDone) return;                                 // uniform
    __builtin_amdgcn_s_waitcnt(0x0F70);                        // vmcnt == 0: what is stored is there
    __syncthreads();
    if (left == kExact) exact_tile<RB, NB, WR, WC, AKN, BKN, WEIGHT>(a, (lds_byte)smem);
    else sum_again<RB, NB, WR, WC, AKN, BKN, WEIGHT>(a, (lds_byte)smem, left);
}

template <int RB, int NB, int WR, int WC>
__global__ void __launch_bounds__(64 * WR * WC, 2) gemm_pair_grad_kernel(GemmF32Args a, GradTail t) {
    extern __shared__ __align__(16) unsigned char smem[];
    if (pair_tile<RB, NB, WR, WC, false, true, false, true>(a, (lds_byte)smem, &t) == kDone) return;         // uniform
    __syncthreads();
    exact_tile<RB, NB, WR, WC, false, true, false>(a, (lds_byte)smem);
    __builtin_amdgcn_s_waitcnt(0x0F70);                        // vmcnt == 0: R is stored
    __syncthreads();
    const uint64_t n0 = (uint64_t)gemm_f32_tile(a).tn * (16 * NB * WC);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t c0 = n0 + (wave % WC) * NB * 16 + 4 * (lane & 15);
    auto r = [&](int i, int j, int e) { return a.C[(uint64_t)((wave / WC * RB + i) * 16 + 4 * (lane >> 4) + e) * a.ldc + c0 + j]; };
    grad_tail<RB, NB, WR, WC, kNothing>(a, t, reinterpret_cast<double*>(smem), n0, r, [](int, int) { return f32x2{}; }, [](int) { return f32x2{}; });
}

template <int RB, int NB, int WR, int WC, bool AKN, bool BKN, bool WEIGHT = false>
static hipError_t launch_pair(GemmF32Args a, hipStream_t st) {
    constexpr uint64_t TM = 16 * RB * WR, TN = 16 * NB * WC;
    constexpr uint64_t lds = 2 * 8 * (TM + TN) * 16 + (TM + TN) * 16 + 32;
    static_assert(lds <= kLdsBytes, "LDS");
    a.tiles_m = (uint32_t)ceil_div(a.M, TM);
    a.tiles_n = (uint32_t)ceil_div(a.N, TN);
    if (a.lower_only && a.tiles_m != a.tiles_n) return hipErrorInvalidValue;
    const uint64_t total = (a.lower_only ? (uint64_t)a.tiles_m * (a.tiles_m + 1) / 2 : (uint64_t)a.tiles_m * a.tiles_n) * a.splits;
    if (total == 0 || total > 0x7FFFFFFFull) return hipErrorInvalidValue;
    static LdsOptIn opt_in;
    hipError_t e = allow_large_lds(opt_in, reinterpret_cast<const void*>(gemm_pair_kernel<RB, NB, WR, WC, AKN, BKN, WEIGHT>));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((gemm_pair_kernel<RB, NB, WR, WC, AKN, BKN, WEIGHT>), dim3((uint32_t)total), dim3(64 * WR * WC), lds, st, a);
    return hipGetLastError();
}

hipError_t gemm_f32_pair_weighted(const GemmF32Args& a, hipStream_t st) {
    if (a.M > 128 || !a.weight || !aligned(a.weight, 16) || gemm_f32_wide(a.lda > a.ldb ? a.lda : a.ldb)) return hipErrorInvalidValue;
    return launch_pair<4, 4, 2, 4, false, false, true>(a, st);
}

template <int RB, int NB, int WR, int WC>
static hipError_t launch_pair_grad(GemmF32Args a, const GradTail& t, hipStream_t st) {
    constexpr uint64_t TM = 16 * RB * WR, TN = 16 * NB * WC;
    constexpr uint64_t lds = 2 * 8 * (TM + TN) * 16 + (TM + TN) * 16 + 32;
    a.tiles_m = 1;
    a.tiles_n = (uint32_t)ceil_div(a.N, TN);
    static LdsOptIn opt_in;
    hipError_t e = allow_large_lds(opt_in, reinterpret_cast<const void*>(gemm_pair_grad_kernel<RB, NB, WR, WC>));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((gemm_pair_grad_kernel<RB, NB, WR, WC>), dim3(a.tiles_n), dim3(64 * WR * WC), lds, st, a, t);
    return hipGetLastError();
}

hipError_t gemm_f32_pair_grad(const GemmF32Args& a, const GradTail& t, hipStream_t st) {
    if (a.M > 128 || a.accumulate || a.splits != 1 || gemm_f32_wide(a.lda > a.ldb ? a.lda : a.ldb)) return hipErrorInvalidValue;
    // Up to 64 rows on tiles of 64 x 128, two workgroups per CU: half the products are not for padding.  Training steps on tiles of
    // 128 x 256 -> 64 x 128 (64 x 256): 43 + 258 rows of 280,270 1.22 -> 1.13 ms (1.15), 64 + 300 of 1,000,003 1.82 -> 1.67 (1.69),
    // 16 + 4,096 of 200,001 2.09 -> 2.04 (2.04).  Above, 128 x 128 is slower: 128 + 1,000 rows of 300,000 0.97 -> 1.00.
    if (a.M <= 64) return launch_pair_grad<2, 4, 2, 2>(a, t, st);
    return launch_pair_grad<4, 4, 2, 4>(a, t, st);
}

hipError_t gemm_f32_pair(bool a_kn, bool b_kn, int tile, const GemmF32Args& a, hipStream_t st) {
    switch (tile) {
        case kTile256:
            if (a_kn) return launch_pair<8, 4, 2, 4, true, true>(a, st);
            if (b_kn) return launch_pair<8, 4, 2, 4, false, true>(a, st);
            return launch_pair<8, 4, 2, 4, false, false>(a, st);
        case kTile128x256:
            if (a_kn) return hipErrorInvalidValue;
            if (b_kn) return launch_pair<4, 4, 2, 4, false, true>(a, st);
            return launch_pair<4, 4, 2, 4, false, false>(a, st);
        case kTile64:
            return hipErrorInvalidValue;
        default:
            if (a_kn) return launch_pair<4, 4, 2, 2, true, true>(a, st);
            if (b_kn) return launch_pair<4, 4, 2, 2, false, true>(a, st);
            return launch_pair<4, 4, 2, 2, false, false>(a, st);
    }
}

}  // namespace grass
