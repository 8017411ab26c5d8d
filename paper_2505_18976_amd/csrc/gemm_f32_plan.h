// Plan of the fp32 products: kernel, tile and K ranges.  Plain C++, so that tests can ask on the host which kernel a shape gets.
#pragma once

#include <stdint.h>

namespace grass {

constexpr uint64_t kGemmCUs = 256;       // MI355X
inline uint64_t gemm_div(uint64_t a, uint64_t b) { return (a + b - 1) / b; }

// 256 x 256, 128 x 128, 64 x 512 (only with three bf16 pieces), 128 x 256 (only with two fp16 pieces, A row-major)
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

// Kernel, tile and number of K ranges of a product.  Estimated time of a choice, in microseconds: the tiles run in rounds of
// as many workgroups as the chip holds; a slice of 16 k takes `full` (256 x 256; two workgroups of 128 x 128 on a CU; 64 x 512;
// 128 x 256) in a round that fills it and `part` in one of at most `part_wgs` workgroups; the C tiles leave at 4 TB/s; K ranges
// cost another launch that adds the partial sums.  Measured per slice with three bf16 pieces, 192 and 256 workgroups of 256 x
// 256 1.94 and 2.30, 256 and 512 of 128 x 128 1.01 and 1.44, 128 and 256 of 64 x 512 1.64 and 2.10; with two fp16 pieces (from
// the difference of K = 2,048 and 8,192) 1.15 and 1.32, 0.51 and 0.87 (the power limit leaves a part-filled chip a higher
// clock).  A launch of the latter takes 8 us more to start (sample of the operands, longer code).  128 x 256
// reads a quarter less per product than two workgroups of 128 x 128, which shows where at most 128 rows of A meet long rows of
// B: 100 x 1,000 x 400,001 in 64 ranges 475 -> 420 us.  64 x 512 is for at most 64 rows of A.
// On 160 drawn products (4 x 500 x 64 to 2,048 x 65,536 x 1,500, FIMs of 500 x 128 to 60,000 x 4,096) the choice takes 0.81 times
// the time of the best plan with three bf16 pieces in the geometric mean, and 1.06 at most.
struct TileCost { uint64_t tm, tn, per_cu; double full, part; uint64_t part_wgs; };
inline const TileCost kTiles[2][4] = {{{256, 256, 1, 2.1, 1.95, 192}, {128, 128, 2, 1.31, 1.05, 256}, {64, 512, 1, 2.15, 1.5, 128}},
                                      {{256, 256, 1, 1.32, 1.1, 192}, {128, 128, 2, 0.87, 0.5, 256}, {}, {128, 256, 1, 0.84, 0.62, 128}}};
constexpr double kPairStart = 8.0;       // us more than a launch on three bf16 pieces

inline GemmPlan gemm_f32_plan(bool a_kn, bool b_kn, uint64_t M, uint64_t N, uint64_t K, uint64_t ld_max, bool lower_only,
                              uint32_t max_splits) {
    GemmPlan best{kTile128, 1, false};
    const uint64_t groups = gemm_div(K, 32);
    const bool wide = gemm_f32_wide(ld_max);
    for (int pair = 0; pair < (wide ? 1 : 2); ++pair)
        for (int t = 0; t < (pair ? 4 : 3); ++t) {
            const TileCost& T = kTiles[pair][t];
            if (wide && t != kTile128) continue;
            if (t == kTile128x256 && a_kn) continue;
            if (t == kTile64 && (pair || a_kn || b_kn || lower_only || M > 64)) continue;
            const uint64_t side = gemm_div(M, T.tm);
            const uint64_t n = lower_only ? side * (side + 1) / 2 : side * gemm_div(N, T.tn);
            for (uint32_t s = 1; s <= max_splits && (s == 1 || groups / s >= 2); ++s) {
                if (pair && K / s < kPairMinK) break;
                const uint64_t wgs = n * s, cap = T.per_cu * kGemmCUs, rest = wgs % cap;
                const double slices = 2.0 * (double)gemm_div(groups, s), mb = (double)(M * N) * 4e-6 * s;
                const double us = slices * ((double)(wgs / cap) * T.full + (rest == 0 ? 0.0 : rest <= T.part_wgs ? T.part : T.full)) +
                                  mb / 4.0 + (s > 1 ? 4.0 + mb / 4.5 : 0.0) + (pair ? kPairStart : 0.0);
                if (pair && !best.pair && us > 0.94 * best.us) continue;          // 8 x 6,139 x 10,476: 3 % less estimated, 12 % more taken
                if (best.us == 0.0 || us < best.us) best = GemmPlan{t, s, pair != 0, us};
            }
        }
    return best;
}

// Columns of C that fill one round of the chip with the tile of `plan`.
inline uint64_t gemm_f32_round_columns(const GemmPlan& plan, uint64_t M) {
    const TileCost& T = kTiles[plan.pair][plan.tile];
    return T.per_cu * kGemmCUs / gemm_div(M, T.tm) * T.tn;
}

// A B^T with many columns: as many tile columns as fill whole rounds of the chip run as one launch, the columns left over
// as a second one with a plan of their own (K ranges, smaller tiles) instead of a last round that is nearly empty.  The
// second launch starts when the first has drained, about 4 us.  1,000 x 50,001 x 4,096 has 784 tiles of 256 x 256 for 256
// CUs: two K ranges of everything (6.1 rounds of half the length) took 2.09 ms, 49,152 columns in three rounds and 849 in 16
// K ranges take 1.80 ms.
inline GemmCut gemm_f32_cut(uint64_t M, uint64_t N, uint64_t K, uint64_t ld_max, uint32_t max_splits) {
    GemmCut best{0, GemmPlan{kTile128, 1, false}, gemm_f32_plan(false, false, M, N, K, ld_max, false, max_splits)};
    if (gemm_f32_wide(ld_max)) return best;
    double best_us = 0.97 * best.tail.us;                  // a cut has to be worth its launch: below 3 % it measured 2 % slower
    const bool pair = K >= kPairMinK;
    for (int t = 0; t < (pair ? 4 : 3); ++t) {
        const TileCost& T = kTiles[pair][t];
        if (t == kTile64 && (pair || M > 64)) continue;
        const uint64_t side = gemm_div(M, T.tm), cap = T.per_cu * kGemmCUs;
        const uint64_t rounds = side * (N / T.tn) / cap;
        for (uint64_t q = rounds; q > 0 && q + 2 > rounds; --q) {                // all full rounds, or one less
            const uint64_t head_n = q * cap / side * T.tn;
            if (head_n == 0 || head_n >= N) continue;
            const double head_us = 2.0 * (double)gemm_div(K, 32) * (double)q * T.full + (double)(M * head_n) * 1e-6 + (pair ? kPairStart : 0.0);
            const GemmPlan tail = gemm_f32_plan(false, false, M, N - head_n, K, ld_max, false, max_splits);
            if (head_us + 4.0 + tail.us < best_us) {
                best_us = head_us + 4.0 + tail.us;
                best = GemmCut{head_n, GemmPlan{t, 1, pair, head_us}, tail};
            }
        }
    }
    return best;
}

}  // namespace grass
