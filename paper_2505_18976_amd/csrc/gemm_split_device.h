// A tile of an fp32 product on three bf16 pieces per operand: device code of gemm_split.hip, where the method is described, and of
// the tiles that gemm_pair.hip gives up.
#pragma once

#include <type_traits>

#include "gemm_f32_device.h"

namespace grass {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
constexpr float kSplitScale = 16777216.0f, kSplitUnscale = 1.0f / (kSplitScale * kSplitScale);

// Two fp32 values times kSplitScale -> their three bf16 pieces, packed in pairs.
__device__ __forceinline__ void split3(float x, float y, uint32_t& p0, uint32_t& p1, uint32_t& p2) {
    x *= kSplitScale;
    y *= kSplitScale;
    const bf16x2 h = __builtin_convertvector((f32x2{x, y}), bf16x2);
    p0 = __builtin_bit_cast(uint32_t, h);
    const float rx = x - __uint_as_float(p0 << 16), ry = y - __uint_as_float(p0 & 0xFFFF0000u);
    const bf16x2 m = __builtin_convertvector((f32x2{rx, ry}), bf16x2);
    p1 = __builtin_bit_cast(uint32_t, m);
    const float sx = rx - __uint_as_float(p1 << 16), sy = ry - __uint_as_float(p1 & 0xFFFF0000u);
    p2 = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{sx, sy}), bf16x2));
}

// One workgroup owns a TM x TN tile of C; its WR x WC wavefronts own 32 MI x 32 NJ each.  K is consumed in slices of 16
// through two LDS stages.  A stage holds the three bf16 planes of every tile row ("slot": the rows of A, then of B) as
// [plane][k half][slot][8 k], so that a fragment (lane l: row l%32, k 8(l/32)..+7) is one 16-byte read at a stride of 16
// bytes; the slots of the upper half are stored at slot ^ 8, which puts the two halves of a store into different banks.
// A slice travels from memory into registers two slices before it is split and stored, and it is stored one slice before
// it is multiplied.  The barrier of a slice sits before its last row of MFMA tiles: by then every wavefront has the
// fragments of this slice in registers and its part of the next slice in LDS; the first fragments of the next slice are
// requested behind it and the last row of tiles covers their latency.
// AKN / BKN: the operand is stored K-major (K x M resp. K x N).  A thread then takes 4 columns of 4 k-rows (16-byte loads
// along the rows) and stores 4 k of each column, the same LDS image, with the columns permuted inside blocks of 32 so
// that the stores spread over the banks.
// SIDE (tiles of 32 or 64 rows of A next to 512 of B): every wavefront loads 64 slots of B and a few of A.
// WIDE: 64-bit lane offsets, for rows so far apart that 16 of them exceed 4 GB (no chunk's lanes span more than 16 rows).
// WEIGHT: columns of A times a.weight on their way in, rounded once as a matrix of products would be.
// The tile's first row and column are m0 and n0, its groups of 32 k g0 .. g0 + ng - 1; a.C is that of the K range.  `smem` has
// split_lds<...>() bytes, `tid` counts the 64 WR WC threads; all of a workgroup's threads that share barriers run the same ng.
template <int MI, int NJ, int WR, int WC>
constexpr uint32_t split_lds() { return 2 * 32 * (MI * WR + NJ * WC) * 96; }

template <int MI, int NJ, int WR, int WC, bool AKN, bool BKN, bool WIDE, bool WEIGHT>
__device__ __forceinline__ void split_tile(const GemmF32Args& a, unsigned char* smem, int tid, uint64_t m0, uint64_t n0, uint64_t g0,
                                           uint64_t ng) {
    constexpr int NW = WR * WC;
    constexpr int TM = 32 * MI * WR, TN = 32 * NJ * WC, SLOTS = TM + TN;
    constexpr bool SIDE = SLOTS != 64 * NW;
    static_assert(SIDE ? (TN == 64 * NW && (TM == 32 || TM == 64) && NW == 8 && !AKN && !BKN) : TM % 64 == 0, "loading map");
    constexpr int NC = SIDE ? 5 : 4;                           // chunks of 4 fp32 per thread and slice
    constexpr int kHalf = SLOTS * 16, kPlane = 2 * kHalf, kStage = 3 * kPlane;
    static_assert(!WEIGHT || (!SIDE && !AKN && !WIDE), "weights");
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WC, wn = wave % WC;

    // ---- loading.  Addresses: per chunk a uniform base that walks along K plus a byte offset per lane inside its 16 rows.
    typedef typename std::conditional<WIDE, uint64_t, uint32_t>::type ofs_t;
    const bool is_a = !SIDE && wave * 64 < TM;                 // uniform per wavefront (the SIDE chunk belongs to A)
    const int unit = SIDE || is_a ? wave : wave - TM / 64;     // which 64 rows of its operand
    const bool kmajor = is_a ? AKN : BKN;
    const float* mat = is_a ? a.A : a.B;
    const uint64_t ld = is_a ? a.lda : a.ldb, rows = is_a ? a.M : a.N, r0 = is_a ? m0 : n0;
    const float* base[NC];                                     // row-major: row 16i of the wavefront's 64; K-major: the same for all
    ofs_t gofs[NC];
    uint32_t wofs[NC];                                         // LDS byte offset of chunk i inside a plane
    // row-major: chunk i = row 16i + lane/4, k 4(lane%4)..+3.  K-major: chunk i = k-row i of the thread's 4 x 4 block on
    // loading and its column i on storing.
    constexpr int GBA = TM / 128 > 0 ? TM / 128 : 1, GBB = TN / 128;                 // K-major: runs of 128 columns
    const int gb = is_a ? GBA : GBB;
    const int kq = kmajor ? (lane & 1) + 2 * (unit / gb) : lane & 3;
    int shift = 0;                                             // K-major, ragged edge: columns the loads were moved back by
    bool ragged = false, narrow = false;
    if (kmajor) {
        const int cq = 4 * ((lane >> 1) + 32 * (unit % gb));   // first of the thread's four columns
        narrow = rows < 4;                                     // too narrow for 16-byte loads
        const uint64_t rb = r0 + 4 <= rows ? r0 : narrow ? 0 : rows - 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) base[i] = mat + g0 * 32 * ld + rb;
        ragged = !narrow && rows % 4 != 0 && r0 + (is_a ? TM : TN) > rows;
        int c = cq;
        if (r0 + cq + 4 > rows && !narrow) {                   // columns past the edge: never stored
            shift = r0 + cq < rows ? (int)(r0 + cq + 4 - rows) : 0;
            c = (int)(rows - 4 - rb);
        }
        const int blk = cq >> 5, slot0 = (is_a ? 0 : TM) + blk * 32 + ((lane >> 1) & 7);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            gofs[i] = ((ofs_t)(4 * kq + i) * (ofs_t)ld + (ofs_t)c) * 4;
            const int slot = (slot0 + ((i ^ (blk & 1)) * 8)) ^ (kq >> 1) * 8;
            wofs[i] = (kq >> 1) * kHalf + slot * 16 + (kq & 1) * 8;
        }
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint64_t rb = r0 + unit * 64 + 16 * i;
            rb = rb < rows ? rb : rows - 1;
            base[i] = mat + rb * ld + g0 * 32;
            uint64_t r = rb + (lane >> 2);
            r = r < rows ? r : rows - 1;                       // rows past the edge re-read the last row; never stored
            gofs[i] = ((ofs_t)(r - rb) * (ofs_t)ld + 4 * kq) * 4;
            const int slot = ((SIDE ? TM : 0) + wave * 64 + 16 * i + (lane >> 2)) ^ (kq >> 1) * 8;
            wofs[i] = (kq >> 1) * kHalf + slot * 16 + (kq & 1) * 8;
        }
    }
    if constexpr (SIDE) {                                      // TM / 8 rows of A per wavefront, by the first lanes
        const uint64_t rb = m0 + wave * (TM / 8) < a.M ? m0 + wave * (TM / 8) : a.M - 1;
        base[4] = a.A + rb * a.lda + g0 * 32;
        const int rl = (lane >> 2) % (TM / 8);                 // the other lanes repeat them
        uint64_t r = rb + rl;
        r = r < a.M ? r : a.M - 1;
        gofs[4] = ((ofs_t)(r - rb) * (ofs_t)a.lda + 4 * kq) * 4;
        wofs[4] = (kq >> 1) * kHalf + ((wave * (TM / 8) + rl) ^ (kq >> 1) * 8) * 16 + (kq & 1) * 8;
    }
    const uint32_t ns = (uint32_t)(2 * ng);                    // slices of 16
    const uint64_t step = kmajor ? 16 * ld : 16;               // from a slice to the next

    // Slices whose 16 k all exist are loaded unconditionally (FULL), so that the compiler's wait counts leave the newer
    // loads in flight; the last slices of a range go through the guarded loads.
    uint32_t ns_full;
    {
        const uint64_t k_full = a.K / 16, first = 2 * g0;                // full slices of the whole K
        ns_full = (uint32_t)(k_full <= first ? 0 : k_full - first < ns ? k_full - first : ns);
        if ((AKN && a.M < 4) || (BKN && a.N < 4)) ns_full = 0;
    }
    f32x4 raw[2][NC], rw[2];                                   // two slices on their way; the weights of the thread's k of these
    auto weights = [&](int u, uint32_t s) {
        if constexpr (WEIGHT) rw[u] = *reinterpret_cast<const f32x4*>(a.weight + g0 * 32 + (uint64_t)s * 16 + 4 * (lane & 3));
    };
    auto at = [&](int i, uint64_t adv) {
        const float* p = base[i] + adv;
        asm volatile("" : "+s"(p));                            // stays a scalar base: no 64-bit lane addresses
        return reinterpret_cast<const unsigned char*>(p) + gofs[i];
    };
    auto fetch_full = [&](int u, uint32_t s) {
        f32x4 (&x)[NC] = raw[u];
        const uint64_t adv = s * step;
        weights(u, s);
#pragma unroll
        for (int i = 0; i < NC; ++i) x[i] = *reinterpret_cast<const f32x4u*>(at(i, adv));
    };
    auto fetch = [&](int u, uint32_t s) {
        f32x4 (&x)[NC] = raw[u];
        if (s < ns_full) { fetch_full(u, s); return; }                                   // uniform
        if (s >= ns) return;                                                             // uniform
        weights(u, s);
        const uint64_t k0 = g0 * 32 + (uint64_t)s * 16;                                  // first k of the slice
        const uint64_t adv = s * step;
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            const float* p = reinterpret_cast<const float*>(at(i, adv));
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                bool ok = k0 + 4 * kq + (kmajor ? i : e) < a.K;
                if (kmajor && narrow) ok = ok && r0 + (gofs[0] / 4 - (ofs_t)(4 * kq) * (ofs_t)ld) + e < rows;
                x[i][e] = ok ? p[e] : 0.0f;
            }
        }
    };
    auto stash = [&](int u, int i, int stage) {
        const f32x4 (&x)[NC] = raw[u];
        unsigned char* st = smem + stage * kStage + wofs[i];
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = kmajor && i < 4 ? x[e][i & 3] : x[i][e];
        if (kmajor && ragged) {                                                          // uniform: edge tile of a ragged width
            const int c = i + shift;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = c == 1 ? x[e][1] : c == 2 ? x[e][2] : c == 3 ? x[e][3] : v[e];
        }
        if constexpr (WEIGHT) {
            if (is_a) {                                                                  // uniform
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] *= rw[u][e];
            }
        }
        u32x2 p0, p1, p2;
        uint32_t q0, q1, q2;
        split3(v[0], v[1], q0, q1, q2);
        p0[0] = q0; p1[0] = q1; p2[0] = q2;
        split3(v[2], v[3], q0, q1, q2);
        p0[1] = q0; p1[1] = q1; p2[1] = q2;
        *reinterpret_cast<u32x2*>(st) = p0;
        *reinterpret_cast<u32x2*>(st + kPlane) = p1;
        *reinterpret_cast<u32x2*>(st + 2 * kPlane) = p2;
    };

    // ---- fragments
    const int fofs = (lane >> 5) * kHalf + (((lane & 31) ^ ((lane >> 5) * 8)) * 16);
    const int a_ofs = fofs + wm * MI * 512, b_ofs = fofs + (TM + wn * NJ * 32) * 16;
    struct FragA { bf16x8 p[3]; };
    struct FragB { bf16x8 p[NJ][3]; };
    auto load_a = [&](FragA& f, int stage, int i) {
#pragma unroll
        for (int q = 0; q < 3; ++q)
            f.p[q] = *reinterpret_cast<const bf16x8*>(smem + stage * kStage + q * kPlane + a_ofs + i * 512);
    };
    auto load_b = [&](FragB& f, int stage) {
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int q = 0; q < 3; ++q)
                f.p[j][q] = *reinterpret_cast<const bf16x8*>(smem + stage * kStage + q * kPlane + b_ofs + j * 512);
    };
    f32x16 acc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
    auto mma = [&](const FragA& fa, const FragB& fb, int i) {
        constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};            // small terms first
#pragma unroll
        for (int t = 0; t < 6; ++t)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa.p[pa[t]], fb.p[j][pb[t]], acc[i][j], 0, 0, 0);
    };

    // ---- pipeline
    fetch(0, 0);
#pragma unroll
    for (int i = 0; i < NC; ++i) stash(0, i, 0);
    fetch(1, 1);
    fetch(0, 2);
    wait_lds();
    f32_barrier();
    FragB fb[2];
    FragA fa[2];
    load_b(fb[0], 0);
    load_a(fa[0], 0, 0);
    auto slice = [&](auto full, int u, uint32_t s) {
        // raw[u ^ 1] holds slice s + 1, whose stage u ^ 1 is free
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int fi = (u * MI + i) & 1;                              // fragment set of this row of tiles
            if (i + 1 < MI) {
                load_a(fa[fi ^ 1], u, i + 1);
                constexpr int per = (NC + MI - 2) / (MI > 1 ? MI - 1 : 1);
#pragma unroll
                for (int q = i * per; q < NC && q < (i + 1) * per; ++q) stash(u ^ 1, q, u ^ 1);
            } else {
                if constexpr (MI == 1) {
#pragma unroll
                    for (int q = 0; q < NC; ++q) stash(u ^ 1, q, u ^ 1);
                }
                if constexpr (decltype(full)::value) fetch_full(u ^ 1, s + 3); else fetch(u ^ 1, s + 3);
                wait_lds();
                f32_barrier();
                load_b(fb[u ^ 1], u ^ 1);
                load_a(fa[fi ^ 1], u ^ 1, 0);
            }
            mma(fa[fi], fb[u], i);
            // Spread the splitting arithmetic and the LDS operations of a slice evenly over its matrix instructions, whose 32
            // cycles each leave room for them; on its own the compiler issues them in blocks of 35 and more while the matrix
            // cores idle (1,024 x 65,536 x 4,096 on 256 x 256 tiles: 2.44 -> 2.25 ms; the 128 x 128 tile gains 2 %).
            constexpr int kValu = MI == 4 ? 4 : 6;
#pragma unroll
            for (int q = 0; q < 6 * NJ; ++q) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);       // one matrix instruction
                __builtin_amdgcn_sched_group_barrier(0x002, kValu, 0);   // vector arithmetic
                __builtin_amdgcn_sched_group_barrier(0x300, 1, 0);       // one LDS read or write
            }
        }
    };
    uint32_t s = 0;
    for (; s + 4 < ns_full; s += 2) {
        slice(std::true_type{}, 0, s);
        slice(std::true_type{}, 1, s + 1);
    }
    for (; s < ns; s += 2) {
        slice(std::false_type{}, 0, s);
        slice(std::false_type{}, 1, s + 1);
    }

    // ---- results.  Element e of a lane: tile row 8(e/4) + 4(lane/32) + e%4, tile column lane%32 (slots: a K-major
    // operand's columns are permuted inside each block of 32).  Sums that are not finite are left for the fp32 matrix
    // instructions below: an operand is infinite or NaN, or operand or sum are too large for the scale of the pieces.
    const int cl = lane & 31;
    auto a_row = [&](int i, int slot) {                        // row of A in slot `slot` of the wavefront's block i
        const int b = wm * MI + i;
        return m0 + b * 32 + (AKN ? 4 * (slot & 7) + ((slot >> 3) ^ (b & 1)) : slot);
    };
    auto row_of = [&](int i, int e) { return a_row(i, 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3)); };
    auto col_of = [&](int j) {
        const int b = wn * NJ + j;
        return n0 + b * 32 + (BKN ? 4 * (cl & 7) + ((cl >> 3) ^ (b & 1)) : cl);
    };
    const bool interior = m0 + TM <= a.M && n0 + TN <= a.N && !a.accumulate;             // uniform
    uint32_t todo[MI * NJ];
    uint32_t any = 0;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const uint64_t col = col_of(j);
            uint32_t bad = 0;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const bool fin = __builtin_isfinite(acc[i][j][e]);
                const float v = acc[i][j][e] * kSplitUnscale;
                const uint64_t row = row_of(i, e);
                float* c = a.C + row * a.ldc + col;
                if (interior) {
                    *c = v;
                    if (!fin) bad |= 1u << e;
                } else if (row < a.M && col < a.N) {
                    if (fin) *c = a.accumulate ? *c + v : v;
                    else bad |= 1u << e;
                }
            }
            todo[i * NJ + j] = bad;
            any |= bad;
        }
    // 32 x 32 blocks with such sums are contracted again with v_mfma_f32_32x32x2_f32, straight from memory, and only those
    // sums replaced.  A lane holds k 4(lane/32)..+3 of every 8 (the order inside a contraction is free).  The loads of 32 k
    // are requested together.  256 x 2,000 x 16,384 with one infinite row of B: 106 -> 176 us, with one in every row 315 us (a
    // loop of one lane per sum: 2,560 and 15,100); 1,000 x 50,001 x 4,096: 2.00 -> 2.06 and 6.99 ms (20.9 and 373).
    if (__builtin_expect(__any(any != 0), 0)) {
        const uint64_t k_end = (g0 + ng) * 32 < a.K ? (g0 + ng) * 32 : a.K;
#pragma unroll 1
        for (int t = 0; t < MI * NJ; ++t) {
            uint32_t bad = 0;
#pragma unroll
            for (int q = 0; q < MI * NJ; ++q) bad = q == t ? todo[q] : bad;
            if (!__any(bad != 0)) continue;                               // uniform
            const int i = t / NJ, j = t % NJ;
            uint64_t row = a_row(i, cl), col = col_of(j);
            row = row < a.M ? row : a.M - 1;                              // past the edge: never stored
            col = col < a.N ? col : a.N - 1;
            const float* pa = AKN ? a.A + row : a.A + row * a.lda;
            const float* pb = BKN ? a.B + col : a.B + col * a.ldb;
            f32x16 sum;
#pragma unroll
            for (int e = 0; e < 16; ++e) sum[e] = 0.0f;
            for (uint64_t k0 = g0 * 32; k0 < k_end; k0 += 32) {
                f32x4 xa[4], xb[4];
                const uint64_t kl = k0 + 4 * (lane >> 5);
                if (k0 + 32 <= k_end) {                                   // uniform
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const uint64_t k = kl + 8 * u;
                        if constexpr (AKN) {
#pragma unroll
                            for (int q = 0; q < 4; ++q) xa[u][q] = pa[(k + q) * a.lda];
                        } else {
                            xa[u] = *reinterpret_cast<const f32x4u*>(pa + k);
                        }
                        if constexpr (BKN) {
#pragma unroll
                            for (int q = 0; q < 4; ++q) xb[u][q] = pb[(k + q) * a.ldb];
                        } else {
                            xb[u] = *reinterpret_cast<const f32x4u*>(pb + k);
                        }
                    }
                } else {
#pragma unroll
                    for (int u = 0; u < 4; ++u)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const uint64_t k = kl + 8 * u + q;
                            xa[u][q] = k < k_end ? pa[AKN ? k * a.lda : k] : 0.0f;
                            xb[u][q] = k < k_end ? pb[BKN ? k * a.ldb : k] : 0.0f;
                        }
                }
                if constexpr (WEIGHT) {
#pragma unroll
                    for (int u = 0; u < 4; ++u)
#pragma unroll
                        for (int q = 0; q < 4; ++q) xa[u][q] *= kl + 8 * u + q < k_end ? a.weight[kl + 8 * u + q] : 0.0f;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        sum = __builtin_amdgcn_mfma_f32_32x32x2f32(xa[u][q], xb[u][q], sum, 0, 0, 0);
            }
#pragma unroll
            for (int e = 0; e < 16; ++e)
                if (bad >> e & 1) {
                    float* c = a.C + row_of(i, e) * a.ldc + col_of(j);
                    *c = a.accumulate ? *c + sum[e] : sum[e];
                }
        }
    }
}

}  // namespace grass
