// Per-symbol body of the FP32 direct-difference demapper (one lane = one symbol).
//
// For every point j the lane forms e_j = 2^(K - c ||y - x_j||^2), c = log2(e)/(2 sigma2): the
// likelihood exp(-||y-x||^2/(2 sigma2)) rescaled by the fixed factor 2^K, so no running maximum
// is needed (e_j <= 2^K because ||y-x||^2 >= 0, and K = 123 - m keeps the sum of M terms below
// 2^123).  The per-bit subset sums S_p^0, S_p^1 come from accumulators indexed by the label's
// low bits (table in label order):
//   bits 0-3: accA[j & 15] (one add per point); group sum T over 16 points (one add);
//   bits 4-5: accB[(j >> 4) & 3] (one add per 16 points);
//   bits >= 6: the 64-point block sum added to the side given by (j >> 6).
// A subset sum under 2^(m-102) may have lost terms below FP32's normal range (v_exp_f32 flushes
// results under 2^-126); such (symbol, bit) pairs are queued for an exact recomputation.
//
// MC is the constellation's size where that is known at compile time (2 .. 256), else 0 (any M).
// With it the loops are unrolled over exactly M points (not padded to 16), the group sums that no
// label bit needs are not formed, the epilogue handles exactly m bits, and the LLRs go out in
// wide stores: for few points per symbol the epilogue, not the exponentials, is the work.
//
// What bounds the point loop: vector issue.  On MI355X an FP32 add or FMA takes 0.88 ns per wave and
// SIMD alone and about 1.3 with exponentials among them, v_exp_f32 3.6 alone and about 8 among FMAs
// (probes of the mixtures); 12 instructions per point at D = 4 measure 18-20 ns.  A 16-byte
// broadcast read from LDS takes 8 cycles of the CU whatever the lanes share, so points read from LDS
// once per symbol and lane come close to that (D = 4: 128 of 177 cycles); tables of up to 8 KiB are
// read through the scalar cache instead, into scalar registers that the subtractions take as they
// are.
#pragma once
#include <type_traits>

#include "device_common.hpp"
#include "fixup_queue.hpp"

namespace dm {

// Label bits of an MC-point constellation (MC == 0: up to 16, known at run time).
constexpr int valu_log2(int v) { return v <= 1 ? 0 : 1 + valu_log2(v / 2); }
constexpr int valu_bits(int mc) { return mc == 0 ? 16 : valu_log2(mc); }

template <int MC>
struct ValuSums {
    static constexpr int R = MC == 0 || MC >= 16 ? 16 : MC;   // accA entries in use
    static constexpr int Q = MC == 0 || MC >= 64 ? 4 : MC / 16;  // accB entries in use
    float accA[16], accB[4];
    __device__ __forceinline__ void init() {
#pragma unroll
        for (int i = 0; i < 16; ++i) accA[i] = 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i) accB[i] = 0.0f;
    }
};

// Sums of one side of label bits 6 and up.  The two sides are objects of their own: as arrays of
// one struct the compiler picks the side by a run-time address, which puts them in scratch memory.
struct ValuHigh {
    float s[10];
    __device__ __forceinline__ void init() {
#pragma unroll
        for (int i = 0; i < 10; ++i) s[i] = 0.0f;
    }
};

// Where the points are read from: LDS (16-byte aligned, all lanes the same address: broadcast), or the
// table itself in constant address space (scalar loads).  Both say so in their type: a generic pointer
// that passes an asm statement is read with flat loads.
typedef const __attribute__((address_space(3))) float* LdsTable;
typedef const __attribute__((address_space(4))) float* ScalarTable;

// G points of the label-ordered table (row stride LS), read as wide as the stride allows.
template <int DP, int LS, int G>
struct ValuPoints {
    float x[G][DP];
    __device__ __forceinline__ void load(LdsTable p) {
        constexpr int W = DP % 4 == 0 && LS % 4 == 0 ? 4 : DP % 2 == 0 && LS % 2 == 0 ? 2 : 1;
        typedef float vec __attribute__((ext_vector_type(W)));
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int d = 0; d < DP; d += W) {
                const vec v = *(const __attribute__((address_space(3))) vec*)(p + g * LS + d);
                if constexpr (W == 1) x[g][d] = v[0];
                else
#pragma unroll
                    for (int w = 0; w < W; ++w) x[g][d + w] = v[w];
            }
    }
    __device__ __forceinline__ void load(ScalarTable p) {
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int d = 0; d < DP; ++d) x[g][d] = p[g * LS + d];
    }
};

// e_j of R consecutive points into e, G points at a time, the next G read while the current ones
// are evaluated.
template <int DP, int LS, int R, typename Table>
__device__ __forceinline__ void valu_terms(Table xg, const float (&y)[DP], float c, float K, float (&e)[R]) {
    // (G DP <= 16: two sets of points stay under 32 registers; at least one point)
    constexpr int G0 = DP <= 4 ? 4 : DP <= 8 ? 2 : 1, G = R < G0 ? R : G0;
    ValuPoints<DP, LS, G> p[2];
    p[0].load(xg);
#pragma unroll
    for (int r = 0; r < R; r += G) {
        if (r + G < R) p[(r / G + 1) & 1].load(xg + (r + G) * LS);
#pragma unroll
        for (int g = 0; g < G; ++g) e[r + g] = hw_exp2(fmaf(-c, sqdist<DP>(y, p[(r / G) & 1].x[g]), K));
    }
}

// Accumulate the points [c0, c0 + cnt) of the label-ordered table `tab` with row stride LS >= DP.
// MC != 0: the whole table (c0 = 0, cnt = MC).  MC == 0: cnt a multiple of 16, c0 of 64.
template <int DP, int LS, int MC, typename Table>
__device__ __forceinline__ void valu_accumulate(Table tab, int c0, int cnt, const float (&y)[DP], float c,
                                                float K, int m, ValuSums<MC>& S, ValuHigh& H0, ValuHigh& H1) {
    constexpr int R = ValuSums<MC>::R;
    if constexpr (MC != 0) {
        constexpr int NB = MC > 64 ? MC / 64 : 1, NQ = MC > 64 ? 4 : (MC + 15) / 16;  // blocks, groups per block
        if constexpr (MC > 64) {
            S.init();
            H0.init();
            H1.init();
        }
#pragma unroll 1
        for (int blk = 0; blk < NB; ++blk) {
            float bt = 0.0f;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                // A table of up to 32 floats may stay in registers across symbols; a larger one is
                // read 16 points at a time (the compiler would otherwise hoist every read out of
                // the symbol loop, or to its top, and spill).
                Table t = tab + (blk * 64 + q * 16) * LS;
                if constexpr (MC * DP > 32 && std::is_same<Table, ScalarTable>::value) asm volatile("" : "+s"(t));
                float e[R], T = 0.0f;
                valu_terms<DP, LS, R>(t, y, c, K, e);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    S.accA[r] = MC <= 64 && q == 0 ? e[r] : S.accA[r] + e[r];
                    T = r == 0 ? e[r] : T + e[r];
                }
                if constexpr (MC * DP > 32) asm volatile("" : "+v"(T)::"memory");
                if constexpr (MC > 16) S.accB[q] = MC <= 64 ? T : S.accB[q] + T;
                bt += T;
            }
            if constexpr (MC > 64) {
#pragma unroll
                for (int p = 6; p < valu_bits(MC); ++p) {
                    const bool one = (blk >> (p - 6)) & 1;
                    H1.s[p - 6] += one ? bt : 0.0f;
                    H0.s[p - 6] += one ? 0.0f : bt;
                }
            }
        }
    } else {
        for (int b0 = 0; b0 < cnt; b0 += 64) {
            float bt = 0.0f;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (b0 + q * 16 < cnt) {
                    float e[16], T = 0.0f;
                    valu_terms<DP, LS, 16>(tab + (b0 + q * 16) * LS, y, c, K, e);
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        S.accA[r] += e[r];
                        T += e[r];
                    }
                    S.accB[q] += T;
                    bt += T;
                }
            }
            const int blk = (c0 + b0) >> 6;
#pragma unroll
            for (int p = 6; p < 16; ++p) {
                if (p < m) {
                    const bool one = (blk >> (p - 6)) & 1;
                    H1.s[p - 6] += one ? bt : 0.0f;
                    H0.s[p - 6] += one ? 0.0f : bt;
                }
            }
        }
    }
}

// Constellations of up to 16 points recompute their flagged bits in the wave when at least this many
// lanes have one: at high SNR nearly all do (DP-QPSK and 4-QAM beyond 20 dB), and an entry and a
// recomputation from the queue then cost more than the symbol itself; fewer lanes are better
// collected in the queue, where they share full waves.  4-QAM, 6 x 742567 symbols up to 22 dB: 67 us
// and 174 us in the fix-up with the queue alone, 134 and 10 with this; from 12 to 22 dB with LLRs now
// 262 and 8.6.
constexpr int kInPlaceLanes = 8;

// Per-bit subset sums -> LLRs, flags, GMI and MI terms of one symbol; queues flagged bits, or (MC <= 16)
// recomputes them at once, their (symbol, bit) pairs added to pairs and their GMI / MI terms to gc,
// mc.  txl: the transmitted label (0 without tx); xtx: its point; LS: row stride of tab and b.table.
template <int DP, int LS, int MC, typename Table>
__device__ __forceinline__ void valu_epilogue(const BlockView& b, const Sinks& k, uint32_t* fill, int64_t n, bool active,
                                              const float (&y)[DP], const ValuSums<MC>& S,
                                              const ValuHigh& H0, const ValuHigh& H1, int txl, const float* xtx,
                                              Table tab, float& g, float& mi, double& gc, double& mc,
                                              uint32_t& pairs) {
    constexpr int MB = valu_bits(MC);
    const int m = MC ? MB : b.m;
    float stot = 0.0f;
#pragma unroll
    for (int r = 0; r < ValuSums<MC>::R; ++r) stot += S.accA[r];
    g = 0.0f;
    mi = 0.0f;
    uint32_t mask = 0;
    [[maybe_unused]] float Lv[MC ? MB : 1];
    float* const out = b.llr && active ? b.llr + (size_t)n * m : nullptr;
    auto bit_of = [&](int p, float s0, float s1) {
        const bool flagged = !(fminf(s0, s1) >= b.flag_thresh);
        const float L = log2_ratio(s1, s0);
        const int bit = (txl >> p) & 1;
        // a flagged bit without LLR output, |L| >= 60 and the transmitted bit on the near side: its
        // GMI term is 1 in FP64
        const bool sure = flagged && !b.want_llr && fmaxf(s0, s1) >= b.near_thresh && (bit ? s1 > s0 : s0 > s1);
        if (b.tx) {
            const float gb = gmi_bit_term(L, bit);
            g += flagged ? (sure ? 1.0f : 0.0f) : gb;
        }
        mask |= flagged && !sure ? flag_bits(p, s0, s1) : 0u;
        // LLRs (a flagged bit's is overwritten by the fix-up): bit p is column m - 1 - p
        if constexpr (MC != 0) Lv[p] = L * 0.69314718055994531f;
        else if (out) out[m - 1 - p] = L * 0.69314718055994531f;
    };
#pragma unroll
    for (int p = 0; p < (MB < 4 ? MB : 4); ++p) {
        if (p < m) {
            float s0 = 0.0f, s1 = 0.0f;
#pragma unroll
            for (int r = 0; r < ValuSums<MC>::R; ++r) {
                if ((r >> p) & 1) s1 += S.accA[r];
                else s0 += S.accA[r];
            }
            bit_of(p, s0, s1);
        }
    }
#pragma unroll
    for (int p = 4; p < (MB < 6 ? MB : 6); ++p) {
        if (p < m) {
            float s0 = 0.0f, s1 = 0.0f;
#pragma unroll
            for (int q = 0; q < ValuSums<MC>::Q; ++q) {
                if ((q >> (p - 4)) & 1) s1 += S.accB[q];
                else s0 += S.accB[q];
            }
            bit_of(p, s0, s1);
        }
    }
    if constexpr (MB > 6) {
#pragma unroll
        for (int p = 6; p < MB; ++p)
            if (p < m) bit_of(p, H0.s[p - 6], H1.s[p - 6]);
    }
    if (b.tx) {
        if (stot >= b.flag_thresh) {
            const float ttx = fmaf(-b.c, sqdist<DP>(y, xtx), b.K);
            const int e = __builtin_amdgcn_frexp_expf(stot);
            const float mant = __builtin_amdgcn_frexp_mantf(stot);
            // m - log2(stot) + t_tx, with log2(stot) = e + log2(mant) split off exactly
            mi = ((float)(m - e) + ttx) - hw_log2(mant);
        } else {
            mask |= kMiFlag;
        }
    }
    if constexpr (MC != 0 && MC <= 16) {
        const bool fix = mask != 0u && active;
        if (__builtin_popcountll(__ballot(fix)) >= kInPlaceLanes && fix) {
            two_pass_symbol<DP, LS, MC>(
                b, tab, y, mask, txl, xtx, [&](int p, float L) { Lv[p] = L * 0.69314718055994531f; }, gc, mc);
            pairs += (uint32_t)__popc(mask & 0xFFFFu);
            mask = 0u;
        }
    }
    if constexpr (MC != 0)
        if (out) {
#pragma unroll
            for (int j = 0; j < MB; ++j) out[j] = Lv[MB - 1 - j];
        }
    // (sizes that are not known here but at D = 1, 2, 4, 8 have more than 64 points)
    constexpr bool kWide = DP <= 8 && (MC ? MC >= 32 && MC <= kFixLaneMaxM : DP == 3 || DP > 4 && DP < 8);
    if (mask && active) queue_or_fix<DP, LS, kWide>(b, k, fill, (uint32_t)n, mask, near_word(stot, m, false), gc, mc);
}

}  // namespace dm
