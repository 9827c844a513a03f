// The fix-up's side of the demapping kernels (gfx950): appending flagged symbols to the queue, the
// recomputation in place of a symbol that finds its region full, and the recomputation in one lane, which
// the queue's drain uses too.
//
// A symbol's recomputed LLRs must not depend on what else is in the call: how many symbols of its wave are
// flagged, how many are queued, whether a region is full.  So each table size has one arithmetic, wherever
// it runs: 2 .. 16 points (and more than 8 dimensions) two passes per flagged bit, 32 and 64 points one
// pass for all bits.  From 128 points on the drain works with several lanes per symbol, and only a
// symbol that finds its region full takes the two passes in one lane.
#pragma once
#include "device_common.hpp"
#include "wide_sums.hpp"

namespace dm {

constexpr int kFixLaneMaxM = 64;  // up to here the drain takes one lane per symbol

// The flagged bits and the MI term of one symbol of MC <= 16 points in one lane, exponents in registers: the
// arithmetic of fixup_one, bit for bit.  put(p, L) takes the log2-unit LLR of bit p; the GMI and MI terms
// are added to g and mi.  LS: row stride of tab; xtx: the transmitted label's point.
template <int DP, int LS, int MC, typename Table, typename Put>
__device__ __forceinline__ void two_pass_symbol(const BlockView& b, Table tab, const float (&y)[DP], uint32_t mask,
                                                int txl, const float* xtx, Put put, double& g, double& mi) {
    constexpr int MB = MC == 2 ? 1 : MC == 4 ? 2 : MC == 8 ? 3 : 4;
    static_assert(MC == 1 << MB, "2 to 16 points");
    float t[MC];
#pragma unroll
    for (int j = 0; j < MC; ++j) {
        float x[DP];
#pragma unroll
        for (int d = 0; d < DP; ++d) x[d] = tab[j * LS + d];
        t[j] = fmaf(-b.c, sqdist<DP>(y, x), b.K);
    }
#pragma unroll
    for (int p = 0; p < MB; ++p) {
        if (!((mask >> p) & 1u)) continue;
        float mx0 = -INFINITY, mx1 = -INFINITY, s0 = 0.0f, s1 = 0.0f;
#pragma unroll
        for (int j = 0; j < MC; ++j) {
            if ((j >> p) & 1) mx1 = fmaxf(mx1, t[j]);
            else mx0 = fmaxf(mx0, t[j]);
        }
#pragma unroll
        for (int j = 0; j < MC; ++j) {
            if ((j >> p) & 1) s1 += hw_exp2(t[j] - mx1);
            else s0 += hw_exp2(t[j] - mx0);
        }
        const float L = (mx1 - mx0) + (hw_log2(s1) - hw_log2(s0));
        put(p, L);
        if (b.tx) g += (double)finite_term(gmi_bit_term(L, (txl >> p) & 1));
    }
    if ((mask & kMiFlag) && b.tx) {
        float mx = -INFINITY, s = 0.0f;
#pragma unroll
        for (int j = 0; j < MC; ++j) mx = fmaxf(mx, t[j]);
#pragma unroll
        for (int j = 0; j < MC; ++j) s += hw_exp2(t[j] - mx);
        const float ttx = fmaf(-b.c, sqdist<DP>(y, xtx), b.K);
        mi += (double)finite_term((float)MB - ((mx - ttx) + hw_log2(s)));
    }
}

// The same for 32 and 64 points: one pass over the points for all bits.  Returns the mask of what is out of
// the wide range, for the form under maxima.  Against two passes per flagged bit (fixup_one): 2^20
// symbols of 64-QAM at 18 dB 29.2 -> 7.6 us, 4096 of them at 20 dB 29.9 -> 7.2; 8 x 2^20 symbols from 6
// to 20 dB 93 -> 27; 64 mixed instances of 2^14 .. 2^22 symbols 153 -> 76.  Bound by vector issue.
template <int DP, int LS, typename Table, typename Put>
__device__ __forceinline__ uint32_t wide_symbol(const BlockView& b, Table tab, const float (&y)[DP], uint32_t mask,
                                                int txl, const float* xtx, Put put, double& g, double& mi) {
    double accA[16], z4 = 0.0, o4 = 0.0, z5 = 0.0, o5 = 0.0;
#pragma unroll
    for (int r = 0; r < 16; ++r) accA[r] = 0.0;
    const int groups = b.M >> 4;
#pragma unroll 1
    for (int q = 0; q < groups; ++q) {
        double T = 0.0;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            float x[DP];
#pragma unroll
            for (int d = 0; d < DP; ++d) x[d] = tab[(q * 16 + r) * LS + d];
            const double w = wide_exp2(fmaf(-b.c, sqdist<DP>(y, x), b.K));
            accA[r] += w;
            T += w;
        }
        if (q & 1) o4 += T;
        else z4 += T;
        if (q & 2) o5 += T;
        else z5 += T;
    }
    uint32_t left = 0u;
    auto finish = [&](int p, double s0, double s1) {
        if (!((mask >> p) & 1u)) return;
        if (!wide_ok(s0, s1)) {
            left |= 1u << p;
            return;
        }
        const float L = wide_log2_ratio(s1, s0);
        put(p, L);
        if (b.tx) g += (double)gmi_bit_term(L, (txl >> p) & 1);
    };
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        double s0 = 0.0, s1 = 0.0;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            if ((r >> p) & 1) s1 += accA[r];
            else s0 += accA[r];
        }
        finish(p, s0, s1);
    }
    finish(4, z4, o4);
    finish(5, z5, o5);
    if ((mask & kMiFlag) && b.tx) {
        const double all = z4 + o4;
        if (wide_ok(all, all)) mi += (double)wide_mi(b.m, all, fmaf(-b.c, sqdist<DP>(y, xtx), b.K));
        else left |= kMiFlag;
    }
    return left;
}

// The flagged bits and MI term of one symbol in one lane, for the symbols that find their region full.
// WIDE: the table may have 32 or 64 points (and D <= 8).  Their results are those of wide_symbol, the same
// numbers added in the same order, but in two walks over the points, which need half of its
// registers: with the sixteen running sums the demapping kernels would spill.
template <int DP, int LS, bool WIDE>
__device__ void fixup_in_place(const BlockView& b, const Sinks& k, uint32_t n, uint32_t mask, double& gcorr,
                               double& mcorr) {
    if constexpr (WIDE) {
        if (b.M == 32 || b.M == 64) {
            float y[DP];
            load_symbol<DP>(y, b.y + (size_t)n * b.D, b.D, true);
            const int txl = b.tx ? tx_label(b, k, n) : 0, groups = b.M >> 4;
            const float* const tab = as_global(b.table);
            auto term = [&](int j) { return wide_exp2(fmaf(-b.c, sqdist<DP>(y, tab + (size_t)j * LS), b.K)); };
            uint32_t left = 0u;
            auto finish = [&](int p, double s0, double s1) {
                if (!((mask >> p) & 1u)) return;
                if (!wide_ok(s0, s1)) {
                    left |= 1u << p;
                    return;
                }
                const float L = wide_log2_ratio(s1, s0);
                if (b.llr) b.llr[(size_t)n * b.m + (b.m - 1 - p)] = L * 0.69314718055994531f;
                if (b.tx) gcorr += (double)gmi_bit_term(L, (txl >> p) & 1);
            };
            // half 0: bits 0 .. 3, by index within 16 points; half 1: bits 4 and 5, by group of 16
#pragma unroll 1
            for (int half = 0; half < 2; ++half) {
                const int outer = half ? groups : 16, inner = half ? 16 : groups, so = half ? 16 : 1, si = half ? 1 : 16;
                double s0[4], s1[4];
#pragma unroll
                for (int p = 0; p < 4; ++p) s0[p] = s1[p] = 0.0;
#pragma unroll 1
                for (int o = 0; o < outer; ++o) {
                    double a = 0.0;
#pragma unroll 2
                    for (int i = 0; i < inner; ++i) a += term(o * so + i * si);
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        const bool one = (o >> p) & 1;
                        s1[p] += one ? a : 0.0;
                        s0[p] += one ? 0.0 : a;
                    }
                }
#pragma unroll
                for (int p = 0; p < 4; ++p)
                    if (!half || p < 2) finish(4 * half + p, s0[p], s1[p]);
                if (half && (mask & kMiFlag) && b.tx) {
                    const double all = s0[0] + s1[0];
                    if (wide_ok(all, all)) {
                        const float ttx = fmaf(-b.c, sqdist<DP>(y, b.table + (size_t)txl * LS), b.K);
                        mcorr += (double)wide_mi(b.m, all, ttx);
                    } else {
                        left |= kMiFlag;
                    }
                }
            }
            if (left == 0u) return;
            mask = left;
        }
    }
    fixup_one<DP, LS>(b, k, b.table, n, mask, gcorr, mcorr);
}

// Queue a symbol for the fix-up (near: FixEntry.near of the symbol) in the workgroup's region, whose
// fill is counted in LDS at *fill; when the region is full the calling lane recomputes the
// symbol in place (slow but exact), counts its pairs, and the corrections come back through
// gc / mc.  Queued pairs are counted by the fix-up when it drains them.  LS: row stride of the block's
// table; WIDE: as for fixup_in_place.
template <int DP, int LS, bool WIDE>
__device__ __forceinline__ void queue_or_fix(const BlockView& b, const Sinks& k, uint32_t* fill, uint32_t n,
                                             uint32_t mask, uint32_t near, double& gc, double& mc) {
    const uint32_t slot = atomicAdd(fill, 1u);
    // (the long form is marked unlikely, which keeps it from the registers of the kernels of D = 3, 5, 6, 7; the
    // short one not: with it 8 points of 2D take a 65th register)
    if (WIDE ? __builtin_expect(slot < k.queue_seg, 1) : slot < k.queue_seg) {
        k.queue[(size_t)blockIdx.x * k.queue_seg + slot] = FixEntry{n, (uint32_t)b.tag, mask, near};
    } else {
        if (k.fix_pairs) atomicAdd(k.fix_pairs + b.tag, (uint32_t)__popc(mask & 0xFFFFu));
        fixup_in_place<DP, LS, WIDE>(b, k, n, mask, gc, mc);
    }
}

// Store the workgroup's region count; every thread calls it once, after its last queue_or_fix.
__device__ __forceinline__ void queue_close(const Sinks& k, const uint32_t* fill) {
    __syncthreads();
    if (threadIdx.x == 0) k.queue_count[blockIdx.x] = min(*fill, k.queue_seg);
}

}  // namespace dm
