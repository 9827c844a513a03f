// Batched exact demapping, FP32 direct differences: a workgroup's part of the list of a plan's FP32
// instances (gfx950).  Work lists, claims and GMI / MI partial sums as in demap_batched.hip; one
// lane per symbol, the body of valu_body.hpp with the coordinates rounded up to 2, 4 or 8 (zeros past
// D; the tables' row stride is 8) and M = 2 .. 64 at compile time.  Padding every instance to 16
// points of 8 coordinates, as one body for all shapes had to, made an 8-QAM symbol five times as long
// (the shaping search's launches of 2^21 symbols: 72 us, now 33).  The twenty-one bodies' loop
// invariants do not all fit the scalar registers: some 20 of the 128 vector registers spill, outside
// the point loops.
#pragma once
#include "device_common.hpp"
#include "kernels.hpp"
#include "valu_body.hpp"
#include "wave_reduce.hpp"

namespace dm {

constexpr int kBatchThreads = 1024;

// Symbols [n0, n0 + len) of one instance; the GMI / MI terms of the lane's symbols are added to gl, ml.
template <int DP, int MC>
__device__ __forceinline__ void valu_item(const float* lds, const BlockView& b, const Sinks& k, uint32_t* fill,
                                          int64_t n0, int len, double& gl, double& ml,
                                          uint32_t& pairs) {
    const int D = b.D, M = MC ? MC : b.M;
    const int Mpad = MC ? MC : M < 16 ? 16 : M;
    float y_nx[DP];
    uint32_t row_nx = 0;
    auto fetch = [&](int64_t n) {
        const size_t nc = (size_t)(n < b.N ? n : 0);
        const float* src = b.y + nc * D;
#pragma unroll
        for (int d = 0; d < DP; ++d) y_nx[d] = src[min(d, D - 1)];
        if (b.tx) row_nx = b.tx[nc];
    };
    fetch(n0 + threadIdx.x);
    for (int o = threadIdx.x; o < len; o += kBatchThreads) {
        const int64_t n = n0 + o;
        const bool active = n < b.N;
        float y[DP];
#pragma unroll
        for (int d = 0; d < DP; ++d) y[d] = active && d < D ? y_nx[d] : 0.0f;
        uint32_t row = row_nx;
        if (o + kBatchThreads < len) fetch(n + kBatchThreads);
        int txl = 0;
        if (b.tx && active) {
            if (row >= (uint32_t)M) {  // out-of-range row: clamped and reported
                if (k.bad_tx) atomicOr(k.bad_tx, 1u);
                row = 0;
            }
            txl = (int)b.row2label[row];
        }
        ValuSums<MC> S;
        S.init();
        ValuHigh H0, H1;
        if constexpr (MC == 0) {
            H0.init();
            H1.init();
        }
        valu_accumulate<DP, 8, MC>((LdsTable)lds, 0, Mpad, y, b.c, b.K, b.m, S, H0, H1);
        float g, mi;
        double gc = 0.0, mc = 0.0;
        valu_epilogue<DP, 8, MC>(b, k, fill, n, active, y, S, H0, H1, txl, lds + txl * 8, (LdsTable)lds, g, mi, gc, mc,
                                 pairs);
        if (active) {
            gl += (double)g + gc;
            ml += (double)mi + mc;
        }
    }
}

template <int DP>
__device__ __forceinline__ void valu_item_m(const float* lds, const BlockView& b, const Sinks& k, uint32_t* fill,
                                            int64_t n0, int len, double& gl, double& ml, uint32_t& pairs) {
    switch (b.M) {  // uniform
        case 2: valu_item<DP, 2>(lds, b, k, fill, n0, len, gl, ml, pairs); break;
        case 4: valu_item<DP, 4>(lds, b, k, fill, n0, len, gl, ml, pairs); break;
        case 8: valu_item<DP, 8>(lds, b, k, fill, n0, len, gl, ml, pairs); break;
        case 16: valu_item<DP, 16>(lds, b, k, fill, n0, len, gl, ml, pairs); break;
        case 32: valu_item<DP, 32>(lds, b, k, fill, n0, len, gl, ml, pairs); break;
        case 64: valu_item<DP, 64>(lds, b, k, fill, n0, len, gl, ml, pairs); break;
        default: valu_item<DP, 0>(lds, b, k, fill, n0, len, gl, ml, pairs); break;
    }
}

// A workgroup of the FP32 list.
__device__ __forceinline__ void batched_valu(const BatchArgs& a, float* lds) {
    __shared__ int s_claim;      // first item of this claim
    __shared__ uint32_t s_fill;  // entries in this block's fix-up queue region
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave_slot = (blockIdx.x * (kBatchThreads / 64) + (tid >> 6)) % kAccSlots;
    const Sinks& k = a.sinks;
    if (tid == 0) s_fill = 0u;
    int staged = -1;
    for (;;) {
        // (asked for when the last claim is done, see demap_batched.hip)
        if (tid == 0) s_claim = (int)atomicAdd(a.next, (uint32_t)a.grab);
        __syncthreads();
        const int i0 = __builtin_amdgcn_readfirstlane(s_claim);
        if (i0 >= a.n_items) break;
        const int i1 = min(i0 + a.grab, a.n_items);
        for (int i = i0; i < i1;) {
            // a run of items of one instance, GMI / MI terms summed per lane, then over the wave once
            const WorkItem it = uniform_copy(a.items[i]);
            const BatchDesc d = uniform_desc(a.desc[it.inst]);
            const BlockView& b = d.view;
            i += it.run;
            if (it.inst != staged) {  // restage the point table (whole block, uniform condition)
                __syncthreads();
                const int Mpad = b.M < 16 ? 16 : b.M;
                for (int j = tid; j < Mpad * 8; j += kBatchThreads)
                    lds[j] = (j < b.M * 8) ? b.table[j] : 1.0e19f;  // padding rows: e_j = 0
                __syncthreads();
                staged = it.inst;
            }
            const int len = it.run * d.sub * kBatchThreads;
            double gl = 0.0, ml = 0.0;
            uint32_t pairs = 0;
            if (b.D <= 2) valu_item_m<2>(lds, b, k, &s_fill, it.n0, len, gl, ml, pairs);
            else if (b.D <= 4) valu_item_m<4>(lds, b, k, &s_fill, it.n0, len, gl, ml, pairs);
            else valu_item_m<8>(lds, b, k, &s_fill, it.n0, len, gl, ml, pairs);
            pairs = wave_sum_u32(pairs);
            if (lane == 0 && pairs && k.fix_pairs) atomicAdd(k.fix_pairs + it.inst, pairs);
            if (k.acc) {
                gl = wave_sum(gl);
                ml = wave_sum(ml);
                if (lane == 0) {
                    acc_add(k.acc, it.inst, wave_slot, 0, gl);
                    acc_add(k.acc, it.inst, wave_slot, 1, ml);
                }
            }
        }
        __syncthreads();  // the claim is read before the next overwrites it
    }
    queue_close(k, &s_fill);
}

}  // namespace dm
