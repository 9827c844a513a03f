// Exact soft demapper for constellations of 32 to 256 points (one to eight 32-point tiles) with
// the distance cross term on MFMA (gfx950): the multi-SNR launch over one constellation with the
// tile count fixed at compile time (tile loop and subset sums in mfma_small.hpp, epilogue in
// mfma_body.hpp).  The whole operand table (at most 8 tiles x 2 MFMAs x 1 KiB), the FP32 points
// (at most 8 KiB) and the row-to-label map are staged in LDS once per block, so that the
// transmitted label and its point, read once per symbol, cost LDS rather than global-memory
// latency.  With split FP16 operands the MI term takes the transmitted point's exponent from the
// direct FP32 differences (a few VALU instructions) instead of a diagonal MFMA product and a
// register select; the other precisions keep the diagonal product (their per-label operand
// rows are staged too).
#include <type_traits>

#include "device_common.hpp"
#include "kernels.hpp"
#include "mfma_body.hpp"
#include "mfma_small.hpp"

namespace dm {

namespace {

// Most threads per block.  A wave takes 64 symbols, one per lane, through the tile loop 32 at a time: what
// is done once per symbol (operand splitting, flags, MI term, FP64 sums, loads) then fills the lanes
// instead of running in both halves, and half the vector instructions of an 8-tile batch were outside
// its tile loop.  The first half's sums wait in registers, so 256 points take 160 of them per lane:
// three waves per SIMD (at four, 18 registers spilled and a third of the gain was lost); fewer points
// fit four.  Measured, DP-16QAM, 8 x 2^20 symbols: split FP16 497 -> 458 us (four waves: 478), split
// BF16 513 -> 480 us; 64-QAM split FP16 226 -> 183 us.
constexpr int kThreads = 256;

template <typename T, int D, bool SPLIT, int NT>
__global__ __launch_bounds__(kThreads, NT == 8 ? 3 : 4) void demap_mfma_small_kernel(const LaunchArgs a, const uint4* __restrict__ frag,
                                                                    const uint16_t* __restrict__ pv) {
    constexpr int S = Slots<D, SPLIT>::S;
    constexpr int MB = SmallBits<NT>::MB;  // label bits of the constellation
    __shared__ uint4 lds_frag[NT * S * 64];     // [tile][s][lane] x 16 bytes
    __shared__ float lds_tab[NT * 32 * D];      // FP32 points in label order
    // the transmitted point's MI exponent from FP32 differences only with split FP16 operands
    constexpr bool kDirectTx = SPLIT && std::is_same<T, _Float16>::value;
    __shared__ uint4 lds_pv[kDirectTx ? 1 : NT * 32 * 2 * S];  // [label][16 S halves]
    __shared__ uint16_t lds_r2l[NT * 32];       // row -> label
    __shared__ uint32_t s_fill;                 // entries in this block's fix-up queue region
    const int tid = threadIdx.x, threads = blockDim.x;
    if (tid == 0) s_fill = 0u;
    const int lane = tid & 63;
    const int wave_slot = (blockIdx.x * (threads >> 6) + (tid >> 6)) % kAccSlots;
    const Sinks& k = a.sinks;
    for (int i = tid; i < NT * S * 64; i += threads) lds_frag[i] = frag[i];
    for (int i = tid; i < NT * 32 * D; i += threads) lds_tab[i] = a.table[i];
    if constexpr (!kDirectTx)
        for (int i = tid; i < NT * 32 * 2 * S; i += threads) lds_pv[i] = reinterpret_cast<const uint4*>(pv)[i];
    for (int i = tid; i < NT * 32; i += threads) lds_r2l[i] = a.row2label[i];
    __syncthreads();

    const int64_t sym_per_blk = threads;
    const int64_t blks_per_snr = (a.N + sym_per_blk - 1) / sym_per_blk;
    const int64_t total = blks_per_snr * a.n_snr;
    double gsum = 0.0, msum = 0.0;
    int cur = -1;
    auto flush = [&]() {
        const double gw = wave_sum(gsum), mw = wave_sum(msum);
        if (lane == 0) {
            acc_add(k.acc, cur, wave_slot, 0, gw);
            acc_add(k.acc, cur, wave_slot, 1, mw);
        }
    };
    int s_idx = (int)(blockIdx.x / blks_per_snr);
    int64_t r = blockIdx.x - (int64_t)s_idx * blks_per_snr;
    // The received symbols and transmitted rows of the next batch are loaded one batch ahead:
    // their latency overlaps the current batch's tile loops and epilogue.
    auto fetch = [&](int s, int64_t rr, float (&yy)[D], uint32_t& row) {
        const int64_t n = rr * sym_per_blk + tid;
        const bool act = n < a.N;
        const float* yrow = a.snr[s].y + (size_t)(act ? n : 0) * D;
#pragma unroll
        for (int d = 0; d < D; ++d) yy[d] = yrow[d];
        row = (a.tx && act) ? (uint32_t)a.tx[n] : 0u;
    };
    float y_nx[D];
    uint32_t row_nx = 0;
    if ((int64_t)blockIdx.x < total) fetch(s_idx, r, y_nx, row_nx);
    for (int64_t bt = blockIdx.x; bt < total; bt += gridDim.x) {
        const int64_t n = r * sym_per_blk + tid;
        if (s_idx != cur) {
            if (cur >= 0 && k.acc) flush();
            gsum = msum = 0.0;
            cur = s_idx;
        }
        const bool active = n < a.N;
        const BlockView b = view_sym(a, s_idx, n, active);
        float y[D];
#pragma unroll
        for (int d = 0; d < D; ++d) y[d] = active ? y_nx[d] : 0.0f;
        uint32_t row = row_nx;
        // next batch: advance (s_idx, r) and issue its loads
        r += gridDim.x;
        while (r >= blks_per_snr) {
            r -= blks_per_snr;
            ++s_idx;
        }
        if (bt + gridDim.x < total) fetch(s_idx, r, y_nx, row_nx);
        int txl = 0;
        if (b.tx && active) {
            if (row >= (uint32_t)b.M) {  // out-of-range row: clamped and reported
                if (k.bad_tx) atomicOr(k.bad_tx, 1u);
                row = 0;
            }
            txl = (int)lds_r2l[row];
        }
        PairSums<MB> P;
        bool bad = false;
        float ttx = 0.0f;
        {
            Frags<T, S> f0, f1;
            build_pair_frags<T, D, SPLIT>(y, b.c, b.K, f0, f1, bad);
            mfma_pair_sums<T, D, SPLIT, NT>(lds_frag, lane, f0, f1, P);
            if constexpr (!kDirectTx)
                if (b.tx) ttx = pair_diagonal<T, D, SPLIT>(reinterpret_cast<const uint16_t*>(lds_pv), f0, f1, txl, lane);
        }
        // The MI term's exponent of the transmitted point: with split FP16 operands from the
        // direct FP32 differences (the MFMA exponents carry ~1e-6 of rounding, which then stays
        // in the MI term instead of cancelling); with the coarser BF16 split and the plain
        // operands from the same MFMA arithmetic as the sum, so that the transmitted point's own
        // rounding cancels (with BF16 splits the direct form was 1.2e-4 bit off in MI on
        // DP-16QAM at high SNR).
        if constexpr (kDirectTx) ttx = fmaf(-b.c, sqdist<D>(y, lds_tab + txl * D), b.K);
        float ge, go, mi;
        uint32_t mask, near;
        mfma_pair_finish<MB>(b, P, n, active, bad, txl, ttx, ge, go, mi, mask, near);
        // far subsets of flagged bits resolved in the wave (at high SNR nearly every batch has
        // some; each would otherwise be a queue entry and a recomputation from the queue)
        mfma_pair_far_pass<T, D, SPLIT, NT>(lds_frag, lane, y, b.c, b.K, bad, b, n, active, txl, near, mask, ge, go);
        if (mask && active) {
            double gc = 0.0, mc = 0.0;
            queue_or_fix<D, D, (MB <= 6)>(b, k, &s_fill, (uint32_t)n, mask, near, gc, mc);
            ge += (float)gc;
            mi += (float)mc;
        }
        if (k.acc && active) {
            gsum += (double)ge + (double)go;
            msum += (double)mi;
        }
    }
    if (cur >= 0 && k.acc) flush();
    queue_close(k, &s_fill);
}

template <typename T, int D, bool SPLIT>
hipError_t launch_nt(const LaunchArgs& a, const void* frag, const void* pv, int grid, int threads, hipStream_t st) {
    const uint4* f = (const uint4*)frag;
    const uint16_t* p = (const uint16_t*)pv;
    switch (a.M) {
        case 32: hipLaunchKernelGGL((demap_mfma_small_kernel<T, D, SPLIT, 1>), dim3(grid), dim3(threads), 0, st, a, f, p); break;
        case 64: hipLaunchKernelGGL((demap_mfma_small_kernel<T, D, SPLIT, 2>), dim3(grid), dim3(threads), 0, st, a, f, p); break;
        case 128: hipLaunchKernelGGL((demap_mfma_small_kernel<T, D, SPLIT, 4>), dim3(grid), dim3(threads), 0, st, a, f, p); break;
        case 256: hipLaunchKernelGGL((demap_mfma_small_kernel<T, D, SPLIT, 8>), dim3(grid), dim3(threads), 0, st, a, f, p); break;
        default: return hipErrorNotSupported;
    }
    return hipGetLastError();
}

template <typename T, bool SPLIT>
hipError_t launch_d(const LaunchArgs& a, const void* frag, const void* pv, int grid, int threads, hipStream_t st) {
    switch (a.D) {
        case 2: return launch_nt<T, 2, SPLIT>(a, frag, pv, grid, threads, st);
        case 4: return launch_nt<T, 4, SPLIT>(a, frag, pv, grid, threads, st);
        case 8: return launch_nt<T, 8, SPLIT>(a, frag, pv, grid, threads, st);
        default: return hipErrorNotSupported;
    }
}

}  // namespace

bool mfma_small_supported(int M, int D) { return M >= 32 && M <= 256 && (D == 2 || D == 4 || D == 8); }

// The fewer the symbols, the smaller the blocks, so that each CU has some; 256 symbols a block (four or
// three blocks per CU) leave the ends of a large launch even.
int mfma_small_threads(int64_t symbols, int cus) {
    int t = 64;
    while (t < kThreads && symbols > (int64_t)cus * t) t *= 2;
    return t;
}

hipError_t launch_demap_mfma_small(const LaunchArgs& a, int prec, const void* frag, const void* pv, int grid,
                                   int threads, hipStream_t st) {
    if (!mfma_small_supported(a.M, a.D)) return hipErrorNotSupported;
    switch (prec) {
        case 1: return launch_d<__bf16, false>(a, frag, pv, grid, threads, st);
        case 2: return launch_d<_Float16, false>(a, frag, pv, grid, threads, st);
        case 3: return launch_d<__bf16, true>(a, frag, pv, grid, threads, st);
        case 4: return launch_d<_Float16, true>(a, frag, pv, grid, threads, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace dm
