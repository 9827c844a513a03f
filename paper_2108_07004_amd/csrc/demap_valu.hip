// Exact soft demapper, FP32 direct-difference variant, plus the far-subset fix-up (gfx950).
//
// One lane owns one received symbol and walks the whole label-ordered point table, read with
// wave-uniform addresses from LDS (broadcast) or, up to 256 points, through the scalar cache; the
// per-symbol arithmetic is in valu_body.hpp.  A persistent grid walks (SNR point, block-sized tile)
// work items; the next tile's symbols and transmitted rows are loaded a tile ahead, and the GMI / MI
// terms are summed per lane in FP64 and over the wave only when the SNR point changes.
//
// Measured (this kernel alone), against one body for all M that stored each LLR by itself and reduced
// the sums over the wave once a tile: DP-16QAM, 11 x 2^20 symbols, 1250 -> 1155 us; DP-QPSK, 6 x 65536
// symbols, 16.2 -> 13.0 us; 64-QAM, 2^20 symbols, 34.1 -> 29.2 us.
#include "device_common.hpp"
#include "fixup_drain.hpp"
#include "kernels.hpp"
#include "valu_body.hpp"
#include "wave_reduce.hpp"

namespace dm {

namespace {

constexpr int kValuThreads = 512;  // most threads per block
constexpr int kLdsFloats = 16384;  // 64 KiB of points per staged chunk

// (D <= 8: at most 128 registers, so that two 512-thread blocks fit a CU)
template <int DP, int MC>
__global__ __launch_bounds__(kValuThreads, DP <= 8 ? 4 : 1) void demap_valu_kernel(const LaunchArgs a) {
    extern __shared__ __align__(16) float lds[];
    __shared__ uint32_t s_fill;  // entries in this block's fix-up queue region
    const int tid = threadIdx.x;
    if (tid == 0) s_fill = 0u;
    const int M = MC ? MC : a.M, D = a.D;
    const int Mpad = MC ? MC : M < 16 ? 16 : M;
    // Chunk = whole table when it fits in 64 KiB, else a multiple of 64 points.
    int chunk = (kLdsFloats / DP) & ~63;
    if (chunk >= Mpad) chunk = Mpad;
    const int nchunks = MC ? 1 : (Mpad + chunk - 1) / chunk;
    const int lane = tid & 63;
    const int wave_slot = (blockIdx.x * (blockDim.x >> 6) + (tid >> 6)) % kAccSlots;
    const Sinks& k = a.sinks;
    const auto stab = (ScalarTable)(uintptr_t)a.table;

    auto stage = [&](int c0, int cnt) {
        for (int i = tid; i < cnt * DP; i += blockDim.x) {
            const int j = c0 + i / DP;
            lds[i] = (j < M) ? a.table[(size_t)c0 * DP + i] : 1.0e19f;  // padding: e_j = 0
        }
    };
    if (nchunks == 1) stage(0, Mpad);
    __syncthreads();

    const int64_t total = a.tiles_per_snr * a.n_snr;
    double gsum = 0.0, msum = 0.0;
    uint32_t pairs = 0;  // (symbol, bit) pairs recomputed in place
    int cur = -1;
    auto flush = [&]() {
        if (cur < 0 || !k.acc) return;
        if constexpr (MC != 0 && MC <= 16) {
            const uint32_t pw = wave_sum_u32(pairs);
            if (lane == 0 && pw) atomicAdd(k.fix_pairs + cur, pw);
            pairs = 0;
        }
        const double gw = wave_sum(gsum), mw = wave_sum(msum);
        if (lane == 0) {
            acc_add(k.acc, cur, wave_slot, 0, gw);
            acc_add(k.acc, cur, wave_slot, 1, mw);
        }
        gsum = msum = 0.0;
    };
    // (s, r) = divmod(tile, tiles_per_snr), advanced incrementally.  Loads are unconditional with
    // clamped indices and selected at use (a load under a branch is waited for at once).
    int s = (int)(blockIdx.x / a.tiles_per_snr);
    int64_t r = blockIdx.x - (int64_t)s * a.tiles_per_snr;
    float y_nx[DP];
    uint32_t row_nx = 0;
    auto fetch = [&](int sf, int64_t rf) {
        const int64_t n = rf * blockDim.x + tid;
        const size_t nc = (size_t)(n < a.N ? n : 0);
        const float* src = a.snr[sf].y + nc * D;
#pragma unroll
        for (int d = 0; d < DP; ++d) y_nx[d] = src[DP <= 8 ? d : min(d, D - 1)];
        if (a.tx) row_nx = a.tx[nc];
    };
    if ((int64_t)blockIdx.x < total) fetch(s, r);
    for (int64_t tile = blockIdx.x; tile < total; tile += gridDim.x) {
        const int64_t n = r * blockDim.x + tid;
        if (s != cur) {
            flush();
            cur = s;
        }
        const bool active = n < a.N;
        const BlockView b = view_sym(a, s, n, active);
        float y[DP];
#pragma unroll
        for (int d = 0; d < DP; ++d) y[d] = active && (DP <= 8 || d < D) ? y_nx[d] : 0.0f;
        uint32_t row = row_nx;
        r += gridDim.x;
        while (r >= a.tiles_per_snr) {
            r -= a.tiles_per_snr;
            ++s;
        }
        if (tile + gridDim.x < total) fetch(s, r);
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
        for (int ch = 0; ch < nchunks; ++ch) {
            const int c0 = ch * chunk;
            const int cnt = min(chunk, Mpad - c0);
            if (nchunks > 1) {
                __syncthreads();
                stage(c0, cnt);
                __syncthreads();
            }
            if constexpr (MC != 0)
                valu_accumulate<DP, DP, MC>(stab, 0, MC, y, b.c, b.K, b.m, S, H0, H1);
            else
                valu_accumulate<DP, DP, MC>((LdsTable)lds, c0, cnt, y, b.c, b.K, b.m, S, H0, H1);
        }
        float g, mi;
        double gc = 0.0, mc = 0.0;
        const float* xtx = nchunks == 1 ? lds + txl * DP : b.table + (size_t)txl * DP;
        valu_epilogue<DP, DP, MC>(b, k, &s_fill, n, active, y, S, H0, H1, txl, xtx, stab, g, mi, gc, mc, pairs);
        if (k.acc && active) {
            gsum += (double)g + gc;
            msum += (double)mi + mc;
        }
    }
    flush();
    queue_close(k, &s_fill);
}

// Exact recomputation of the queued symbols (one lane or one wavefront per symbol).
template <int DP>
__global__ __launch_bounds__(kFixThreads) void fixup_kernel(const LaunchArgs a, int cache_pts) {
    extern __shared__ float s_t[];  // per-wave exponent caches, 4 x cache_pts floats
    drain_fix_queue<DP>(a.sinks, [&](const FixEntry& e) { return view_sym(a, (int)e.tag, e.n, true); },
                        s_t + (threadIdx.x >> 6) * cache_pts, cache_pts, a.M, a.table);
}

template <int DP, int MC>
hipError_t launch_valu_mc(const LaunchArgs& a, int grid, int threads, hipStream_t st) {
    const int Mpad = MC ? MC : a.M < 16 ? 16 : a.M;
    int chunk = (kLdsFloats / DP) & ~63;
    if (chunk >= Mpad) chunk = Mpad;
    const size_t lds = (size_t)chunk * DP * sizeof(float);
    hipLaunchKernelGGL((demap_valu_kernel<DP, MC>), dim3(grid), dim3(threads), lds, st, a);
    return hipGetLastError();
}

// Sizes known at compile time for M = 2 .. 256 and D = 1, 2, 4, 8 (the formats with few points per
// symbol, where the loop and epilogue overheads matter most, and tables within the scalar cache);
// any other shape takes the general kernel.
template <int DP>
hipError_t launch_valu_t(const LaunchArgs& a, int grid, int threads, hipStream_t st) {
    if constexpr (DP == 1 || DP == 2 || DP == 4 || DP == 8) {
        switch (a.M) {
            case 2: return launch_valu_mc<DP, 2>(a, grid, threads, st);
            case 4: return launch_valu_mc<DP, 4>(a, grid, threads, st);
            case 8: return launch_valu_mc<DP, 8>(a, grid, threads, st);
            case 16: return launch_valu_mc<DP, 16>(a, grid, threads, st);
            case 32: return launch_valu_mc<DP, 32>(a, grid, threads, st);
            case 64: return launch_valu_mc<DP, 64>(a, grid, threads, st);
            case 128: return launch_valu_mc<DP, 128>(a, grid, threads, st);
            case 256: return launch_valu_mc<DP, 256>(a, grid, threads, st);
            default: break;
        }
    }
    return launch_valu_mc<DP, 0>(a, grid, threads, st);
}

template <int DP>
hipError_t launch_fixup_t(const LaunchArgs& a, int grid, hipStream_t st) {
    hipLaunchKernelGGL(fixup_kernel<DP>, dim3(grid), dim3(kFixThreads), fixup_lds_bytes(a.M), st, a, fixup_cache_points(a.M));
    return hipGetLastError();
}

}  // namespace

int padded_dim(int D) {
    if (D <= 8) return D;
    return D <= 16 ? 16 : 32;
}

int valu_tile_symbols(int64_t symbols, int cus) {
    int t = 64;
    while (t < kValuThreads && symbols > (int64_t)cus * t) t *= 2;
    return t;
}

#define DM_DISPATCH_DP(FN, ...)                          \
    switch (padded_dim(a.D)) {                          \
        case 1: return FN<1>(__VA_ARGS__);              \
        case 2: return FN<2>(__VA_ARGS__);              \
        case 3: return FN<3>(__VA_ARGS__);              \
        case 4: return FN<4>(__VA_ARGS__);              \
        case 5: return FN<5>(__VA_ARGS__);              \
        case 6: return FN<6>(__VA_ARGS__);              \
        case 7: return FN<7>(__VA_ARGS__);              \
        case 8: return FN<8>(__VA_ARGS__);              \
        case 16: return FN<16>(__VA_ARGS__);            \
        case 32: return FN<32>(__VA_ARGS__);            \
        default: return hipErrorInvalidValue;           \
    }

hipError_t launch_demap_valu(const LaunchArgs& a, int grid, int threads, hipStream_t st) {
    DM_DISPATCH_DP(launch_valu_t, a, grid, threads, st)
}

hipError_t launch_fixup(const LaunchArgs& a, int grid, hipStream_t st) {
    DM_DISPATCH_DP(launch_fixup_t, a, grid, st)
}

}  // namespace dm
