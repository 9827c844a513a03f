// Batched exact demapping: one persistent launch over many (constellation, noise level, block) instances
// of uneven M, D and N (gfx950).
//
// Work items are (instance, sub consecutive symbol tiles) pairs listed instance by instance,
// the most costly instance first (sub per instance, from the plan's shape choice).  There are three
// lists, each with its own body: MFMA instances of more than 256 points, of 32 .. 256 points (the
// compile-time tile loop of mfma_small.hpp), and FP32 instances (batched_valu.hpp).  A workgroup belongs to
// one list, and fills a CU; the launch has the large tables' workgroups first, so those of the next
// list start as CUs run out of work.  As three kernels one after the other, each list's tail left the chip
// idle (12 instances of 2^12 .. 2^17 symbols: 271 us, now 191; 64 of 2^14 .. 2^22: 6.43 ms, now 6.32),
// and as one loop over one list the bodies' registers spilled in each other's loops (228 us; 8.11 ms).
//
// Workgroups claim fixed chunks of `grab` consecutive items of their list from a counter
// (dynamic balance: the cheap items at the end fill the tail) and restage their LDS table only
// when the next item belongs to another instance.  They ask when the last claim is done: a claim ahead,
// the first workgroups hold two of the last claims and others none (as many claims as workgroups, 2^20
// symbols of 8D with 2048 points in FP32: 2046 us ahead, 960 so; 2^19 on MFMA 305 and 168), and
// asking while a claim for each is left gains 0 to 6% on long lists but costs registers that spill.  GMI / MI
// partial sums are flushed per chunk and instance, so every fixed-point contribution covers a fixed
// set of symbols whichever workgroup runs it: the totals are bit-reproducible.  On MFMA one wave takes
// 32 symbols, a block 512 per tile.  Batched tables use a row stride of 8 (D <= 8 zero-padded): the
// padded coordinates contribute exact zeros, and the MFMA operand vectors of every instance have the same
// K layout.  Some 40 of the 128 vector registers spill, outside the tile and point loops.
#include "batched_valu.hpp"
#include "device_common.hpp"
#include "fixup_drain.hpp"
#include "kernels.hpp"
#include "mfma_body.hpp"
#include "mfma_small.hpp"

namespace dm {

namespace {

constexpr int kThreads = kBatchThreads;
constexpr int kWaves = kThreads / 64;

// One 32-symbol batch of an instance with 32 * NT points (D padded to 8): compile-time tile loop
// and epilogue.
template <typename T, bool SPLIT, int NT>
__device__ __forceinline__ void small_item(const uint4* lds, const BlockView& b, const Sinks& k, uint32_t* fill, const uint16_t* pv,
                                           const Frags<T, Slots<8, SPLIT>::S>& bfr, int64_t n, bool active, bool bad,
                                           int txl, int lane, float& g, float& mi) {
    constexpr int MB = SmallBits<NT>::MB;
    float S0[MB], S1[MB], tot;
    mfma_small_sums<T, 8, SPLIT, NT>(lds, lane, bfr, S0, S1, tot);
    mfma_finish<T, 8, SPLIT, MB>(b, k, fill, pv, bfr, S0, S1, tot, n, active, bad, txl, lane, g, mi);
}

// A workgroup of the list of small (SMALL) or large MFMA tables.
template <typename T, bool SPLIT, bool SMALL>
__device__ __forceinline__ void batched_mfma(const BatchArgs& a, uint4* lds_raw) {
    constexpr int S = Slots<8, SPLIT>::S;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int h = lane >> 5;
    const int wave = tid >> 6;
    const int wave_slot = (blockIdx.x * kWaves + wave) % kAccSlots;  // integer slots: any spread sums alike
    const Sinks& k = a.sinks;
    __shared__ int s_claim;      // first item of this claim
    __shared__ uint32_t s_fill;  // entries in this block's fix-up queue region
    if (tid == 0) s_fill = 0u;
    int staged = -1;
    for (;;) {
        // (asked for when the last claim is done, see the file's head)
        if (tid == 0) s_claim = (int)atomicAdd(a.next, (uint32_t)a.grab);
        __syncthreads();
        const int i0 = __builtin_amdgcn_readfirstlane(s_claim);
        if (i0 >= a.n_items) break;
        const int i1 = min(i0 + a.grab, a.n_items);
        for (int i = i0; i < i1;) {
            // a run of items of one instance: its symbol tiles one after the other, GMI / MI terms
            // summed per lane, then over the wave once
            const WorkItem it = uniform_copy(a.items[i]);
            const BatchDesc d = uniform_desc(a.desc[it.inst]);
            const BlockView& b = d.view;
            i += it.run;
            if (it.inst != staged) {  // restage the point table (whole block, uniform condition)
                __syncthreads();
                const int n16 = (b.M >> 5) * S * 64;
                for (int j = tid; j < n16; j += kThreads) lds_raw[j] = d.frag[j];
                __syncthreads();
                staged = it.inst;
            }
            const int tiles = it.run * d.sub;
            const int sub = wave * 32 + (lane & 31);
            // (the small tables' kernel has the registers to load a tile's symbols a tile ahead)
            float y_nx[8];
            uint32_t row_nx = 0;
            auto fetch = [&](int t) {
                const int64_t n = it.n0 + (int64_t)t * (kWaves * 32) + sub;
                const size_t nc = (size_t)(n < b.N ? n : 0);
                const float* src = b.y + nc * b.D;
#pragma unroll
                for (int q = 0; q < 8; ++q) y_nx[q] = src[min(q, b.D - 1)];
                if (b.tx) row_nx = b.tx[nc];
            };
            if constexpr (SMALL) fetch(0);
            double gl = 0.0, ml = 0.0;
            for (int t = 0; t < tiles; ++t) {
                float g = 0.0f, mi = 0.0f;
                const int64_t n = it.n0 + (int64_t)t * (kWaves * 32) + sub;
                const bool active = n < b.N;
                float y[8];
                int txl = 0;
                if constexpr (SMALL) {
#pragma unroll
                    for (int q = 0; q < 8; ++q) y[q] = active && q < b.D ? y_nx[q] : 0.0f;
                    uint32_t row = row_nx;
                    if (t + 1 < tiles) fetch(t + 1);
                    if (b.tx && active) {
                        if (row >= (uint32_t)b.M) {  // out-of-range row: clamped and reported
                            if (k.bad_tx) atomicOr(k.bad_tx, 1u);
                            row = 0;
                        }
                        txl = (int)b.row2label[row];
                    }
                } else {
                    load_symbol<8>(y, b.y + (size_t)(active ? n : 0) * b.D, b.D, active);
                    txl = (b.tx && active) ? tx_label(b, k, n) : 0;
                }
                bool bad = false;
                const Frags<T, S> bfr = build_symbol_frags<T, 8, SPLIT>(y, b.c, b.K, h, bad);
                if constexpr (SMALL) {
                    switch (b.M) {  // uniform
                        case 32: small_item<T, SPLIT, 1>(lds_raw, b, k, &s_fill, d.pv, bfr, n, active, bad, txl, lane, g, mi); break;
                        case 64: small_item<T, SPLIT, 2>(lds_raw, b, k, &s_fill, d.pv, bfr, n, active, bad, txl, lane, g, mi); break;
                        case 128: small_item<T, SPLIT, 4>(lds_raw, b, k, &s_fill, d.pv, bfr, n, active, bad, txl, lane, g, mi); break;
                        default: small_item<T, SPLIT, 8>(lds_raw, b, k, &s_fill, d.pv, bfr, n, active, bad, txl, lane, g, mi); break;
                    }
                } else {
                    MfmaAcc A;
                    A.init();
                    mfma_tiles<T, 8, SPLIT>(lds_raw, lane, 0, b.M >> 5, b.m, bfr, A);
                    mfma_epilogue<T, 8, SPLIT>(b, k, &s_fill, d.pv, bfr, A, n, active, bad, txl, lane, g, mi);
                }
                if (active) {
                    gl += (double)g;
                    ml += (double)mi;
                }
            }
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

template <typename T, bool SPLIT>
__global__ __launch_bounds__(kThreads) void demap_batched_kernel(const BatchLists p) {
    extern __shared__ __align__(16) uint4 lds_raw[];
    const int at = (int)blockIdx.x;
    const int large = p.grid[kBatchLarge], small = p.grid[kBatchSmall];
    if (at < large) batched_mfma<T, SPLIT, false>(p.list[kBatchLarge], lds_raw);
    else if (at < large + small) batched_mfma<T, SPLIT, true>(p.list[kBatchSmall], lds_raw);
    else batched_valu(p.list[kBatchValu], reinterpret_cast<float*>(lds_raw));
}

// Exact recomputation of the queued symbols of every instance (one lane or one wavefront per symbol).
__global__ __launch_bounds__(kFixThreads) void batched_fixup_kernel(const BatchArgs a) {
    __shared__ float s_t[4][kFixCached];  // per-wave exponent cache (32 KiB per block)
    drain_fix_queue<8>(a.sinks, [&](const FixEntry& e) { return a.desc[e.tag].view; }, s_t[threadIdx.x >> 6],
                       kFixCached);
}

// Zero the accumulators and counters with a kernel (a graph must not hold memset nodes).
__global__ void zero_words(uint32_t* p, size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}

template <typename T, bool SPLIT>
hipError_t prepare_t() {
    return hipFuncSetAttribute((const void*)demap_batched_kernel<T, SPLIT>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               kBatchedLdsAlloc);
}

template <typename T, bool SPLIT>
hipError_t launch_batched_t(const BatchLists& p, hipStream_t st) {
    // the largest table of the lists at hand; a large table also has the one fragment tile that its pipeline
    // reads past a 16-tile block
    size_t lds = p.grid[kBatchValu] ? p.list[kBatchValu].lds_bytes : 0;
    if (p.grid[kBatchSmall]) lds = std::max<size_t>(lds, 8 * Slots<8, SPLIT>::S * 1024);
    if (p.grid[kBatchLarge]) lds = std::max<size_t>(lds, kBatchedLdsAlloc);
    const int grid = p.grid[kBatchValu] + p.grid[kBatchSmall] + p.grid[kBatchLarge];
    hipLaunchKernelGGL((demap_batched_kernel<T, SPLIT>), dim3(grid), dim3(kThreads), lds, st, p);
    return hipGetLastError();
}

}  // namespace

int batched_tile_symbols(int kind) { return kind == kKindMfma ? kWaves * 32 : 1024; }

hipError_t launch_demap_batched(const BatchLists& p, int prec, hipStream_t st) {
    if (p.grid[kBatchSmall] + p.grid[kBatchLarge] == 0)
        return p.grid[kBatchValu] ? launch_demap_batched_valu(p.list[kBatchValu], p.grid[kBatchValu], st) : hipSuccess;
    switch (prec) {
        case 4: return launch_batched_t<_Float16, true>(p, st);
        case 1: return launch_batched_t<__bf16, false>(p, st);
        case 2: return launch_batched_t<_Float16, false>(p, st);
        case 3: return launch_batched_t<__bf16, true>(p, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t prepare_batched(int prec) {
    const hipError_t e = prepare_batched_valu();
    if (e != hipSuccess) return e;
    switch (prec) {
        case 0: return hipSuccess;  // every instance runs the FP32 body
        case 4: return prepare_t<_Float16, true>();
        case 1: return prepare_t<__bf16, false>();
        case 2: return prepare_t<_Float16, false>();
        case 3: return prepare_t<__bf16, true>();
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_batched_fixup(const BatchArgs& a, int grid, hipStream_t st) {
    hipLaunchKernelGGL(batched_fixup_kernel, dim3(grid), dim3(kFixThreads), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_zero_words(uint32_t* p, size_t n, hipStream_t st) {
    const int blocks = (int)std::max<size_t>(1, std::min<size_t>(64, (n + 255) / 256));
    hipLaunchKernelGGL(zero_words, dim3(blocks), dim3(256), 0, st, p, n);
    return hipGetLastError();
}

}  // namespace dm
