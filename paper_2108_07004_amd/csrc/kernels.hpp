// Host-visible launchers of the demapping kernels (defined next to each kernel).
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device_common.hpp"

namespace dm {

// Table row stride used by the kernels for a dimensionality D (1..8 exact, else 16 or 32).
int padded_dim(int D);

// Symbols per tile (threads per block) of the FP32 kernel, one lane per symbol: 512, or down to 64
// when that many would leave CUs without a tile.
int valu_tile_symbols(int64_t symbols, int cus);
int hard_tile_symbols();
hipError_t launch_hard_demap(const HardArgs& a, int grid, hipStream_t st);
// MFMA decisions (split-FP16 operand table `frag` of the label-order points, r_max = max ||x||).
hipError_t launch_hard_mfma(const HardArgs& a, const void* frag, float r_max, int cus, hipStream_t st);

// FP32 direct-difference demapper (one lane per symbol, persistent grid).
hipError_t launch_demap_valu(const LaunchArgs& a, int grid, int threads, hipStream_t st);

// Most blocks that a launch's symbols give the fix-up kernel work for, so that an empty pass costs little: a
// lane per symbol up to 64 points; for 128 and 256 points (rows) chunks of 32 on up to 512 blocks, then
// of 256; else a wavefront per symbol.  (With 256 symbols per block for every form, 64 per wavefront: 4096
// symbols of 8D, 4096 points at 21 dB 4040 us a call, now 476; of 256-QAM 22.5, now 18.3.  Rows over more
// than 512 blocks: an empty pass over 200000 symbols takes 1.6 us more.)
inline int64_t fixup_most_blocks(int M, int64_t symbols) {
    auto blocks = [symbols](int per) { return (symbols + per - 1) / per; };
    if (M <= 64) return blocks(256);
    if (M <= 256) return std::max(blocks(256), std::min<int64_t>(blocks(32), 512));
    return blocks(4);
}

// Exact recomputation of the queued (symbol, bit) pairs whose far-subset sum underflowed.
hipError_t launch_fixup(const LaunchArgs& a, int grid, hipStream_t st);
// The same for large tables (512 points and more that fit its LDS): one launch of at most cus blocks.
bool fixup_large_supported(int M, int D);
hipError_t launch_fixup_large(const LaunchArgs& a, int cus, hipStream_t st);
// Exponent cache of the fix-up kernel (per wave, 4 waves per block) for an M-point constellation,
// and the blocks per CU that fit it within 160 KiB of LDS and the kernel's 8 waves per SIMD.
inline int fixup_cache_points(int M) { return M <= kFixCached ? ((M + 63) / 64) * 64 : 64; }
inline size_t fixup_lds_bytes(int M) { return (size_t)4 * fixup_cache_points(M) * sizeof(float); }
inline int fixup_blocks_per_cu(int M) { return (int)std::min<size_t>(8, (160 * 1024) / (fixup_lds_bytes(M) + 1024)); }

// K slots (multiple of 16) of the MFMA operand vectors for dimensionality D.
int mfma_slots(int D, bool split);

// Symbols per block iteration of the MFMA kernel.
int mfma_block_symbols(int M, int D, int64_t symbols, int cus);

// MFMA demapper specialised for M = 32..256 points and D in {2, 4, 8} (tile count and label
// bits known at compile time); hipErrorNotSupported for other shapes.
bool mfma_small_supported(int M, int D);
hipError_t launch_demap_mfma_small(const LaunchArgs& a, int prec, const void* frag, const void* pv, int grid,
                                   int threads, hipStream_t st);
// Threads (and symbols) per block of that kernel for a launch of so many symbols.
int mfma_small_threads(int64_t symbols, int cus);

// MFMA demapper: prec 1 = BF16, 2 = FP16, 3 = BF16 split, 4 = FP16 split.  `frag` is the
// point-side operand table in fragment order ([tile][mfma][lane] x 16 bytes); `pv` the same
// operands per label ([label][K slots], 16-bit), read for the transmitted points.
hipError_t launch_demap_mfma(const LaunchArgs& a, int prec, const void* frag, const void* pv, int grid, int tile,
                             hipStream_t st);

// Symbols per work item of the batched kernel for an instance kind (kKindValu / kKindMfma).
int batched_tile_symbols(int kind);

// Allow the batched kernel of a precision its 128 KiB of dynamic LDS (call before launching or
// capturing it).
hipError_t prepare_batched(int prec);

// The persistent batched kernel over a plan's lists; prec selects the MFMA operand variant.
hipError_t launch_demap_batched(const BatchLists& p, int prec, hipStream_t st);
hipError_t launch_demap_batched_valu(const BatchArgs& a, int grid, hipStream_t st);
hipError_t prepare_batched_valu();

// Fix-up of queued symbols of any instance (tables with row stride 8).
hipError_t launch_batched_fixup(const BatchArgs& a, int grid, hipStream_t st);

// p[0..n) = 0 with a kernel (usable inside a captured graph).
hipError_t launch_zero_words(uint32_t* p, size_t n, hipStream_t st);

}  // namespace dm
