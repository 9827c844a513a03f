// Minimum-distance decisions with the distance cross term on MFMA (gfx950), exact by proof.
//
// The split-FP16 MFMA (three products per term, FP32 accumulation) yields for every symbol and
// point u~ = K + 2 y.x - ||x||^2 - ||y||^2 = K - ||y - x||^2, with a per-symbol offset
// K = (||y|| + r_max)^2 + 1 that keeps every u~ positive, so the bit patterns of the u~ order
// like their values.  The 16 result registers of a lane are the labels 32 t + 16 h + r of tile t
// (h the lane half): one group of 16 consecutive labels.  The matrix pass only ranks groups: the
// group's largest u~ (8 max / max3 instructions for 16 values), with the complemented tile
// index in its low 7 bits, updates the lane's best and second-best groups (and_or, med3, max), so
// a 32-point tile costs 11 vector instructions per lane instead of one and a quarter per value.
// The winning group's 16 points are then compared by the reference FP32 distance itself, eight
// per lane half, ties to the lowest label.
//
// Exactness.  Per value, |u~ - u| is at most 3.5e-6 K (FP32 accumulation of 3D + 5 terms bounded
// by 2K) + 1e-6 K (operand splitting, dropped lo*lo products) + 5.4e-7 K (rounding of the
// reference FP32 distance) + 1.5e-5 K (the 7 packed bits: 127 ulp, at most 2^-16 of the value),
// under 2.1e-5 K in all; with eps = 2^-15 K (+ a floor for FP16 subnormal lo parts) a gap between
// the two best groups above 2 eps proves that the minimiser of the reference distance lies in the
// winning group.  Otherwise (near or exact ties between groups, values out of FP16 range,
// non-finite inputs) the whole table is scanned for that symbol with the reference formula (lowest label
// among equal distances): by the wave, 64 points at a time, or where that is less work for so many
// of its symbols, by each lane for its own.  No queue and no second launch.  (All symbols unproven, as
// with points of 1e-3: 2^20 symbols of 8D with 2048 points 1930 us by the wave alone, 990 so;
// 4096 of 32-QAM 47 and 29.)
//
// A wave takes 64 symbols, one per lane, as two sets of 32 MFMA columns, so that each point
// tile read from LDS serves both (with one set the LDS reads, 16 cycles a tile and wave, took as
// long as the MFMAs).
//
// What bounds it: the matrix cores.  On real operands they are power-limited (a 32x32x16 product
// of random values takes 20.8 ns per SIMD, of zeros 13.6 ns; a large BF16 matrix product reaches
// 1.1 PFLOP/s on the same card), and one chain of MFMAs runs under each set's maxima.
// Measured, 2^24 symbols of 8D M = 2048: 4.2 -> 2.25 ms (1.0 PFLOP/s) against the earlier
// per-value ranking with a queue and a second kernel; 2^23 symbols of 128-QAM: 1304 -> 169 us,
// most of which had been atomics on the queue's and the error counts' few addresses.
#include "device_common.hpp"
#include "kernels.hpp"
#include "mfma_body.hpp"
#include "wave_reduce.hpp"

namespace dm {

namespace {

constexpr int kHardMfmaThreads = 1024;
constexpr int kHardMfmaLds = 131072;   // staged chunk: at most 128 tiles, so 7 bits hold its tile index
constexpr uint32_t kTileMask = 0x7Fu;

// Reference FP32 distance of the library's hard decisions.
template <int D>
__device__ __forceinline__ float ref_dist(const float (&y)[D], const float* x) {
    float acc = 0.0f;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const float t = y[d] - x[d];
        acc = __builtin_fmaf(t, t, acc);
    }
    return acc;
}

template <int D>
__global__ __launch_bounds__(kHardMfmaThreads) void hard_mfma_kernel(const HardArgs a, const uint4* __restrict__ frag,
                                                                     float r_max) {
    using T = _Float16;
    constexpr int S = Slots<D, true>::S;
    using V = typename Mma<T>::V;
    extern __shared__ uint4 lds_frag[];
    const int ntiles = a.M >> 5;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int waves = blockDim.x >> 6;
    const int wave_slot = (blockIdx.x * waves + wave) % kAccSlots;
    const int chunk_tiles = min(ntiles, kHardMfmaLds / (S * 64 * 16));
    const int nchunks = (ntiles + chunk_tiles - 1) / chunk_tiles;
    auto stage = [&](int t0, int cnt) {
        const uint4* src = frag + (size_t)t0 * S * 64;
        for (int i = tid; i < cnt * S * 64; i += blockDim.x) lds_frag[i] = src[i];
    };
    if (nchunks == 1) {
        stage(0, ntiles);
        __syncthreads();
    }
    const int64_t sym_per_blk = blockDim.x;
    const int64_t blks = (a.N + sym_per_blk - 1) / sym_per_blk;
    const int64_t total = blks * a.n_blk;
    // Error counts accumulate per lane and go out once per received block and wave, spread over
    // kAccSlots addresses (device-scope atomics on one address serialise at ~11 ns each).
    uint32_t se = 0, be = 0, exact = 0;
    int cur = -1;
    auto flush = [&]() {
        if (cur >= 0 && a.counts) hard_flush(a.counts, cur, wave_slot, lane, se, be);
        se = be = 0;
    };
    // (s, r) = divmod(bt, blks), advanced incrementally; the next symbol and its transmitted row
    // are loaded one batch ahead.
    int s = (int)(blockIdx.x / blks);
    int64_t r = blockIdx.x - (int64_t)s * blks;
    float y_nx[D];
    uint32_t row_nx = 0;
    auto fetch = [&](int sf, int64_t rf) {
        const int64_t n = rf * sym_per_blk + tid;
        const size_t nc = (size_t)(n < a.N ? n : 0);
        const float* yrow = a.y[sf] + nc * D;
#pragma unroll
        for (int d = 0; d < D; ++d) y_nx[d] = yrow[d];
        if (a.counts) row_nx = a.tx[nc];
    };
    if ((int64_t)blockIdx.x < total) fetch(s, r);
    for (int64_t bt = blockIdx.x; bt < total; bt += gridDim.x) {
        const int64_t n = r * sym_per_blk + tid;
        if (s != cur) {
            flush();
            cur = s;
        }
        const bool active = n < a.N;
        float y[D];
#pragma unroll
        for (int d = 0; d < D; ++d) y[d] = active ? y_nx[d] : 0.0f;
        uint32_t row = row_nx;
        uint16_t* const out = a.labels_out[s];
        r += gridDim.x;
        while (r >= blks) {
            r -= blks;
            ++s;
        }
        if (bt + gridDim.x < total) fetch(s, r);
        int txl = 0;
        if (a.counts) {  // sent label, used after the decision
            if (row >= (uint32_t)a.M) {
                if (active) atomicOr(a.bad_tx, 1u);
                row = 0;
            }
            txl = a.row2label[row];
        }
        float ysq = 0.0f;
#pragma unroll
        for (int d = 0; d < D; ++d) ysq = fmaf(y[d], y[d], ysq);
        const float rr = sqrtf(ysq) + r_max;
        const float K = fmaf(rr, rr, 1.0f);
        bool bad = false;
        // symbols of lanes 0..31 (f0) and 32..63 (f1): every point tile read from LDS serves both
        Frags<T, S> f0, f1;
        build_pair_frags<T, D, true>(y, 1.0f, K, f0, f1, bad);
        // the mask lives in a register so that masking and inserting the (scalar) tile field is
        // one v_and_or_b32 (a literal mask and a scalar field would need two instructions)
        uint32_t keep = ~kTileMask;
        asm volatile("" : "+v"(keep));
        // per symbol set and lane half (16 labels of every tile): best and second-best groups
        uint32_t best0 = 0u, sec0 = 0u, best1 = 0u, sec1 = 0u;
        int tw0 = 0, tw1 = 0;  // tile of the best group
        for (int ch = 0; ch < nchunks; ++ch) {
            const int t0 = ch * chunk_tiles;
            const int cnt = min(chunk_tiles, ntiles - t0);
            if (nchunks > 1) {
                __syncthreads();
                stage(t0, cnt);
                __syncthreads();
            }
            auto read = [&](int t, V (&x)[S]) {
                const uint4* fp = lds_frag + (size_t)t * S * 64 + lane;
#pragma unroll
                for (int q = 0; q < S; ++q) x[q] = __builtin_bit_cast(V, fp[q * 64]);
            };
            auto mma = [&](const V (&x)[S], const Frags<T, S>& f) {
                f32x16 acc = Mma<T>::run(x[0], f.v[0]);
#pragma unroll
                for (int q = 1; q < S; ++q) acc = Mma<T>::run(x[q], f.v[q], acc);
                return acc;
            };
            auto rank = [&](const f32x16& x, int t, uint32_t& cb, uint32_t& cs) {
                uint32_t u[16];
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    const float f = x[q];
                    u[q] = __float_as_uint(f);
                }
                uint32_t g = max(max(u[0], u[1]), u[2]);
#pragma unroll
                for (int q = 3; q < 15; q += 2) g = max(max(g, u[q]), u[q + 1]);
                g = max(g, u[15]);
                g = (g & keep) | (kTileMask - (uint32_t)t);
                uint32_t med;  // second largest of {cb, cs, g}
                asm("v_med3_u32 %0, %1, %2, %3" : "=v"(med) : "v"(cb), "v"(cs), "v"(g));
                cs = med;
                cb = max(cb, g);
            };
            uint32_t cb0 = 0u, cs0 = 0u, cb1 = 0u, cs1 = 0u;  // the chunk's groups
            V xa[S], xb[S];
            read(0, xa);
            f32x16 acc0 = mma(xa, f0), acc1;
            // one chain of MFMAs runs under each set's maxima; the next tile is read a tile ahead
            for (int t = 0; t < cnt; t += 2) {
                read(min(t + 1, cnt - 1), xb);
                acc1 = mma(xa, f1);
                rank(acc0, t, cb0, cs0);
                if (t + 1 < cnt) acc0 = mma(xb, f0);
                rank(acc1, t, cb1, cs1);
                if (t + 1 < cnt) {
                    read(min(t + 2, cnt - 1), xa);
                    acc1 = mma(xb, f1);
                    rank(acc0, t + 1, cb0, cs0);
                    if (t + 2 < cnt) acc0 = mma(xa, f0);
                    rank(acc1, t + 1, cb1, cs1);
                }
            }
            auto merge = [&](uint32_t cb, uint32_t cs, uint32_t& best, uint32_t& sec, int& tw) {
                const bool lead = cb > best;
                sec = lead ? max(best, cs) : max(sec, cb);
                tw = lead ? t0 + (int)(kTileMask - (cb & kTileMask)) : tw;
                best = lead ? cb : best;
            };
            merge(cb0, cs0, best0, sec0, tw0);
            merge(cb1, cs1, best1, sec1, tw1);
        }
        // each lane's own symbol: the two label halves' groups meet (b0, s0, w0 the lower half's)
        uint32_t b0, b1, s0, s1, w0, w1;
        swap_halves(best0, best1, b0, b1);
        swap_halves(sec0, sec1, s0, s1);
        swap_halves((uint32_t)tw0, (uint32_t)tw1, w0, w1);
        const bool hi = b1 > b0;
        const uint32_t bg = max(b0, b1), sg = max(max(s0, s1), min(b0, b1));
        const float gap = __uint_as_float(bg & ~kTileMask) - __uint_as_float(sg & ~kTileMask);
        const float eps = 0x1p-15f * K + 0x1p-18f * (1.0f + rr);
        const bool ok = !bad && (gap > 2.0f * eps) && (gap < __builtin_inff());
        const int base = ok ? 32 * (int)(hi ? w1 : w0) + (hi ? 16 : 0) : 0;
        // reference distances of the winning group
        const float* cand = a.table + (size_t)base * D;
        float bd = __builtin_inff();
        int dec = 0;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const float d = ref_dist<D>(y, cand + q * D);
            const bool better = d < bd;
            bd = better ? d : bd;
            dec = better ? q : dec;
            // at most four points in flight
            if (q % 4 == 3) asm volatile("" : "+v"(bd), "+v"(dec)::"memory");
        }
        dec += base;
        // symbols without a proven group: the whole wave scans the table for each
        uint64_t todo = __ballot(active && !ok);
        if (a.exact) {  // also counts the symbols whose runner-up inside the group is that near
            const float lim = bd + 2.0f * eps;
            int near = 0;
#pragma unroll 1
            for (int q = 0; q < 16; ++q) near += ref_dist<D>(y, cand + q * D) <= lim;
            if (active && (!ok || near > 1)) ++exact;
        }
        // (in issue slots: 2 D + 3 per point by lanes, 2 D + 5 per 64 points and some 60 to reduce per symbol)
        if (__builtin_popcountll(todo) * (((a.M + 63) >> 6) * (2 * D + 5) + 60) > a.M * (2 * D + 3)) {
            // many: each lane scans it for its own symbol, points read as scalars
            const auto tab = (const __attribute__((address_space(4))) float*)(uintptr_t)a.table;
            float best_d = __builtin_inff();
            int best_l = 0;
            constexpr int G = D <= 4 ? 16 : 8;  // points in flight (64 scalars): few waves may be there to hide the reads
#pragma unroll 1
            for (int l = 0; l < a.M; l += G) {
                float x[G][D];
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int d = 0; d < D; ++d) x[g][d] = tab[(size_t)(l + g) * D + d];
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const float d = ref_dist<D>(y, x[g]);
                    const bool better = d < best_d;
                    best_d = better ? d : best_d;
                    best_l = better ? l + g : best_l;
                }
            }
            if (!ok) dec = best_l;
            todo = 0;
        }
        while (todo) {
            const int j = __builtin_ctzll(todo);
            todo &= todo - 1;
            float ys[D];
#pragma unroll
            for (int d = 0; d < D; ++d)
                ys[d] = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(y[d]), j));
            float best_d = __builtin_inff();
            uint32_t best_l = 0;
#pragma unroll 4
            for (int l = lane; l < a.M; l += 64) {
                const float d = ref_dist<D>(ys, a.table + (size_t)l * D);
                const bool better = d < best_d;
                best_d = better ? d : best_d;
                best_l = better ? (uint32_t)l : best_l;
            }
            const float dm = wave_reduce_f(best_d, [](float p, float q) { return fminf(p, q); });
            const uint32_t lm = wave_min_u32(best_d == dm ? best_l : 0xFFFFFFFFu);
            if (lane == j) dec = (int)lm;
        }
        if (active) {
            if (out) out[n] = (uint16_t)dec;
            if (a.counts) {
                se += dec != txl;
                be += __builtin_popcount((uint32_t)(dec ^ txl));
            }
        }
    }
    flush();
    if (a.exact) {
        exact = wave_sum_u32(exact);
        if (lane == 0 && exact) atomicAdd(a.exact + wave_slot, exact);
    }
}

template <int D>
hipError_t launch_hard_mfma_t(const HardArgs& a, const void* frag, float r_max, int cus, hipStream_t st) {
    constexpr int S = Slots<D, true>::S;
    const int ntiles = a.M >> 5;
    const int chunk_tiles = std::min(ntiles, kHardMfmaLds / (S * 64 * 16));
    const size_t lds = (size_t)chunk_tiles * S * 64 * 16;
    auto kern = hard_mfma_kernel<D>;
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    // 16 waves per block (one block per CU) when the symbols fill the GPU; fewer, down to four
    // (one per SIMD), when they would otherwise leave CUs without a block.
    const int64_t want = (a.N * a.n_blk + (int64_t)cus * 64 - 1) / ((int64_t)cus * 64);
    int threads = 256;
    while (threads < kHardMfmaThreads && threads < 64 * want) threads *= 2;
    const int64_t work = (a.N + threads - 1) / threads * a.n_blk;
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(work, cus));
    hipLaunchKernelGGL(kern, dim3(grid), dim3(threads), lds, st, a, (const uint4*)frag, r_max);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_hard_mfma(const HardArgs& a, const void* frag, float r_max, int cus, hipStream_t st) {
    switch (a.D) {
        case 1: return launch_hard_mfma_t<1>(a, frag, r_max, cus, st);
        case 2: return launch_hard_mfma_t<2>(a, frag, r_max, cus, st);
        case 3: return launch_hard_mfma_t<3>(a, frag, r_max, cus, st);
        case 4: return launch_hard_mfma_t<4>(a, frag, r_max, cus, st);
        case 5: return launch_hard_mfma_t<5>(a, frag, r_max, cus, st);
        case 6: return launch_hard_mfma_t<6>(a, frag, r_max, cus, st);
        case 7: return launch_hard_mfma_t<7>(a, frag, r_max, cus, st);
        case 8: return launch_hard_mfma_t<8>(a, frag, r_max, cus, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace dm
