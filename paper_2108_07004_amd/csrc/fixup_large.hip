// The fix-up of constellations of 512 points and more (gfx950): exact recomputation of the queued
// (symbol, bit) pairs, one queued symbol per lane.
//
// At high SNR (8D formats beyond 15 dB) nearly every symbol has bits whose far subset underflowed, and
// the recomputation takes longer than the demapping.  With one wavefront per symbol every symbol reads
// the whole table (64 KiB at 2048 points of 8D) from L2.  Here 64 symbols share each point read (from LDS,
// broadcast), and one pass serves all bits (wide_sums.hpp: FP32 exponents, sums with the exponent range
// of a double).  The sums are taken over indexed accumulators as in valu_body.hpp: two FP64 additions
// per point.  A sum below 2^-1860 sends that bit to the two-pass form (fixup_wave).
//
// A workgroup is four groups of four waves.  A group takes 64 queued symbols; wave q of it walks the
// points with top label bits q (a quarter of the table), which are then no sums of its own but its
// total.  The four partial sums of every other bit meet in LDS, and each wave finishes its own bits.
//
// What bounds it: vector issue, some 30 instructions per (point, 64 symbols) at 8D.  Measured, sweeps of
// 8 x 262144 symbols of 8D, 2048 points, with LLRs: the product format from 6 to 20 dB 6050 us with two
// passes by wavefronts, now 690; random points from 8 to 22 dB 6730, now 590 (the demapping before it: 630
// on MFMA).  881619 symbols of the product format at 20 dB, whole call: 21.2 -> 1.5 ms.
//
// A lane takes its quarter of the table point by point, some 25 us at 2048 points of 8D however few
// symbols there are, so few symbols go by wavefronts: row q of the wave takes quarter q, lane r of
// it the points of index r modulo 16.  Both forms add the same numbers in the same order (sixteen points
// by a pairwise tree, which is what the lanes of a row can do), so a symbol's results do not depend on
// how many are queued with it.
#include "device_common.hpp"
#include "fixup_drain.hpp"
#include "kernels.hpp"
#include "wave_reduce.hpp"
#include "wide_sums.hpp"

namespace dm {

namespace {

constexpr int kThreads = 1024;
constexpr int kGroups = kThreads / 256;
constexpr int kTabFloats = 16384;                // table in LDS: at most 64 KiB
constexpr int kHighBits = 6;                     // label bits 6 and up of a quarter (M <= 16384)
constexpr int kRound = 4;                        // label bits that a group's waves exchange at a time
constexpr int kXchg = kGroups * 4 * 2 * kRound * 64;  // doubles
constexpr int kTot = kGroups * 4 * 64;
constexpr size_t kLdsBytes = (size_t)kTabFloats * 4 + (size_t)(kXchg + kTot) * 8;
static_assert(kLdsBytes >= (size_t)(kThreads / 64) * kFixCached * 4, "the wavefront form's exponent caches");

// Sum of v over the 16 lanes of each row, every lane receiving it: pairs, pairs of pairs, ..
__device__ __forceinline__ double row_tree(double v) {
    v += dpp_d<0xB1>(v);   // quad_perm [1,0,3,2]
    v += dpp_d<0x4E>(v);   // quad_perm [2,3,0,1]
    v += dpp_d<0x141>(v);  // row_half_mirror (the quads are uniform)
    v += dpp_d<0x140>(v);  // row_mirror
    return v;
}

// The same tree over the values f(0) .. f(15) of one lane.
template <int N, int R = 0, typename Fn>
__device__ __forceinline__ double lane_tree(Fn&& f) {
    if constexpr (N == 1) {
        return f(R);
    } else {
        const double a = lane_tree<N / 2, R>(f);
        const double b = lane_tree<N / 2, R + N / 2>(f);
        return a + b;
    }
}

// Value v of lane src, uniform.
__device__ __forceinline__ double read_lane(double v, int src) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, src);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), src);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// One queued symbol by a whole wavefront (all lanes active).  Returns the mask of what is out of range here;
// gcorr, mcorr: the corrections, in every lane.
template <int DP>
__device__ uint32_t wide_wave(const BlockView& b, const Sinks& k, uint32_t n, uint32_t mask, double& gcorr,
                              double& mcorr) {
    const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
    const int M = b.M, m = b.m, ml = m - 2;
    float y[DP];
    load_symbol<DP>(y, b.y + (size_t)n * b.D, b.D, true);
    const int txl = b.tx ? tx_label(b, k, n) : 0;
    const float* const pts = b.table + ((size_t)q * (M >> 2) + r) * DP;
    double acc = 0.0, accB[4], h0[kHighBits], h1[kHighBits], tot = 0.0;
#pragma unroll
    for (int g = 0; g < 4; ++g) accB[g] = 0.0;
#pragma unroll
    for (int p = 0; p < kHighBits; ++p) h0[p] = h1[p] = 0.0;
#pragma unroll 1
    for (int blk = 0; blk < (M >> 8); ++blk) {
        double bt = 0.0;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const double w = wide_exp2(fmaf(-b.c, sqdist<DP>(y, pts + (size_t)(blk * 64 + g * 16) * DP), b.K));
            acc += w;
            const double T = row_tree(w);
            accB[g] += T;
            bt += T;
        }
        tot += bt;
#pragma unroll
        for (int p = 0; p < kHighBits; ++p) {
            if ((blk >> p) & 1) h1[p] += bt;
            else h0[p] += bt;
        }
    }
    uint32_t left = 0u;
    auto finish = [&](int p, double s0, double s1) {
        if (!wide_ok(s0, s1)) {
            left |= 1u << p;
            return;
        }
        const float L = wide_log2_ratio(s1, s0);
        if (b.llr && lane == 0) b.llr[(size_t)n * m + (m - 1 - p)] = L * 0.69314718055994531f;
        if (b.tx) gcorr += (double)gmi_bit_term(L, (txl >> p) & 1);
    };
#pragma unroll
    for (int p = 0; p < 6 + kHighBits; ++p) {
        if (p >= ml || !((mask >> p) & 1u)) continue;  // uniform
        double s0 = 0.0, s1 = 0.0;
        if (p < 4) {
            const bool one = (r >> p) & 1;
            s0 = row_tree(one ? 0.0 : acc);
            s1 = row_tree(one ? acc : 0.0);
        } else if (p < 6) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                if ((g >> (p - 4)) & 1) s1 += accB[g];
                else s0 += accB[g];
            }
        } else {
            s0 = h0[p - 6];
            s1 = h1[p - 6];
        }
        double t0 = 0.0, t1 = 0.0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            t0 += read_lane(s0, 16 * w);
            t1 += read_lane(s1, 16 * w);
        }
        finish(p, t0, t1);
    }
    const double t0 = read_lane(tot, 0), t1 = read_lane(tot, 16), t2 = read_lane(tot, 32), t3 = read_lane(tot, 48);
    if ((mask >> (m - 2)) & 1u) finish(m - 2, t0 + t2, t1 + t3);
    if ((mask >> (m - 1)) & 1u) finish(m - 1, t0 + t1, t2 + t3);
    if ((mask & kMiFlag) && b.tx) {
        const double all = (t0 + t1) + (t2 + t3);
        if (wide_ok(all, all)) {
            const float ttx = fmaf(-b.c, sqdist<DP>(y, b.table + (size_t)txl * DP), b.K);
            mcorr += (double)wide_mi(m, all, ttx);
        } else {
            left |= kMiFlag;
        }
    }
    return left;
}

template <int DP>
__global__ __launch_bounds__(kThreads) void fixup_large_kernel(const LaunchArgs a, uint32_t lanes_from) {
    extern __shared__ __align__(16) float dyn[];
    __shared__ unsigned long long s_acc[kMaxSnrPerLaunch * 2];
    __shared__ uint32_t s_pairs[kMaxSnrPerLaunch];
    __shared__ uint32_t s_qpre[kMaxQueueRegions + 1];
    const Sinks& k = a.sinks;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    if (tid < kMaxSnrPerLaunch * 2) s_acc[tid] = 0ull;
    if (tid < kMaxSnrPerLaunch) s_pairs[tid] = 0u;
    queue_prefix<kThreads>(k, s_qpre);
    __syncthreads();
    const uint32_t count = s_qpre[kMaxQueueRegions];
    auto view = [&](const FixEntry& e) { return view_sym(a, (int)e.tag, e.n, true); };
    auto count_pairs = [&](const FixEntry& e) {
        if (k.fix_pairs) atomicAdd(&s_pairs[e.tag], (uint32_t)__popc(e.mask & 0xFFFFu));
    };
    auto add = [&](uint32_t tag, int which, double v) {
        const long long q = __double2ll_rn(v * kFixScale);
        if (k.acc && q != 0) atomicAdd(&s_acc[tag * 2 + which], (unsigned long long)q);
    };
    if (count < lanes_from) {
        // few symbols: a wavefront each
        const uint32_t waves = gridDim.x * (kThreads / 64);
        for (uint32_t i = wv * gridDim.x + blockIdx.x; i < count; i += waves) {
            const FixEntry e = uniform_copy(k.queue[queue_index(k, s_qpre, i)]);
            double gc = 0.0, mc = 0.0;
            const uint32_t left = wide_wave<DP>(view(e), k, e.n, e.mask, gc, mc);
            if (lane == 0) {
                add(e.tag, 0, gc);
                add(e.tag, 1, mc);
            }
            gc = mc = 0.0;
            if (left) fixup_wave<DP>(view(e), k, e.n, left, dyn + wv * kFixCached, kFixCached, gc, mc);
            if (lane == 0) {
                count_pairs(e);
                add(e.tag, 0, gc);
                add(e.tag, 1, mc);
            }
        }
    } else {
        const int M = a.M, m = a.m, ml = m - 2;  // ml: label bits below the wave's quarter
        float* const tab = dyn;
        double* const xchg = reinterpret_cast<double*>(dyn + kTabFloats);
        const int group = wv >> 2, q = wv & 3;
        double* const gx = xchg + group * (4 * 2 * kRound * 64);
        double* const gt = xchg + kXchg + group * (4 * 64);
        const uint32_t batches = (count + 63) / 64;
        if (blockIdx.x < batches)
            for (int i = tid; i < M * DP; i += kThreads) tab[i] = a.table[i];
        __syncthreads();
        // batch b: group b / gridDim.x % kGroups of block b % gridDim.x, so that few batches spread over the CUs
        for (uint32_t b0 = blockIdx.x; b0 < batches; b0 += gridDim.x * kGroups) {  // uniform over the block
            const uint32_t i = (b0 + group * gridDim.x) * 64 + lane;
            const bool live = i < count;
            const FixEntry e = k.queue[queue_index(k, s_qpre, live ? i : count - 1)];
            const uint32_t mask = live ? e.mask : 0u;
            const BlockView b = view(e);
            float y[DP];
            load_symbol<DP>(y, b.y + (size_t)e.n * b.D, b.D, true);
            const int txl = b.tx ? tx_label(b, k, e.n) : 0;
            if (live && q == 0) count_pairs(e);
            // sums of this wave's quarter: labels bits 0-3 by register, 4-5 per 16 points, 6 and up per 64
            double accA[16], accB[4], h0[kHighBits], h1[kHighBits], tot = 0.0;
#pragma unroll
            for (int r = 0; r < 16; ++r) accA[r] = 0.0;
#pragma unroll
            for (int r = 0; r < 4; ++r) accB[r] = 0.0;
#pragma unroll
            for (int r = 0; r < kHighBits; ++r) h0[r] = h1[r] = 0.0;
            const float* const pts = tab + (size_t)q * (M >> 2) * DP;
#pragma unroll 1
            for (int blk = 0; blk < (M >> 8); ++blk) {
                double bt = 0.0;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    double T = lane_tree<16>([&](int r) {
                        const float t = fmaf(-b.c, sqdist<DP>(y, pts + (size_t)(blk * 64 + g * 16 + r) * DP), b.K);
                        const double w = wide_exp2(t);
                        accA[r] += w;
                        return w;
                    });
                    asm volatile("" : "+v"(T)::"memory");  // the next group's points are read here, not before
                    accB[g] += T;
                    bt += T;
                }
                tot += bt;
#pragma unroll
                for (int p = 0; p < kHighBits; ++p) {
                    if ((blk >> p) & 1) h1[p] += bt;
                    else h0[p] += bt;
                }
            }
            gt[q * 64 + lane] = tot;
            double gc = 0.0, mc = 0.0;
            uint32_t left = 0u;  // flagged bits out of range here
            auto finish = [&](int p, double s0, double s1) {
                if (!((mask >> p) & 1u)) return;
                if (!wide_ok(s0, s1)) {
                    left |= 1u << p;
                    return;
                }
                const float L = wide_log2_ratio(s1, s0);
                if (b.llr) b.llr[(size_t)e.n * m + (m - 1 - p)] = L * 0.69314718055994531f;
                if (b.tx) gc += (double)gmi_bit_term(L, (txl >> p) & 1);
            };
            // bits below the quarter, kRound at a time: the wave's partial sums of each go to LDS, wave q
            // adds up and finishes bit p0 + q
#pragma unroll
            for (int p0 = 0; p0 < 6 + kHighBits; p0 += kRound) {
                if (p0 >= ml) break;
#pragma unroll
                for (int j = 0; j < kRound; ++j) {
                    const int p = p0 + j;
                    double s0 = 0.0, s1 = 0.0;
                    if (p < 4) {  // the eight registers of each side
                        const int low = (1 << p) - 1;
                        s0 = lane_tree<8>([&](int i) { return accA[((i & ~low) << 1) | (i & low)]; });
                        s1 = lane_tree<8>([&](int i) { return accA[((i & ~low) << 1) | (i & low) | (1 << p)]; });
                    } else if (p < 6) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            if ((r >> (p - 4)) & 1) s1 += accB[r];
                            else s0 += accB[r];
                        }
                    } else {
                        s0 = h0[p - 6];
                        s1 = h1[p - 6];
                    }
                    gx[((q * kRound + j) * 2 + 0) * 64 + lane] = s0;
                    gx[((q * kRound + j) * 2 + 1) * 64 + lane] = s1;
                }
                __syncthreads();
                if (p0 + q < ml) {
                    double s0 = 0.0, s1 = 0.0;
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        s0 += gx[((w * kRound + q) * 2 + 0) * 64 + lane];
                        s1 += gx[((w * kRound + q) * 2 + 1) * 64 + lane];
                    }
                    finish(p0 + q, s0, s1);
                }
                __syncthreads();
            }
            // the quarter's two bits and the MI term, from the totals
            const double t0 = gt[lane], t1 = gt[64 + lane], t2 = gt[128 + lane], t3 = gt[192 + lane];
            if (q == 1) finish(m - 2, t0 + t2, t1 + t3);
            if (q == 2) finish(m - 1, t0 + t1, t2 + t3);
            if (q == 3 && (mask & kMiFlag) && b.tx) {
                const double all = (t0 + t1) + (t2 + t3);
                if (wide_ok(all, all)) {
                    const float ttx = fmaf(-b.c, sqdist<DP>(y, tab + (size_t)txl * DP), b.K);
                    mc += (double)wide_mi(m, all, ttx);
                } else {
                    left |= kMiFlag;
                }
            }
            if (live) {
                add(e.tag, 0, gc);
                add(e.tag, 1, mc);
            }
            for (uint64_t todo = __ballot(left != 0u); todo; todo &= todo - 1) {  // uniform over the wave
                const int src = __ffsll((unsigned long long)todo) - 1;
                FixEntry o;
                o.n = (uint32_t)__builtin_amdgcn_readlane((int)e.n, src);
                o.tag = (uint32_t)__builtin_amdgcn_readlane((int)e.tag, src);
                o.mask = (uint32_t)__builtin_amdgcn_readlane((int)left, src);
                double og = 0.0, om = 0.0;
                fixup_wave<DP>(view(o), k, o.n, o.mask, nullptr, 0, og, om);
                if (lane == 0) {
                    add(o.tag, 0, og);
                    add(o.tag, 1, om);
                }
            }
            __syncthreads();  // the totals are read before the next batch overwrites them
        }
    }
    __syncthreads();
    const int bslot = (int)(blockIdx.x % kAccSlots);
    if (k.acc)
        for (int i = tid; i < kMaxSnrPerLaunch * 2; i += kThreads)
            if (s_acc[i] != 0ull) atomicAdd(k.acc + ((size_t)(i >> 1) * kAccSlots + bslot) * 2 + (i & 1), s_acc[i]);
    if (k.fix_pairs)
        for (int i = tid; i < kMaxSnrPerLaunch; i += kThreads)
            if (s_pairs[i] != 0u) atomicAdd(k.fix_pairs + i, s_pairs[i]);
}

template <int DP>
hipError_t launch_t(const LaunchArgs& a, int cus, hipStream_t st) {
    const hipError_t e = hipFuncSetAttribute((const void*)fixup_large_kernel<DP>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBytes);
    if (e != hipSuccess) return e;
    const int64_t most = (a.N * a.n_snr + kThreads / 64 - 1) / (kThreads / 64);  // a wave per symbol
    const int grid = (int)std::min<int64_t>(cus, most);
    // Up to 24 queued symbols per CU by wavefronts: 2048 points of 8D at 21 dB, a whole call of 4096 symbols
    // 57 us, of 6000 61 us; by lanes 8192 symbols 63 us, and no less for fewer.
    hipLaunchKernelGGL(fixup_large_kernel<DP>, dim3(grid), dim3(kThreads), kLdsBytes, st, a, (uint32_t)(24 * cus));
    return hipGetLastError();
}

}  // namespace

// M is a power of two: four quarters of whole 64-point blocks.
bool fixup_large_supported(int M, int D) {
    return M >= 512 && D <= 8 && (int64_t)M * padded_dim(D) <= kTabFloats;
}

hipError_t launch_fixup_large(const LaunchArgs& a, int cus, hipStream_t st) {
    switch (padded_dim(a.D)) {
        case 1: return launch_t<1>(a, cus, st);
        case 2: return launch_t<2>(a, cus, st);
        case 3: return launch_t<3>(a, cus, st);
        case 4: return launch_t<4>(a, cus, st);
        case 5: return launch_t<5>(a, cus, st);
        case 6: return launch_t<6>(a, cus, st);
        case 7: return launch_t<7>(a, cus, st);
        case 8: return launch_t<8>(a, cus, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace dm
