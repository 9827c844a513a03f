// Kernels of the learned demapper: an MLP (D+1) -> H -> H -> m with GELU, BF16 weights and
// activations, FP32 accumulation on v_mfma_f32_32x32x16_bf16 (gfx950).
//
// A training step is three launches:
//   train_pass_kernel   forward and backward of 32 samples per workgroup.  Wave w owns hidden units
//                       32 w .. 32 w + 31 of both hidden layers: their pre-activations stay in its
//                       registers from the forward to the backward pass, activations and deltas
//                       pass between the layers through LDS, and every matrix that the weight
//                       gradients read goes out in MFMA operand order;
//   weight_grad_kernel  the three weight gradients, one wavefront per 32 x 32 tile and K split
//                       (K = the batch), and the bias gradients (row sums over the batch);
//   adam_kernel         sums the K splits in a fixed order (deterministic), updates the FP32 master
//                       weights and rewrites their BF16 copies.
// It was sixteen launches, one GEMM per layer, with activations written twice (row-major and
// transposed, two bytes a lane) and read back: 139 us per step of 4096 samples, most of it launch
// gaps and partial-line stores.  Now 36 us: 14.7 + 10 + 5.3 us of kernels and the gaps.  Every
// product and sum keeps its operands and its order, so the results are the same bit for bit.
//
// Activations and back-propagated deltas are stored as BF16 pairs hi + lo (lo = the rounding
// remainder, about 16 significant bits together) and enter every product that reads them as
// such: hi.b + lo.b, or hi.hi + hi.lo + lo.hi when both operands are pairs.  Only the weights
// (BF16 copies of the FP32 masters) and the network inputs are single BF16 words, so the
// gradients are those of the network on BF16-rounded weights and inputs, with activations and
// deltas carried to about 2^-16 relative instead of BF16's 2^-8.
//
// Operand order ("fragments"): a matrix of rows by K columns is stored as [32-row tile][16-column
// step][lane][8], lane l holding row l % 32 and the 8 columns starting at 8 (l / 32), so that a wave
// reads an MFMA operand as one contiguous KiB.  The weights' BF16 copies have that order; the
// matrices over the batch (rows = units or inputs, columns = samples, the K dimension of a weight
// gradient) have it with [hi, lo] between step and lane.
#include <hip/hip_runtime.h>

#include "mlp_kernels.hpp"

namespace dm {

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

__device__ __forceinline__ float rcp_f(float x) { return __builtin_amdgcn_rcpf(x); }

__device__ __forceinline__ float gelu_f(float x) {
    // 0.5 x (1 + tanh(u)) = x * sigmoid(2u), u = sqrt(2/pi) (x + 0.044715 x^3)
    const float u2 = 1.5957691216057308f * x * fmaf(0.044715f, x * x, 1.0f);
    return x * rcp_f(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * u2));
}

__device__ __forceinline__ float gelu_grad_f(float x) {
    const float x2 = x * x;
    const float u2 = 1.5957691216057308f * x * fmaf(0.044715f, x2, 1.0f);  // 2u
    const float s = rcp_f(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * u2));  // sigmoid(2u)
    // d/dx [x sigmoid(2u)] = s + x s (1 - s) d(2u)/dx,  d(2u)/dx = 2 sqrt(2/pi) (1 + 3 * 0.044715 x^2)
    return s + x * s * (1.0f - s) * 1.5957691216057308f * fmaf(0.134145f, x2, 1.0f);
}

__device__ __forceinline__ float sigmoid_f(float x) { return rcp_f(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * x)); }

__device__ __forceinline__ float softplus_f(float x) {
    return fmaxf(x, 0.0f) + 0.69314718055994531f * __builtin_amdgcn_logf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * fabsf(x)));
}

typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;

// Two values as BF16 pairs hi = bf16(v), lo = bf16(v - hi) (the difference is exact in FP32), packed
// in one word each.  The values are pinned in registers: the compiler would otherwise fold the
// products that they come from into the subtractions and take lo from the unrounded products.
__device__ __forceinline__ void bf16_pairs(float v0, float v1, uint32_t& hi, uint32_t& lo) {
    asm("" : "+v"(v0), "+v"(v1));
    hi = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)v0, (__bf16)v1});
    const float f0 = __builtin_bit_cast(float, hi << 16), f1 = __builtin_bit_cast(float, hi & 0xFFFF0000u);
    lo = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)(v0 - f0), (__bf16)(v1 - f1)});
}

__device__ __forceinline__ f32x16 mma(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ bf16x8 load8(const __bf16* p) { return *reinterpret_cast<const bf16x8*>(p); }
__device__ __forceinline__ bf16x8 load8(const uint16_t* p) { return *reinterpret_cast<const bf16x8*>(p); }

// Workgroup barrier for data in LDS only: unlike __syncthreads it does not wait for global loads and
// stores in flight (the next layer's weights, the operands written for weight_grad_kernel).
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Row (sample) of MFMA result register q in lane half h.
__device__ __forceinline__ int result_row(int q, int h) { return 8 * (q >> 2) + 4 * h + (q & 3); }

constexpr int kPassThreads = 512;          // 8 waves: one per 32 hidden units
constexpr int kHidden = 256;
constexpr int kActLd = kHidden + 8;        // LDS row stride of an activation tile (16-byte rows, no bank conflicts)
constexpr int kOutLd = 32 + 8;

// A 32-sample tile in LDS, hi and lo words, row-major by sample.
template <int LD>
struct alignas(16) Tile {
    alignas(16) uint16_t hi[32 * LD];
    alignas(16) uint16_t lo[32 * LD];
};

// Store one wave's 32 x 32 result (lane = column j of the tile's columns, registers = samples) as
// pairs: into an LDS tile (LDS; for the next layer's A operand) and, in fragment order, to global
// memory.  A lane's registers 4g .. 4g+3 are samples 8g + 4h .. + 3; swapping the halves' packed
// words (g even for the lower half, odd for the upper) gives each lane 8 consecutive samples.
template <bool LDS, int LD>
__device__ __forceinline__ void store_pairs(const float (&v)[16], int col, int lane, Tile<LD>& tile, __bf16* frag) {
    const int h = lane >> 5;
    uint32_t w[2][8];  // [hi, lo][2 g + pair]: samples 8g + 4h + 2 pair, + 1
#pragma unroll
    for (int q = 0; q < 16; q += 2) {
        uint32_t& hw = w[0][q >> 1];
        uint32_t& lw = w[1][q >> 1];
        bf16_pairs(v[q], v[q + 1], hw, lw);
        if constexpr (LDS) {
            const int r = result_row(q, h);
            tile.hi[r * LD + col] = (uint16_t)hw;
            tile.lo[r * LD + col] = (uint16_t)lw;
            tile.hi[(r + 1) * LD + col] = (uint16_t)(hw >> 16);
            tile.lo[(r + 1) * LD + col] = (uint16_t)(lw >> 16);
        }
    }
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            // samples 16 s ..: registers' groups g = 2 s (words 4 s, 4 s + 1) and g = 2 s + 1
            const auto x = __builtin_amdgcn_permlane32_swap(w[k][4 * s], w[k][4 * s + 2], false, false);
            const auto y = __builtin_amdgcn_permlane32_swap(w[k][4 * s + 1], w[k][4 * s + 3], false, false);
            *reinterpret_cast<uint4*>(frag + (s * 2 + k) * 512 + lane * 8) = uint4{x[0], y[0], x[1], y[1]};
        }
}

// Sample tile of workgroup b out of T = B / 32: workgroups b, b + 8, .. run on one XCD (round robin),
// whose L2 then holds the operands of the batch's K splits (sixteenths of the batch) that
// weight_grad_kernel reads on the same XCD.
__device__ __forceinline__ int sample_tile(int b, int T) {
    if (T % 16) return b;
    const int per = T / 16, n = b >> 3;
    return ((b & 7) + 8 * (n / per)) * per + n % per;
}

// Forward and backward of 32 samples; B / 32 workgroups.  Wave w computes unit columns 32 w .. of
// both hidden layers, wave 0 the output layer.  Weights are read straight from L2 in operand
// order, a whole layer's ahead of the barrier that its inputs wait for; LDS holds two activation
// tiles and the output deltas.  The output layer is one chain of MFMAs on wave 0; its losses and
// deltas (eight transcendentals a value) are spread over all waves through LDS.
// Bound: the latency of the chain, not a rate: of 25,000 cycles (128 workgroups at a batch of 4096)
// 10,000 go by before layer 2 has its inputs and weights (128 KiB of them per workgroup and layer
// out of L2), 6,600 in layer 2, 3,900 in the output layer's 32 dependent MFMAs and its losses.
__global__ __launch_bounds__(kPassThreads) void train_pass_kernel(const TrainPassArgs a) {
    __shared__ Tile<kActLd> act[2];
    __shared__ Tile<kOutLd> dout;
    __shared__ float outs[16][64], losses[16][64];  // [result register][lane] of the output layer
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 31, h = lane >> 5;
    const int tile = sample_tile(blockIdx.x, a.B / 32), m0 = 32 * tile;
    const int j = 32 * wave + r;  // this lane's hidden unit (both layers)
    const size_t steps = (size_t)a.B / 16;
    // fragment base of row tile t, samples m0 ..
    auto frag_at = [&](__bf16* f, int t) { return f + ((size_t)t * steps + 2 * tile) * 1024; };
    // the 16 operands (K = 256) of weight row tile t
    auto load_w = [&](const __bf16* w, int t, bf16x8 (&f)[16]) {
#pragma unroll
        for (int k = 0; k < 16; ++k) f[k] = load8(w + (size_t)(t * 16 + k) * 512 + lane * 8);
    };
    // acc = tile . w^T over K = 256, low words first in every step
    auto gemm256 = [&](const Tile<kActLd>& t, const bf16x8 (&w)[16]) {
        f32x16 acc = {};
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int o = r * kActLd + 16 * k + 8 * h;
            acc = mma(load8(t.lo + o), w[k], acc);
            acc = mma(load8(t.hi + o), w[k], acc);
        }
        return acc;
    };

    // ---- inputs: X[b][0..D) = y, X[b][D] = SNR feature, rest 0, as BF16 ----
    // The SNR feature is (s - 7.5) / 7.5 with s = -10 log10(2 sigma2), the SNR in dB at unit energy
    // per two dimensions: -10 log10(2 s2) = -(10 / log2(10)) (1 + log2 s2).
    auto feature = [&](float s2) {
        const float snr_db = -3.0102999566398120f * (1.0f + __builtin_amdgcn_logf(s2));
        return (snr_db - 7.5f) * (1.0f / 7.5f);
    };
    bf16x8 wf[16];
    const bf16x8 w1 = load8(a.W1t + (size_t)wave * 1024 + lane * 8);
    // (loads with clamped indices, selected at use: a load under a branch is waited for at once)
    float yv[8], yt[8], st[8];
    const float s2 = a.sigma2[m0 + r];
#pragma unroll
    for (int q = 0; q < 8; ++q) yv[q] = a.y[(size_t)(m0 + r) * a.D + min(8 * h + q, a.D - 1)];
    if (wave < 2) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int b = m0 + 16 * wave + 8 * h + q;
            yt[q] = a.y[(size_t)b * a.D + min(r, a.D - 1)];
            st[q] = a.sigma2[b];
        }
    }
    load_w(a.W2t, wave, wf);
    const float b1 = a.b1[j], b2 = a.b2[j];
    bf16x8 x;
    {
        const float sf = feature(s2);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int k = 8 * h + q;
            x[q] = (__bf16)(k < a.D ? yv[q] : k == a.D ? sf : 0.0f);
        }
    }
    if (wave < 2) {  // the transposed inputs (rows 16..31 zero) for the layer-1 weight gradient
        bf16x8 xt;
#pragma unroll
        for (int q = 0; q < 8; ++q) xt[q] = (__bf16)(r < a.D ? yt[q] : r == a.D ? feature(st[q]) : 0.0f);
        *reinterpret_cast<bf16x8*>(a.Xf + ((size_t)2 * tile + wave) * 512 + lane * 8) = xt;
    }

    // ---- layer 1 ----
    float h1[16], h2[16], v[16];
    {
        const f32x16 acc = mma(x, w1, f32x16{});
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            h1[q] = acc[q] + b1;
            v[q] = gelu_f(h1[q]);
        }
        store_pairs<true>(v, j, lane, act[0], frag_at(a.A1f, wave));
    }
    lds_barrier();

    // ---- layer 2 ----
    {
        const f32x16 acc = gemm256(act[0], wf);
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            h2[q] = acc[q] + b2;
            v[q] = gelu_f(h2[q]);
        }
        store_pairs<true>(v, j, lane, act[1], frag_at(a.A2f, wave));
    }
    const bf16x8 w3a = load8(a.W3 + (size_t)wave * 1024 + lane * 8), w3b = load8(a.W3 + (size_t)wave * 1024 + 512 + lane * 8);
    if (wave == 0) load_w(a.W3t, 0, wf);
    else load_w(a.W2, wave, wf);
    // this wave's share of the outputs: registers 2 wave and 2 wave + 1, lane = output r
    float tgt[2];
#pragma unroll
    for (int e = 0; e < 2; ++e)
        tgt[e] = a.target[(size_t)(m0 + result_row(2 * wave + e, h)) * a.m + min(r, a.m - 1)];
    const float b3 = a.b3[r];
    lds_barrier();

    // ---- output layer, loss and output deltas ----
    if (wave == 0) {
        const f32x16 acc = gemm256(act[1], wf);
#pragma unroll
        for (int q = 0; q < 16; ++q) outs[q][lane] = acc[q];
        load_w(a.W2, wave, wf);
    }
    lds_barrier();
    {
        float d[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const float o = outs[2 * wave + e][lane] + b3;
            const float t = tgt[e];
            const float p = sigmoid_f(t);
            d[e] = r < a.m ? (sigmoid_f(o) - p) * a.scale : 0.0f;
            losses[2 * wave + e][lane] = r < a.m ? (softplus_f(o) - p * o) - (softplus_f(t) - p * t) : 0.0f;
        }
        uint32_t hw, lw;
        bf16_pairs(d[0], d[1], hw, lw);
        const int row = result_row(2 * wave, h);
        dout.hi[row * kOutLd + r] = (uint16_t)hw;
        dout.lo[row * kOutLd + r] = (uint16_t)lw;
        dout.hi[(row + 1) * kOutLd + r] = (uint16_t)(hw >> 16);
        dout.lo[(row + 1) * kOutLd + r] = (uint16_t)(lw >> 16);
    }
    lds_barrier();
    if (wave == 0) {  // losses in register order, then over the wave
        float loss = 0.0f;
#pragma unroll
        for (int q = 0; q < 16; ++q) loss += losses[q][lane];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) loss += __shfl_xor(loss, off, 64);
        if (lane == 0) a.loss_tiles[tile] = loss;
    } else if (wave < 5) {  // the output deltas in operand order: step (wave - 1) / 2, hi or lo
        const int s = (wave - 1) >> 1;
        const uint16_t* src = (wave & 1) ? dout.hi : dout.lo;
        uint32_t f[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = 16 * s + 8 * h + 2 * e;
            f[e] = src[row * kOutLd + r] | ((uint32_t)src[(row + 1) * kOutLd + r] << 16);
        }
        *reinterpret_cast<uint4*>(frag_at(a.dOf, 0) + (s * 2 + (wave & 1 ? 0 : 1)) * 512 + lane * 8) =
            uint4{f[0], f[1], f[2], f[3]};
    }

    // ---- back through layer 3 and GELU 2 ----
    {
        const int o = r * kOutLd + 8 * h;
        f32x16 acc = mma(load8(dout.lo + o), w3a, f32x16{});
        acc = mma(load8(dout.hi + o), w3a, acc);
        acc = mma(load8(dout.lo + o + 16), w3b, acc);
        acc = mma(load8(dout.hi + o + 16), w3b, acc);
#pragma unroll
        for (int q = 0; q < 16; ++q) v[q] = acc[q] * gelu_grad_f(h2[q]);
        store_pairs<true>(v, j, lane, act[0], frag_at(a.dH2f, wave));
    }
    lds_barrier();

    // ---- back through layer 2 and GELU 1 ----
    {
        const f32x16 acc = gemm256(act[0], wf);
#pragma unroll
        for (int q = 0; q < 16; ++q) v[q] = acc[q] * gelu_grad_f(h1[q]);
        store_pairs<false>(v, j, lane, act[0], frag_at(a.dH1f, wave));
    }
}

constexpr int kGradThreads = 256;

// One 32 x 32 tile of a weight gradient over one K split: C[i][j] = sum_b A[i][b] Bt[j][b], both in
// fragment order; hi.lo and hi.hi after lo.hi in every 16-sample step.
template <bool BLO>
__device__ __forceinline__ void grad_tile(const __bf16* A, const __bf16* Bt, int step0, int nsteps, float* out, int ldc,
                                          int lane) {
    constexpr size_t bstep = BLO ? 1024 : 512;
    const __bf16* ap = A + (size_t)step0 * 1024 + lane * 8;
    const __bf16* bp = Bt + (size_t)step0 * bstep + lane * 8;
    f32x16 acc = {};
#pragma unroll 8
    for (int k = 0; k < nsteps; ++k) {
        const bf16x8 ah = load8(ap), al = load8(ap + 512), bh = load8(bp);
        acc = mma(al, bh, acc);
        if constexpr (BLO) acc = mma(ah, load8(bp + 512), acc);
        acc = mma(ah, bh, acc);
        ap += 1024;
        bp += bstep;
    }
    const int r = lane & 31, h = lane >> 5;
#pragma unroll
    for (int q = 0; q < 16; ++q) out[(size_t)result_row(q, h) * ldc + r] = acc[q];
}

// Bias gradients are sums over the batch, hi + lo: kSums partial sums per row, partial sum t over the
// 8-sample chunks t, t + kSums, .. in order, then (row_sum) a pairwise tree over t: the order is
// fixed by the batch alone.  Here the partial sums of steps k0 .. k0 + 3 (chunks 2 k, 2 k + 1) of one
// 32-row tile.
constexpr int kSums = 256;

__device__ __forceinline__ void partial_sums(const __bf16* F, int steps, int k0, float* out, int lane) {
    const int r = lane & 31, h = lane >> 5;
    float s[4] = {};
    for (int k1 = k0; k1 < steps; k1 += kSums / 2) {
        bf16x8 v[4], l[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            v[q] = load8(F + (size_t)(k1 + q) * 1024 + lane * 8);
            l[q] = load8(F + (size_t)(k1 + q) * 1024 + 512 + lane * 8);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int e = 0; e < 8; ++e) s[q] += (float)v[q][e] + (float)l[q][e];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) out[(size_t)(2 * (k0 + q) + h) * 32 + r] = s[q];
}

// Waves of four per block: first the 2 x 2 tiles of dW2 (a quarter of the operand reads of a tile
// hit the CU's cache), then dW1 and dW3, then the bias sums of the 17 row tiles of the three
// deltas.  A K split's blocks sit on the XCD (block index modulo 8) that wrote its operands.
// Bound: operand traffic through the CUs' caches, 4 KiB per three MFMAs, and its latency.
__global__ __launch_bounds__(kGradThreads) void weight_grad_kernel(const WeightGradArgs a) {
    const size_t steps = (size_t)a.B / 16;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int b = blockIdx.x;
    if (b < 16 * a.splits2) {  // dW2[u][i]: tile (u / 32, i / 32)
        const int n = b >> 3, split = (b & 7) + 8 * (n >> 4), ns = (int)steps / a.splits2;
        const int row = 2 * ((n >> 2) & 3) + (wave >> 1), col = 2 * (n & 3) + (wave & 1);
        grad_tile<true>(a.dH2f + (size_t)row * steps * 1024, a.A1f + (size_t)col * steps * 1024, split * ns, ns,
                        a.part2 + (size_t)split * 65536 + (size_t)row * 32 * kHidden + col * 32, kHidden, lane);
        return;
    }
    b -= 16 * a.splits2;
    if (b < 4 * a.splits13) {
        // per: splits of dW1 / dW3 per sixteenth of the batch; the four blocks of a split on one XCD
        const int per = a.splits13 / 16, n = b >> 5, m = (b >> 3) & 3;
        const int split = ((b & 7) + 8 * (n / per)) * per + n % per, ns = (int)steps / a.splits13;
        const int t = 4 * (m & 1) + wave;
        if (m < 2)  // dW1[u][input]: tile u / 32
            grad_tile<false>(a.dH1f + (size_t)t * steps * 1024, a.Xf, split * ns, ns,
                             a.part1 + (size_t)split * 8192 + (size_t)t * 32 * 32, 32, lane);
        else  // dW3[o][i]: tile i / 32
            grad_tile<true>(a.dOf, a.A2f + (size_t)t * steps * 1024, split * ns, ns,
                            a.part3 + (size_t)split * 8192 + t * 32, kHidden, lane);
        return;
    }
    b -= 4 * a.splits13;
    // kSums / 2 / 16 blocks per row tile: 16 steps each, 4 per wave (batches under 2048 have fewer)
    const int t = b / (kSums / 32), k0 = 16 * (b % (kSums / 32)) + 4 * wave;
    const __bf16* F = t < 8 ? a.dH1f + (size_t)t * steps * 1024 : t < 16 ? a.dH2f + (size_t)(t - 8) * steps * 1024 : a.dOf;
    partial_sums(F, (int)steps, k0, a.sums + (size_t)t * kSums * 32, lane);
}

// Sum of row r (of 32) of a tile's partial sums over t, by one wave: pairs 32, 16, .. 1 apart within
// each 64, then the four groups.
__device__ __forceinline__ float row_sum(const float* sums, int r, int lane) {
    float p[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) p[w] = sums[(size_t)(64 * w + lane) * 32 + r];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
#pragma unroll
        for (int w = 0; w < 4; ++w) p[w] += __shfl_xor(p[w], off, 64);
    return (p[0] + p[1]) + (p[2] + p[3]);
}

// Sum of SPLITS partials of element i, in split order, every load in flight at once.
template <int SPLITS>
__device__ __forceinline__ float reduce_splits(const float* part, size_t n, size_t i) {
    float v[SPLITS], s = 0.0f;
#pragma unroll
    for (int q = 0; q < SPLITS; ++q) v[q] = part[(size_t)q * n + i];
#pragma unroll
    for (int q = 0; q < SPLITS; ++q) s += v[q];
    return s;
}

// Gradient of element i of a weight tensor of n: summed over the K splits.
__device__ __forceinline__ float reduce_element(const AdamArgs& a, size_t n, size_t i) {
    const float s = a.splits == 64   ? reduce_splits<64>(a.part, n, i)
                    : a.splits == 32 ? reduce_splits<32>(a.part, n, i)
                                     : reduce_splits<16>(a.part, n, i);
    a.grad[i] = s;
    return s;
}

// Index of element (row, col) of a matrix of `cols` columns in operand order.
__device__ __forceinline__ size_t frag_index(int row, int col, int cols) {
    return ((size_t)((row >> 5) * (cols >> 4) + (col >> 4)) * 64 + (row & 31) + 32 * ((col >> 3) & 1)) * 8 + (col & 7);
}

// Adam on one parameter element (rows x cols, row-major FP32 master), then the BF16 copies in
// operand order: copy (rows x cols) and copyT (cols x rows), either may be null.  mask_rows /
// mask_cols: entries outside [0, mask_rows) x [0, mask_cols) are padding and stay zero.
__device__ __forceinline__ void adam_element(const AdamArgs& a, size_t i, float g) {
    const int rr = (int)(i / a.cols), cc = (int)(i % a.cols);
    float w = a.w[i];
    if (rr < a.mask_rows && cc < a.mask_cols) {
        const float m = a.beta1 * a.m[i] + (1.0f - a.beta1) * g;
        const float v = a.beta2 * a.v[i] + (1.0f - a.beta2) * g * g;
        a.m[i] = m;
        a.v[i] = v;
        const float mh = m / a.bc1, vh = v / a.bc2;
        w -= a.lr * mh / (sqrtf(vh) + a.eps);
        a.w[i] = w;
    }
    if (a.copy) a.copy[frag_index(rr, cc, a.cols)] = (__bf16)w;
    if (a.copyT) a.copyT[frag_index(cc, rr, a.rows)] = (__bf16)w;
}

// Every tensor of a batch: the gradient's reduction (reduce), then the Adam step (update).  Weights take
// one element per thread, biases (splits 0) one per wave.  Tensors start at whole blocks, so a
// block's arguments are scalar loads.
constexpr int kAdamThreads = 256;

__global__ __launch_bounds__(kAdamThreads) void adam_kernel(const AdamBatch b) {
    int k = 0;
    while (k + 1 < b.count && (int)blockIdx.x >= b.first_block[k + 1]) ++k;
    const AdamArgs& a = b.t[k];
    const size_t n = (size_t)a.rows * a.cols;
    const size_t t = (size_t)(blockIdx.x - b.first_block[k]) * kAdamThreads + threadIdx.x;
    const size_t i = a.splits ? t : t >> 6;
    if (i >= n) return;  // (whole waves for a bias)
    float g = 0.0f;
    if (b.reduce) {
        if (a.splits) {
            g = reduce_element(a, n, i);
        } else {
            g = row_sum(a.part + (i >> 5) * kSums * 32, (int)(i & 31), threadIdx.x & 63);
            if ((t & 63) == 0) a.grad[i] = g;
        }
    }
    if (b.update && (a.splits || (t & 63) == 0)) adam_element(a, i, g);
}

}  // namespace

size_t mlp_sum_floats() { return (size_t)17 * kSums * 32; }

hipError_t launch_train_pass(const TrainPassArgs& a, hipStream_t st) {
    if (a.B < 256 || a.B % 256 || a.D < 1 || a.D > 13 || a.m < 1 || a.m > 32) return hipErrorInvalidValue;
    hipLaunchKernelGGL(train_pass_kernel, dim3(a.B / 32), dim3(kPassThreads), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_weight_grad(const WeightGradArgs& a, hipStream_t st) {
    // B a multiple of 256 has 16 splits of dW2 and 16, 32 or 64 of dW1 and dW3
    const int steps = a.B / 16;
    if (a.B < 256 || a.B % 256 || a.splits2 != 16 || a.splits13 % 16 || a.splits13 < 16 || a.splits13 > 64 ||
        steps % a.splits13)
        return hipErrorInvalidValue;
    const int blocks = 16 * a.splits2 + 4 * a.splits13 + 17 * (kSums / 32);
    hipLaunchKernelGGL(weight_grad_kernel, dim3(blocks), dim3(kGradThreads), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_adam_batch(AdamBatch b, hipStream_t st) {
    if (b.count < 1 || b.count > kAdamMaxTensors) return hipErrorInvalidValue;
    int blocks = 0;
    for (int k = 0; k < b.count; ++k) {
        b.first_block[k] = blocks;
        const int per_block = b.t[k].splits ? kAdamThreads : kAdamThreads / 64;
        blocks += (b.t[k].rows * b.t[k].cols + per_block - 1) / per_block;
    }
    hipLaunchKernelGGL(adam_kernel, dim3(blocks), dim3(kAdamThreads), 0, st, b);
    return hipGetLastError();
}

}  // namespace dm
