// Geometric-shaping search driven by the AWGN GMI (Sec. 5): starting from a given constellation,
// each iteration proposes K candidates, each either the baseline with one randomly chosen point
// moved by Gaussian noise or with the labels of two randomly chosen points swapped, rescaled to
// unit energy per two dimensions; the candidates' GMIs are estimated in one batched launch on a
// common transmitted block and noise draw, and the best candidate replaces the baseline if its
// GMI is higher.  The paper evaluates one modification per iteration; evaluating K at once and
// keeping the best is the data-parallel form of the same greedy acceptance rule.
//
// Device side: one allocation holds the K candidates' point tables (label order, identity
// labelling, row stride 8), rewritten by one copy from pinned memory per iteration; the K received
// blocks are regenerated by gs_channel_kernel, and one FP32 batched plan (hipGraph) runs over the K
// instances.  An iteration waits for the GPU once, for the GMIs.  (With a constellation object
// per candidate, each rewriting its own tables with synchronous copies, 64 copies took 0.9 of the
// 1.0 ms of an iteration of 32 candidates.)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "api_internal.hpp"
#include "kernels.hpp"

namespace {

constexpr int kMaxCand = 64;

struct GsChannelArgs {
    const float* table;  // K label-order tables, row stride 8, table_stride floats apart
    float* y;            // K received blocks (N x D), y_stride floats apart
    const uint16_t* tx;  // N transmitted labels
    const float* z;      // N x D unit-variance noise
    int64_t N, table_stride, y_stride;
    int D, M, K;
    double s;            // noise standard deviation
};

// y_k[n][d] = fl32(x_k[tx_n][d] + s z[n][d]), one FP64 multiply-add.  One symbol per thread, all
// its candidates: tx and z are read once, and the writes of a wave are contiguous.  An
// out-of-range tx reads row 0 here; the GMI launch that follows reports it as an error.
__global__ __launch_bounds__(256) void gs_channel_kernel(const GsChannelArgs a) {
    // grid: x over the symbols, y over groups of candidates
    const int per = (a.K + gridDim.y - 1) / gridDim.y;
    const int k0 = blockIdx.y * per, k1 = min(a.K, k0 + per);
    for (int64_t n = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; n < a.N; n += (int64_t)gridDim.x * blockDim.x) {
        uint32_t row = a.tx[n];
        if (row >= (uint32_t)a.M) row = 0;
        double zs[8];
#pragma unroll
        for (int d = 0; d < 8; ++d) zs[d] = d < a.D ? (double)a.z[n * a.D + d] : 0.0;
        for (int k = k0; k < k1; ++k) {
            const float* x = a.table + k * a.table_stride + (size_t)row * 8;
            float* o = a.y + k * a.y_stride + n * a.D;
#pragma unroll
            for (int d = 0; d < 8; ++d)
                if (d < a.D) o[d] = (float)__builtin_fma(a.s, zs[d], (double)x[d]);
        }
    }
}

// SplitMix64 (Steele, Lea and Flood, 2014) and draws built on it.
struct SplitMix64 {
    uint64_t s;
    uint64_t next() {
        uint64_t z = (s += 0x9E3779B97F4A7C15ull);
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        return z ^ (z >> 31);
    }
    double uniform() { return (double)(next() >> 11) * 0x1.0p-53; }  // [0, 1)
    int below(int n) { return (int)(uniform() * n); }
    double normal() {  // Box-Muller, u1 in (0, 1]
        const double u1 = 1.0 - uniform(), u2 = uniform();
        return std::sqrt(-2.0 * std::log(u1)) * std::cos(6.283185307179586 * u2);
    }
};

void normalise(std::vector<double>& t, int M, int D) {
    double e = 0.0;
    for (double v : t) e += v * v;
    const double scale = std::sqrt((D / 2.0) / (e / M));
    for (double& v : t) v *= scale;
}

struct GsState {
    std::vector<dm_constellation*> cons;
    float *tables = nullptr, *ys = nullptr;  // K tables, K received blocks
    uint16_t* ident = nullptr;
    float* h_tables = nullptr;               // pinned
    dm_plan* plan = nullptr;
    ~GsState() {
        if (plan) dm_plan_destroy(plan);
        for (auto* c : cons) dm_constellation_destroy(c);
        (void)hipFree(tables);
        (void)hipFree(ys);
        (void)hipFree(ident);
        if (h_tables) (void)hipHostFree(h_tables);
    }
};

}  // namespace

extern "C" {

int dm_gs_optimize(const float* points, const uint16_t* labels, int32_t M, int32_t D, const dm_gs_config* cfg,
                   const uint16_t* tx, const float* z, int64_t N, float* out_points, double* gmi_trace,
                   int32_t* accepted, void* stream) {
    dmapi::clear_error();
    using dmapi::fail;
    if (!points || !labels || !cfg || !tx || !z || !out_points || !gmi_trace) return fail(DM_EINVAL, "null argument");
    if (M < 2 || (M & (M - 1)) || M > 4096) return fail(DM_EINVAL, "M=%d must be a power of two in [2, 4096]", M);
    if (D < 1 || D > 8) return fail(DM_EUNSUPPORTED, "the shaping search supports 1 <= D <= 8 (D=%d)", D);
    const int K = cfg->candidates;
    if (K < 1 || K > kMaxCand) return fail(DM_EINVAL, "candidates=%d outside [1, %d]", K, kMaxCand);
    if (cfg->iters < 0) return fail(DM_EINVAL, "iters < 0");
    if (!(cfg->perturb_sd >= 0.0) || !(cfg->swap_prob >= 0.0 && cfg->swap_prob <= 1.0) || !std::isfinite(cfg->snr_db))
        return fail(DM_EINVAL, "perturb_sd must be >= 0, swap_prob in [0, 1], snr_db finite");
    if (N < 1 || N >= (int64_t(1) << 31)) return fail(DM_EINVAL, "N=%lld out of range", (long long)N);
    std::vector<int> row_of(M, -1);
    for (int j = 0; j < M; ++j) {
        if (labels[j] >= (uint32_t)M || row_of[labels[j]] >= 0) return fail(DM_EINVAL, "labels are not a bijection");
        row_of[labels[j]] = j;
    }
    const double sigma2 = 1.0 / (2.0 * std::pow(10.0, cfg->snr_db / 10.0));
    hipStream_t st = (hipStream_t)stream;
    int dev = 0;
    DM_HIP_TRY(hipGetDevice(&dev));
    int r;
    if ((r = dmapi::check_device_ptr(tx, "tx", dev)) || (r = dmapi::check_device_ptr(z, "z", dev))) return r;

    // baseline in label order, FP64, unit energy per 2D
    std::vector<double> base((size_t)M * D);
    for (int l = 0; l < M; ++l)
        for (int d = 0; d < D; ++d) base[(size_t)l * D + d] = points[(size_t)row_of[l] * D + d];
    normalise(base, M, D);
    std::vector<uint16_t> ident(M);
    for (int l = 0; l < M; ++l) ident[l] = (uint16_t)l;

    GsState g;
    // tables and received blocks start on 256-byte boundaries
    const int64_t table_stride = ((int64_t)M * 8 + 63) / 64 * 64, y_stride = (N * D + 63) / 64 * 64;
    const size_t table_bytes = sizeof(float) * (size_t)table_stride * K;
    if (hipMalloc(&g.tables, table_bytes) != hipSuccess || hipMalloc(&g.ident, sizeof(uint16_t) * M) != hipSuccess ||
        hipMalloc(&g.ys, sizeof(float) * (size_t)y_stride * K) != hipSuccess ||
        hipHostMalloc((void**)&g.h_tables, table_bytes, hipHostMallocDefault) != hipSuccess) {
        (void)hipGetLastError();
        return fail(DM_ENOMEM, "allocation of the candidates' tables and received blocks failed");
    }
    std::memset(g.h_tables, 0, table_bytes);
    // Candidate k's table into the staging buffer.
    auto stage = [&](int k, const std::vector<double>& t) -> int {
        float* h = g.h_tables + k * table_stride;
        for (int l = 0; l < M; ++l)
            for (int d = 0; d < D; ++d) {
                const float v = (float)t[(size_t)l * D + d];
                if (!std::isfinite(v) || std::fabs(v) > 1e15f)
                    return fail(DM_EINVAL, "point coordinate is not finite or exceeds 1e15");
                h[(size_t)l * 8 + d] = v;
            }
        return DM_OK;
    };
    for (int k = 0; k < K; ++k)
        if ((r = stage(k, base))) return r;
    DM_HIP_TRY(hipMemcpy(g.ident, ident.data(), sizeof(uint16_t) * M, hipMemcpyHostToDevice));
    int m = 0, cus = 0;
    while ((1 << m) < M) ++m;
    DM_HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    g.cons.assign(K, nullptr);
    std::vector<dm_instance> inst(K);
    for (int k = 0; k < K; ++k) {  // views of the shared tables: all that an FP32 plan reads
        auto* c = new (std::nothrow) dm_constellation();
        if (!c) return fail(DM_ENOMEM, "host allocation failed");
        g.cons[k] = c;
        c->M = M;
        c->D = D;
        c->m = m;
        c->DP = dm::padded_dim(D);
        c->device = dev;
        c->cus = cus;
        c->borrowed = true;
        c->d_table8 = g.tables + k * table_stride;
        c->d_row2label = g.ident;
        inst[k] = dm_instance{c, sigma2, g.ys + k * y_stride, tx, N, nullptr};
    }
    if ((r = dm_plan_create(inst.data(), K, DM_PREC_FP32, DM_PLAN_FORCE_VALU, &g.plan))) return r;

    GsChannelArgs ca;
    std::memset(&ca, 0, sizeof ca);
    ca.table = g.tables;
    ca.y = g.ys;
    ca.tx = tx;
    ca.z = z;
    ca.N = N;
    ca.table_stride = table_stride;
    ca.y_stride = y_stride;
    ca.D = D;
    ca.M = M;
    ca.K = K;
    ca.s = std::sqrt(sigma2);
    // about 8 blocks per CU: the candidates are split where the symbols alone give fewer
    const int gx = (int)std::min<int64_t>((N + 255) / 256, (int64_t)cus * 8);
    const int gy = std::max(1, std::min(K, cus * 8 / gx));
    std::vector<double> gmi(K), mi(K);
    auto evaluate = [&]() -> int {
        DM_HIP_TRY(hipMemcpyAsync(g.tables, g.h_tables, table_bytes, hipMemcpyHostToDevice, st));
        hipLaunchKernelGGL(gs_channel_kernel, dim3(gx, gy), dim3(256), 0, st, ca);
        DM_HIP_TRY(hipGetLastError());
        int rr = dm_plan_launch(g.plan, stream);
        if (rr) return rr;
        return dm_plan_results(g.plan, gmi.data(), mi.data(), nullptr, stream);
    };
    // the baseline's own GMI on the common block (every table equals the baseline here)
    if ((r = evaluate())) return r;
    double cur = gmi[0];
    gmi_trace[0] = cur;
    int32_t acc = 0;
    SplitMix64 rng{cfg->seed};
    std::vector<std::vector<double>> cand(K);
    for (int it = 1; it <= cfg->iters; ++it) {
        for (int k = 0; k < K; ++k) {
            cand[k] = base;
            if (rng.uniform() < cfg->swap_prob) {
                const int a = rng.below(M);
                int b = rng.below(M - 1);
                if (b >= a) ++b;
                for (int d = 0; d < D; ++d) std::swap(cand[k][(size_t)a * D + d], cand[k][(size_t)b * D + d]);
            } else {
                const int a = rng.below(M);
                for (int d = 0; d < D; ++d) cand[k][(size_t)a * D + d] += cfg->perturb_sd * rng.normal();
                normalise(cand[k], M, D);
            }
            if ((r = stage(k, cand[k]))) return r;
        }
        if ((r = evaluate())) return r;
        int best = 0;
        for (int k = 1; k < K; ++k)
            if (gmi[k] > gmi[best]) best = k;
        if (gmi[best] > cur) {
            cur = gmi[best];
            base = cand[best];
            ++acc;
        }
        gmi_trace[it] = cur;
    }
    for (size_t i = 0; i < base.size(); ++i) out_points[i] = (float)base[i];
    if (accepted) *accepted = acc;
    return DM_OK;
}

}  // extern "C"
