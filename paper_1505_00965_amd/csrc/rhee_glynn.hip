// Randomised single-term multilevel estimator (Sec. 7 cites Rhee and
// Glynn's extra randomisation, which removes the bias of a fixed finest
// level).  Every one of the N samples draws its level L from the geometric
// law p_l ~ q^l cut at the finest grid Lc and contributes Z = Y_L / p_L, so
// E[Z] = sum_l E[Y_l] = E[P_Lc] (eq. (eq:mlmc:ident)).
//
// GPU form: one kernel draws the N levels (word i mod 4 of the Philox block
// at counter (0, i / 4, 0, stream 7), inverted against the cumulative law)
// into a per-level histogram.  fp32 paths without the twin then run every
// level in one launch of the all-levels sampler, planned on the device from
// the histogram, so the host waits once (2^22 samples, Milstein, M = 4, seven
// levels: 45 us; with the histogram read back and a launch per level 125).
// Other estimates, timed ones and any under a level shape that the caller fixed
// read the histogram back and run every level with a non-zero count on the
// ordinary sampler's samples 0 .. n_l - 1, one launch each.  The host forms
//   estimate = (1/N) sum_l S1_l / p_l,  E[Z^2] = (1/N) sum_l S2_l / p_l^2.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>

#include "context.hpp"
#include "philox.hpp"

namespace mlmc {

constexpr int kRgLevels = 16;

// Levels above l are drawn by the words x with (x >> 8) >= T[l]: the uniform
// ((x >> 8) + 1/2) 2^-24 is at least the cumulative probability F_l exactly
// when the integer is at least T_l = ceil(F_l 2^24 - 1/2).
struct RgLaw {
    uint32_t T[kRgLevels];
    int Lc;
};

// The counts of "above l" come from wave ballots, word by word until no lane
// is above (most draws stop at level 0): an LDS counter per level serialised
// the lanes that hit the same one (4e6 draws: 33 us, now 12.5).
__global__ __launch_bounds__(1024) void level_draw_kernel(uint64_t seed, uint64_t N, RgLaw law,
                                                          unsigned long long* counts)
{
    __shared__ unsigned long long above[kRgLevels + 1];   // [l + 1]: draws above l; [0]: all
    if (threadIdx.x <= kRgLevels) above[threadIdx.x] = 0;
    __syncthreads();
    const uint64_t nblk = (N + 3) / 4, stride = (uint64_t)gridDim.x * blockDim.x;
    uint32_t c[kRgLevels] = {}, all = 0;                   // wave-uniform
    const uint64_t wave0 = blockIdx.x * (uint64_t)blockDim.x + (threadIdx.x & ~63u);
    for (uint64_t b0 = wave0; b0 < nblk; b0 += stride) {   // whole waves
        const uint64_t b = b0 + (threadIdx.x & 63);
        const u32x4 w = path_block(make_path_key(seed, 0, b, kStreamLevelDraw), 0);
        const uint32_t words[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const bool in = 4 * b + k < N;
            const uint32_t x = words[k] >> 8;
            all += (uint32_t)__popcll(__ballot(in));
#pragma unroll
            for (int l = 0; l < kRgLevels - 1; ++l) {
                if (l >= law.Lc) break;                    // uniform
                const uint64_t m = __ballot(in && x >= law.T[l]);
                if (!m) break;
                c[l] += (uint32_t)__popcll(m);
            }
        }
    }
    if ((threadIdx.x & 63) == 0) {
        atomicAdd(&above[0], (unsigned long long)all);
#pragma unroll
        for (int l = 0; l < kRgLevels - 1; ++l)
            if (c[l]) atomicAdd(&above[l + 1], (unsigned long long)c[l]);
    }
    __syncthreads();
    if (threadIdx.x < kRgLevels) {
        const unsigned long long n = above[threadIdx.x] - above[threadIdx.x + 1];
        // adds to one line serialise at ~3 ns: a copy for every eighth block
        if (n) atomicAdd(&counts[(blockIdx.x % kCountCopies) * kRgLevels + threadIdx.x], n);
    }
}

// The estimator's form with a launch per level.
static mlmc_status run_levels(mlmc_ctx* ctx, const mlmc_model& m, const mlmc_payoff& p, int L, int M, uint64_t seed,
                              int precision, unsigned long long* counts, uint64_t* N)
{
    // the counts alone, published
    mlmc_status st = publish_groups(ctx, ctx->d_acc, 0, counts, false);
    if (st) return st;
    counts_published(ctx);
    for (int l = 0; l <= L; ++l) N[l] = ctx->h_pub->count[l];
    static_assert(kRgLevels * kSpread <= kAccSlots, "one spread group per level");
    int clean = 0;
    st = claim_records(ctx, L + 1, &clean);
    for (int l = 0; l <= L && !st; ++l) {
        if (!N[l]) continue;
        st = enqueue_level(ctx, m, p, l, M, N[l], seed, 0, precision, kStreamNormal, 1,
                           ctx->d_acc + l * kSpread, nullptr, nullptr, nullptr);
    }
    if (!st) st = publish_groups(ctx, ctx->d_acc, L + 1, nullptr, false);
    if (!st) release_records(ctx, L + 1, clean);
    return st;
}

}  // namespace mlmc

using namespace mlmc;

extern "C" {

mlmc_status mlmc_rhee_glynn(mlmc_ctx* ctx, const mlmc_model* model, const mlmc_payoff* payoff,
                            int M, int L_cap, double q, uint64_t N, uint64_t seed, int precision,
                            mlmc_rg_result* out)
{
    if (!ctx) return MLMC_EINVAL;
    if (!out) return fail(ctx, MLMC_EINVAL, "out must not be NULL");
    mlmc_status st = check_level_args(ctx, model, payoff, L_cap, M, precision);
    if (st) return st;
    if (L_cap >= kRgLevels) return fail(ctx, MLMC_EINVAL, "L_cap must be at most 15");
    if (!(q > 0.0 && q < 1.0)) return fail(ctx, MLMC_EINVAL, "q must lie in (0, 1)");
    if (N == 0 || N > (1ull << 40)) return fail(ctx, MLMC_EINVAL, "N must be in 1..2^40");
    ctx->err.clear();
    const auto t0 = std::chrono::steady_clock::now();
    MLMC_ENTER(ctx);
    std::memset(out, 0, sizeof(*out));
    // the law and its cumulative sums, in the same order as the oracle's
    RgLaw law;
    const double norm = 1.0 - std::pow(q, (double)(L_cap + 1));
    double acc = 0.0;
    for (int l = 0; l <= L_cap; ++l) {
        out->p[l] = (1.0 - q) * std::pow(q, (double)l) / norm;
        acc += out->p[l];
        // every word is below 2^24: level L_cap takes what is left
        law.T[l] = (uint32_t)std::max(0.0, std::min(std::ceil(std::ldexp(acc, 24) - 0.5), 16777216.0));
    }
    for (int l = L_cap; l < kRgLevels; ++l) law.T[l] = 1u << 24;
    law.Lc = L_cap;
    unsigned long long* d_counts = nullptr;
    st = level_counts(ctx, &d_counts);
    if (st) return st;
    const uint64_t nblk = (N + 3) / 4;
    // a block per compute unit: each adds its counts once
    const unsigned grid = (unsigned)std::min<uint64_t>((nblk + 1023) / 1024, (uint64_t)ctx->num_cu);
    hipLaunchKernelGGL(level_draw_kernel, dim3(grid), dim3(1024), 0, ctx->stream, seed, N, law, d_counts);
    MLMC_HIP(ctx, hipGetLastError());
    // stamped launches and a fixed level shape belong to the per-level form
    if (precision == 32 && !model->antithetic && !ctx->launch_block && !(ctx->timing && !ctx->timing_paused)) {
        st = run_counts(ctx, *model, *payoff, L_cap, M, seed, d_counts);
        for (int l = 0; l <= L_cap; ++l) out->N[l] = ctx->h_pub->count[l];
    } else {
        st = run_levels(ctx, *model, *payoff, L_cap, M, seed, precision, d_counts, out->N);
    }
    if (st) return st;
    double z1 = 0.0, z2 = 0.0;
    for (int l = 0; l <= L_cap; ++l) {
        if (!out->N[l]) continue;
        const double* sum = ctx->h_pub->sum[l];
        out->sum_y[l] = sum[0];
        out->sum_y2[l] = sum[1];
        out->n_nonfinite += ctx->h_pub->n_nonfinite[l];
        out->cost += (double)out->N[l] * level_cost(*model, l, M);
        z1 += sum[0] / out->p[l];
        z2 += sum[1] / (out->p[l] * out->p[l]);
    }
    out->L_cap = L_cap;
    out->estimate = z1 / (double)N;
    out->variance = z2 / (double)N - out->estimate * out->estimate;
    out->rmse_est = std::sqrt(std::max(out->variance, 0.0) / (double)N);
    out->wall_s = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    if (out->n_nonfinite)
        return fail(ctx, MLMC_ENONFINITE, "non-finite samples were left out of the sums");
    return MLMC_OK;
}

}  // extern "C"
