// Learned control variate: parameters, the samplers with the control variate
// and the table (training: cv_train.hip).
//
// Level estimators with the control variate (eqs. (eq:mlmc:Yzero),
// (eq:Yldef) with each payoff replaced by P - sum_n phi(t_n, X_n) dW1_n on
// its own grid): the fine path uses its fine increments, the coarse path its
// coarse (summed) increments, both evaluated at the left point of each step.
// At t = 0 every sample sits at (0, S0), so level 0 needs only the one value
// phi(0, S0), computed once per launch.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>

#include "cv_state.hpp"
#include "cv_tab.hpp"
#include "sampler_impl.hpp"

using namespace mlmc::cvnet;

namespace mlmc {

// ------------------------------------------------------------ parameters
// Xavier-uniform weights from the init stream: parameter i takes word i % 4
// of generator block i / 4 at (sample 0, level 0); biases zero.
__global__ void cv_init_kernel(float* params, int D, uint64_t seed)
{
    const int np = nparams(D);
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= np) return;
    float a = 0.0f;
    if (i < off_b1(D)) a = sqrtf(6.0f / (float)(D + H));
    else if (i >= off_W2(D) && i < off_b2(D)) a = sqrtf(6.0f / (float)(2 * H));
    else if (i >= off_w3(D) && i < off_b3(D)) a = sqrtf(6.0f / (float)(H + 1));
    if (a == 0.0f) {
        params[i] = 0.0f;
        return;
    }
    const u32x4 w = path_block(make_path_key(seed, 0, 0, kStreamInit), (uint32_t)(i / 4));
    const uint32_t word = (i % 4 == 0) ? w.x : (i % 4 == 1) ? w.y : (i % 4 == 2) ? w.z : w.w;
    params[i] = a * (2.0f * (float)u01d(word) - 1.0f);
}

// bf16 operand arrays from the fp32 W2 (round to nearest even).
__global__ void cv_prepare_kernel(const float* params, int D, bf16x8* afwd, bf16x8* abwd)
{
    const float* W2 = params + off_W2(D);
    const int t = threadIdx.x;            // 64 lanes x 8 operand sets
    for (int idx = t; idx < 8 * 64; idx += blockDim.x) {
        const int set = idx / 64, lane = idx % 64;
        const int hi = lane / 32;
        const int tile = set / 4, kb = set % 4;
        bf16x8 f, b;
        for (int i = 0; i < 8; ++i) {
            const int j = 32 * tile + lane % 32, k = 16 * kb + 8 * hi + i;
            f[i] = (__bf16)W2[j * H + k];
            b[i] = (__bf16)W2[k * H + j];    // the transposed product's operand
        }
        afwd[idx] = f;
        abwd[idx] = b;
    }
}

// Grid of the tabulated network for a model (host): 256 time rows x 32 stock
// values for GBM; 16 rows x 16 stock values x 32 variances for Heston (32 KiB
// of fp32 either way; a level's sampler copies the rows it reads into LDS).
// Stock values span S0 exp(+-4 sref sqrt T) (sref = sigma, or sqrt(theta) for
// Heston), variances [0, 4 max(theta, v0)].  The network varies slowly in S
// at these scales; Heston's variance axis and the time rows of deep levels
// decide how much of its variance reduction the table keeps.
struct TableGrid {
    int rows, ns, nv;
    double s_lo, s_hi, v_lo, v_hi;
};

static TableGrid table_grid(const mlmc_model& m)
{
    TableGrid g;
    const bool heston = m.kind == MLMC_HESTON;
    const double sref = heston ? std::sqrt(m.theta) : m.sigma;
    const double w = 4.0 * sref * std::sqrt(m.T);
    g.rows = heston ? 16 : 256;
    g.ns = heston ? 16 : 32;
    g.nv = heston ? 32 : 1;
    g.s_lo = m.S0 * std::exp(-w);
    g.s_hi = m.S0 * std::exp(w);
    g.v_lo = 0.0;
    g.v_hi = heston ? 4.0 * std::max(m.theta, m.v0) : 1.0;
    return g;
}

static TableSpec table_spec(const TableGrid& g)
{
    TableSpec t;
    t.rows = g.rows;
    t.ns = g.ns;
    t.nv = g.nv;
    t.s_lo = (float)g.s_lo;
    t.s_inv = (float)((g.ns - 1) / (g.s_hi - g.s_lo));
    t.v_lo = (float)g.v_lo;
    t.v_inv = g.nv > 1 ? (float)((g.nv - 1) / (g.v_hi - g.v_lo)) : 0.0f;
    return t;
}

static size_t table_size(const TableGrid& g) { return (size_t)g.rows * g.ns * g.nv; }

// Fill the table: point p = (row j, variance k, stock i), p = (j nv + k) ns + i,
// holds phi(j T / rows, S_i, v_k) from the network (64 points per wave
// through phi_eval; every lane of a wave evaluates, lanes past the end drop
// their value).
template <int D>
__global__ void cv_table_kernel(CvKernelArgs c, TableGrid g, float* tab)
{
    __shared__ NetShared sh;
    __shared__ bf16x8 s_afwd[8 * 64];
    load_shared<D>(sh, c.params, c.nc);
    for (int i = threadIdx.x; i < 8 * 64; i += blockDim.x) s_afwd[i] = c.afwd[i];
    __syncthreads();
    const int npts = g.rows * g.nv * g.ns;
    const double ds = (g.s_hi - g.s_lo) / (g.ns - 1);
    const double dv = g.nv > 1 ? (g.v_hi - g.v_lo) / (g.nv - 1) : 0.0;
    for (int base = blockIdx.x * blockDim.x; base < npts; base += gridDim.x * blockDim.x) {
        const int p = min(base + (int)threadIdx.x, npts - 1);
        const int i = p % g.ns, jk = p / g.ns;
        const int k = jk % g.nv, j = jk / g.nv;
        const float S = (float)(g.s_lo + i * ds);
        const float v = (float)(g.v_lo + k * dv);
        const float x0 = (float)j / (float)g.rows;
        // a wave may span two time rows: every lane brings its own time
        const float phi = phi_eval<D, true>(sh, s_afwd, x0, S, v);
        if (base + (int)threadIdx.x < npts) tab[p] = phi;
    }
}

// phi at (0, S0, v0) read from the table (level 0 of the tabulated form).
__global__ void cv_table_point_kernel(const float* tab, TableSpec t, float S0, float v0, float* out)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) *out = table_phi(tab, t, 0, S0, v0);
}

template <int D>
__global__ void cv_phi0_kernel(CvKernelArgs c, float S0, float v0, float* out)
{
    __shared__ NetShared sh;
    load_shared<D>(sh, c.params, c.nc);
    __syncthreads();
    const float phi = phi_eval<D>(sh, c.afwd, 0.0f, S0, v0);
    if (threadIdx.x == 0) *out = phi;
}

// One sample per lane; every lane runs every network evaluation (samples
// past the range are simulated and dropped), so waves stay converged.  Two
// blocks per compute unit (two waves per SIMD): with the network constants
// and W2 operands read from LDS per evaluation the kernel fits 256 registers
// per lane without spilling, and the second wave hides the matrix-core and
// transcendental latencies of the first.
template <int MODEL, int PAYOFF, int M>
__global__ __launch_bounds__(256, 2) void cv_level_kernel(LevelArgs<float> a, CvKernelArgs c)
{
    constexpr int D = (MODEL == kGBM) ? 2 : 3;
    __shared__ NetShared sh;
    __shared__ bf16x8 s_afwd[8 * 64];   // W2 operands, read at every evaluation
    load_shared<D>(sh, c.params, c.nc);
    for (int i = threadIdx.x; i < 8 * 64; i += blockDim.x) s_afwd[i] = c.afwd[i];
    __syncthreads();
    const StepParams<float>& P = a.P;
    const bool coupled = a.coupled && a.l > 0;
    double sums[kNumSums] = {0, 0, 0, 0, 0, 0};
    unsigned nonfinite = 0;
    const uint64_t nchunks = (a.N + blockDim.x - 1) / blockDim.x;
    for (uint64_t ch = blockIdx.x; ch < nchunks; ch += gridDim.x) {
        const uint64_t idx = ch * blockDim.x + threadIdx.x;
        const uint64_t s = a.offset + idx;
        PathPair<float> q;
        init_pair<float, MODEL, PAYOFF>(q, P);
        float phic = 0.0f;
        for (uint32_t g = 0; g < a.ngroups; ++g) {
            float dw1[4], dwp[4], e[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            fetch_group<MODEL, PAYOFF>(a, s, g, dw1, dwp, e);
            // not unrolled: one copy of each network evaluation in the code
#pragma unroll 1
            for (int k = 0; k < 4; ++k) {
                const int n = 4 * (int)g + k;
                if (n >= a.nf) break;                       // wave-uniform
                const float d1 = k == 0 ? dw1[0] : k == 1 ? dw1[1] : k == 2 ? dw1[2] : dw1[3];
                const float dp = k == 0 ? dwp[0] : k == 1 ? dwp[1] : k == 2 ? dwp[2] : dwp[3];
                const float ek = k == 0 ? e[0] : k == 1 ? e[1] : k == 2 ? e[2] : e[3];
                const float x0 = (float)n * P.h * sh.inv_T;
                const float phif = phi_eval<D>(sh, s_afwd, x0, q.S, q.v);
                q.cvf = __builtin_fmaf(phif, d1, q.cvf);
                if (coupled && (n & (M - 1)) == 0) phic = phi_eval<D>(sh, s_afwd, x0, q.Sc, q.vc);
                fine_step<float, MODEL, PAYOFF>(q, P, d1, dp, ek, n & (M - 1), coupled);
                if (coupled && ((n + 1) & (M - 1)) == 0) {
                    q.cvc = __builtin_fmaf(phic, q.dw1c, q.cvc);
                    coarse_step<float, MODEL, PAYOFF>(q, P);
                }
            }
        }
        const float pf = payoff_value<float, PAYOFF>(P, q.S, q.asum, q.acomp, q.mn, P.h) - q.cvf;
        const float pc = coupled
                             ? payoff_value<float, PAYOFF>(P, q.Sc, q.csum, q.ccomp, q.mnc, P.H) - q.cvc
                             : 0.0f;
        if (idx < a.N) accumulate(a, idx, pf, pc, sums, nonfinite);
    }
    block_reduce_add(sums, nonfinite, a.acc + (blockIdx.x & a.spread_mask));
}

// Levels with n_f >= 4: PPT samples per lane, blocks walk the chunks.
template <int MODEL, int PAYOFF, int M, int PPT>
__global__ __launch_bounds__(256) void cv_tab_level_kernel(LevelArgs<float> a, const float* table,
                                                           TableSpec t)
{
    extern __shared__ __attribute__((aligned(16))) float s_tab[];
    const TabView tv = load_level_table(s_tab, table, t, a.nf);
    double sums[kNumSums] = {0, 0, 0, 0, 0, 0};
    unsigned nonfinite = 0;
    const uint64_t chunk = (uint64_t)blockDim.x * PPT;
    const uint64_t nchunks = (a.N + chunk - 1) / chunk;
    for (uint64_t ch = blockIdx.x; ch < nchunks; ch += gridDim.x)
        process_chunk_tab<MODEL, PAYOFF, M, PPT>(a, ch * chunk, tv, sums, nonfinite);
    block_reduce_add(sums, nonfinite, a.acc + (blockIdx.x & a.spread_mask));
}

template <int PAYOFF, int M>
__global__ __launch_bounds__(256) void cv_tab_split_kernel(LevelArgs<float> a, const float* table,
                                                           TableSpec t)
{
    extern __shared__ __attribute__((aligned(16))) float s_tab[];
    const TabView tv = load_level_table(s_tab, table, t, a.nf);
    double sums[kNumSums] = {0, 0, 0, 0, 0, 0};
    unsigned nonfinite = 0;
    const uint64_t per_block = blockDim.x / a.split;
    const uint64_t nchunks = (a.N + per_block - 1) / per_block;
    for (uint64_t c = blockIdx.x; c < nchunks; c += gridDim.x)
        process_split_tab<PAYOFF, M>(a, c * per_block, tv, sums, nonfinite);
    block_reduce_add(sums, nonfinite, a.acc + (blockIdx.x & a.spread_mask));
}

// Levels with n_f < 4 (level 1 at M = 2): one sample per lane, the level's
// table rows in LDS.
template <int MODEL, int PAYOFF, int M>
__global__ __launch_bounds__(256) void cv_tab_short_kernel(LevelArgs<float> a, const float* table,
                                                           TableSpec t)
{
    extern __shared__ __attribute__((aligned(16))) float s_tab[];
    const TabView tv = load_level_table(s_tab, table, t, a.nf);
    double sums[kNumSums] = {0, 0, 0, 0, 0, 0};
    unsigned nonfinite = 0;
    const uint64_t nchunks = (a.N + blockDim.x - 1) / blockDim.x;
    for (uint64_t ch = blockIdx.x; ch < nchunks; ch += gridDim.x)
        process_short_tab<MODEL, PAYOFF, M>(a, ch * blockDim.x, tv, sums, nonfinite);
    block_reduce_add(sums, nonfinite, a.acc + (blockIdx.x & a.spread_mask));
}

// ----------------------------------------------------------- dispatch
using CvFn = void (*)(LevelArgs<float>, CvKernelArgs);

template <int MODEL, int PAYOFF>
static CvFn pick_cv_m(int M)
{
    return M == 2 ? cv_level_kernel<MODEL, PAYOFF, 2> : cv_level_kernel<MODEL, PAYOFF, 4>;
}

template <int MODEL>
static CvFn pick_cv_payoff(int payoff, int M)
{
    switch (payoff) {
    case kCall: return pick_cv_m<MODEL, kCall>(M);
    case kAsian: return pick_cv_m<MODEL, kAsian>(M);
    case kLookback: return pick_cv_m<MODEL, kLookback>(M);
    default: return pick_cv_m<MODEL, kDigital>(M);
    }
}

using CvTabFn = void (*)(LevelArgs<float>, const float*, TableSpec);

// Tabulated sampler for one payoff: the short-level kernel (n_f < 4), the
// split kernel (GBM, split > 1) or the per-lane kernel with ppt samples.
template <int MODEL, int PAYOFF, int M>
static CvTabFn pick_tab_m(int nf, int split, int ppt)
{
    if (nf < 4) return cv_tab_short_kernel<MODEL, PAYOFF, M>;
    if constexpr (MODEL == kGBM)
        if (split > 1) return cv_tab_split_kernel<PAYOFF, M>;
    return ppt == 2 ? cv_tab_level_kernel<MODEL, PAYOFF, M, 2> : cv_tab_level_kernel<MODEL, PAYOFF, M, 1>;
}

template <int MODEL>
static CvTabFn pick_tab_payoff(int payoff, int M, int nf, int split, int ppt)
{
    switch (payoff) {
    case kCall: return M == 2 ? pick_tab_m<MODEL, kCall, 2>(nf, split, ppt) : pick_tab_m<MODEL, kCall, 4>(nf, split, ppt);
    case kAsian: return M == 2 ? pick_tab_m<MODEL, kAsian, 2>(nf, split, ppt) : pick_tab_m<MODEL, kAsian, 4>(nf, split, ppt);
    case kLookback:
        return M == 2 ? pick_tab_m<MODEL, kLookback, 2>(nf, split, ppt) : pick_tab_m<MODEL, kLookback, 4>(nf, split, ppt);
    default: return M == 2 ? pick_tab_m<MODEL, kDigital, 2>(nf, split, ppt) : pick_tab_m<MODEL, kDigital, 4>(nf, split, ppt);
    }
}

NetConsts net_consts(const mlmc_model& m)
{
    NetConsts c;
    const double sref = m.kind == MLMC_GBM ? m.sigma : std::sqrt(m.theta);
    c.scale = (float)(sref * m.S0);
    const double a = std::log(2.0) / (sref * std::sqrt(m.T));
    c.x1a = (float)a;
    c.x1b = (float)(std::log2(m.S0) * a);
    c.x2a = m.kind == MLMC_HESTON ? (float)(1.0 / m.theta) : 0.0f;
    c.x2b = m.kind == MLMC_HESTON ? 1.0f : 0.0f;
    c.inv_T = (float)(1.0 / m.T);
    c.s_floor = (float)(m.S0 * std::ldexp(1.0, -40));
    return c;
}

static bool same_model(const mlmc_model& a, const mlmc_model& b)
{
    return a.kind == b.kind && a.S0 == b.S0 && a.r == b.r && a.sigma == b.sigma && a.T == b.T &&
           a.kappa == b.kappa && a.theta == b.theta && a.xi == b.xi && a.rho == b.rho && a.v0 == b.v0;
}

// The table of the current parameters for model m in cv->d_table, rebuilt
// when the parameters, the model or the stream changed (the same caching rule
// as phi(0, S0)).
static hipError_t cv_ensure_table(mlmc_cv* cv, const mlmc_model& m, hipStream_t st)
{
    if (cv->table_version == cv->version && cv->table_stream == st && same_model(cv->table_model, m))
        return hipSuccess;
    const TableGrid g = table_grid(m);
    const size_t n = table_size(g);
    if (cv->table_cap < n) {
        // the previous table may still be read by queued launches
        hipError_t e = hipStreamSynchronize(st);
        if (e != hipSuccess) return e;
        if (cv->d_table) hipFree(cv->d_table);
        cv->d_table = nullptr;
        cv->table_cap = 0;
        e = hipMalloc(&cv->d_table, sizeof(float) * n);
        if (e != hipSuccess) return e;
        cv->table_cap = n;
    }
    CvKernelArgs c{cv->d_params, cv->d_afwd, net_consts(m), cv->D};
    const int blocks = (int)((n + 255) / 256);
    if (cv->D == 2)
        hipLaunchKernelGGL(cv_table_kernel<2>, dim3(blocks), dim3(256), 0, st, c, g, cv->d_table);
    else
        hipLaunchKernelGGL(cv_table_kernel<3>, dim3(blocks), dim3(256), 0, st, c, g, cv->d_table);
    const hipError_t e = hipGetLastError();
    if (e == hipSuccess) {
        cv->table_version = cv->version;
        cv->table_stream = st;
        cv->table_model = m;
    }
    return e;
}

// phi(0, S0) for level 0 in cv->d_phi0[0] (from the network) or, for the
// tabulated form, cv->d_phi0[1] (from the table).  The value depends only on
// the parameters and the model, so it is computed once per parameter change,
// model and stream (a launch on another stream would not be ordered after
// the write) and level-0 launches reuse it.
hipError_t cv_ensure_phi0(const mlmc_cv* ccv, const mlmc_model& m, hipStream_t st, bool tab)
{
    mlmc_cv* cv = const_cast<mlmc_cv*>(ccv);
    const int w = tab ? 1 : 0;
    if (cv->phi0_version[w] == cv->version && cv->phi0_stream[w] == st &&
        same_model(cv->phi0_model[w], m))
        return hipSuccess;
    if (tab) {
        hipError_t e = cv_ensure_table(cv, m, st);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(cv_table_point_kernel, dim3(1), dim3(64), 0, st, (const float*)cv->d_table,
                           table_spec(table_grid(m)), (float)m.S0, (float)m.v0, cv->d_phi0 + 1);
    } else {
        CvKernelArgs c{cv->d_params, cv->d_afwd, net_consts(m), cv->D};
        if (cv->D == 2)
            hipLaunchKernelGGL(cv_phi0_kernel<2>, dim3(1), dim3(64), 0, st, c, (float)m.S0,
                               (float)m.v0, cv->d_phi0);
        else
            hipLaunchKernelGGL(cv_phi0_kernel<3>, dim3(1), dim3(64), 0, st, c, (float)m.S0,
                               (float)m.v0, cv->d_phi0);
    }
    const hipError_t e = hipGetLastError();
    if (e == hipSuccess) {
        cv->phi0_version[w] = cv->version;
        cv->phi0_stream[w] = st;
        cv->phi0_model[w] = m;
    }
    return e;
}

bool cv_tabulated(const mlmc_cv* cv) { return cv->tabulated != 0; }

hipError_t cv_table_view(const mlmc_cv* ccv, const mlmc_model& m, hipStream_t st, int max_nf,
                         const float** table, TableSpec* spec, const float** phi0, size_t* lds_bytes)
{
    const hipError_t e = cv_ensure_phi0(ccv, m, st, true);   // builds the table first
    if (e != hipSuccess) return e;
    const TableGrid g = table_grid(m);
    const int lr = max_nf < g.rows ? max_nf : g.rows;
    *table = ccv->d_table;
    *spec = table_spec(g);
    *phi0 = ccv->d_phi0 + 1;
    *lds_bytes = sizeof(float) * (size_t)lr * g.ns * g.nv;
    return hipSuccess;
}

hipError_t cv_launch_level(const mlmc_cv* ccv, const mlmc_model& m, const mlmc_payoff& p, int M,
                           const LevelArgs<float>& a, int grid, hipStream_t st, bool tab, int ppt)
{
    mlmc_cv* cv = const_cast<mlmc_cv*>(ccv);
    if (tab) {
        hipError_t e = cv_ensure_table(cv, m, st);
        if (e != hipSuccess) return e;
        const TableGrid g = table_grid(m);
        const int lr = a.nf < g.rows ? a.nf : g.rows;    // rows the level reads
        const size_t lds = sizeof(float) * (size_t)lr * g.ns * g.nv;
        CvTabFn fn = m.kind == MLMC_GBM ? pick_tab_payoff<kGBM>(p.kind, M, a.nf, (int)a.split, ppt)
                                        : pick_tab_payoff<kHeston>(p.kind, M, a.nf, 1, ppt);
        hipLaunchKernelGGL(fn, dim3(grid), dim3(256), lds, st, a, (const float*)cv->d_table,
                           table_spec(g));
        return hipGetLastError();
    }
    CvKernelArgs c{cv->d_params, cv->d_afwd, net_consts(m), cv->D};
    CvFn fn = m.kind == MLMC_GBM ? pick_cv_payoff<kGBM>(p.kind, M) : pick_cv_payoff<kHeston>(p.kind, M);
    hipLaunchKernelGGL(fn, dim3(grid), dim3(256), 0, st, a, c);
    return hipGetLastError();
}

const float* cv_phi0_ptr(const mlmc_cv* cv, bool tab) { return cv->d_phi0 + (tab ? 1 : 0); }
int cv_in_dim(const mlmc_cv* cv) { return cv->D; }

static hipError_t cv_prepare(mlmc_cv* cv, hipStream_t st)
{
    ++cv->version;
    hipLaunchKernelGGL(cv_prepare_kernel, dim3(1), dim3(256), 0, st, (const float*)cv->d_params,
                       cv->D, cv->d_afwd, cv->d_abwd);
    return hipGetLastError();
}

}  // namespace mlmc

using namespace mlmc;

namespace {
const mlmc_payoff kAnyPayoff{MLMC_CALL, 100.0, 1.0};
}

extern "C" {

mlmc_status mlmc_cv_destroy(mlmc_cv* cv)
{
    if (!cv) return MLMC_OK;
    if (cv->ctx) hipSetDevice(cv->ctx->device);
    for (void* p : {(void*)cv->d_params, (void*)cv->d_m1, (void*)cv->d_m2, (void*)cv->d_afwd,
                    (void*)cv->d_abwd, (void*)cv->d_phi0, (void*)cv->d_train, (void*)cv->d_loss,
                    (void*)cv->d_table})
        if (p) hipFree(p);
    delete cv;
    return MLMC_OK;
}

mlmc_status mlmc_cv_create(mlmc_ctx* ctx, int in_dim, int hidden, uint64_t init_seed, mlmc_cv** out)
{
    if (!ctx) return MLMC_EINVAL;
    if (!out) return fail(ctx, MLMC_EINVAL, "out must not be NULL");
    *out = nullptr;
    if ((in_dim != 2 && in_dim != 3) || hidden != H)
        return fail(ctx, MLMC_EINVAL, "in_dim must be 2 (GBM) or 3 (Heston) and hidden 64");
    MLMC_ENTER(ctx);
    mlmc_cv* cv = new (std::nothrow) mlmc_cv();
    if (!cv) return fail(ctx, MLMC_ENOMEM, "host allocation failed");
    cv->ctx = ctx;
    cv->D = in_dim;
    cv->np = nparams(in_dim);
    hipError_t e = hipMalloc(&cv->d_params, sizeof(float) * cv->np);
    if (e == hipSuccess) e = hipMalloc(&cv->d_m1, sizeof(float) * cv->np);
    if (e == hipSuccess) e = hipMalloc(&cv->d_m2, sizeof(float) * cv->np);
    if (e == hipSuccess) e = hipMalloc(&cv->d_afwd, sizeof(bf16x8) * 8 * 64);
    if (e == hipSuccess) e = hipMalloc(&cv->d_abwd, sizeof(bf16x8) * 8 * 64);
    if (e == hipSuccess) e = hipMalloc(&cv->d_phi0, sizeof(float) * 4);
    if (e == hipSuccess) e = hipMalloc(&cv->d_loss, sizeof(double) * 64);
    if (e == hipSuccess) e = hipMemsetAsync(cv->d_m1, 0, sizeof(float) * cv->np, ctx->stream);
    if (e == hipSuccess) e = hipMemsetAsync(cv->d_m2, 0, sizeof(float) * cv->np, ctx->stream);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(cv_init_kernel, dim3((cv->np + 255) / 256), dim3(256), 0, ctx->stream,
                           cv->d_params, in_dim, init_seed);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = cv_prepare(cv, ctx->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) {
        mlmc_cv_destroy(cv);
        return hip_fail(ctx, e, "control variate allocation/initialisation");
    }
    *out = cv;
    return MLMC_OK;
}

mlmc_status mlmc_cv_get_params(const mlmc_cv* cv, float* host, size_t n)
{
    if (!cv) return MLMC_EINVAL;
    mlmc_ctx* ctx = cv->ctx;
    if (!host || n != (size_t)cv->np) return fail(ctx, MLMC_EINVAL, "need a host array of nparams floats");
    MLMC_ENTER(ctx);
    MLMC_HIP(ctx, hipMemcpyAsync(host, cv->d_params, sizeof(float) * n, hipMemcpyDeviceToHost,
                                 ctx->stream));
    MLMC_HIP(ctx, hipStreamSynchronize(ctx->stream));
    return MLMC_OK;
}

mlmc_status mlmc_cv_set_params(mlmc_cv* cv, const float* host, size_t n)
{
    if (!cv) return MLMC_EINVAL;
    mlmc_ctx* ctx = cv->ctx;
    if (!host || n != (size_t)cv->np) return fail(ctx, MLMC_EINVAL, "need a host array of nparams floats");
    for (size_t i = 0; i < n; ++i)
        if (!std::isfinite(host[i])) return fail(ctx, MLMC_EINVAL, "parameters must be finite");
    MLMC_ENTER(ctx);
    MLMC_HIP(ctx, hipMemcpyAsync(cv->d_params, host, sizeof(float) * n, hipMemcpyHostToDevice,
                                 ctx->stream));
    MLMC_HIP(ctx, cv_prepare(cv, ctx->stream));
    MLMC_HIP(ctx, hipStreamSynchronize(ctx->stream));
    return MLMC_OK;
}

size_t mlmc_cv_nparams(const mlmc_cv* cv) { return cv ? (size_t)cv->np : 0; }

mlmc_status mlmc_cv_set_tabulated(mlmc_cv* cv, int on)
{
    if (!cv) return MLMC_EINVAL;
    if (on != 0 && on != 1) return fail(cv->ctx, MLMC_EINVAL, "on must be 0 or 1");
    cv->tabulated = on;
    return MLMC_OK;
}

mlmc_status mlmc_cv_get_table(mlmc_cv* cv, const mlmc_model* model, float* host, size_t n,
                              int* dims)
{
    if (!cv) return MLMC_EINVAL;
    mlmc_ctx* ctx = cv->ctx;
    mlmc_status st = check_level_args(ctx, model, &kAnyPayoff, 0, 2, 32);
    if (st) return st;
    if (cv->D != (model->kind == MLMC_HESTON ? 3 : 2))
        return fail(ctx, MLMC_EINVAL, "network inputs do not match the model (2: GBM, 3: Heston)");
    const TableGrid g = table_grid(*model);
    if (dims) {
        dims[0] = g.rows;
        dims[1] = g.nv;
        dims[2] = g.ns;
    }
    if (!host) return MLMC_OK;
    if (n != table_size(g)) return fail(ctx, MLMC_EINVAL, "need a host array of rows * nv * ns floats");
    MLMC_ENTER(ctx);
    MLMC_HIP(ctx, cv_ensure_table(cv, *model, ctx->stream));
    MLMC_HIP(ctx, hipMemcpyAsync(host, cv->d_table, sizeof(float) * n, hipMemcpyDeviceToHost,
                                 ctx->stream));
    MLMC_HIP(ctx, hipStreamSynchronize(ctx->stream));
    return MLMC_OK;
}

}  // extern "C"
