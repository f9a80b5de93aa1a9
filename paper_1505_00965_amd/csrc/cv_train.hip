// Training of the control-variate network: one loss/gradient evaluation (and
// Adam step) in five launches.
//
// Loss over levels 0..lmax (the MLMC cost functional; total cost scales as
// (sum_l sqrt(V_l C_l))^2):  loss = sum_l sqrt(C_l Var_batch(Y_l)), with Y the
// level sample with the control variate (eq. (eq:Yldef), each payoff replaced
// by P - sum_n phi(t_n, X_n) dW1_n), so dLoss/dY_i = sqrt(C_l / V_l)
// (Y_i - mean_l) / (B - 1).
//
// The network is evaluated at points (t_n, X_n) that do not depend on it, so
// a step is cut at the points, not at the paths:
//   train_paths    every path of the batch once: per point the network's
//                  inputs and the coefficient c of phi in Y (-dW1 on the fine
//                  path, +dW1 on the coarse one), per sample the payoffs
//   train_forward  phi at every point, 64 points of one time per wave
//   train_combine  Y per sample, the level sums; phi(0, S0) once
//   train_backward the parameter gradient over all points, one partial row
//                  per block
//   train_update   the rows' sum, Adam, the bf16 operands of the new W2
// Points are independent units of equal cost: both network passes deal them
// out evenly whatever the levels (a launch per level, in runs of steps, left
// the device a fifth full: 0.50 ms per step of 16384 samples on levels 0..3,
// now 0.20), and the paths are stepped twice a step at most instead of
// once per run.  Every path starts at (0, S0), so the points at t = 0 share
// one network evaluation: level 0 needs no other.
//
// The paths do not depend on the parameters either: train_paths makes those
// of several Adam steps in one launch (as many as fit kMaxPoints), whose
// time is one path's chain of steps whatever their number.  A batch whose
// points exceed kMaxPoints is worked off in chunks of samples instead (the
// points of a chunk are made again for the backward pass), of kTrainChunk
// samples at least: every chunk takes the deepest level's chain twice, 0.5 ms
// (Heston 0.9) at 4096 steps however few its samples, and kMaxPoints alone
// holds 2432 of them there.  Adam step on levels 0..6, M = 4, ms, by
// kMaxPoints alone and with at least 32768 samples:
//   16384 samples, GBM 20.9  11.6, Heston 27.1  12.9
//   131072 samples     175   93,          223   102
// (131072 with at least 16384, 32768 and 65536, the backward pass in one launch
// a chunk: 98, 91 and 88, Heston 111, 100 and 95.)
// 32768 there need 2.7 GB (Heston 3.6) of scratch, kept by the network.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "cv_state.hpp"
#include "cv_tab.hpp"
#include "sampler_impl.hpp"
#include "trace.hpp"

using namespace mlmc::cvnet;

namespace mlmc {

constexpr int kTrainLevels = 7;               // lmax <= 6
constexpr uint64_t kMaxPoints = 1ull << 24;   // points in memory at once
constexpr int kMaxSteps = 16;                 // steps whose paths one launch makes
constexpr int kGradRow = 4544;                // floats per partial row (>= nparams, 16-byte rows)
// Times of the backward kernel's blocks: 34 ns per (level, sample) pair of the
// start point, 4.8 us per 64 points (four blocks per compute unit).
constexpr double kStartPairCost = 34.0, kTaskCost = 4800.0;
constexpr int kBwdBlocksPerCu = 4;            // the backward kernel's residency (registers, LDS)
constexpr int kFwdBlocksPerCu = 4;

struct TrainLevel {
    StepParams<float> P;
    int nf, ngroups;
    uint32_t row0;      // first point row of the level: fine steps 1.., then coarse steps 1..
    uint32_t blk0;      // first block of the level's samples (256 per block)
    uint32_t runs;      // runs of generator groups a sample's sums are taken in
};

// One chunk of a training batch: samples offset .. offset + n - 1 of every
// level, point rows of `stride` samples (n rounded up to whole waves).
struct TrainArgs {
    TrainLevel lev[kTrainLevels];
    int nlev, M;
    uint32_t n, stride, nrows;
    uint32_t first;         // position of the chunk in the batch
    uint32_t task0, tasks;  // a backward launch's part of the chunk's (row, 64 samples) tasks
    uint64_t B, Bpad;       // batch size, row length of y
    uint64_t seed, offset;
    float S0, v0;
    float *x1, *x2;         // [nrows][stride] network inputs of each point
    float *c;               // [nrows][stride] coefficient of phi in Y
    float *phi;             // [nrows][stride] phi of each point
    float *x0;              // [nrows] time input
    float2 *pay;            // [nlev][stride] fine and coarse payoff
    float2 *c0;             // [nlev][stride] coefficients of phi(0, S0): fine, coarse
    double *y;              // [nlev][Bpad]
    float *phi0;            // phi(0, S0)
    // per level: sums of Y and Y^2 over the batch
    LevelAcc *rec;
};

// The arguments of step k of a group: its samples and its buffers (all but
// phi, x0, y and phi0, which every step shares).
__host__ __device__ __forceinline__ TrainArgs for_step(TrainArgs a, uint32_t k)
{
    const uint64_t pts = (uint64_t)k * a.nrows * a.stride, smp = (uint64_t)k * a.nlev * a.stride;
    a.offset += (uint64_t)k * a.B;
    a.x1 += pts;
    a.x2 += pts;
    a.c += pts;
    a.pay += smp;
    a.c0 += smp;
    a.rec += k * (uint32_t)a.nlev;
    return a;
}

// Level whose blocks of 256 samples hold block b (levels deepest first).
__device__ __forceinline__ int block_level(const TrainArgs& a, uint32_t b)
{
    int l = a.nlev - 1;
    while (l > 0 && b >= a.lev[l - 1].blk0) --l;
    return l;
}

// ------------------------------------------------------------------ paths
// One sample per lane, as the estimation samplers step it.  Bound by the
// longest path's chain of steps (64 at level 3, ~7 us); the stores are
// coalesced rows.  blockIdx.y: the step of a group, with buffers of its own
// (for_step).  The first blocks clear the level sums.
template <int MODEL, int PAYOFF, int M>
__global__ __launch_bounds__(256) void train_paths_kernel(TrainArgs a, NetConsts nc, int clear)
{
    // (the arguments stay as they were passed: a changed copy of them would be
    // indexed by level in private memory)
    const uint64_t pts = (uint64_t)blockIdx.y * a.nrows * a.stride;
    const uint64_t smp = (uint64_t)blockIdx.y * a.nlev * a.stride;
    if (clear && blockIdx.x == 0 && threadIdx.x < (unsigned)a.nlev)
        a.rec[blockIdx.y * (uint32_t)a.nlev + threadIdx.x] = LevelAcc{};
    const int l = block_level(a, blockIdx.x);
    const TrainLevel& L = a.lev[l];
    const uint32_t i = (blockIdx.x - L.blk0) * 256u + threadIdx.x;
    if (i >= a.stride) return;                      // wave-uniform
    LevelArgs<float> la;                            // what fetch_group reads
    la.P = L.P;
    la.seed = a.seed;
    la.l = l;
    la.nf = L.nf;
    la.stream = kStreamTrainNormal;
    const StepParams<float>& P = la.P;
    const uint64_t s = a.offset + (uint64_t)blockIdx.y * a.B + i;
    const bool in = i < a.n, coupled = l > 0;
    const int nf = L.nf;
    float* const x1 = a.x1 + pts + (uint64_t)L.row0 * a.stride + i;
    float* const x2 = a.x2 + pts + (uint64_t)L.row0 * a.stride + i;
    float* const cs = a.c + pts + (uint64_t)L.row0 * a.stride + i;
    auto x1_of = [&](float S) {
        return __builtin_fmaf(__builtin_amdgcn_logf(S > nc.s_floor ? S : nc.s_floor), nc.x1a, -nc.x1b);
    };
    // point of row r (coefficient stored apart for the coarse points)
    auto put = [&](uint32_t r, float S, float v) {
        const uint64_t at = (uint64_t)r * a.stride;
        x1[at] = in ? x1_of(S) : 0.0f;
        if (MODEL == kHeston) x2[at] = in ? __builtin_fmaf(v, nc.x2a, -nc.x2b) : 0.0f;
    };
    auto put_c = [&](uint32_t r, float c) { cs[(uint64_t)r * a.stride] = in ? c : 0.0f; };
    PathPair<float> q;
    init_pair<float, MODEL, PAYOFF>(q, P);
    float2 c0 = make_float2(0.0f, 0.0f);
    for (uint32_t g = 0; g < (uint32_t)L.ngroups; ++g) {
        float dw1[4], dwp[4], e[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        fetch_group<MODEL, PAYOFF>(la, s, g, dw1, dwp, e);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int n = 4 * (int)g + k;
            if (n >= nf) break;                     // block-uniform
            if (n > 0) {
                put(n - 1, q.S, q.v);
                put_c(n - 1, -dw1[k]);
                if (coupled && n % M == 0) put(nf - 1 + n / M - 1, q.Sc, q.vc);
            } else {
                c0.x = -dw1[0];
            }
            fine_step<float, MODEL, PAYOFF>(q, P, dw1[k], dwp[k], e[k], n % M, coupled);
            if (coupled && (n + 1) % M == 0) {
                const int m = n / M;
                if (m > 0) put_c(nf - 1 + m - 1, q.dw1c);
                else c0.y = q.dw1c;
                coarse_step<float, MODEL, PAYOFF>(q, P);
            }
        }
    }
    const float pf = payoff_value<float, PAYOFF>(P, q.S, q.asum, q.acomp, q.mn, P.h);
    const float pc = coupled ? payoff_value<float, PAYOFF>(P, q.Sc, q.csum, q.ccomp, q.mnc, P.H) : 0.0f;
    a.pay[smp + (uint64_t)l * a.stride + i] = make_float2(pf, pc);
    a.c0[smp + (uint64_t)l * a.stride + i] = c0;
    // time inputs of the level's rows, by its first block
    if (blockIdx.x == L.blk0 && blockIdx.y == 0) {
        const int nrow = (nf - 1) + (coupled ? nf / M - 1 : 0);
        for (int r = (int)threadIdx.x; r < nrow; r += (int)(a.stride < 256u ? a.stride : 256u)) {
            const int n = r < nf - 1 ? r + 1 : (r - (nf - 1) + 1) * M;
            a.x0[L.row0 + r] = (float)n * P.h * nc.inv_T;
        }
    }
}

// ---------------------------------------------------------------- forward
// phi for 64 points of one row per wave.  Bound by the vector ALU: ~900
// instructions a point of which 256 transcendental (two issue slots each),
// so four waves per SIMD (128 registers: the network's constants stay in
// LDS) keep it issuing.
template <int D>
__global__ __launch_bounds__(256, kFwdBlocksPerCu) void train_forward_kernel(TrainArgs a, CvKernelArgs c)
{
    __shared__ NetShared sh;
    __shared__ bf16x8 s_afwd[8 * 64];
    load_shared<D>(sh, c.params, c.nc);
    for (int i = threadIdx.x; i < 8 * 64; i += blockDim.x) s_afwd[i] = c.afwd[i];
    __syncthreads();
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t cw = a.stride / 64, total = a.nrows * cw, nw = gridDim.x * (blockDim.x / 64);
    if (blockIdx.x == gridDim.x - 1 && wave == 3) {
        // the point all paths share (the last wave has the fewest tasks)
        const float phi = phi_eval<D>(sh, s_afwd, 0.0f, a.S0, a.v0);
        if (lane == 0) *a.phi0 = phi;
    }
    for (uint32_t t = blockIdx.x * (blockDim.x / 64) + wave; t < total; t += nw) {
        const uint32_t row = __builtin_amdgcn_readfirstlane(t / cw), ch = t - row * cw;
        const uint64_t at = (uint64_t)row * a.stride + ch * 64 + lane;
        a.phi[at] = phi_eval_x<D>(sh, s_afwd, a.x0[row], a.x1[at], D == 3 ? a.x2[at] : 0.0f);
    }
}

// Y of every sample and the level sums.  The two paths' sums of phi dW are
// taken in fp32 as the samplers take them, step by step with fused
// multiply-adds, and on levels of several runs run by run, the runs' sums
// added in order: the sums' rounding decides which way d2 rounds to bf16 in
// the backward pass, so it does not depend on the launches' shapes.  Bound by
// the latency of the loads: a block of four waves takes 64 samples, a run per
// wave at a time (16384 samples on levels 0..3: 12.6 us; with a lane for all of a
// sample's runs 27).
__global__ __launch_bounds__(256) void train_combine_kernel(TrainArgs a)
{
    __shared__ float s_run[2][4][64];
    const uint32_t cw = a.stride / 64;
    const int l = a.nlev - 1 - (int)(blockIdx.x / cw);          // deepest level first
    const TrainLevel& L = a.lev[l];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t i = (blockIdx.x % cw) * 64 + lane;
    const float phi0 = *a.phi0;
    const float2 c0 = a.c0[(uint64_t)l * a.stride + i];
    // run r of the sum of phi dW over the points s = 0 .. runs per - 1 of a
    // path whose rows (from s = 1) start at `row`; the coefficients hold sign dW
    auto run_of = [&](uint32_t row, int per, int r, float start, float sign) {
        const float* ph = a.phi + (uint64_t)row * a.stride + i;
        const float* cc = a.c + (uint64_t)row * a.stride + i;
        float run = r ? 0.0f : __builtin_fmaf(phi0, sign * start, 0.0f);
#pragma unroll 8
        for (int s = r ? r * per : 1; s < (r + 1) * per; ++s) {
            const uint64_t at = (uint64_t)(s - 1) * a.stride;
            run = __builtin_fmaf(ph[at], sign * cc[at], run);
        }
        return run;
    };
    float cf = 0.0f, cc = 0.0f;
    const int runs = l ? (int)L.runs : 0, nc = l ? L.nf / a.M : 0;
    for (int r0 = 0; r0 < runs; r0 += 4) {                      // block-uniform
        const int r = r0 + wave;
        if (r < runs) {
            s_run[0][wave][lane] = run_of(L.row0, L.nf / runs, r, c0.x, -1.0f);
            s_run[1][wave][lane] = run_of(L.row0 + L.nf - 1, nc / runs, r, c0.y, 1.0f);
        }
        __syncthreads();
        for (int k = 0; k < 4 && r0 + k < runs; ++k) {          // 0 + x is exact
            cf += s_run[0][k][lane];
            cc += s_run[1][k][lane];
        }
        __syncthreads();
    }
    double sums[kNumSums] = {0, 0, 0, 0, 0, 0};
    unsigned nonfinite = 0;
    if (wave == 0) {
        const float2 p = a.pay[(uint64_t)l * a.stride + i];
        const float pf = l ? p.x - cf : __builtin_fmaf(phi0, c0.x, p.x);
        const float pc = l ? p.y - cc : 0.0f;
        const bool in = i < a.n;
        const double y = in ? (double)pf - (double)pc : 0.0;
        a.y[(uint64_t)l * a.Bpad + a.first + i] = y;
        if (in && isfinite(y)) {
            sums[0] = y;
            sums[1] = y * y;
        } else if (in) {
            nonfinite = 1;
        }
    }
    block_reduce_add(sums, nonfinite, &a.rec[l]);
}

// --------------------------------------------------------------- backward
// With g = dLoss/dphi at a point (w c, w = dLoss/dY of its sample) and
// dy = scale g:
//   gb3 += dy,  gw3 += dy h2,  d2 = dy w3 (1 - h2^2),  gb2 += d2,
//   gW2 += d2 h1^T,  d1 = (W2^T d2) (1 - h1^2),  gb1 += d1,  gW1 += d1 x^T.
// d2 and h1 are rounded to bf16 where the matrix cores read them; 1 - h1^2
// uses the fp32 h1 and the vector gradients fp32 sums.
//
// A block of two waves takes 64 points: wave ut holds the 32 units of tile
// ut for all of them, so a lane keeps 16 units (its gradient sums and G fill
// 112 registers; a wave that holds 64 x 64 needs 225 and runs alone on its
// SIMD, where a wave issues at little more than half rate) with two
// independent points' chains in flight, and four blocks fit a compute unit.
// The layers exchange h1 and d2 through LDS rows (row: point, column: unit,
// 144 bytes so that 16-byte reads of eight rows meet no bank twice), and gW2
// reads them transposed (ds_read_b64_tr_b16: 24 reads a wave in place of
// 128 two-byte ones).  Two buffers: a point's writes need no barrier after
// the reads of the point before it.
// 16384 samples on levels 0..3 (25344 tasks): 127 us, 74% of it issuing VALU; with one wave per block, two-byte
// transposed reads and a launch per level 300, with four waves of 32 x 32
// (the constants read twice as often) 143.
constexpr int kRowPad = 72;     // bf16 per staged row (64 + 8)

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// Operand fragment (lane: column lane % 32 of tile t, rows 16 kb + 8 h + i of
// the staged array) of a transposed read; `at` is the lane's element for
// kb = 0, t = 0.
__device__ __forceinline__ bf16x8 read_tr(const __bf16* at, int kb, int t)
{
    const __bf16* p = at + (16 * kb) * kRowPad + 32 * t;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * kRowPad));
    bf16x8 v;
    __builtin_memcpy(&v, &lo, 8);
    __builtin_memcpy((char*)&v + 8, &hi, 8);
    return v;
}

__device__ __forceinline__ float sum32(float v)
{
    // over the 32 lanes of the half: rows of 16 by DPP, then the other row
    auto add = [](float x, int y) { return x + __builtin_bit_cast(float, y); };
    v = add(v, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), kQuadPerm1032, 0xF, 0xF, false));
    v = add(v, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), kQuadPerm2301, 0xF, 0xF, false));
    v = add(v, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), kRowRor4, 0xF, 0xF, false));
    v = add(v, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), kRowRor8, 0xF, 0xF, false));
    return v + __shfl_xor(v, 16);
}

// Mean and dLoss/dY scale of every level, and the loss.
struct LevelStats {
    double mean[kTrainLevels], scale[kTrainLevels], var[kTrainLevels], cost[kTrainLevels];
};

__device__ __forceinline__ void level_stats(const TrainArgs& a, int l, LevelStats& s)
{
    const double n = (double)a.B;
    const LevelAcc& r = a.rec[l];
    const double mean = r.sum[0] / n;
    double var = (r.sum[1] - n * mean * mean) / (n - 1.0);
    if (var < 0) var = 0;
    double C = 1.0;
    if (l > 0) {
        double b = 1.0;
        for (int i = 0; i < l - 1; ++i) b *= a.M;
        C = b * a.M + b;
    }
    s.mean[l] = mean;
    s.var[l] = var;
    s.cost[l] = C;
    s.scale[l] = var > 0 ? sqrt(C / var) / (n - 1.0) : 0.0;
}

// The gradient at the one point (0, S0) all paths share: start block `b` of
// `ns` takes its share of the chunk's (level, sample) pairs, fine and coarse
// point each.  Only dy differs between them, so a pair costs the 64 units'
// d2 = dy w3 (1 - h2^2), rounded to bf16 as at every other point and summed in
// fp32; the products with W2 and h1 follow once from the sums.
template <int D>
__device__ __forceinline__ void start_point_row(const TrainArgs& a, const CvKernelArgs& c, const NetShared& sh,
                                                const LevelStats& st, uint32_t b, uint32_t ns, float* row)
{
    __shared__ __attribute__((aligned(16))) float s_dy[256];
    __shared__ float s_h1[H], s_d2[2][H], s_sum[2];
    const float x1 = input_x1(sh, a.S0);
    const float x2 = D == 3 ? __builtin_fmaf(a.v0, sh.x2a, -sh.x2b) : 0.0f;
    const float* W2 = c.params + off_W2(D);
    const int u = threadIdx.x & 63, half = threadIdx.x >> 6;
    {
        // the time input is zero
        float z = __builtin_fmaf(sh.w1[u][1], x1, sh.w1[u][2]);
        if (D == 3) z = __builtin_fmaf(sh.w1[u][3], x2, z);
        s_h1[u] = tanh_fast(z);
    }
    __syncthreads();
    float z = sh.b2[u];
    for (int k = 0; k < H; ++k) z = __builtin_fmaf((float)(__bf16)W2[u * H + k], (float)(__bf16)s_h1[k], z);
    const float hv = tanh_fast(z), dd = 1.0f - hv * hv, w3 = sh.w3[u];
    // 128 pairs at a time: a thread forms a pair's two dy, then each half
    // block adds up one unit per thread over half of them
    const uint32_t pairs = (uint32_t)a.nlev * a.n;
    const uint32_t e0 = (uint32_t)((uint64_t)pairs * b / ns), e1 = (uint32_t)((uint64_t)pairs * (b + 1) / ns);
    float d2 = 0.0f, sum = 0.0f;
    for (uint32_t e = e0; e < e1; e += 128) {
        const uint32_t k = e + threadIdx.x;
        float dyf = 0.0f, dyc = 0.0f;
        if (k < e1) {
            const uint32_t l = k / a.n, i = k - l * a.n;
            const float2 c0 = a.c0[(uint64_t)l * a.stride + i];
            const float w = (float)(st.scale[l] * (a.y[(uint64_t)l * a.Bpad + a.first + i] - st.mean[l]));
            dyf = sh.scale * (w * c0.x);
            dyc = sh.scale * (w * c0.y);
        }
        sum += dyf + dyc;
        *(float2*)&s_dy[2 * threadIdx.x] = make_float2(dyf, dyc);
        __syncthreads();
#pragma unroll 4
        for (int i = 0; i < 128; i += 4) {
            const float4 v = *(const float4*)&s_dy[128 * half + i];
            d2 += (float)(__bf16)(v.x * w3 * dd);
            d2 += (float)(__bf16)(v.y * w3 * dd);
            d2 += (float)(__bf16)(v.z * w3 * dd);
            d2 += (float)(__bf16)(v.w * w3 * dd);
        }
        __syncthreads();
    }
    sum = sum32(sum);
    sum += __shfl_xor(sum, 32);
    s_d2[half][u] = d2;
    if (u == 0) s_sum[half] = sum;
    __syncthreads();
    const bool add = a.first != 0;              // a later chunk of the batch
    auto put = [&](int i, float v) { row[i] = add ? row[i] + v : v; };
    if (half == 0) {
        const float dy = s_sum[0] + s_sum[1];
        put(off_w3(D) + u, dy * hv);
        put(off_b2(D) + u, dy * w3 * dd);
        if (u == 0) put(off_b3(D), dy);
        float e = 0.0f;
        for (int j = 0; j < H; ++j)
            e = __builtin_fmaf((float)(__bf16)W2[j * H + u], s_d2[0][j] + s_d2[1][j], e);
        const float d1 = e * (1.0f - s_h1[u] * s_h1[u]);
        put(off_b1(D) + u, d1);
        put(u * D + 0, 0.0f);
        put(u * D + 1, d1 * x1);
        if (D == 3) put(u * D + 2, d1 * x2);
    }
    for (int i = threadIdx.x; i < H * H; i += blockDim.x)
        put(off_W2(D) + i, (s_d2[0][i / H] + s_d2[1][i / H]) * (float)(__bf16)s_h1[i % H]);
}

// Blocks 0 .. ns - 1: the start point's rows of gpart and (block 0, first
// chunk) the loss.  Block ns + b: points of share b of the launch's tasks.  A
// block's row is added to after the batch's first launch: a chunk of more than
// kMaxPoints takes several, so that no lane sums more points in fp32 than one
// of that size gives it.  Gradients on levels 0..6 of 16384 and 32000 samples in
// one launch lay 0.8e-6 to 4e-6 from those of chunks of kMaxPoints and of
// launches per level, which lie 3.5e-7 to 4.5e-7 apart; so as far as those.
template <int D>
__global__ __launch_bounds__(128, 2) void train_backward_kernel(TrainArgs a, CvKernelArgs c,
                                                                const bf16x8* abwd, float* gpart, uint32_t ns,
                                                                double* loss, double* loss_hist)
{
    __shared__ NetShared sh;
    __shared__ LevelStats st;
    __shared__ __attribute__((aligned(16))) __bf16 s_h1[2][64 * kRowPad], s_d2[2][64 * kRowPad];
    load_shared<D>(sh, c.params, c.nc);
    if (threadIdx.x < (unsigned)a.nlev) level_stats(a, (int)threadIdx.x, st);
    __syncthreads();
    float* grow = gpart + (uint64_t)blockIdx.x * kGradRow;
    if (blockIdx.x < ns) {
        if (a.task0) return;                    // in the chunk's first launch
        start_point_row<D>(a, c, sh, st, blockIdx.x, ns, grow);
        if (blockIdx.x == 0 && threadIdx.x == 0 && a.first == 0) {
            double t = 0.0;
            for (int l = 0; l < a.nlev; ++l) {
                t += sqrt(st.cost[l] * st.var[l]);
                loss[1 + l] = st.var[l];
            }
            loss[0] = t;
            if (loss_hist) *loss_hist = t;
        }
        return;
    }
    const uint32_t nb = gridDim.x - ns, b = blockIdx.x - ns;
    const int lane = threadIdx.x & 63, h = lane >> 5, col = lane & 31;
    const int ut = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    bf16x8 af[4], ab[4];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
        af[kb] = c.afwd[(ut * 4 + kb) * 64 + lane];
        ab[kb] = abwd[(ut * 4 + kb) * 64 + lane];
    }
    f32x16 G[2];
    float gw3[16], gb2[16], gb1[16], gw1[D][16], gb3 = 0.0f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        G[0][r] = G[1][r] = gw3[r] = gb2[r] = gb1[r] = 0.0f;
#pragma unroll
        for (int d = 0; d < D; ++d) gw1[d][r] = 0.0f;
    }
    // the lane's staged elements: its own rows col, 32 + col (written and
    // read by row) and its corner of a transposed read
    const int own = col * kRowPad;
    const int tr = (8 * h + ((lane & 15) >> 2)) * kRowPad + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
    const uint32_t cw = a.stride / 64;
    const uint32_t t0 = a.task0 + (uint32_t)((uint64_t)a.tasks * b / nb);
    const uint32_t t1 = a.task0 + (uint32_t)((uint64_t)a.tasks * (b + 1) / nb);
    // a task's points: network inputs, coefficient, Y; with two inputs the
    // next task's loads are in flight while this one's points are worked off
    // (with three the registers for it would spill)
    constexpr bool kAhead = D == 2;
    struct Points {
        uint32_t row;
        int l;
        float x0, x1[2], x2[2], c[2];
        double y[2];
    };
    auto load = [&](uint32_t t) {
        Points p;
        p.row = __builtin_amdgcn_readfirstlane(t / cw);
        const uint32_t ch = t - p.row * cw;
        p.l = a.nlev - 1;
        while (p.l > 0 && p.row < a.lev[p.l].row0) --p.l;
        p.x0 = a.x0[p.row];
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            const uint32_t i = ch * 64 + 32 * nt + col;
            const uint64_t at = (uint64_t)p.row * a.stride + i;
            p.x1[nt] = a.x1[at];
            p.x2[nt] = D == 3 ? a.x2[at] : 0.0f;
            p.c[nt] = a.c[at];
            p.y[nt] = a.y[(uint64_t)p.l * a.Bpad + a.first + i];
        }
        return p;
    };
    int buf = 0;
    Points next = load(t0 < t1 ? t0 : 0);       // every block has a task, but in a short last chunk
    for (uint32_t t = t0; t < t1; ++t) {
        // the network's constants are read from LDS at every point (see phi_eval_x)
        __asm__ volatile("" ::: "memory");
        const Points p = kAhead ? next : load(t);
        if (kAhead && t + 1 < t1) next = load(t + 1);
        const float x0 = p.x0;
        float x1[2], x2[2], dy[2];
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            x1[nt] = p.x1[nt];
            x2[nt] = p.x2[nt];
            dy[nt] = sh.scale * ((float)(st.scale[p.l] * (p.y[nt] - st.mean[p.l])) * p.c[nt]);
            gb3 += dy[nt];
        }
        __bf16* h1 = s_h1[buf];
        __bf16* d2 = s_d2[buf];
        buf ^= 1;
        float h1f[2][16];
#pragma unroll
        for (int r4 = 0; r4 < 16; r4 += 4) {
            __bf16 v4[2][4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float4 w = *(const float4*)sh.w1[row_d(h, ut, r4 + k)];
                const float c0 = __builtin_fmaf(w.x, x0, w.z);
#pragma unroll
                for (int nt = 0; nt < 2; ++nt) {
                    float z = __builtin_fmaf(w.y, x1[nt], c0);
                    if (D == 3) z = __builtin_fmaf(w.w, x2[nt], z);
                    h1f[nt][r4 + k] = tanh_fast(z);
                    v4[nt][k] = (__bf16)h1f[nt][r4 + k];
                }
            }
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
                __builtin_memcpy(&h1[own + 32 * nt * kRowPad + row_d(h, ut, r4)], v4[nt], 8);
        }
        __syncthreads();
        f32x16 z[2];
#pragma unroll
        for (int r4 = 0; r4 < 16; r4 += 4) {
            four(z[0], r4, sh.b2 + row_d(h, ut, r4));
            four(z[1], r4, sh.b2 + row_d(h, ut, r4));
        }
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)          // two chains of products side by side
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                const bf16x8 b = *(const bf16x8*)&h1[own + 32 * nt * kRowPad + 16 * kb + 8 * h];
                z[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[kb], b, z[nt], 0, 0, 0);
            }
#pragma unroll
        for (int r4 = 0; r4 < 16; r4 += 4) {
            const float4 w4 = *(const float4*)(sh.w3 + row_d(h, ut, r4));
            const float w3[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                __bf16 v4[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int r = r4 + k;
                    const float hv = tanh_fast(z[nt][r]), dd = 1.0f - hv * hv;
                    gw3[r] = __builtin_fmaf(dy[nt], hv, gw3[r]);
                    gb2[r] = __builtin_fmaf(dy[nt], dd, gb2[r]);
                    v4[k] = (__bf16)(dy[nt] * w3[k] * dd);
                }
                __builtin_memcpy(&d2[own + 32 * nt * kRowPad + row_d(h, ut, r4)], v4, 8);
            }
        }
        __syncthreads();
        // e1 = W2^T d2, and gW2 as G[j][u] += d2[j][p] h1[u][p] over the 64
        // points (unit tile ut): four chains of products
        f32x16 e1[2];
#pragma unroll
        for (int r = 0; r < 16; ++r) e1[0][r] = e1[1][r] = 0.0f;
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                const bf16x8 b = *(const bf16x8*)&d2[own + 32 * nt * kRowPad + 16 * kb + 8 * h];
                e1[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ab[kb], b, e1[nt], 0, 0, 0);
            }
            const bf16x8 u = read_tr(h1 + tr, kb, ut);
#pragma unroll
            for (int jt = 0; jt < 2; ++jt)
                G[jt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_tr(d2 + tr, kb, jt), u, G[jt], 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float d10 = e1[0][r] * (1.0f - h1f[0][r] * h1f[0][r]);
            const float d11 = e1[1][r] * (1.0f - h1f[1][r] * h1f[1][r]);
            const float sum = d10 + d11;
            gb1[r] += sum;
            gw1[0][r] = __builtin_fmaf(x0, sum, gw1[0][r]);
            gw1[1][r] = __builtin_fmaf(d10, x1[0], __builtin_fmaf(d11, x1[1], gw1[1][r]));
            if (D == 3)
                gw1[D - 1][r] = __builtin_fmaf(d10, x2[0], __builtin_fmaf(d11, x2[1], gw1[D - 1][r]));
        }
    }
    // the block's row: a unit's sums over the 32 lanes of its half
    const bool add = a.first != 0 || a.task0 != 0;
    auto put = [&](int i, float v) { grow[i] = add ? grow[i] + v : v; };
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int u = row_d(h, ut, r);
        const float s3 = sum32(gw3[r]), s2 = sum32(gb2[r]), s1 = sum32(gb1[r]);
        float w1s[D];
#pragma unroll
        for (int d = 0; d < D; ++d) w1s[d] = sum32(gw1[d][r]);
        if (col == 0) {
            put(off_w3(D) + u, s3);
            put(off_b2(D) + u, s2 * sh.w3[u]);
            put(off_b1(D) + u, s1);
#pragma unroll
            for (int d = 0; d < D; ++d) put(u * D + d, w1s[d]);
        }
#pragma unroll
        for (int jt = 0; jt < 2; ++jt)          // rows of G are layer-2 units, columns (lanes) layer-1 units
            put(off_W2(D) + row_d(h, jt, r) * H + 32 * ut + col, G[jt][r]);
    }
    gb3 = sum32(gb3);                           // every half wave holds all the points
    if (threadIdx.x == 0) put(off_b3(D), gb3);
}

// ----------------------------------------------------------------- update
struct AdamArgs {
    float *params, *m1, *m2;
    bf16x8 *afwd, *abwd;
    float lr, b1, b2, eps, c1, c2;
};

// Sum of the partial rows (fixed order: 32 runs of rows, then the runs) and,
// with `step`, Adam (Kingma and Ba 2015) on the fp32 master parameters and
// the new W2 in both operand arrays; the gradient goes to grad.  32
// parameters per block, 32 runs of rows side by side.
__global__ __launch_bounds__(1024) void train_update_kernel(const float* gpart, int rows, int D, float* grad,
                                                            AdamArgs p, int step)
{
    __shared__ float part[32][33];
    const int np = nparams(D);
    const int col = threadIdx.x & 31, run = threadIdx.x >> 5;
    const int i = blockIdx.x * 32 + col;        // < kGradRow
    const int per = (rows + 31) / 32;
    const int r1 = (run + 1) * per < rows ? (run + 1) * per : rows;
    float s = 0.0f;
    if (i < np) {
#pragma unroll 8
        for (int r = run * per; r < r1; ++r) s += gpart[(uint64_t)r * kGradRow + i];
    }
    part[run][col] = s;
    __syncthreads();
    if (run || i >= np) return;
    float g = 0.0f;
#pragma unroll
    for (int r = 0; r < 32; ++r) g += part[r][col];
    grad[i] = g;
    if (!step) return;
    const float a = p.b1 * p.m1[i] + (1.0f - p.b1) * g;
    const float v = p.b2 * p.m2[i] + (1.0f - p.b2) * g * g;
    p.m1[i] = a;
    p.m2[i] = v;
    const float q = p.params[i] - p.lr * (a / p.c1) / (sqrtf(v / p.c2) + p.eps);
    p.params[i] = q;
    const int w = i - off_W2(D);
    if (w >= 0 && w < H * H) {
        const int j = w / H, k = w % H;         // W2[j][k]
        ((__bf16*)p.afwd)[w2_operand_at(j, k)] = (__bf16)q;
        ((__bf16*)p.abwd)[w2_operand_at(k, j)] = (__bf16)q;
    }
}

// ------------------------------------------------------------------- host
using TrainPathsFn = void (*)(TrainArgs, NetConsts, int);

template <int MODEL>
static TrainPathsFn pick_paths(int payoff, int M)
{
    switch (payoff) {
    case kCall: return M == 2 ? train_paths_kernel<MODEL, kCall, 2> : train_paths_kernel<MODEL, kCall, 4>;
    case kAsian: return M == 2 ? train_paths_kernel<MODEL, kAsian, 2> : train_paths_kernel<MODEL, kAsian, 4>;
    case kLookback:
        return M == 2 ? train_paths_kernel<MODEL, kLookback, 2> : train_paths_kernel<MODEL, kLookback, 4>;
    default: return M == 2 ? train_paths_kernel<MODEL, kDigital, 2> : train_paths_kernel<MODEL, kDigital, 4>;
    }
}

// Runs a sample's sums of phi dW are taken in on a level of nf steps: a power
// of two dividing its generator groups, while 64 samples of one run each make
// at most 2048 pieces of the batch.
static uint32_t sum_runs(uint64_t B, uint64_t nf)
{
    const uint64_t groups = (nf + 3) / 4, pieces = (B + 63) / 64;
    uint32_t runs = 1;
    while (2ull * runs <= groups && groups % (2ull * runs) == 0 && pieces * runs * 2 <= 2048) runs *= 2;
    return runs;
}

// The scratch of one step, cut from cv->d_train (256-byte pieces).
struct TrainScratch {
    float *x1, *x2, *c, *phi, *x0;
    float2 *pay, *c0;
    double* y;
    float* phi0;
    LevelAcc* rec;
    float *gpart, *grad;
    size_t bytes;
};

static TrainScratch cut_scratch(char* base, uint64_t nrows, uint64_t stride, int nlev, uint64_t Bpad, int D,
                                int grows, uint64_t group)
{
    TrainScratch s;
    size_t at = 0;
    auto take = [&](size_t bytes) {
        char* p = base + at;
        at += (bytes + 255) / 256 * 256;
        return p;
    };
    const size_t pts = nrows * stride * sizeof(float);
    s.x1 = (float*)take(group * pts);
    s.x2 = (float*)take(D == 3 ? group * pts : 0);
    s.c = (float*)take(group * pts);
    s.phi = (float*)take(pts);
    s.x0 = (float*)take(nrows * sizeof(float));
    s.pay = (float2*)take(group * nlev * stride * sizeof(float2));
    s.c0 = (float2*)take(group * nlev * stride * sizeof(float2));
    s.y = (double*)take(nlev * Bpad * sizeof(double));
    s.phi0 = (float*)take(sizeof(float));
    s.rec = (LevelAcc*)take(group * nlev * sizeof(LevelAcc));
    s.gpart = (float*)take((size_t)grows * kGradRow * sizeof(float));
    s.grad = (float*)take(kGradRow * sizeof(float));
    s.bytes = at;
    return s;
}

// The evaluations of steps step .. step + nsteps - 1 of a batch of B samples
// per level: sizes, scratch and the arguments common to all of them.
struct TrainPlan {
    TrainArgs a;
    TrainScratch s;
    uint64_t chunk;      // samples worked off at once
    uint32_t group;      // steps whose paths one launch makes (1 with chunks)
    uint32_t parts;      // backward launches of a chunk
    int nb, ns;          // backward blocks: points, start point
    NetConsts nc;
    TrainPathsFn paths;
};

// Samples per chunk (`most` of them at most, rounded down to whole waves), the
// steps in a group and the backward blocks.
static void size_chunk(TrainPlan& t, int num_cu, uint64_t most, int nsteps)
{
    const TrainArgs& a = t.a;
    const uint64_t nrows = a.nrows;
    t.chunk = std::min<uint64_t>(a.Bpad, std::max<uint64_t>(64, most / 64 * 64));
    const uint64_t pts = std::max<uint64_t>(t.chunk * std::max<uint64_t>(nrows, (uint64_t)a.nlev), 1);
    t.group = t.chunk < a.B ? 1u
                            : (uint32_t)std::max<uint64_t>(
                                  1, std::min<uint64_t>({(uint64_t)nsteps, kMaxPoints / pts, (uint64_t)kMaxSteps}));
    // backward blocks: the start point's, and beside them what fills the
    // device's residency (one more would wait for another's end) or a task each
    // so that both kinds end together: one start block in fifty for
    // 16384 samples on levels 0..3, one in four on levels 0..1
    const uint64_t resident = (uint64_t)num_cu * kBwdBlocksPerCu, tasks = nrows * (t.chunk / 64);
    const uint64_t pairs = t.chunk * a.nlev;
    const double sc = kStartPairCost * (double)pairs, share = sc / (sc + kTaskCost * (double)tasks);
    // (times the chunk's backward launches: the start point is worked off beside
    // the first of them, and a block of it sums as many samples as in one of
    // kMaxPoints)
    t.parts = (uint32_t)std::max<uint64_t>(1, (nrows * t.chunk + kMaxPoints - 1) / kMaxPoints);
    t.ns = (int)std::max<uint64_t>(1, std::min<uint64_t>({(uint64_t)(share * (double)resident + 0.5),
                                                          (pairs + 127) / 128, resident / 2}));
    t.ns = (int)std::min<uint64_t>({(uint64_t)t.ns * t.parts, (pairs + 127) / 128, resident / 2});
    t.nb = (int)std::min<uint64_t>(tasks, resident - t.ns);
}

static mlmc_status plan_train(mlmc_cv* cv, const mlmc_model& m, const mlmc_payoff& p, int M, int lmax, uint64_t B,
                              uint64_t seed, int nsteps, TrainPlan* out)
{
    mlmc_ctx* ctx = cv->ctx;
    TrainPlan& t = *out;
    TrainArgs& a = t.a;
    std::memset(&a, 0, sizeof(a));
    a.nlev = lmax + 1;
    a.M = M;
    uint64_t nrows = 0, nf = 1;
    for (int l = 0; l <= lmax; ++l, nf *= M) {
        TrainLevel& L = a.lev[l];
        L.P = make_step_params<float>(m, p, l, M);
        L.nf = (int)nf;
        L.ngroups = (int)((nf + 3) / 4);
        L.row0 = (uint32_t)nrows;
        L.runs = sum_runs(B, nf);
        nrows += (nf - 1) + (l ? nf / M - 1 : 0);
    }
    a.nrows = (uint32_t)nrows;
    a.B = B;
    a.Bpad = (B + 63) / 64 * 64;
    a.seed = seed;
    a.S0 = (float)m.S0;
    a.v0 = (float)m.v0;
    // Samples per chunk: whole waves, as many as fit kMaxPoints, but kTrainChunk
    // at least while the memory is there (halved on each refusal, for the
    // network's later steps as well).
    for (;; cv->train_least /= 2) {
        const uint64_t least = cv->train_least;
        size_chunk(t, ctx->num_cu, std::max<uint64_t>(least, kMaxPoints / std::max<uint64_t>(nrows, 1)), nsteps);
        t.s = cut_scratch(nullptr, nrows, t.chunk, a.nlev, a.Bpad, cv->D, t.nb + t.ns, t.group);
        if (cv->train_cap >= t.s.bytes) break;
        // queued launches may still use the old scratch
        MLMC_HIP(ctx, hipStreamSynchronize(ctx->stream));
        if (cv->d_train) hipFree(cv->d_train);
        cv->d_train = nullptr;
        cv->train_cap = 0;
        const hipError_t e = hipMalloc(&cv->d_train, t.s.bytes);
        if (e == hipSuccess) {
            cv->train_cap = t.s.bytes;
            break;
        }
        cv->d_train = nullptr;
        if (e != hipErrorOutOfMemory || least <= 64 || t.chunk * nrows <= kMaxPoints)
            return hip_fail(ctx, e, "training scratch allocation");
        (void)hipGetLastError();
    }
    t.s = cut_scratch(cv->d_train, nrows, t.chunk, a.nlev, a.Bpad, cv->D, t.nb + t.ns, t.group);
    a.x1 = t.s.x1;
    a.x2 = t.s.x2;
    a.c = t.s.c;
    a.phi = t.s.phi;
    a.x0 = t.s.x0;
    a.pay = t.s.pay;
    a.c0 = t.s.c0;
    a.y = t.s.y;
    a.phi0 = t.s.phi0;
    a.rec = t.s.rec;
    t.nc = net_consts(m);
    t.paths = m.kind == MLMC_GBM ? pick_paths<kGBM>(p.kind, M) : pick_paths<kHeston>(p.kind, M);
    return MLMC_OK;
}

// The chunk of step `step` from sample `first` of the batch; returns its
// blocks of 256 samples.
static uint32_t set_chunk(TrainPlan& t, uint64_t step, uint64_t first)
{
    TrainArgs& a = t.a;
    a.first = (uint32_t)first;
    a.offset = step * a.B + first;
    a.n = (uint32_t)std::min(t.chunk, a.B - first);
    a.stride = (a.n + 63) / 64 * 64;
    const uint32_t per = (a.stride + 255) / 256;
    for (int l = 0; l < a.nlev; ++l) a.lev[l].blk0 = (uint32_t)(a.nlev - 1 - l) * per;   // deepest first
    return per * (uint32_t)a.nlev;
}

// One loss/gradient evaluation (and, with adam, the parameter update),
// enqueued on the context's stream: step `step`, number k of a group of
// `group` whose paths the group's first evaluation makes.  hist: device
// address that receives the loss, or null.
static mlmc_status enqueue_loss_grad(mlmc_cv* cv, TrainPlan& t, uint64_t step, uint32_t k, uint32_t group,
                                     const AdamArgs* adam, double* hist)
{
    mlmc_ctx* ctx = cv->ctx;
    const hipStream_t q = ctx->stream;
    const uint64_t B = t.a.B;
    const bool d3 = cv->D == 3, one_chunk = t.chunk >= B;
    const CvKernelArgs c{cv->d_params, cv->d_afwd, t.nc, cv->D};
    for (uint64_t first = 0; first < B; first += t.chunk) {
        const uint32_t blocks = set_chunk(t, step - k, first);
        if (k == 0) {
            hipLaunchKernelGGL(t.paths, dim3(blocks, group), dim3(256), 0, q, t.a, t.nc, first == 0 ? 1 : 0);
            MLMC_HIP(ctx, hipGetLastError());
        }
        const TrainArgs a = for_step(t.a, k);
        const uint64_t waves = (uint64_t)a.nrows * (a.stride / 64) + 1;
        const unsigned grid = (unsigned)std::min<uint64_t>((waves + 3) / 4, (uint64_t)ctx->num_cu * kFwdBlocksPerCu);
        hipLaunchKernelGGL(d3 ? train_forward_kernel<3> : train_forward_kernel<2>, dim3(grid), dim3(256), 0, q, a, c);
        MLMC_HIP(ctx, hipGetLastError());
        hipLaunchKernelGGL(train_combine_kernel, dim3(a.stride / 64 * (uint32_t)a.nlev), dim3(256), 0, q, a);
        MLMC_HIP(ctx, hipGetLastError());
    }
    const int tix = timed_begin(ctx, 18, 0.0, 0.0);
    for (uint64_t first = 0; first < B; first += t.chunk) {
        const uint32_t blocks = set_chunk(t, step - k, first);
        if (!one_chunk) {
            hipLaunchKernelGGL(t.paths, dim3(blocks), dim3(256), 0, q, t.a, t.nc, 0);
            MLMC_HIP(ctx, hipGetLastError());
        }
        TrainArgs a = for_step(t.a, k);
        const uint32_t total = a.nrows * (a.stride / 64);
        for (uint32_t part = 0; part < t.parts; ++part) {
            a.task0 = (uint32_t)((uint64_t)total * part / t.parts);
            a.tasks = (uint32_t)((uint64_t)total * (part + 1) / t.parts) - a.task0;
            if (part && !a.tasks) continue;
            hipLaunchKernelGGL(d3 ? train_backward_kernel<3> : train_backward_kernel<2>, dim3(t.nb + t.ns), dim3(128),
                               0, q, a, c, (const bf16x8*)cv->d_abwd, t.s.gpart, (uint32_t)t.ns, cv->d_loss, hist);
            MLMC_HIP(ctx, hipGetLastError());
        }
    }
    hipLaunchKernelGGL(train_update_kernel, dim3((cv->np + 31) / 32), dim3(1024), 0, q, (const float*)t.s.gpart,
                       t.nb + t.ns, cv->D, t.s.grad, adam ? *adam : AdamArgs{}, adam ? 1 : 0);
    MLMC_HIP(ctx, hipGetLastError());
    timed_end(ctx, tix);
    return MLMC_OK;
}

static mlmc_status check_train_args(mlmc_cv* cv, const mlmc_model* m, const mlmc_payoff* p, int M,
                                    int lmax, uint64_t B)
{
    mlmc_ctx* ctx = cv->ctx;
    mlmc_status st = check_level_args(ctx, m, p, lmax < 0 ? 0 : lmax, M, 32);
    if (st) return st;
    if (lmax < 0 || lmax > 6) return fail(ctx, MLMC_EINVAL, "lmax must be in 0..6");
    if (B < 2 || B > (1ull << 24)) return fail(ctx, MLMC_EINVAL, "batch must be in 2..2^24 per level");
    if (cv->D != (m->kind == MLMC_HESTON ? 3 : 2))
        return fail(ctx, MLMC_EINVAL, "network inputs do not match the model (2: GBM, 3: Heston)");
    if (m->scheme != MLMC_EULER || m->antithetic || p->kind == MLMC_DIGITAL_COND)
        return fail(ctx, MLMC_EINVAL, "the control variate trains on plain Euler paths and payoffs");
    return MLMC_OK;
}

}  // namespace mlmc

using namespace mlmc;

extern "C" {

mlmc_status mlmc_cv_loss_grad(mlmc_cv* cv, const mlmc_model* model, const mlmc_payoff* payoff,
                              int M, int lmax, uint64_t batch, uint64_t seed, uint64_t step,
                              float* grad, double* var, double* loss)
{
    if (!cv) return MLMC_EINVAL;
    mlmc_ctx* ctx = cv->ctx;
    mlmc_status st = check_train_args(cv, model, payoff, M, lmax, batch);
    if (st) return st;
    ctx->err.clear();
    MLMC_ENTER(ctx);
    TrainPlan t;
    st = plan_train(cv, *model, *payoff, M, lmax, batch, seed, 1, &t);
    if (!st) st = enqueue_loss_grad(cv, t, step, 0, 1, nullptr, nullptr);
    if (st) return st;
    if (grad)
        MLMC_HIP(ctx, hipMemcpyAsync(grad, t.s.grad, sizeof(float) * cv->np, hipMemcpyDeviceToHost,
                                     ctx->stream));
    double hl[64];
    MLMC_HIP(ctx, hipMemcpyAsync(hl, cv->d_loss, sizeof(hl), hipMemcpyDeviceToHost, ctx->stream));
    MLMC_HIP(ctx, hipStreamSynchronize(ctx->stream));
    harvest_timing(ctx);
    if (loss) *loss = hl[0];
    if (var)
        for (int l = 0; l <= lmax; ++l) var[l] = hl[1 + l];
    return MLMC_OK;
}

mlmc_status mlmc_cv_train(mlmc_cv* cv, const mlmc_model* model, const mlmc_payoff* payoff, int M,
                          int lmax, int steps, uint64_t batch, double lr, uint64_t seed,
                          float* loss_hist)
{
    if (!cv) return MLMC_EINVAL;
    mlmc_ctx* ctx = cv->ctx;
    mlmc_status st = check_train_args(cv, model, payoff, M, lmax, batch);
    if (st) return st;
    if (steps < 0 || !(lr > 0)) return fail(ctx, MLMC_EINVAL, "need steps >= 0 and lr > 0");
    ctx->err.clear();
    MLMC_ENTER(ctx);
    double* d_hist = nullptr;
    if (loss_hist && steps > 0) MLMC_HIP(ctx, hipMalloc(&d_hist, sizeof(double) * steps));
    AdamArgs adam{cv->d_params, cv->d_m1, cv->d_m2, cv->d_afwd, cv->d_abwd, (float)lr,
                  0.9f, 0.999f, 1e-8f, 0.0f, 0.0f};
    TrainPlan t;
    st = plan_train(cv, *model, *payoff, M, lmax, batch, seed, steps, &t);
    for (int k = 0; k < steps && !st; ++k) {
        const TraceRange step_range("mlmc_cv_train step");
        const uint32_t in_group = (uint32_t)k % t.group;
        const uint32_t group = std::min<uint32_t>(t.group, (uint32_t)steps - ((uint32_t)k - in_group));
        adam.c1 = 1.0f - std::pow(adam.b1, (float)(cv->adam_t + 1));
        adam.c2 = 1.0f - std::pow(adam.b2, (float)(cv->adam_t + 1));
        // each step draws fresh training samples: indices t * batch .. (t+1) * batch - 1
        st = enqueue_loss_grad(cv, t, (uint64_t)cv->adam_t, in_group, group, &adam, d_hist ? d_hist + k : nullptr);
        if (st) break;
        cv->adam_t += 1;
        ++cv->version;
    }
    if (!st && d_hist) {
        std::vector<double> h(steps);
        hipError_t e = hipMemcpyAsync(h.data(), d_hist, sizeof(double) * steps,
                                      hipMemcpyDeviceToHost, ctx->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
        if (e != hipSuccess) st = hip_fail(ctx, e, "loss history copy");
        for (int k = 0; k < steps; ++k) loss_hist[k] = (float)h[k];
    }
    if (!st) {
        hipError_t e = hipStreamSynchronize(ctx->stream);
        if (e != hipSuccess) st = hip_fail(ctx, e, "training");
        harvest_timing(ctx);
    }
    if (d_hist) hipFree(d_hist);
    return st;
}

}  // extern "C"
