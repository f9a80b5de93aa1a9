// Learned martingale control variate: the MLP phi(t, X) evaluated for the 64
// samples of a wavefront at once, layer 2 on the bf16 matrix cores.
//
// The control variate is the discrete martingale sum_n phi(t_n, X_n) dW_n
// (left-point evaluation, so every term has conditional mean zero and the
// level estimators of eqs. (eq:mlmc:Yzero), (eq:Yldef) keep their means; the
// control-variate idea is Sec. 5, "Exploiting Structure").  Network:
//   x = (t/T, ln(max(S, S0 2^-40)/S0)/(sref sqrt T) [, (v - theta)/theta])
//   h1 = tanh(W1 x + b1), h2 = tanh(W2 h1 + b2), phi = sref S0 (w3.h2 + b3)
// with H = 64 hidden units.  Layer 1 and 3 run in fp32 on the vector ALUs;
// layer 2 is a 64x64x64 product per evaluation (units x units x samples) on
// v_mfma_f32_32x32x16_bf16: W2 and h1 in bf16, fp32 accumulation.
//
// Lane layouts (wave of 64 lanes, lane l, half h = l / 32):
//   bf16 B operand (K = 16 units x N = 32 samples): lane l holds column
//     n = l % 32, rows 8h + i (i < 8) of the K block;
//   A operand (M = 32 rows x K = 16): lane l holds row l % 32, columns
//     8h + i;
//   fp32 accumulator (32 x 32): register r of lane l is row
//     8 (r / 4) + 4h + r % 4, column l % 32.
// Sample p of the wave lives in lane p.  Lane l computes layer 1 for samples
// l % 32 and 32 + l % 32 (its own and lane l ^ 32's), at the 32 units
// unit_b(h, s) of its B-operand slots s = 8 kb + i, so no data moves between
// layer 1 and the matrix product; layer 3 sums each half-column of h2 and one
// exchange with lane l ^ 32 completes phi.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mlmc {
namespace cvnet {

constexpr int H = 64;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Unit at B-operand slot s (0..31) of lane half h (k block s / 8, element s % 8).
__host__ __device__ constexpr int unit_b(int h, int s) { return 16 * (s / 8) + 8 * h + s % 8; }
// Row of accumulator register r (0..15) of row tile t for lane half h.
__host__ __device__ constexpr int row_d(int h, int t, int r) { return 32 * t + 8 * (r / 4) + 4 * h + r % 4; }

// Parameter offsets in the flat vector (same order as the CPU reference):
// W1[H][D], b1[H], W2[H][H] (row = output unit), b2[H], w3[H], b3.
__host__ __device__ constexpr int off_b1(int D) { return H * D; }
__host__ __device__ constexpr int off_W2(int D) { return H * D + H; }
__host__ __device__ constexpr int off_b2(int D) { return H * D + H + H * H; }
__host__ __device__ constexpr int off_w3(int D) { return H * D + 2 * H + H * H; }
__host__ __device__ constexpr int off_b3(int D) { return H * D + 3 * H + H * H; }
__host__ __device__ constexpr int nparams(int D) { return H * D + 3 * H + H * H + 1; }

// Network constants shared by a block (loaded into LDS once); read four
// floats at a time.
struct alignas(16) NetShared {
    float w1[H][4];       // unit u: weights of t and log S, b1[u], weight of v (or 0)
    float b2[H], w3[H];
    float b3, scale;      // scale = sref * S0
    float x1a, x1b;       // x1 = log2(max(S, floor)) * x1a - x1b
    float x2a, x2b;       // x2 = v * x2a - x2b
    float inv_T, s_floor;
};

// Host-side description of the network inputs and output scale.
struct NetConsts {
    float scale, x1a, x1b, x2a, x2b, inv_T, s_floor;
};

__device__ __forceinline__ float tanh_fast(float x)
{
    // 1 - 2 / (e^{2x} + 1); e^{2x} = 2^{2x log2 e}.  Exact limits +-1.
    const float e = __builtin_amdgcn_exp2f(x * 2.8853900817779268f);
    return __builtin_fmaf(-2.0f, __builtin_amdgcn_rcpf(e + 1.0f), 1.0f);
}

template <int D>
__device__ __forceinline__ void load_shared(NetShared& sh, const float* params, const NetConsts& c)
{
    for (int i = threadIdx.x; i < H; i += blockDim.x) {
        sh.w1[i][0] = params[i * D];
        sh.w1[i][1] = params[i * D + 1];
        sh.w1[i][2] = params[off_b1(D) + i];
        sh.w1[i][3] = D == 3 ? params[i * D + 2] : 0.0f;
        sh.b2[i] = params[off_b2(D) + i];
        sh.w3[i] = params[off_w3(D) + i];
    }
    if (threadIdx.x == 0) {
        sh.b3 = params[off_b3(D)];
        sh.scale = c.scale;
        sh.x1a = c.x1a;
        sh.x1b = c.x1b;
        sh.x2a = c.x2a;
        sh.x2b = c.x2b;
        sh.inv_T = c.inv_T;
        sh.s_floor = c.s_floor;
    }
}

// Element W2[j][k] in the A operand array of a product W2 b, kept in lane
// order: afwd[(jt * 4 + kb) * 64 + lane][i] = W2[32 jt + l%32][16 kb + 8h + i].
__host__ __device__ constexpr int w2_operand_at(int j, int k)
{
    return (((j / 32) * 4 + k / 16) * 64 + (k % 16) / 8 * 32 + j % 32) * 8 + k % 8;
}

// Registers r .. r + 3 of an accumulator from four consecutive floats (rows
// row_d(h, t, r) .. + 3).
__device__ __forceinline__ void four(f32x16& acc, int r, const float* p)
{
    const float4 v = *(const float4*)p;
    acc[r] = v.x;
    acc[r + 1] = v.y;
    acc[r + 2] = v.z;
    acc[r + 3] = v.w;
}

// Network inputs x1 (and x2) of one sample; x0 = t/T is wave-uniform.
__device__ __forceinline__ float input_x1(const NetShared& sh, float S)
{
    const float s = S > sh.s_floor ? S : sh.s_floor;
    return __builtin_fmaf(__builtin_amdgcn_logf(s), sh.x1a, -sh.x1b);
}

// Layer-1 activations of the lane's two samples, packed as B operands.
// x0 is the time input of both samples (wave-uniform in the samplers); with
// X0LANE the two samples have their own, x0p[nt].
template <int D, bool X0LANE = false>
__device__ __forceinline__ void layer1(const NetShared& sh, float x0, const float (&x1)[2],
                                       const float (&x2)[2], bf16x8 (&b)[2][4],
                                       const float* x0p = nullptr)
{
    const int h = (threadIdx.x & 63) >> 5;
#pragma unroll
    for (int s = 0; s < 32; ++s) {
        const float4 w = *(const float4*)sh.w1[unit_b(h, s)];
        const float c = __builtin_fmaf(w.x, x0, w.z);
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            const float cn = X0LANE ? __builtin_fmaf(w.x, x0p[nt], w.z) : c;
            float a = __builtin_fmaf(w.y, x1[nt], cn);
            if (D == 3) a = __builtin_fmaf(w.w, x2[nt], a);
            b[nt][s / 8][s % 8] = (__bf16)tanh_fast(a);
        }
    }
}

// Samples handled by this lane's two B columns: nt = h is its own sample,
// nt = 1 - h the sample of lane l ^ 32.
template <int D>
__device__ __forceinline__ void pair_inputs(float own1, float own2, float (&x1)[2], float (&x2)[2])
{
    const int h = (threadIdx.x & 63) >> 5;
    const float oth1 = __shfl_xor(own1, 32);
    x1[0] = h == 0 ? own1 : oth1;
    x1[1] = h == 0 ? oth1 : own1;
    if (D == 3) {
        const float oth2 = __shfl_xor(own2, 32);
        x2[0] = h == 0 ? own2 : oth2;
        x2[1] = h == 0 ? oth2 : own2;
    } else {
        x2[0] = x2[1] = 0.0f;
    }
}

// phi of this lane's sample from its network inputs; every lane of the wave
// must call it.  afwd: the bf16 W2 operands in lane order (in LDS in the
// sampler).  Layer 2 and layer 3 run one 32-row tile at a time, so only half
// of the matrix accumulators are live.
template <int D, bool X0LANE = false>
__device__ __forceinline__ float phi_eval_x(const NetShared& sh, const bf16x8* afwd, float x0,
                                            float own1, float own2)
{
    // The network constants are read from LDS at every evaluation: kept in
    // registers across the path loop they would take ~190 VGPRs and leave a
    // single wave per SIMD.  The empty asm (a compiler-only memory clobber,
    // no instruction) stops the loads from being hoisted out of the loop.
    __asm__ volatile("" ::: "memory");
    const int lane = threadIdx.x & 63;
    const int h = lane >> 5;
    float x1[2], x2[2];
    pair_inputs<D>(own1, own2, x1, x2);
    bf16x8 b[2][4];
    float x0p[2] = {x0, x0};
    if (X0LANE) {
        // this lane's sample and lane l ^ 32's, in B-column order
        const float oth = __shfl_xor(x0, 32);
        x0p[0] = h == 0 ? x0 : oth;
        x0p[1] = h == 0 ? oth : x0;
    }
    layer1<D, X0LANE>(sh, x0, x1, x2, b, x0p);
    float part[2] = {0.0f, 0.0f};
#pragma unroll
    for (int jt = 0; jt < 2; ++jt) {
        bf16x8 a[4];
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) a[kb] = afwd[(jt * 4 + kb) * 64 + lane];
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            f32x16 acc;
#pragma unroll
            for (int r = 0; r < 16; r += 4) four(acc, r, sh.b2 + row_d(h, jt, r));
#pragma unroll
            for (int kb = 0; kb < 4; ++kb)
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kb], b[nt][kb], acc, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 16; r += 4) {
                const float4 w3 = *(const float4*)(sh.w3 + row_d(h, jt, r));
                part[nt] = __builtin_fmaf(w3.x, tanh_fast(acc[r]), part[nt]);
                part[nt] = __builtin_fmaf(w3.y, tanh_fast(acc[r + 1]), part[nt]);
                part[nt] = __builtin_fmaf(w3.z, tanh_fast(acc[r + 2]), part[nt]);
                part[nt] = __builtin_fmaf(w3.w, tanh_fast(acc[r + 3]), part[nt]);
            }
        }
    }
    const float send = h == 0 ? part[1] : part[0];
    const float recv = __shfl_xor(send, 32);
    const float mine = h == 0 ? part[0] : part[1];
    return sh.scale * (mine + recv + sh.b3);
}

// phi(t, X) of this lane's sample.
template <int D, bool X0LANE = false>
__device__ __forceinline__ float phi_eval(const NetShared& sh, const bf16x8* afwd, float x0,
                                          float S, float v)
{
    return phi_eval_x<D, X0LANE>(sh, afwd, x0, input_x1(sh, S),
                                 D == 3 ? __builtin_fmaf(v, sh.x2a, -sh.x2b) : 0.0f);
}

// ------------------------------------------------------------ tabulated
// The sampler may read phi from a table instead of evaluating the network at
// every point: phi on a grid of `rows` times t_j = j T / rows, ns stock values
// S_i = s_lo + i dS (and nv variances v_k = v_lo + k dv for Heston), filled by
// the network itself (cv_table_kernel), and interpolated linearly in S (and v)
// within the row of the last grid time at or before the evaluation time.  Any
// function of (t_n, X_n) keeps the control variate's mean at zero, so the
// table changes only how much variance it removes, not the level means.
struct TableSpec {
    int rows, ns, nv;
    float s_lo, s_inv;    // u = (S - s_lo) s_inv, grid index in S
    float v_lo, v_inv;    // w = (v - v_lo) v_inv (nv > 1)
};

// Row of step n of a path with nf fine steps: floor(n rows / nf).
__device__ __forceinline__ int table_row(int n, int nf, int rows)
{
    return (int)(((unsigned)n * (unsigned)rows) / (unsigned)nf);
}

// Linear (bilinear for nv > 1) interpolation in one row; points outside the
// grid take the nearest edge of it (a non-finite S or v reads the low edge:
// fmin/fmax return the other operand of a NaN, so the index stays in range).
__device__ __forceinline__ float table_phi(const float* tab, const TableSpec& t, int row, float S,
                                           float v)
{
    const float u = __builtin_fminf(__builtin_fmaxf((S - t.s_lo) * t.s_inv, 0.0f), (float)(t.ns - 1));
    const int i = min((int)u, t.ns - 2);
    const float f = u - (float)i;
    if (t.nv == 1) {
        const float* r = tab + row * t.ns + i;
        return __builtin_fmaf(f, r[1] - r[0], r[0]);
    }
    const float w = __builtin_fminf(__builtin_fmaxf((v - t.v_lo) * t.v_inv, 0.0f), (float)(t.nv - 1));
    const int k = min((int)w, t.nv - 2);
    const float g = w - (float)k;
    const float* r = tab + (row * t.nv + k) * t.ns + i;
    const float a = __builtin_fmaf(f, r[1] - r[0], r[0]);
    const float b = __builtin_fmaf(f, r[t.ns + 1] - r[t.ns], r[t.ns]);
    return __builtin_fmaf(g, b - a, a);
}

}  // namespace cvnet
}  // namespace mlmc
