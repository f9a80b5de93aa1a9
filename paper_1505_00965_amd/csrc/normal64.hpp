// Box--Muller in fp64 on 24-bit uniforms, for the fp64 sampler.
//
// Both uniforms are odd multiples of 2^-25, so neither function meets a
// special value, a denormal or a large argument, and the general library
// routines (two head-and-tail logarithm and sine/cosine expansions: 97 vector
// instructions per fine step, 195 us for 2^20 samples of level 3, M = 4; with these
// 44 and 102) do more
// than is needed.  Here:
//   -2 ln u:  u = z 2^e with z in [0.69, 1.39) and a table of 64 intervals of
//             z (1/c short enough that r = z/c - 1 is exact; c = 1 around
//             z = 1, so small logarithms keep their relative accuracy), then
//             a polynomial in r: the table-driven logarithm of P. T. P. Tang
//             (ACM TOMS 16, 1990);
//   cos, sin: a table of 64 angles and the exact residual, at most pi/64, by
//             polynomials and the addition theorem, the angles chosen so that
//             the tabulated values are nearly exact (the accurate tables of S.
//             Gal and B. Bachelis, ACM TOMS 17, 1991; the logarithm's too);
//   sqrt:     the hardware's reciprocal square root and Goldschmidt's iteration
//             with a last correction by the exact residual (P. W. Markstein,
//             IBM J. Res. Dev. 34, 1990), without scaling (the argument lies in
//             [5.9e-8, 35]).
// Largest errors over all 2^24 values: -2 ln u 0.79 ulp, cos and sin 0.61 2^-53;
// of 2^21 normals against 80-bit arithmetic, in units of rho 2^-53: 2.77, root
// mean square 0.513 (the library routines: 2.77 and 0.515).
// The 3 KiB of tables are copied into LDS by each block (load_normal_tables).
// tests/golden/make_normal_tables.py makes every constant (coefficients:
// interpolation at Chebyshev nodes in 60-digit arithmetic).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mlmc {

// {1/c, 25 kTwoLn2Hi - 2 ln c} for z in interval i, whose high word starts at
// kLogOff + i 2^14: 1/c has 26 fractional bits and is, of the values near the
// interval's centre, one whose -2 ln c lies within 2^-62 of a multiple of
// 2^-47, so that its sum with a multiple of kTwoLn2Hi is exact.
constexpr uint32_t kLogOff = 0x3fe62000u;
constexpr double kLogTable[64][2] = {
    {0x1.701f1a0000000p+0, 0x1.1b12158ecc30ap+5}, {0x1.6c30a30000000p+0, 0x1.1ae61aa246148p+5},
    {0x1.67e7eac000000p+0, 0x1.1ab5a2d70ad79p+5}, {0x1.6432b3c000000p+0, 0x1.1a8b38078809ep+5},
    {0x1.602943c000000p+0, 0x1.1a5c88733ed20p+5}, {0x1.5c696a0000000p+0, 0x1.1a30b0891f548p+5},
    {0x1.58c43e4000000p+0, 0x1.1a059c3218f12p+5}, {0x1.55309b0000000p+0, 0x1.19dae523cd090p+5},
    {0x1.51bf310000000p+0, 0x1.19b159f8ce998p+5}, {0x1.4e3dc8c000000p+0, 0x1.19869ddbe1264p+5},
    {0x1.4b1bdcc000000p+0, 0x1.19600c45bf683p+5}, {0x1.47ae6a0000000p+0, 0x1.19356d2dcda6fp+5},
    {0x1.4465e7c000000p+0, 0x1.190c2ddf3fac0p+5}, {0x1.416d618000000p+0, 0x1.18e67ee604858p+5},
    {0x1.3e01af8000000p+0, 0x1.18baabf79e991p+5}, {0x1.3b2cc48000000p+0, 0x1.1896090851177p+5},
    {0x1.383b0f8000000p+0, 0x1.186f97d9625a7p+5}, {0x1.34f442c000000p+0, 0x1.184461e7d63bap+5},
    {0x1.324f800000000p+0, 0x1.18212f0e1e9c8p+5}, {0x1.2f3e6d4000000p+0, 0x1.17f7f81c7e75ep+5},
    {0x1.2cce52c000000p+0, 0x1.17d6e819dc62cp+5}, {0x1.29c1338000000p+0, 0x1.17ad257147b6cp+5},
    {0x1.273c430000000p+0, 0x1.178a57b8e7a71p+5}, {0x1.24b8060000000p+0, 0x1.176747756cd18p+5},
    {0x1.22154a0000000p+0, 0x1.17423b2bd9d09p+5}, {0x1.1f5e548000000p+0, 0x1.171bb81592ecfp+5},
    {0x1.1cf4c10000000p+0, 0x1.16f93051f9235p+5}, {0x1.1a9b68c000000p+0, 0x1.16d748adf1801p+5},
    {0x1.17f9440000000p+0, 0x1.16b0f0170e8adp+5}, {0x1.15be130000000p+0, 0x1.16902a1d59ef4p+5},
    {0x1.137c178000000p+0, 0x1.166ebb801b106p+5}, {0x1.10e8d0c000000p+0, 0x1.1648430d4d7bfp+5},
    {0x1.0eba344000000p+0, 0x1.1627615b74c02p+5}, {0x1.0c94d24000000p+0, 0x1.1606c84a07950p+5},
    {0x1.0a5773c000000p+0, 0x1.15e47b758a0e3p+5}, {0x1.084a8c0000000p+0, 0x1.15c4d3d76ad10p+5},
    {0x1.06018ac000000p+0, 0x1.15a141faa0c2ap+5}, {0x1.04014a8000000p+0, 0x1.1581db1b32313p+5},
    {0x1.0214f20000000p+0, 0x1.156372171630dp+5}, {0x1.0000000000000p+0, 0x1.1542457337bc0p+5},
    {0x1.f837040000000p-1, 0x1.1503831de1d97p+5}, {0x1.f064eb8000000p-1, 0x1.14c37b9964c74p+5},
    {0x1.e9028d8000000p-1, 0x1.1486180a3d99ap+5}, {0x1.e210908000000p-1, 0x1.144b80a6402a5p+5},
    {0x1.da8aa00000000p-1, 0x1.140b1351ee0d5p+5}, {0x1.d472cb8000000p-1, 0x1.13d6247acfeadp+5},
    {0x1.cd70690000000p-1, 0x1.1398643f359dcp+5}, {0x1.c77ad10000000p-1, 0x1.136325fd51bbdp+5},
    {0x1.c089d60000000p-1, 0x1.13243f1818874p+5}, {0x1.bab58c8000000p-1, 0x1.12eeaa60c1593p+5},
    {0x1.b53a7b8000000p-1, 0x1.12bba402a9c8bp+5}, {0x1.aed8f70000000p-1, 0x1.127f6c4a0cca1p+5},
    {0x1.a94a3d0000000p-1, 0x1.124a3ea8a73a2p+5}, {0x1.a422f38000000p-1, 0x1.12184ee4d89f5p+5},
    {0x1.9ed4100000000p-1, 0x1.11e43a65ecbc7p+5}, {0x1.99bb0d8000000p-1, 0x1.11b194f39c02cp+5},
    {0x1.9491d78000000p-1, 0x1.117da92acf1abp+5}, {0x1.8fd4038000000p-1, 0x1.114d5f6156648p+5},
    {0x1.8ac68b8000000p-1, 0x1.111948219606cp+5}, {0x1.8601630000000p-1, 0x1.10e77cd0aee2dp+5},
    {0x1.81bfba0000000p-1, 0x1.10ba89d72fe8ap+5}, {0x1.7cd30c0000000p-1, 0x1.1085e960ed808p+5},
    {0x1.78dd808000000p-1, 0x1.105b1b04dff4dp+5}, {0x1.7429a50000000p-1, 0x1.1027ac729517bp+5},
};

// {cos, sin, -d} of 2 pi (i 2^26 + d) / 2^32: of the angles a little past
// 2 pi i / 64 one whose cosine and sine both lie within 1/100 of a half unit
// in the last place of their fp64 values.
constexpr double kTrigTable[64][3] = {
    {0x1.0000000000000p+0, 0x0.0p+0, 0.0}, {0x1.fd8833739b523p-1, 0x1.91af5392a69a9p-4, -34656.0},
    {0x1.f624a65ce06b0p-1, 0x1.8fecc3a0d3bc9p-3, -129280.0}, {0x1.e9ec7aaafe278p-1, 0x1.2972817f7f1ecp-2, -136576.0},
    {0x1.d90614a25bddep-1, 0x1.87e1571a31899p-2, -8960.0}, {0x1.c37f3971a9d96p-1, 0x1.e2e290b95e1ecp-2, -132288.0},
    {0x1.a9ae9bce714dap-1, 0x1.1c7f56a4a3e73p-1, -72992.0}, {0x1.8bbadf2f8c607p-1, 0x1.44df38f8d8118p-1, -108128.0},
    {0x1.69fc420b08970p-1, 0x1.6a178a414b2ddp-1, -100608.0}, {0x1.44c20eaf7b958p-1, 0x1.8bd2cec9710b2p-1, -88640.0},
    {0x1.1c5e9fe23fad5p-1, 0x1.a9c4771dfe99fp-1, -132192.0}, {0x1.e275f788e9068p-2, 0x1.c39c3eba56b70p-1, -188800.0},
    {0x1.87b02d9ad350bp-2, 0x1.d910428646fb6p-1, -129792.0}, {0x1.28fc248003c0bp-2, 0x1.e9fe6dec8d96ap-1, -185952.0},
    {0x1.8f13144ad02ccp-3, 0x1.f62f79401be70p-1, -160096.0}, {0x1.9088a78d8d94dp-4, 0x1.fd8bd350a2253p-1, -158368.0},
    {0x0.0p+0, 0x1.0000000000000p+0, 0.0}, {-0x1.91af5392a69a9p-4, 0x1.fd8833739b523p-1, -34656.0},
    {-0x1.8fecc3a0d3bc9p-3, 0x1.f624a65ce06b0p-1, -129280.0}, {-0x1.2972817f7f1ecp-2, 0x1.e9ec7aaafe278p-1, -136576.0},
    {-0x1.87e1571a31899p-2, 0x1.d90614a25bddep-1, -8960.0}, {-0x1.e2e290b95e1ecp-2, 0x1.c37f3971a9d96p-1, -132288.0},
    {-0x1.1c7f56a4a3e73p-1, 0x1.a9ae9bce714dap-1, -72992.0}, {-0x1.44df38f8d8118p-1, 0x1.8bbadf2f8c607p-1, -108128.0},
    {-0x1.6a178a414b2ddp-1, 0x1.69fc420b08970p-1, -100608.0}, {-0x1.8bd2cec9710b2p-1, 0x1.44c20eaf7b958p-1, -88640.0},
    {-0x1.a9c4771dfe99fp-1, 0x1.1c5e9fe23fad5p-1, -132192.0}, {-0x1.c39c3eba56b70p-1, 0x1.e275f788e9068p-2, -188800.0},
    {-0x1.d910428646fb6p-1, 0x1.87b02d9ad350bp-2, -129792.0}, {-0x1.e9fe6dec8d96ap-1, 0x1.28fc248003c0bp-2, -185952.0},
    {-0x1.f62f79401be70p-1, 0x1.8f13144ad02ccp-3, -160096.0}, {-0x1.fd8bd350a2253p-1, 0x1.9088a78d8d94dp-4, -158368.0},
    {-0x1.0000000000000p+0, 0x0.0p+0, 0.0}, {-0x1.fd8833739b523p-1, -0x1.91af5392a69a9p-4, -34656.0},
    {-0x1.f624a65ce06b0p-1, -0x1.8fecc3a0d3bc9p-3, -129280.0}, {-0x1.e9ec7aaafe278p-1, -0x1.2972817f7f1ecp-2, -136576.0},
    {-0x1.d90614a25bddep-1, -0x1.87e1571a31899p-2, -8960.0}, {-0x1.c37f3971a9d96p-1, -0x1.e2e290b95e1ecp-2, -132288.0},
    {-0x1.a9ae9bce714dap-1, -0x1.1c7f56a4a3e73p-1, -72992.0}, {-0x1.8bbadf2f8c607p-1, -0x1.44df38f8d8118p-1, -108128.0},
    {-0x1.69fc420b08970p-1, -0x1.6a178a414b2ddp-1, -100608.0}, {-0x1.44c20eaf7b958p-1, -0x1.8bd2cec9710b2p-1, -88640.0},
    {-0x1.1c5e9fe23fad5p-1, -0x1.a9c4771dfe99fp-1, -132192.0}, {-0x1.e275f788e9068p-2, -0x1.c39c3eba56b70p-1, -188800.0},
    {-0x1.87b02d9ad350bp-2, -0x1.d910428646fb6p-1, -129792.0}, {-0x1.28fc248003c0bp-2, -0x1.e9fe6dec8d96ap-1, -185952.0},
    {-0x1.8f13144ad02ccp-3, -0x1.f62f79401be70p-1, -160096.0}, {-0x1.9088a78d8d94dp-4, -0x1.fd8bd350a2253p-1, -158368.0},
    {0x0.0p+0, -0x1.0000000000000p+0, 0.0}, {0x1.91af5392a69a9p-4, -0x1.fd8833739b523p-1, -34656.0},
    {0x1.8fecc3a0d3bc9p-3, -0x1.f624a65ce06b0p-1, -129280.0}, {0x1.2972817f7f1ecp-2, -0x1.e9ec7aaafe278p-1, -136576.0},
    {0x1.87e1571a31899p-2, -0x1.d90614a25bddep-1, -8960.0}, {0x1.e2e290b95e1ecp-2, -0x1.c37f3971a9d96p-1, -132288.0},
    {0x1.1c7f56a4a3e73p-1, -0x1.a9ae9bce714dap-1, -72992.0}, {0x1.44df38f8d8118p-1, -0x1.8bbadf2f8c607p-1, -108128.0},
    {0x1.6a178a414b2ddp-1, -0x1.69fc420b08970p-1, -100608.0}, {0x1.8bd2cec9710b2p-1, -0x1.44c20eaf7b958p-1, -88640.0},
    {0x1.a9c4771dfe99fp-1, -0x1.1c5e9fe23fad5p-1, -132192.0}, {0x1.c39c3eba56b70p-1, -0x1.e275f788e9068p-2, -188800.0},
    {0x1.d910428646fb6p-1, -0x1.87b02d9ad350bp-2, -129792.0}, {0x1.e9fe6dec8d96ap-1, -0x1.28fc248003c0bp-2, -185952.0},
    {0x1.f62f79401be70p-1, -0x1.8f13144ad02ccp-3, -160096.0}, {0x1.fd8bd350a2253p-1, -0x1.9088a78d8d94dp-4, -158368.0},
};

// (-2 ln(1 + r) + 2 r) / r^2 for |r| <= 2^-6.9 (relative error of the
// logarithm 2^-56), and sin(w R) / R, (cos(w R) - 1) / R^2 in R^2 for
// |R| <= 2^25 + 2^18, w = 2 pi / 2^32 (absolute errors 2^-64).
constexpr double kLogPoly[6] = {0x1.0000000000009p+0, -0x1.5555555555566p-1, 0x1.fffffff623b03p-2, -0x1.99999990d5c38p-2, 0x1.555b9d209a5a4p-2, -0x1.2497de4b82eb1p-2};
constexpr double kSinPoly[4] = {0x1.921fb54442d18p-30, -0x1.4abbce625bcf7p-91, 0x1.466bc669e8725p-154, -0x1.32cd7b9daf0fep-218};
constexpr double kCosPoly[4] = {-0x1.3bd3cc9be45dep-60, 0x1.03c1f081b5a56p-122, -0x1.55d3c7db592a4p-186, 0x1.e1ee57e355f1ap-251};
// 2 ln 2 as a multiple of 2^-42 and the rest
constexpr double kTwoLn2Hi = 0x1.62e42fefa3800p+0, kTwoLn2Lo = 0x1.ef35793c76730p-44;

struct NormalTables {
    double2 log[64];
    struct alignas(32) {
        double2 cs;
        double shift;
    } trig[64];
};

// The block's copy of the tables (LDS).
__device__ __forceinline__ NormalTables& normal_tables()
{
    __shared__ NormalTables t;
    return t;
}

// Fills the calling block's copy; every thread calls it before the block's
// first fp64 normal.  Ends with a barrier.
__device__ __forceinline__ void load_normal_tables()
{
    NormalTables& t = normal_tables();
    for (int i = threadIdx.x; i < 64; i += blockDim.x) {
        t.log[i] = make_double2(kLogTable[i][0], kLogTable[i][1]);
        t.trig[i].cs = make_double2(kTrigTable[i][0], kTrigTable[i][1]);
        t.trig[i].shift = kTrigTable[i][2];
    }
    __syncthreads();
}

// The uniform of a generator word, ((x >> 8) + 1/2) 2^-24, times 2^32: the
// word with its low byte replaced by 0x80 ((a & b) | c in one instruction).
__device__ __forceinline__ uint32_t u01_32(uint32_t x)
{
    return __builtin_amdgcn_bitop3_b32(x, 0xffffff00u, 0x80u, 0xEA);
}

// -2 ln(n 2^-32) of n = u01_32(x).
__device__ __forceinline__ double neg2_log32(uint32_t n)
{
    const double v = (double)n;
    const uint64_t bits = __builtin_bit_cast(uint64_t, v);
    const uint32_t hi = (uint32_t)(bits >> 32), off = hi - (kLogOff + (7u << 20));
    const int e = (int)off >> 20;                     // v = z 2^(e + 7)
    const double z = __builtin_bit_cast(
        double, ((uint64_t)(hi - (7u << 20) - (off & 0xfff00000u)) << 32) | (uint32_t)bits);
    const double2 t = normal_tables().log[(off >> 14) & 63u];
    const double r = __builtin_fma(z, t.x, -1.0);     // exact
    double q = __builtin_fma(r, kLogPoly[5], kLogPoly[4]);
    q = __builtin_fma(r, q, kLogPoly[3]);
    q = __builtin_fma(r, q, kLogPoly[2]);
    q = __builtin_fma(r, q, kLogPoly[1]);
    q = __builtin_fma(r, q, kLogPoly[0]);
    // 2 (25 - e) ln 2 - 2 ln c: the high part is exact (zero where z is near
    // 1 and e = 25), so the result has one rounding of its own size
    const double k = (double)e;
    const double lo = __builtin_fma(r * r, q, __builtin_fma(k, -kTwoLn2Lo, 25.0 * kTwoLn2Lo));
    return __builtin_fma(k, -kTwoLn2Hi, t.y) + __builtin_fma(-2.0, r, lo);
}

// cos and sin of 2 pi n 2^-32 of n = u01_32(x): nearest of the 64 angles, and
// the residual from the low 26 bits (signed).
__device__ __forceinline__ void cos_sin32(uint32_t n, double& c, double& s)
{
    const auto& t = normal_tables().trig[(n + (1u << 25)) >> 26];
    const double R = (double)((int)(n << 6) >> 6) + t.shift;   // exact
    const double y = R * R;
    const double sr = R * __builtin_fma(y, __builtin_fma(y, __builtin_fma(y, kSinPoly[3], kSinPoly[2]),
                                                         kSinPoly[1]), kSinPoly[0]);
    const double cr = y * __builtin_fma(y, __builtin_fma(y, __builtin_fma(y, kCosPoly[3], kCosPoly[2]),
                                                         kCosPoly[1]), kCosPoly[0]);
    c = t.cs.x + __builtin_fma(t.cs.x, cr, -t.cs.y * sr);
    s = t.cs.y + __builtin_fma(t.cs.y, cr, t.cs.x * sr);
}

// Square root of x in [2^-500, 2^500]: the last step's correction is exact to
// 2^-90, so the result is the rounded root but for ties closer than that.
__device__ __forceinline__ double sqrt_normal(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double r = __builtin_fma(-h, g, 0.5);
    g = __builtin_fma(g, r, g);
    h = __builtin_fma(h, r, h);
    return __builtin_fma(__builtin_fma(-g, g, x), h, g);
}

}  // namespace mlmc
