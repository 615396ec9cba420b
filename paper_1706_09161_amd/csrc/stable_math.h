// stable_math.h -- FP64 evaluation of Weron's stable variable (random_walk.hip)
// from logarithms kept in two doubles: one exponential instead of two powers.
//
// Both powers of the formula
//   S = Sc sin(a (V + B)) cos(V)^(-1/a) (cos(V - a (V + B)) / W)^((1 - a)/a),  W = -log u2,
// are formed as exp(L), L = -(1/a) log cos V + ((1 - a)/a) (log cos(V - a (V + B)) - log W),
// with logarithms of about 2^-60 absolute error, so L (up to 75 in size) costs
// the exponential no more than a rounding.  The arguments V, a (V + B) and
// V - a (V + B) lie in [-pi, pi]: sine and cosine need one fold and one
// polynomial, no reduction by multiples of pi/2.  Methods: table-driven
// logarithm (P. T. P. Tang, ACM TOMS 16, 1990; its reduction, x 2^-k from 0.6875
// indexed by 7 bits of the high word with c = 1 next to 1 and log 2 cut at a
// multiple of 2^-42, makes the choices of the open log of Arm's optimized
// routines, which glibc has too; the table, with c of 24 bits, and what follows
// it are this file's), Taylor polynomials of sine and exponential on [0, pi/2]
// and [-log 2 / 2, log 2 / 2] (truncation below 2^-58), error-free sums and
// products (Dekker 1971, Knuth).
//
// Relative error of S against 128-bit arithmetic on the same rounded arguments,
// 4e6 draws over a in (1, 2], beta in [-1, 1] and the ends of the uniforms, rms
// / largest (units of 2^-53): 0.94 / 4.5; with glibc's log, sin, cos and pow
// 1.06 / 5.6.
#pragma once
#include <math.h>
#include <stdint.h>

namespace lbm {
namespace stable_math {

// Entry j of the table of -log c: c is 1 / m to 24 bits for mantissas m in the
// j-th of 128 equal steps of the high word from 0.6875 to 1.375 (c = 1 in the
// two next to m = 1, where the logarithm is small), hi a multiple of 2^-42.
struct alignas(16) LogEntry {
    double hi;
    float c, lo;
};
#define LBM_LOG_TABLE \
    {-0x1.7cc7f6f347000p-2, 0x1.734f0c0000000p+0f, 0x1.7d01640000000p-44f}, {-0x1.76feea5d47000p-2, 0x1.7137860000000p+0f, -0x1.69997c0000000p-46f}, \
    {-0x1.713e35386a000p-2, 0x1.6f26020000000p+0f, -0x1.76a0060000000p-46f}, {-0x1.6b85b3abfa000p-2, 0x1.6d1a620000000p+0f, -0x1.fd1a400000000p-45f}, \
    {-0x1.65d556f4ce000p-2, 0x1.6b14900000000p+0f, -0x1.cd3f4a0000000p-53f}, {-0x1.602d09a709000p-2, 0x1.6914740000000p+0f, -0x1.ea08980000000p-46f}, \
    {-0x1.5a8caf83ee000p-2, 0x1.6719f40000000p+0f, 0x1.95dbb00000000p-48f}, {-0x1.54f430c7be000p-2, 0x1.6524f80000000p+0f, -0x1.a6d34c0000000p-46f}, \
    {-0x1.4f638013aa000p-2, 0x1.63356c0000000p+0f, 0x1.fcfcac0000000p-44f}, {-0x1.49da7dbfcc000p-2, 0x1.614b360000000p+0f, -0x1.06992c0000000p-44f}, \
    {-0x1.4459202d3a000p-2, 0x1.5f66440000000p+0f, 0x1.812e8a0000000p-47f}, {-0x1.3edf458417000p-2, 0x1.5d867c0000000p+0f, 0x1.f0a9e20000000p-44f}, \
    {-0x1.396ce231bc000p-2, 0x1.5babcc0000000p+0f, 0x1.5d92c60000000p-47f}, {-0x1.3401e3eaed000p-2, 0x1.59d6200000000p+0f, 0x1.1b8f360000000p-44f}, \
    {-0x1.2e9e2b8e12000p-2, 0x1.5805600000000p+0f, -0x1.42f0c20000000p-45f}, {-0x1.2941b0b987000p-2, 0x1.56397c0000000p+0f, 0x1.21944c0000000p-44f}, \
    {-0x1.23ec584dec000p-2, 0x1.54725e0000000p+0f, 0x1.6e8b4c0000000p-44f}, {-0x1.1e9e183c8a000p-2, 0x1.52aff60000000p+0f, 0x1.8479f60000000p-44f}, \
    {-0x1.1956d385bc000p-2, 0x1.50f22e0000000p+0f, -0x1.7d24e40000000p-45f}, {-0x1.14167e6767000p-2, 0x1.4f38f60000000p+0f, -0x1.e09a300000000p-44f}, \
    {-0x1.0edd064378000p-2, 0x1.4d843c0000000p+0f, -0x1.016a520000000p-47f}, {-0x1.09aa57a26c000p-2, 0x1.4bd3ee0000000p+0f, -0x1.b4efd60000000p-44f}, \
    {-0x1.047e5e31e8000p-2, 0x1.4a27fa0000000p+0f, -0x1.d510000000000p-45f}, {-0x1.feb22276a0000p-3, 0x1.4880520000000p+0f, -0x1.f31a7e0000000p-45f}, \
    {-0x1.f474b5c4e0000p-3, 0x1.46dce40000000p+0f, 0x1.bd7ec00000000p-44f}, {-0x1.ea4448d84a000p-3, 0x1.453d9e0000000p+0f, -0x1.5e6b1e0000000p-44f}, \
    {-0x1.e020d27236000p-3, 0x1.43a2740000000p+0f, 0x1.5be04a0000000p-45f}, {-0x1.d60a157104000p-3, 0x1.420b520000000p+0f, 0x1.5e3b0e0000000p-44f}, \
    {-0x1.cc001295b4000p-3, 0x1.40782e0000000p+0f, 0x1.e8a5a60000000p-46f}, {-0x1.c20289a180000p-3, 0x1.3ee8f40000000p+0f, 0x1.93292e0000000p-45f}, \
    {-0x1.b81178d382000p-3, 0x1.3d5d9a0000000p+0f, -0x1.d850640000000p-46f}, {-0x1.ae2ca9be72000p-3, 0x1.3bd60e0000000p+0f, -0x1.7995d20000000p-44f}, \
    {-0x1.a4540b3e6a000p-3, 0x1.3a52440000000p+0f, -0x1.5f7b5c0000000p-44f}, {-0x1.9a877e06ba000p-3, 0x1.38d22e0000000p+0f, -0x1.43bcdc0000000p-44f}, \
    {-0x1.90c6e177cc000p-3, 0x1.3755be0000000p+0f, 0x1.a472780000000p-46f}, {-0x1.8712139d0e000p-3, 0x1.35dce60000000p+0f, -0x1.328dec0000000p-44f}, \
    {-0x1.7d68fe72f6000p-3, 0x1.34679a0000000p+0f, 0x1.532a420000000p-45f}, {-0x1.73cb8adcfe000p-3, 0x1.32f5ce0000000p+0f, 0x1.da53d80000000p-44f}, \
    {-0x1.6a39a0a3be000p-3, 0x1.3187760000000p+0f, 0x1.90ad560000000p-44f}, {-0x1.60b30b830a000p-3, 0x1.301c820000000p+0f, 0x1.73d6740000000p-44f}, \
    {-0x1.5737cbb818000p-3, 0x1.2eb4ea0000000p+0f, -0x1.9b93b20000000p-44f}, {-0x1.4dc7b817bc000p-3, 0x1.2d50a00000000p+0f, -0x1.c75b600000000p-47f}, \
    {-0x1.4462b3bc9c000p-3, 0x1.2bef980000000p+0f, 0x1.89360a0000000p-44f}, {-0x1.3b08bc0d80000p-3, 0x1.2a91ca0000000p+0f, 0x1.aec7d80000000p-44f}, \
    {-0x1.31b996aba4000p-3, 0x1.2937260000000p+0f, -0x1.f02c260000000p-44f}, {-0x1.28753ef11a000p-3, 0x1.27dfa40000000p+0f, -0x1.734fc40000000p-44f}, \
    {-0x1.1f3b93bf26000p-3, 0x1.268b380000000p+0f, 0x1.6066ea0000000p-46f}, {-0x1.160c80c4b2000p-3, 0x1.2539d80000000p+0f, -0x1.ec142a0000000p-45f}, \
    {-0x1.0ce7f0c4cc000p-3, 0x1.23eb7a0000000p+0f, -0x1.3eb1ba0000000p-46f}, {-0x1.03cdbf7d1e000p-3, 0x1.22a0120000000p+0f, -0x1.817f080000000p-44f}, \
    {-0x1.f57bc79900000p-4, 0x1.2157980000000p+0f, -0x1.76a4ca0000000p-46f}, {-0x1.e3708b5304000p-4, 0x1.2012020000000p+0f, -0x1.05bd3e0000000p-45f}, \
    {-0x1.d1797ba218000p-4, 0x1.1ecf440000000p+0f, -0x1.35f51c0000000p-44f}, {-0x1.bf9680f9fc000p-4, 0x1.1d8f560000000p+0f, -0x1.3f81b80000000p-45f}, \
    {-0x1.adc78265b0000p-4, 0x1.1c52300000000p+0f, 0x1.579d200000000p-44f}, {-0x1.9c0c2ba4d4000p-4, 0x1.1b17c60000000p+0f, 0x1.ad19520000000p-44f}, \
    {-0x1.8a647d391c000p-4, 0x1.19e0120000000p+0f, -0x1.c194820000000p-44f}, {-0x1.78d01f23d8000p-4, 0x1.18ab080000000p+0f, -0x1.67117a0000000p-47f}, \
    {-0x1.674f0ee364000p-4, 0x1.1778a20000000p+0f, -0x1.a65acc0000000p-44f}, {-0x1.55e10e20e0000p-4, 0x1.1648d60000000p+0f, -0x1.9225000000000p-47f}, \
    {-0x1.4485dc8dbc000p-4, 0x1.151b9a0000000p+0f, -0x1.fa67a60000000p-44f}, {-0x1.333d734184000p-4, 0x1.13f0e80000000p+0f, 0x1.ff3b6a0000000p-49f}, \
    {-0x1.2207ac8784000p-4, 0x1.12c8b80000000p+0f, -0x1.472c500000000p-44f}, {-0x1.10e4612cb0000p-4, 0x1.11a3020000000p+0f, 0x1.7e109a0000000p-44f}, \
    {-0x1.ffa694dab8000p-5, 0x1.107fbc0000000p+0f, -0x1.2fd08a0000000p-45f}, {-0x1.dda8b7c680000p-5, 0x1.0f5ee00000000p+0f, 0x1.1caac60000000p-45f}, \
    {-0x1.bbced3a690000p-5, 0x1.0e40660000000p+0f, 0x1.8850880000000p-46f}, {-0x1.9a188df740000p-5, 0x1.0d24460000000p+0f, 0x1.0ed8ac0000000p-44f}, \
    {-0x1.7885892358000p-5, 0x1.0c0a780000000p+0f, 0x1.0d92d00000000p-46f}, {-0x1.5715df4040000p-5, 0x1.0af2f80000000p+0f, 0x1.8e055e0000000p-44f}, \
    {-0x1.35c8b2ca10000p-5, 0x1.09ddba0000000p+0f, -0x1.820c4e0000000p-44f}, {-0x1.149e568008000p-5, 0x1.08cabc0000000p+0f, 0x1.3030ca0000000p-44f}, \
    {-0x1.e72bccc140000p-6, 0x1.07b9f20000000p+0f, 0x1.9306240000000p-45f}, {-0x1.a55f624c60000p-6, 0x1.06ab5a0000000p+0f, 0x1.dec41a0000000p-45f}, \
    {-0x1.63d615c690000p-6, 0x1.059eea0000000p+0f, -0x1.7ab2f80000000p-47f}, {-0x1.228f827ea0000p-6, 0x1.04949c0000000p+0f, -0x1.686df20000000p-45f}, \
    {-0x1.c3177b4c80000p-7, 0x1.038c6c0000000p+0f, 0x1.4424600000000p-44f}, {-0x1.4192bb9680000p-7, 0x1.0286500000000p+0f, -0x1.95f4760000000p-46f}, \
    {-0x1.8121bb4580000p-8, 0x1.0182440000000p+0f, -0x1.a1bbb80000000p-46f}, {0x0.0p+0, 0x1.0000000000000p+0f, 0x0.0p+0f}, \
    {0x0.0p+0, 0x1.0000000000000p+0f, 0x0.0p+0f}, {0x1.7dc49e7820000p-7, 0x1.fa11ca0000000p-1f, -0x1.ea453e0000000p-44f}, \
    {0x1.3cea5df470000p-6, 0x1.f6310a0000000p-1f, -0x1.68e0bc0000000p-44f}, {0x1.b9fc0afb00000p-6, 0x1.f25f640000000p-1f, -0x1.b97bf00000000p-44f}, \
    {0x1.1b0d909240000p-5, 0x1.ee9c800000000p-1f, -0x1.3381ea0000000p-44f}, {0x1.58a5b57c90000p-5, 0x1.eae8080000000p-1f, -0x1.b23e3a0000000p-45f}, \
    {0x1.95c836cc90000p-5, 0x1.e741aa0000000p-1f, -0x1.c0be1a0000000p-45f}, {0x1.d276b22db0000p-5, 0x1.e3a9180000000p-1f, 0x1.6b943c0000000p-46f}, \
    {0x1.0759824990000p-4, 0x1.e01e020000000p-1f, -0x1.b8e3f60000000p-44f}, {0x1.253f6120a0000p-4, 0x1.dca01e0000000p-1f, 0x1.4189d80000000p-44f}, \
    {0x1.42edcd9a64000p-4, 0x1.d92f220000000p-1f, 0x1.bc6a0e0000000p-46f}, {0x1.60658ad374000p-4, 0x1.d5cac80000000p-1f, 0x1.0c3b9e0000000p-44f}, \
    {0x1.7da76907b0000p-4, 0x1.d272ca0000000p-1f, 0x1.2cee8c0000000p-44f}, {0x1.9ab4225204000p-4, 0x1.cf26e60000000p-1f, -0x1.8a20720000000p-45f}, \
    {0x1.b78c7d2b10000p-4, 0x1.cbe6da0000000p-1f, -0x1.24f7f40000000p-44f}, {0x1.d4313a96cc000p-4, 0x1.c8b2660000000p-1f, -0x1.93d5a80000000p-45f}, \
    {0x1.f0a3039118000p-4, 0x1.c5894e0000000p-1f, -0x1.d360600000000p-44f}, {0x1.06714f3ca6000p-3, 0x1.c26b540000000p-1f, -0x1.a3853a0000000p-45f}, \
    {0x1.14785c6e74000p-3, 0x1.bf583e0000000p-1f, 0x1.5ed7720000000p-46f}, {0x1.2266f328a6000p-3, 0x1.bc4fd60000000p-1f, -0x1.4c7e1c0000000p-45f}, \
    {0x1.303d74c648000p-3, 0x1.b951e20000000p-1f, -0x1.15295c0000000p-50f}, {0x1.3dfc2c26cc000p-3, 0x1.b65e2e0000000p-1f, 0x1.8abf360000000p-45f}, \
    {0x1.4ba37269a6000p-3, 0x1.b374840000000p-1f, -0x1.420f9c0000000p-44f}, {0x1.5933896982000p-3, 0x1.b094b40000000p-1f, 0x1.2eb88c0000000p-48f}, \
    {0x1.66acd4072a000p-3, 0x1.adbe880000000p-1f, 0x1.aa1c5c0000000p-44f}, {0x1.740f93fc04000p-3, 0x1.aaf1d20000000p-1f, -0x1.08b1020000000p-44f}, \
    {0x1.815c059c36000p-3, 0x1.a82e660000000p-1f, -0x1.0026280000000p-44f}, {0x1.8e92902886000p-3, 0x1.a574100000000p-1f, 0x1.a8b74c0000000p-44f}, \
    {0x1.9bb36547e0000p-3, 0x1.a2c2a80000000p-1f, -0x1.1dc18a0000000p-45f}, {0x1.a8becdf082000p-3, 0x1.a01a020000000p-1f, 0x1.e385240000000p-44f}, \
    {0x1.b5b51740fc000p-3, 0x1.9d79f20000000p-1f, -0x1.4a90660000000p-44f}, {0x1.c2968890c2000p-3, 0x1.9ae24e0000000p-1f, -0x1.cd402e0000000p-45f}, \
    {0x1.cf6359209c000p-3, 0x1.9852f00000000p-1f, 0x1.7b963a0000000p-45f}, {0x1.dc1bcdcabe000p-3, 0x1.95cbb00000000p-1f, 0x1.916e1a0000000p-44f}, \
    {0x1.e8c0250aa6000p-3, 0x1.934c680000000p-1f, -0x1.6804b80000000p-45f}, {0x1.f550a0ecb8000p-3, 0x1.90d4f20000000p-1f, -0x1.2d402a0000000p-45f}, \
    {0x1.00e6c38ad5000p-2, 0x1.8e65280000000p-1f, 0x1.e188d60000000p-50f}, {0x1.071b860cd6000p-2, 0x1.8bfce80000000p-1f, -0x1.bcb83a0000000p-44f}, \
    {0x1.0d46b3d9ab000p-2, 0x1.899c100000000p-1f, 0x1.d41a200000000p-44f}, {0x1.13686fa13b000p-2, 0x1.87427c0000000p-1f, -0x1.d3c42a0000000p-44f}, \
    {0x1.1980d34542000p-2, 0x1.84f00c0000000p-1f, 0x1.b7dde80000000p-45f}, {0x1.1f8ffa248a000p-2, 0x1.82a4a00000000p-1f, 0x1.7956c00000000p-45f}, \
    {0x1.2596011df7000p-2, 0x1.8060180000000p-1f, 0x1.8e7c420000000p-44f}, {0x1.2b9301378a000p-2, 0x1.7e22560000000p-1f, -0x1.67ac9e0000000p-45f}, \
    {0x1.31871a4144000p-2, 0x1.7beb3a0000000p-1f, 0x1.8fd1da0000000p-46f}, {0x1.37726827fe000p-2, 0x1.79baa60000000p-1f, -0x1.e74b620000000p-44f}, \
    {0x1.3d54f7e81f000p-2, 0x1.7790820000000p-1f, 0x1.c6e4160000000p-44f}, {0x1.432ef2f84f000p-2, 0x1.756cac0000000p-1f, -0x1.fb037a0000000p-44f},

constexpr int kLogEntries = 128;
constexpr double kLn2Hi = 0x1.62e42fefa3800p-1, kLn2Lo = 0x1.ef35793c76730p-45;  // log 2, hi a multiple of 2^-42
constexpr double kPiHi = 0x1.921fb54442d18p+1, kPiLo = 0x1.1a62633145c07p-53;

// log x = h + l for a positive normal x
__host__ __device__ inline void log2d(const LogEntry* table, double x, double& h, double& l)
{
#pragma clang fp contract(off)
    const uint64_t bits = __builtin_bit_cast(uint64_t, x);
    const uint32_t top = (uint32_t)(bits >> 32) - 0x3FE60000u;
    const int32_t k = (int32_t)top >> 20;
    const double m = __builtin_bit_cast(double, bits - ((uint64_t)(uint32_t)(k << 20) << 32));  // x 2^-k, in [0.6875, 1.375)
    const LogEntry e = table[(top >> 13) & (kLogEntries - 1)];
    const double z = fma(m, (double)e.c, -1.0);  // |z| < 2^-7
    const double kd = (double)k, t = fma(kd, kLn2Hi, e.hi);  // exact
    h = t + z;  // |t| > |z| or t = 0
    const double tail = (t - h) + z;
    double p = -1.0 / 8;
    p = fma(p, z, 1.0 / 7);
    p = fma(p, z, -1.0 / 6);
    p = fma(p, z, 1.0 / 5);
    p = fma(p, z, -1.0 / 4);
    p = fma(p, z, 1.0 / 3);
    p = fma(p, z, -1.0 / 2);
    l = fma(z * z, p, tail + fma(kd, kLn2Lo, (double)e.lo));
}

// sin(y + e), y in [0, pi/2], |e| a rounding of y
__host__ __device__ inline double sin_fold(double y, double e)
{
#pragma clang fp contract(off)
    const double s = y * y;
    double p = 1.0 / 51090942171709440000.0;  // 1 / 21!
    p = fma(p, s, -1.0 / 121645100408832000.0);
    p = fma(p, s, 1.0 / 355687428096000.0);
    p = fma(p, s, -1.0 / 1307674368000.0);
    p = fma(p, s, 1.0 / 6227020800.0);
    p = fma(p, s, -1.0 / 39916800.0);
    p = fma(p, s, 1.0 / 362880.0);
    p = fma(p, s, -1.0 / 5040.0);
    p = fma(p, s, 1.0 / 120.0);
    p = fma(p, s, -1.0 / 6.0);
    const double c = fma(s, fma(s, 1.0 / 24, -0.5), 1.0);  // cos y to 2 %
    return y + fma(y * s, p, e * c);
}

// cos x, |x| <= pi/2 (and a rounding more: negative there)
__host__ __device__ inline double cos_half(double x)
{
#pragma clang fp contract(off)
    const double a = fabs(x), y = 0.5 * kPiHi - a;
    return sin_fold(y, ((0.5 * kPiHi - y) - a) + 0.5 * kPiLo);
}

// sin x, |x| <= pi (and a few roundings more)
__host__ __device__ inline double sin_full(double x)
{
#pragma clang fp contract(off)
    const double a = fabs(x);
    const bool far = a > 0.5 * kPiHi;
    const double y = far ? kPiHi - a : a;  // exact: a >= pi / 2
    return copysign(1.0, x) * sin_fold(y, far ? kPiLo : 0.0);
}

// exp(h + l), |l| a rounding of h
__host__ __device__ inline double exp2d(double h, double l)
{
#pragma clang fp contract(off)
    const double n = rint(h * 1.4426950408889634);
    const double r0 = fma(-n, kLn2Hi, h);  // exact
    const double low = fma(-n, kLn2Lo, l), r = r0 + low, rl = (r0 - r) + low;
    double q = 1.0 / 6227020800.0;  // 1 / 13!
    q = fma(q, r, 1.0 / 479001600.0);
    q = fma(q, r, 1.0 / 39916800.0);
    q = fma(q, r, 1.0 / 3628800.0);
    q = fma(q, r, 1.0 / 362880.0);
    q = fma(q, r, 1.0 / 40320.0);
    q = fma(q, r, 1.0 / 5040.0);
    q = fma(q, r, 1.0 / 720.0);
    q = fma(q, r, 1.0 / 120.0);
    q = fma(q, r, 1.0 / 24.0);
    q = fma(q, r, 1.0 / 6.0);
    q = fma(q, r, 0.5);
    return ldexp(1.0 + (r + fma(r * r, q, rl)), (int)n);
}

// S from the uniforms u1, u2; a, B, Sc as in the formula, ia = 1 / a, ex = (1 - a) / a
__host__ __device__ inline double stable(const LogEntry* table, double a, double ia, double ex, double B, double Sc,
                                         double u1, double u2)
{
#pragma clang fp contract(off)
    const double V = 3.14159265358979323846 * (u1 - 0.5);
    double wh, wl;
    log2d(table, u2, wh, wl);
    const double W = -(wh + wl);
    const double arg = a * (V + B);
    const double c1 = cos_half(V), c2 = cos_half(V - arg);
    double h1, l1, h2, l2, h3, l3;
    log2d(table, c1, h1, l1);
    log2d(table, c2, h2, l2);
    log2d(table, W, h3, l3);
    const double d = h2 - h3, db = h2 - d;
    const double dl = ((h2 - (d + db)) + (db - h3)) + (l2 - l3);  // h2 + l2 - h3 - l3 = d + dl
    const double p = -ia * h1, pl = fma(-ia, h1, -p) - ia * l1;
    const double q = ex * d, ql = fma(ex, d, -q) + ex * dl;
    const double L = p + q, Lb = L - p;
    const double Ll = ((p - (L - Lb)) + (q - Lb)) + (pl + ql);
    double P = exp2d(L, Ll);
    // the ends of the range, as the powers have them (the exponent is in
    // [-1/2, 0)): u2 that rounds to 1, W = 0, gives 0, and an argument past
    // pi/2, where the cosine is negative, no number
    if (!(c2 > 0.0)) P = __builtin_nan("");
    if (!(W > 0.0)) P = 0.0;
    return Sc * sin_full(arg) * P;
}

}  // namespace stable_math
}  // namespace lbm
