// normal_math.hpp -- the binary64 functions of the closed-form sweeps' normals:
// Box-Muller from two 32-bit words, and log of the accept uniform.
//
// The sweeps are bound by VALU issue, and the library's log, sqrt and sincospi
// were most of it: 124 binary64 and 70 other instructions a pair of normals
// against 51 and 50 here.  The arguments make the difference: a uniform is a
// 32-bit integer plus 1/2 over 2^32, so nothing is zero, subnormal, infinite or
// NaN, reductions are exact, and accurate tables in LDS (4.5 KB; points moved to
// where the tabulated values lie close to binary64 numbers, S. Gal 1986) take what
// a long polynomial would.  On the GPU against 64-bit-mantissa references over 2^23
// random words, as many near the axes of the circle and the extreme ones, errors in
// units in the last place (largest / root mean square over the random words):
// -2 log 0.570 / 0.289 (the library's 0.641 / 0.292), sine and cosine 0.632 / 0.290
// (0.884 / 0.301), the normals 2.38 / 0.533 (2.65 / 0.539).  The d = 10 Gaussian
// sweep of 2^22 particles and 64 steps: 13.15 -> 9.15 ms when they came in, and later
// 7.67 -> 7.77 ms for the closer sine and cosine below.
//   * log: u = m 2^k, c near 1 / m with at most 29 bits, so that r = m c - 1 is
//     exact, and -2 log u = -2 k log 2 + h + (-2 log(1 + r)) with h = 2 log c
//     (plus 2 log 2 where the octave counts up) stored to 2^-44: each c was
//     searched near 1 / m so that h lies within 2^-57 of such a multiple (2^-60
//     in the upper half octave), which makes the sum with the multiple of 2 log 2 exact.
//     The last entry is c = 1/2, h = 0: near u = 1 the result is the series alone.
//     |r| < 2^-7.9, Taylor series to r^7.
//   * sqrt: the hardware's reciprocal root and two coupled Newton steps, without
//     the scaling that arguments beyond 2^+-767 would need.
//   * sin and cos of 2 pi u: the nearest of 128 points of the circle, each displaced
//     by a few 2^-32 turns to where its sine and cosine both lie within 0.006 units
//     in the last place of binary64 numbers; then the remaining angle x, from an exact
//     integer difference, by Taylor series to x^9 and x^8, joined by the addition
//     theorems.  sin x enters as x and the rest, each multiplied by itself, so that
//     its rounding does not enter; and the points next to an axis stand at the axis
//     (|x| < 0.074 there, 0.025 elsewhere), where the small one of the two would
//     otherwise be a difference of terms as large as itself.  (Rounding sin x and
//     keeping those points had left 1.48 units.)
#pragma once
#include "device_common.hpp"

namespace oasmc {

constexpr int kLogEntries = 128;
constexpr int kCircle = 128;

// {c, h} of the mantissas [1 + i / 128, 1 + (i + 1) / 128)
__device__ const double2 kLogTable[kLogEntries] = {
    {0x1.fded100000000p-1, -0x1.0a02044678000p-7}, {0x1.fa1a790000000p-1, -0x1.7b92600a3c000p-6},
    {0x1.f619f18000000p-1, -0x1.3fdbee99be000p-5}, {0x1.f24fda0000000p-1, -0x1.bbfaebb230000p-5},
    {0x1.ee9dcc8000000p-1, -0x1.1af80d917e000p-4}, {0x1.ead82f0000000p-1, -0x1.59ae2ef140000p-4},
    {0x1.e730820000000p-1, -0x1.96e8ac60d7000p-4}, {0x1.e3a6150000000p-1, -0x1.d2a9b5264f000p-4},
    {0x1.e01c608000000p-1, -0x1.07676c1b9a000p-3}, {0x1.dca70f0000000p-1, -0x1.2503ba77da800p-3},
    {0x1.d91d898000000p-1, -0x1.4386208380000p-3}, {0x1.d5b6430000000p-1, -0x1.61187653cc000p-3},
    {0x1.d269ca0000000p-1, -0x1.7df671caee000p-3}, {0x1.cf1a3c0000000p-1, -0x1.9b242349f8000p-3},
    {0x1.cbe4ea0000000p-1, -0x1.b79dbeb457000p-3}, {0x1.c8bca70000000p-1, -0x1.d3d544a723800p-3},
    {0x1.c575498000000p-1, -0x1.f157d0322b000p-3}, {0x1.c263268000000p-1, -0x1.06967e7507000p-2},
    {0x1.bf43ad8000000p-1, -0x1.14d68422af800p-2}, {0x1.bc3c128000000p-1, -0x1.22c20e5175400p-2},
    {0x1.b9432b0000000p-1, -0x1.3081bf25d9c00p-2}, {0x1.b64bba0000000p-1, -0x1.3e5263e769c00p-2},
    {0x1.b37a088000000p-1, -0x1.4b897f69b1000p-2}, {0x1.b0aad90000000p-1, -0x1.58cab4ec9a000p-2},
    {0x1.adb3360000000p-1, -0x1.66e2c78514000p-2}, {0x1.aae9f20000000p-1, -0x1.74355ad54a400p-2},
    {0x1.a8298f0000000p-1, -0x1.817363ca49400p-2}, {0x1.a589958000000p-1, -0x1.8e29fe19e5000p-2},
    {0x1.a2b8fa8000000p-1, -0x1.9be2ba59f2400p-2}, {0x1.a01f7f8000000p-1, -0x1.a8a3c86c2c000p-2},
    {0x1.9d805d8000000p-1, -0x1.b5954b0a37c00p-2}, {0x1.9adba18000000p-1, -0x1.c2b7cca3f8800p-2},
    {0x1.983ba88000000p-1, -0x1.cfd81f130a000p-2}, {0x1.95c9ab8000000p-1, -0x1.dc25fc873e800p-2},
    {0x1.9350aa0000000p-1, -0x1.e8aa85ffddc00p-2}, {0x1.90ddc30000000p-1, -0x1.f523958fa1c00p-2},
    {0x1.8e6f9c0000000p-1, -0x1.00cbe5bd15000p-1}, {0x1.8be7588000000p-1, -0x1.075348a675a00p-1},
    {0x1.898b6e8000000p-1, -0x1.0d71f8ea9f600p-1}, {0x1.87325d0000000p-1, -0x1.1392a1a1c0200p-1},
    {0x1.84f2e78000000p-1, -0x1.19794d6554800p-1}, {0x1.8297238000000p-1, -0x1.1fb3b27f08400p-1},
    {0x1.806a508000000p-1, -0x1.257ac6f5a2000p-1}, {0x1.7e34908000000p-1, -0x1.2b62299ede600p-1},
    {0x1.7be4988000000p-1, -0x1.3198f9b427800p-1}, {0x1.79c8668000000p-1, -0x1.374d20faa2000p-1},
    {0x1.77a0d28000000p-1, -0x1.3d287d6289600p-1}, {0x1.7571760000000p-1, -0x1.4321d121dc000p-1},
    {0x1.7346ef8000000p-1, -0x1.4916c7c393400p-1}, {0x1.712cc60000000p-1, -0x1.4ee7467130c00p-1},
    {0x1.6f2f2a0000000p-1, -0x1.5470a1686ae00p-1}, {0x1.6d07d80000000p-1, -0x1.5a76ac915ae00p-1},
    {0x1.6b036e8000000p-1, -0x1.60235a8962000p-1}, {0x1.68fd330000000p-1, -0x1.65dd4aade4200p-1},
    {0x1.6724108000000p-1, -0x1.6b1edb7e4f400p-1}, {0x1.6537390000000p-1, -0x1.709fda0fd7a00p-1},
    {0x1.63394e0000000p-1, -0x1.7659ae574ac00p-1}, {0x1.614ec30000000p-1, -0x1.7be3977eb4800p-1},
    {0x1.5f7b548000000p-1, -0x1.8131df7418000p-1}, {0x1.5d8a548000000p-1, -0x1.86ddd6240ca00p-1},
    {0x1.5b971b8000000p-1, -0x1.8c986f56d9200p-1}, {0x1.59e4040000000p-1, -0x1.919d5bafe4e00p-1},
    {0x1.57fdfc8000000p-1, -0x1.974032b8ad400p-1}, {0x1.5624b50000000p-1, -0x1.9cc4dc7ae6600p-1},
    {0x1.546b6a2000000p-1, 0x1.23d76e8f7a000p-1}, {0x1.52b55e3000000p-1, 0x1.1eae711c3ae00p-1},
    {0x1.50e49f1000000p-1, 0x1.192d9e4c1a000p-1}, {0x1.4f3a3cd000000p-1, 0x1.141a64b4e1600p-1},
    {0x1.4d84109000000p-1, 0x1.0edc80e58f600p-1}, {0x1.4bcb68d000000p-1, 0x1.09900c49e3a00p-1},
    {0x1.4a30c32000000p-1, 0x1.04999da26b000p-1}, {0x1.488caac000000p-1, 0x1.feff1a5161c00p-2},
    {0x1.46d6434000000p-1, 0x1.f44b2e262c000p-2}, {0x1.45335e9000000p-1, 0x1.ea03c05ebc400p-2},
    {0x1.4398561000000p-1, 0x1.dfe0cbff75400p-2}, {0x1.42171bf000000p-1, 0x1.d6550c441cc00p-2},
    {0x1.4076da6000000p-1, 0x1.cbf79826bc000p-2}, {0x1.3eed88f000000p-1, 0x1.c21ff5e0a8000p-2},
    {0x1.3d59f3c000000p-1, 0x1.b7f9ebdbe9400p-2}, {0x1.3bd8043000000p-1, 0x1.ae39621391800p-2},
    {0x1.3a49049000000p-1, 0x1.a417c905d2400p-2}, {0x1.38dc1de000000p-1, 0x1.9ac88b6c91000p-2},
    {0x1.3756d79000000p-1, 0x1.90ce1d9bc1000p-2}, {0x1.35ea2e0000000p-1, 0x1.8769d99b83400p-2},
    {0x1.3474d7c000000p-1, 0x1.7dc0ea9f03800p-2}, {0x1.32f1f0a000000p-1, 0x1.73b1c1b6dcc00p-2},
    {0x1.317ab5c000000p-1, 0x1.69e4262e3a800p-2}, {0x1.300e941000000p-1, 0x1.60553b008a000p-2},
    {0x1.2eb7781000000p-1, 0x1.574914c9ae000p-2}, {0x1.2d46b30000000p-1, 0x1.4d84401f3ac00p-2},
    {0x1.2bef9d8000000p-1, 0x1.4462d94a9b000p-2}, {0x1.2a9731c000000p-1, 0x1.3b2dcf607b400p-2},
    {0x1.2938abf000000p-1, 0x1.31c4158e80000p-2}, {0x1.27e7d67000000p-1, 0x1.28adfb4713400p-2},
    {0x1.2681694000000p-1, 0x1.1ef7610d85400p-2}, {0x1.254167e000000p-1, 0x1.164150f6d9000p-2},
    {0x1.23eeb1c000000p-1, 0x1.0cfe83c3e7800p-2}, {0x1.229ecbe000000p-1, 0x1.03c4c54e94000p-2},
    {0x1.214b5cc000000p-1, 0x1.f4ce9d2df8000p-3}, {0x1.200d41f000000p-1, 0x1.e32cffe127800p-3},
    {0x1.1ed6f08000000p-1, 0x1.d1e711aeb7800p-3}, {0x1.1d886bf000000p-1, 0x1.bf335270ef000p-3},
    {0x1.1c543cd000000p-1, 0x1.ade50adee6800p-3}, {0x1.1b1d075000000p-1, 0x1.9c5833edcc000p-3},
    {0x1.19dad7b000000p-1, 0x1.8a18852a5f000p-3}, {0x1.189d1c4000000p-1, 0x1.7804f19fba800p-3},
    {0x1.1777939000000p-1, 0x1.673f93426e000p-3}, {0x1.16427b5000000p-1, 0x1.5583864153000p-3},
    {0x1.1527ef1000000p-1, 0x1.453c21d424000p-3}, {0x1.13ed40d000000p-1, 0x1.33073934f6800p-3},
    {0x1.12cea29000000p-1, 0x1.225fdc0731000p-3}, {0x1.11a1a40000000p-1, 0x1.10cfea0f9f800p-3},
    {0x1.105c776000000p-1, 0x1.fb82112ee1000p-4}, {0x1.0f3ee0c000000p-1, 0x1.d9e295754e000p-4},
    {0x1.0e1d453000000p-1, 0x1.b7a5bbcdc7000p-4}, {0x1.0d0178b000000p-1, 0x1.95f5004424000p-4},
    {0x1.0bed04f000000p-1, 0x1.75014b13b6000p-4}, {0x1.0ad5dea000000p-1, 0x1.5398b3e207000p-4},
    {0x1.09bd3f8000000p-1, 0x1.31dfb71b41000p-4}, {0x1.08a62ec000000p-1, 0x1.10333683a8000p-4},
    {0x1.079eda0000000p-1, 0x1.e098434160000p-5}, {0x1.068c880000000p-1, 0x1.9ddc86bc98000p-5},
    {0x1.0590b5f000000p-1, 0x1.605c813676000p-5}, {0x1.04750f4000000p-1, 0x1.1acf58b0ac000p-5},
    {0x1.036e87c000000p-1, 0x1.b458d163f0000p-6}, {0x1.027b7e5000000p-1, 0x1.3c374d011c000p-6},
    {0x1.0199ea1000000p-1, 0x1.98a33dd370000p-7}, {0x1.0000000000000p-1, -0x0.0p+0},
};

// The circle's points: displacements from i / 128 of a turn in units of 2^-32 turns,
// and {sin, cos} there
__device__ const int32_t kCircleOffset[kCircle] = {
    0, -33554432, 8596, 5965, -249, 17459, 82, 109,
    5076, -1018, -3533, 1803, -9185, -9660, -15705, -5729,
    -2838, 5729, 15705, 9660, 9185, -1803, 3533, 1018,
    -5076, -109, -82, -17459, 249, -5965, -8596, 33554432,
    0, -33554432, 8596, 5965, -249, 17459, 82, 109,
    5076, -1018, -3533, 1803, -9185, -9660, -15705, -5729,
    2838, 5729, 15705, 9660, 9185, -1803, 3533, 1018,
    -5076, -109, -82, -17459, 249, -5965, -8596, 33554432,
    0, -33554432, 8596, 5965, -249, 17459, 82, 109,
    5076, -1018, -3533, 1803, -9185, -9660, -15705, -5729,
    -2838, 5729, 15705, 9660, 9185, -1803, 3533, 1018,
    -5076, -109, -82, -17459, 249, -5965, -8596, 33554432,
    0, -33554432, 8596, 5965, -249, 17459, 82, 109,
    5076, -1018, -3533, 1803, -9185, -9660, -15705, -5729,
    2838, 5729, 15705, 9660, 9185, -1803, 3533, 1018,
    -5076, -109, -82, -17459, 249, -5965, -8596, 33554432,
};
__device__ const double2 kCircleTable[kCircle] = {
    {0x0.0p+0, 0x1.0000000000000p+0}, {0x0.0p+0, 0x1.0000000000000p+0},
    {0x1.91878b250fc49p-4, 0x1.fd88b0e08872fp-1}, {0x1.2c858d751049ap-3, 0x1.fa752cf988fb9p-1},
    {0x1.8f8b53d2fdac6p-3, 0x1.f6297f61e6fe2p-1}, {0x1.f1ac95044bda9p-3, 0x1.f0a71f7979aa5p-1},
    {0x1.29406aa17ebc6p-2, 0x1.e9f4144143b63p-1}, {0x1.58f9b16e069a3p-2, 0x1.e2120e81f54d4p-1},
    {0x1.87dff6d18d7d2p-2, 0x1.d9065d98c07d3p-1}, {0x1.b5d0a64564951p-2, 0x1.ced7c4a151080p-1},
    {0x1.e2b4a19b084f3p-2, 0x1.c38b80d88a442p-1}, {0x1.0738c57bdf2ecp-1, 0x1.b72806d173d43p-1},
    {0x1.1c723cb87d434p-1, 0x1.a9b75d0d5c4a9p-1}, {0x1.30fe02ef4d09fp-1, 0x1.9b3f1ef7263a5p-1},
    {0x1.44ccde61c4e32p-1, 0x1.8bc9efc0284bdp-1}, {0x1.57d5c2e981679p-1, 0x1.7b5eaf01cfce2p-1},
    {0x1.6a0983e618a02p-1, 0x1.6a0a48e9b40bfp-1}, {0x1.7b5eaf01cfce2p-1, 0x1.57d5c2e981679p-1},
    {0x1.8bc9efc0284bdp-1, 0x1.44ccde61c4e32p-1}, {0x1.9b3f1ef7263a5p-1, 0x1.30fe02ef4d09fp-1},
    {0x1.a9b75d0d5c4a9p-1, 0x1.1c723cb87d434p-1}, {0x1.b72806d173d43p-1, 0x1.0738c57bdf2ecp-1},
    {0x1.c38b80d88a442p-1, 0x1.e2b4a19b084f3p-2}, {0x1.ced7c4a151080p-1, 0x1.b5d0a64564951p-2},
    {0x1.d9065d98c07d3p-1, 0x1.87dff6d18d7d2p-2}, {0x1.e2120e81f54d4p-1, 0x1.58f9b16e069a3p-2},
    {0x1.e9f4144143b63p-1, 0x1.29406aa17ebc6p-2}, {0x1.f0a71f7979aa5p-1, 0x1.f1ac95044bda9p-3},
    {0x1.f6297f61e6fe2p-1, 0x1.8f8b53d2fdac6p-3}, {0x1.fa752cf988fb9p-1, 0x1.2c858d751049ap-3},
    {0x1.fd88b0e08872fp-1, 0x1.91878b250fc49p-4}, {0x1.0000000000000p+0, 0x0.0p+0},
    {0x1.0000000000000p+0, 0x0.0p+0}, {0x1.0000000000000p+0, 0x0.0p+0},
    {0x1.fd88b0e08872fp-1, -0x1.91878b250fc49p-4}, {0x1.fa752cf988fb9p-1, -0x1.2c858d751049ap-3},
    {0x1.f6297f61e6fe2p-1, -0x1.8f8b53d2fdac6p-3}, {0x1.f0a71f7979aa5p-1, -0x1.f1ac95044bda9p-3},
    {0x1.e9f4144143b63p-1, -0x1.29406aa17ebc6p-2}, {0x1.e2120e81f54d4p-1, -0x1.58f9b16e069a3p-2},
    {0x1.d9065d98c07d3p-1, -0x1.87dff6d18d7d2p-2}, {0x1.ced7c4a151080p-1, -0x1.b5d0a64564951p-2},
    {0x1.c38b80d88a442p-1, -0x1.e2b4a19b084f3p-2}, {0x1.b72806d173d43p-1, -0x1.0738c57bdf2ecp-1},
    {0x1.a9b75d0d5c4a9p-1, -0x1.1c723cb87d434p-1}, {0x1.9b3f1ef7263a5p-1, -0x1.30fe02ef4d09fp-1},
    {0x1.8bc9efc0284bdp-1, -0x1.44ccde61c4e32p-1}, {0x1.7b5eaf01cfce2p-1, -0x1.57d5c2e981679p-1},
    {0x1.6a0983e618a02p-1, -0x1.6a0a48e9b40bfp-1}, {0x1.57d5c2e981679p-1, -0x1.7b5eaf01cfce2p-1},
    {0x1.44ccde61c4e32p-1, -0x1.8bc9efc0284bdp-1}, {0x1.30fe02ef4d09fp-1, -0x1.9b3f1ef7263a5p-1},
    {0x1.1c723cb87d434p-1, -0x1.a9b75d0d5c4a9p-1}, {0x1.0738c57bdf2ecp-1, -0x1.b72806d173d43p-1},
    {0x1.e2b4a19b084f3p-2, -0x1.c38b80d88a442p-1}, {0x1.b5d0a64564951p-2, -0x1.ced7c4a151080p-1},
    {0x1.87dff6d18d7d2p-2, -0x1.d9065d98c07d3p-1}, {0x1.58f9b16e069a3p-2, -0x1.e2120e81f54d4p-1},
    {0x1.29406aa17ebc6p-2, -0x1.e9f4144143b63p-1}, {0x1.f1ac95044bda9p-3, -0x1.f0a71f7979aa5p-1},
    {0x1.8f8b53d2fdac6p-3, -0x1.f6297f61e6fe2p-1}, {0x1.2c858d751049ap-3, -0x1.fa752cf988fb9p-1},
    {0x1.91878b250fc49p-4, -0x1.fd88b0e08872fp-1}, {0x0.0p+0, -0x1.0000000000000p+0},
    {0x0.0p+0, -0x1.0000000000000p+0}, {0x0.0p+0, -0x1.0000000000000p+0},
    {-0x1.91878b250fc49p-4, -0x1.fd88b0e08872fp-1}, {-0x1.2c858d751049ap-3, -0x1.fa752cf988fb9p-1},
    {-0x1.8f8b53d2fdac6p-3, -0x1.f6297f61e6fe2p-1}, {-0x1.f1ac95044bda9p-3, -0x1.f0a71f7979aa5p-1},
    {-0x1.29406aa17ebc6p-2, -0x1.e9f4144143b63p-1}, {-0x1.58f9b16e069a3p-2, -0x1.e2120e81f54d4p-1},
    {-0x1.87dff6d18d7d2p-2, -0x1.d9065d98c07d3p-1}, {-0x1.b5d0a64564951p-2, -0x1.ced7c4a151080p-1},
    {-0x1.e2b4a19b084f3p-2, -0x1.c38b80d88a442p-1}, {-0x1.0738c57bdf2ecp-1, -0x1.b72806d173d43p-1},
    {-0x1.1c723cb87d434p-1, -0x1.a9b75d0d5c4a9p-1}, {-0x1.30fe02ef4d09fp-1, -0x1.9b3f1ef7263a5p-1},
    {-0x1.44ccde61c4e32p-1, -0x1.8bc9efc0284bdp-1}, {-0x1.57d5c2e981679p-1, -0x1.7b5eaf01cfce2p-1},
    {-0x1.6a0983e618a02p-1, -0x1.6a0a48e9b40bfp-1}, {-0x1.7b5eaf01cfce2p-1, -0x1.57d5c2e981679p-1},
    {-0x1.8bc9efc0284bdp-1, -0x1.44ccde61c4e32p-1}, {-0x1.9b3f1ef7263a5p-1, -0x1.30fe02ef4d09fp-1},
    {-0x1.a9b75d0d5c4a9p-1, -0x1.1c723cb87d434p-1}, {-0x1.b72806d173d43p-1, -0x1.0738c57bdf2ecp-1},
    {-0x1.c38b80d88a442p-1, -0x1.e2b4a19b084f3p-2}, {-0x1.ced7c4a151080p-1, -0x1.b5d0a64564951p-2},
    {-0x1.d9065d98c07d3p-1, -0x1.87dff6d18d7d2p-2}, {-0x1.e2120e81f54d4p-1, -0x1.58f9b16e069a3p-2},
    {-0x1.e9f4144143b63p-1, -0x1.29406aa17ebc6p-2}, {-0x1.f0a71f7979aa5p-1, -0x1.f1ac95044bda9p-3},
    {-0x1.f6297f61e6fe2p-1, -0x1.8f8b53d2fdac6p-3}, {-0x1.fa752cf988fb9p-1, -0x1.2c858d751049ap-3},
    {-0x1.fd88b0e08872fp-1, -0x1.91878b250fc49p-4}, {-0x1.0000000000000p+0, 0x0.0p+0},
    {-0x1.0000000000000p+0, 0x0.0p+0}, {-0x1.0000000000000p+0, 0x0.0p+0},
    {-0x1.fd88b0e08872fp-1, 0x1.91878b250fc49p-4}, {-0x1.fa752cf988fb9p-1, 0x1.2c858d751049ap-3},
    {-0x1.f6297f61e6fe2p-1, 0x1.8f8b53d2fdac6p-3}, {-0x1.f0a71f7979aa5p-1, 0x1.f1ac95044bda9p-3},
    {-0x1.e9f4144143b63p-1, 0x1.29406aa17ebc6p-2}, {-0x1.e2120e81f54d4p-1, 0x1.58f9b16e069a3p-2},
    {-0x1.d9065d98c07d3p-1, 0x1.87dff6d18d7d2p-2}, {-0x1.ced7c4a151080p-1, 0x1.b5d0a64564951p-2},
    {-0x1.c38b80d88a442p-1, 0x1.e2b4a19b084f3p-2}, {-0x1.b72806d173d43p-1, 0x1.0738c57bdf2ecp-1},
    {-0x1.a9b75d0d5c4a9p-1, 0x1.1c723cb87d434p-1}, {-0x1.9b3f1ef7263a5p-1, 0x1.30fe02ef4d09fp-1},
    {-0x1.8bc9efc0284bdp-1, 0x1.44ccde61c4e32p-1}, {-0x1.7b5eaf01cfce2p-1, 0x1.57d5c2e981679p-1},
    {-0x1.6a0983e618a02p-1, 0x1.6a0a48e9b40bfp-1}, {-0x1.57d5c2e981679p-1, 0x1.7b5eaf01cfce2p-1},
    {-0x1.44ccde61c4e32p-1, 0x1.8bc9efc0284bdp-1}, {-0x1.30fe02ef4d09fp-1, 0x1.9b3f1ef7263a5p-1},
    {-0x1.1c723cb87d434p-1, 0x1.a9b75d0d5c4a9p-1}, {-0x1.0738c57bdf2ecp-1, 0x1.b72806d173d43p-1},
    {-0x1.e2b4a19b084f3p-2, 0x1.c38b80d88a442p-1}, {-0x1.b5d0a64564951p-2, 0x1.ced7c4a151080p-1},
    {-0x1.87dff6d18d7d2p-2, 0x1.d9065d98c07d3p-1}, {-0x1.58f9b16e069a3p-2, 0x1.e2120e81f54d4p-1},
    {-0x1.29406aa17ebc6p-2, 0x1.e9f4144143b63p-1}, {-0x1.f1ac95044bda9p-3, 0x1.f0a71f7979aa5p-1},
    {-0x1.8f8b53d2fdac6p-3, 0x1.f6297f61e6fe2p-1}, {-0x1.2c858d751049ap-3, 0x1.fa752cf988fb9p-1},
    {-0x1.91878b250fc49p-4, 0x1.fd88b0e08872fp-1}, {0x0.0p+0, 0x1.0000000000000p+0},
};

// The tables in LDS.
struct NormalTables {
    double2 log[kLogEntries];
    double2 circle[kCircle];
    int32_t offset[kCircle];
};

// Copied by the whole workgroup; the caller's next barrier publishes them.
__device__ __forceinline__ void stage_tables(NormalTables& t)
{
    for (int i = threadIdx.x; i < kLogEntries; i += blockDim.x) t.log[i] = kLogTable[i];
    for (int i = threadIdx.x; i < kCircle; i += blockDim.x) {
        t.circle[i] = kCircleTable[i];
        t.offset[i] = kCircleOffset[i];
    }
}

// -2 log((w + 1/2) 2^-32), positive.
__device__ __forceinline__ double minus2_log_word(const NormalTables& tb, uint32_t w)
{
    const double v = (double)w + 0.5;  // in [1/2, 2^32)
    const uint32_t hi = (uint32_t)__double2hiint(v);
    const double2 t = tb.log[(hi >> 13) & (kLogEntries - 1)];
    const double m = __hiloint2double((int)((hi & 0x000FFFFFu) | 0x3FF00000u), __double2loint(v));
    // octaves below u = 1; the upper half of an octave counts to the next
    const double k = (double)((1023 + 32) - (int)((hi + 0x00080000u) >> 20));
    const double r = fma(m, t.x, -1.0);
    const double r2 = r * r;
    double p = fma(r, -2.0 / 7.0, 1.0 / 3.0);
    p = fma(p, r, -2.0 / 5.0);
    p = fma(p, r, 1.0 / 2.0);
    p = fma(p, r, -2.0 / 3.0);
    p = fma(p, r, 1.0);
    const double q = fma(r2, p, k * -0x1.0ca86c3898d00p-48);  // 2 log 2 = high + low
    // T - 2 r with its rounding (|T| > |2 r| or T = 0, so the difference is exact)
    const double T = fma(k, 0x1.62e42fefa3a00p+0, t.y);
    const double a = fma(-2.0, r, T);
    return a + (fma(-2.0, r, T - a) + q);
}

// sqrt of x in [2^-40, 2^6].
__device__ __forceinline__ double sqrt_plain(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double e = fma(-h, g, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
    return fma(fma(-g, g, x), h, g);
}

// sin and cos of 2 pi (w + 1/2) 2^-32.
__device__ __forceinline__ void circle_word(const NormalTables& tb, uint32_t w, double& s, double& c)
{
    const uint32_t i = (w + (1u << 24)) >> 25;  // nearest point (128 is point 0)
    const double2 t = tb.circle[i & (kCircle - 1)];
    const double d = (double)((int32_t)(w - (i << 25)) - tb.offset[i & (kCircle - 1)]) + 0.5;
    const double x = d * 0x1.921fb54442d18p-30;  // 2 pi 2^-32
    const double z = x * x;
    double sp = fma(z, 1.0 / 362880.0, -1.0 / 5040.0);
    double cp = fma(z, 1.0 / 40320.0, -1.0 / 720.0);
    sp = fma(sp, z, 1.0 / 120.0);
    cp = fma(cp, z, 1.0 / 24.0);
    sp = fma(sp, z, -1.0 / 6.0);
    cp = fma(cp, z, -1.0 / 2.0);
    // sin x = x + sl (with the low parts of the product and of 2 pi), cos x - 1 = cm
    const double lo = fma(d, 0x1.1a62633145c07p-84, fma(d, 0x1.921fb54442d18p-30, -x));
    const double sl = fma(x * z, sp, lo);
    const double cm = z * cp;
    s = t.x + fma(t.y, x, fma(t.y, sl, t.x * cm));
    c = t.y + fma(-t.x, x, fma(-t.x, sl, t.y * cm));
}

// Box-Muller: (wa, wb) -> (r cos 2 pi u_b, r sin 2 pi u_b), r = sqrt(-2 log u_a).
__device__ __forceinline__ void box_muller(const NormalTables& tb, uint32_t wa, uint32_t wb, double& zc,
                                           double& zs)
{
    const double r = sqrt_plain(minus2_log_word(tb, wa));
    double s, c;
    circle_word(tb, wb, s, c);
    zc = r * c;
    zs = r * s;
}

}  // namespace oasmc
