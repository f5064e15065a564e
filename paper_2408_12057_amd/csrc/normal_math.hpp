// normal_math.hpp -- the binary64 functions of the closed-form sweeps' normals:
// Box-Muller from two 32-bit words, and log of the accept uniform.
//
// The sweeps are bound by VALU issue, and the library's log, sqrt and sincospi
// were most of it: 124 binary64 and 70 other instructions a pair of normals
// against 48 and 50 here.  The arguments make the difference: a uniform is a
// 32-bit integer plus 1/2 over 2^32, so nothing is zero, subnormal, infinite or
// NaN, reductions are exact, and a table in LDS (4 KB) takes what a long
// polynomial would.  Against 64-bit-mantissa references over 2^24 random words
// and the extreme ones, errors in units in the last place (largest / root mean
// square): log 0.57 / 0.288 (the library's 0.64 / 0.291), sine and cosine
// 1.49 / 0.296 (0.88 / 0.302), the normals 2.97 / 0.537 (2.54 / 0.540).  The d = 10
// Gaussian sweep of 2^22 particles and 64 steps: 13.15 -> 9.15 ms.
//   * log: u = m 2^k, c near 1 / m with at most 29 bits, so that r = m c - 1 is
//     exact, and -2 log u = -2 k log 2 + h + (-2 log(1 + r)) with h = 2 log c
//     (plus 2 log 2 where the octave counts up) stored to 2^-44: each c was
//     searched near 1 / m so that h lies within 2^-58 of such a multiple (2^-61
//     in the upper half octave), which makes the sum with the multiple of 2 log 2 exact.
//     The last entry is c = 1/2, h = 0: near u = 1 the result is the series alone.
//     |r| < 2^-7.9, Taylor series to r^7.
//   * sqrt: the hardware's reciprocal root and two coupled Newton steps, without
//     the scaling that arguments beyond 2^+-767 would need.
//   * sin and cos of 2 pi u: the nearest of 128 points of the circle, each displaced
//     by a few 2^-32 turns to where its sine and cosine both lie within 0.006 units
//     in the last place of binary64 numbers; then the remaining angle (|x| < pi / 127,
//     from an exact integer difference) by Taylor series to x^7 and x^6, joined by
//     the addition theorems.
#pragma once
#include "device_common.hpp"

namespace oasmc {

constexpr int kExpEntries = 128;
constexpr int kLogEntries = 128;
constexpr int kCircle = 128;

// 2^(j / 128) and what its rounding leaves
__device__ const double2 kExpTable[kExpEntries] = {
    {0x1.0000000000000p+0, 0x0.0p+0}, {0x1.0163da9fb3335p+0, 0x1.b61299ab8cdb7p-54},
    {0x1.02c9a3e778061p+0, -0x1.19083535b085dp-56}, {0x1.04315e86e7f85p+0, -0x1.0a31c1977c96ep-54},
    {0x1.059b0d3158574p+0, 0x1.d73e2a475b465p-55}, {0x1.0706b29ddf6dep+0, -0x1.c91dfe2b13c27p-55},
    {0x1.0874518759bc8p+0, 0x1.186be4bb284ffp-57}, {0x1.09e3ecac6f383p+0, 0x1.1487818316136p-54},
    {0x1.0b5586cf9890fp+0, 0x1.8a62e4adc610bp-54}, {0x1.0cc922b7247f7p+0, 0x1.01edc16e24f71p-54},
    {0x1.0e3ec32d3d1a2p+0, 0x1.03a1727c57b53p-59}, {0x1.0fb66affed31bp+0, -0x1.b9bedc44ebd7bp-57},
    {0x1.11301d0125b51p+0, -0x1.6c51039449b3ap-54}, {0x1.12abdc06c31ccp+0, -0x1.1b514b36ca5c7p-58},
    {0x1.1429aaea92de0p+0, -0x1.32fbf9af1369ep-54}, {0x1.15a98c8a58e51p+0, 0x1.2406ab9eeab0ap-55},
    {0x1.172b83c7d517bp+0, -0x1.19041b9d78a76p-55}, {0x1.18af9388c8deap+0, -0x1.11023d1970f6cp-54},
    {0x1.1a35beb6fcb75p+0, 0x1.e5b4c7b4968e4p-55}, {0x1.1bbe084045cd4p+0, -0x1.95386352ef607p-54},
    {0x1.1d4873168b9aap+0, 0x1.e016e00a2643cp-54}, {0x1.1ed5022fcd91dp+0, -0x1.1df98027bb78cp-54},
    {0x1.2063b88628cd6p+0, 0x1.dc775814a8495p-55}, {0x1.21f49917ddc96p+0, 0x1.2a97e9494a5eep-55},
    {0x1.2387a6e756238p+0, 0x1.9b07eb6c70573p-54}, {0x1.251ce4fb2a63fp+0, 0x1.ac155bef4f4a4p-55},
    {0x1.26b4565e27cddp+0, 0x1.2bd339940e9d9p-55}, {0x1.284dfe1f56381p+0, -0x1.a4c3a8c3f0d7ep-54},
    {0x1.29e9df51fdee1p+0, 0x1.612e8afad1255p-55}, {0x1.2b87fd0dad990p+0, -0x1.10adcd6381aa4p-59},
    {0x1.2d285a6e4030bp+0, 0x1.0024754db41d5p-54}, {0x1.2ecafa93e2f56p+0, 0x1.1ca0f45d52383p-56},
    {0x1.306fe0a31b715p+0, 0x1.6f46ad23182e4p-55}, {0x1.32170fc4cd831p+0, 0x1.a9ce78e18047cp-55},
    {0x1.33c08b26416ffp+0, 0x1.32721843659a6p-54}, {0x1.356c55f929ff1p+0, -0x1.b5cee5c4e4628p-55},
    {0x1.371a7373aa9cbp+0, -0x1.63aeabf42eae2p-54}, {0x1.38cae6d05d866p+0, -0x1.e958d3c9904bdp-54},
    {0x1.3a7db34e59ff7p+0, -0x1.5e436d661f5e3p-56}, {0x1.3c32dc313a8e5p+0, -0x1.efff8375d29c3p-54},
    {0x1.3dea64c123422p+0, 0x1.ada0911f09ebcp-55}, {0x1.3fa4504ac801cp+0, -0x1.7d023f956f9f3p-54},
    {0x1.4160a21f72e2ap+0, -0x1.ef3691c309278p-58}, {0x1.431f5d950a897p+0, -0x1.1c7dde35f7999p-55},
    {0x1.44e086061892dp+0, 0x1.89b7a04ef80d0p-59}, {0x1.46a41ed1d0057p+0, 0x1.c944bd1648a76p-54},
    {0x1.486a2b5c13cd0p+0, 0x1.3c1a3b69062f0p-56}, {0x1.4a32af0d7d3dep+0, 0x1.9cb62f3d1be56p-54},
    {0x1.4bfdad5362a27p+0, 0x1.d4397afec42e2p-56}, {0x1.4dcb299fddd0dp+0, 0x1.8ecdbbc6a7833p-54},
    {0x1.4f9b2769d2ca7p+0, -0x1.4b309d25957e3p-54}, {0x1.516daa2cf6642p+0, -0x1.f768569bd93efp-55},
    {0x1.5342b569d4f82p+0, -0x1.07abe1db13cadp-55}, {0x1.551a4ca5d920fp+0, -0x1.d689cefede59bp-55},
    {0x1.56f4736b527dap+0, 0x1.9bb2c011d93adp-54}, {0x1.58d12d497c7fdp+0, 0x1.295e15b9a1de8p-55},
    {0x1.5ab07dd485429p+0, 0x1.6324c054647adp-54}, {0x1.5c9268a5946b7p+0, 0x1.c4b1b816986a2p-60},
    {0x1.5e76f15ad2148p+0, 0x1.ba6f93080e65ep-54}, {0x1.605e1b976dc09p+0, -0x1.3e2429b56de47p-54},
    {0x1.6247eb03a5585p+0, -0x1.383c17e40b497p-54}, {0x1.6434634ccc320p+0, -0x1.c483c759d8933p-55},
    {0x1.6623882552225p+0, -0x1.bb60987591c34p-54}, {0x1.68155d44ca973p+0, 0x1.038ae44f73e65p-57},
    {0x1.6a09e667f3bcdp+0, -0x1.bdd3413b26456p-54}, {0x1.6c012750bdabfp+0, -0x1.2895667ff0b0dp-56},
    {0x1.6dfb23c651a2fp+0, -0x1.bbe3a683c88abp-57}, {0x1.6ff7df9519484p+0, -0x1.83c0f25860ef6p-55},
    {0x1.71f75e8ec5f74p+0, -0x1.16e4786887a99p-55}, {0x1.73f9a48a58174p+0, -0x1.0a8d96c65d53cp-54},
    {0x1.75feb564267c9p+0, -0x1.0245957316dd3p-54}, {0x1.780694fde5d3fp+0, 0x1.866b80a02162dp-54},
    {0x1.7a11473eb0187p+0, -0x1.41577ee04992fp-55}, {0x1.7c1ed0130c132p+0, 0x1.f124cd1164dd6p-54},
    {0x1.7e2f336cf4e62p+0, 0x1.05d02ba15797ep-56}, {0x1.80427543e1a12p+0, -0x1.27c86626d972bp-54},
    {0x1.82589994cce13p+0, -0x1.d4c1dd41532d8p-54}, {0x1.8471a4623c7adp+0, -0x1.8d684a341cdfbp-55},
    {0x1.868d99b4492edp+0, -0x1.fc6f89bd4f6bap-54}, {0x1.88ac7d98a6699p+0, 0x1.994c2f37cb53ap-54},
    {0x1.8ace5422aa0dbp+0, 0x1.6e9f156864b27p-54}, {0x1.8cf3216b5448cp+0, -0x1.0d55e32e9e3aap-56},
    {0x1.8f1ae99157736p+0, 0x1.5cc13a2e3976cp-55}, {0x1.9145b0b91ffc6p+0, -0x1.dd6792e582524p-54},
    {0x1.93737b0cdc5e5p+0, -0x1.75fc781b57ebcp-57}, {0x1.95a44cbc8520fp+0, -0x1.64b7c96a5f039p-56},
    {0x1.97d829fde4e50p+0, -0x1.d185b7c1b85d1p-54}, {0x1.9a0f170ca07bap+0, -0x1.173bd91cee632p-54},
    {0x1.9c49182a3f090p+0, 0x1.c7c46b071f2bep-56}, {0x1.9e86319e32323p+0, 0x1.824ca78e64c6ep-56},
    {0x1.a0c667b5de565p+0, -0x1.359495d1cd533p-54}, {0x1.a309bec4a2d33p+0, 0x1.6305c7ddc36abp-54},
    {0x1.a5503b23e255dp+0, -0x1.d2f6edb8d41e1p-54}, {0x1.a799e1330b358p+0, 0x1.bcb7ecac563c7p-54},
    {0x1.a9e6b5579fdbfp+0, 0x1.0fac90ef7fd31p-54}, {0x1.ac36bbfd3f37ap+0, -0x1.f9234cae76cd0p-55},
    {0x1.ae89f995ad3adp+0, 0x1.7a1cd345dcc81p-54}, {0x1.b0e07298db666p+0, -0x1.bdef54c80e425p-54},
    {0x1.b33a2b84f15fbp+0, -0x1.2805e3084d708p-57}, {0x1.b59728de5593ap+0, -0x1.c71dfbbba6de3p-54},
    {0x1.b7f76f2fb5e47p+0, -0x1.5584f7e54ac3bp-56}, {0x1.ba5b030a1064ap+0, -0x1.efcd30e54292ep-54},
    {0x1.bcc1e904bc1d2p+0, 0x1.23dd07a2d9e84p-55}, {0x1.bf2c25bd71e09p+0, -0x1.efdca3f6b9c73p-54},
    {0x1.c199bdd85529cp+0, 0x1.11065895048ddp-55}, {0x1.c40ab5fffd07ap+0, 0x1.b4537e083c60ap-54},
    {0x1.c67f12e57d14bp+0, 0x1.2884dff483cadp-54}, {0x1.c8f6d9406e7b5p+0, 0x1.1acbc48805c44p-56},
    {0x1.cb720dcef9069p+0, 0x1.503cbd1e949dbp-56}, {0x1.cdf0b555dc3fap+0, -0x1.dd83b53829d72p-55},
    {0x1.d072d4a07897cp+0, -0x1.cbc3743797a9cp-54}, {0x1.d2f87080d89f2p+0, -0x1.d487b719d8578p-54},
    {0x1.d5818dcfba487p+0, 0x1.2ed02d75b3707p-55}, {0x1.d80e316c98398p+0, -0x1.11ec18beddfe8p-54},
    {0x1.da9e603db3285p+0, 0x1.c2300696db532p-54}, {0x1.dd321f301b460p+0, 0x1.2da5778f018c3p-54},
    {0x1.dfc97337b9b5fp+0, -0x1.1a5cd4f184b5cp-54}, {0x1.e264614f5a129p+0, -0x1.7b627817a1496p-54},
    {0x1.e502ee78b3ff6p+0, 0x1.39e8980a9cc8fp-55}, {0x1.e7a51fbc74c83p+0, 0x1.2d522ca0c8de2p-54},
    {0x1.ea4afa2a490dap+0, -0x1.e9c23179c2893p-54}, {0x1.ecf482d8e67f1p+0, -0x1.c93f3b411ad8cp-54},
    {0x1.efa1bee615a27p+0, 0x1.dc7f486a4b6b0p-54}, {0x1.f252b376bba97p+0, 0x1.3a1a5bf0d8e43p-54},
    {0x1.f50765b6e4540p+0, 0x1.9d3e12dd8a18bp-54}, {0x1.f7bfdad9cbe14p+0, -0x1.dbb12d006350ap-54},
    {0x1.fa7c1819e90d8p+0, 0x1.74853f3a5931ep-55}, {0x1.fd3c22b8f71f1p+0, 0x1.2eb74966579e7p-57},
};

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
    0, -941, 8596, 5965, -249, 17459, 82, 109,
    5076, -1018, -3533, 1803, -9185, -9660, -15705, -5729,
    -2838, 5729, 15705, 9660, 9185, -1803, 3533, 1018,
    -5076, -109, -82, -17459, 249, -5965, -8596, 941,
    0, -941, 8596, 5965, -249, 17459, 82, 109,
    5076, -1018, -3533, 1803, -9185, -9660, -15705, -5729,
    2838, 5729, 15705, 9660, 9185, -1803, 3533, 1018,
    -5076, -109, -82, -17459, 249, -5965, -8596, 941,
    0, -941, 8596, 5965, -249, 17459, 82, 109,
    5076, -1018, -3533, 1803, -9185, -9660, -15705, -5729,
    -2838, 5729, 15705, 9660, 9185, -1803, 3533, 1018,
    -5076, -109, -82, -17459, 249, -5965, -8596, 941,
    0, -941, 8596, 5965, -249, 17459, 82, 109,
    5076, -1018, -3533, 1803, -9185, -9660, -15705, -5729,
    2838, 5729, 15705, 9660, 9185, -1803, 3533, 1018,
    -5076, -109, -82, -17459, 249, -5965, -8596, 941,
};
__device__ const double2 kCircleTable[kCircle] = {
    {0x0.0p+0, 0x1.0000000000000p+0}, {0x1.91f37ce57b513p-5, 0x1.ff62207bcddb8p-1},
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
    {0x1.fd88b0e08872fp-1, 0x1.91878b250fc49p-4}, {0x1.ff62207bcddb8p-1, 0x1.91f37ce57b513p-5},
    {0x1.0000000000000p+0, 0x0.0p+0}, {0x1.ff62207bcddb8p-1, -0x1.91f37ce57b513p-5},
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
    {0x1.91878b250fc49p-4, -0x1.fd88b0e08872fp-1}, {0x1.91f37ce57b513p-5, -0x1.ff62207bcddb8p-1},
    {0x0.0p+0, -0x1.0000000000000p+0}, {-0x1.91f37ce57b513p-5, -0x1.ff62207bcddb8p-1},
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
    {-0x1.fd88b0e08872fp-1, -0x1.91878b250fc49p-4}, {-0x1.ff62207bcddb8p-1, -0x1.91f37ce57b513p-5},
    {-0x1.0000000000000p+0, 0x0.0p+0}, {-0x1.ff62207bcddb8p-1, 0x1.91f37ce57b513p-5},
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
    {-0x1.91878b250fc49p-4, 0x1.fd88b0e08872fp-1}, {-0x1.91f37ce57b513p-5, 0x1.ff62207bcddb8p-1},
};

// The tables in LDS.
struct NormalTables {
    double2 exp[kExpEntries];
    double2 log[kLogEntries];
    double2 circle[kCircle];
    int32_t offset[kCircle];
};

// Copied by the whole workgroup; the caller's next barrier publishes them.
__device__ __forceinline__ void stage_tables(NormalTables& t)
{
    for (int i = threadIdx.x; i < kExpEntries; i += blockDim.x) t.exp[i] = kExpTable[i];
    for (int i = threadIdx.x; i < kLogEntries; i += blockDim.x) t.log[i] = kLogTable[i];
    for (int i = threadIdx.x; i < kCircle; i += blockDim.x) {
        t.circle[i] = kCircleTable[i];
        t.offset[i] = kCircleOffset[i];
    }
}

// -2 log(v 2^-SHIFT) of a positive, finite, normal v.
template <int SHIFT>
__device__ __forceinline__ double minus2_log(const NormalTables& tb, double v)
{
    const uint32_t hi = (uint32_t)__double2hiint(v);
    const double2 t = tb.log[(hi >> 13) & (kLogEntries - 1)];
    const double m = __hiloint2double((int)((hi & 0x000FFFFFu) | 0x3FF00000u), __double2loint(v));
    // octaves below v = 2^SHIFT; the upper half of an octave counts to the next
    const double k = (double)((1023 + SHIFT) - (int)((hi + 0x00080000u) >> 20));
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

// -2 log((w + 1/2) 2^-32), positive.
__device__ __forceinline__ double minus2_log_word(const NormalTables& tb, uint32_t w)
{
    return minus2_log<32>(tb, (double)w + 0.5);
}

// log of a sum of weights relative to their largest, in [1, 2^10] (or NaN: NaN).
__device__ __forceinline__ double log_sum(const NormalTables& tb, double s)
{
    return (s == s) ? -0.5 * minus2_log<0>(tb, s) : s;
}

// exp(x) for x <= 0, -inf (0) and NaN (NaN): x = (128 n + j) log 2 / 128 + r, the
// table's 2^(j / 128) and the series of exp(r) to r^5 (|r| < 0.0028).
__device__ __forceinline__ double exp_neg(const NormalTables& tb, double x)
{
    x = (x < -1100.0) ? -1100.0 : x;
    const double magic = 0x1.8p+52;  // the sum's low word is the nearest integer
    const double t = fma(x, 0x1.71547652b82fep+7, magic);
    const double k = t - magic;
    const int n = __double2loint(t);
    const double r = fma(k, -0x1.1cf79abc9e3b4p-43, fma(k, -0x1.62e42fef80000p-8, x));
    const double2 e = tb.exp[n & (kExpEntries - 1)];
    double p = fma(r, 1.0 / 120.0, 1.0 / 24.0);
    p = fma(p, r, 1.0 / 6.0);
    p = fma(p, r, 0.5);
    const double q = fma(r * r, p, r);
    return ldexp(e.x + fma(e.x, q, e.y), n >> 7);
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
    const double sp = fma(fma(z, -1.0 / 5040.0, 1.0 / 120.0), z, -1.0 / 6.0);
    const double cp = fma(fma(z, -1.0 / 720.0, 1.0 / 24.0), z, -1.0 / 2.0);
    // sin x (with the low parts of the product and of 2 pi) and cos x - 1
    const double lo = fma(d, 0x1.1a62633145c07p-84, fma(d, 0x1.921fb54442d18p-30, -x));
    const double sx = x + fma(x * z, sp, lo);
    const double cm = z * cp;
    s = t.x + fma(t.y, sx, t.x * cm);
    c = t.y + fma(-t.x, sx, t.y * cm);
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
