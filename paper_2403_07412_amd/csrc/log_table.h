// Table of the logarithm log_staged in device_common.h: for the 64 intervals
// [1/2 + j/128, 1/2 + (j + 1)/128) of the mantissa, c = 1 / midpoint rounded to
// ten fractional bits and -log c rounded to the nearest double.
#pragma once

namespace vecchia {

constexpr int kLogTableSize = 64;

struct LogTableEntry {
    double c, neg_log_c;
};

constexpr LogTableEntry kLogMant64[kLogTableSize] = {
    {0x1.fc00000000000p+0, -0x1.5ee02a9241675p-1},
    {0x1.f440000000000p+0, -0x1.5701226128af8p-1},
    {0x1.ecc0000000000p+0, -0x1.4f45283594e19p-1},
    {0x1.e580000000000p+0, -0x1.47ae52544ae44p-1},
    {0x1.de40000000000p+0, -0x1.3ffa411a427c1p-1},
    {0x1.d780000000000p+0, -0x1.38b3216b5778ep-1},
    {0x1.d0c0000000000p+0, -0x1.3151241c2fc5fp-1},
    {0x1.ca40000000000p+0, -0x1.2a1b06a9db6dap-1},
    {0x1.c400000000000p+0, -0x1.23130d7bebf43p-1},
    {0x1.bdc0000000000p+0, -0x1.1bf2042752c42p-1},
    {0x1.b7c0000000000p+0, -0x1.1501bebf93522p-1},
    {0x1.b200000000000p+0, -0x1.0e44985d1cc8cp-1},
    {0x1.ac40000000000p+0, -0x1.07706f9625913p-1},
    {0x1.a6c0000000000p+0, -0x1.00d22dfc0e10bp-1},
    {0x1.a180000000000p+0, -0x1.f4d87dd7b97e6p-2},
    {0x1.9c40000000000p+0, -0x1.e7e32b29c349ep-2},
    {0x1.9700000000000p+0, -0x1.dac353e2c5954p-2},
    {0x1.9200000000000p+0, -0x1.ce1af0b85f3ebp-2},
    {0x1.8d40000000000p+0, -0x1.c1ef05c1dfd59p-2},
    {0x1.8880000000000p+0, -0x1.b59d9f3bea7c2p-2},
    {0x1.83c0000000000p+0, -0x1.a925d37a8c58bp-2},
    {0x1.7f40000000000p+0, -0x1.9d31bea13ed3bp-2},
    {0x1.7ac0000000000p+0, -0x1.9119850995d54p-2},
    {0x1.7680000000000p+0, -0x1.858b57725cc43p-2},
    {0x1.7240000000000p+0, -0x1.79db6681afacbp-2},
    {0x1.6e00000000000p+0, -0x1.6e08eaa2ba1e4p-2},
    {0x1.6a00000000000p+0, -0x1.62c82f2b9c795p-2},
    {0x1.6600000000000p+0, -0x1.5767717455a6cp-2},
    {0x1.6240000000000p+0, -0x1.4c9f09e152c3cp-2},
    {0x1.5e80000000000p+0, -0x1.41b941cce0beep-2},
    {0x1.5ac0000000000p+0, -0x1.36b5776bc1117p-2},
    {0x1.5700000000000p+0, -0x1.2b9303ab89d25p-2},
    {0x1.5380000000000p+0, -0x1.211255986160cp-2},
    {0x1.5000000000000p+0, -0x1.1675cababa60ep-2},
    {0x1.4cc0000000000p+0, -0x1.0c81d4860a869p-2},
    {0x1.4940000000000p+0, -0x1.01ade39139ef7p-2},
    {0x1.4600000000000p+0, -0x1.ef0adcbdc5936p-3},
    {0x1.42c0000000000p+0, -0x1.da85d620ce500p-3},
    {0x1.3fc0000000000p+0, -0x1.c765b9e4d68d6p-3},
    {0x1.3c80000000000p+0, -0x1.b2797ee46320cp-3},
    {0x1.3980000000000p+0, -0x1.9ef83d2769a34p-3},
    {0x1.3680000000000p+0, -0x1.8b46f8223625bp-3},
    {0x1.33c0000000000p+0, -0x1.790ed4ee26333p-3},
    {0x1.30c0000000000p+0, -0x1.64fee8825fc4bp-3},
    {0x1.2e00000000000p+0, -0x1.526e5e3a1b438p-3},
    {0x1.2b40000000000p+0, -0x1.3fb25a59528cbp-3},
    {0x1.2880000000000p+0, -0x1.2cca0f5f5f251p-3},
    {0x1.2600000000000p+0, -0x1.1b72ad52f67a0p-3},
    {0x1.2340000000000p+0, -0x1.08338affa282ap-3},
    {0x1.20c0000000000p+0, -0x1.ed1794e83780cp-4},
    {0x1.1e40000000000p+0, -0x1.c97978d78e920p-4},
    {0x1.1bc0000000000p+0, -0x1.a58b60c2b2324p-4},
    {0x1.1940000000000p+0, -0x1.814be23f8c036p-4},
    {0x1.1700000000000p+0, -0x1.60658a93750c4p-4},
    {0x1.1480000000000p+0, -0x1.3b87598b1b6eep-4},
    {0x1.1240000000000p+0, -0x1.1a0fba1bf8a52p-4},
    {0x1.1000000000000p+0, -0x1.f0a30c01162a6p-5},
    {0x1.0dc0000000000p+0, -0x1.ac97221711f8dp-5},
    {0x1.0b80000000000p+0, -0x1.67f94f094bd98p-5},
    {0x1.0940000000000p+0, -0x1.22c71bcea83a5p-5},
    {0x1.0740000000000p+0, -0x1.c98d18d00c814p-6},
    {0x1.0500000000000p+0, -0x1.3cea44346a575p-6},
    {0x1.0300000000000p+0, -0x1.7dc475f810a77p-7},
    {0x1.0100000000000p+0, -0x1.ff00aa2b10bc0p-9},
};

// -ln(c_j / 2) of the first entries, for mantissas below 0.703: the logarithm
// takes these as twice the mantissa under an exponent one less, so that
// arguments just above 1 do not add ln2 to a -ln c near -ln2.
constexpr int kLogLowEntries = 26;
constexpr double kLogMantLow[kLogLowEntries] = {
    0x1.010157588de71p-7, 0x1.7c61b1cf5dee0p-6, 0x1.39f07ba0ebd62p-5,
    0x1.b35dd9b58baadp-5, 0x1.174f76ab09171p-4, 0x1.518874226130ap-4,
    0x1.8c985e9b9ec84p-4, 0x1.c6494a2e418a6p-4, 0x1.fe89139dbd566p-4,
    0x1.1bc8af21436b3p-3, 0x1.3789c4c041337p-3, 0x1.527e5e4a1b58dp-3,
    0x1.6dcf0165f8373p-3, 0x1.884807ce5638fp-3, 0x1.a1dfc40f1b7f1p-3,
    0x1.bbca696b07e80p-3, 0x1.d60a17f903515p-3, 0x1.ef5ade4dcffe6p-3,
    0x1.03d95a1d67686p-2, 0x1.102ac0a35cc1cp-2, 0x1.1ca28c64bae54p-2,
    0x1.2896a13e086a4p-2, 0x1.34aedad5b168bp-2, 0x1.403d086cea79cp-2,
    0x1.4becf95d97913p-2, 0x1.57bf753c8d1fbp-2,
};

}  // namespace vecchia
