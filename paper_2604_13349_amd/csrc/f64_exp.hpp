// Exponentials in double precision for the exact scores, shorter than the math library's: their arguments are a logit less its row's
// maximum or log-sum-exp, so nothing above about zero matters and what lies below exp(-690) adds nothing to a sum that is at least one or
// that ends in single precision.
//
// exp(x) = 2^(k / 64) exp(x - k ln2 / 64), k the nearest whole number to 64 x / ln2: 2^((k mod 64) / 64) from a table in LDS (512 bytes:
// the lanes' reads spread over the banks), the Taylor series to the fifth power on |r| <= ln2 / 128 (the sixth is 3.5e-17), the rest of k
// into the exponent.  k comes out of the low word of a sum with 1.5 * 2^52.  k ln2 / 64 is subtracted in one step: its error, 1.1e-16 |x|,
// is that of the logit itself.
#pragma once
#include "common.hpp"

namespace obf {

constexpr int kExpTab = 64;
constexpr double kExpFloor = -690.0;      // smaller arguments are raised to this one (no denormal appears); not-a-number passes through

__device__ const double kExp2Frac[kExpTab] = {
    0x1.0000000000000p+0, 0x1.02c9a3e778061p+0, 0x1.059b0d3158574p+0, 0x1.0874518759bc8p+0,
    0x1.0b5586cf9890fp+0, 0x1.0e3ec32d3d1a2p+0, 0x1.11301d0125b51p+0, 0x1.1429aaea92de0p+0,
    0x1.172b83c7d517bp+0, 0x1.1a35beb6fcb75p+0, 0x1.1d4873168b9aap+0, 0x1.2063b88628cd6p+0,
    0x1.2387a6e756238p+0, 0x1.26b4565e27cddp+0, 0x1.29e9df51fdee1p+0, 0x1.2d285a6e4030bp+0,
    0x1.306fe0a31b715p+0, 0x1.33c08b26416ffp+0, 0x1.371a7373aa9cbp+0, 0x1.3a7db34e59ff7p+0,
    0x1.3dea64c123422p+0, 0x1.4160a21f72e2ap+0, 0x1.44e086061892dp+0, 0x1.486a2b5c13cd0p+0,
    0x1.4bfdad5362a27p+0, 0x1.4f9b2769d2ca7p+0, 0x1.5342b569d4f82p+0, 0x1.56f4736b527dap+0,
    0x1.5ab07dd485429p+0, 0x1.5e76f15ad2148p+0, 0x1.6247eb03a5585p+0, 0x1.6623882552225p+0,
    0x1.6a09e667f3bcdp+0, 0x1.6dfb23c651a2fp+0, 0x1.71f75e8ec5f74p+0, 0x1.75feb564267c9p+0,
    0x1.7a11473eb0187p+0, 0x1.7e2f336cf4e62p+0, 0x1.82589994cce13p+0, 0x1.868d99b4492edp+0,
    0x1.8ace5422aa0dbp+0, 0x1.8f1ae99157736p+0, 0x1.93737b0cdc5e5p+0, 0x1.97d829fde4e50p+0,
    0x1.9c49182a3f090p+0, 0x1.a0c667b5de565p+0, 0x1.a5503b23e255dp+0, 0x1.a9e6b5579fdbfp+0,
    0x1.ae89f995ad3adp+0, 0x1.b33a2b84f15fbp+0, 0x1.b7f76f2fb5e47p+0, 0x1.bcc1e904bc1d2p+0,
    0x1.c199bdd85529cp+0, 0x1.c67f12e57d14bp+0, 0x1.cb720dcef9069p+0, 0x1.d072d4a07897cp+0,
    0x1.d5818dcfba487p+0, 0x1.da9e603db3285p+0, 0x1.dfc97337b9b5fp+0, 0x1.e502ee78b3ff6p+0,
    0x1.ea4afa2a490dap+0, 0x1.efa1bee615a27p+0, 0x1.f50765b6e4540p+0, 0x1.fa7c1819e90d8p+0,
};

// the table into LDS, by the first threads of a workgroup; a barrier follows before the first use
__device__ __forceinline__ void exp_table(double* tab, int tid) { if (tid < kExpTab) tab[tid] = kExp2Frac[tid]; }

// exp(x), x not below kExpFloor
__device__ __forceinline__ double exp_tab(double x, const double* tab) {
  const double magic = 6755399441055744.0;                                                     // 1.5 * 2^52
  const double t = fma(x, 0x1.71547652b82fep+6, magic);                                 // 64 / ln2
  const double r = fma(t - magic, -0x1.62e42fefa39efp-7, x);                                // ln2 / 64
  const uint32_t k = (uint32_t)__double2loint(t);
  const double e = tab[k & (kExpTab - 1)];
  const double f = __hiloint2double(__double2hiint(e) + (int)((k >> 6) << 20), __double2loint(e));
  const double p = fma(r, fma(r, fma(r, fma(r, 1.0 / 120, 1.0 / 24), 1.0 / 6), 0.5), 1.0);
  return fma(f, p * r, f);
}

// x[0..3] raised to the floor: the comparison is all that usually runs
__device__ __forceinline__ void exp_clamp(double (&x)[4]) {
  const bool low = x[0] < kExpFloor || x[1] < kExpFloor || x[2] < kExpFloor || x[3] < kExpFloor;
  if (__ballot(low)) {
    asm volatile("");                                          // a branch, not twelve selects on the usual way
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = x[i] < kExpFloor ? kExpFloor : x[i];
  }
}

}  // namespace obf
