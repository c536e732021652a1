// Exponentials in double precision for the exact scores, shorter than the math library's: their arguments are a logit less its row's
// maximum or log-sum-exp, so nothing above about zero matters and what lies below exp(-690) adds nothing to a sum that is at least one or
// that ends in single precision.
//
// exp(x) = 2^(k / 256) exp(x - k ln2 / 256), k the nearest whole number to 256 x / ln2: 2^((k mod 256) / 256) from a table in LDS (the
// lanes' reads spread over the banks), the Taylor series to the fourth power on |r| <= h = ln2 / 512 (its fifth term, 3.8e-17, is put on the
// third: 0.87 h^2 r^3 is within a seventh of h^5 of r^5), the rest of k into the exponent.  k comes out of the low word of a sum with
// 1.5 * 2^52.  k ln2 / 256 is subtracted in two parts and the table's own rounding is added back before the last step: the error is at most
// 1.2e-16 of the result for every argument (the library's: 1.4e-16; with one part and the table as it is 2.3e-16 near zero and 2.3e-14 at
// -690).  The score passes of 96 heads x 2048 tokens x 128 rows at head_dim 64: 153 us (149 without these two, 170 with the library's).
#pragma once
#include "common.hpp"

namespace obf {

constexpr int kExpTab = 256;           // a power of two, the workgroup's threads at most
constexpr double kExpFloor = -690.0;      // smaller arguments are raised to this one (no denormal appears); not-a-number passes through

__device__ const double kExp2Frac[kExpTab] = {
    0x1.0000000000000p+0, 0x1.00b1afa5abcbfp+0, 0x1.0163da9fb3335p+0, 0x1.02168143b0281p+0,
    0x1.02c9a3e778061p+0, 0x1.037d42e11bbccp+0, 0x1.04315e86e7f85p+0, 0x1.04e5f72f654b1p+0,
    0x1.059b0d3158574p+0, 0x1.0650a0e3c1f89p+0, 0x1.0706b29ddf6dep+0, 0x1.07bd42b72a836p+0,
    0x1.0874518759bc8p+0, 0x1.092bdf66607e0p+0, 0x1.09e3ecac6f383p+0, 0x1.0a9c79b1f3919p+0,
    0x1.0b5586cf9890fp+0, 0x1.0c0f145e46c85p+0, 0x1.0cc922b7247f7p+0, 0x1.0d83b23395decp+0,
    0x1.0e3ec32d3d1a2p+0, 0x1.0efa55fdfa9c5p+0, 0x1.0fb66affed31bp+0, 0x1.1073028d7233ep+0,
    0x1.11301d0125b51p+0, 0x1.11edbab5e2ab6p+0, 0x1.12abdc06c31ccp+0, 0x1.136a814f204abp+0,
    0x1.1429aaea92de0p+0, 0x1.14e95934f312ep+0, 0x1.15a98c8a58e51p+0, 0x1.166a45471c3c2p+0,
    0x1.172b83c7d517bp+0, 0x1.17ed48695bbc0p+0, 0x1.18af9388c8deap+0, 0x1.1972658375d2fp+0,
    0x1.1a35beb6fcb75p+0, 0x1.1af99f8138a1cp+0, 0x1.1bbe084045cd4p+0, 0x1.1c82f95281c6bp+0,
    0x1.1d4873168b9aap+0, 0x1.1e0e75eb44027p+0, 0x1.1ed5022fcd91dp+0, 0x1.1f9c18438ce4dp+0,
    0x1.2063b88628cd6p+0, 0x1.212be3578a819p+0, 0x1.21f49917ddc96p+0, 0x1.22bdda27912d1p+0,
    0x1.2387a6e756238p+0, 0x1.2451ffb82140ap+0, 0x1.251ce4fb2a63fp+0, 0x1.25e85711ece75p+0,
    0x1.26b4565e27cddp+0, 0x1.2780e341ddf29p+0, 0x1.284dfe1f56381p+0, 0x1.291ba7591bb70p+0,
    0x1.29e9df51fdee1p+0, 0x1.2ab8a66d10f13p+0, 0x1.2b87fd0dad990p+0, 0x1.2c57e39771b2fp+0,
    0x1.2d285a6e4030bp+0, 0x1.2df961f641589p+0, 0x1.2ecafa93e2f56p+0, 0x1.2f9d24abd886bp+0,
    0x1.306fe0a31b715p+0, 0x1.31432edeeb2fdp+0, 0x1.32170fc4cd831p+0, 0x1.32eb83ba8ea32p+0,
    0x1.33c08b26416ffp+0, 0x1.3496266e3fa2dp+0, 0x1.356c55f929ff1p+0, 0x1.36431a2de883bp+0,
    0x1.371a7373aa9cbp+0, 0x1.37f26231e754ap+0, 0x1.38cae6d05d866p+0, 0x1.39a401b7140efp+0,
    0x1.3a7db34e59ff7p+0, 0x1.3b57fbfec6cf4p+0, 0x1.3c32dc313a8e5p+0, 0x1.3d0e544ede173p+0,
    0x1.3dea64c123422p+0, 0x1.3ec70df1c5175p+0, 0x1.3fa4504ac801cp+0, 0x1.40822c367a024p+0,
    0x1.4160a21f72e2ap+0, 0x1.423fb2709468ap+0, 0x1.431f5d950a897p+0, 0x1.43ffa3f84b9d4p+0,
    0x1.44e086061892dp+0, 0x1.45c2042a7d232p+0, 0x1.46a41ed1d0057p+0, 0x1.4786d668b3237p+0,
    0x1.486a2b5c13cd0p+0, 0x1.494e1e192aed2p+0, 0x1.4a32af0d7d3dep+0, 0x1.4b17dea6db7d7p+0,
    0x1.4bfdad5362a27p+0, 0x1.4ce41b817c114p+0, 0x1.4dcb299fddd0dp+0, 0x1.4eb2d81d8abffp+0,
    0x1.4f9b2769d2ca7p+0, 0x1.508417f4531eep+0, 0x1.516daa2cf6642p+0, 0x1.5257de83f4eefp+0,
    0x1.5342b569d4f82p+0, 0x1.542e2f4f6ad27p+0, 0x1.551a4ca5d920fp+0, 0x1.56070dde910d2p+0,
    0x1.56f4736b527dap+0, 0x1.57e27dbe2c4cfp+0, 0x1.58d12d497c7fdp+0, 0x1.59c0827ff07ccp+0,
    0x1.5ab07dd485429p+0, 0x1.5ba11fba87a03p+0, 0x1.5c9268a5946b7p+0, 0x1.5d84590998b93p+0,
    0x1.5e76f15ad2148p+0, 0x1.5f6a320dceb71p+0, 0x1.605e1b976dc09p+0, 0x1.6152ae6cdf6f4p+0,
    0x1.6247eb03a5585p+0, 0x1.633dd1d1929fdp+0, 0x1.6434634ccc320p+0, 0x1.652b9febc8fb7p+0,
    0x1.6623882552225p+0, 0x1.671c1c70833f6p+0, 0x1.68155d44ca973p+0, 0x1.690f4b19e9538p+0,
    0x1.6a09e667f3bcdp+0, 0x1.6b052fa75173ep+0, 0x1.6c012750bdabfp+0, 0x1.6cfdcddd47645p+0,
    0x1.6dfb23c651a2fp+0, 0x1.6ef9298593ae5p+0, 0x1.6ff7df9519484p+0, 0x1.70f7466f42e87p+0,
    0x1.71f75e8ec5f74p+0, 0x1.72f8286ead08ap+0, 0x1.73f9a48a58174p+0, 0x1.74fbd35d7cbfdp+0,
    0x1.75feb564267c9p+0, 0x1.77024b1ab6e09p+0, 0x1.780694fde5d3fp+0, 0x1.790b938ac1cf6p+0,
    0x1.7a11473eb0187p+0, 0x1.7b17b0976cfdbp+0, 0x1.7c1ed0130c132p+0, 0x1.7d26a62ff86f0p+0,
    0x1.7e2f336cf4e62p+0, 0x1.7f3878491c491p+0, 0x1.80427543e1a12p+0, 0x1.814d2add106d9p+0,
    0x1.82589994cce13p+0, 0x1.8364c1eb941f7p+0, 0x1.8471a4623c7adp+0, 0x1.857f4179f5b21p+0,
    0x1.868d99b4492edp+0, 0x1.879cad931a436p+0, 0x1.88ac7d98a6699p+0, 0x1.89bd0a478580fp+0,
    0x1.8ace5422aa0dbp+0, 0x1.8be05bad61778p+0, 0x1.8cf3216b5448cp+0, 0x1.8e06a5e0866d9p+0,
    0x1.8f1ae99157736p+0, 0x1.902fed0282c8ap+0, 0x1.9145b0b91ffc6p+0, 0x1.925c353aa2fe2p+0,
    0x1.93737b0cdc5e5p+0, 0x1.948b82b5f98e5p+0, 0x1.95a44cbc8520fp+0, 0x1.96bdd9a7670b3p+0,
    0x1.97d829fde4e50p+0, 0x1.98f33e47a22a2p+0, 0x1.9a0f170ca07bap+0, 0x1.9b2bb4d53fe0dp+0,
    0x1.9c49182a3f090p+0, 0x1.9d674194bb8d5p+0, 0x1.9e86319e32323p+0, 0x1.9fa5e8d07f29ep+0,
    0x1.a0c667b5de565p+0, 0x1.a1e7aed8eb8bbp+0, 0x1.a309bec4a2d33p+0, 0x1.a42c980460ad8p+0,
    0x1.a5503b23e255dp+0, 0x1.a674a8af46052p+0, 0x1.a799e1330b358p+0, 0x1.a8bfe53c12e59p+0,
    0x1.a9e6b5579fdbfp+0, 0x1.ab0e521356ebap+0, 0x1.ac36bbfd3f37ap+0, 0x1.ad5ff3a3c2774p+0,
    0x1.ae89f995ad3adp+0, 0x1.afb4ce622f2ffp+0, 0x1.b0e07298db666p+0, 0x1.b20ce6c9a8952p+0,
    0x1.b33a2b84f15fbp+0, 0x1.b468415b749b1p+0, 0x1.b59728de5593ap+0, 0x1.b6c6e29f1c52ap+0,
    0x1.b7f76f2fb5e47p+0, 0x1.b928cf22749e4p+0, 0x1.ba5b030a1064ap+0, 0x1.bb8e0b79a6f1fp+0,
    0x1.bcc1e904bc1d2p+0, 0x1.bdf69c3f3a207p+0, 0x1.bf2c25bd71e09p+0, 0x1.c06286141b33dp+0,
    0x1.c199bdd85529cp+0, 0x1.c2d1cd9fa652cp+0, 0x1.c40ab5fffd07ap+0, 0x1.c544778fafb22p+0,
    0x1.c67f12e57d14bp+0, 0x1.c7ba88988c933p+0, 0x1.c8f6d9406e7b5p+0, 0x1.ca3405751c4dbp+0,
    0x1.cb720dcef9069p+0, 0x1.ccb0f2e6d1675p+0, 0x1.cdf0b555dc3fap+0, 0x1.cf3155b5bab74p+0,
    0x1.d072d4a07897cp+0, 0x1.d1b532b08c968p+0, 0x1.d2f87080d89f2p+0, 0x1.d43c8eacaa1d6p+0,
    0x1.d5818dcfba487p+0, 0x1.d6c76e862e6d3p+0, 0x1.d80e316c98398p+0, 0x1.d955d71ff6075p+0,
    0x1.da9e603db3285p+0, 0x1.dbe7cd63a8315p+0, 0x1.dd321f301b460p+0, 0x1.de7d5641c0658p+0,
    0x1.dfc97337b9b5fp+0, 0x1.e11676b197d17p+0, 0x1.e264614f5a129p+0, 0x1.e3b333b16ee12p+0,
    0x1.e502ee78b3ff6p+0, 0x1.e653924676d76p+0, 0x1.e7a51fbc74c83p+0, 0x1.e8f7977cdb740p+0,
    0x1.ea4afa2a490dap+0, 0x1.eb9f4867cca6ep+0, 0x1.ecf482d8e67f1p+0, 0x1.ee4aaa2188510p+0,
    0x1.efa1bee615a27p+0, 0x1.f0f9c1cb6412ap+0, 0x1.f252b376bba97p+0, 0x1.f3ac948dd7274p+0,
    0x1.f50765b6e4540p+0, 0x1.f6632798844f8p+0, 0x1.f7bfdad9cbe14p+0, 0x1.f91d802243c89p+0,
    0x1.fa7c1819e90d8p+0, 0x1.fbdba3692d514p+0, 0x1.fd3c22b8f71f1p+0, 0x1.fe9d96b2a23d9p+0,
};

// (2^(i / 256) - the entry) over the entry: high words of doubles whose low words are zero
__device__ const uint32_t kExp2Rest[kExpTab] = {
    0x00000000, 0xbc84e830, 0x3c9b3b4f, 0xbc82985e, 0xbc716014, 0x3c651e61, 0xbc905e7a, 0x3c845fad,
    0x3c8cd252, 0xbc954529, 0xbc8bce80, 0x3c829371, 0x3c60f74e, 0xbc95b928, 0x3c90a3e4, 0x3c84f31f,
    0x3c979aa6, 0x3c9407fb, 0x3c8eb51b, 0xbc9a5d05, 0x3c3ebe3d, 0xbc937a02, 0xbc6a0335, 0x3c8b8269,
    0xbc955652, 0xbc9ac46e, 0xbc5080f0, 0xbc65704f, 0xbc91c924, 0xbc897cea, 0x3c80d3e4, 0x3c56f014,
    0xbc801b16, 0x3c6e653b, 0xbc8f1ff0, 0x3c92cc7f, 0x3c8b898c, 0x3c957bfb, 0xbc96d99c, 0x3c8cdc18,
    0x3c9aecf7, 0xbc949368, 0xbc8fe783, 0xbc98e28a, 0x3c8a6f41, 0x3c9120fd, 0x3c807a06, 0x3c89b789,
    0x3c968efe, 0x3c877afc, 0x3c875e19, 0x3c91512f, 0x3c80472c, 0x3c9a02f1, 0xbc96b87b, 0xbc803298,
    0x3c82f7e1, 0xbc95b77e, 0xbc3d219b, 0xbc91e75c, 0x3c8b3782, 0x3c98a912, 0x3c6e1493, 0xbc61e7ca,
    0x3c834d75, 0x3c85425c, 0x3c864202, 0xbc979518, 0x3c8fdd39, 0xbc800e2a, 0xbc86a380, 0xbc874308,
    0xbc924aee, 0xbc954de3, 0xbc9907f8, 0xbc94f248, 0xbc71d1e8, 0x3c914a54, 0xbc99191a, 0x3c79c3bc,
    0x3c859f49, 0xbc85a716, 0xbc931260, 0x3c86421f, 0xbc58a78f, 0xbc9348a7, 0xbc7c2c9b, 0x3c835c44,
    0x3c4363ed, 0xbc632afd, 0x3c966609, 0xbc95fc5e, 0x3c6ecce2, 0xbc7ea015, 0x3c93ff8e, 0xbc7a843b,
    0x3c7690cf, 0x3c892ca4, 0x3c931dbe, 0xbc902c9a, 0xbc8f9434, 0x3c73e34f, 0xbc87decd, 0xbc75a3b1,
    0xbc78dec7, 0x3c81bd29, 0xbc861247, 0xbc896be9, 0x3c933505, 0xbc88e6ad, 0x3c7b98b7, 0xbc91af7f,
    0x3c9063e2, 0xbc943a35, 0x3c34c785, 0xbc951f59, 0x3c9432e6, 0xbc82e165, 0xbc8ce44a, 0x3c95f30f,
    0xbc8c33c5, 0x3c917ece, 0xbc845379, 0xbc9345f4, 0xbc93cedd, 0xbc85c340, 0x3c5710ab, 0x3c81079b,
    0xbc93b3f0, 0x3c727df1, 0xbc6a12ae, 0x3c93f992, 0xbc6367f0, 0xbc875579, 0xbc80dc3d, 0x3c51ed2f,
    0xbc781f64, 0xbc88e67b, 0xbc86ee4b, 0x3c865975, 0xbc861932, 0x3c92c0b7, 0x3c909ccb, 0x3c8a30fb,
    0xbc7b32dd, 0xbc92dad3, 0x3c94ecfd, 0x3c87d514, 0x3c65ebe2, 0xbc760a36, 0xbc88a1c5, 0x3c8b18c7,
    0xbc9369b7, 0x3c90ec1e, 0xbc805e84, 0xbc522cea, 0xbc94d451, 0x3c7c8855, 0x3c90ad67, 0x3c931144,
    0x3c8db730, 0x3c93e9e9, 0xbc65b661, 0xbc8dac43, 0x3c7bf683, 0x3c8b99de, 0xbc930920, 0xbc7885ad,
    0xbc5da9b9, 0xbc82d5e8, 0xbc6c23f9, 0xbc516694, 0xbc924343, 0x3c71f2b3, 0xbc85ca6d, 0xbc9294f3,
    0x3c71affc, 0xbc8a1e58, 0x3c6dd236, 0xbc79740b, 0xbc87c504, 0x3c916583, 0x3c8b1c87, 0xbc903d5d,
    0xbc91bbd2, 0x3c598618, 0x3c90cc32, 0xbc894729, 0x3c846984, 0x3c7d8158, 0xbc82dfce, 0x3c8c8a4e,
    0x3c8c1a78, 0xbc888c8d, 0xbc907b8f, 0x3c889c2f, 0xbc55c3d9, 0xbc7274af, 0xbc90a40e, 0x3c85c621,
    0xbc68d6f4, 0xbc8fda53, 0xbc91eee2, 0xbc32141a, 0x3c74ffd7, 0xbc302899, 0xbc91bdfc, 0xbc80dda3,
    0x3c736eae, 0xbc8a007e, 0x3c8ee332, 0x3c836909, 0x3c84e090, 0xbc811cd8, 0x3c63cdaf, 0xbc7ac28b,
    0x3c676b2c, 0xbc703058, 0xbc808a19, 0xbc8cc734, 0xbc8fad5d, 0x3c87752a, 0xbc900dae, 0x3c85b670,
    0x3c74a386, 0x3c5159da, 0xbc82919e, 0x3c8c254d, 0x3c8e5a51, 0xbc8d8c33, 0x3c843a5a, 0xbc8ea6e7,
    0xbc82d521, 0xbc63e8e4, 0xbc892ab9, 0xbc8b7967, 0x3c74b604, 0xbc776caa, 0x3c83c5ec, 0xbc81d5fc,
    0xbc8ff713, 0x3c855cd9, 0xbc8dae99, 0x3c826994, 0x3c8ec3bc, 0xbc83b613, 0x3c842b95, 0xbc69fa75,
    0x3c8a64a9, 0x3c901f3a, 0xbc8e37bb, 0xbc516a9d, 0x3c77893b, 0xbc699c7e, 0x3c5305c1, 0x3c64b458,
};

struct ExpTable {
  double frac[kExpTab];
  uint32_t rest[kExpTab];
};

// the table into LDS, by the first threads of a workgroup; a barrier follows before the first use
__device__ __forceinline__ void exp_table(ExpTable& tab, int tid) {
  if (tid < kExpTab) { tab.frac[tid] = kExp2Frac[tid]; tab.rest[tid] = kExp2Rest[tid]; }
}

// exp(x), x not below kExpFloor
__device__ __forceinline__ double exp_tab(double x, const ExpTable& tab) {
  const double magic = 6755399441055744.0;                                                     // 1.5 * 2^52
  const double t = fma(x, 0x1.71547652b82fep+8, magic), n = t - magic;                  // 256 / ln2
  const double r = fma(n, -0x1.abc9e3b39803fp-64, fma(n, -0x1.62e42fefa39efp-9, x));        // ln2 / 256: the double, and what it lacks
  const uint32_t k = (uint32_t)__double2loint(t);
  const double e = tab.frac[k & (kExpTab - 1)], rest = __hiloint2double((int)tab.rest[k & (kExpTab - 1)], 0);
  const double f = __hiloint2double(__double2hiint(e) + (int)((k >> 8) << 20), __double2loint(e));
  const double p = fma(r, fma(r, fma(r, 1.0 / 24, 0x1.5555571de4f61p-3), 0.5), 1.0);
  return fma(f, fma(p, r, rest), f);
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
