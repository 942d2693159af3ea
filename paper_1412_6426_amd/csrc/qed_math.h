// qed_math.h -- FP64 elementary functions of the sub-step path.
//
// A lepton sub-step is bound by the instructions it issues: one wavefront holds a SIMD for 4
// cycles per FP64 instruction, and a sub-step is a chain with little to overlap.  The library
// takes 17 instructions for a square root, 10 for a division, 75 for a log2 (it carries a
// double-double), 26 for an exp and 45 for a cube root; the forms here, whose operands the
// callers keep within the ranges that each states, take 3 to 20, x^(2/3) 45.  log2 and exp are
// table-driven (P. T. P. Tang, ACM TOMS 15, 144 (1989) and 16, 378 (1990)).
//
// None is less exact than what it stands for.  Largest errors over 10^6 arguments each against
// extended precision, in units of 2^-53 of the result (in brackets the library's, over 2^22):
//   rsqrt_normal 1.24 (1.5 for 1 / sqrt), rcp_normal 1.00 (1.0), exp_neg 1.00 (1.2),
//   pow23_normal 1.00 (1.3 for the cube root of the square);
//   log2_affine: 2^-53 |scale| and the two roundings that its comment names (the library's log2,
//   a subtraction and a product took three).
// sqrt_from_rsqrt and div_normal agreed with the correctly rounded result in every one of them.
// That is no proof: their last step starts from an inverse good to 1.2 units, where Markstein's
// theorem asks for the correctly rounded one, so that an argument whose root or quotient lies
// within 2^-52 units of a rounding boundary may still round the other way.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace qedk {

constexpr int kMathN = 64;  // entries of each table

// Mantissa interval j of [1, 2): an inverse c_j of its middle 1 + (j + 1/2) / 64 and -log2 of
// the rounded c_j; and 2^(j / 64).
static __device__ const double kLog2Tab[kMathN][2] = {
    {0x1.fc07f01fc07f0p-1, 0x1.6fe50b6ef085dp-7}, {0x1.f44659e4a4271p-1, 0x1.11cd1d513341bp-5},
    {0x1.ecc07b301ecc0p-1, 0x1.c4dfab90aab6ap-5}, {0x1.e573ac901e574p-1, 0x1.3aa2fdd27f1bfp-4},
    {0x1.de5d6e3f8868ap-1, 0x1.918a16e46335ep-4}, {0x1.d77b654b82c34p-1, 0x1.e72ec117fa5adp-4},
    {0x1.d0cb58f6ec074p-1, 0x1.1dcd197552b7dp-3}, {0x1.ca4b3055ee191p-1, 0x1.476a9f983f74dp-3},
    {0x1.c3f8f01c3f8f0p-1, 0x1.70742d4ef0280p-3}, {0x1.bdd2b899406f7p-1, 0x1.98edd077e70e1p-3},
    {0x1.b7d6c3dda338bp-1, 0x1.c0db6cdd94defp-3}, {0x1.b2036406c80d9p-1, 0x1.e840be74e6a4dp-3},
    {0x1.ac5701ac5701bp-1, 0x1.0790adbb03009p-2}, {0x1.a6d01a6d01a6dp-1, 0x1.1ac05b291f070p-2},
    {0x1.a16d3f97a4b02p-1, 0x1.2db10fc4d9aaep-2}, {0x1.9c2d14ee4a102p-1, 0x1.406463b1b0448p-2},
    {0x1.970e4f80cb872p-1, 0x1.52dbdfc4c96b5p-2}, {0x1.920fb49d0e229p-1, 0x1.6518fe4677ba6p-2},
    {0x1.8d3018d3018d3p-1, 0x1.771d2ba7efb3cp-2}, {0x1.886e5f0abb04ap-1, 0x1.88e9c72e0b224p-2},
    {0x1.83c977ab2beddp-1, 0x1.9a802391e2330p-2}, {0x1.7f405fd017f40p-1, 0x1.abe18797f1f4ap-2},
    {0x1.7ad2208e0ecc3p-1, 0x1.bd0f2e9e79032p-2}, {0x1.767dce434a9b1p-1, 0x1.ce0a4923a587dp-2},
    {0x1.724287f46debcp-1, 0x1.ded3fd442364cp-2}, {0x1.6e1f76b4337c7p-1, 0x1.ef6d67328e220p-2},
    {0x1.6a13cd1537290p-1, 0x1.ffd799a83ff9cp-2}, {0x1.661ec6a5122f9p-1, 0x1.0809cf27f703dp-1},
    {0x1.623fa77016240p-1, 0x1.10113b153c8eap-1}, {0x1.5e75bb8d015e7p-1, 0x1.18028cf72976bp-1},
    {0x1.5ac056b015ac0p-1, 0x1.1fde3d30e8127p-1}, {0x1.571ed3c506b3ap-1, 0x1.27a4c0585cbf7p-1},
    {0x1.5390948f40febp-1, 0x1.2f56875eb3f26p-1}, {0x1.5015015015015p-1, 0x1.36f3ffb6d9162p-1},
    {0x1.4cab88725af6ep-1, 0x1.3e7d9379f7017p-1}, {0x1.49539e3b2d067p-1, 0x1.45f3a98a20738p-1},
    {0x1.460cbc7f5cf9ap-1, 0x1.4d56a5b33cec5p-1}, {0x1.42d6625d51f87p-1, 0x1.54a6e8ca5438ep-1},
    {0x1.3fb013fb013fbp-1, 0x1.5be4d0cb51435p-1}, {0x1.3c995a47babe7p-1, 0x1.6310b8f553049p-1},
    {0x1.3991c2c187f63p-1, 0x1.6a2af9e5a0f0bp-1}, {0x1.3698df3de0748p-1, 0x1.7133e9b156c7bp-1},
    {0x1.33ae45b57bcb2p-1, 0x1.782bdbfdda657p-1}, {0x1.30d190130d190p-1, 0x1.7f1322182cf16p-1},
    {0x1.2e025c04b8097p-1, 0x1.85ea0b0b27b26p-1}, {0x1.2b404ad012b40p-1, 0x1.8cb0e3b4b3bbep-1},
    {0x1.288b01288b013p-1, 0x1.9367f6da0ab2dp-1}, {0x1.25e22708092f1p-1, 0x1.9a0f8d3b0e050p-1},
    {0x1.23456789abcdfp-1, 0x1.a0a7eda4c112dp-1}, {0x1.20b470c67c0d9p-1, 0x1.a7315d02f20c7p-1},
    {0x1.1e2ef3b3fb874p-1, 0x1.adac1e711c833p-1}, {0x1.1bb4a4046ed29p-1, 0x1.b418734a9008cp-1},
    {0x1.19453808ca29cp-1, 0x1.ba769b39e4964p-1}, {0x1.16e0689427379p-1, 0x1.c0c6d447c5dd3p-1},
    {0x1.1485f0e0acd3bp-1, 0x1.c7095ae91e1c8p-1}, {0x1.12358e75d3033p-1, 0x1.cd3e6a0ca8908p-1},
    {0x1.0fef010fef011p-1, 0x1.d3663b27f31d5p-1}, {0x1.0db20a88f4696p-1, 0x1.d9810643d6614p-1},
    {0x1.0b7e6ec259dc8p-1, 0x1.df8f02086af2bp-1}, {0x1.0953f39010954p-1, 0x1.e59063c8822cep-1},
    {0x1.073260a47f7c6p-1, 0x1.eb855f8ca88fcp-1}, {0x1.05197f7d73404p-1, 0x1.f16e281db7630p-1},
    {0x1.03091b51f5e1ap-1, 0x1.f74aef0efafafp-1}, {0x1.0101010101010p-1, 0x1.fd1be4c7f2af9p-1},
};
static __device__ const double kExp2Tab[kMathN][2] = {
    {0x1.0000000000000p+0, 0x0.0p+0}, {0x1.02c9a3e778061p+0, -0x1.19083535b085dp-56},
    {0x1.059b0d3158574p+0, 0x1.d73e2a475b465p-55}, {0x1.0874518759bc8p+0, 0x1.186be4bb284ffp-57},
    {0x1.0b5586cf9890fp+0, 0x1.8a62e4adc610bp-54}, {0x1.0e3ec32d3d1a2p+0, 0x1.03a1727c57b53p-59},
    {0x1.11301d0125b51p+0, -0x1.6c51039449b3ap-54}, {0x1.1429aaea92de0p+0, -0x1.32fbf9af1369ep-54},
    {0x1.172b83c7d517bp+0, -0x1.19041b9d78a76p-55}, {0x1.1a35beb6fcb75p+0, 0x1.e5b4c7b4968e4p-55},
    {0x1.1d4873168b9aap+0, 0x1.e016e00a2643cp-54}, {0x1.2063b88628cd6p+0, 0x1.dc775814a8495p-55},
    {0x1.2387a6e756238p+0, 0x1.9b07eb6c70573p-54}, {0x1.26b4565e27cddp+0, 0x1.2bd339940e9d9p-55},
    {0x1.29e9df51fdee1p+0, 0x1.612e8afad1255p-55}, {0x1.2d285a6e4030bp+0, 0x1.0024754db41d5p-54},
    {0x1.306fe0a31b715p+0, 0x1.6f46ad23182e4p-55}, {0x1.33c08b26416ffp+0, 0x1.32721843659a6p-54},
    {0x1.371a7373aa9cbp+0, -0x1.63aeabf42eae2p-54}, {0x1.3a7db34e59ff7p+0, -0x1.5e436d661f5e3p-56},
    {0x1.3dea64c123422p+0, 0x1.ada0911f09ebcp-55}, {0x1.4160a21f72e2ap+0, -0x1.ef3691c309278p-58},
    {0x1.44e086061892dp+0, 0x1.89b7a04ef80d0p-59}, {0x1.486a2b5c13cd0p+0, 0x1.3c1a3b69062f0p-56},
    {0x1.4bfdad5362a27p+0, 0x1.d4397afec42e2p-56}, {0x1.4f9b2769d2ca7p+0, -0x1.4b309d25957e3p-54},
    {0x1.5342b569d4f82p+0, -0x1.07abe1db13cadp-55}, {0x1.56f4736b527dap+0, 0x1.9bb2c011d93adp-54},
    {0x1.5ab07dd485429p+0, 0x1.6324c054647adp-54}, {0x1.5e76f15ad2148p+0, 0x1.ba6f93080e65ep-54},
    {0x1.6247eb03a5585p+0, -0x1.383c17e40b497p-54}, {0x1.6623882552225p+0, -0x1.bb60987591c34p-54},
    {0x1.6a09e667f3bcdp+0, -0x1.bdd3413b26456p-54}, {0x1.6dfb23c651a2fp+0, -0x1.bbe3a683c88abp-57},
    {0x1.71f75e8ec5f74p+0, -0x1.16e4786887a99p-55}, {0x1.75feb564267c9p+0, -0x1.0245957316dd3p-54},
    {0x1.7a11473eb0187p+0, -0x1.41577ee04992fp-55}, {0x1.7e2f336cf4e62p+0, 0x1.05d02ba15797ep-56},
    {0x1.82589994cce13p+0, -0x1.d4c1dd41532d8p-54}, {0x1.868d99b4492edp+0, -0x1.fc6f89bd4f6bap-54},
    {0x1.8ace5422aa0dbp+0, 0x1.6e9f156864b27p-54}, {0x1.8f1ae99157736p+0, 0x1.5cc13a2e3976cp-55},
    {0x1.93737b0cdc5e5p+0, -0x1.75fc781b57ebcp-57}, {0x1.97d829fde4e50p+0, -0x1.d185b7c1b85d1p-54},
    {0x1.9c49182a3f090p+0, 0x1.c7c46b071f2bep-56}, {0x1.a0c667b5de565p+0, -0x1.359495d1cd533p-54},
    {0x1.a5503b23e255dp+0, -0x1.d2f6edb8d41e1p-54}, {0x1.a9e6b5579fdbfp+0, 0x1.0fac90ef7fd31p-54},
    {0x1.ae89f995ad3adp+0, 0x1.7a1cd345dcc81p-54}, {0x1.b33a2b84f15fbp+0, -0x1.2805e3084d708p-57},
    {0x1.b7f76f2fb5e47p+0, -0x1.5584f7e54ac3bp-56}, {0x1.bcc1e904bc1d2p+0, 0x1.23dd07a2d9e84p-55},
    {0x1.c199bdd85529cp+0, 0x1.11065895048ddp-55}, {0x1.c67f12e57d14bp+0, 0x1.2884dff483cadp-54},
    {0x1.cb720dcef9069p+0, 0x1.503cbd1e949dbp-56}, {0x1.d072d4a07897cp+0, -0x1.cbc3743797a9cp-54},
    {0x1.d5818dcfba487p+0, 0x1.2ed02d75b3707p-55}, {0x1.da9e603db3285p+0, 0x1.c2300696db532p-54},
    {0x1.dfc97337b9b5fp+0, -0x1.1a5cd4f184b5cp-54}, {0x1.e502ee78b3ff6p+0, 0x1.39e8980a9cc8fp-55},
    {0x1.ea4afa2a490dap+0, -0x1.e9c23179c2893p-54}, {0x1.efa1bee615a27p+0, 0x1.dc7f486a4b6b0p-54},
    {0x1.f50765b6e4540p+0, 0x1.9d3e12dd8a18bp-54}, {0x1.fa7c1819e90d8p+0, 0x1.74853f3a5931ep-55},
};

// The tables in LDS (1.5 KB a workgroup): the first wavefront's loads go out at the kernel's
// start, under its first reads of the step's header, and are stored once they are needed; a
// barrier follows.
struct MathTab {
  double2 lg[kMathN];
  double2 ex[kMathN];
};
struct MathRow {
  double2 l, e;
};
__device__ __forceinline__ MathRow load_math() {
  const int j = (int)threadIdx.x & (kMathN - 1);
  return {make_double2(kLog2Tab[j][0], kLog2Tab[j][1]),
          make_double2(kExp2Tab[j][0], kExp2Tab[j][1])};
}
__device__ __forceinline__ void store_math(MathTab& m, const MathRow& r) {
  if (threadIdx.x < kMathN) {
    m.lg[threadIdx.x] = r.l;
    m.ex[threadIdx.x] = r.e;
  }
}
__device__ __forceinline__ void stage_math(MathTab& m) { store_math(m, load_math()); }

// Operands of the functions below lie in [2^-900, 2^900].
constexpr double kFastLo = 0x1p-900, kFastHi = 0x1p900;

// x^(-1/2): the hardware estimate y (24 bits) and one third-order step; with
// e = 1 - x y^2, x^(-1/2) = y (1 - e)^(-1/2) = y (1 + e/2 + 3 e^2/8 + O(e^3)).
__device__ __forceinline__ double rsqrt_normal(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-(x * y), y, 1.0);
  return fma(y * e, fma(e, 0.375, 0.5), y);
}
// x^(1/2) from y = rsqrt_normal(x): the product's remainder is exact, so that one correction
// rounds correctly.
__device__ __forceinline__ double sqrt_from_rsqrt(double x, double y) {
  const double g = x * y;
  return fma(fma(-g, g, x), 0.5 * y, g);
}
// 1/x: with e = 1 - x y, 1/x = y (1 + e + e^2 + O(e^3)).
__device__ __forceinline__ double rcp_normal(double x) {
  const double y = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, y, 1.0);
  return fma(y, fma(e, e, e), y);
}

// a / b from ib, 1/b to a unit in the last place: the quotient's remainder is exact and its
// correction rounds once, so the result is the correctly rounded quotient (a, b and a / b
// normal).
__device__ __forceinline__ double div_normal(double a, double b, double ib) {
  const double q = a * ib;
  return fma(fma(-q, b, a), ib, q);
}

// Fraction part of log2 for a mantissa m in [1, 2): log2(m) = lg + log2(1 + r), r = m c - 1,
// |r| < 2^-7: the series to r^7 / 7 leaves 3e-18.
__device__ __forceinline__ double log2_mantissa(const MathTab& t, uint32_t hi, uint32_t lo) {
  const double2 c = t.lg[(hi >> 14) & (kMathN - 1)];
  const double m = __hiloint2double((int)((hi & 0x000FFFFFu) | 0x3FF00000u), (int)lo);
  const double r = fma(m, c.x, -1.0);
  double p = 0x1.a61762a7aded9p-3;
  p = fma(p, r, -0x1.ec709dc3a03fdp-3);
  p = fma(p, r, 0x1.2776c50ef9bfep-2);
  p = fma(p, r, -0x1.71547652b82fep-2);
  p = fma(p, r, 0x1.ec709dc3a03fdp-2);
  p = fma(p, r, -0x1.71547652b82fep-1);
  p = fma(p, r, 0x1.71547652b82fep+0);
  return fma(p, r, c.y);
}
// (log2 x - lo) scale + offset for an integer lo: one rounding of the whole octaves' part, one
// of the sum, and scale times the fraction's error.
__device__ __forceinline__ double log2_affine(const MathTab& t, double x, int lo, double scale,
                                              double offset) {
  const uint32_t xh = (uint32_t)__double2hiint(x), xl = (uint32_t)__double2loint(x);
  const double octaves = (double)((int)(xh >> 20) - 1023 - lo);
  return fma(log2_mantissa(t, xh, xl), scale, fma(octaves, scale, offset));
}

// e^r 2^(k / 64) for |r| <= ln 2 / 128 (the series to r^6 / 720 leaves 3e-20)
__device__ __forceinline__ double exp_reduced(const MathTab& t, double r, int k) {
  const double2 f = t.ex[k & (kMathN - 1)];
  double p = 1.0 / 720.0;
  p = fma(p, r, 1.0 / 120.0);
  p = fma(p, r, 1.0 / 24.0);
  p = fma(p, r, 1.0 / 6.0);
  p = fma(p, r, 0.5);
  p = fma(p, r, 1.0);
  return ldexp(f.x + fma(f.x, r * p, f.y), k >> 6);
}
// e^-x for 0 <= x <= 600
__device__ __forceinline__ double exp_neg(const MathTab& t, double x) {
  const double n = rint(x * -0x1.71547652b82fep+6);
  double r = fma(n, -0x1.62e42fefa39efp-7, -x);
  r = fma(n, -0x1.abc9e3b39803fp-62, r);
  return exp_reduced(t, r, (int)n);
}
// x^(2/3) for 2^-400 <= x <= 2^400.  With x = 2^(3q + s) m, the power is
// 2^(2q) 2^(2/3 (s + log2 m)); that is good to 4 units of 2^-53, and one Newton step of
// y^3 = x^2, whose residual is taken with both squares' low parts, leaves a rounding.
constexpr double kPow23Lo = 0x1p-400, kPow23Hi = 0x1p400;
__device__ __forceinline__ double pow23_normal(const MathTab& t, double x) {
  const uint32_t hi = (uint32_t)__double2hiint(x), lo = (uint32_t)__double2loint(x);
  const int b = (int)(hi >> 20);  // exponent + 1023, and 1023 = 3 * 341
  const int q = b / 3;
  const double l = (2.0 / 3.0) * ((double)(b - 3 * q) + log2_mantissa(t, hi, lo));
  const double n = rint(64.0 * l);
  const double y = exp_reduced(t, fma(n, -1.0 / 64.0, l) * 0x1.62e42fefa39efp-1,
                               (int)n + 128 * (q - 341));
  const double x2 = x * x, y2 = y * y;
  const double xe = fma(x, x, -x2), ye = fma(y, y, -y2);
  const double res = fma(-y, y2, x2) + fma(-y, ye, xe);
  return fma(res * __builtin_amdgcn_rcp(y2), 1.0 / 3.0, y);
}

}  // namespace qedk
