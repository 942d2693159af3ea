// The functions of qed_math.h compiled for the CPU: the hardware's estimates are replaced by
// values off by the given fraction of their documented error (2^-23 of the result).  Prints
// each function's largest error over n arguments, in units of 2^-53 of the result (log2:
// absolute), and how often sqrt and the quotient were not the correctly rounded ones.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>

#define __device__
#define __forceinline__ inline
struct double2 {
  double x, y;
};
static inline double2 make_double2(double x, double y) { return {x, y}; }
static inline uint64_t word(double x) {
  uint64_t u;
  std::memcpy(&u, &x, 8);
  return u;
}
static inline int __double2hiint(double x) { return (int)(word(x) >> 32); }
static inline int __double2loint(double x) { return (int)(uint32_t)word(x); }
static inline double __hiloint2double(int h, int l) {
  const uint64_t u = ((uint64_t)(uint32_t)h << 32) | (uint32_t)l;
  double x;
  std::memcpy(&x, &u, 8);
  return x;
}
static struct {
  unsigned x;
} threadIdx;
static double off = 0.0;
static inline double __builtin_amdgcn_rsq(double x) {
  return (double)(1.0L / sqrtl(x)) * (1.0 + off);
}
static inline double __builtin_amdgcn_rcp(double x) { return 1.0 / x * (1.0 + off); }
using std::fma;
using std::ldexp;
using std::rint;

#include "qed_math.h"

using namespace qedk;

static uint64_t state;
static double uniform() {  // splitmix64
  uint64_t z = (state += 0x9E3779B97F4A7C15ull);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return (double)((z ^ (z >> 31)) >> 11) * 0x1p-53;
}
static double spread(double lo, double hi) { return exp2(lo + (hi - lo) * uniform()); }

int main(int argc, char** argv) {
  const long n = argc > 1 ? atol(argv[1]) : 100000;
  MathTab t;
  for (threadIdx.x = 0; threadIdx.x < kMathN; ++threadIdx.x) store_math(t, load_math());
  const char* names[] = {"rsqrt", "rcp", "exp", "pow23", "log2", "affine", "sqrt", "div"};
  for (int f = 0; f < 8; ++f) {
    double worst = 0.0;
    long wrong = 0;
    state = 100 + f;
    for (long i = 0; i < n; ++i) {
      off = (2.0 * uniform() - 1.0) * 0x1p-23;
      const double x = f == 2   ? 128.0 * uniform()
                       : f == 3 ? spread(-400, 400)
                       : f == 4 ? 1.0 + uniform()
                       : f == 5 ? spread(-20, 7)
                                : spread(-899, 899);
      long double got = 0, want = 1, unit = 0;
      if (f == 0) got = rsqrt_normal(x), want = 1 / sqrtl(x);
      if (f == 1) got = rcp_normal(x), want = 1 / (long double)x;
      if (f == 2) got = exp_neg(t, x), want = expl(-(long double)x);
      if (f == 3) {
        got = pow23_normal(t, x);
        want = cbrtl((long double)x * x);
      }
      if (f == 4) {
        got = log2_mantissa(t, (uint32_t)__double2hiint(x), (uint32_t)__double2loint(x));
        want = log2l(x), unit = 1;
      }
      if (f == 5) {
        const double scale = 4095.0 / 27.0;
        got = log2_affine(t, x, -20, scale, 0.0);
        want = (log2l(x) + 20) * (long double)scale, unit = 4096;  // half an ulp: one unit
      }
      if (f == 6) {
        got = sqrt_from_rsqrt(x, rsqrt_normal(x));
        wrong += (double)got != sqrt(x);
        want = sqrtl(x);
      }
      if (f == 7) {
        const double a = spread(-400, 400), b = spread(-400, 400);
        got = div_normal(a, b, rcp_normal(b));
        wrong += (double)got != a / b;
        want = (long double)a / b;
      }
      if (unit == 0) unit = fabsl(want);
      const double e = (double)(fabsl(got - want) / unit * 0x1p53L);
      if (!(e <= worst)) worst = e;  // (a NaN sticks)
    }
    printf("%s %.6f %ld\n", names[f], worst, wrong);
  }
  // beyond the fast ranges' edges the callers take the library: the edges themselves are in
  const double edge[] = {kFastLo, kFastHi};
  off = 0.0;
  double worst = 0.0;
  for (double x : edge) {
    const double e[] = {fabs(rcp_normal(x) * x - 1.0),
                        fabs(rsqrt_normal(x) * sqrt(x) - 1.0)};
    for (double v : e) worst = v > worst || v != v ? v : worst;
  }
  const double ends[] = {kPow23Lo, kPow23Hi};
  for (double x : ends) {
    const double v = (double)(fabsl(pow23_normal(t, x) / cbrtl((long double)x * x) - 1));
    worst = v > worst || v != v ? v : worst;
  }
  printf("edges %.6f 0\n", worst * 0x1p53);
  return 0;
}
