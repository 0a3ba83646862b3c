// Host build of quotient (cones.hpp) against the division it stands for: prints
// how many of `count` random pairs differ in any bit.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>

#define __device__
#define __noinline__ __attribute__((noinline))
#define __forceinline__ inline
using std::isfinite;
using std::isnan;
struct Dim {
  int x;
};
static Dim threadIdx, blockIdx;
static double __builtin_amdgcn_rcp(double x) { return 1.0 / x; }
static int __builtin_amdgcn_update_dpp(int, int, int, int, int, bool) { return 0; }
static int __builtin_amdgcn_ds_swizzle(int, int) { return 0; }
static int __builtin_amdgcn_readlane(int v, int) { return v; }
static int __double2loint(double) { return 0; }
static int __double2hiint(double) { return 0; }
static double __hiloint2double(int, int) { return 0; }
static unsigned atomicAdd(unsigned* p, unsigned v) { return (*p += v) - v; }
enum { PDHCG_CONE_EXP = 4, PDHCG_CONE_POW = 5 };
#include "cones.hpp"

int main(int argc, char** argv) {
  const long count = atol(argv[1]);
  std::mt19937_64 g(3);
  std::uniform_real_distribution<double> u(0.0, 1.0);
  long differ = 0;
  for (long i = 0; i < count; ++i) {
    const double a = (u(g) - 0.5) * std::pow(10.0, 200.0 * u(g) - 100.0), b = (0.5 + u(g)) * std::pow(10.0, 40.0 * u(g) - 20.0);
    const double q = pdhcg::quotient(a, b, 1.0 / b), d = a / b;
    differ += std::memcmp(&q, &d, sizeof(q)) != 0;
  }
  printf("%ld\n", differ);
  return 0;
}
