// Host build of the POW cone's membership test (cones.hpp) at points within a few
// ulps of the boundary.  Prints how many points further than 4 ulps from it are
// taken for the other side.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
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
static double __builtin_amdgcn_rcp(double x) { return 1.0 / x * (1.0 + 1e-8); }
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
  std::mt19937_64 g(5);
  std::uniform_real_distribution<double> u(0.0, 1.0);
  long wrong = 0;
  for (long i = 0; i < count; ++i) {
    const double al = 0.1 + 0.8 * u(g), bl = 1.0 - al, x = std::pow(10.0, 160.0 * u(g) - 80.0);
    const double y = std::pow(10.0, 160.0 * u(g) - 80.0);
    const long double edge = expl(al * logl(x) + bl * logl(y));
    const double z = (double)(edge * (1.0L + (40.0 * u(g) - 20.0) * 2.2e-16L));
    const long double off = ((long double)z - edge) / edge / 2.2e-16L;
    const bool in = pdhcg::pow_reaches(x, y, al, z);
    if (off > 4.0L && in) ++wrong;
    if (off < -4.0L && !in) ++wrong;
  }
  printf("%ld\n", wrong);
  return 0;
}
