// Host build of the device root-finders (cones.hpp): every block is projected
// cold and from warm starts of all kinds, and the largest difference relative
// to max(1, ||r||_inf) is printed.
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
// the hardware's reciprocal is approximate: 1e-8 relative here
static double __builtin_amdgcn_rcp(double x) { return 1.0 / x * (1.0 + 1e-8); }
// cross-lane operations of the blocks that a group of lanes shares: not run
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
  const bool pow_block = atoi(argv[1]) != 0;
  const long count = atol(argv[2]);
  std::mt19937_64 g(11);
  std::normal_distribution<double> nd;
  std::uniform_real_distribution<double> u(0.0, 1.0);
  double worst = 0.0, last = 0.0;
  for (long i = 0; i < count; ++i) {
    double r[3], m[3];
    const double sc = std::pow(10.0, 4.0 * u(g) - 2.0), al = 0.1 + 0.8 * u(g);
    for (int k = 0; k < 3; ++k) {
      r[k] = nd(g) * sc * (u(g) < 0.2 ? std::pow(10.0, -6.0 * u(g)) : 1.0);
      m[k] = std::pow(10.0, 2.0 * u(g) - 1.0);
    }
    auto project = [&](double* warm, double* o) {
      if (pow_block) pdhcg::project_pow_body(r[0], r[1], r[2], al, m[0], m[1], m[2], o, warm);
      else pdhcg::project_exp_body(r[0], r[1], r[2], m[0], m[1], m[2], o, warm);
    };
    double cold[3];
    project(nullptr, cold);
    const double starts[] = {0.0, last, 40.0 * nd(g), 700.0 * (2.0 * u(g) - 1.0), 1e9, -1e9, NAN, INFINITY};
    for (double w : starts) {
      double o[3], slot = w;
      for (int again = 0; again < 2; ++again) {   // then from the root it left
        project(&slot, o);
        double d = 0.0, s = 1.0;
        for (int k = 0; k < 3; ++k) {
          d = std::max(d, std::fabs(o[k] - cold[k]));
          s = std::max(s, std::fabs(r[k]));
          if (!isfinite(o[k])) d = INFINITY;
        }
        worst = std::max(worst, d / s);
      }
      if (isfinite(slot)) last = slot;
    }
  }
  printf("%.3e\n", worst);
  return 0;
}
