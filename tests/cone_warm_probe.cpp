// Host build of the device root-finders (cones.hpp) on one lane (a group of
// one needs no cross-lane step): projections from warm roots that are nearly
// right, as the slots of a converging solve are, against the projection in
// extended precision.  argv: mode, blocks, spread of the metric in a block.
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
// the hardware's reciprocal is approximate: 1e-8 relative here
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

typedef __float128 Q;
constexpr int N = 6;

struct Src {
  const double *rr, *mm;
  double r(int j) const { return rr[j]; }
  double m(int j) const { return mm[j]; }
};

static Q q_sqrt(Q x) {
  if (x <= 0) return 0;
  Q s = std::sqrt((double)x);
  for (int i = 0; i < 4; ++i) s = (s + x / s) / 2;
  return s;
}

// the metric projection onto ||v|| <= t by bisection of the secular equation
static void soc_exact(const Q* r, const Q* m, Q* out) {
  const int d = N - 1;
  Q a = 0, b = 0;
  for (int j = 0; j < d; ++j) {
    a += r[j] * r[j];
    b += m[j] * r[j] * m[j] * r[j];
  }
  const Q rt = r[d], mt = m[d];
  if (q_sqrt(a) <= rt) {
    for (int j = 0; j < N; ++j) out[j] = r[j];
    return;
  }
  if (q_sqrt(b) <= -mt * rt) {
    for (int j = 0; j < N; ++j) out[j] = 0;
    return;
  }
  const int sg = rt > 0 ? 1 : -1;
  const Q art = rt > 0 ? rt : -rt;
  auto psi = [&](Q del) {
    Q s = 0;
    for (int j = 0; j < d; ++j) {
      const Q v = m[j] * r[j] / (m[j] + mt - sg * del);
      s += v * v;
    }
    return del * q_sqrt(s) - mt * art;
  };
  Q lo = 0, hi = mt;
  if (sg < 0)
    while (psi(hi) < 0) hi *= 2;
  for (int i = 0; i < 220; ++i) {
    const Q mid = (lo + hi) / 2;
    if (psi(mid) < 0) lo = mid;
    else hi = mid;
  }
  const Q del = (lo + hi) / 2;
  for (int j = 0; j < d; ++j) out[j] = m[j] * r[j] / (m[j] + mt - sg * del);
  out[d] = mt * art / del;
}

static void rsoc_exact(const Q* r, const Q* m, Q* out) {
  const Q ms = q_sqrt(m[N - 2]), mt = q_sqrt(m[N - 1]), q = ms * mt, sq = q_sqrt(q), h = q_sqrt(Q(0.5));
  Q rr[N], mm[N], o[N];
  for (int j = 0; j < N - 2; ++j) {
    rr[j] = sq * r[j];
    mm[j] = m[j] / q;
  }
  rr[N - 2] = (ms * r[N - 2] - mt * r[N - 1]) * h;
  rr[N - 1] = (ms * r[N - 2] + mt * r[N - 1]) * h;
  mm[N - 2] = mm[N - 1] = 1;
  soc_exact(rr, mm, o);
  for (int j = 0; j < N - 2; ++j) out[j] = o[j] / sq;
  out[N - 2] = (o[N - 1] + o[N - 2]) * h / ms;
  out[N - 1] = (o[N - 1] - o[N - 2]) * h / mt;
}

static void project(int type, const double* r, const double* m, double* warm, double* out) {
  pdhcg::project_wave_item(type, N, false, Src{r, m}, [&](int j, double v) { out[j] = v; }, warm, 1);
}

static double error(int type, const double* r, const double* m, const double* o) {
  Q rq[N], mq[N], ex[N];
  for (int j = 0; j < N; ++j) {
    rq[j] = r[j];
    mq[j] = m[j];
  }
  if (type == 2) soc_exact(rq, mq, ex);
  else rsoc_exact(rq, mq, ex);
  double d = 0.0, s = 0.0;
  for (int j = 0; j < N; ++j) {
    d = std::max(d, std::fabs((double)(o[j] - ex[j])));
    s = std::max(s, std::fabs(r[j]));
    if (!isfinite(o[j])) d = INFINITY;
  }
  return d / s;
}

int main(int argc, char** argv) {
  const char* mode = argv[1];
  const long count = atol(argv[2]);
  const double spread = atof(argv[3]);
  std::mt19937_64 g(7);
  std::normal_distribution<double> nd;
  std::uniform_real_distribution<double> u(0.0, 1.0);
  double worst = 0.0;
  for (long i = 0; i < count; ++i) {
    double r[N], m[N], o[N];
    for (int j = 0; j < N; ++j) {
      r[j] = nd(g) * std::pow(10.0, -2.0 * u(g));
      m[j] = std::pow(spread, u(g) - 0.5);
    }
    if (!strcmp(mode, "soc") || !strcmp(mode, "rsoc")) {
      // a root that is off by 3e-10 to 9e-10
      const int type = mode[0] == 's' ? 2 : 3;
      double slot = NAN;
      project(type, r, m, &slot, o);
      if (!isfinite(slot)) continue;
      project(type, r, m, &slot, o);
      slot *= 1.0 + (u(g) < 0.5 ? -1.0 : 1.0) * (3e-10 + 6e-10 * u(g));
      project(type, r, m, &slot, o);
      worst = std::max(worst, error(type, r, m, o));
    } else if (!strcmp(mode, "soc_path") || !strcmp(mode, "rsoc_path")) {
      // the slot carried along a geometrically converging sequence of points
      const int type = mode[0] == 's' ? 2 : 3;
      double d[N], rate = 0.3 + 0.6 * u(g), slot = NAN, f = 1.0;
      for (int j = 0; j < N; ++j) {
        d[j] = 0.1 * nd(g);
        m[j] = 1.0 + std::pow(spread, u(g));
      }
      for (int k = 0; k < 60; ++k, f *= rate) {
        double p[N];
        for (int j = 0; j < N; ++j) p[j] = r[j] + f * d[j];
        project(type, p, m, &slot, o);
        worst = std::max(worst, error(type, p, m, o));
      }
    } else {
      // EXP, POW: against the projection from the root itself
      const bool pw = !strcmp(mode, "pow");
      const double al = 0.1 + 0.8 * u(g);
      double slot = NAN, ref[3], again[3];
      auto run = [&](double* w, double* to) {
        if (pw) pdhcg::project_pow_body(r[0], r[1], r[2], al, m[0], m[1], m[2], to, w);
        else pdhcg::project_exp_body(r[0], r[1], r[2], m[0], m[1], m[2], to, w);
      };
      run(&slot, ref);
      if (!isfinite(slot)) continue;
      run(&slot, ref);
      slot += std::max(1.0, std::fabs(slot)) * (u(g) < 0.5 ? -1.0 : 1.0) * (3e-10 + 6e-10 * u(g));
      run(&slot, again);
      double e = 0.0, s = 0.0;
      for (int k = 0; k < 3; ++k) {
        e = std::max(e, std::fabs(again[k] - ref[k]));
        s = std::max(s, std::fabs(r[k]));
        if (!isfinite(again[k])) e = INFINITY;
      }
      worst = std::max(worst, e / s);
    }
  }
  printf("%.3e\n", worst);
  return 0;
}
