// Host build of the grid's all-reduce (exchange.hpp): workgroups of one thread,
// run one after another.  Thread 0 of a wave polls the partials of workgroups
// 0, 64, ...; the grid has 65, of which 0 (which adds up the slot) and 64 are
// run.  Prints one line per scenario:
//   returned by 0, returned by 64, total seen by 64, abort word, total stored
#include <cmath>
#include <cstdio>
#include <cstring>

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
static int __builtin_amdgcn_update_dpp(int, int, int, int, int, bool) { return 0; }   // the other lanes hold 0
static int __builtin_amdgcn_ds_swizzle(int, int) { return 0; }
static int __builtin_amdgcn_readlane(int v, int l) { return l == 0 ? v : 0; }
static int __builtin_amdgcn_readfirstlane(int v) { return v; }
static void __builtin_amdgcn_s_waitcnt(int) {}
static unsigned long long bits(double v) {
  unsigned long long b;
  std::memcpy(&b, &v, 8);
  return b;
}
static int __double2loint(double v) { return (int)(unsigned)bits(v); }
static int __double2hiint(double v) { return (int)(unsigned)(bits(v) >> 32); }
static double __hiloint2double(int h, int l) {
  const unsigned long long b = ((unsigned long long)(unsigned)h << 32) | (unsigned)l;
  double v;
  std::memcpy(&v, &b, 8);
  return v;
}
static long long __double_as_longlong(double v) { return (long long)bits(v); }
static unsigned atomicAdd(unsigned* p, unsigned v) { return (*p += v) - v; }
static unsigned long long ticks;
static unsigned long long wall_clock64() { return ++ticks; }
static bool __all(bool b) { return b; }
static void __syncthreads() {}
static void __builtin_amdgcn_fence(int, const char*) {}
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_store(p, v, order, scope) (*(p) = (v))
#define __hip_atomic_load(p, order, scope) (*(p))
#include "pdhcg.h"
#include "cones.hpp"
namespace pdhcg {
constexpr int BLOCK = 512, NWAVE = 8;
static int thread_here() { return 0; }
}  // namespace pdhcg
#include "exchange.hpp"
using namespace pdhcg;

constexpr int G = 65;
struct TestLds {
  unsigned epoch = 0;
  int flag = 0;
  double mine[SL_COUNT] = {};
};

struct Grid {
  unsigned long long in[SL_COUNT * G * 2] = {}, out[COMM_COPIES * SL_COUNT * 2] = {};
  CtlBlock ctl = {};
  TestLds L[G];
  double got[G] = {};
  bool run(int rank, double mine, unsigned long long limit) {
    Comm c{};
    c.abort = &ctl.abort;
    c.in = in;
    c.out = out;
    const GridTeam T{c, limit, rank, G};
    L[rank].mine[SL_DELTA2] = mine;
    return allreduce(T, L[rank], 1, [](int) { return (int)SL_DELTA2; }, [&](int) { return &got[rank]; }, true);
  }
  // a workgroup that has stored its partial and waits for the total
  void arrive(int rank, double mine, unsigned ep) { put_pair(in + ((size_t)SL_DELTA2 * G + rank) * 2, mine, ep); }
  bool stored(unsigned ep) {
    double v;
    return get_pair(out + (size_t)SL_DELTA2 * 2, ep, v);
  }
  void print(bool a, bool b) {
    printf("%d %d %g %d %d\n", a, b, got[64], ctl.abort, stored(1));
  }
};

int main() {
  {   // everyone arrives
    static Grid g;
    g.arrive(64, 5.0, 1);
    const bool a = g.run(0, 2.0, 1000000);
    const bool b = g.run(64, 5.0, 1000000);
    g.print(a, b);
  }
  {   // 0 gives up; 64 arrives afterwards, with a clock of its own
    static Grid g;
    const bool a = g.run(0, 2.0, 50);
    const bool b = g.run(64, 5.0, 1000000);
    g.print(a, b);
  }
  {   // the same after a good epoch, whose words are still there
    static Grid g;
    g.arrive(64, 5.0, 1);
    g.run(0, 2.0, 1000000);
    g.run(64, 5.0, 1000000);
    g.got[64] = 0.0;
    const bool a = g.run(0, 3.0, 50);
    const bool b = g.run(64, 6.0, 1000000);
    printf("%d %d %g %d %d\n", a, b, g.got[64], g.ctl.abort, g.stored(2));
  }
  {   // a launch that ended normally on workgroup 0 while another gave up
    CtlBlock b{};
    b.c.status = PDHCG_OPTIMAL;
    const int fine = launch_status(b);
    b.abort = 1;
    printf("%d %d\n", fine == PDHCG_OPTIMAL, launch_status(b) == PDHCG_ABORTED);
  }
  return 0;
}
