// Host check of ring_start (common.hpp): a ring buffer begins on a line of its own
// inside an allocation that begins anywhere and holds RES_RING_ALIGN more.
#include <cstdio>
#include "common.hpp"
using namespace pdhcg;

int main() {
  alignas(256) static double mem[256];
  int bad = 0;
  for (int off = 0; off < 64; ++off)
    for (int need = 1; need <= 128; ++need) {
      double* p = mem + off;
      double* q = ring_start(p);
      bad += reinterpret_cast<uintptr_t>(q) % (RES_RING_ALIGN * sizeof(double)) != 0;
      bad += q < p || q + need > p + need + RES_RING_ALIGN;
    }
  printf("%d\n", bad);
  return 0;
}
