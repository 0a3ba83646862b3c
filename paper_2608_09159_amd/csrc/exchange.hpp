// What the workgroups of a grid exchange: stores that other workgroups read,
// and the all-reduce, which is also the grid's barrier.  Included after
// cones.hpp (wave_sum) and thread_here().
#pragma once
#include "common.hpp"

namespace pdhcg {

// ---------------------------------------------------------------------------
// Exchange between the workgroups of a grid.
//
// Data that other workgroups read -- the iterates x, y, u, w_x, w_y and the
// words of the all-reduce -- is written with agent-scope stores, which go
// through the XCD's L2 to memory, so a release needs only the wait for the
// thread's own stores and no write-back of the L2.  Everything else is read
// by the workgroup that wrote it alone.
// ---------------------------------------------------------------------------
template <bool WT>
__device__ __forceinline__ void put(double* p, double v) {
  if constexpr (WT)
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), (unsigned long long)__double_as_longlong(v),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else
    *p = v;
}

__device__ __forceinline__ void put_pair(unsigned long long* p, double v, unsigned ep) {
  __hip_atomic_store(p, ((unsigned long long)(unsigned)__double2hiint(v) << 32) | ep, __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(p + 1, ((unsigned long long)(unsigned)__double2loint(v) << 32) | ep, __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}

// one try: v is the pair's value when both words carry epoch ep
__device__ __forceinline__ bool get_pair(const unsigned long long* p, unsigned ep, double& v) {
  const unsigned long long a = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const unsigned long long b = __hip_atomic_load(p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  v = __hiloint2double((int)(a >> 32), (int)(b >> 32));
  return (unsigned)a == ep && (unsigned)b == ep;
}

// This thread's stores are done.  The wait is not a fence to the compiler, so
// nothing that touches memory may move across it: a store of an iterate that sank
// below it would be published by the all-reduce before it is in memory.
__device__ __forceinline__ void stores_done() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
  asm volatile("" ::: "memory");
}

struct GridTeam {
  Comm C;
  unsigned long long limit;
  int rank, size;
};

struct SoloTeam {
  int rank = 0, size = 1;
};

// Sum over the team of `ns` slots of L.mine (slot q's index slot_of(q)), the
// totals to *dst_of(q); also the team's barrier.  acq: what other workgroups
// stored before it may be read (as plain loads) after it.
//
// Grids: two trips through memory.  Every workgroup stores its partials as
// value/epoch pairs; slot q is summed in a fixed order by one wave of
// workgroup q mod G, which polls the G pairs themselves and stores the total;
// every workgroup polls the totals (one of COMM_COPIES copies, so that a line
// is polled by a quarter of the grid).  A total carries everyone's arrival,
// so no flag, no L2 write-back and no second read of the partials is needed:
// a barrier of 256 workgroups with 23 slots takes 3.4 us against 12.1 us for
// arrival flags, a release word, the fences and a read of all partials by
// every workgroup (1 slot: 2.3 against 6.6 us).  A workgroup overwrites its
// pairs only after it has read a total of the same slot and epoch, or has
// passed a later all-reduce, so a poll cannot miss its epoch.
//
// Waits are bounded: after `limit` ticks of the constant-rate wall clock the
// abort word is set and the workgroup leaves the kernel, and the others
// follow.  A sum that lacks a partial is not stored, so no workgroup can take
// it for a total.  Others may still end their launch normally (the wait that
// failed may have been for a total on its way), so the host takes a launch
// with a raised abort word for aborted whatever its status says
// (launch_status).
template <class LdsT, class SlotFn, class DstFn>
__device__ __forceinline__ bool allreduce(const GridTeam& T, LdsT& L, int ns, SlotFn slot_of, DstFn dst_of,
                                          bool acq) {
  const int tid = thread_here(), lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = T.size, me = T.rank;
  stores_done();
  if (tid == 0) {
    L.epoch += 1u;
    L.flag = 0;
  }
  __syncthreads();
  const unsigned ep = L.epoch;
  const unsigned long long t0 = wall_clock64();
  bool ok = true;
  if (tid < ns) {
    const int s = slot_of(tid);
    put_pair(T.C.in + ((size_t)s * G + me) * 2, L.mine[s], ep);
  }
  for (int q = me + G * wv; q < ns; q += G * NWAVE) {
    const int s = slot_of(q);
    const unsigned long long* in = T.C.in + (size_t)s * G * 2;
    double sum = 0.0;
    for (int w0 = 0; w0 < G && ok; w0 += 256) {
      double v[4] = {0.0, 0.0, 0.0, 0.0};
      while (true) {
        bool all = true;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int w = w0 + 64 * t + lane;
          if (w < G) all = get_pair(in + (size_t)w * 2, ep, v[t]) && all;
        }
        if (__all(all)) break;
        if (wall_clock64() - t0 > T.limit) {
          ok = false;
          break;
        }
      }
      sum += (v[0] + v[1]) + (v[2] + v[3]);
    }
    if (!ok) break;
    sum = wave_sum(sum);
    if (lane < COMM_COPIES) put_pair(T.C.out + ((size_t)lane * SL_COUNT + s) * 2, sum, ep);
  }
  if (tid < ns) {
    const unsigned long long* out = T.C.out + ((size_t)(me & (COMM_COPIES - 1)) * SL_COUNT + slot_of(tid)) * 2;
    double v = 0.0;
    int n = 0;
    while (!get_pair(out, ep, v)) {
      if (wall_clock64() - t0 > T.limit) { ok = false; break; }
      if ((++n & 255) == 0 && __hip_atomic_load(T.C.abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
        ok = false;
        break;
      }
    }
    *dst_of(tid) = v;
  }
  if (!ok) {
    __hip_atomic_store(T.C.abort, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    L.flag = 1;
  }
  if (acq && tid == 0) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  __syncthreads();
  return L.flag == 0;
}

// what other workgroups stored before the last all-reduce may be read after it
__device__ __forceinline__ void acquire(const GridTeam&) {
  if (threadIdx.x == 0) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  __syncthreads();
}
__device__ __forceinline__ void acquire(const SoloTeam&) {}

template <class LdsT, class SlotFn, class DstFn>
__device__ __forceinline__ bool allreduce(const SoloTeam&, LdsT& L, int ns, SlotFn slot_of, DstFn dst_of, bool) {
  const int tid = thread_here();
  __syncthreads();
  if (tid < ns) *dst_of(tid) = L.mine[slot_of(tid)];
  __syncthreads();
  return true;
}

}  // namespace pdhcg
