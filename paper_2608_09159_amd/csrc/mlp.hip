// Kernels of the warm-start network: a ReLU MLP trained and evaluated with
// BF16 matrix operands on the gfx950 matrix cores (FP32 accumulation), FP32
// master weights and Adam.
//
// GEMM: C[M x N] = op(A)[M x K] * op(B)[K x N], all matrices row-major.
//   A: M x K (TA = false) or stored K x M (TA = true, used transposed)
//   B: K x N (TB = false) or stored N x K (TB = true, used transposed)
// The sum over K is cut into chunks (chunk_k below): a chunk is one chain of
// v_mfma_f32_32x32x16_bf16 from zero, and the chunks' sums are added in order
// to zero.  Three kernels form the same sums:
//   gemm_kernel<128>  tiles of 128 x 128 staged in LDS, one chunk: large M x N,
//                     or long chunks
//   gemm_kernel<64>   several chunks one after another, tiles of 64 x 64 (and
//                     one chunk where tiles of 128 leave the chip idle)
//   gemm_rows_kernel  a chunk per wave, tiles of 32 x 32, fragments straight
//                     from memory: few tiles and long K, or up to 32 rows
// so the chunks travel through memory only where that is the cheapest way (few
// tiles, long K): then they are spread over workgroups and added by a second
// kernel.  (As partial tiles they were 20 to 44 MB a product.)
//
// In the staged kernels each of the four waves owns a quarter of the tile;
// both operand tiles are staged with K contiguous (row stride padded by 8
// elements), so every lane reads its 8-element fragment with one 16-byte LDS
// load; global loads are 4-element runs along the contiguous dimension.
//
// Bound by staging: a stage of 64 of K takes a tile of 128 about 2 us at three
// workgroups a CU, of which the matrix instructions are a quarter.  6000 x 6000
// at 256 rows: 60 us, 0.31 PFLOP/s.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "mlp.hpp"

namespace pdhcg {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int TK = 64, LDK = TK + 8;
constexpr int GT = 256;   // threads per staged GEMM workgroup (4 waves, 2 x 2)
constexpr int RT = 32;    // tile of gemm_rows_kernel
constexpr int CUS = 256;      // compute units
constexpr int VW = 4;     // elements per vector load (8 bytes)

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
// vectors at addresses that are a multiple of four bytes only
typedef bf16x4 __attribute__((aligned(4))) bf16x4_a4;
typedef bf16x8 __attribute__((aligned(4))) bf16x8_a4;

struct GemmArgs {
  const __bf16* A;
  const __bf16* B;
  long lda, ldb;
  int M, N, K;
  int kchunk;             // K range of one chunk (multiple of TK)
  int epi;
  bool vec_a, vec_b;      // vector loads (stage_load)
  const float* bias;      // EPI_BIAS_*
  const __bf16* mask;     // EPI_MASK_BF16: M x N, ld = N
  float* outf;            // FP32 output (ld = N) or partials [chunks][M][N]
  __bf16* outb;           // BF16 output (ld = N)
  int partial;            // 1: write the chunks' sums
  GradStep gs;            // EPI_GRAD
};

__device__ __forceinline__ float adam_update(float w, float g, float& m, float& v, const AdamStep& a) {
  const float mi = fmaf(a.omb1, g, a.b1 * m);   // written out: the same rounding wherever it is inlined
  const float vi = fmaf(a.omb2 * g, g, a.b2 * v);
  m = mi;
  v = vi;
  return w - a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
}

__device__ __forceinline__ void epilogue(const GemmArgs& g, int m, int n, float acc) {
  const size_t o = (size_t)m * g.N + n;
  switch (g.epi) {
    case EPI_BIAS_F32: g.outf[o] = acc + g.bias[n]; break;
    case EPI_BIAS_RELU_BF16: g.outb[o] = (__bf16)fmaxf(acc + g.bias[n], 0.0f); break;
    case EPI_MASK_BF16: g.outb[o] = (__bf16)((float)g.mask[o] > 0.0f ? acc : 0.0f); break;
    default: break;
  }
}

// LDS column of element (row r, k): the 8-element k groups of a row are
// XOR-permuted by (r / 16) so that both the staging writes and the
// fragment reads spread over the banks (2-way and 4-way, the minimum for
// 8- and 16-byte accesses of a wave)
__device__ __forceinline__ int kswz(int r, int k) {
  return ((((k >> 3) ^ (r >> 4)) & (TK / 8 - 1)) << 3) | (k & 7);
}

// one operand tile of R rows (m or n) x TK (k), staged through registers:
// k-contiguous storage (element (r, k) at P[r * ld + k]) as VW-runs of k;
// r-contiguous storage (element (r, k) at P[k * ld + r]) as 4 x 4 blocks,
// four runs of 4 rows transposed in registers into four runs of 4 k.
template <int T>
constexpr int NRUN = (T * TK / VW) / GT;   // runs of VW elements per thread
static_assert((64 / 4) * (TK / 4) / GT * 4 == NRUN<64>, "both staging forms use NRUN runs per thread");

// global -> registers: zero past kend, anything past rmax (those rows and
// columns of C are dropped).  A run's address is a scalar part and a 32-bit
// offset of the thread, clamped into the matrix only in the tiles and the stage
// at its edges: no branches around the loads, which were most of a stage's
// time, next to no address arithmetic, and registers for three workgroups of
// T = 128 a CU (with an address per run in registers, 203, two).
// VEC: the contiguous dimension and the leading dimension are even and at
// least 4, so a run of 4 is one load, at the matrix's last 4 elements where it
// would pass the end (by 2, or altogether).
template <int T, bool KCONTIG, bool VEC>
__device__ __forceinline__ void stage_load(bf16x4 (&x)[NRUN<T>], const __bf16* P, long ld, int r0, int rmax,
                                           int k0, int kend) {
  const __bf16 z = (__bf16)0.0f;
  constexpr int RUNS = TK / VW, RB = T / 4;
  constexpr int RSTEP = GT / RUNS, KSTEP = GT / RB * 4;   // rows (k) between a thread's runs
  constexpr unsigned ES = sizeof(__bf16);
  using Off = std::conditional_t<VEC, unsigned, size_t>;   // VEC: 64 lines within 32 bits (gemm_args)
  const unsigned t = threadIdx.x;
  const Off row = (Off)ld * ES;
  // this thread's run begins at `at` of the contiguous dimension, which ends at
  // `end`; it is loaded from `st`
  const int at = KCONTIG ? k0 + (int)(t % RUNS) * VW : r0 + (int)(t % RB) * VW, end = KCONTIG ? kend : rmax;
  const int st = min(at, end - (VEC ? VW : 1));
  const bool cut = KCONTIG ? k0 + TK > kend : r0 + T > rmax;   // some run passes the end (uniform)
  const unsigned n = t / (KCONTIG ? RUNS : RB) * (KCONTIG ? 1 : 4), so = (unsigned)st * ES;
  const auto run = [&](int line, unsigned n, auto clamp) {
    const char* p = reinterpret_cast<const char*>(P + line * ld) + ((Off)n * row + so);
    bf16x4 v;
    if constexpr (VEC) {
      v = *reinterpret_cast<const bf16x4_a4*>(p);
    } else {
#pragma unroll
      for (int j = 0; j < VW; ++j)
        v[j] = *reinterpret_cast<const __bf16*>(p + (clamp.value ? min(j, end - 1 - st) : j) * ES);
    }
    return v;
  };
  // line q of the thread: its scalar part, and how many lines there are
  const auto line = [&](int q) { return KCONTIG ? r0 + q * RSTEP : k0 + q / 4 * KSTEP + q % 4; };
  const int lines = KCONTIG ? rmax : kend;
  const bool inside = KCONTIG ? r0 + T <= rmax : k0 + TK <= kend;
  if (inside && (VEC || !cut)) {
#pragma unroll
    for (int q = 0; q < NRUN<T>; ++q) x[q] = run(line(q), n, std::false_type{});
  } else {
#pragma unroll
    for (int q = 0; q < NRUN<T>; ++q) {
      const int l = min(line(q), lines - 1);
      x[q] = run(l, min(n, (unsigned)(lines - 1 - l)), std::true_type{});
      if (!KCONTIG && line(q) + (int)n >= kend) x[q] = bf16x4{z, z, z, z};
    }
  }
  if (VEC && cut && (KCONTIG || end % VW != 0)) {
#pragma unroll
    for (int q = 0; q < NRUN<T>; ++q)
      x[q] = st == at ? x[q] : st + 2 == at ? bf16x4{x[q][2], x[q][3], z, z} : bf16x4{z, z, z, z};
  }
  if (!VEC && KCONTIG && cut) {
#pragma unroll
    for (int q = 0; q < NRUN<T>; ++q)
#pragma unroll
      for (int j = 0; j < VW; ++j) x[q][j] = at + j < kend ? x[q][j] : z;
  }
}

// registers -> S[row][k] (swizzled k groups)
template <int T, bool KCONTIG>
__device__ __forceinline__ void stage_store(__bf16 (*S)[LDK], const bf16x4 (&x)[NRUN<T>]) {
  const int tid = threadIdx.x;
  if (KCONTIG) {
    constexpr int RUNS = TK / VW;
#pragma unroll
    for (int q = 0; q < NRUN<T>; ++q) {
      const int v = tid + q * GT;
      const int r = v / RUNS, kq = (v % RUNS) * VW;
      *reinterpret_cast<bf16x4*>(&S[r][kswz(r, kq)]) = x[q];
    }
  } else {
    constexpr int RB = T / 4;
#pragma unroll
    for (int q = 0; q < NRUN<T> / 4; ++q) {
      const int b = tid + q * GT;
      const int rb = (b % RB) * 4, kb = (b / RB) * 4;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        *reinterpret_cast<bf16x4*>(&S[rb + j][kswz(rb + j, kb)]) =
            bf16x4{x[4 * q][j], x[4 * q + 1][j], x[4 * q + 2][j], x[4 * q + 3][j]};
    }
  }
}

// a barrier for LDS alone: loads from memory stay in flight across it
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Tiles of T x T.  T = 64 where K has several chunks: half the tile in each
// direction, so that a chunk's sums and their total both stay in registers and
// a product of a few thousand columns covers the chip (512 x 5450 x 256: 688
// workgroups, 172 with T = 128).
// EPI_GRAD (C = dW): the workgroups of the first tile row add up the columns of
// B (the bias gradient) from the staged tiles, in row order, and the Adam step
// is taken where the gradient is: dW, W, m and v pass through memory once
// (512 x 5450 x 256: 24 us, bound by those 84 MB; 57 us in five kernels).
// VA, VB: vector loads of A and B (stage_load).
template <int T, bool TA, bool TB, bool VA, bool VB>
__global__ __launch_bounds__(GT, 3) void gemm_kernel(GemmArgs g) {
  constexpr bool CHUNKS = T == 64;
  constexpr int NB = T / 64;        // 32 x 32 blocks per wave and direction
  __shared__ __attribute__((aligned(16))) __bf16 As[T][LDK];
  __shared__ __attribute__((aligned(16))) __bf16 Bs[T][LDK];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int m0 = blockIdx.y * T, n0 = blockIdx.x * T;
  const int wm = (wv >> 1) * (T / 2), wn = (wv & 1) * (T / 2);
  constexpr bool GRAD = TA;         // the one product with a transposed A
  const bool colsum = GRAD && blockIdx.y == 0 && tid < T;
  float db = 0.0f;
  f32x16 acc[NB][NB] = {}, tot[CHUNKS ? NB : 1][CHUNKS ? NB : 1] = {};
  // the next stage's global loads are in flight while this stage computes
  bf16x4 xa[NRUN<T>], xb[NRUN<T>];
  const int kb = CHUNKS ? 0 : blockIdx.z * g.kchunk, ke = CHUNKS ? g.K : min(g.K, kb + g.kchunk);
  stage_load<T, !TA, VA>(xa, g.A, g.lda, m0, g.M, kb, g.K);
  stage_load<T, TB, VB>(xb, g.B, g.ldb, n0, g.N, kb, g.K);
  int kend = g.kchunk;              // of the current chunk
#pragma unroll 1
  for (int k0 = kb; k0 < ke; k0 += TK) {
    stage_store<T, !TA>(As, xa);
    stage_store<T, TB>(Bs, xb);
    lds_barrier();
    if (k0 + TK < ke) {
      stage_load<T, !TA, VA>(xa, g.A, g.lda, m0, g.M, k0 + TK, g.K);
      stage_load<T, TB, VB>(xb, g.B, g.ldb, n0, g.N, k0 + TK, g.K);
    }
    // lane l holds row/col (l % 32), k (l / 32) * 8 + j of each 32 x 32 x 16 step
#pragma unroll
    for (int ks = 0; ks < TK; ks += 16) {
      bf16x8 a[NB], b[NB];
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const int ra = wm + 32 * i + (lane & 31), rb = wn + 32 * i + (lane & 31);
        a[i] = *reinterpret_cast<const bf16x8*>(&As[ra][kswz(ra, ks + (lane >> 5) * 8)]);
        b[i] = *reinterpret_cast<const bf16x8*>(&Bs[rb][kswz(rb, ks + (lane >> 5) * 8)]);
      }
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    if (colsum) {
#pragma unroll
      for (int k = 0; k < TK; k += 8) {
        const bf16x8 v = *reinterpret_cast<const bf16x8*>(&Bs[tid][kswz(tid, k)]);
#pragma unroll
        for (int j = 0; j < 8; ++j) db += (float)v[j];
      }
    }
    if (CHUNKS && (k0 + TK >= kend || k0 + TK >= g.K)) {
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            tot[i][j][e] += acc[i][j][e];
            acc[i][j][e] = 0.0f;
          }
      kend += g.kchunk;
    }
    lds_barrier();
  }
  // ---- output: acc[i][j][e] is row (e / 4) * 8 + (l / 32) * 4 + e % 4 of block
  // i, column l % 32 of block j
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const f32x16& c = CHUNKS ? tot[CHUNKS ? i : 0][CHUNKS ? j : 0] : acc[i][j];
      const int n = n0 + wn + 32 * j + (lane & 31);
      const int mb = m0 + wm + 32 * i + (lane >> 5) * 4;
      if (n >= g.N) continue;
      if (!GRAD) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int m = mb + (e >> 2) * 8 + (e & 3);
          if (m >= g.M) continue;
          if (!CHUNKS && g.partial) g.outf[((size_t)blockIdx.z * g.M + m) * g.N + n] = c[e];
          else epilogue(g, m, n, c[e]);
        }
      } else {
#pragma unroll
        for (int q = 0; q < 16; q += 8) {     // eight rows' loads in flight
          float w[8], m1[8], m2[8];
          if (g.gs.on) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const int m = min(mb + ((q + e) >> 2) * 8 + (e & 3), g.M - 1);
              const size_t o = (size_t)m * g.N + n;
              w[e] = g.gs.W[o];
              m1[e] = g.gs.mW[o];
              m2[e] = g.gs.vW[o];
            }
          }
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int m = mb + ((q + e) >> 2) * 8 + (e & 3);
            if (m >= g.M) continue;
            const size_t o = (size_t)m * g.N + n;
            g.outf[o] = c[q + e];
            if (g.gs.on) {
              const float wi = adam_update(w[e], c[q + e], m1[e], m2[e], g.gs.a);
              g.gs.W[o] = wi;
              g.gs.Wb[o] = (__bf16)wi;
              g.gs.mW[o] = m1[e];
              g.gs.vW[o] = m2[e];
            }
          }
        }
      }
    }
  if (colsum && n0 + tid < g.N) {
    const int n = n0 + tid;
    g.gs.db[n] = db;
    if (g.gs.on) {
      float m1 = g.gs.mb[n], m2 = g.gs.vb[n];
      g.gs.b[n] = adam_update(g.gs.b[n], db, m1, m2, g.gs.a);
      g.gs.mb[n] = m1;
      g.gs.vb[n] = m2;
    }
  }
}

// 8 consecutive elements along k of a row, zero past `lim`
__device__ __forceinline__ bf16x8 load_k8(const __bf16* src, int lim) {
  bf16x8 v;
#pragma unroll
  for (int j = 0; j < 8; ++j) v[j] = j < lim ? src[j] : (__bf16)0.0f;
  return v;
}

// C tile of 32 x 32 with a chunk of K per wave, W waves a round; the chunks'
// sums meet in LDS and are added in order.  The fragments are loaded in the
// layout of the matrix instruction straight from memory: each is used once by
// the workgroup, and the waves with U steps of loads each cover the latency,
// so staging them would add a barrier per 64 of K and save nothing.
// Rows and columns past the edge repeat the last one; their results are dropped.
// A row of B gives a tile 64 bytes, half a line, so neighbouring tiles run on
// one XCD (workgroups go to the eight XCDs in turn) and share it in the L2.
template <bool TB, int W>
__global__ __launch_bounds__(W * 64) void gemm_rows_kernel(GemmArgs g) {
  constexpr int E = RT * RT / (W * 64), U = W == 1 ? 8 : 4;
  __shared__ float part[W][RT * RT];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int bx = blockIdx.x, pair = bx & 15;
  const int m0 = blockIdx.y * RT;
  const int n0 = (bx - pair + 16 <= (int)gridDim.x ? bx - pair + (pair & 7) * 2 + (pair >> 3) : bx) * RT;
  const int chunks = (g.K + g.kchunk - 1) / g.kchunk;
  const __bf16* a_row = g.A + (size_t)min(m0 + (lane & 31), g.M - 1) * g.lda;
  const int bn = min(n0 + (lane & 31), g.N - 1);
  const __bf16* b_base = TB ? g.B + (size_t)bn * g.ldb : g.B + bn;
  const int kl = (lane >> 5) * 8;
  float tot[E] = {};
  for (int c0 = blockIdx.z * W; c0 < chunks; c0 += gridDim.z * W) {
    const int c = c0 + wv;
    f32x16 acc = {};
    if (c < chunks) {
      const int ke = min(g.K, (c + 1) * g.kchunk);
      int k0 = c * g.kchunk;
      bf16x8 a[U], b[U];
      const bool vec = g.vec_a && (!TB || g.vec_b);
      for (; vec && k0 + 16 * U <= ke; k0 += 16 * U) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int k = k0 + 16 * u + kl;
          a[u] = *reinterpret_cast<const bf16x8_a4*>(a_row + k);
          if (!TB) {
#pragma unroll
            for (int j = 0; j < 8; ++j) b[u][j] = b_base[(size_t)(k + j) * g.ldb];
          } else {
            b[u] = *reinterpret_cast<const bf16x8_a4*>(b_base + k);
          }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[u], b[u], acc, 0, 0, 0);
      }
      for (; k0 < ke; k0 += 16) {
        const int k = k0 + kl, lim = ke - k;
        a[0] = load_k8(a_row + k, lim);
        if (TB) {
          b[0] = load_k8(b_base + k, lim);
        } else {
#pragma unroll
          for (int j = 0; j < 8; ++j) b[0][j] = j < lim ? b_base[(size_t)(k + j) * g.ldb] : (__bf16)0.0f;
        }
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[0], acc, 0, 0, 0);
      }
    }
#pragma unroll
    for (int e = 0; e < 16; ++e)
      part[wv][((e >> 2) * 8 + (lane >> 5) * 4 + (e & 3)) * RT + (lane & 31)] = acc[e];
    __syncthreads();
    if (g.partial) {
      for (int j = 0; j < min(W, chunks - c0); ++j)
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const int o = tid + e * W * 64, m = m0 + o / RT, n = n0 + o % RT;
          if (m < g.M && n < g.N) g.outf[((size_t)(c0 + j) * g.M + m) * g.N + n] = part[j][o];
        }
    } else {
      for (int j = 0; j < min(W, chunks - c0); ++j)
#pragma unroll
        for (int e = 0; e < E; ++e) tot[e] += part[j][tid + e * W * 64];
    }
    __syncthreads();
  }
  if (g.partial) return;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int o = tid + e * W * 64, m = m0 + o / RT, n = n0 + o % RT;
    if (m < g.M && n < g.N) epilogue(g, m, n, tot[e]);
  }
}

// the chunks' sums added in order, then the epilogue; 16 loads in flight and
// one wave a workgroup, since there are few outputs and many chunks (512
// outputs of 114 chunks: 27 us with one load at a time on two workgroups)
__global__ __launch_bounds__(64) void chunk_sum_kernel(GemmArgs g, const float* part, int chunks) {
  const long total = (long)g.M * g.N, o = (long)blockIdx.x * 64 + threadIdx.x;
  if (o >= total) return;
  float s = 0.0f;
  int z = 0;
  for (; z + 16 <= chunks; z += 16) {
    float v[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = part[(size_t)(z + j) * total + o];
#pragma unroll
    for (int j = 0; j < 16; ++j) s += v[j];
  }
  for (; z < chunks; ++z) s += part[(size_t)z * total + o];
  epilogue(g, (int)(o / g.N), (int)(o % g.N), s);
}

__global__ __launch_bounds__(256) void to_bf16_kernel(const float* x, __bf16* y, long n) {
  for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long)gridDim.x * 256) y[i] = (__bf16)x[i];
}

// dZ = bf16(scale * (yhat - y)); per-block partial of sum (yhat - y)^2 in FP64
__global__ __launch_bounds__(256) void mse_grad_kernel(const float* yhat, const float* y, __bf16* dz, long n,
                                                      float scale, double* part) {
  __shared__ double red[4];
  double s = 0.0;
  for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long)gridDim.x * 256) {
    const float d = yhat[i] - y[i];
    dz[i] = (__bf16)(scale * d);
    s += (double)d * (double)d;
  }
  for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

__global__ __launch_bounds__(64) void sum_partials_kernel(const double* part, int np, double* out) {
  // lane-strided sums, then a fixed-order wave reduction (deterministic)
  double s = 0.0;
  for (int i = threadIdx.x; i < np; i += 64) s += part[i];
  for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o, 64);
  if (threadIdx.x == 0) out[0] = s;
}

int grid_for(long n, int per, int cap) {
  long g = (n + per - 1) / per;
  return (int)std::max<long>(1, std::min<long>(g, cap));
}

// The chunks of a product's sum over K: as many (a power of two, in steps of
// TK) as keep 128 x 128 tiles within three workgroups a CU and the chunks' sums
// within `work_floats`.  This is the definition of the sum: it fixes the order
// of the additions, whichever kernel carries them out.
int chunk_k(int M, int N, int K, size_t work_floats) {
  const int tiles = ((M + 127) / 128) * ((N + 127) / 128);
  const int ksteps = std::max(1, (K + TK - 1) / TK);
  int splits = 1;
  while (tiles * splits * 2 <= 768 && splits * 2 <= ksteps &&
         (size_t)(splits * 2) * (size_t)M * (size_t)N <= work_floats)
    splits *= 2;
  return (ksteps + splits - 1) / splits * TK;
}

GemmArgs gemm_args(const __bf16* A, bool ta, long lda, const __bf16* B, bool tb, long ldb, int M, int N, int K,
                   int epi, size_t work_floats) {
  const int ca = ta ? M : K, cb = tb ? K : N;   // contiguous dimensions
  GemmArgs g{};
  g.A = A;
  g.B = B;
  g.lda = lda;
  g.ldb = ldb;
  g.M = M;
  g.N = N;
  g.K = K;
  g.epi = epi;
  // up to 64 rows of the matrix within the 32-bit offsets of stage_load
  constexpr long LD_MAX = 1l << 25;
  g.vec_a = lda % 2 == 0 && lda <= LD_MAX && ca % 2 == 0 && ca >= VW;
  g.vec_b = ldb % 2 == 0 && ldb <= LD_MAX && cb % 2 == 0 && cb >= VW;
  g.kchunk = chunk_k(M, N, K, work_floats);
  return g;
}

template <bool TB>
void launch_rows(const GemmArgs& g, dim3 grid, int chunks, hipStream_t st) {
  if (chunks > 8) hipLaunchKernelGGL((gemm_rows_kernel<TB, 16>), grid, dim3(16 * 64), 0, st, g);
  else if (chunks > 1) hipLaunchKernelGGL((gemm_rows_kernel<TB, 8>), grid, dim3(8 * 64), 0, st, g);
  else hipLaunchKernelGGL((gemm_rows_kernel<TB, 1>), grid, dim3(64), 0, st, g);
}

// How to carry out a product of several chunks: a wave per chunk, staged
// tiles of 128 whose sums go through memory, or staged tiles of 64 with the
// chunks one after another.  The cost of each in microseconds: what the last
// workgroup takes for its part of K, or what the chip takes for all of them,
// and the passes over C.  The numbers are a fit to 2,200 products of 33 to
// 1,024 rows, K from 96 to 56,500 and N from 100 to 26,557, timed in all three
// ways with B in either layout; the choice is 1% above the best way on average
// (512 columns, K = 4800, 256 rows: 22 us in waves, 24 through memory, 85 in
// tiles of 64; 6000 columns, K = 6000: 158, 60, 107; 12800 columns, K = 512:
// 38, 33, 20).
//  - waves: rounds of 8 or 16 chunks a workgroup (one, and a pass more, where
//    they are spread); tiles of 32 read A and B four times as often as tiles of
//    128, and 64 bytes of a row of B at a time, which straddle lines unless
//    the rows begin on them; A in single elements takes five times as long
//  - staged: single elements take several loads where a run takes one
enum Way { WAY_ROWS, WAY_SPREAD, WAY_STAGED };
bool rows_spread(const GemmArgs& g, int chunks) {
  // fewer than 64 tiles of 32 x 32: the chunks go to several workgroups
  return chunks > 16 && (long)((g.N + RT - 1) / RT) * ((g.M + RT - 1) / RT) < 64;
}
Way cheapest(const GemmArgs& g, int chunks) {
  const double M = g.M, N = g.N, K = g.K, mn = M * N * 1e-6;
  const auto tiles = [&](int t) { return std::ceil(M / t) * std::ceil(N / t); };
  const bool vec = g.vec_a && g.vec_b, spread = rows_spread(g, chunks);
  const double rounds = spread ? 1.0 : std::ceil(chunks / (chunks > 8 ? 16.0 : 8.0));
  const double rows = 3.3 + 16.8e-3 * (g.vec_a ? 1.0 : 5.3) * g.kchunk * (1.0 + 1.65 * (rounds - 1.0)) +
                      13.2e-6 * (g.ldb % 64 == 0 ? 1.0 : 1.27) * tiles(RT) * K + 0.9 * mn +
                      (spread ? 1.9 + 1.2 * chunks * mn : 0.0);
  const double through = 10.0 + std::max(26.9e-3 * std::ceil(tiles(128) * chunks / (3.0 * CUS)) * g.kchunk,
                                         33.8e-6 * (vec ? 1.0 : 3.2) * tiles(128) * K) + 1.2 * chunks * mn;
  const double inside = 4.7 + (vec ? 1.0 : 2.0) * std::max(11.7e-3 * std::ceil(tiles(64) / (5.0 * CUS)) * K,
                                                           23.5e-6 * tiles(64) * K) + 0.8 * mn;
  return rows <= through && rows <= inside ? WAY_ROWS : through <= inside ? WAY_SPREAD : WAY_STAGED;
}

// Which tile: 64 x 64 for several chunks one after another.  One chunk: tiles
// of 128 read the operands half as often, three of them a CU; tiles of 64
// where those are too few, up to one and a half a CU (64 x 20000, 192 rows, 314
// tiles: 18 us in tiles of 128, 11 in tiles of 64; 512 x 31000, 160 rows, 486
// tiles: 29 and 38; 512 x 49000, 256 rows, 766 tiles: 40 and 63), and for up to
// 64 rows, unless K is long and one turn of the chip holds the tiles (2048 x
// 65000, 33 rows, 508 tiles: 72 and 84; 2048 x 100000, 782 tiles: 151 and 114).
// Single elements are staged at half the rate: tiles of 64 up to a tile on
// every fourth CU (512 x 26557, 128 rows, 208 tiles: 41 and 48).
template <bool TA, bool TB>
void launch_staged(const GemmArgs& g, int chunks, hipStream_t st) {
  const long t128 = (long)((g.N + 127) / 128) * ((g.M + 127) / 128);
  const bool small = t128 <= (g.vec_a && g.vec_b ? CUS + CUS / 2 : CUS / 4) || (g.M <= 64 && (g.K <= 1024 || t128 > 3 * CUS));
  const bool inside = !g.partial && (chunks > 1 || small);
  const int T = inside ? 64 : 128;
  const dim3 grid((g.N + T - 1) / T, (g.M + T - 1) / T, inside ? 1 : chunks);
  const auto launch = [&](auto va, auto vb) {
    constexpr bool VA = va.value, VB = vb.value;
    if (inside) hipLaunchKernelGGL((gemm_kernel<64, TA, TB, VA, VB>), grid, dim3(GT), 0, st, g);
    else hipLaunchKernelGGL((gemm_kernel<128, TA, TB, VA, VB>), grid, dim3(GT), 0, st, g);
  };
  using yes = std::true_type;
  using no = std::false_type;
  if (g.vec_a && g.vec_b) {
    launch(yes{}, yes{});
  } else if constexpr (TB) {
    launch(no{}, no{});   // both operands are stored along K
  } else {
    if (g.vec_a) launch(yes{}, no{});
    else if (g.vec_b) launch(no{}, yes{});
    else launch(no{}, no{});
  }
}

}  // namespace

hipError_t mlp_gemm(const __bf16* A, long lda, const __bf16* B, bool tb, long ldb, int M, int N, int K, int epi,
                    const float* bias, const __bf16* mask, float* outf, __bf16* outb, float* work,
                    size_t work_floats, hipStream_t st) {
  if (M <= 0 || N <= 0) return hipSuccess;
  GemmArgs g = gemm_args(A, false, lda, B, tb, ldb, M, N, K, epi, work_floats);
  g.bias = bias;
  g.mask = mask;
  g.outf = outf;
  g.outb = outb;
  const int chunks = (K + g.kchunk - 1) / g.kchunk;
  // up to 32 rows: a wave per chunk, since a staged tile would hold mostly
  // padding; several chunks: the cheapest of the three
  const Way way = M <= RT ? WAY_ROWS : chunks > 1 ? cheapest(g, chunks) : WAY_STAGED;
  const bool rows = way == WAY_ROWS;
  dim3 grid((N + RT - 1) / RT, (M + RT - 1) / RT);
  const bool spread = rows ? rows_spread(g, chunks) : way == WAY_SPREAD;
  GemmArgs p = g;
  if (spread) {
    p.partial = 1;
    p.outf = work;
  }
  if (rows && spread) {
    grid.z = (chunks + 7) / 8;
    if (tb) hipLaunchKernelGGL((gemm_rows_kernel<true, 8>), grid, dim3(8 * 64), 0, st, p);
    else hipLaunchKernelGGL((gemm_rows_kernel<false, 8>), grid, dim3(8 * 64), 0, st, p);
  } else if (rows) {
    if (tb) launch_rows<true>(g, grid, chunks, st);
    else launch_rows<false>(g, grid, chunks, st);
  } else {
    if (tb) launch_staged<false, true>(p, chunks, st);
    else launch_staged<false, false>(p, chunks, st);
  }
  if (spread)
    hipLaunchKernelGGL(chunk_sum_kernel, dim3((unsigned)(((long)M * N + 63) / 64)), dim3(64), 0, st, g, work, chunks);
  return hipGetLastError();
}

hipError_t mlp_grad(const __bf16* in, const __bf16* dz, int rows, int K, int N, float* dW, const GradStep& s,
                    size_t work_floats, hipStream_t st) {
  if (K <= 0 || N <= 0) return hipSuccess;
  GemmArgs g = gemm_args(in, true, K, dz, false, N, K, N, rows, EPI_GRAD, work_floats);
  g.outf = dW;
  g.gs = s;
  launch_staged<true, false>(g, (rows + g.kchunk - 1) / g.kchunk, st);
  return hipGetLastError();
}

hipError_t mlp_to_bf16(const float* x, __bf16* y, long n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(to_bf16_kernel, dim3(grid_for(n, 256, 4096)), dim3(256), 0, st, x, y, n);
  return hipGetLastError();
}

hipError_t mlp_mse_grad(const float* yhat, const float* y, __bf16* dz, long n, float scale, double* part,
                        double* loss, hipStream_t st) {
  const int grid = grid_for(n, 256, 1024);
  hipLaunchKernelGGL(mse_grad_kernel, dim3(grid), dim3(256), 0, st, yhat, y, dz, n, scale, part);
  hipLaunchKernelGGL(sum_partials_kernel, dim3(1), dim3(64), 0, st, part, grid, loss);
  return hipGetLastError();
}

}  // namespace pdhcg
