// Solver core for problems whose iterates fit in registers: thread t of a
// workgroup keeps coordinates c0 + t + 512 j (j < CPT) and rows
// r0 + t + 512 j (j < RPT) for the whole launch, and meets memory only for
// the matrices, the gathers and the sums.  The method is run_solver's (see
// solver.hip), pass by pass.
//
// At up to a thousand coordinates a workgroup every pass of run_solver is a
// chain of dependent loads of a few hundred nanoseconds each (row pointer,
// column, gather, state, state again), of spills, and of an L2 emptied by the
// acquire of every barrier.  Here a product is one streaming pass over the
// workgroup's nonzeros, all of a thread's gathers in flight at once, into an
// LDS buffer from which each row is summed; the state needs no loads; and
// between workgroups only the gathered vectors travel, through a ring of
// buffers: a buffer that no cache has held before needs no invalidation, so
// the L2 is invalidated once per turn of the ring and the matrices stay in it.
// Each workgroup's part of a ring buffer begins on a cache line of its own.
//
// Bound by latency: two to three products and three to six all-reduces an
// iteration, 2.5 to 3 us each, in sequence.  Whole solves, run_solver with a
// counting barrier and separate sums before, this core after: 200 coordinates
// and 256 iterations on one workgroup 10.0 to 5.6 ms; sparse Q, 20,011
// coordinates 3.6 to 1.8 ms; boxes and row bounds, 60,001 coordinates 5.7 to
// 2.5 ms; all cones with rank-10 Q, 100,000 coordinates 8.8 to 5.0 ms.
#pragma once

namespace pdhcg {

constexpr int RES_T = 8;        // nonzeros per thread and chunk of a product
static_assert(RES_T * BLOCK == RES_CHUNK_MAX, "");

struct LdsRes : Lds {
  // rows of A^T, P and A longer than RES_LONG: summed by a wave each
  int ls[3][RES_LMAX], le[3][RES_LMAX];
  unsigned short li[3][RES_LMAX];
  int ln[3];
};
static_assert(sizeof(LdsRes) <= RES_LDS_STATIC, "dynamic LDS budget");

// x read anew through the scalar cache: what the compiler cannot see to be
// loop-invariant it does not keep in registers across the whole solve
// (x: constant during the kernel)
template <class X>
__device__ __forceinline__ const X& fresh(const X& x) {
  typedef const __attribute__((address_space(4))) X* Cp;
  Cp p = (Cp)&x;
  asm volatile("" : "+s"(p));
  return *(const X*)p;
}

// A CSR slice of one workgroup.  Nonzero tid + 512 t is thread tid's in every
// product, so its first REG nonzeros stay in registers; later ones are
// streamed from the L2.
template <int REG>
struct ResMat {
  const int* col;
  const double* val;
  int nnz;
  int c[REG];
  double v[REG];
  __device__ __forceinline__ void load(const int* col_, const double* val_, int nnz_) {
    col = col_;
    val = val_;
    nnz = nnz_;
#pragma unroll
    for (int t = 0; t < REG; ++t) {
      const int k = (int)threadIdx.x + t * BLOCK;
      c[t] = k < nnz ? col[k] : 0;
      v[t] = k < nnz ? val[k] : 0.0;
    }
  }
};

// the sum of prod[s..e), eight at a time in a tree
__device__ __forceinline__ double res_row_sum(const double* prod, int s, int e) {
  double sum = 0.0;
  for (int k = s; k < e; k += 8) {
    double a[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) a[i] = prod[min(k + i, e - 1)];
#pragma unroll
    for (int i = 1; i < 8; ++i) a[i] = k + i < e ? a[i] : 0.0;
    sum += ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
  }
  return sum;
}

// out[j] = row (tid + 512 j) of M times src; row bounds st/en count from the
// slice's first nonzero; list q of L holds the long rows.  prod: `chunk`
// products; rs: one double per row.  What a product costs is its chain of
// latencies: the gather, two LDS passes, the longest row's sum.
template <int K, int REG>
__device__ __forceinline__ void res_spmv(const ResMat<REG>& M, const double* src, const int (&st)[K], const int (&en)[K],
                                         int nrows, LdsRes& L, int q, double* prod, double* rs, int chunk,
                                         double (&out)[K]) {
  const int tid = thread_here(), lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
#pragma unroll
  for (int j = 0; j < K; ++j) out[j] = 0.0;
  const int nlong = __builtin_amdgcn_readfirstlane(L.ln[q]);
  for (int cb = 0; cb < M.nnz; cb += chunk) {
    const int cn = min(chunk, M.nnz - cb);
    int c[RES_T];
    double v[RES_T];
#pragma unroll
    for (int t = 0; t < RES_T; ++t)
      if (t * BLOCK < cn) {
        if (t < REG && cb == 0) {
          c[t] = M.c[t];
          v[t] = M.v[t];
        } else {
          const int k = cb + min(tid + t * BLOCK, cn - 1);
          c[t] = M.col[k];
          v[t] = M.val[k];
        }
      }
#pragma unroll
    for (int t = 0; t < RES_T; ++t)
      if (t * BLOCK < cn) v[t] *= src[c[t]];
    lds_sync();                 // the readers of the last products are done
#pragma unroll
    for (int t = 0; t < RES_T; ++t)
      if (tid + t * BLOCK < cn) prod[tid + t * BLOCK] = v[t];
    lds_sync();
#pragma unroll
    for (int j = 0; j < K; ++j) {
      if (wv * 64 + j * BLOCK >= nrows) break;
      const int s = max(st[j], cb) - cb, e = min(en[j], cb + cn) - cb;
      if (en[j] - st[j] <= RES_LONG) out[j] += res_row_sum(prod, s, e);
    }
    for (int i = wv; i < nlong; i += NWAVE) {
      const int s = L.ls[q][i], a = max(s, cb) - cb, e = min(L.le[q][i], cb + cn) - cb;
      if (a >= e) continue;
      double sum = 0.0;
      for (int k = a + lane; k < e; k += 64) sum += prod[k];
      sum = wave_sum(sum);
      const int row = L.li[q][i];
      if (lane == 0) rs[row] = s >= cb ? sum : rs[row] + sum;
    }
  }
  if (nlong > 0) {
    lds_sync();
#pragma unroll
    for (int j = 0; j < K; ++j)
      if (en[j] - st[j] > RES_LONG) out[j] = rs[tid + j * BLOCK];
  }
}

// columns of R of the workgroup's coordinates, by local index: one type per
// address space (a pointer that may be either is read by flat loads, one at a
// time)
struct RLocal {
  const double* l;
  int nl;
  __device__ __forceinline__ double operator()(int k, int i) const { return l[k * nl + i]; }
};
struct RGlobal {
  const double* g;   // the workgroup's first column
  long n;
  __device__ __forceinline__ double operator()(int k, int i) const { return g[(size_t)k * n + i]; }
};

// R u (and R s) of the workgroup's coordinates into L.mine: a wave per sum,
// three at a time; u and s in LDS
template <class RT>
__device__ __forceinline__ void res_factor_sums(Lds& L, const RT& R, int r, const double* u, const double* s,
                                                int nl) {
  const int tid = thread_here(), lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nsum = s ? 2 * r : r;
  for (int q0 = wv; q0 < nsum; q0 += 3 * NWAVE) {
    int kk[3], off[3];
    double t[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      const int q = q0 + e * NWAVE < nsum ? q0 + e * NWAVE : q0;
      kk[e] = q >= r ? q - r : q;
      off[e] = q >= r ? (int)(s - u) : 0;
    }
#pragma unroll 2
    for (int i = lane; i < nl; i += 64)
#pragma unroll
      for (int e = 0; e < 3; ++e) t[e] += R(kk[e], i) * u[off[e] + i];
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      const int q = q0 + e * NWAVE;
      const double sum = wave_sum(t[e]);
      if (lane == 0 && q < nsum) L.mine[(q >= r ? (int)SL_HS0 : (int)SL_H0) + kk[e]] = sum;
    }
  }
}

// staged points and metric of the cone items (LDS, workgroup-local)
struct LocalSrc {
  const double* z;
  const double* mt;
  int o;
  __device__ double r(int j) const { return z[o + j]; }
  __device__ double m(int j) const { return mt[o + j]; }
};
struct LocalNegSrc {
  const double* z;
  int o;
  __device__ double r(int j) const { return -z[o + j]; }
  __device__ double m(int) const { return 1.0; }
};

// Q: which objectives the code covers (diagonal Q^ has no inner loop, and
// without that loop's vectors more of the matrix stays in registers)
enum : int { Q_DIAG = 0, Q_GENERAL, Q_ANY };

template <int CPT, int RPT, bool CONES, int Q, class Team>
__device__ __forceinline__ void run_resident(const Run& A, const DevProblem& P, const DevVec& V, Ctl* ctl,
                                             const Team& T, LdsRes& L, const Own& own, bool prof, double* dyn) {
  constexpr bool SOLO = std::is_same<Team, SoloTeam>::value;
  // lt: the thread's index, opaque anew in every iteration, so that the
  // addresses and masks formed from it are not kept in registers between uses
  const int tid = threadIdx.x, rank = T.rank;
  int lt = tid;
  const int wbase = __builtin_amdgcn_readfirstlane(tid & ~63);   // the wave's first thread
  const long n = P.n, m = P.m, c0 = own.c0, r0 = own.r0;
  const int nl = (int)(own.c1 - c0), ml = (int)(own.r1 - r0), r = Q == Q_DIAG ? 0 : P.r;
  const DevSettings& S = *A.S;
  // dynamic LDS (res_lds_bytes): products (R s between them), own iterate,
  // the rows' dual iterate (one workgroup), staged cone points and metric,
  // long-row sums, columns of R
  const int chunk = P.res_chunk;
  double* const prod = dyn;
  double* const ul = prod + (r > 0 && nl > chunk ? nl : chunk);
  double* const yl = ul + nl;
  double* const zl = yl + (SOLO ? ml : 0);
  double* const mt = zl + (CONES ? nl : 0);
  double* const rs = mt + (CONES ? nl : 0);
  double* const rl = rs + (nl > ml ? nl : ml);
  const bool r_lds = r > 0 && P.res_r_lds;
  if (r_lds)
    for (int e = tid; e < r * nl; e += BLOCK) rl[e] = P.R[(size_t)(e / nl) * n + c0 + e % nl];
  const RLocal RL{rl, nl};
  const RGlobal RG{P.R + c0, n};
  auto factor_sums = [&](const double* u, const double* w) __attribute__((always_inline)) {
    if (r_lds) res_factor_sums(L, RL, r, u, w, nl);
    else res_factor_sums(L, RG, r, u, w, nl);
  };
  for (int e = tid; e < r * r; e += BLOCK) L.Dl[e] = P.Dm[e];
  if (tid < 3) L.ln[tid] = 0;
  const Items IT = CONES ? cache_items(P, own.it, L) : own.it;
  const bool has_items = CONES && ((IT.w1 > IT.w0) || (IT.l1 > IT.l0));
  __syncthreads();

  const bool qdiag = Q == Q_DIAG || (Q == Q_ANY && P.q_diag != 0), pdiag = P.p_diag != 0, sparse_p = !qdiag && P.P_ptr && !pdiag;
  const bool fuse = !qdiag && !sparse_p;
  const bool jac = S.inner == PDHCG_INNER_JACOBI;
  const double rho = S.rho;
  const int cap = A.T->cap;

  // ---- own coordinates and rows
  double x[CPT], ax[CPT], u[CPT], v[CPT], up[CPT], gp[CPT], c[CPT], qd[CPT], pd[CPT], xlo[CPT], xhi[CPT];
  int ct[CPT], ts[CPT], te[CPT], ps[CPT], pe[CPT];
  double y[RPT], ay[RPT], Ax[RPT], Aa[RPT], wy[RPT], aw[RPT], b[RPT], lo[RPT], hi[RPT];
  int as[RPT], ae[RPT];
  const bool started = L.C.started != 0;
  const int64_t tb = nl > 0 ? P.AT_ptr[c0] : 0, ab = ml > 0 ? P.A_ptr[r0] : 0;
  const int64_t pb = sparse_p && nl > 0 ? P.P_ptr[c0] : 0;
  const int tn = nl > 0 ? (int)(P.AT_ptr[own.c1] - tb) : 0, an = ml > 0 ? (int)(P.A_ptr[own.r1] - ab) : 0;
  const int pn = sparse_p && nl > 0 ? (int)(P.P_ptr[own.c1] - pb) : 0;
  auto add_long = [&](int q, int i, int s, int e) {
    if (e - s > RES_LONG) {
      const int k = atomicAdd(&L.ln[q], 1);
      if (k < RES_LMAX) {
        L.ls[q][k] = s;
        L.le[q][k] = e;
        L.li[q][k] = (unsigned short)i;
      }
    }
  };
#pragma unroll
  for (int j = 0; j < CPT; ++j) {
    const int l = tid + j * BLOCK;
    const long i = c0 + l;
    x[j] = ax[j] = u[j] = v[j] = up[j] = gp[j] = c[j] = qd[j] = pd[j] = xlo[j] = xhi[j] = 0.0;
    ct[j] = CT_FREE;
    ts[j] = te[j] = ps[j] = pe[j] = 0;
    if (l < nl) {
      if (started) {
        x[j] = V.x[i];
        ax[j] = V.ax[i];
      } else {
        x[j] = V.zb[i];
      }
      c[j] = P.c[i];
      qd[j] = P.qd[i];
      if (pdiag) pd[j] = P.Pd[i];
      ct[j] = P.ctype[i];
      if (P.xlo) {
        xlo[j] = P.xlo[i];
        xhi[j] = P.xhi[i];
      }
      ts[j] = (int)(P.AT_ptr[i] - tb);
      te[j] = (int)(P.AT_ptr[i + 1] - tb);
      add_long(0, l, ts[j], te[j]);
      if (sparse_p) {
        ps[j] = (int)(P.P_ptr[i] - pb);
        pe[j] = (int)(P.P_ptr[i + 1] - pb);
        add_long(1, l, ps[j], pe[j]);
      }
    }
  }
#pragma unroll
  for (int j = 0; j < RPT; ++j) {
    const int l = tid + j * BLOCK;
    const long i = r0 + l;
    y[j] = ay[j] = Ax[j] = Aa[j] = wy[j] = aw[j] = b[j] = lo[j] = hi[j] = 0.0;
    as[j] = ae[j] = 0;
    if (l < ml) {
      y[j] = V.y[i];
      if (started) {
        ay[j] = V.ay[i];
        Ax[j] = V.Ax[i];
        Aa[j] = V.Aa[i];
      }
      b[j] = P.b[i];
      if (P.rlo) {
        lo[j] = P.rlo[i];
        hi[j] = P.rhi[i];
      }
      as[j] = (int)(P.A_ptr[i] - ab);
      ae[j] = (int)(P.A_ptr[i + 1] - ab);
      add_long(2, l, as[j], ae[j]);
    }
  }
  auto own_c = [&](int j) { return lt + j * BLOCK < nl; };
  auto own_r = [&](int j) { return lt + j * BLOCK < ml; };
  // whether the wave has any (uniform: a pass is as long as its instructions,
  // and most waves of a workgroup with few rows have none)
  auto wave_c = [&](int j) { return wbase + j * BLOCK < nl; };
  auto wave_r = [&](int j) { return wbase + j * BLOCK < ml; };
  auto eproj_j = [&](int j, double z) {
    return ct[j] == CT_NONNEG ? fmax(z, 0.0) : (ct[j] == CT_BOX ? fmin(fmax(z, xlo[j]), xhi[j]) : z);
  };
  const bool bounded = P.rlo != nullptr;   // two-sided rows (dual_candidate)

  // ---- what other workgroups gather: ring buffers (grids), LDS (one
  // workgroup).  need: a buffer is reused, so the next all-reduce acquires
  int rn = -1, rm = -1;
  bool need = false;
  const long pc = SOLO ? 0 : P.pad_c[rank], pr = SOLO ? 0 : P.pad_r[rank];
  auto next_n = [&]() {
    if constexpr (!SOLO) {
      rn = rn + 1 == V.nring ? 0 : rn + 1;
      need = need || rn == 0;
    }
  };
  auto next_m = [&]() {
    if constexpr (!SOLO) {
      rm = rm + 1 == V.nring ? 0 : rm + 1;
      need = need || rm == 0;
    }
  };
  auto give_n = [&](const double (&w)[CPT]) {
#pragma unroll
    for (int j = 0; j < CPT; ++j)
      if (own_c(j)) {
        if constexpr (!SOLO) put<true>(V.ring_n + rn * V.ld_n + pc + lt + j * BLOCK, w[j]);
        ul[lt + j * BLOCK] = w[j];
      }
  };
  auto give_m = [&](const double (&w)[RPT]) {
#pragma unroll
    for (int j = 0; j < RPT; ++j)
      if (own_r(j)) {
        if constexpr (SOLO) yl[lt + j * BLOCK] = w[j];
        else put<true>(V.ring_m + rm * V.ld_m + pr + lt + j * BLOCK, w[j]);
      }
  };
  auto local_n = [&](const double (&w)[CPT]) {
#pragma unroll
    for (int j = 0; j < CPT; ++j)
      if (own_c(j)) ul[lt + j * BLOCK] = w[j];
  };
  auto take = [&]() {
    const bool t = need;
    need = false;
    return t;
  };
  constexpr int REG = Q == Q_DIAG ? 4 : 2;   // as many as do not spill
  ResMat<REG> MT, MP, MA;
  MT.load((SOLO ? P.AT_col : P.AT_colx) + tb, P.AT_val + tb, tn);
  MA.load((SOLO ? P.A_col : P.A_colx) + ab, P.A_val + ab, an);
  if (sparse_p) MP.load((SOLO ? P.P_col : P.P_colx) + pb, P.P_val + pb, pn);
  else MP.load(nullptr, nullptr, 0);
  auto mul_at = [&](double (&o)[CPT]) __attribute__((always_inline)) {
    if constexpr (SOLO) res_spmv(MT, yl, ts, te, nl, L, 0, prod, rs, chunk, o);
    else res_spmv(MT, V.ring_m + rm * V.ld_m, ts, te, nl, L, 0, prod, rs, chunk, o);
  };
  auto mul_p = [&](double (&o)[CPT]) __attribute__((always_inline)) {
    if constexpr (SOLO) res_spmv(MP, ul, ps, pe, nl, L, 1, prod, rs, chunk, o);
    else res_spmv(MP, V.ring_n + rn * V.ld_n, ps, pe, nl, L, 1, prod, rs, chunk, o);
  };
  auto mul_a = [&](double (&o)[RPT]) __attribute__((always_inline)) {
    if constexpr (SOLO) res_spmv(MA, ul, as, ae, ml, L, 2, prod, rs, chunk, o);
    else res_spmv(MA, V.ring_n + rn * V.ld_n, as, ae, ml, L, 2, prod, rs, chunk, o);
  };

#define REDUCE_OR_EXIT(call)                   \
  do {                                         \
    const int _cat = L.pcat;                   \
    tmark(L, prof, PT_BAR);                    \
    const bool _ok = (call);                   \
    tmark(L, prof, _cat);                      \
    if (!_ok) {                                \
      if (rank == 0 && tid == 0) {             \
        L.C.status = PDHCG_ABORTED;            \
        *ctl = L.C;                            \
      }                                        \
      return;                                  \
    }                                          \
  } while (0)
  const long dbase = c0;
  // the staged points projected in place (metric mt, or Euclidean)
  auto project = [&](bool force) {
    if constexpr (CONES) {
      lds_sync();
      const int cat = L.pcat;
      tmark(L, prof, PT_PROJ);
      project_items<true, false, false, true>(P, IT, force, [&](long st) { return LocalSrc{zl, mt, (int)(st - c0)}; }, zl,
                          L.C.started ? V.warm : nullptr, nullptr, dbase);
      tmark(L, prof, cat);
    }
  };

  // ------------------------------------------------------------------ init
  if (!started) {
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      if (ct[j] != CT_CONE) x[j] = eproj_j(j, x[j]);
      else if (CONES) zl[lt + j * BLOCK] = x[j];
    }
    if (has_items) {
      project(true);
#pragma unroll
      for (int j = 0; j < CPT; ++j)
        if (ct[j] == CT_CONE) x[j] = zl[lt + j * BLOCK];
    }
  }
  next_n();
  give_n(x);
  next_m();
  give_m(y);
  if (!started) {
    if (r > 0) {
      lds_sync();
      factor_sums(ul, nullptr);
    }
    REDUCE_OR_EXIT(reduce_sh(T, L, 0, 0, r, L.C.hx, take()));
    mul_a(Ax);
#pragma unroll
    for (int j = 0; j < CPT; ++j) ax[j] = x[j];
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
      Aa[j] = Ax[j];
      ay[j] = y[j];
    }
    if (tid == 0) {
      L.C.started = 1;
      if (!L.C.resume) {
        L.C.omega = P.omega0;
        L.C.eps_in = S.eps_in0;
        L.C.ktot = 0;
        L.C.inner_total = 0;
        L.C.restarts = 0;
        L.C.pid_I = 0.0;
        L.C.e_prev = 0.0;
      }
      L.C.resume = 0;
      L.C.k = 0;
      L.C.E0 = L.C.Eprev = L.C.lastE = 0.0;
    }
    lds_sync();
  } else {
    REDUCE_OR_EXIT(reduce_sh(T, L, 0, 0, 0, nullptr, take()));
  }

  // Q^ w on own coordinates: w in registers, its gathered copy the last given
  auto mul_q = [&](const double (&w)[CPT], const double* h, double (&o)[CPT]) __attribute__((always_inline)) {
    if (qdiag) {
#pragma unroll
      for (int j = 0; j < CPT; ++j) if (wave_c(j)) o[j] = qd[j] * w[j];
      return;
    }
    if (sparse_p) {
      mul_p(o);
    } else {
#pragma unroll
      for (int j = 0; j < CPT; ++j) if (wave_c(j)) o[j] = pd[j] * w[j];
    }
    if (r > 0) {
      lds_sync();
      times_d(L, P, h);
      lds_sync();
#pragma unroll
      for (int j = 0; j < CPT; ++j)
        if (own_c(j)) {
          double d = 0.0;
          if (r_lds) {
#pragma unroll 4
            for (int k = 0; k < r; ++k) d += RL(k, lt + j * BLOCK) * L.ht[k];
          } else {
#pragma unroll 4
            for (int k = 0; k < r; ++k) d += RG(k, lt + j * BLOCK) * L.ht[k];
          }
          o[j] += d;
        }
    }
  };
  // the sums of a projected step u - w0 (and R u, R s) into L.mine
  auto step_sums = [&](const double (&w0)[CPT], const double (&mi)[CPT]) __attribute__((always_inline)) {
    double acc[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      if (!wave_c(j)) break;
      const double s = u[j] - w0[j];
      acc[0] += s * s;
      if (fuse) {
        acc[1] += s * (mi[j] * s);
        acc[2] += s * (pd[j] * s);
        if (r > 0 && own_c(j)) prod[lt + j * BLOCK] = s;
      }
    }
    give_n(u);
    const unsigned long long sl = slot_list(SL_DELTA2, SL_SJS, SL_SPS);
    block_store(L, acc, sl, fuse ? 3 : 1);
    if (r > 0) factor_sums(ul, fuse ? prod : nullptr);
  };

  double mi[CPT], im[CPT], itau = 0.0, isig = 0.0, omega_m = 0.0;   // a primal weight is positive
  while (L.C.ktot < A.stop_at && L.C.status == 0) {
    asm volatile("" : "+v"(lt));
    const double omega = L.C.omega;
    const double tau = P.eta / omega, sigma = P.eta * omega;
    const long long k = L.C.k;
    const long long kt1 = L.C.ktot + 1;
    const bool check = (k == 0) || (kt1 % S.check_every == 0) || (kt1 >= S.max_iter);
    const double eps_in = L.C.eps_in;
    const bool tracing = L.C.ktot < cap;
    const double alpha0 = jac ? 1.0 : 1.0 / (A.qmax + 1.0 / tau);
    // the metric and its inverse change with the primal weight alone
    if (omega != omega_m) {
      omega_m = omega;
      itau = 1.0 / tau;
      isig = 1.0 / sigma;
#pragma unroll
      for (int j = 0; j < CPT; ++j) {
        mi[j] = qdiag ? 1.0 + tau * qd[j] : (jac ? itau + qd[j] : 1.0);
        im[j] = 1.0 / mi[j];
      }
    }
    if (tracing) {
      const TraceBufs& TB = fresh(*A.T);
      const long kk = kt1 - 1;
#pragma unroll
      for (int j = 0; j < CPT; ++j)
        if (own_c(j)) TB.x[kk * n + c0 + lt + j * BLOCK] = x[j];
#pragma unroll
      for (int j = 0; j < RPT; ++j)
        if (own_r(j)) TB.y[kk * m + r0 + lt + j * BLOCK] = y[j];
    }
    // u[j] = projection of z[j]; cone coordinates go through the staged points
    auto step_to = [&](const double (&z)[CPT], bool force) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < CPT; ++j) {
        if (!wave_c(j)) break;
        if (ct[j] != CT_CONE) {
          u[j] = eproj_j(j, z[j]);
        } else if (CONES) {
          zl[lt + j * BLOCK] = z[j];
          mt[lt + j * BLOCK] = mi[j];
        }
      }
      if (has_items) {
        project(force);
#pragma unroll
        for (int j = 0; j < CPT; ++j)
          if (ct[j] == CT_CONE) u[j] = zl[lt + j * BLOCK];
      }
    };

    // -------------------------------------------------------------- P1
    tmark(L, prof, PT_P1);
    int jcount = 0;
    double t[CPT], z[CPT];
    mul_at(t);
    if (qdiag) {
#pragma unroll
      for (int j = 0; j < CPT; ++j) if (wave_c(j)) z[j] = quotient(x[j] + tau * t[j] - tau * c[j], mi[j], im[j]);
      step_to(z, false);
      next_n();
      give_n(u);
      REDUCE_OR_EXIT(reduce_sh(T, L, 0, 0, 0, nullptr, take()));
    } else {
      double q[CPT];
#pragma unroll
      for (int j = 0; j < CPT; ++j) if (wave_c(j)) v[j] = x[j] + tau * t[j];
      mul_q(x, L.C.hx, q);
#pragma unroll
      for (int j = 0; j < CPT; ++j) {
        if (!wave_c(j)) break;
        gp[j] = q[j] + c[j] + quotient(x[j] - v[j], tau, itau);
        up[j] = x[j];
        z[j] = x[j] - quotient(alpha0 * gp[j], mi[j], im[j]);
      }
      step_to(z, !jac);
      next_n();
      step_sums(up, mi);
      const unsigned long long sl_d = slot_list(SL_DELTA2);
      if (fuse) REDUCE_OR_EXIT(reduce_step(T, L, r, tau));
      else REDUCE_OR_EXIT(reduce_sh(T, L, sl_d, 1, r, L.hu, take()));
      jcount = 1;
      bool done = (S.fixed_inner <= 0) && (sqrt(L.scal[SL_DELTA2]) <= eps_in);
      const int jmax = S.fixed_inner > 0 ? S.fixed_inner : S.j_max;
      while (!done && jcount < jmax) {
        tmark(L, prof, PT_P3);
        double g[CPT], alpha;
        mul_q(u, L.hu, q);
#pragma unroll
        for (int j = 0; j < CPT; ++j) if (wave_c(j)) g[j] = q[j] + c[j] + quotient(u[j] - v[j], tau, itau);
        if (fuse) {
          const double den = L.scal[SL_SDG];
          alpha = den > 0.0 ? (jac ? L.scal[SL_SJS] : L.scal[SL_DELTA2]) / den : 1.0;
        } else {
          double acc[3] = {0.0, 0.0, 0.0};
#pragma unroll
          for (int j = 0; j < CPT; ++j) {
            if (!wave_c(j)) break;
            const double s = u[j] - up[j];
            acc[0] += s * (mi[j] * s);
            acc[1] += s * (g[j] - gp[j]);
            acc[2] += s * s;
            gp[j] = g[j];
          }
          const unsigned long long sl = slot_list(SL_SJS, SL_SDG, SL_SS);
          block_store(L, acc, sl, 3);
          REDUCE_OR_EXIT(reduce_sh(T, L, sl, 3, 0, nullptr, false));
          const double den = L.scal[SL_SDG];
          alpha = den > 0.0 ? (jac ? L.scal[SL_SJS] : L.scal[SL_SS]) / den : 1.0;
          next_n();
        }
        tmark(L, prof, PT_P4);
#pragma unroll
        for (int j = 0; j < CPT; ++j) {
          if (!wave_c(j)) break;
          z[j] = u[j] - quotient(alpha * g[j], mi[j], im[j]);
          up[j] = u[j];
        }
        step_to(z, !jac);
        step_sums(up, mi);
        if (fuse) REDUCE_OR_EXIT(reduce_step(T, L, r, tau));
        else REDUCE_OR_EXIT(reduce_sh(T, L, sl_d, 1, r, L.hu, take()));
        ++jcount;
        done = (S.fixed_inner <= 0) && (sqrt(L.scal[SL_DELTA2]) <= eps_in);
      }
      if (fuse && take()) acquire(T);
    }

    // -------------------------------------------------------------- P6
    tmark(L, prof, PT_P6);
    const double c1h = (double)(k + 1) / (double)(k + 2);
    const double c3h = 1.0 / (double)(k + 2);
    mul_a(aw);
    auto halpern = [&](double w, double z0, double a0) {
      return c1h * (2.0 * rho * w + (1.0 - 2.0 * rho) * z0) + c3h * a0;
    };
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
      if (!wave_r(j)) break;
      const long l = r0 + lt + j * BLOCK;
      if (!own_r(j)) continue;
      const double axb = 2.0 * aw[j] - Ax[j];
      if (bounded && lo[j] != hi[j]) {
        const double q = axb - quotient(y[j], sigma, isig);
        wy[j] = sigma * (fmin(fmax(q, lo[j]), hi[j]) - q);
      } else {
        wy[j] = y[j] + sigma * (b[j] - axb);
      }
      if (tracing) fresh(*A.T).wy[(kt1 - 1) * m + l] = wy[j];
      if (check) {
        const double dy = y[j] - wy[j];
        acc[0] += dy * dy;                               // SL_DY2
        acc[1] += (Ax[j] - aw[j]) * dy;                  // SL_ADXDY
        const DevProblem& F = fresh(P);
        const double rp = F.nu_b * row_residual<true>(F, l, aw[j]) / F.Sy[l];
        acc[2] += rp * rp;                               // SL_RP2
        acc[3] += row_dual_term<true>(F, l, wy[j]);      // SL_BY
        const double my = wy[j] - ay[j];
        acc[4] += my * my;                               // SL_MOVY2
      } else {
        y[j] = halpern(wy[j], y[j], ay[j]);
        Ax[j] = halpern(aw[j], Ax[j], Aa[j]);
      }
    }
    if (tracing) {
      const TraceBufs& TB = fresh(*A.T);
#pragma unroll
      for (int j = 0; j < CPT; ++j)
        if (own_c(j)) TB.wx[(kt1 - 1) * n + c0 + lt + j * BLOCK] = u[j];
    }
    if (check) {
#pragma unroll
      for (int j = 0; j < CPT; ++j) {
        const double dx = x[j] - u[j];
        acc[5] += dx * dx;                               // SL_DX2
        const double mx = u[j] - ax[j];
        acc[6] += mx * mx;                               // SL_MOVX2
        acc[7] += c[j] * u[j];                           // SL_CX
      }
      next_m();
      give_m(wy);
      const unsigned long long sl = slot_list(SL_DY2, SL_ADXDY, SL_RP2, SL_BY, SL_MOVY2, SL_DX2, SL_MOVX2, SL_CX);
      block_store(L, acc, sl, 8);
      REDUCE_OR_EXIT(reduce_sh(T, L, sl, 8, 0, nullptr, take()));
      if (tid == 0) {
        L.C.inner_total += jcount;
        L.C.ktot = kt1;
      }

      // -------------------------------------------------------- check
      tmark(L, prof, PT_CHECK);
      const DevProblem& F = fresh(P);
      {
        double q[CPT], ac[3] = {0.0, 0.0, 0.0};
        mul_at(t);
        mul_q(u, L.hu, q);
#pragma unroll
        for (int j = 0; j < CPT; ++j) {
          const long i = c0 + lt + j * BLOCK;
          if (!own_c(j)) continue;
          const double si = q[j] + c[j] - t[j];
          ac[0] += u[j] * q[j];                          // SL_XQX
          const double so = F.nu_c * F.Sx[i] * si;
          if (ct[j] == CT_FREE) {
            ac[1] += so * so;                            // SL_RD2
          } else if (ct[j] == CT_NONNEG) {
            const double d = fmax(-so, 0.0);
            ac[1] += d * d;
          } else if (ct[j] == CT_BOX) {
            const double d = so - box_dual_proj(xlo[j], xhi[j], so);
            ac[1] += d * d;
            const double lam = box_dual_proj(xlo[j], xhi[j], si);
            ac[2] += lam > 0.0 ? lam * xlo[j] : (lam < 0.0 ? lam * xhi[j] : 0.0);   // SL_BOXD
          } else if (CONES) {
            zl[lt + j * BLOCK] = si;
          }
        }
        if (has_items) {
          lds_sync();
          // fixed-middle EXP blocks: distance of the reduced cost to its set
          // and the set's support term (run_solver's dual_check)
          for (int it = IT.l0 + tid; it < IT.l1; it += BLOCK) {
            if (li_type(F, IT, it) != PDHCG_CONE_EXP1) continue;
            const long st = li_start(F, IT, it);
            const int o = (int)(st - c0);
            const double f = F.nu_c * F.Sx[st];
            const double sa = f * zl[o], sb = f * zl[o + 1], sc = f * zl[o + 2];
            const double la = fmin(sa, 0.0), lc = fmax(sc, 0.0);
            ac[1] += (sa - la) * (sa - la) + (sc - lc) * (sc - lc);
            const double term = la == 0.0 ? sb : (lc == 0.0 ? -INFINITY : sb + la * (log_call(-la / lc) - 1.0));
            ac[2] += term / (F.nu_b * F.nu_c);
          }
          lds_sync();
          project_items<true, false, false, true>(F, IT, true, [&](long st) { return LocalNegSrc{zl, (int)(st - c0)}; }, zl,
                              V.warm + (F.n_wave + F.n_lane), nullptr, dbase, true);
#pragma unroll
          for (int j = 0; j < CPT; ++j)
            if (ct[j] == CT_CONE) {
              const double f = F.nu_c * F.Sx[c0 + lt + j * BLOCK] * zl[lt + j * BLOCK];
              ac[1] += f * f;
            }
        }
        const unsigned long long sk = slot_list(SL_XQX, SL_RD2, SL_BOXD);
        block_store(L, ac, sk, 3);
        REDUCE_OR_EXIT(reduce_sh(T, L, sk, 3, 0, nullptr, false));
      }
      if (tid == 0) {
        double E;
        const bool rst = check_step<true>(F, A, L, k, kt1, omega, E);
        L.done = rst ? 1 : 0;
        if (tracing && rank == 0) {
          double* tr = fresh(*A.T).sc + (kt1 - 1) * 8;
          tr[0] = tau; tr[1] = sigma; tr[2] = omega; tr[3] = eps_in;
          tr[4] = jcount; tr[5] = rst ? 1.0 : 0.0; tr[6] = 1.0; tr[7] = E;
        }
      }
      lds_sync();
      const bool restart = L.done != 0;
      if (L.C.status != 0) break;
      tmark(L, prof, PT_HALP);
#pragma unroll
      for (int j = 0; j < RPT; ++j) {
        if (restart) {
          y[j] = ay[j] = wy[j];
          Ax[j] = Aa[j] = aw[j];
        } else {
          y[j] = halpern(wy[j], y[j], ay[j]);
          Ax[j] = halpern(aw[j], Ax[j], Aa[j]);
        }
      }
      if (restart) {
#pragma unroll
        for (int j = 0; j < CPT; ++j) x[j] = ax[j] = u[j];
        next_m();
        give_m(y);
        if (sparse_p) {
          next_n();
          give_n(x);
        }
        REDUCE_OR_EXIT(reduce_sh(T, L, 0, 0, 0, nullptr, take()));
        if (tid < r) L.C.hx[tid] = L.hu[tid];
        lds_sync();
        continue;
      }
    } else {
      if (tid == 0) {
        L.C.inner_total += jcount;
        L.C.ktot = kt1;
      }
    }
    // ---------------------------------------------------------- Halpern
    double mov = 0.0;
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      if (!wave_c(j)) break;
      const double xn = halpern(u[j], x[j], ax[j]);
      mov += (xn - x[j]) * (xn - x[j]);
      x[j] = xn;
    }
    next_m();
    give_m(y);
    if (sparse_p) {
      next_n();
      give_n(x);
    } else if (r > 0) {
      lds_sync();          // the A product has read the LDS iterate
      local_n(x);
    }
    const unsigned long long sl = slot_list(SL_XMOV2);
    block_store(L, &mov, sl, 1);
    if (r > 0) factor_sums(ul, nullptr);
    REDUCE_OR_EXIT(reduce_sh(T, L, sl, 1, r, L.C.hx, take()));
    if (tid == 0) {
      L.C.eps_in = fmin(L.C.eps_in, fmax(S.gamma_in * sqrt(L.scal[SL_XMOV2]) / tau, S.eps_min));
      L.C.k = k + 1;
      if (!check && tracing && rank == 0) {
        double* tr = fresh(*A.T).sc + (kt1 - 1) * 8;
        tr[0] = tau; tr[1] = sigma; tr[2] = omega; tr[3] = eps_in;
        tr[4] = jcount; tr[5] = 0.0; tr[6] = 0.0; tr[7] = 0.0;
      }
    }
    lds_sync();
  }

  // ---- the state of the next launch and the candidate
  const DevVec& W = fresh(V);
#pragma unroll
  for (int j = 0; j < CPT; ++j) {
    const long i = c0 + lt + j * BLOCK;
    if (!own_c(j)) continue;
    W.x[i] = x[j];
    W.ax[i] = ax[j];
    (qdiag ? W.wx : W.u)[i] = u[j];
  }
#pragma unroll
  for (int j = 0; j < RPT; ++j) {
    const long i = r0 + lt + j * BLOCK;
    if (!own_r(j)) continue;
    W.y[i] = y[j];
    W.ay[i] = ay[j];
    W.Ax[i] = Ax[j];
    W.Aa[i] = Aa[j];
    W.wy[i] = wy[j];
  }
#undef REDUCE_OR_EXIT
}

}  // namespace pdhcg
