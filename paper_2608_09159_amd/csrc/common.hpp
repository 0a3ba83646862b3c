// Internal structures shared by the host setup, the driver and the kernels.
#pragma once
#include <stdint.h>

#include "pdhcg.h"

namespace pdhcg {

constexpr int RMAX = 32;          // largest supported rank of the dense factor R
constexpr int MAX_BLOCK = 1024;

// per-coordinate kind used by elementwise passes
enum : uint8_t { CT_FREE = 0, CT_NONNEG = 1, CT_CONE = 2, CT_BOX = 3 };

// reduction slots (one double per workgroup, summed over the team)
enum Slot : int {
  SL_DELTA2 = 0,   // ||u_new - u||^2                (inner stop test)
  SL_SJS,          // <s, J s>                       (BB numerator)
  SL_SDG,          // <s, dg>                        (BB denominator)
  SL_SS,           // ||s||^2                        (Euclidean BB numerator)
  SL_DX2,          // ||x - w_x||^2                  (restart metric)
  SL_DY2,          // ||y - w_y||^2
  SL_ADXDY,        // <A(x - w_x), y - w_y>
  SL_XMOV2,        // ||x_new - x||^2                (inner tolerance)
  SL_RP2,          // ||A x - b||^2 (unscaled)
  SL_RD2,          // ||Pi_K(-s)||^2 (unscaled)
  SL_XQX,          // <x, Q x>   (scaled)
  SL_CX,           // <c, x>     (scaled)
  SL_BY,           // <b, y>     (scaled)
  SL_MOVX2,        // ||w_x - a_x||^2                (PID)
  SL_MOVY2,        // ||w_y - a_y||^2
  SL_NAN,          // count of non-finite values
  SL_SPS,          // <s, P s>, diagonal P          (one-sync inner step)
  SL_BOXD,         // sum(lambda+ l^x - lambda- u^x) over box coordinates (scaled)
  SL_H0,           // R u : RMAX slots
  SL_HS0 = SL_H0 + RMAX,   // R s : RMAX slots (one-sync inner step)
  SL_COUNT = SL_HS0 + RMAX
};

struct DevProblem {
  int n, m, r;
  int at_lanes, a_lanes;
  const int64_t* A_ptr;  const int* A_col;  const double* A_val;
  const int64_t* AT_ptr; const int* AT_col; const double* AT_val;
  const int64_t* P_ptr;  const int* P_col;  const double* P_val;  // nullable
  const double* Pd;      // diag(P^) when p_diag (P u is then Pd * u)
  int p_diag;
  const double* R;       // r x n row-major (scaled)
  // FP32 copies of the values of A, A^T, P, R (FP32 mode only; else null)
  const float* A_valf; const float* AT_valf; const float* P_valf; const float* Rf;
  const double* Dm;      // r x r (scaled)
  const double* b;       // m (scaled; the combined row bounds when rows are bounded)
  const double* rlo;     // m scaled row bounds (nullable: A x = b)
  const double* rhi;
  const double* xlo;     // n scaled box bounds (nullable: no box block)
  const double* xhi;
  int ext;               // row bounds, box or fixed-middle EXP blocks present, or the
                         // rescaled-cone mode: the kernel variant compiled with them
                         // (others leave them out)
  int resc;              // rescaled-cone mode: SOC/RSOC/EXP/POW block j is S_j K_j,
                         // S_j = diag(Sx on the block)
  const double* c;       // n (scaled)
  const double* qd;      // n diag(Q^)
  const double* Sx;      // n
  const double* Sy;      // m
  const uint8_t* ctype;  // n
  int n_wave, n_lane;
  const int* wave_start; const int* wave_dim; const uint8_t* wave_type;
  const uint8_t* wave_euclid;
  const int* lane_start; const uint8_t* lane_type; const double* lane_alpha;
  const uint8_t* lane_euclid;
  double nu_b, nu_c, norm_b, norm_c;   // norm_b, norm_c: ||b||, ||c|| of the original data
  double eta, omega0;
  int q_diag;            // Q^ diagonal (includes Q = 0): one metric projection per prox
  // ownership of workgroup w: coordinates [part_c[w], part_c[w+1]), rows
  // [part_r[w], part_r[w+1]), wave items [part_w[w], ...), lane items
  // [part_l[w], ...)
  const long* part_c;
  const long* part_r;
  const int* part_w;
  const int* part_l;
  // A^T rows of each workgroup grouped by length class (skewed row lengths
  // only; else null): at_perm[n], at_seg[(classes + 1) * G]
  const int* at_perm;
  const int* at_seg;
  // register-resident core: its form, products staged at a time, whether the
  // owned columns of R are staged; grids: column indices as positions in the
  // ring buffers, and where each workgroup's part of them starts
  int res, res_chunk, res_r_lds;
  const int *A_colx, *AT_colx, *P_colx;
  const long *pad_c, *pad_r;
  const unsigned short* part_lanes;  // per workgroup: lanes for A^T/P rows (up to
                                     // 512: the whole workgroup), A rows,
                                    // SOC/RSOC group width, pad
};

// the register-resident core (resident.hpp): which form runs a problem, and
// what its workgroups need of LDS
enum : int { RES_NONE = 0, RES_GRID1, RES_GRID2, RES_ONE };
constexpr int RES_LONG = 32;          // rows longer than this are summed by a wave
constexpr int RES_LMAX = 192;         // at most so many of them a workgroup and matrix
constexpr int RES_CHUNK_MAX = 4096;   // products staged at a time
constexpr int RES_LDS_STATIC = 32 * 1024;
constexpr size_t RES_LDS_DYN = 160 * 1024 - RES_LDS_STATIC;
constexpr int RES_RING_ALIGN = 32;    // doubles: a workgroup's part of a ring buffer starts a line
// the first such start in an allocation that holds RES_RING_ALIGN more than it needs
// (memory of a caller's allocator may begin anywhere)
inline double* ring_start(double* p) {
  const uintptr_t line = RES_RING_ALIGN * sizeof(double);
  return reinterpret_cast<double*>((reinterpret_cast<uintptr_t>(p) + line - 1) / line * line);
}

// coordinates and rows of one workgroup, rank of R (0: its columns stay in
// global memory), products staged; one: the whole problem on one workgroup
constexpr size_t res_lds_bytes(long nl, long ml, int r, bool r_lds, long chunk, bool cones, bool one) {
  const long prod = (r > 0 && nl > chunk) ? nl : chunk;
  return sizeof(double) * (size_t)(prod + nl + (one ? ml : 0) + (cones ? 2 * nl : 0) + (nl > ml ? nl : ml) +
                                   (r_lds ? (long)r * nl : 0));
}

struct DevVec {
  double *x, *y, *ax, *ay, *wx, *wy;
  double *Ax, *Aa, *Aw;          // A^ x, A^ a, A^ w_x (m)
  double *v, *u, *up, *g, *gp;   // inner-solve vectors (n)
  double *zb;                    // pre-projection buffer (n)
  double *s;                     // KKT dual slack (n)
  double *t1, *t2;               // SpMV results of the current pass (n)
  double *warm;                  // root-finding warm starts, 2 x (n_wave + n_lane)
  double *xb, *yb, *Axb;         // averaged scheme
  double *ring_n, *ring_m;       // register-resident grids: nring gather buffers of ld_n, ld_m
  long ld_n, ld_m;
  int nring;
};

struct DevSettings {
  double tol;
  long long max_iter;
  int check_every;
  int scheme;
  double rho;
  int avg_epoch;
  int inner;
  int fixed_inner;
  int j_max;
  double eps_in0, gamma_in, eps_min;
  double beta_s, beta_n, beta_a;
  double pid_beta_i, pid_kp, pid_ki, pid_kd;
  int trace_iters;
};

// scalar state persisted in device memory between launches
struct Ctl {
  double omega, eps_in, E0, Eprev, pid_I, e_prev;
  double rel_p, rel_d, rel_gap, pobj, dobj, lastE;
  long long k, ktot, inner_total, restarts;
  int status;       // 0 running, else PDHCG_* status
  int started;
  int resume;       // with started = 0: re-initialise from zb / y, keep counters
  unsigned epoch;   // grid all-reduces done on the handle's exchange words
  double hx[RMAX];  // R^ x of the current Halpern primal state
  double hxb[RMAX]; // R^ xbar (averaged scheme)
  unsigned long long pt[16];  // phase timers (wall-clock ticks, workgroup 0)
};

// phase-timer categories
enum : int { PT_INIT = 0, PT_P1, PT_P2, PT_P3, PT_P4, PT_P6, PT_CHECK, PT_HALP, PT_BAR,
             PT_PROJ, PT_WCALL, PT_NCALL, PT_COUNT };

struct TraceBufs {
  int cap;                       // 0 = off
  double *x, *y, *wx, *wy;       // cap*n, cap*m
  double *sc;                    // cap * 8 scalars
};

// what a launch on one problem leaves for the host: the scalar state, and on
// a line of its own the abort word of the grid
struct CtlBlock {
  Ctl c;
  alignas(128) int abort;   // a workgroup's wait ended without its data
};

// the status of a launch: no workgroup may have left it on its own
inline int launch_status(const CtlBlock& b) { return b.abort != 0 ? PDHCG_ABORTED : b.c.status; }

// what the workgroups of a grid exchange (one allocation): COMM_COPIES copies
// of one pair of words per slot for the totals, and one pair per slot and
// workgroup for its partial.  A pair carries the two halves of a double, each
// beside the epoch of the all-reduce that wrote it.
constexpr int COMM_COPIES = 4;
struct Comm {
  int* abort;                // CtlBlock::abort
  unsigned long long* in;    // [SL_COUNT][G][2]
  unsigned long long* out;   // [COMM_COPIES][SL_COUNT][2]
};

struct KArgs {
  DevProblem P;
  DevVec V;
  DevSettings S;
  Ctl* ctl;
  Comm comm;
  unsigned epoch;      // all-reduces done on these words before this launch
  TraceBufs T;
  long long stop_at;   // return to the host when ktot reaches this
  unsigned long long spin_limit;  // all-reduce wait bound, wall-clock ticks
  double qmax;         // max_i diag(Q^)_i (first Euclidean BB step)
  int lds_bytes;       // dynamic LDS per workgroup (R slice; 0 = none)
  int profile;         // accumulate phase timers in ctl->pt and ptimes
  unsigned long long* ptimes;   // [G][PT_COUNT] per-workgroup timers (profile)
};

// what one solver run reads besides the problem and its vectors
struct Run {
  const DevSettings* S;
  const TraceBufs* T;
  long long stop_at;             // return when ktot reaches this
  double qmax;                   // max_i diag(Q^)_i (first Euclidean BB step)
  unsigned long long deadline;   // wall-clock tick; 0 = none (checked at checks)
  void* lds;                     // dynamic LDS for the workgroup's slice of R (nullable)
  int lds_bytes;
};

// one instance of a batch: its problem, vectors, trace buffers and control
// block, solved by a single workgroup that owns every coordinate and row
struct InstDesc {
  DevProblem P;
  DevVec V;
  TraceBufs T;
  Ctl* ctl;
  double qmax;
  const double* x0;   // scaled warm start (nullable), copied into zb at reset
  const double* y0;   // scaled dual warm start (nullable)
  int la, lr, lg;     // lanes per row of A^T / P and of A, SOC/RSOC group width
  int n_warm;         // root warm-start slots (2 x (wave + lane items))
  const int* perm;    // caller index of each internal coordinate (nullable)
};

struct BatchArgs {
  const InstDesc* desc;
  int first, count;        // queue positions [first, count) of this launch
  const int* order;        // queue position -> instance (largest first)
  int* queue;              // positions taken (reset to 0 before a launch)
  DevSettings S;
  long long stop_at;       // per-instance iteration cap of this launch
  const unsigned long long* deadline;   // wall-clock tick of the whole batch, set at its reset (0: none)
  unsigned long long* ptimes;       // [grid][PT_COUNT] phase timers, nullable
};

}  // namespace pdhcg
