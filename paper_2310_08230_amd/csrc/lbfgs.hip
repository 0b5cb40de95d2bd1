// Quasi-Newton powered MMA (Sec. 4.1, Alg. 1; Appendix "Quasi-Newton
// Updates") on top of the Jacobi sweep of dual.hip.
//
// Vectors with one value per multiplier (the subgradient g, the history pairs
// s and y, the direction q / d) are five slot planes of n_free values: slot k
// of variable i (slots at or above the variable's row count are zero) at
// k * n_free + i, so every pass reads and
// writes whole planes coalesced.  What the row passes read and write (the
// direction, the row minimisers) is one value per cell: the last direction
// pass also scatters d to the cells, which up to seven row passes then read in
// order, and the history pass gathers the new g.  g and y only take the values 0/1 and -1/0/1 and
// are stored as bytes, so a history pair costs 5 reals and 5 bytes per
// variable.  In FP32 i counts in variable order (layout.hip), where the gathers
// are cheapest.  In FP64 i is canonical and the bounds' terms are added in one
// fixed order (bound_order): where the relaxation is tight the search compares
// sums that differ in their last bits only, and its steps should not hang on how
// the launch deals the rows.
//
// One iteration, as launched by the host loop below:
//  1. direction: 2h + 1 variable-major passes over the last h accepted pairs.
//     Each pass first sums the previous pass's per-block dot partials in a
//     fixed order (every block computes the same value, so no extra launch is
//     needed for the reduction), applies one step of the two-loop recursion
//     and emits the per-block partials of the next dot; the last pass removes
//     every variable's mean (dual-feasible direction).  Dots are FP64.
//  2. FindStepSize: K + 1 bound-only sweeps at lambda + gamma d, each followed
//     by a one-block kernel that sums the bound and takes the search decision
//     on the device; sweeps after the search has stopped exit at once.
//  3. the MMA sweep at lambda + step d (step = 0 unless a trial improved).
//  4. the subgradient sweep at the new lambda, which also yields its bound.
//  5. the history pass s = lambda_new - lambda_old, y = g_old - g_new with the
//     dots s^T y and y^T y, and a one-block kernel for the curvature test; its
//     verdict is the only value read back by the host per iteration.
#include <algorithm>
#include <cmath>
#include <vector>

#include "dm_internal.h"

namespace {

constexpr int VB = 256;      // threads per block of the variable-major passes
constexpr int VGRID = 1024;  // at most this many blocks, hence partials per dot

// state of the step-size search, on the device
struct QnState {
  double E_init;  // E(lambda) of the current iteration
  double E0;      // E(lambda^0)
  double dmin;    // Delta_min
  double gamma;   // trial step size of the next probe
  double gm, Em;  // best trial so far and its objective
  double step;    // step applied before the MMA update
  int32_t done;   // search finished (later probes skip)
  int32_t pad;
};

__device__ inline double bsum(double v, double* red) { return block_sum_256(v, red); }

// sum of n per-block partials in a fixed order; every block gets the same value
__device__ inline double sum_partials(const double* p, int n, double* red) { return sum_partials_256(p, n, red); }

// vectors hold five slot planes of n values: slot k of variable i at k n + i
template <typename R>
__device__ inline void load5(const R* __restrict__ a, int64_t i, int64_t n, double v[5]) {
#pragma unroll
  for (int k = 0; k < 5; ++k) v[k] = double(a[k * n + i]);
}

template <typename R>
__device__ inline void store5(R* __restrict__ a, int64_t i, int64_t n, const double v[5]) {
#pragma unroll
  for (int k = 0; k < 5; ++k) a[k * n + i] = R(v[k]);
}

__device__ inline void load5_u8(const uint8_t* __restrict__ a, int64_t i, int64_t n, double v[5]) {
#pragma unroll
  for (int k = 0; k < 5; ++k) v[k] = double(a[k * n + i]);
}

__device__ inline void load5_i8(const int8_t* __restrict__ a, int64_t i, int64_t n, double v[5]) {
#pragma unroll
  for (int k = 0; k < 5; ++k) v[k] = double(a[k * n + i]);
}

__device__ inline double dot5(const double a[5], const double b[5]) {
  return (((a[0] * b[0] + a[1] * b[1]) + a[2] * b[2]) + a[3] * b[3]) + a[4] * b[4];
}

// subtract the mean over the variable's d rows (slots 0 to d - 1; the others
// stay zero)
__device__ inline void project5(double v[5], int d) {
  double sum = 0.0;
  for (int k = 0; k < 5; ++k) sum += k < d ? v[k] : 0.0;
  const double mean = sum / double(d);
  for (int k = 0; k < 5; ++k) v[k] = k < d ? v[k] - mean : 0.0;
}

// ---------------------------------------------------------------- direction passes
// the used slots of d into the variable's cells
template <typename R>
__device__ inline void scatter5(const uint32_t* vpos, int64_t i, int64_t n, const double v[5], int d, R* cells) {
#pragma unroll
  for (int k = 0; k < 5; ++k)
    if (k < d) cells[vpos[k * n + i]] = R(v[k]);
}

// row minimisers of the cells into slot planes (zero in unused slots)
__global__ __launch_bounds__(VB) void k_qn_gather_g(const uint8_t* gcell, const uint32_t* vpos, const uint8_t* deg,
                                                    int64_t n, uint8_t* g8) {
  for (int64_t i = int64_t(blockIdx.x) * VB + threadIdx.x; i < n; i += int64_t(gridDim.x) * VB) {
    const int d = deg[i];
#pragma unroll
    for (int k = 0; k < 5; ++k) g8[k * n + i] = k < d ? gcell[vpos[k * n + i]] : 0;
  }
}

// h = 0: d = g minus its per-variable mean
template <typename R>
__global__ __launch_bounds__(VB) void k_qn_project_g(const uint8_t* g8, const uint8_t* deg, int64_t n, R* d,
                                                     const uint32_t* vpos, R* dcell) {
  for (int64_t i = int64_t(blockIdx.x) * VB + threadIdx.x; i < n; i += int64_t(gridDim.x) * VB) {
    double v[5];
    load5_u8(g8, i, n, v);
    project5(v, deg[i]);
    store5<R>(d, i, n, v);
    if (dcell) scatter5<R>(vpos, i, n, v, deg[i], dcell);
  }
}

// partials of s^T g (first dot of the first loop)
template <typename R>
__global__ __launch_bounds__(VB) void k_qn_first(const uint8_t* g8, const R* s, int64_t n, double* part_out) {
  __shared__ double red[4];
  double acc = 0.0;
  for (int64_t i = int64_t(blockIdx.x) * VB + threadIdx.x; i < n; i += int64_t(gridDim.x) * VB) {
    double gv[5], sv[5];
    load5_u8(g8, i, n, gv);
    load5<R>(s, i, n, sv);
    acc += dot5(sv, gv);
  }
  const double b = bsum(acc, red);
  if (threadIdx.x == 0) part_out[blockIdx.x] = b;
}

// first loop, pair j: alpha_j = rho_j s_j^T q (from the partials), q -= alpha_j
// y_j, then the partials of the next dot: s_{j-1}^T q, or y_oldest^T q after
// the last pair (for beta of the second loop)
template <typename R>
__global__ __launch_bounds__(VB) void k_qn_loop1(const uint8_t* g8, const R* q_in, const int8_t* y,
                                                 const R* s_next, const int8_t* y_next, const double* part_in,
                                                 int32_t n_in, const double* sy, double* alpha_out, int64_t n,
                                                 R* q_out, double* part_out) {
  __shared__ double red[4];
  const double alpha = sum_partials(part_in, n_in, red) / *sy;
  if (blockIdx.x == 0 && threadIdx.x == 0) *alpha_out = alpha;
  double acc = 0.0;
  for (int64_t i = int64_t(blockIdx.x) * VB + threadIdx.x; i < n; i += int64_t(gridDim.x) * VB) {
    double qv[5], yv[5], nv[5];
    if (g8) load5_u8(g8, i, n, qv);
    else load5<R>(q_in, i, n, qv);
    load5_i8(y, i, n, yv);
    for (int k = 0; k < 5; ++k) qv[k] = double(R(qv[k] - alpha * yv[k]));
    store5<R>(q_out, i, n, qv);
    if (s_next) load5<R>(s_next, i, n, nv);
    else load5_i8(y_next, i, n, nv);
    acc += dot5(nv, qv);
  }
  const double b = bsum(acc, red);
  if (threadIdx.x == 0) part_out[blockIdx.x] = b;
}

// second loop, pair j: beta = rho_j y_j^T q, q += (alpha_j - beta) s_j; the
// first pass scales q by H0 = s^T y / y^T y of the newest pair; then the
// partials of y_{j+1}^T q, or after the newest pair the projection of d
template <typename R>
__global__ __launch_bounds__(VB) void k_qn_loop2(const R* q_in, const R* s, const int8_t* y_next,
                                                 const double* part_in, int32_t n_in, const double* sy,
                                                 const double* alpha, const double* h0_sy, const double* h0_yy,
                                                 const uint8_t* deg, int64_t n, R* q_out, double* part_out,
                                                 const uint32_t* vpos, R* dcell) {
  __shared__ double red[4];
  const double h0 = h0_sy ? *h0_sy / *h0_yy : 1.0;
  const double beta = h0 * sum_partials(part_in, n_in, red) / *sy;
  const double coef = *alpha - beta;
  double acc = 0.0;
  for (int64_t i = int64_t(blockIdx.x) * VB + threadIdx.x; i < n; i += int64_t(gridDim.x) * VB) {
    double qv[5], sv[5];
    load5<R>(q_in, i, n, qv);
    load5<R>(s, i, n, sv);
    for (int k = 0; k < 5; ++k) qv[k] = h0 * qv[k] + coef * sv[k];
    if (y_next) {
      for (int k = 0; k < 5; ++k) qv[k] = double(R(qv[k]));
      double yv[5];
      load5_i8(y_next, i, n, yv);
      acc += dot5(yv, qv);
    } else {
      project5(qv, deg[i]);
      if (dcell) scatter5<R>(vpos, i, n, qv, deg[i], dcell);
    }
    store5<R>(q_out, i, n, qv);
  }
  if (y_next) {
    const double b = bsum(acc, red);
    if (threadIdx.x == 0) part_out[blockIdx.x] = b;
  }
}

// ---------------------------------------------------------------- history
// s + t / |J| in one rounding, as the row passes form it
template <typename R>
__device__ inline R restored(R s, R t, R rd) {
  if constexpr (sizeof(R) == 4) return __builtin_fmaf(t, rd, s);
  else return __builtin_fma(t, rd, s);
}

// s = lambda_new - lambda_old (both with feasibility restored exactly as the
// sweeps see them), y = g_old - g_new, and the partials of s^T y and y^T y; the
// new g comes from the cells and goes to its planes
template <typename R>
__global__ __launch_bounds__(VB) void k_qn_hist_pass(const R* cell_old, const R* t_old, const R* cell_new,
                                                     const R* t_new, const int32_t* vinv, const uint32_t* vpos,
                                                     const uint8_t* g_old, const uint8_t* gcell,
                                                     const uint8_t* deg, int64_t n, uint8_t* g_new, R* s_out,
                                                     int8_t* y_out, double* part_sy, double* part_yy) {
  __shared__ double red[4];
  double a_sy = 0.0, a_yy = 0.0;
  for (int64_t i = int64_t(blockIdx.x) * VB + threadIdx.x; i < n; i += int64_t(gridDim.x) * VB) {
    const int d = deg[i];
    const int64_t v = vinv ? int64_t(vinv[i]) : i;
    const R rd = R(1) / R(d), to = t_old[v], tn = t_new[v];
    uint32_t p[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) p[k] = vpos[k * n + i];
    R so[5], sn[5];
    double go[5], gn[5], sv[5], yv[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      so[k] = cell_old[p[k]];
      sn[k] = cell_new[p[k]];
      gn[k] = k < d ? double(gcell[p[k]]) : 0.0;
    }
    load5_u8(g_old, i, n, go);
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      sv[k] = k < d ? double(R(restored<R>(sn[k], tn, rd) - restored<R>(so[k], to, rd))) : 0.0;
      yv[k] = go[k] - gn[k];
      y_out[k * n + i] = int8_t(yv[k]);
      g_new[k * n + i] = uint8_t(gn[k]);
    }
    store5<R>(s_out, i, n, sv);
    a_sy += dot5(sv, yv);
    a_yy += dot5(yv, yv);
  }
  const double b_sy = bsum(a_sy, red);
  const double b_yy = bsum(a_yy, red);
  if (threadIdx.x == 0) {
    part_sy[blockIdx.x] = b_sy;
    part_yy[blockIdx.x] = b_yy;
  }
}

// partials of s^T y and y^T y of a given pair
template <typename R>
__global__ __launch_bounds__(VB) void k_qn_pair_dots(const R* s, const int8_t* y, int64_t n, double* part_sy,
                                                     double* part_yy) {
  __shared__ double red[4];
  double a_sy = 0.0, a_yy = 0.0;
  for (int64_t i = int64_t(blockIdx.x) * VB + threadIdx.x; i < n; i += int64_t(gridDim.x) * VB) {
    double sv[5], yv[5];
    load5<R>(s, i, n, sv);
    load5_i8(y, i, n, yv);
    a_sy += dot5(sv, yv);
    a_yy += dot5(yv, yv);
  }
  const double b_sy = bsum(a_sy, red);
  const double b_yy = bsum(a_yy, red);
  if (threadIdx.x == 0) {
    part_sy[blockIdx.x] = b_sy;
    part_yy[blockIdx.x] = b_yy;
  }
}

__global__ __launch_bounds__(1024) void k_qn_pair_fin(const double* part_sy, const double* part_yy, int32_t n,
                                                    double* sy, double* yy) {
  __shared__ double red[16];
  const double a = sum_partials_1024(part_sy, n, red);
  const double b = sum_partials_1024(part_yy, n, red);
  if (threadIdx.x == 0) {
    *sy = a;
    *yy = b;
  }
}

// ---------------------------------------------------------------- one-block decisions
// Sum of a sweep's bound: of the n block sums p, or (T.terms) of the terms in their
// own order.  Up to FOLD_BLOCKS blocks of terms one workgroup adds all; more are
// dealt out, four to a workgroup, and the last workgroup to arrive adds their sums
// (in index order, so it does not matter which).  Returns false in the others, which
// are done: whatever the launch changes, it changes after all have arrived.
// 320-face pair (12k rows, 100k entries), FP64, a call of six iterations: 996 us; with
// a launch of its own for the block sums, 39 a call, 1023 (and up to 1180 where the
// host is slower); with all of it in one workgroup 1078; with every thread
// fencing, not one, 1267.  At 4k rows one workgroup is as good.
constexpr int FOLD_BLOCKS = 32, FOLD_LONG = 1024;

inline unsigned sum_grid(const TermSums& T) {
  if (!T.terms || (T.n_blocks <= FOLD_BLOCKS && T.n_long_blocks <= FOLD_LONG)) return 1u;
  return unsigned(std::max((T.n_blocks + 3) / 4, (T.n_long_blocks + 1023) / 1024));
}

__device__ inline bool bound_sum(const TermSums& T, const double* p, int n, double* red, double* E) {
  __shared__ double part[FOLD_BLOCKS + FOLD_LONG];
  __shared__ double waves[4 * FOLD_BLOCKS];
  __shared__ bool last;
  if (!T.terms) {   // uniform across the grid
    *E = sum_partials_1024(p, n, red);
    return true;
  }
  constexpr int PER = FOLD_BLOCKS / 4;
  const int t = int(threadIdx.x);
  if (gridDim.x == 1) {
    double v[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) v[u] = 4 * u + t / 256 < T.n_blocks ? T.terms[u * 1024 + t] : 0.0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      if (4 * u >= T.n_blocks) break;   // uniform
      v[u] = wave_sum(v[u]);
      if ((t & 63) == 0) waves[u * 16 + t / 64] = v[u];
    }
    for (int q = t; q < T.n_long_blocks; q += 1024) part[T.n_blocks + q] = T.long_block(q);
    __syncthreads();
    if (t < T.n_blocks) part[t] = ((waves[4 * t] + waves[4 * t + 1]) + waves[4 * t + 2]) + waves[4 * t + 3];
    __syncthreads();
    *E = sum_partials_1024(part, T.n_blocks + T.n_long_blocks, red);
    return true;
  }
  const int b0 = 4 * int(blockIdx.x);
  const double v = wave_sum(b0 + t / 256 < T.n_blocks ? T.terms[size_t(b0) * 256 + t] : 0.0);
  if ((t & 63) == 0) waves[t / 64] = v;
  for (int q = int(blockIdx.x) * 1024 + t; q < T.n_long_blocks; q += int(gridDim.x) * 1024)
    T.part[T.n_blocks + q] = T.long_block(q);
  __syncthreads();
  if (t < 4 && b0 + t < T.n_blocks)
    T.part[b0 + t] = ((waves[4 * t] + waves[4 * t + 1]) + waves[4 * t + 2]) + waves[4 * t + 3];
  __syncthreads();   // the workgroup's sums are in its L2; one thread hands them on
  if (t == 0) {
    last = __hip_atomic_fetch_add(T.arrived, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1u;
    if (last) *T.arrived = 0u;   // for the next launch
  }
  __syncthreads();
  if (!last) return false;   // uniform
  *E = sum_partials_1024(T.part, T.n_blocks + T.n_long_blocks, red);
  return true;
}

// start of a call: the bound at the imported lambda; a fresh search also
// resets the step size and Delta_min (a resumed one keeps them)
__global__ __launch_bounds__(1024) void k_qn_begin(TermSums T, const double* sp, int32_t sn, double offset, QnState* st,
                                                 double* etrace, double gamma0, int32_t resume) {
  __shared__ double red[16];
  double E = 0.0;
  if (!bound_sum(T, sp, sn, red, &E)) return;   // uniform
  E += offset;
  if (threadIdx.x == 0) {
    etrace[0] = E;
    if (!resume) {
      st->E0 = E;
      st->dmin = INFINITY;
      st->gamma = gamma0;
      st->gm = gamma0;
    }
    st->E_init = E;
    st->Em = -INFINITY;
    st->step = 0.0;
    st->done = 0;
  }
}

// FindStepSize after probe t (t = 0: the previous step size; t = 1..K: the
// rescaled ones): keep the best trial, stop after a gain of Delta_min or at
// t = K, otherwise rescale gamma by the verdict of this trial against E(lambda)
__global__ __launch_bounds__(1024) void k_qn_probe(TermSums T, const double* sp, int32_t sn, double offset, int32_t t,
                                                 int32_t K,
                                                 double up, double down, QnState* st, double* gtrace,
                                                 int32_t* taken) {
  __shared__ double red[16];
  if (st->done) return;   // uniform across the grid
  double E = 0.0;
  if (!bound_sum(T, sp, sn, red, &E)) return;   // uniform
  E += offset;
  if (threadIdx.x != 0) return;
  if (t == 0 || E >= st->Em) {
    st->gm = st->gamma;
    st->Em = E;
  }
  const bool stop = t == K || (t > 0 && E - st->E_init >= st->dmin);
  if (stop) {
    const bool improve = st->Em > st->E_init;
    st->done = 1;
    st->step = improve ? st->gm : 0.0;
    st->gamma = st->gm;
    if (gtrace) *gtrace = st->gm;
    if (taken) *taken = improve ? 1 : 0;
  } else {
    st->gamma = (E <= st->E_init) ? down * st->gamma : up * st->gamma;
  }
}

// after the subgradient sweep at lambda_{k+1} and the history pass: the bound
// E(lambda_{k+1}), Delta_min after the first iteration, the curvature test
__global__ __launch_bounds__(1024) void k_qn_hist(TermSums T, const double* sp, int32_t sn, double offset,
                                                const double* part_sy, const double* part_yy, int32_t hn, int32_t k,
                                                int32_t set_dmin,
                                                double eps, QnState* st, double* etrace, double* sy_out,
                                                double* yy_out, int32_t* accepted) {
  __shared__ double red[16];
  double E = 0.0;
  if (!bound_sum(T, sp, sn, red, &E)) return;   // uniform
  E += offset;
  const double sy = sum_partials_1024(part_sy, hn, red);
  const double yy = sum_partials_1024(part_yy, hn, red);
  if (threadIdx.x != 0) return;
  etrace[k + 1] = E;
  if (set_dmin) st->dmin = 1e-6 * (E - st->E0);
  st->E_init = E;
  st->done = 0;
  st->Em = -INFINITY;
  const bool ok = hn > 0 && sy >= eps;
  if (ok) {
    *sy_out = sy;
    *yy_out = yy;
  }
  *accepted = ok ? 1 : 0;
}

// ---------------------------------------------------------------- layout conversion
// entry order <-> slot planes
template <typename T>
__global__ void k_scatter(const T* v, const uint32_t* word, const int32_t* vinv, int64_t nnz, int64_t n, T* planes) {
  const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= nnz) return;
  const int32_t i = int32_t(word[e] & W_VAR_MASK);
  planes[int64_t((word[e] >> W_SLOT_SHIFT) & 7u) * n + (vinv ? vinv[i] : i)] = v[e];
}

template <typename T>
__global__ void k_gather(const T* planes, const uint32_t* word, const int32_t* vinv, int64_t nnz, int64_t n, T* v) {
  const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= nnz) return;
  const int32_t i = int32_t(word[e] & W_VAR_MASK);
  v[e] = planes[int64_t((word[e] >> W_SLOT_SHIFT) & 7u) * n + (vinv ? vinv[i] : i)];
}

// entry order from cells
__global__ void k_gather_cells(const uint8_t* cells, const uint32_t* ent_cell, int64_t nnz, uint8_t* v) {
  const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e < nnz) v[e] = cells[ent_cell[e]];
}

__global__ void k_fill_f64(double* a, int64_t n, double v) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) a[i] = v;
}

__global__ void k_fill_i32(int32_t* a, int64_t n, int32_t v) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) a[i] = v;
}

// device scalars per history buffer b: s^T y, y^T y, alpha
struct Scal {
  double* p;
  int nb;
  double* sy(int b) const { return p + b; }
  double* yy(int b) const { return p + nb + b; }
  double* alpha(int b) const { return p + 2 * nb + b; }
};

// the numbering of the variables in the planes: cells of variable i, its row
// count; its place in variable order (NULL: i itself) and in the planes from the
// canonical index (NULL: the index itself)
struct Numbering {
  const uint32_t* pos;
  const uint8_t* deg;
  const int32_t* to_v;
  const int32_t* from_i;
};

template <typename R>
dm_status numbering(dm_ctx* ctx, Numbering& N) {
  if constexpr (sizeof(R) == 8) {
    DM_TRY(bound_order(ctx));
    N = {ctx->cpos, ctx->var_deg.p, ctx->vinv.p, nullptr};
  } else {
    N = {ctx->vpos.p, ctx->vdeg.p, nullptr, ctx->vinv.p};
  }
  return DM_OK;
}

unsigned vgrid(int64_t n) {
  return unsigned(std::max<int64_t>(1, std::min<int64_t>(VGRID, (n + VB - 1) / VB)));
}

// d = projected H g into q, over the pairs in `order` (oldest first); part
// holds two VGRID halves; dcell (optional) takes d per cell as well
template <typename R>
dm_status direction(dm_ctx* ctx, const std::vector<int>& order, R* const* S, int8_t* const* Y, const uint8_t* g8,
                    R* q, const Scal& sc, double* part, R* dcell, const Numbering& N) {
  const int64_t n = ctx->n_free;
  const unsigned G = vgrid(n);
  const uint8_t* deg = N.deg;
  hipStream_t st = ctx->stream;
  const int h = int(order.size());
  if (h == 0) {
    k_qn_project_g<R><<<G, VB, 0, st>>>(g8, deg, n, q, N.pos, dcell);
    DM_LAUNCH_CHECK(ctx);
    return DM_OK;
  }
  double* pin = part;
  double* pout = part + VGRID;
  k_qn_first<R><<<G, VB, 0, st>>>(g8, S[order[h - 1]], n, pin);
  for (int i = h - 1; i >= 0; --i) {
    const int b = order[i];
    const R* s_next = i > 0 ? S[order[i - 1]] : nullptr;
    const int8_t* y_next = i > 0 ? nullptr : Y[order[0]];
    k_qn_loop1<R><<<G, VB, 0, st>>>(i == h - 1 ? g8 : nullptr, q, Y[b], s_next, y_next, pin, int32_t(G),
                                     sc.sy(b), sc.alpha(b), n, q, pout);
    std::swap(pin, pout);
  }
  const int newest = order[h - 1];
  for (int i = 0; i < h; ++i) {
    const int b = order[i];
    const int8_t* y_next = i + 1 < h ? Y[order[i + 1]] : nullptr;
    k_qn_loop2<R><<<G, VB, 0, st>>>(q, S[b], y_next, pin, int32_t(G), sc.sy(b), sc.alpha(b),
                                     i == 0 ? sc.sy(newest) : nullptr, i == 0 ? sc.yy(newest) : nullptr, deg, n,
                                     q, pout, N.pos, y_next ? nullptr : dcell);
    std::swap(pin, pout);
  }
  DM_LAUNCH_CHECK(ctx);
  return DM_OK;
}

template <typename R>
struct QnBuffers {
  DArr<unsigned char> mem;   // everything below
  R* q = nullptr;
  uint8_t* g[2] = {nullptr, nullptr};
  double *part = nullptr, *scal = nullptr;
  std::vector<R*> Sp;
  std::vector<int8_t*> Yp;
};

// zeroed buffers of nb pairs
template <typename R>
dm_status qn_alloc(dm_ctx* ctx, int nb, QnBuffers<R>& B) {
  const int64_t rec = std::max<int64_t>(ctx->n_free, 1) * 5;   // five slot planes
  Slab k;
  k.add<R>(rec * nb);
  k.add<int8_t>(rec * nb);
  k.add<R>(rec);
  k.add<uint8_t>(rec);
  k.add<uint8_t>(rec);
  k.add<double>(4 * VGRID);
  k.add<double>(3 * nb);
  DM_ALLOC(ctx, B.mem, k.bytes);
  DM_HIP(ctx, hipMemsetAsync(B.mem.p, 0, k.bytes, ctx->stream));
  k.at = B.mem.p;
  R* S = k.take<R>(rec * nb);
  int8_t* Y = k.take<int8_t>(rec * nb);
  B.q = k.take<R>(rec);
  B.g[0] = k.take<uint8_t>(rec);
  B.g[1] = k.take<uint8_t>(rec);
  B.part = k.take<double>(4 * VGRID);
  B.scal = k.take<double>(3 * nb);
  B.Sp.resize(nb);
  B.Yp.resize(nb);
  for (int b = 0; b < nb; ++b) {
    B.Sp[b] = S + rec * b;
    B.Yp[b] = Y + rec * b;
  }
  return DM_OK;
}

// search state kept on the context between calls (history pairs, step size,
// Delta_min), one per message precision
template <typename R>
struct QnSession {
  QnBuffers<R> B;
  DArr<QnState> st;
  DArr<int32_t> flag;
  std::vector<int> order;   // accepted pairs, oldest first
  int spare = 0;            // buffer of the next candidate pair
  int m = -1;
  int64_t n_free = -1, generation = -1;
};

struct QnSessions {
  QnSession<float> f32;
  QnSession<double> f64;
};

void qn_delete(void* p) { delete static_cast<QnSessions*>(p); }

template <typename R>
QnSession<R>& session(dm_ctx* ctx) {
  if (!ctx->qn) {
    ctx->qn = new QnSessions;
    ctx->qn_free = qn_delete;
  }
  QnSessions* q = static_cast<QnSessions*>(ctx->qn);
  if constexpr (sizeof(R) == 4) return q->f32;
  else return q->f64;
}

template <typename R>
dm_status lbfgs_impl(dm_ctx* ctx, int32_t iters, const dm_lbfgs_params& P, R* lam, double* lb_trace,
                     double* gamma_trace, int32_t* taken) {
  hipStream_t stream = ctx->stream;
  if (ctx->n_rows == 0) {   // nothing free: the bound is the constant
    if (lb_trace) k_fill_f64<<<grid_for(iters + 1, 256), 256, 0, stream>>>(lb_trace, iters + 1, ctx->offset);
    if (gamma_trace && iters > 0)
      k_fill_f64<<<grid_for(iters, 256), 256, 0, stream>>>(gamma_trace, iters, P.gamma0);
    if (taken && iters > 0) k_fill_i32<<<grid_for(iters, 256), 256, 0, stream>>>(taken, iters, 0);
    DM_LAUNCH_CHECK(ctx);
    return DM_OK;
  }
  const int m = P.history;
  const int nb = m + 1;   // m history pairs and one candidate
  QnSession<R>& S = session<R>(ctx);
  const bool resume = P.resume != 0 && S.m == m && S.n_free == ctx->n_free &&
                      S.generation == ctx->cost_generation;
  if (P.resume != 0 && !resume)
    return dm_fail(ctx, DM_ERR_STATE,
                   "resume needs an earlier dm_lbfgs_solve on the same costs with the same precision and history");
  if (!resume) {
    DM_TRY(qn_alloc<R>(ctx, nb, S.B));
    DM_ALLOC(ctx, S.st, 1);
    DM_ALLOC(ctx, S.flag, 1);
    S.order.clear();
    S.spare = 0;
    S.m = m;
    S.n_free = ctx->n_free;
    S.generation = ctx->cost_generation;
  }
  QnBuffers<R>& B = S.B;
  QnState* st = S.st.p;
  const Scal sc{B.scal, nb};
  const int64_t n = ctx->n_free;
  const unsigned G = vgrid(n);
  DM_TRY(dual_flush(ctx));
  CellState& C = ctx->cells;
  DM_TRY(cells_import<R>(ctx, lam, C, true));
  // row minimisers and direction, one value per cell; the bounds
  Slab slab;
  slab.add<uint8_t>(ctx->n_cells + 1);
  slab.add<R>(ctx->n_cells + 1);
  slab.add<double>(int64_t(iters) + 1);
  DArr<unsigned char> mem;
  DM_ALLOC(ctx, mem, slab.bytes);
  slab.at = mem.p;
  uint8_t* gcell = slab.take<uint8_t>(ctx->n_cells + 1);
  R* dcell = slab.take<R>(ctx->n_cells + 1);
  double* etrace = slab.take<double>(int64_t(iters) + 1);
  int cur = 0, gc = 0;
  R* none = nullptr;
  Numbering N;
  DM_TRY(numbering<R>(ctx, N));
  // the bound of a sweep: its block sums, or in FP64 the terms
  constexpr bool ordered = sizeof(R) == 8;
  const TermSums T = ordered ? term_sums(ctx) : TermSums();
  const unsigned SG = sum_grid(T);
  SweepExt sub;
  sub.gsub = gcell;
  sub.terms = ordered ? ctx->terms : nullptr;
  DM_TRY(cells_vars<R>(ctx, C.cells<R>(0), C.costs<R>(), C.ts<R>(0), true));
  DM_TRY(cells_rows<R>(ctx, SWEEP_SUBGRAD, C.cells<R>(0), C.ts<R>(0), none, R(0), nullptr, &sub));
  k_qn_begin<<<SG, 1024, 0, stream>>>(T, ctx->pend_partial, ctx->pend_n, ctx->offset, st, etrace, P.gamma0, resume ? 1 : 0);
  k_qn_gather_g<<<G, VB, 0, stream>>>(gcell, N.pos, N.deg, n, B.g[0]);
  DM_LAUNCH_CHECK(ctx);
  for (int32_t k = 0; k < iters; ++k) {
    DM_TRY(direction<R>(ctx, S.order, B.Sp.data(), B.Yp.data(), B.g[gc], B.q, sc, B.part, dcell, N));
    SweepExt pe;
    pe.dir = dcell;
    pe.gamma = &st->gamma;
    pe.skip = &st->done;
    pe.terms = sub.terms;
    for (int t = 0; t <= P.max_search; ++t) {
      DM_TRY(cells_rows<R>(ctx, SWEEP_BOUND, C.cells<R>(cur), C.ts<R>(cur), none, R(0), nullptr, &pe));
      k_qn_probe<<<SG, 1024, 0, stream>>>(T, ctx->pend_partial, ctx->pend_n, ctx->offset, t, P.max_search, P.step_up,
                                          P.step_down, st, gamma_trace ? gamma_trace + k : nullptr,
                                          taken ? taken + k : nullptr);
      DM_LAUNCH_CHECK(ctx);
      // the search usually stops at the second trial: one read of the flag
      // then spares launching the remaining probes (a skipped launch still
      // dispatches every workgroup of the sweep grid)
      if (t == 1 && t < P.max_search) {
        int32_t done = 0;
        DM_HIP(ctx, hipMemcpyAsync(&done, &st->done, sizeof(int32_t), hipMemcpyDeviceToHost, stream));
        DM_HIP(ctx, hipStreamSynchronize(stream));
        if (done) break;
      }
    }
    SweepExt me;
    me.dir = dcell;
    me.gamma = &st->step;
    const int nxt = cur ^ 1;
    DM_TRY(cells_rows<R>(ctx, SWEEP_UPDATE, C.cells<R>(cur), C.ts<R>(cur), C.cells<R>(nxt), R(P.omega), nullptr, &me));
    DM_TRY(cells_vars<R>(ctx, C.cells<R>(nxt), C.costs<R>(), C.ts<R>(nxt), true));
    DM_TRY(cells_rows<R>(ctx, SWEEP_SUBGRAD, C.cells<R>(nxt), C.ts<R>(nxt), none, R(0), nullptr, &sub));
    double* psy = B.part + 2 * VGRID;
    double* pyy = B.part + 3 * VGRID;
    const int spare = S.spare;
    if (m > 0)
      k_qn_hist_pass<R><<<G, VB, 0, stream>>>(C.cells<R>(cur), C.ts<R>(cur), C.cells<R>(nxt), C.ts<R>(nxt), N.to_v, N.pos,
                                               B.g[gc], gcell, N.deg, n, B.g[gc ^ 1], B.Sp[spare],
                                               B.Yp[spare], psy, pyy);
    else
      k_qn_gather_g<<<G, VB, 0, stream>>>(gcell, N.pos, N.deg, n, B.g[gc ^ 1]);
    k_qn_hist<<<SG, 1024, 0, stream>>>(T, ctx->pend_partial, ctx->pend_n, ctx->offset, psy, pyy, m > 0 ? int32_t(G) : 0, k,
                                    (k == 0 && !resume) ? 1 : 0, P.eps, st, etrace, sc.sy(spare),
                                    sc.yy(spare), S.flag.p);
    DM_LAUNCH_CHECK(ctx);
    cur ^= 1;
    gc ^= 1;
    if (m > 0) {
      int32_t ok = 0;
      DM_TRY(read_i32(ctx, S.flag.p, &ok));
      if (ok) {
        S.order.push_back(spare);
        if (int(S.order.size()) > m) {
          S.spare = S.order.front();
          S.order.erase(S.order.begin());
        } else {
          for (int b = 0; b < nb; ++b)
            if (std::find(S.order.begin(), S.order.end(), b) == S.order.end()) {
              S.spare = b;
              break;
            }
        }
      }
    }
  }
  if (lb_trace)
    DM_HIP(ctx, hipMemcpyAsync(lb_trace, etrace, (size_t(iters) + 1) * sizeof(double), hipMemcpyDeviceToDevice,
                               stream));
  DM_TRY(cells_export<R>(ctx, C.cells<R>(cur), C.ts<R>(cur), lam));
  // the per-call trace buffer is freed on return: wait for the queued work
  DM_HIP(ctx, hipStreamSynchronize(stream));
  return DM_OK;
}

template <typename R>
dm_status subgradient_impl(dm_ctx* ctx, const R* lam, uint8_t* g, double* lb) {
  CellState C;
  DArr<uint8_t> gcell;
  DM_TRY(dual_flush(ctx));
  DM_TRY(cells_import<R>(ctx, lam, C, false));
  DM_ALLOC(ctx, gcell, size_t(ctx->n_cells) + 1);
  DM_ALLOC(ctx, ctx->scal, 16);
  SweepExt sub;
  sub.gsub = gcell.p;
  DM_TRY(cells_vars<R>(ctx, C.cells<R>(0), C.costs<R>(), C.ts<R>(0), true));
  DM_TRY(cells_rows<R>(ctx, SWEEP_SUBGRAD, C.cells<R>(0), C.ts<R>(0), static_cast<R*>(nullptr), R(0), ctx->scal.p,
                       &sub));
  DM_TRY(dual_flush(ctx));
  if (ctx->nnz > 0)
    k_gather_cells<<<grid_for(ctx->nnz, 256), 256, 0, ctx->stream>>>(gcell.p, ctx->ent_cell.p, ctx->nnz, g);
  DM_LAUNCH_CHECK(ctx);
  double v = 0.0;
  DM_HIP(ctx, hipMemcpyAsync(&v, ctx->scal.p, sizeof(double), hipMemcpyDeviceToHost, ctx->stream));
  DM_HIP(ctx, hipStreamSynchronize(ctx->stream));
  if (lb) *lb = v;
  return DM_OK;
}

template <typename R>
dm_status direction_impl(dm_ctx* ctx, int32_t h, const R* S, const int8_t* Y, const uint8_t* g, R* d) {
  const int64_t n = ctx->n_free, nnz = ctx->nnz;
  if (nnz == 0) return DM_OK;
  QnBuffers<R> B;
  DM_TRY(qn_alloc<R>(ctx, std::max(h, 1), B));
  const Scal sc{B.scal, std::max(h, 1)};
  const unsigned G = vgrid(n);
  const unsigned E = grid_for(nnz, 256);
  Numbering N;
  DM_TRY(numbering<R>(ctx, N));
  std::vector<int> order;
  k_scatter<uint8_t><<<E, 256, 0, ctx->stream>>>(g, ctx->rent_word.p, N.from_i, nnz, n, B.g[0]);
  for (int b = 0; b < h; ++b) {
    k_scatter<R><<<E, 256, 0, ctx->stream>>>(S + size_t(b) * nnz, ctx->rent_word.p, N.from_i, nnz, n, B.Sp[b]);
    k_scatter<int8_t><<<E, 256, 0, ctx->stream>>>(Y + size_t(b) * nnz, ctx->rent_word.p, N.from_i, nnz, n, B.Yp[b]);
    k_qn_pair_dots<R><<<G, VB, 0, ctx->stream>>>(B.Sp[b], B.Yp[b], n, B.part, B.part + VGRID);
    k_qn_pair_fin<<<1, 1024, 0, ctx->stream>>>(B.part, B.part + VGRID, int32_t(G), sc.sy(b), sc.yy(b));
    order.push_back(b);
  }
  DM_LAUNCH_CHECK(ctx);
  DM_TRY(direction<R>(ctx, order, B.Sp.data(), B.Yp.data(), B.g[0], B.q, sc, B.part,
                         static_cast<R*>(nullptr), N));
  k_gather<R><<<E, 256, 0, ctx->stream>>>(B.q, ctx->rent_word.p, N.from_i, nnz, n, d);
  DM_LAUNCH_CHECK(ctx);
  DM_HIP(ctx, hipStreamSynchronize(ctx->stream));
  return DM_OK;
}

dm_status check_ready(dm_ctx* ctx, int32_t msg_prec) {
  if (!ctx) return DM_ERR_INVALID_ARG;
  if (!ctx->has_space) return dm_fail(ctx, DM_ERR_STATE, "no product space built");
  if (!ctx->has_cost) return dm_fail(ctx, DM_ERR_STATE, "no costs built");
  if (msg_prec != DM_PREC_FP32 && msg_prec != DM_PREC_FP64)
    return dm_fail(ctx, DM_ERR_INVALID_ARG, "message precision must be FP32 or FP64");
  return DM_OK;
}

}  // namespace

extern "C" dm_status dm_lbfgs_solve(dm_ctx* ctx, int32_t iters, const dm_lbfgs_params* params, int32_t msg_prec,
                                    void* lambda, double* lb_trace, double* gamma_trace, int32_t* taken) {
  DM_TRY(check_ready(ctx, msg_prec));
  ctx->err.clear();
  if (!params || (!lambda && ctx->nnz > 0) || iters < 0)
    return dm_fail(ctx, DM_ERR_INVALID_ARG, "dm_lbfgs_solve: bad arguments");
  const dm_lbfgs_params& P = *params;
  if (P.history < 0 || P.history > 64) return dm_fail(ctx, DM_ERR_INVALID_ARG, "history must be in [0, 64]");
  if (P.max_search < 1 || P.max_search > 64)
    return dm_fail(ctx, DM_ERR_INVALID_ARG, "max_search must be in [1, 64]");
  if (!(P.omega > 0.0 && P.omega <= 1.0)) return dm_fail(ctx, DM_ERR_INVALID_ARG, "omega must be in (0, 1]");
  if (!(P.step_up > 1.0) || !(P.step_down > 0.0 && P.step_down < 1.0) || !(P.gamma0 >= 0.0) ||
      !std::isfinite(P.gamma0) || !std::isfinite(P.step_up) || !std::isfinite(P.eps))
    return dm_fail(ctx, DM_ERR_INVALID_ARG, "need step_up > 1, 0 < step_down < 1, finite gamma0 >= 0, finite eps");
  DM_HIP(ctx, hipSetDevice(ctx->device));
  if (msg_prec == DM_PREC_FP32)
    return lbfgs_impl<float>(ctx, iters, P, static_cast<float*>(lambda), lb_trace, gamma_trace, taken);
  return lbfgs_impl<double>(ctx, iters, P, static_cast<double*>(lambda), lb_trace, gamma_trace, taken);
}

extern "C" dm_status dm_subgradient(dm_ctx* ctx, int32_t msg_prec, const void* lambda, uint8_t* g, double* lb) {
  DM_TRY(check_ready(ctx, msg_prec));
  ctx->err.clear();
  if ((!lambda || !g) && ctx->nnz > 0) return dm_fail(ctx, DM_ERR_INVALID_ARG, "dm_subgradient: NULL argument");
  DM_HIP(ctx, hipSetDevice(ctx->device));
  if (msg_prec == DM_PREC_FP32) return subgradient_impl<float>(ctx, static_cast<const float*>(lambda), g, lb);
  return subgradient_impl<double>(ctx, static_cast<const double*>(lambda), g, lb);
}

extern "C" dm_status dm_lbfgs_direction(dm_ctx* ctx, int32_t msg_prec, int32_t h, const void* S, const int8_t* Y,
                                        const uint8_t* g, void* d) {
  DM_TRY(check_ready(ctx, msg_prec));
  ctx->err.clear();
  if (h < 0 || h > 64 || !g || !d || (h > 0 && (!S || !Y)))
    return dm_fail(ctx, DM_ERR_INVALID_ARG, "dm_lbfgs_direction: bad arguments");
  DM_HIP(ctx, hipSetDevice(ctx->device));
  if (msg_prec == DM_PREC_FP32)
    return direction_impl<float>(ctx, h, static_cast<const float*>(S), Y, g, static_cast<float*>(d));
  return direction_impl<double>(ctx, h, static_cast<const double*>(S), Y, g, static_cast<double*>(d));
}
