// Jacobi min-marginal averaging on the Lagrangean dual (Sec. 3.2, Eq. (D);
// the MMA step of Alg. 1) and the dual bound.
//
// State layout (hard minimum).  Every entry of the presolved rows owns one
// cell with its multiplier s^j_i; the cells are in row order (layout.hip).  One
// iteration is two passes:
//   1. k_vars, one thread per variable: gathers the variable's s from its (at
//      most five) cells and writes one value, the residual t_i = c_i - sum_k s_k;
//   2. k_sweep, over the rows: each entry reads its cell and its variable's t
//      and restores dual feasibility, lambda^j_i = s_j + t_i / |J_i|; the row
//      computes its minimum and the min-marginal differences M^j_i =
//      min_{s_i=1} - min_{s_i=0} (Appendix "Coarse-to-fine"); each entry writes
//      s_j' = lambda^j_i - omega M^j_i back to its cell.  Row minima are summed
//      into an FP64 bound in a fixed order.
// Together they are lambda <- lambda - omega (M - mean_j M): the mean of the
// min-marginals is exactly what the projection adds back.
//
// What bounds an iteration and why two passes: an entry needs its variable's
// sum, and a single pass has to gather the variable's whole 32-byte record for
// it and scatter 4 bytes into another (measured: 3.7 times the algorithmic
// bytes through the L2 at the 2000/3000-face pair, 253 us).  Split in two, the
// row pass streams its cells coalesced, in place, and every random access is a
// 4-byte read of a small array (t: 4 bytes per variable) or of cells that
// neighbouring variables share.  Measured, one iteration of a long solve before
// and after: 13.2 -> 9.2 to 9.7 us at the 500-face pair (two launches of 2.4 us
// each are half of it), 41.6 -> 22.6 at 1000 faces, 253 -> 108 at 2000/3000 (row
// pass 66, variable pass 43; 5.0 TB/s through the L2s, a plain copy reaches 4.7 to
// 4.9), 837 -> 342 with K = 144 candidates.
//
// Problems of few entries take other forms of the same iteration, bit for bit: one
// workgroup that runs all of them from LDS (k_small), or one launch each, in
// which every entry sums its variable's cells itself (k_iterate); see hard_form.
//
// Rows: closedness rows (short, coefficients +-1, right-hand side b) with b = 0
// and few entries run one lane per row (tiles), the others one lane per entry
// in wave chunks, with the row minimum from sorted prefix sums: choosing k
// entries with coefficient +1 and k-b with -1 costs at least S+(k) + S-(k-b),
// the sums of the k and k-b smallest multipliers.  Projection rows (all +1,
// b = 1) get one wave or one block each and reduce (min, argmin, second min).
//
// With a temperature T > 0 every min becomes the soft-min -T log sum
// exp(-./T); short rows then run a partial-sum recursion with one lane per
// partial sum.  That sweep is bound by its arithmetic and keeps one record of
// REC reals per variable (slots 0-2 for its three closedness rows, then its
// projection rows, slot 5 the cost, slot 6 the reciprocal row count) in two
// buffers that alternate between iterations, one launch per iteration.
#include <hip/hip_ext.h>

#include <cmath>

#include "dm_internal.h"
#include "small_layout.h"

namespace {

constexpr int MODE_UPDATE = SWEEP_UPDATE, MODE_EVAL = SWEEP_EVAL, MODE_BOUND = SWEEP_BOUND,
              MODE_SUBGRAD = SWEEP_SUBGRAD;

template <typename R>
__device__ inline R rinf() {
  return R(INFINITY);
}

template <typename R>
__device__ inline R r_exp(R x);
template <>
__device__ inline float r_exp<float>(float x) { return expf(x); }
template <>
__device__ inline double r_exp<double>(double x) { return exp(x); }
template <typename R>
__device__ inline R r_log(R x);
template <>
__device__ inline float r_log<float>(float x) { return logf(x); }
template <>
__device__ inline double r_log<double>(double x) { return log(x); }

// Scaled soft-min arithmetic for the short-row recursion.  Values are kept in
// units u = x / (T ln 2) (FP32) or u = x / T (FP64), so that the soft-min of
// two values is min - L(1 + E(-|a - b|)) and of many min - L(sum E(u - min))
// with E = 2^x, L = log2 (FP32: the hardware exp2 / log2 instructions, about
// one ulp) or E = exp, L = log (FP64).
template <typename R>
struct SoftUnits;
template <>
struct SoftUnits<float> {
  // a state that cannot be reached holds none; while a row's values are at most
  // most, every sum of them is below lim and every such state above it
  static constexpr float none = 1e37f, lim = 1e36f, most = 1e34f, big = 3.402823466e+38f;
  static __device__ float unit(float T) { return T * 0.693147180559945309f; }   // x = u * unit
  static __device__ float E(float x) { return __builtin_amdgcn_exp2f(x); }
  static __device__ float L(float x) { return __builtin_amdgcn_logf(x); }
  static __device__ float L1p(float x) { return __builtin_amdgcn_logf(1.0f + x); }
};
template <>
struct SoftUnits<double> {
  static constexpr double none = 1e307, lim = 1e306, most = 1e304, big = 1.7976931348623157e+308;
  static __device__ double unit(double T) { return T; }
  static __device__ double E(double x) { return exp(x); }
  static __device__ double L(double x) { return log(x); }
  static __device__ double L1p(double x) { return log1p(x); }
};

// soft-min of two values in scaled units, without branches.  Neither is +inf and
// both at once: a state that cannot be reached holds SoftUnits::none, so large
// that E of its distance to any value is 0, and finite.
template <typename R>
__device__ inline R smin2u(R a, R b) {
  return fmin(a, b) - SoftUnits<R>::L1p(SoftUnits<R>::E(-fabs(a - b)));
}

// The same where a state that cannot be reached holds +inf: clamped to the
// largest finite value, an infinite operand leaves the other, and two give +inf.
template <typename R>
__device__ inline R smin2u_inf(R a, R b) {
  constexpr R big = SoftUnits<R>::big;
  return fmin(a, b) - SoftUnits<R>::L1p(SoftUnits<R>::E(-fabs(fmin(a, big) - fmin(b, big))));
}

// multiplier of entry word w from the previous record buffer, with dual
// feasibility restored
template <typename R>
__device__ inline R cur_lambda(const R* __restrict__ rec, uint32_t w) {
  R lam[5];
  rec_lambdas<R>(rec, size_t(w & W_VAR_MASK), lam);
  const int k = int((w >> W_SLOT_SHIFT) & 7u);
  return k == 0 ? lam[0] : k == 1 ? lam[1] : k == 2 ? lam[2] : k == 3 ? lam[3] : lam[4];
}

template <typename R>
__device__ inline void write_out(R* __restrict__ out, uint32_t w, R v) {
  out[size_t(w & W_VAR_MASK) * REC + ((w >> W_SLOT_SHIFT) & 7u)] = v;
}

// block-wide FP64 sum of a 256-thread block in a fixed order (the waves in
// index order); red is not reused after it
__device__ inline double block_sum(double v, double* red) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return ((red[0] + red[1]) + red[2]) + red[3];
}

// Each block stores the sum of its row minima; the per-block partials of one
// launch are summed in index order by block 0 of the next launch (the kernel
// boundary makes them visible without atomics or cache maintenance) or by a
// one-block kernel after the last launch.
__device__ inline void store_partial(double part, double* partial, int32_t item) {
  if (threadIdx.x == 0) partial[item] = part;
}

__device__ inline void reduce_partials(const double* partial, int n, double offset, double* out, double* red) {
  const double tot = sum_partials_256(partial, n, red);
  if (threadIdx.x == 0) *out = offset + tot;
}

struct SweepArgs {
  // ---- hard minimum: cells
  const uint32_t* word;     // per cell: variable and row count, CHUNK_PAD for padding
  int32_t n_tiles[TILE_FORMS];   // 64-row tiles of each form
  uint32_t tile_cell0[TILE_FORMS], chunk_cell0, long_cell0;   // first cells
  int32_t n_chunks;         // wave chunks of short rows
  const unsigned long long* chunk_mask;   // bit e: entry e of the chunk starts a row
  const unsigned long long* chunk_neg;    // bit e: entry e has coefficient -1
  const int8_t* chunk_b;    // 64 per chunk: right-hand side of the entry's row
  int32_t n_long_y;         // of the projection rows in launch order, the Y rows come first
  int32_t per[3 + TILE_FORMS];   // blocks per XCD: Y rows, X rows, chunks, tiles from the widest form down
  const int2* long_row;     // first cell and length of the projection rows in launch order
  const int32_t* long_ent;  // entry of each projection-row cell (ties in MODE_SUBGRAD), or NULL: in order
  // quasi-Newton extensions: rows see lambda + gamma * dir when dir is set
  // (one value per cell; gamma a device scalar); the launch does nothing when
  // *skip is nonzero; MODE_SUBGRAD writes the row's minimising assignment
  // (1 / 0 per entry) to its cells of gsub
  const void* dir;
  const double* gamma;
  const int32_t* skip;
  uint8_t* gsub;
  // FP64 bounds of the quasi-Newton search: every row's term goes to its place
  double* terms;
  const int32_t *term_row, *term_long;
  int32_t tile_rows[TILE_FORMS], term_chunk0, term_long0;
  // ---- smoothed: records
  const uint32_t* ent_word;   // per entry: sign, slot, variable
  const int32_t* soft_row;  // short rows in order of length
  int32_t soft_c8, soft_c16;  // short rows of at most 7 / of 8 to 15 entries
  const int32_t* rrow_b;
  int32_t n_short_blocks;   // blocks of short rows
  int32_t n_items;          // short-row blocks + long-row blocks
  // ---- both
  const int32_t* rrow_ptr;
  int32_t n_short;
  int32_t long_wpr;         // waves per projection row: 1 or 4
  int32_t n_long;           // projection rows
  const int32_t* long_perm; // projection rows (relative to n_short) in launch order
  double* partial;          // this launch's per-block partials
  const double* prev_partial; // smoothed: previous launch's partials still to be summed, or NULL
  int32_t prev_n;
  double prev_offset;
  double* prev_out;
};

// multiplier of a cell with dual feasibility restored: s + t (1/|J|) in one
// rounding, as rec_lambdas forms it
template <typename R>
__device__ inline R feasible(R s, R t, R rdeg) {
  if constexpr (sizeof(R) == 4) return __builtin_fmaf(t, rdeg, s);
  else return __builtin_fma(t, rdeg, s);
}

template <typename R>
__device__ inline R fma_r(R a, R b, R c) {
  if constexpr (sizeof(R) == 4) return __builtin_fmaf(a, b, c);
  else return __builtin_fma(a, b, c);
}

// 1/|J| of a cell word.  A product triangle lies in four or five rows; the
// top bit of the count tells those from the fewer rows of a generic variable.
template <typename R>
__device__ inline R rdeg_hi(uint32_t w) {
  return (w >> CELL_DEG_SHIFT) & 1u ? R(1) / R(5) : R(1) / R(4);
}
template <typename R>
__device__ inline R rdeg_of(uint32_t w) {
  const uint32_t d = w >> CELL_DEG_SHIFT;
  const R lo = d == 1u ? R(1) : (d == 2u ? R(1) / R(2) : R(1) / R(3));
  return (w >> 31) ? rdeg_hi<R>(w) : lo;
}

// Where a row pass takes the residuals from: the array that the variable pass
// wrote, or the variable's cost and cells, added in the variable pass's order.
template <typename R>
using Written = const R* __restrict__;

template <typename R>
struct Summed {
  const uint32_t* __restrict__ vpos;
  const R* __restrict__ cells;
  const R* __restrict__ cost;
  uint32_t n;
  __device__ R operator[](uint32_t v) const {
    uint32_t p[5];
    R s[5];
#pragma unroll
    for (uint32_t q = 0; q < 5; ++q) p[q] = vpos[q * n + v];
    const R c = cost[v];
#pragma unroll
    for (int q = 0; q < 5; ++q) s[q] = cells[p[q]];
    return c - ((((s[0] + s[1]) + s[2]) + s[3]) + s[4]);
  }
};

// multiplier of cell c (word w, not padding) as the rows see it: feasible, and
// moved along dir when one is set
template <typename R, typename RT>
__device__ inline R cell_lambda(const SweepArgs& A, const R* cells, RT t, uint32_t c, uint32_t w, R gam) {
  R v = feasible<R>(cells[c], t[w & W_VAR_MASK], rdeg_of<R>(w));
  if (A.dir) v = fma_r<R>(gam, static_cast<const R*>(A.dir)[c], v);
  return v;
}

// ---------------------------------------------------------------- short rows, hard min
// One wave per chunk of whole closedness rows (<= 64 entries, one per lane),
// four chunks per block, with an LDS slice per wave and no barrier until the
// bound.  Every cross-lane step runs in a wave-uniform loop, so no lane ever
// reads from an inactive lane:
//  1. lane e holds entry e (multiplier, sign, word) and finds its row in the
//     chunk's mask of row starts;
//  2. rank inside the row's sign group by comparing with the row's values, which
//     the wave's slice holds; if every row of the chunk has b = 0, a closed form
//     of the ranks gives the rest;
//  3. ds_permute moves every value to its sorted position;
//  4. a segmented inclusive scan gives S(k), the sum of the k smallest of a
//     group, at the lane of the k-th smallest;
//  5. each lane evaluates its two constrained minima over k.
// 16-byte LDS read of four FP32 or two FP64 values
template <typename R>
struct LdsVec;
template <>
struct LdsVec<float> {
  using type = float4;
  static __device__ float get(const float4& v, int u) { return u == 0 ? v.x : u == 1 ? v.y : u == 2 ? v.z : v.w; }
};
template <>
struct LdsVec<double> {
  using type = double2;
  static __device__ double get(const double2& v, int u) { return u == 0 ? v.x : v.y; }
};

template <typename R>
__device__ inline R permute_to(int dst_lane, R v) {   // push v to lane dst_lane
  if constexpr (sizeof(R) == 4) {
    return __int_as_float(__builtin_amdgcn_ds_permute(dst_lane << 2, __float_as_int(v)));
  } else {
    const long long bits = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_ds_permute(dst_lane << 2, int(bits & 0xFFFFFFFFll));
    const int hi = __builtin_amdgcn_ds_permute(dst_lane << 2, int(bits >> 32));
    return __longlong_as_double((static_cast<long long>(hi) << 32) | (static_cast<long long>(lo) & 0xFFFFFFFFll));
  }
}

template <typename R, typename RT, int MODE>
__device__ inline double short_chunk_hard(const SweepArgs& A, const R* cells, RT t_, R* out, R omega, R gam,
                                          int32_t wc, R* wave_vals) {
  const int lane = threadIdx.x & 63;
  double rowpart = 0.0;
  if (wc < A.n_chunks) {   // uniform across the wave
    // the padded chunk: words and right-hand sides straight from the chunk index
    const unsigned long long starts = A.chunk_mask[wc];
    const unsigned long long negm = A.chunk_neg[wc];
    const uint32_t cell = A.chunk_cell0 + uint32_t(wc) * 64u + uint32_t(lane);
    const uint32_t w = A.word[cell];
    const int32_t b = A.chunk_b[size_t(wc) * 64 + lane];
    const bool act = w != CHUNK_PAD;
    const int32_t ne = __popcll(__ballot(act));
    const R lam = act ? cell_lambda<R, RT>(A, cells, t_, cell, w, gam) : R(0);
    const int g = int((negm >> lane) & 1ull);
    // my row from the chunk's row-start mask: its start is the last set bit at
    // or below this lane, its end the next set bit (or the chunk's end)
    const unsigned long long le = lane == 63 ? ~0ull : ((2ull << lane) - 1ull);
    const unsigned long long below = starts & le, above = starts & ~le;
    const int32_t s = 63 - __clzll(static_cast<long long>(below));   // entry 0 always starts a row
    const int32_t n = (above ? __ffsll(static_cast<long long>(above)) - 1 : ne) - s;

    const unsigned long long rowm = act ? (((n >= 64) ? ~0ull : ((1ull << n) - 1ull)) << s) : 0ull;
    const int32_t P = __popcll(rowm & ~negm);
    const int32_t N = n - P;
    // rank of this entry in its sign group (ties broken by lane): the wave's
    // values go to its own 64-entry LDS slice, and each lane reads its row in
    // aligned 16-byte pieces (lanes of one row read the same addresses: a
    // broadcast); only this wave touches the slice, so a wave-level fence
    // orders the writes before the reads
    wave_vals[lane] = lam;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    constexpr int V = 16 / int(sizeof(R));   // values per 16-byte read
    using Vec = typename LdsVec<R>::type;
    if (__ballot(act && b != 0) == 0ull) {   // uniform: every row of the chunk has b = 0
      // Rows with b = 0 choose k entries of each sign.  With P and Q the
      // sorted +1 and -1 groups, the pair sums p_(j) + q_(j) never decrease,
      // so the minimiser takes the k* pairs with negative sums.  An entry of
      // rank r (1-based, ties by lane) is taken iff the other group holds at
      // least r values whose sum with it is negative.  Its min-marginal needs
      // only the order statistics around k*: with U = min(p_(k*+1), -q_(k*))
      // and V = min(q_(k*+1), -p_(k*)) (empty terms +inf),
      //   taken +1: p - U,  left +1: p + V,  taken -1: q - V,  left -1: q + U,
      // and the row minimum is the sum of the taken values.
      int32_t rank = 0, cnt = 0;
      if (act) {
        const R nlam = -lam;
        for (int a = s & ~(V - 1); a < s + n; a += V) {
          const Vec v = *reinterpret_cast<const Vec*>(wave_vals + a);
#pragma unroll
          for (int u = 0; u < V; ++u) {
            const int src = a + u;
            const R lq = LdsVec<R>::get(v, u);
            const int gq = int((negm >> src) & 1ull);
            if (src >= s && src < s + n) {
              if (gq == g) rank += (lq < lam) || (lq == lam && src < lane);
              else cnt += lq < nlam;
            }
          }
        }
      }
      const bool sel = act && cnt > rank;
      // U collects left +1 and taken -1 entries, V left -1 and taken +1
      // entries, each as +-lambda
      const R t = sel ? -lam : lam;
      R* uvals = wave_vals + 64;
      R* vvals = wave_vals + 128;
      uvals[lane] = (act && g == int(sel)) ? t : rinf<R>();
      vvals[lane] = (act && g != int(sel)) ? t : rinf<R>();
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      if (act) {
        R U = rinf<R>(), Vv = rinf<R>();
        if (MODE == MODE_UPDATE || MODE == MODE_EVAL) {
          for (int a = s & ~(V - 1); a < s + n; a += V) {
            const Vec uv = *reinterpret_cast<const Vec*>(uvals + a);
            const Vec vv = *reinterpret_cast<const Vec*>(vvals + a);
#pragma unroll
            for (int u = 0; u < V; ++u) {
              const int src = a + u;
              if (src >= s && src < s + n) {
                U = fmin(U, LdsVec<R>::get(uv, u));
                Vv = fmin(Vv, LdsVec<R>::get(vv, u));
              }
            }
          }
          const R Wm = g == int(sel) ? Vv : U;
          const R M = sel ? lam - Wm : lam + Wm;
          if (MODE == MODE_UPDATE) out[cell] = fma_r<R>(-omega, M, lam);
          if (MODE == MODE_EVAL) out[cell] = M;
        }
        if (MODE == MODE_SUBGRAD) A.gsub[cell] = uint8_t(sel ? 1 : 0);
        if (sel) rowpart = double(lam);
      }
      return rowpart;
    }
    // general right-hand sides: the rank as above, then a sort of the chunk
    int32_t rank = 0;
    if (act) {
      for (int a = s & ~(V - 1); a < s + n; a += V) {   // a + V <= 64: the slice's end
        const Vec v = *reinterpret_cast<const Vec*>(wave_vals + a);
#pragma unroll
        for (int u = 0; u < V; ++u) {
          const int src = a + u;
          const R lq = LdsVec<R>::get(v, u);
          const int gq = int((negm >> src) & 1ull);
          if (src >= s && src < s + n && gq == g) rank += (lq < lam) || (lq == lam && src < lane);
        }
      }
    }
    // sorted position: positive group first, then negative group
    const int dst = act ? s + (g ? P + rank : rank) : lane;
    const R srt = permute_to<R>(dst, lam);
    // segmented inclusive scan over the sorted groups: lane j of row [s, s+n)
    // belongs to the +1 group if j - s < P
    const int32_t seg = act ? s + (lane - s < P ? 0 : P) : lane;
    R pre = srt;
    for (int off = 1; off < 64; off <<= 1) {
      const R t = __shfl(pre, lane >= off ? lane - off : 0);
      if (lane - off >= seg) pre += t;
    }
    // pre at lane (group start + k - 1) = S_group(k).
    // Choosing k of the own group and k - bb of the other costs
    // f(k) = S_own(k) + S_oth(k - bb) for k in [klo, khi]; its increments
    // o_k + q_{k-bb} (sorted values of the two groups) never decrease, so f is
    // convex and its smallest minimiser is klo plus the number of negative
    // increments.  The constrained minima of an entry at sorted position t are
    // minima of two more convex sequences over ranges that depend on t:
    //   A(k) = S_own(k-1) + S_oth(k-bb)  (increments o_{k-1} + q_{k-bb}),
    //   B(k) = S_own(k+1) + S_oth(k-bb)  (increments o_{k+1} + q_{k-bb}),
    // so they too come from counts of negative increments, clamped to the range.
    // 1. sorted role: lane L holds the k-th smallest of its group
    const int32_t j = lane - s;
    const int gs = act && j >= P;
    const int32_t ks = j - (gs ? P : 0) + 1;
    const int32_t own_s = gs ? N : P, oth_s = gs ? P : N, bb_s = gs ? -b : b;
    const int32_t klo_s = bb_s > 0 ? bb_s : 0;
    const int32_t khi_s = own_s < oth_s + bb_s ? own_s : oth_s + bb_s;
    const int32_t qi = s + (gs ? 0 : P) + (ks - bb_s) - 1;
    const R qv = __shfl(srt, qi >= 0 && qi < 64 ? qi : 0);
    const R om1 = __shfl(srt, lane > 0 ? lane - 1 : 0);
    const R op1 = __shfl(srt, lane < 63 ? lane + 1 : 63);
    const int32_t alo_s = klo_s > 1 ? klo_s : 1;
    const int32_t bhi_s = khi_s < own_s - 1 ? khi_s : own_s - 1;
    const unsigned long long mF = __ballot(act && ks > klo_s && ks <= khi_s && srt + qv < R(0));
    const unsigned long long mA = __ballot(act && ks > alo_s && ks <= khi_s && om1 + qv < R(0));
    const unsigned long long mB = __ballot(act && ks > klo_s && ks <= bhi_s && op1 + qv < R(0));
    // 2. entry role: this lane's entry has own-group position t = rank + 1
    const int32_t own = g ? N : P, oth = g ? P : N, bb = g ? -b : b;
    const int32_t obase = s + (g ? P : 0), tbase = s + (g ? 0 : P);
    const int32_t klo = bb > 0 ? bb : 0;
    const int32_t khi = own < oth + bb ? own : oth + bb;
    const unsigned long long gmask = act ? (((own >= 64) ? ~0ull : ((1ull << own) - 1ull)) << obase) : 0ull;
    const int32_t kbest = klo + __popcll(mF & gmask);   // smallest minimiser
    auto s_own = [&](int32_t k) {   // every lane shuffles; k == 0 gives 0
      const int i = obase + k - 1;
      const R v = __shfl(pre, i >= 0 && i < 64 ? i : 0);
      return k <= 0 ? R(0) : v;
    };
    auto s_oth = [&](int32_t k) {
      const int i = tbase + k - 1;
      const R v = __shfl(pre, i >= 0 && i < 64 ? i : 0);
      return k <= 0 ? R(0) : v;
    };
    const R rmin = s_own(kbest) + s_oth(kbest - bb);
    R m1 = rmin, m0 = rmin;
    if (MODE == MODE_UPDATE || MODE == MODE_EVAL) {
      const int32_t t = rank + 1;
      const bool sel = t <= kbest;   // the minimiser takes this entry
      // the other side's minimum: f at the nearest k on that side, and A or B
      // at their convex minimiser clamped to the side's range
      const int32_t x1 = sel ? t - 1 : t;
      const bool c1ok = sel ? (t - 1 >= klo) : (t <= khi);
      const R c1 = s_own(x1) + s_oth(x1 - bb);
      int32_t lo2, hi2, kst;
      if (sel) {
        lo2 = t > klo ? t : klo;
        hi2 = khi < own - 1 ? khi : own - 1;
        kst = klo + __popcll(mB & gmask);
      } else {
        lo2 = klo > 1 ? klo : 1;
        hi2 = t - 1 < khi ? t - 1 : khi;
        kst = lo2 + __popcll(mA & gmask);
      }
      const bool c2ok = lo2 <= hi2;
      const int32_t k2 = kst < lo2 ? lo2 : (kst > hi2 ? hi2 : kst);
      const R so2 = s_own(sel ? k2 + 1 : k2 - 1);
      const R st2 = s_oth(k2 - bb);
      const R c2 = sel ? (so2 - lam) + st2 : (lam + so2) + st2;
      R other = rinf<R>();
      if (c1ok) other = c1;
      if (c2ok && c2 < other) other = c2;
      if (sel) m0 = other;
      else m1 = other;
    }
    if (act) {
      const R M = m1 - m0;
      if (MODE == MODE_UPDATE) out[cell] = fma_r<R>(-omega, M, lam);
      if (MODE == MODE_EVAL) out[cell] = M;
      if (MODE == MODE_SUBGRAD)
        A.gsub[cell] = uint8_t(rank < kbest ? 1 : 0);
      if (lane == s) rowpart = double(rmin);
    }
  }
  return rowpart;
}

// the four waves of a block take four adjacent chunks
template <typename R, typename RT, int MODE>
__device__ __forceinline__ double chunk_block(const SweepArgs& A, const R* cells, RT t, R* out, R omega, R gam,
                                              unsigned char* smem, int32_t item) {
  const int wave = threadIdx.x >> 6;
  R* wave_vals = reinterpret_cast<R*>(smem) + wave * CHUNK_SLICE;
  [[clang::always_inline]] return short_chunk_hard<R, RT, MODE>(A, cells, t, out, omega, gam, item * 4 + wave, wave_vals);
}

// ---------------------------------------------------------------- short rows with b = 0, one lane per row
// Rows with right-hand side 0 and at most H entries of each sign run one lane
// per row, 64 rows per wave (a tile).  Pair j of lane l holds the row's j-th +1
// and j-th -1 entry, each group in row order, in cells j * 128 + 2 l and the
// next one (one 8-byte access per pair and lane, 512 bytes per wave).  The
// multipliers stay in registers and the closed form of the b = 0 rows (see
// short_chunk_hard) is evaluated over pairs: within a group the earlier
// entry's rank rises if it is larger, the later one's if it is not smaller;
// across the groups both counts rise if the pair sums to a negative value.
// d = count - rank decides whether an entry is taken (d > 0).  A missing entry
// holds +inf: it is never taken, never ranked before a value and never pairs
// to a negative sum.
// Several widths, because the cells of a tile are streamed whether they are
// used or not and the comparisons grow with the square of the width: 76 % of
// the rows of the 2000/3000-face pair have at most 5 entries of each sign,
// 99.4 % at most 8; of the small pairs that the exact search meets, most have 3.
template <typename R>
struct Pair2;
template <>
struct Pair2<float> {
  using type = float2;
};
template <>
struct Pair2<double> {
  using type = double2;
};

template <typename R, typename RT, int MODE, int H>
__device__ inline double tile_rows(const SweepArgs& A, const R* cells, RT t, R* out, R omega, R gam, uint32_t cell0) {
  using P2 = typename Pair2<R>::type;
  const uint32_t c0 = cell0 + 2u * (threadIdx.x & 63u);
  uint2 wv[H];
  P2 sv[H];
#pragma unroll
  for (int j = 0; j < H; ++j) wv[j] = *reinterpret_cast<const uint2*>(A.word + c0 + 128u * j);
#pragma unroll
  for (int j = 0; j < H; ++j) sv[j] = *reinterpret_cast<const P2*>(cells + c0 + 128u * j);
  R lp[H], lq[H];
#pragma unroll
  for (int j = 0; j < H; ++j) {   // a missing entry reads t of variable 0 and is replaced below
    lp[j] = t[wv[j].x != CHUNK_PAD ? wv[j].x & W_VAR_MASK : 0u];
    lq[j] = t[wv[j].y != CHUNK_PAD ? wv[j].y & W_VAR_MASK : 0u];
  }
  uint32_t all = 0xFFFFFFFFu;
#pragma unroll
  for (int j = 0; j < H; ++j) all &= wv[j].x & wv[j].y;
  if (__all(int(all >> 31))) {   // every variable in four or five rows (padding reads as seven)
#pragma unroll
    for (int j = 0; j < H; ++j) {
      lp[j] = feasible<R>(sv[j].x, lp[j], rdeg_hi<R>(wv[j].x));
      lq[j] = feasible<R>(sv[j].y, lq[j], rdeg_hi<R>(wv[j].y));
    }
  } else {
#pragma unroll
    for (int j = 0; j < H; ++j) {
      lp[j] = feasible<R>(sv[j].x, lp[j], rdeg_of<R>(wv[j].x));
      lq[j] = feasible<R>(sv[j].y, lq[j], rdeg_of<R>(wv[j].y));
    }
  }
  if (A.dir) {   // uniform: rows see lambda + gamma * dir
    P2 dv[H];
#pragma unroll
    for (int j = 0; j < H; ++j) dv[j] = *reinterpret_cast<const P2*>(static_cast<const R*>(A.dir) + c0 + 128u * j);
#pragma unroll
    for (int j = 0; j < H; ++j) {
      lp[j] = fma_r<R>(gam, dv[j].x, lp[j]);
      lq[j] = fma_r<R>(gam, dv[j].y, lq[j]);
    }
  }
#pragma unroll
  for (int j = 0; j < H; ++j) {
    lp[j] = wv[j].x != CHUNK_PAD ? lp[j] : rinf<R>();
    lq[j] = wv[j].y != CHUNK_PAD ? lq[j] : rinf<R>();
  }
  int32_t dp[H], dq[H];
#pragma unroll
  for (int j = 0; j < H; ++j) dp[j] = dq[j] = 0;
#pragma unroll
  for (int j = 1; j < H; ++j)
#pragma unroll
    for (int k = 0; k < j; ++k) {
      const bool lep = lp[k] <= lp[j], leq = lq[k] <= lq[j];   // k is earlier: a tie ranks j after k
      dp[j] -= lep ? 1 : 0;
      dp[k] -= lep ? 0 : 1;
      dq[j] -= leq ? 1 : 0;
      dq[k] -= leq ? 0 : 1;
    }
#pragma unroll
  for (int j = 0; j < H; ++j)
#pragma unroll
    for (int k = 0; k < H; ++k) {
      const int ng = lp[j] + lq[k] < R(0) ? 1 : 0;   // the pair's sum (its sign is exact)
      dp[j] += ng;
      dq[k] += ng;
    }
  // U: left +1 and taken -1 entries, V: left -1 and taken +1 entries (as +-lambda)
  R U = rinf<R>(), V = rinf<R>();
  double rowmin = 0.0;
#pragma unroll
  for (int j = 0; j < H; ++j) {
    if (dp[j] > 0) {
      V = fmin(V, -lp[j]);
      rowmin += double(lp[j]);
    } else {
      U = fmin(U, lp[j]);
    }
    if (dq[j] > 0) {
      U = fmin(U, -lq[j]);
      rowmin += double(lq[j]);
    } else {
      V = fmin(V, lq[j]);
    }
  }
  if (MODE == MODE_SUBGRAD) {
#pragma unroll
    for (int j = 0; j < H; ++j)
      *reinterpret_cast<uchar2*>(A.gsub + c0 + 128u * j) = make_uchar2(dp[j] > 0 ? 1 : 0, dq[j] > 0 ? 1 : 0);
  }
  if (MODE == MODE_UPDATE || MODE == MODE_EVAL) {
#pragma unroll
    for (int j = 0; j < H; ++j) {
      // taken +1: p - U, left +1: p + V, taken -1: q - V, left -1: q + U;
      // padding cells take what comes out, they are never read
      P2 m;
      m.x = dp[j] > 0 ? lp[j] - U : lp[j] + V;
      m.y = dq[j] > 0 ? lq[j] - V : lq[j] + U;
      if (MODE == MODE_UPDATE) {
        m.x = fma_r<R>(-omega, m.x, lp[j]);
        m.y = fma_r<R>(-omega, m.y, lq[j]);
      }
      *reinterpret_cast<P2*>(out + c0 + 128u * j) = m;
    }
  }
  return rowmin;
}

// the four waves of a block take four adjacent tiles of one form
template <typename R, typename RT, int MODE, int FORM>
__device__ __forceinline__ double tile_block(const SweepArgs& A, const R* cells, RT t, R* out, R omega, R gam,
                                             int32_t item) {
  constexpr int H = TILE_HALF[FORM];
  const int32_t tile = item * 4 + int32_t(threadIdx.x >> 6);
  if (tile >= A.n_tiles[FORM]) return 0.0;   // uniform across the wave
  // inlined here whatever else calls it: as a function it costs the sweep 40
  // registers and 6 % of its time
  [[clang::always_inline]] return tile_rows<R, RT, MODE, H>(A, cells, t, out, omega, gam,
                                                             A.tile_cell0[FORM] + uint32_t(tile) * (128u * H));
}

// The same rows with a lane per entry, for the form that has one launch per
// iteration: a row's 2 H cells go to SPREAD lanes, so that each gathers one
// residual, not 2 H of them one after the other.  The entries see each other by
// lane exchange; every comparison is that of tile_rows.
template <int H>
constexpr int SPREAD = H <= 4 ? 8 : 16;

template <typename R, typename RT, int H>
__device__ inline double tile_spread(const SweepArgs& A, const R* cells, RT t, R* out, R omega, uint32_t cell0,
                                     uint32_t row0) {
  constexpr int W = SPREAD<H>;
  static_assert(2 * H <= W, "a row's cells need a lane each");
  const uint32_t lane = threadIdx.x & 63u, k = lane % W, j = k / 2;
  const bool neg = k & 1u;
  const uint32_t cell = cell0 + 128u * j + 2u * (row0 + lane / W) + (k & 1u);
  const uint32_t w = k < 2 * H ? A.word[cell] : CHUNK_PAD;
  const bool act = w != CHUNK_PAD;
  const R lam = act ? cell_lambda<R, RT>(A, cells, t, cell, w, R(0)) : rinf<R>();
  int32_t d = 0;   // count - rank
#pragma unroll
  for (uint32_t q = 0; q < 2 * H; ++q) {
    const R other = __shfl(lam, int(q), W);
    if (bool(q & 1u) != neg) d += lam + other < R(0) ? 1 : 0;
    else if (q < k) d -= other <= lam ? 1 : 0;   // earlier: a tie ranks this one behind it
    else if (q > k) d -= lam <= other ? 0 : 1;
  }
  const bool sel = d > 0;
  // U: left +1 and taken -1 entries, V: left -1 and taken +1 entries
  const R v = sel ? -lam : lam;
  R U = sel == neg ? v : rinf<R>(), V = sel == neg ? rinf<R>() : v;
  U = fmin(U, dpp_move<0xB1>(U)), V = fmin(V, dpp_move<0xB1>(V));
  U = fmin(U, dpp_move<0x4E>(U)), V = fmin(V, dpp_move<0x4E>(V));
  U = fmin(U, dpp_move<0x141>(U)), V = fmin(V, dpp_move<0x141>(V));
  if (W > 8) U = fmin(U, dpp_move<0x140>(U)), V = fmin(V, dpp_move<0x140>(V));
  if (act) {
    const R B = sel == neg ? V : U;
    out[cell] = fma_r<R>(-omega, sel ? lam - B : lam + B, lam);
  }
  return sel ? double(lam) : 0.0;
}

// the four waves of a block take adjacent rows of one tile
template <typename R, typename RT, int FORM>
__device__ __forceinline__ double spread_block(const SweepArgs& A, const R* cells, RT t, R* out, R omega,
                                               int32_t item) {
  constexpr int H = TILE_HALF[FORM], BPT = SPREAD<H> / 4, ROWS = 64 / SPREAD<H>;   // blocks per tile, rows per wave
  const int32_t tile = item / BPT;
  if (tile >= A.n_tiles[FORM]) return 0.0;   // uniform across the block
  return tile_spread<R, RT, H>(A, cells, t, out, omega, A.tile_cell0[FORM] + uint32_t(tile) * (128u * H),
                               uint32_t(item % BPT) * (4u * ROWS) + (threadIdx.x >> 6) * ROWS);
}

// ---------------------------------------------------------------- short rows, soft min
// One W-lane segment per row (W = 8, 16, 32 for rows of at most 7, 15, 24
// entries; the rows are taken in order of length from soft_row; a block holds
// soft_rpb<W>() rows).  In the two recursions lane j holds the partial sum
// sigma = j - N:
//   F_{l+1}(sigma) = smin(F_l(sigma), F_l(sigma - a_l) + lam_l),
//   B_l(sigma) = smin(B_{l+1}(sigma), B_{l+1}(sigma + a_l) + lam_l).
// Their tables pass through one LDS table, F first, and then lane l holds entry
// l: its soft-mins for x_l = 0 and 1 run over the states in its own registers,
//   min_sigma F_l(sigma) + B_{l+1}(sigma),  lam_l + min_sigma F_l(sigma) + B_{l+1}(sigma + a_l).
// Bound by vector instructions and, the longest rows first, evenly spread: 1000-
// face pair, a launch 93 us with 46.6 M of them; 119 us with 69.5 M where every
// entry's two soft-mins were reductions over the segment's lanes, entry after
// entry (FP64: 485 and 615 us).  A table each for F and B leaves a CU fewer
// blocks (FP32 119 us against 92, FP64 661 against 592, in one launch order).
// Every sum is formed as those reductions formed it: pairs, fours, eights.
// Rows [row0, row1) of soft_row belong to this width; blk counts the blocks of
// this width, item is the block's index among all blocks.
template <int W>
constexpr int soft_rpb() {   // rows per 256-thread block
  return W == 32 ? 4 : 256 / W;
}
template <int W>
constexpr int soft_nmax() {  // entries per row at most
  return W == 32 ? SOFT_MAX_ROW : W - 1;
}
template <int W>
constexpr int soft_stride() {   // values per table row: 16 lanes' 16-byte reads of 16 rows touch every bank once
  return W == 32 ? 28 : W + 4;
}
// values of one table per block: the largest of the three widths
constexpr int SOFT_TAB = 16 * 15 * 20;
static_assert(soft_rpb<8>() * soft_nmax<8>() * soft_stride<8>() <= SOFT_TAB &&
                  soft_rpb<32>() * soft_nmax<32>() * soft_stride<32>() <= SOFT_TAB && SOFT_MAX_ROW < soft_stride<32>(),
              "table too small");

// orders this wave's LDS accesses (a row's lanes are in one wave)
__device__ inline void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The recursions of one row per W-lane segment where a multiplier passes
// SoftUnits::most in units (1e34 temperatures in FP32): the states that cannot be
// reached are +inf, so that every finite sum counts, and each entry's soft-mins
// are reductions over the lanes, for few registers rather than speed.  Kept out
// of the sweep's own code (1000-face pair, which never comes here: 93.2 us a
// launch against 93.0 without it and 93.9 with it inlined).  lamL: the row's n
// multipliers in units, +inf behind them; neg: its signs; N negative ones, nm
// entries in the wave's longest row.  Returns the row's value; lane l gets entry
// l's soft-mins for x = 1 and 0.
template <typename R, int W>
__device__ __attribute__((noinline)) R soft_states_wide(R* tab, const R* lamL, int lane, int32_t n, int32_t b, uint32_t neg, int32_t N,
                                     int32_t nm, R* my1, R* my0) {
  using U = SoftUnits<R>;
  constexpr int ST = soft_stride<W>();
  auto shifted = [&](R v, int from) {   // v of the segment's lane from, none outside
    const R x = __shfl(v, from & (W - 1), W);
    return from >= 0 && from <= n ? x : rinf<R>();
  };
  auto softmin = [&](R x) {
    R m = x, e;
#pragma unroll 1
    for (int o = 1; o < W; o <<= 1) m = fmin(m, __shfl_xor(m, o, W));
    m = fmin(m, U::big);
    e = U::E(m - x);
#pragma unroll 1
    for (int o = 1; o < W; o <<= 1) e += __shfl_xor(e, o, W);
    return m - U::L(e);
  };
  R F = lane == N ? R(0) : rinf<R>();
#pragma unroll 1
  for (int l = 0; l < nm; ++l) {
    if (W < 32 || lane < ST) tab[l * ST + lane] = F;
    F = smin2u_inf<R>(F, shifted(F, lane - ((neg >> l) & 1u ? -1 : 1)) + lamL[l]);
  }
  wave_lds_fence();
  R Bv = lane - N == b && lane <= n ? R(0) : rinf<R>();
#pragma unroll 1
  for (int l = nm - 1; l >= 0; --l) {
    const R Fl = W < 32 || lane < ST ? tab[l * ST + lane] : rinf<R>();
    const R sh = shifted(Bv, lane + ((neg >> l) & 1u ? -1 : 1));
    const R one = softmin((Fl + lamL[l]) + sh), zero = softmin(Fl + Bv);
    if (lane == l) {
      *my1 = one;
      *my0 = zero;
    }
    Bv = smin2u_inf<R>(Bv, sh + lamL[l]);
  }
  return __shfl(Bv, N, W);
}

template <typename R, int MODE, int W>
__device__ void short_rows_soft(const SweepArgs& A, const R* __restrict__ rin, R* __restrict__ out, R omega,
                                R T, unsigned char* smem, double* red, int32_t item, int32_t blk, int32_t row0,
                                int32_t row1) {
  using U = SoftUnits<R>;
  constexpr int RPB = soft_rpb<W>(), NMAX = soft_nmax<W>(), ST = soft_stride<W>();
  const int seg = threadIdx.x / W, lane = threadIdx.x % W;
  R* tab = reinterpret_cast<R*>(smem) + seg * (NMAX * ST);
  R* lamL = reinterpret_cast<R*>(smem) + SOFT_TAB + seg * W;
  const int32_t r = row0 + blk * RPB + seg;
  const bool act = seg < RPB && r < row1;
  int32_t s = 0, n = 0, b = 0;
  uint32_t w = 0;
  R mylam = R(0);
  double rowpart = 0.0;
  const R unit = U::unit(T), inv_unit = R(1) / unit;
  if (act) {
    const int32_t j = A.soft_row[r];
    s = A.rrow_ptr[j];
    n = A.rrow_ptr[j + 1] - s;
    b = A.rrow_b[j];
    if (lane < n) {
      w = A.ent_word[s + lane];
      mylam = cur_lambda<R>(rin, w);
    }
  }
  lamL[lane] = lane < n ? mylam * inv_unit : rinf<R>();   // past the row's end a step changes nothing
  // signs of the row's entries, and the longest row of the wave (the rows are
  // in order of length, so they hardly differ)
  const unsigned long long neg_wave = __ballot(lane < n && (w >> 31) != 0u);
  const int32_t N = __popc(uint32_t(neg_wave >> ((threadIdx.x & 63u) / W * W)) & (W == 32 ? ~0u : (1u << (W & 31)) - 1u));
  int32_t nm = n;
  for (int off = W; off < 64; off <<= 1) nm = max(nm, __shfl_xor(nm, off));
  nm = __builtin_amdgcn_readfirstlane(nm);
  wave_lds_fence();
  if (__builtin_expect(__any(fabs(mylam) > U::most * unit), 0)) {   // uniform across the wave
    R my1 = R(0), my0 = R(0);
    const R rowv = soft_states_wide<R, W>(tab, lamL, lane, n, b, uint32_t(neg_wave >> ((threadIdx.x & 63u) / W * W)), N, nm,
                                          &my1, &my0);
    if (MODE == MODE_UPDATE && lane < n) write_out<R>(out, w, mylam - omega * ((my1 - my0) * unit));
    if (MODE == MODE_EVAL && lane < n) write_out<R>(out, w, U::E(rowv - my1));
    rowpart = act && lane == 0 ? double(rowv * unit) : 0.0;
  } else {
    // per entry the lanes whose row has it negative, as a mask of the wave
    constexpr unsigned long long LOW = W == 8 ? 0x0101010101010101ull : (W == 16 ? 0x0001000100010001ull : 0x0000000100000001ull);
    unsigned long long neg[NMAX];
#pragma unroll
    for (int l = 0; l < NMAX; ++l) {
      const unsigned long long t = (neg_wave >> l) & LOW;
      neg[l] = (t << W) - t;
    }
    // value of the state above (lanes of up) or below, none past the segment's ends
    auto beside = [&](R v, unsigned long long up) {
      const R lo = dpp_move<0x138>(v), hi = dpp_move<0x130>(v);   // v[lane - 1], v[lane + 1]
      const R x = __builtin_amdgcn_inverse_ballot_w64(up) ? hi : lo;
      return __builtin_amdgcn_inverse_ballot_w64((up & (LOW << (W - 1))) | (~up & LOW)) ? U::none : x;
    };
    constexpr int Q = (W == 32 ? ST : W) / 4;   // states in fours
    R f[4 * Q];   // the entry's F_l of every state
    auto load4 = [](const R* p, R* v) {
      using Vec = typename LdsVec<R>::type;
      constexpr int V = 16 / int(sizeof(R));
#pragma unroll
      for (int g = 0; g < 4; g += V) {
        const Vec x = *reinterpret_cast<const Vec*>(p + g);
#pragma unroll
        for (int u = 0; u < V; ++u) v[g + u] = LdsVec<R>::get(x, u);
      }
    };
    if (MODE != MODE_BOUND) {
      R F = lane == N ? R(0) : U::none;
#pragma unroll
      for (int l = 0; l < NMAX; ++l) {
        if (l >= nm) break;   // uniform
        if (W < 32 || lane < ST) tab[l * ST + lane] = F;
        F = smin2u<R>(F, beside(F, neg[l]) + lamL[l]);
      }
      wave_lds_fence();
      if (lane < n) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          if (4 * q > nm) break;   // uniform: no row of the wave has such states
          load4(tab + lane * ST + 4 * q, f + 4 * q);
        }
      }
      wave_lds_fence();   // the table now takes B
    }
    R Bv = lane - N == b && lane <= n ? R(0) : U::none;
#pragma unroll
    for (int l = NMAX - 1; l >= 0; --l) {
      if (l < nm) {   // uniform
        if (MODE != MODE_BOUND && (W < 32 || lane < ST)) tab[l * ST + lane] = Bv;
        Bv = smin2u<R>(Bv, beside(Bv, ~neg[l]) + lamL[l]);
      }
    }
    // the soft row value B_0(0) sits on lane N
    R rowv = __shfl(Bv, N, W);
    rowv = rowv < U::lim ? rowv : rinf<R>();
    if (MODE != MODE_BOUND) {
      wave_lds_fence();
      if (lane < n) {
        const bool up = !(w >> 31);
        const R* Bl = tab + lane * ST;
        const R mine = lamL[lane];
        R x1[4 * Q];   // the sums for x = 1; f becomes those for x = 0
        R m0 = U::none, m1 = U::none;
        R below = U::none;   // B of the state below the four
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          if (4 * q > nm) break;
          R B[6];
          B[0] = below;
          load4(Bl + 4 * q, B + 1);
          B[5] = q + 1 < Q ? Bl[4 * q + 4] : U::none;
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            R& x = f[4 * q + u];
            x1[4 * q + u] = (x + mine) + (up ? B[u + 2] : B[u]);
            x = x + B[u + 1];
            m0 = fmin(m0, x);
            m1 = fmin(m1, x1[4 * q + u]);
          }
          below = B[4];
        }
        // one exponential per state, added in pairs, fours, eights, ...
        R e0[8], e1[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          e0[q] = e1[q] = R(0);
          if (q < Q && 4 * q <= nm) {
            const R *x = f + 4 * (q < Q ? q : 0), *y = x1 + 4 * (q < Q ? q : 0);
            e0[q] = (U::E(m0 - x[0]) + U::E(m0 - x[1])) + (U::E(m0 - x[2]) + U::E(m0 - x[3]));
            e1[q] = (U::E(m1 - y[0]) + U::E(m1 - y[1])) + (U::E(m1 - y[2]) + U::E(m1 - y[3]));
          }
        }
#pragma unroll
        for (int h = 1; h < W / 4; h *= 2)
#pragma unroll
          for (int q = 0; q < W / 4; q += 2 * h) {
            e0[q] += e0[q + h];
            e1[q] += e1[q + h];
          }
        const R my1 = m1 < U::lim ? m1 - U::L(e1[0]) : rinf<R>();
        const R my0 = m0 < U::lim ? m0 - U::L(e0[0]) : rinf<R>();
        if (MODE == MODE_UPDATE) write_out<R>(out, w, mylam - omega * ((my1 - my0) * unit));
        if (MODE == MODE_EVAL) write_out<R>(out, w, U::E(rowv - my1));
      }
    }
    rowpart = act && lane == 0 ? double(rowv * unit) : 0.0;
  }
  store_partial(block_sum(rowpart, red), A.partial, item);
}

// a multiplier record as loaded (two 16-byte loads for FP32, four for FP64)
template <typename R>
struct RecRaw;
template <>
struct RecRaw<float> {
  float4 lo, hi;
  __device__ void load(const float* __restrict__ rec, uint32_t i) {
    lo = *reinterpret_cast<const float4*>(rec + size_t(i) * REC);
    hi = *reinterpret_cast<const float4*>(rec + size_t(i) * REC + 4);
  }
  // lambda of slot k with dual feasibility restored, in the arithmetic of rec_lambdas
  __device__ float lambda(int k) const {
    const float sum = (((lo.x + lo.y) + lo.z) + lo.w) + hi.x;
    const float corr = (hi.y - sum) * hi.z;
    const float sk = k == 0 ? lo.x : k == 1 ? lo.y : k == 2 ? lo.z : k == 3 ? lo.w : hi.x;
    return sk + corr;
  }
};
template <>
struct RecRaw<double> {
  double2 a, b, c, d;
  __device__ void load(const double* __restrict__ rec, uint32_t i) {
    const double* r = rec + size_t(i) * REC;
    a = *reinterpret_cast<const double2*>(r);
    b = *reinterpret_cast<const double2*>(r + 2);
    c = *reinterpret_cast<const double2*>(r + 4);
    d = *reinterpret_cast<const double2*>(r + 6);
  }
  __device__ double lambda(int k) const {
    const double sum = (((a.x + a.y) + b.x) + b.y) + c.x;
    const double corr = (c.y - sum) * d.x;
    const double sk = k == 0 ? a.x : k == 1 ? a.y : k == 2 ? b.x : k == 3 ? b.y : c.x;
    return sk + corr;
  }
};

// ---------------------------------------------------------------- long rows (exactly one)
template <typename R>
struct MinState {   // hard: (m, a, m2); soft adds s = sum_{k != a} exp(-(lam_k - m2)/T)
  R m, m2, s;
  int32_t a;
};

template <typename R, bool SOFT>
__device__ inline MinState<R> ms_combine(MinState<R> x, MinState<R> y, R T) {
  if (y.m < x.m || (y.m == x.m && y.a < x.a)) {
    MinState<R> t = x;
    x = y;
    y = t;
  }
  MinState<R> r;
  r.m = x.m;
  r.a = x.a;
  r.m2 = x.m2 < y.m ? x.m2 : y.m;
  r.s = R(0);
  if (SOFT && r.m2 != rinf<R>()) {
    R sx = (x.m2 == rinf<R>()) ? R(0) : x.s * r_exp<R>(-(x.m2 - r.m2) / T);
    R ys = (y.m2 == rinf<R>()) ? R(0) : y.s * r_exp<R>(-(y.m2 - y.m) / T);
    R sy = (y.m == rinf<R>()) ? R(0) : (R(1) + ys) * r_exp<R>(-(y.m - r.m2) / T);
    r.s = sx + sy;
  }
  return r;
}

template <typename R, bool SOFT>
__device__ inline MinState<R> ms_shfl_xor(MinState<R> v, int off) {
  MinState<R> o;
  o.m = __shfl_xor(v.m, off);
  o.m2 = __shfl_xor(v.m2, off);
  o.s = SOFT ? __shfl_xor(v.s, off) : R(0);
  o.a = __shfl_xor(v.a, off);
  return o;
}

// The hard minimum and second minimum alone.  Which entry holds the minimum
// needs no index: an entry that equals it either is the only one, or the second
// minimum equals it too.
template <typename R>
struct TwoMin {
  R m, m2;
  __device__ void take(R v) {   // a NaN is passed over
    m2 = fmin(m2, m > v ? m : v);
    m = fmin(m, v);
  }
  __device__ void join(R om, R om2) {
    m2 = fmin(fmax(m, om), fmin(m2, om2));
    m = fmin(m, om);
  }
  template <int CTRL>
  __device__ void join_dpp() {
    join(dpp_move<CTRL>(m), dpp_move<CTRL>(m2));
  }
  // over the first 4, 16 or 64 lanes of every aligned group
  __device__ void join_group(int group) {
    join_dpp<0xB1>();
    join_dpp<0x4E>();
    if (group > 4) {
      join_dpp<0x141>();
      join_dpp<0x140>();
    }
    if (group > 16) {
      join(__shfl_xor(m, 16), __shfl_xor(m2, 16));
      join(__shfl_xor(m, 32), __shfl_xor(m2, 32));
    }
  }
};

// one wave per projection row (four rows per block), or for long rows one
// block per row (long_wpr = 4); each lane keeps up to LONG_REG of its row's
// multipliers in registers between the two passes
constexpr int LONG_REG = 8;
constexpr int32_t LONG_GROUP = 8;   // consecutive projection-row blocks per XCD turn (smoothed)

// Hard: the row's cells d.x .. d.x + d.y - 1 (d from long_row: first cell and
// length, so that the words follow the descriptor at once).  A launch over few
// blocks takes as long as its longest chain of loads and reductions: descriptor,
// words, cells and residuals, six exchange steps of (m, m2), four of them as
// register moves.  With row number, offsets and an exchange of (m, m2, index)
// through the LDS an FP32 iteration of two launches took 7.5-8.1 us with 8k-30k
// entries, 9.4 with 231k; so 6.5-6.8 and 9.1.  In place where cells and dst are
// one array: a lane reads its own cells before it writes them.
// Returns the row minimum on one lane of the row.
template <typename R, typename RT, int MODE>
__device__ __forceinline__ double long_cells(const SweepArgs& A, const R* cells, RT t, R* dst, R omega, R gam,
                                             int32_t lr, bool has) {
  __shared__ R xm[4], xm2[4];
  __shared__ int32_t xa[4];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int wpr = A.long_wpr;   // uniform
  const int sub = wave & (wpr - 1);
  const int2 d = has ? A.long_row[lr] : make_int2(0, 0);
  const uint32_t c0 = uint32_t(d.x);
  const int32_t n = d.y, step = 64 * wpr, i0 = sub * 64 + lane;
  const uint32_t* words = A.word + c0;
  // the first LONG_REG entries of every lane without branches (past the row's
  // end a lane reads the row's first entry and ignores it), the loads of a
  // batch in flight together
  constexpr int BATCH = 4;
  uint32_t wv[LONG_REG];
  R lv[LONG_REG];
#pragma unroll
  for (int u = 0; u < LONG_REG; ++u) {
    const int32_t i = i0 + step * u;
    wv[u] = n > 0 ? words[i < n ? i : 0] : 0u;
  }
  TwoMin<R> st{rinf<R>(), rinf<R>()};
#pragma unroll
  for (int u0 = 0; u0 < LONG_REG; u0 += BATCH) {
    if (sub * 64 + step * u0 >= n) break;   // uniform: no lane of the wave has entries left
#pragma unroll
    for (int u = u0; u < u0 + BATCH; ++u) {
      const int32_t i = i0 + step * u;
      lv[u] = cell_lambda<R, RT>(A, cells, t, c0 + uint32_t(i < n ? i : 0), wv[u], gam);
    }
#pragma unroll
    for (int u = u0; u < u0 + BATCH; ++u)
      if (i0 + step * u < n) st.take(lv[u]);
  }
  auto value = [&](int32_t i) { return cell_lambda<R, RT>(A, cells, t, c0 + uint32_t(i), words[i], gam); };
  for (int32_t i = i0 + step * LONG_REG; i < n; i += step) st.take(value(i));   // longer rows
  st.join_group(64);
  // which of several equal minima a row takes shows only in its assignment: the
  // first in the row's entry order
  int32_t first = INT32_MAX;
  const int32_t* ent = A.long_ent ? A.long_ent + (c0 - A.long_cell0) : nullptr;
  auto place = [&](int32_t i) { return ent ? ent[i] : i; };
  if (wpr > 1) {   // the row's waves join: every wave ends with the same state
    if (lane == 0) {
      xm[wave] = st.m;
      xm2[wave] = st.m2;
    }
    __syncthreads();
    const int w0 = wave & ~(wpr - 1);
    TwoMin<R> all{xm[w0], xm2[w0]};
    for (int q = 1; q < wpr; ++q) all.join(xm[w0 + q], xm2[w0 + q]);
    st = all;
  }
  if constexpr (MODE == MODE_SUBGRAD) {
#pragma unroll
    for (int u = 0; u < LONG_REG; ++u)
      if (i0 + step * u < n && lv[u] == st.m) first = min(first, place(i0 + step * u));
    for (int32_t i = i0 + step * LONG_REG; i < n; i += step)
      if (value(i) == st.m) first = min(first, place(i));
    for (int off = 32; off > 0; off >>= 1) first = min(first, __shfl_xor(first, off));
    if (wpr > 1) {
      if (lane == 0) xa[wave] = first;
      __syncthreads();
      for (int q = 0; q < wpr; ++q) first = min(first, xa[(wave & ~(wpr - 1)) + q]);
    }
  }
  if (MODE != MODE_BOUND) {
    auto finish = [&](int32_t i, R lam) {
      const R M = lam - (lam == st.m ? st.m2 : st.m);
      if (MODE == MODE_UPDATE) dst[c0 + uint32_t(i)] = fma_r<R>(-omega, M, lam);
      if (MODE == MODE_EVAL) dst[c0 + uint32_t(i)] = M;
      if (MODE == MODE_SUBGRAD) A.gsub[c0 + uint32_t(i)] = uint8_t(place(i) == first ? 1 : 0);
    };
#pragma unroll
    for (int u = 0; u < LONG_REG; ++u) {
      const int32_t i = i0 + step * u;
      if (i < n) finish(i, lv[u]);
    }
    for (int32_t i = i0 + step * LONG_REG; i < n; i += step) finish(i, value(i));
  }
  return has && lane == 0 && sub == 0 ? double(st.m) : 0.0;
}

// Smoothed: row lr of the launch order on records; lanes stride the row's
// entries as above.
template <typename R, int MODE>
__device__ double long_records(const SweepArgs& A, const R* __restrict__ src, R* __restrict__ dst, R omega, R T,
                               int32_t lr, bool has) {
  __shared__ R xm[4], xm2[4], xs[4];
  __shared__ int32_t xa[4];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int wpr = A.long_wpr;   // uniform
  const int sub = wave & (wpr - 1);
  const int32_t j = has ? A.n_short + A.long_perm[lr] : 0;
  const int32_t step = 64 * wpr, i0 = sub * 64 + lane;
  const int32_t s = has ? A.rrow_ptr[j] : 0;
  const int32_t n = has ? A.rrow_ptr[j + 1] - s : 0;
  MinState<R> st;
  st.m = rinf<R>();
  st.m2 = rinf<R>();
  st.s = R(0);
  st.a = INT32_MAX;
  const uint32_t* words = A.ent_word + s;
  auto take = [&](int32_t i, R v) {
    MinState<R> one;
    one.m = v;
    one.m2 = rinf<R>();
    one.s = R(0);
    one.a = i;
    st = ms_combine<R, true>(st, one, T);
  };
  constexpr int LONG_BATCH = 2;   // record loads in flight together
  uint32_t wv[LONG_REG];
  R lv[LONG_REG];
#pragma unroll
  for (int u = 0; u < LONG_REG; ++u) {
    const int32_t i = i0 + step * u;
    wv[u] = n > 0 ? words[i < n ? i : 0] : 0u;
  }
#pragma unroll
  for (int u0 = 0; u0 < LONG_REG; u0 += LONG_BATCH) {
    if (sub * 64 + step * u0 >= n) break;   // uniform: no lane of the wave has entries left
    RecRaw<R> raw[LONG_BATCH];
#pragma unroll
    for (int u = 0; u < LONG_BATCH; ++u) raw[u].load(src, wv[u0 + u] & W_VAR_MASK);
#pragma unroll
    for (int u = 0; u < LONG_BATCH; ++u) lv[u0 + u] = raw[u].lambda(int((wv[u0 + u] >> W_SLOT_SHIFT) & 7u));
#pragma unroll
    for (int u = 0; u < LONG_BATCH; ++u) {
      const int32_t i = i0 + step * (u0 + u);
      if (i < n) take(i, lv[u0 + u]);
    }
  }
  for (int32_t i = i0 + step * LONG_REG; i < n; i += step) take(i, cur_lambda<R>(src, words[i]));   // longer rows
  for (int off = 32; off > 0; off >>= 1) st = ms_combine<R, true>(st, ms_shfl_xor<R, true>(st, off), T);
  if (wpr > 1) {
    // the row's waves combine their states in index order: every wave of
    // the row ends with the same state
    if (lane == 0) {
      xm[wave] = st.m;
      xm2[wave] = st.m2;
      xs[wave] = st.s;
      xa[wave] = st.a;
    }
    __syncthreads();
    const int w0 = wave & ~(wpr - 1);
    MinState<R> acc;
    acc.m = xm[w0];
    acc.m2 = xm2[w0];
    acc.s = xs[w0];
    acc.a = xa[w0];
    for (int q = 1; q < wpr; ++q) {
      MinState<R> o;
      o.m = xm[w0 + q];
      o.m2 = xm2[w0 + q];
      o.s = xs[w0 + q];
      o.a = xa[w0 + q];
      acc = ms_combine<R, true>(acc, o, T);
    }
    st = acc;
  }
  double rowpart = 0.0;
  if (has) {
    const R tot = (st.m2 == rinf<R>()) ? R(0) : st.s * r_exp<R>(-(st.m2 - st.m) / T);
    const R rowv = st.m - T * r_log<R>(R(1) + tot);
    if (MODE != MODE_BOUND) {
      auto finish = [&](int32_t i, uint32_t w, R lam) {
        R others;
        if (i == st.a) {
          others = st.m2 - T * r_log<R>(st.s);
        } else {
          R e = r_exp<R>(-(lam - st.m) / T);
          others = st.m - T * r_log<R>((R(1) + tot) - e);
        }
        const R M = lam - others;
        if (MODE == MODE_UPDATE) write_out<R>(dst, w, lam - omega * M);
        if (MODE == MODE_EVAL) write_out<R>(dst, w, r_exp<R>(-(lam - rowv) / T));
      };
#pragma unroll
      for (int u = 0; u < LONG_REG; ++u) {
        const int32_t i = i0 + step * u;
        if (i < n) finish(i, wv[u], lv[u]);
      }
      for (int32_t i = i0 + step * LONG_REG; i < n; i += step) {
        const uint32_t w = words[i];
        finish(i, w, cur_lambda<R>(src, w));
      }
    }
    if (lane == 0 && sub == 0) rowpart = double(rowv);
  }
  return rowpart;
}

template <typename R, bool SOFT>
constexpr size_t smem_bytes() {
  return SOFT ? (SOFT_TAB + 256) * sizeof(R) : 4 * CHUNK_SLICE * sizeof(R);
}

// First pass of a hard iteration: t_i = c_i - sum_k s_k, one thread per
// variable in variable order; unused slots read the zero cell.  Bound by the
// index planes and the gathered lines (2000/3000-face pair: 20 + 16 bytes per
// variable, 43 us, 5 TB/s; 9 us more with the variables in canonical order).
// Blocks 8 and up take the variables, each XCD a contiguous eighth; block 0
// sums the previous row pass's partials, so that no other launch has to.
template <typename R>
__global__ __launch_bounds__(256) void k_vars(const uint32_t* __restrict__ vpos, const R* __restrict__ cells,
                                              const R* __restrict__ cost, int64_t n, int32_t per, R* __restrict__ t,
                                              const double* prev_partial, int32_t prev_n, double prev_offset,
                                              double* prev_out) {
  __shared__ double red[4];
  if (blockIdx.x < 8) {
    if (blockIdx.x == 0 && prev_partial) reduce_partials(prev_partial, prev_n, prev_offset, prev_out, red);
    return;
  }
  const int32_t k = int32_t(blockIdx.x / 8u) - 1;
  const int64_t v = (int64_t(blockIdx.x % 8u) * per + k) * 256 + threadIdx.x;
  if (v >= n) return;
  uint32_t p[5];
#pragma unroll
  for (int q = 0; q < 5; ++q) p[q] = vpos[size_t(q) * n + v];
  const R c = cost[v];
  R s[5];
#pragma unroll
  for (int q = 0; q < 5; ++q) s[q] = cells[p[q]];
  t[v] = c - ((((s[0] + s[1]) + s[2]) + s[3]) + s[4]);
}

// the terms of the tile rows of a block to their places
template <int FORM>
__device__ __forceinline__ void tile_term(const SweepArgs& A, double part, int32_t item) {
  if (!A.terms) return;   // uniform
  const int32_t row0 = (FORM > 0 ? A.tile_rows[0] : 0) + (FORM > 1 ? A.tile_rows[1] : 0);
  const int32_t r = item * 256 + int32_t(threadIdx.x);
  if (r < A.tile_rows[FORM]) A.terms[A.term_row[row0 + r]] = part;
}

// block k of XCD x of the hard row pass: the sum of its row minima, in parts
template <typename R, typename RT, int MODE, bool SPREAD_TILES>
__device__ __forceinline__ double hard_block(SweepArgs A, const R* cells, RT t, R* out, R omega, R gam,
                                             unsigned char* smem, int32_t x, int32_t k) {
  // Every XCD takes a contiguous eighth of each kind of rows, the heavier
  // kinds first.  (Y projection rows too: they span all variables, but
  // neighbouring rows need neighbouring ones of them.)
  const int wave = threadIdx.x >> 6;
  constexpr bool TERMS = sizeof(R) == 8 && (MODE == MODE_BOUND || MODE == MODE_SUBGRAD);
  double part = 0.0;
  if (k < A.per[0] + A.per[1]) {
    const bool yrow = k < A.per[0];
    const int32_t rpb = 4 / A.long_wpr;
    const int32_t item = yrow ? x * A.per[0] + k : x * A.per[1] + (k - A.per[0]);
    const int32_t r = item * rpb + wave / A.long_wpr;
    const int32_t lr = yrow ? r : A.n_long_y + r;
    const bool has = lr < (yrow ? A.n_long_y : A.n_long);
    part = long_cells<R, RT, MODE>(A, cells, t, out, omega, gam, lr, has);
    if constexpr (TERMS)
      if (A.terms && has && (threadIdx.x & (64 * A.long_wpr - 1)) == 0) A.terms[A.term_long0 + A.term_long[lr]] = part;
  } else if ((k -= A.per[0] + A.per[1]) < A.per[2]) {
    part = chunk_block<R, RT, MODE>(A, cells, t, out, omega, gam, smem, x * A.per[2] + k);
    if constexpr (TERMS) {
      const int32_t c = (x * A.per[2] + k) * 4 + wave;
      if (A.terms && c < A.n_chunks) A.terms[A.term_chunk0 + c * 64 + int32_t(threadIdx.x & 63)] = part;
    }
  } else if ((k -= A.per[2]) < A.per[3]) {
    if constexpr (SPREAD_TILES) part = spread_block<R, RT, 2>(A, cells, t, out, omega, x * A.per[3] + k);
    else part = tile_block<R, RT, MODE, 2>(A, cells, t, out, omega, gam, x * A.per[3] + k);
    if constexpr (TERMS) tile_term<2>(A, part, x * A.per[3] + k);
  } else if ((k -= A.per[3]) < A.per[4]) {
    if constexpr (SPREAD_TILES) part = spread_block<R, RT, 1>(A, cells, t, out, omega, x * A.per[4] + k);
    else part = tile_block<R, RT, MODE, 1>(A, cells, t, out, omega, gam, x * A.per[4] + k);
    if constexpr (TERMS) tile_term<1>(A, part, x * A.per[4] + k);
  } else {
    if constexpr (SPREAD_TILES) part = spread_block<R, RT, 0>(A, cells, t, out, omega, x * A.per[5] + (k - A.per[4]));
    else part = tile_block<R, RT, MODE, 0>(A, cells, t, out, omega, gam, x * A.per[5] + (k - A.per[4]));
    if constexpr (TERMS) tile_term<0>(A, part, x * A.per[5] + (k - A.per[4]));
  }
  return part;
}

template <typename R, bool SOFT, int MODE>
__global__ __launch_bounds__(256) void k_sweep(SweepArgs A, const R* rin, const R* __restrict__ t, R* out, R omega,
                                               R T) {
  __shared__ __align__(16) unsigned char smem[smem_bytes<R, SOFT>()];
  __shared__ double red[256];
  if (A.skip && *A.skip) return;   // uniform across the grid
  if (SOFT && blockIdx.x == 0 && A.prev_partial)
    reduce_partials(A.prev_partial, A.prev_n, A.prev_offset, A.prev_out, red);
  // Workgroups are dealt to the 8 XCDs round-robin (block b runs on XCD b % 8).
  const int32_t x = int32_t(blockIdx.x % 8u), k0 = int32_t(blockIdx.x / 8u);
  if constexpr (!SOFT) {
    const R gam = A.gamma ? R(*A.gamma) : R(0);
    const double part = hard_block<R, Written<R>, MODE, false>(A, rin, t, out, omega, gam, smem, x, k0);
    store_partial(block_sum(part, red), A.partial, int32_t(blockIdx.x));
  } else {
    // The smoothed form deals the projection-row blocks in groups of LONG_GROUP,
    // group g to XCD g % 8, then the short rows' blocks one by one, the widest
    // rows first.  Each width is dealt by itself and in order of length, so that
    // a wave's rows are equally long and the XCDs get equal work (contiguous
    // eighths of all short rows in order of length: half the chip was idle at the
    // end, 1000-face pair 119 us a launch against 90).
    int32_t item;
    const int32_t n_long_blocks = A.n_items - A.n_short_blocks;
    const int32_t lx = (n_long_blocks + 8 * LONG_GROUP - 1) / (8 * LONG_GROUP) * LONG_GROUP;
    const int32_t nb8 = (A.soft_c8 + soft_rpb<8>() - 1) / soft_rpb<8>();
    const int32_t nb16 = (A.soft_c16 + soft_rpb<16>() - 1) / soft_rpb<16>();
    if (k0 < lx) {
      const int32_t li = ((k0 / LONG_GROUP) * 8 + x) * LONG_GROUP + k0 % LONG_GROUP;
      if (li >= n_long_blocks) return;
      item = A.n_short_blocks + li;
    } else {
      item = A.n_short_blocks - 1 - ((k0 - lx) * 8 + x);   // in order of length: the longest are the last
      if (item < 0) return;
    }
    if (item < A.n_short_blocks) {
      const int32_t c816 = A.soft_c8 + A.soft_c16;
      if (item < nb8)
        short_rows_soft<R, MODE, 8>(A, rin, out, omega, T, smem, red, item, item, 0, A.soft_c8);
      else if (item < nb8 + nb16)
        short_rows_soft<R, MODE, 16>(A, rin, out, omega, T, smem, red, item, item - nb8, A.soft_c8, c816);
      else
        short_rows_soft<R, MODE, 32>(A, rin, out, omega, T, smem, red, item, item - nb8 - nb16, c816, A.n_short);
    } else {
      const int32_t lr = (item - A.n_short_blocks) * (4 / A.long_wpr) + int32_t(threadIdx.x >> 6) / A.long_wpr;
      const double part = long_records<R, MODE>(A, rin, out, omega, T, lr, lr < A.n_long);
      store_partial(block_sum(part, red), A.partial, item);
    }
  }
}

// ---------------------------------------------------------------- middle sizes: one launch per iteration
// Hard iteration in one launch, from one cell buffer to the other: each entry
// forms its variable's residual itself, from the cost and the old cells, with the
// additions of the variable pass (same bits).  The gathers are five times as many,
// but a launch less is what counts as long as the iteration is a chain of launches
// (hard_form).  With a lane per row the gathers of a tile are one lane's chain:
// 101k entries 16.4 us an iteration so, 5.9 with a lane per entry (tile_spread).
// Blocks 8 and up take the rows; block 0 sums the previous launch's partials.
template <typename R>
__global__ __launch_bounds__(256) void k_iterate(SweepArgs A, const R* __restrict__ cells,
                                                 const uint32_t* __restrict__ vpos, const R* __restrict__ cost,
                                                 uint32_t n, R* __restrict__ out, R omega) {
  __shared__ __align__(16) unsigned char smem[smem_bytes<R, false>()];
  __shared__ double red[4];
  if (blockIdx.x < 8) {
    if (blockIdx.x == 0 && A.prev_partial)
      reduce_partials(A.prev_partial, A.prev_n, A.prev_offset, A.prev_out, red);
    return;
  }
  const Summed<R> t{vpos, cells, cost, n};
  const double part = hard_block<R, Summed<R>, MODE_UPDATE, true>(A, cells, t, out, omega, R(0), smem,
                                                                  int32_t(blockIdx.x % 8u), int32_t(blockIdx.x / 8u) - 1);
  store_partial(block_sum(part, red), A.partial, int32_t(blockIdx.x) - 8);
}

// ---------------------------------------------------------------- small problems: one workgroup
// A problem whose cells and residuals fit one CU's LDS runs all its iterations
// in one launch of one workgroup: the two passes alternate between barriers
// (some 0.1 us) instead of launches (2.4 to 3 us each, which is nearly all of a
// small problem's iteration).  The values are those of the two-launch form; the
// bound sums the waves' row minima in wave order.
// Exactly-one rows take a group of 4, 16 or 64 lanes each, a quarter of their
// mean length, so that a lane holds about four entries of its row.
// As many waves as their registers leave room for without spilling.
template <typename R>
constexpr int SMALL_THREADS = sizeof(R) == 4 ? 768 : 512;
constexpr int SMALL_LREG = 4;

template <typename R, int NT>
__global__ __launch_bounds__(NT) void k_small(SweepArgs A, const uint32_t* __restrict__ vpos, R* gcells,
                                              const R* __restrict__ cost, int32_t n, uint32_t n_cells, int32_t iters,
                                              R omega, double offset, int32_t group, double* trace) {
  extern __shared__ __align__(16) unsigned char lds[];
  A.dir = nullptr;   // a constant from here on
  __shared__ double part[2][NT / 64];
  R* cells = reinterpret_cast<R*>(lds);
  R* t = cells + n_cells + 1;
  R* wave_vals = cells + small_slices_at<R>(n_cells, n) + (threadIdx.x >> 6) * CHUNK_SLICE;   // chunks only
  constexpr int NW = NT / 64;
  const int tid = int(threadIdx.x), wave = tid >> 6, lane = tid & 63;
  for (uint32_t c = uint32_t(tid); c <= n_cells; c += NT) cells[c] = gcells[c];
  // the first two variables of every thread keep their cell indices in registers
  constexpr int KEEP = sizeof(R) == 4 ? 2 : 1;
  uint32_t kp[KEEP][5];
  R kc[KEEP];
#pragma unroll
  for (int u = 0; u < KEEP; ++u) {
    const int32_t v = tid + u * NT;
#pragma unroll
    for (int q = 0; q < 5; ++q) kp[u][q] = v < n ? vpos[size_t(q) * n + v] : n_cells;
    kc[u] = v < n ? cost[v] : R(0);
  }
  __syncthreads();
#pragma unroll 1
  for (int32_t it = 0; it < iters; ++it) {
#pragma unroll
    for (int u = 0; u < KEEP; ++u) {
      const int32_t v = tid + u * NT;
      R s[5];
#pragma unroll
      for (int q = 0; q < 5; ++q) s[q] = cells[kp[u][q]];
      if (v < n) t[v] = kc[u] - ((((s[0] + s[1]) + s[2]) + s[3]) + s[4]);
    }
    for (int32_t v = tid + KEEP * NT; v < n; v += NT) {
      R s[5];
#pragma unroll
      for (int q = 0; q < 5; ++q) s[q] = cells[vpos[size_t(q) * n + v]];
      t[v] = cost[v] - ((((s[0] + s[1]) + s[2]) + s[3]) + s[4]);
    }
    __syncthreads();
    double sum = 0.0;
    int32_t w0 = wave;   // the waves take the items of all kinds in turn
#pragma unroll 1
    for (; w0 < A.n_tiles[2]; w0 += NW)
      sum += tile_rows<R, Written<R>, MODE_UPDATE, TILE_HALF[2]>(A, cells, t, cells, omega, R(0),
                                                     A.tile_cell0[2] + uint32_t(w0) * (128u * TILE_HALF[2]));
    w0 -= A.n_tiles[2];
#pragma unroll 1
    for (; w0 < A.n_chunks; w0 += NW)
      sum += short_chunk_hard<R, Written<R>, MODE_UPDATE>(A, cells, t, cells, omega, R(0), w0, wave_vals);
    w0 -= A.n_chunks;
#pragma unroll 1
    for (; w0 < A.n_tiles[1]; w0 += NW)
      sum += tile_rows<R, Written<R>, MODE_UPDATE, TILE_HALF[1]>(A, cells, t, cells, omega, R(0),
                                                     A.tile_cell0[1] + uint32_t(w0) * (128u * TILE_HALF[1]));
    w0 -= A.n_tiles[1];
#pragma unroll 1
    for (; w0 < A.n_tiles[0]; w0 += NW)
      sum += tile_rows<R, Written<R>, MODE_UPDATE, TILE_HALF[0]>(A, cells, t, cells, omega, R(0),
                                                     A.tile_cell0[0] + uint32_t(w0) * (128u * TILE_HALF[0]));
    w0 -= A.n_tiles[0];
    const int32_t rpw = 64 / group;
#pragma unroll 1
    for (; w0 * rpw < A.n_long; w0 += NW) {
      const int32_t lr = w0 * rpw + lane / group, i0 = lane & (group - 1);
      const bool has = lr < A.n_long;
      const int2 d = has ? A.long_row[lr] : make_int2(0, 0);
      const uint32_t c0 = uint32_t(d.x);
      const int32_t len = d.y;
      auto value = [&](int32_t i) { return cell_lambda<R, Written<R>>(A, cells, t, c0 + uint32_t(i), A.word[c0 + uint32_t(i)], R(0)); };
      R lv[SMALL_LREG];
      TwoMin<R> st{rinf<R>(), rinf<R>()};
#pragma unroll
      for (int u = 0; u < SMALL_LREG; ++u) {
        const int32_t i = i0 + u * group;
        lv[u] = i < len ? value(i) : rinf<R>();
      }
#pragma unroll
      for (int u = 0; u < SMALL_LREG; ++u) st.take(lv[u]);
      for (int32_t i = i0 + SMALL_LREG * group; i < len; i += group) st.take(value(i));
      st.join_group(group);
      auto finish = [&](int32_t i, R v) {
        cells[c0 + uint32_t(i)] = fma_r<R>(-omega, v - (v == st.m ? st.m2 : st.m), v);
      };
#pragma unroll
      for (int u = 0; u < SMALL_LREG; ++u) {
        const int32_t i = i0 + u * group;
        if (i < len) finish(i, lv[u]);
      }
      for (int32_t i = i0 + SMALL_LREG * group; i < len; i += group) finish(i, value(i));
      if (has && i0 == 0) sum += double(st.m);
    }
    if (trace) {
      sum = wave_sum(sum);
      if (lane == 0) part[it & 1][wave] = sum;
    }
    __syncthreads();
    if (trace && tid == 0) {
      double b = part[it & 1][0];
#pragma unroll
      for (int w = 1; w < NW; ++w) b += part[it & 1][w];
      trace[it] = offset + b;
    }
  }
  for (uint32_t c = uint32_t(tid); c < n_cells; c += NT) gcells[c] = cells[c];
}

// ---------------------------------------------------------------- state import / export (records)
template <typename R>
__global__ void k_rec_import(const R* lam, const uint32_t* word, int64_t nnz, R* rec) {
  int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e < nnz) write_out<R>(rec, word[e], lam[e]);
}

template <typename R>
__global__ void k_rec_cost(const int32_t* free_var, const double* c64, const uint8_t* deg, int64_t nfree, R* rec0,
                           R* rec1) {
  int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= nfree) return;
  const R c = R(c64[free_var[i]]), rd = R(1) / R(deg[i]);
  rec0[size_t(i) * REC + REC_COST] = c;
  rec0[size_t(i) * REC + REC_RDEG] = rd;
  if (rec1) {
    rec1[size_t(i) * REC + REC_COST] = c;
    rec1[size_t(i) * REC + REC_RDEG] = rd;
  }
}

template <typename R>
__global__ void k_rec_export(const R* rec, const uint32_t* word, int64_t nnz, R* lam) {
  int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e < nnz) lam[e] = cur_lambda<R>(rec, word[e]);
}

// ---------------------------------------------------------------- state import / export (cells)
// entries' multipliers into their cells, costs in variable order, the zero cell
template <typename R>
__global__ void k_cell_import(const R* lam, const uint32_t* ent_cell, int64_t nnz, const int32_t* vperm,
                              const int32_t* free_var, const double* c64, int64_t n, uint32_t zero_cell, R* cells,
                              R* other, R* cost) {
  const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e < nnz) cells[ent_cell[e]] = lam[e];
  if (e < n) cost[e] = R(c64[free_var[vperm[e]]]);
  if (e == 0) {
    cells[zero_cell] = R(0);
    if (other) other[zero_cell] = R(0);   // its other cells are written before they are read
  }
}

// multipliers in entry order, with dual feasibility restored; block 0 sums the
// previous launch's partials where there are any (the others then start behind it)
template <typename R, typename RT>
__global__ __launch_bounds__(256) void k_cell_export(const R* cells, RT t, const uint32_t* ent_cell, const uint32_t* word,
                                                     int64_t nnz, R* lam, const double* prev_partial, int32_t prev_n,
                                                     double prev_offset, double* prev_out) {
  __shared__ double red[4];
  if (prev_partial && blockIdx.x == 0) {
    reduce_partials(prev_partial, prev_n, prev_offset, prev_out, red);
    return;
  }
  const int64_t e = (int64_t(blockIdx.x) - (prev_partial ? 1 : 0)) * blockDim.x + threadIdx.x;
  if (e >= nnz) return;
  const uint32_t c = ent_cell[e], w = word[c];
  lam[e] = feasible<R>(cells[c], t[w & W_VAR_MASK], rdeg_of<R>(w));
}

// c_i / |J_i| per variable, then per entry: the division and the two gathers
// behind the cost run once per variable, not per entry (157 us at the
// 2000/3000-face pair when they ran per entry).  Up to INIT_ENTRY_NNZ entries one
// launch that does so per entry is as good as the launch that it saves: 8.1
// against 10.3 us with 2k to 690k entries, 19.2 against 13.6 with 2.6 M.
constexpr int64_t INIT_ENTRY_NNZ = 1000000;

template <typename R>
__global__ void k_init_entry(const uint32_t* word, const int32_t* free_var, const double* c64, const uint8_t* deg,
                             int64_t nnz, R* lam) {
  const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= nnz) return;
  const uint32_t i = word[e] & W_VAR_MASK;
  lam[e] = R(c64[free_var[i]]) / R(deg[i]);
}

template <typename R>
__global__ void k_share(const int32_t* free_var, const double* c64, const uint8_t* deg, int64_t n, R* share) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) share[i] = R(c64[free_var[i]]) / R(deg[i]);
}

template <typename R>
__global__ void k_init_lambda(const uint32_t* word, const R* share, int64_t nnz, R* lam) {
  const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e < nnz) lam[e] = share[word[e] & W_VAR_MASK];
}

__global__ void k_write_offset(double* out, int32_t n, double v) {
  const int32_t i = int32_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) out[i] = v;
}

__global__ __launch_bounds__(256) void k_reduce_last(const double* partial, int n, double offset, double* out) {
  __shared__ double red[256];
  reduce_partials(partial, n, offset, out, red);
}

}  // namespace

// ============================================================================
// host side (shared with rounding, the quasi-Newton layer and the backward pass)
// ============================================================================
// blocks per XCD of each kind of rows of the hard sweep, in launch order
static void hard_blocks(const dm_ctx* ctx, bool spread, int32_t per[3 + TILE_FORMS]) {
  const int64_t n_long = ctx->n_rows - ctx->n_short, rpb = 4 / ctx->long_wpr;
  const auto xcd = [](int64_t items) { return int32_t((items + 7) / 8); };
  per[0] = xcd((ctx->n_long_y + rpb - 1) / rpb);
  per[1] = xcd((n_long - ctx->n_long_y + rpb - 1) / rpb);
  per[2] = xcd((ctx->n_chunks + 3) / 4);
  constexpr int BPT[TILE_FORMS] = {SPREAD<TILE_HALF[0]> / 4, SPREAD<TILE_HALF[1]> / 4, SPREAD<TILE_HALF[2]> / 4};
  for (int f = TILE_FORMS - 1; f >= 0; --f)
    per[2 + TILE_FORMS - f] = xcd(spread ? int64_t(ctx->n_tiles[f]) * BPT[f] : (ctx->n_tiles[f] + 3) / 4);
}

static int64_t hard_grid(const dm_ctx* ctx, bool spread = false) {
  int32_t per[3 + TILE_FORMS];
  hard_blocks(ctx, spread, per);
  int64_t n = 0;
  for (int32_t p : per) n += p;
  return 8 * n;
}

static int64_t soft_short_blocks(const dm_ctx* ctx) {
  const int64_t c32 = ctx->n_short - ctx->soft_c8 - ctx->soft_c16;
  return (ctx->soft_c8 + soft_rpb<8>() - 1) / soft_rpb<8>() + (ctx->soft_c16 + soft_rpb<16>() - 1) / soft_rpb<16>() +
         (c32 + soft_rpb<32>() - 1) / soft_rpb<32>();
}

static int64_t long_blocks(const dm_ctx* ctx) {
  const int64_t rpb = 4 / ctx->long_wpr;
  return (ctx->n_rows - ctx->n_short + rpb - 1) / rpb;
}

// per-launch partials of one sweep (hard and smoothed forms): the partial
// buffer holds two halves of this many doubles
static int64_t sweep_partial_cap(const dm_ctx* ctx) {
  const bool spread = ctx->nnz <= ONE_LAUNCH_NNZ;
  return std::max<int64_t>(hard_grid(ctx, spread), soft_short_blocks(ctx) + long_blocks(ctx));
}

static size_t align256(size_t b) { return (b + 255) / 256 * 256; }

SolverLayout solver_layout(const dm_ctx* ctx, size_t real_bytes) {
  SolverLayout L;
  const size_t n = size_t(std::max<int64_t>(ctx->n_free, 1));
  L.rec_bytes = align256(n * REC * real_bytes);
  L.cell_bytes = align256(size_t(ctx->n_cells + 1) * real_bytes);
  L.var_bytes = align256(n * real_bytes);
  L.part_off = std::max(2 * L.rec_bytes, 2 * L.cell_bytes + 3 * L.var_bytes);
  L.part_count = size_t(2 * std::max<int64_t>(sweep_partial_cap(ctx), 1));
  L.total = L.part_off + align256(L.part_count * sizeof(double));
  return L;
}

// the caller's workspace of this precision, checked against the current
// problem (NULL when none is attached)
static dm_status solver_workspace(dm_ctx* ctx, size_t real_bytes, unsigned char** base, SolverLayout* L) {
  const int k = real_bytes == 4 ? 0 : 1;
  *base = static_cast<unsigned char*>(ctx->ws_ptr[k]);
  *L = solver_layout(ctx, real_bytes);
  if (*base && ctx->ws_bytes[k] < L->total)
    return dm_fail(ctx, DM_ERR_WORKSPACE, "the attached %s solver workspace has %zu bytes; the current problem needs %zu",
                   k == 0 ? "FP32" : "FP64", ctx->ws_bytes[k], L->total);
  return DM_OK;
}

// Which form runs the hard iterations of a problem, by its entries.  An iteration
// in us, of 190 in one call.  One workgroup against one launch per iteration: FP32
// 1934 entries 2.8 and 4.5, 3782 4.1 and 4.4, 5844 4.5 and 4.6, 6983 5.7 and 4.5;
// FP64 1934 3.9 and 4.8, 3649 4.9 and 5.0, 3782 5.7 and 5.1, 5844 6.7 and 4.9.  One
// launch against two: FP32 10k 4.8 and 6.7 to 7.4, 45k 5.9 and 7.4, 101k 5.9 and
// 7.8, 168k 7.1 and 8.1, 206k 10.4 and 8.7, 349k 9.9 and 8.9; FP64 10k 5.4 and 7.5,
// 168k 8.2 and 9.0, 206k 10.7 and 9.5.  (Two launches are bound by the host, 3.6 us
// each, up to some 100k entries; beside the launch one launch saves the last
// variable pass of a call, and five gathers per entry are what it costs.)
enum HardForm { ONE_WORKGROUP, ONE_LAUNCH, TWO_PASSES };

// LDS of the one-workgroup form
template <typename R>
static int64_t small_lds(const dm_ctx* ctx) {
  return small_reals<R>(ctx->n_cells, ctx->n_free, ctx->n_chunks > 0, SMALL_THREADS<R> / 64) * int64_t(sizeof(R));
}

template <typename R>
static HardForm hard_form(const dm_ctx* ctx) {
  constexpr int F = sizeof(R) == 4 ? 0 : 1;
  if (ctx->nnz <= SMALL_NNZ[F] && small_lds<R>(ctx) <= SMALL_LDS) return ONE_WORKGROUP;
  return ctx->nnz <= ONE_LAUNCH_NNZ ? ONE_LAUNCH : TWO_PASSES;
}

template <typename R>
dm_status cells_import(dm_ctx* ctx, const R* lam, CellState& S, bool two) {
  const int64_t n = ctx->n_free;
  two = two || hard_form<R>(ctx) == ONE_LAUNCH;   // whose iterations alternate
  const size_t cb = size_t(ctx->n_cells + 1) * sizeof(R), vb = size_t(std::max<int64_t>(n, 1)) * sizeof(R);
  unsigned char* ws = nullptr;
  SolverLayout L;
  if (&S == &ctx->cells) DM_TRY(solver_workspace(ctx, sizeof(R), &ws, &L));
  for (int b = 0; b < (two ? 2 : 1); ++b) {
    if (ws) {   // the solver's state lives in the caller's workspace
      S.cell[b].attach(ws + b * L.cell_bytes, cb);
      S.t[b].attach(ws + 2 * L.cell_bytes + b * L.var_bytes, vb);
    } else {
      DM_ALLOC(ctx, S.cell[b], cb);
      DM_ALLOC(ctx, S.t[b], vb);
    }
  }
  if (ws) S.cost.attach(ws + 2 * L.cell_bytes + 2 * L.var_bytes, vb);
  else DM_ALLOC(ctx, S.cost, vb);
  const int64_t m = std::max<int64_t>(std::max<int64_t>(ctx->nnz, n), 1);
  k_cell_import<R><<<grid_for(m, 256), 256, 0, ctx->stream>>>(
      lam, ctx->ent_cell.p, ctx->nnz, ctx->vperm.p, ctx->free_var.p, ctx->cost64.p, n, uint32_t(ctx->n_cells),
      S.cells<R>(0), two ? S.cells<R>(1) : nullptr, S.costs<R>());
  DM_LAUNCH_CHECK(ctx);
  return DM_OK;
}

template <typename R>
dm_status cells_export(dm_ctx* ctx, const R* cells, const R* t, R* lam) {
  if (ctx->nnz > 0)
    k_cell_export<R, const R*><<<grid_for(ctx->nnz, 256), 256, 0, ctx->stream>>>(
        cells, t, ctx->ent_cell.p, ctx->cell_word.p, ctx->nnz, lam, nullptr, 0, 0.0, nullptr);
  DM_LAUNCH_CHECK(ctx);
  return DM_OK;
}

template <typename R>
dm_status records_import(dm_ctx* ctx, const R* lam, DArr<unsigned char>* bufs) {
  const size_t bytes = size_t(std::max<int64_t>(ctx->n_free, 1)) * REC * sizeof(R);
  unsigned char* ws = nullptr;
  SolverLayout L;
  if (bufs == ctx->rec) DM_TRY(solver_workspace(ctx, sizeof(R), &ws, &L));
  if (ws) {   // the solver's records live in the caller's workspace
    bufs[0].attach(ws, bytes);
    bufs[1].attach(ws + L.rec_bytes, bytes);
  } else {
    DM_ALLOC(ctx, bufs[0], bytes);
    DM_ALLOC(ctx, bufs[1], bytes);
  }
  DM_HIP(ctx, hipMemsetAsync(bufs[0].p, 0, bytes, ctx->stream));
  DM_HIP(ctx, hipMemsetAsync(bufs[1].p, 0, bytes, ctx->stream));
  R* r0 = reinterpret_cast<R*>(bufs[0].p);
  R* r1 = reinterpret_cast<R*>(bufs[1].p);
  if (ctx->n_free > 0)
    k_rec_cost<R><<<grid_for(ctx->n_free, 256), 256, 0, ctx->stream>>>(ctx->free_var.p, ctx->cost64.p,
                                                                       ctx->var_deg.p, ctx->n_free, r0, r1);
  if (ctx->nnz > 0)
    k_rec_import<R><<<grid_for(ctx->nnz, 256), 256, 0, ctx->stream>>>(lam, ctx->rent_word.p, ctx->nnz, r0);
  DM_LAUNCH_CHECK(ctx);
  return DM_OK;
}

template <typename R>
dm_status records_export(dm_ctx* ctx, const unsigned char* rec, R* lam) {
  if (ctx->nnz > 0)
    k_rec_export<R><<<grid_for(ctx->nnz, 256), 256, 0, ctx->stream>>>(reinterpret_cast<const R*>(rec),
                                                                  ctx->rent_word.p, ctx->nnz, lam);
  DM_LAUNCH_CHECK(ctx);
  return DM_OK;
}

// the half of the partial buffer the next launch writes; two halves of it
// alternate between consecutive launches, and with a caller workspace of this
// precision they live there
static dm_status next_partials(dm_ctx* ctx, size_t real_bytes, double** mine) {
  const int64_t cap = sweep_partial_cap(ctx);
  unsigned char* ws = nullptr;
  SolverLayout L;
  DM_TRY(solver_workspace(ctx, real_bytes, &ws, &L));
  if (ws) {
    double* want = reinterpret_cast<double*>(ws + L.part_off);
    if (ctx->partial.p != want || ctx->partial.n < size_t(2 * cap)) {
      DM_TRY(dual_flush(ctx));
      ctx->partial.attach(want, L.part_count);
    }
  } else if (ctx->partial.view || ctx->partial.n < size_t(2 * cap)) {
    DM_TRY(dual_flush(ctx));
    DM_ALLOC(ctx, ctx->partial, size_t(2 * cap));
  }
  *mine = ctx->partial.p + (ctx->pend_half ^ 1) * cap;
  return DM_OK;
}

static void pend(dm_ctx* ctx, double* mine, int64_t n, double* bound_out) {
  ctx->pend_half ^= 1;
  ctx->pend_partial = mine;
  ctx->pend_n = int32_t(n);
  ctx->pend_offset = ctx->offset;
  ctx->pend_out = bound_out;
}

// timing: start and stop event of the next kernel (the runtime records the
// kernel's own start and end), which ends so many sweeps
static dm_status timing_events(dm_ctx* ctx, hipEvent_t* e0, hipEvent_t* e1, int64_t sweeps) {
  while (ctx->ev_pool.size() < ctx->ev_used + 2) {
    hipEvent_t e;
    DM_HIP(ctx, hipEventCreate(&e));
    ctx->ev_pool.push_back(e);
  }
  *e0 = ctx->ev_pool[ctx->ev_used];
  *e1 = ctx->ev_pool[ctx->ev_used + 1];
  ctx->ev_used += 2;
  ctx->ev_sweeps += sweeps;
  return DM_OK;
}

// t of every variable from the cells; takes over the bound of the last row
// pass that has not been summed yet.  sweep: a row pass follows, which counts it
// as its own (timing)
template <typename R>
dm_status cells_vars(dm_ctx* ctx, const R* cells, const R* cost, R* t, bool sweep) {
  const int64_t n = ctx->n_free;
  const int32_t per = int32_t((n + 8 * 256 - 1) / (8 * 256));
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (ctx->timing && sweep && hard_grid(ctx) > 0) DM_TRY(timing_events(ctx, &e0, &e1, 0));
  const double* pp = ctx->pend_out ? ctx->pend_partial : nullptr;
  const unsigned grid = 8u * unsigned(per + 1);
  if (e0)
    hipExtLaunchKernelGGL(k_vars<R>, dim3(grid), dim3(256), 0, ctx->stream, e0, e1, 0, ctx->vpos.p, cells, cost,
                          n, per, t, pp, ctx->pend_n, ctx->pend_offset, ctx->pend_out);
  else
    k_vars<R><<<grid, 256, 0, ctx->stream>>>(ctx->vpos.p, cells, cost, n, per, t, pp, ctx->pend_n, ctx->pend_offset,
                                             ctx->pend_out);
  DM_LAUNCH_CHECK(ctx);
  ctx->pend_out = nullptr;
  return DM_OK;
}

template <typename R, bool SOFT, int MODE>
static void launch_sweep(hipStream_t st, unsigned grid, hipEvent_t e0, hipEvent_t e1, const SweepArgs& A, const R* ri,
                         const R* t, R* ro, R omega, R T) {
  if (e0 || e1)
    hipExtLaunchKernelGGL((k_sweep<R, SOFT, MODE>), dim3(grid), dim3(256), 0, st, e0, e1, 0, A, ri, t, ro, omega, T);
  else
    k_sweep<R, SOFT, MODE><<<grid, 256, 0, st>>>(A, ri, t, ro, omega, T);
}

static void common_args(const dm_ctx* ctx, SweepArgs& A) {
  A = SweepArgs();
  A.rrow_ptr = ctx->rrow_ptr.p;
  A.n_short = int32_t(ctx->n_short);
  A.long_wpr = ctx->long_wpr;
  A.n_long = int32_t(ctx->n_rows - ctx->n_short);
  A.long_perm = ctx->long_perm.p;
}

// no rows: the bound is the constant
static dm_status empty_sweep(dm_ctx* ctx, double* bound_out) {
  DM_TRY(dual_flush(ctx));
  if (bound_out) k_write_offset<<<1, 1, 0, ctx->stream>>>(bound_out, 1, ctx->offset);
  DM_LAUNCH_CHECK(ctx);
  return DM_OK;
}

static void hard_args(const dm_ctx* ctx, bool spread, SweepArgs& A) {
  common_args(ctx, A);
  A.word = ctx->cell_word.p;
  for (int f = 0; f < TILE_FORMS; ++f) {
    A.n_tiles[f] = ctx->n_tiles[f];
    A.tile_cell0[f] = uint32_t(ctx->tile_cell0[f]);
  }
  A.chunk_cell0 = uint32_t(ctx->chunk_cell0);
  A.long_cell0 = uint32_t(ctx->long_cell0);
  A.n_chunks = ctx->n_chunks;
  A.chunk_mask = ctx->chunk_mask.p;
  A.chunk_neg = ctx->chunk_neg.p;
  A.chunk_b = ctx->chunk_b.p;
  A.n_long_y = ctx->n_long_y;
  A.long_row = ctx->long_row.p;
  A.long_ent = ctx->long_ent.p;
  hard_blocks(ctx, spread, A.per);
}

// one hard row pass: mode update cells -> out (which may be cells itself),
// write M per cell to out, bound only, or the minimising assignment to
// ext->gsub; the bound goes to *bound_out (device)
template <typename R>
dm_status cells_rows(dm_ctx* ctx, int mode, const R* cells, const R* t, R* out, R omega, double* bound_out,
                     const SweepExt* ext) {
  SweepArgs A;
  hard_args(ctx, false, A);
  if (ext) {
    A.dir = ext->dir;
    A.gamma = ext->gamma;
    A.skip = ext->skip;
    A.gsub = ext->gsub;
    if (ext->terms) {
      A.terms = ext->terms;
      A.term_row = ctx->term_row;
      A.term_long = ctx->term_long;
      for (int f = 0; f < TILE_FORMS; ++f) A.tile_rows[f] = ctx->tile_rows[f];
      A.term_chunk0 = ctx->term_tiles * 256;
      A.term_long0 = (ctx->term_tiles + ctx->term_chunks) * 256;
    }
  }
  const int64_t grid = hard_grid(ctx);
  if (grid == 0) return empty_sweep(ctx, bound_out);
  DM_TRY(dual_flush(ctx));
  double* mine = nullptr;
  DM_TRY(next_partials(ctx, sizeof(R), &mine));
  A.partial = mine;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (ctx->timing) DM_TRY(timing_events(ctx, &e0, &e1, 1));
  hipStream_t st = ctx->stream;
  const unsigned g = unsigned(grid);
  if (mode == MODE_UPDATE) launch_sweep<R, false, MODE_UPDATE>(st, g, e0, e1, A, cells, t, out, omega, R(0));
  else if (mode == MODE_EVAL) launch_sweep<R, false, MODE_EVAL>(st, g, e0, e1, A, cells, t, out, omega, R(0));
  else if (mode == MODE_BOUND) launch_sweep<R, false, MODE_BOUND>(st, g, e0, e1, A, cells, t, out, omega, R(0));
  else launch_sweep<R, false, MODE_SUBGRAD>(st, g, e0, e1, A, cells, t, out, omega, R(0));
  DM_LAUNCH_CHECK(ctx);
  pend(ctx, mine, grid, bound_out);
  return DM_OK;
}

// iters hard iterations on S, whose buffer 0 holds the result (their t is left to
// the next cells_vars); the bounds go to trace (device, may be NULL), the last
// one perhaps with the next launch
template <typename R>
dm_status cells_iterate(dm_ctx* ctx, CellState& S, int32_t iters, R omega, double* trace) {
  R *cells = S.cells<R>(0), *t = S.ts<R>(0);
  if (hard_grid(ctx) == 0) {   // presolve left no rows: every bound is the constant
    DM_TRY(dual_flush(ctx));
    if (trace && iters > 0)
      k_write_offset<<<grid_for(iters, 256), 256, 0, ctx->stream>>>(trace, iters, ctx->offset);
    DM_LAUNCH_CHECK(ctx);
    return DM_OK;
  }
  const HardForm form = hard_form<R>(ctx);
  if (form == ONE_WORKGROUP && iters > 0) {
    const size_t lds = size_t(small_lds<R>(ctx));
    DM_TRY(dual_flush(ctx));
    SweepArgs A;
    hard_args(ctx, false, A);
    constexpr int NT = SMALL_THREADS<R>;
    const int64_t n_long = ctx->n_rows - ctx->n_short, mean = (ctx->nnz - ctx->nnz_short) / std::max<int64_t>(n_long, 1);
    const int32_t group = mean <= 16 ? 4 : (mean <= 64 ? 16 : 64);
    // the most that any launch of it takes, whatever this one needs: the limit
    // belongs to the function, which other threads' contexts launch too
    if (lds > 48 * 1024)
      DM_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(&k_small<R, NT>),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, int(SMALL_LDS)));
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (ctx->timing) DM_TRY(timing_events(ctx, &e0, &e1, iters));
    if (e0)
      hipExtLaunchKernelGGL((k_small<R, NT>), dim3(1), dim3(NT), lds, ctx->stream, e0, e1, 0, A, ctx->vpos.p, cells,
                            S.costs<R>(), int32_t(ctx->n_free), uint32_t(ctx->n_cells), iters, omega, ctx->offset, group, trace);
    else
      k_small<R, NT><<<1, NT, lds, ctx->stream>>>(A, ctx->vpos.p, cells, S.costs<R>(), int32_t(ctx->n_free),
                                                  uint32_t(ctx->n_cells), iters, omega, ctx->offset, group, trace);
    DM_LAUNCH_CHECK(ctx);
    return DM_OK;
  }
  if (form == ONE_LAUNCH) {
    SweepArgs A;
    hard_args(ctx, true, A);
    const int64_t grid = hard_grid(ctx, true);
    for (int32_t k = 0; k < iters; ++k) {
      double* mine = nullptr;
      DM_TRY(next_partials(ctx, sizeof(R), &mine));
      A.partial = mine;
      A.prev_partial = ctx->pend_out ? ctx->pend_partial : nullptr;
      A.prev_n = ctx->pend_n;
      A.prev_offset = ctx->pend_offset;
      A.prev_out = ctx->pend_out;
      hipEvent_t e0 = nullptr, e1 = nullptr;
      if (ctx->timing) DM_TRY(timing_events(ctx, &e0, &e1, 1));
      if (e0)
        hipExtLaunchKernelGGL(k_iterate<R>, dim3(unsigned(grid + 8)), dim3(256), 0, ctx->stream, e0, e1, 0, A,
                              S.cells<R>(0), ctx->vpos.p, S.costs<R>(), uint32_t(ctx->n_free), S.cells<R>(1), omega);
      else
        k_iterate<R><<<unsigned(grid + 8), 256, 0, ctx->stream>>>(A, S.cells<R>(0), ctx->vpos.p, S.costs<R>(),
                                                                  uint32_t(ctx->n_free), S.cells<R>(1), omega);
      DM_LAUNCH_CHECK(ctx);
      pend(ctx, mine, grid, trace ? trace + k : nullptr);
      S.swap();
    }
    return DM_OK;
  }
  for (int32_t k = 0; k < iters; ++k) {
    DM_TRY(cells_vars<R>(ctx, cells, S.costs<R>(), t, true));
    DM_TRY(cells_rows<R>(ctx, MODE_UPDATE, cells, t, cells, omega, trace ? trace + k : nullptr, nullptr));
  }
  return DM_OK;
}

// one smoothed sweep over all rows: mode update rec_in -> out, write mu to out
// per slot, or bound only; the bound goes to *bound_out (device)
template <typename R>
dm_status soft_sweep(dm_ctx* ctx, int mode, const unsigned char* rin, unsigned char* out, R omega, R T,
                     double* bound_out) {
  if (ctx->max_short > SOFT_MAX_ROW)
    return dm_fail(ctx, DM_ERR_WORKSPACE, "smoothed rows support at most %d entries (found %d)", SOFT_MAX_ROW,
                   ctx->max_short);
  SweepArgs A;
  common_args(ctx, A);
  A.ent_word = ctx->rent_word.p;
  A.rrow_b = ctx->rrow_b.p;
  A.soft_row = ctx->soft_row.p;
  A.soft_c8 = int32_t(ctx->soft_c8);
  A.soft_c16 = int32_t(ctx->soft_c16);
  A.n_short_blocks = int32_t(soft_short_blocks(ctx));
  const int64_t nl = long_blocks(ctx), nblocks = int64_t(A.n_short_blocks) + nl;
  A.n_items = int32_t(nblocks);
  if (nblocks == 0) return empty_sweep(ctx, bound_out);
  double* mine = nullptr;
  DM_TRY(next_partials(ctx, sizeof(R), &mine));
  A.partial = mine;
  A.prev_partial = ctx->pend_out ? ctx->pend_partial : nullptr;
  A.prev_n = ctx->pend_n;
  A.prev_offset = ctx->pend_offset;
  A.prev_out = ctx->pend_out;
  // 8 XCDs x blocks per XCD, see k_sweep
  const int64_t long_slots = (nl + 8 * LONG_GROUP - 1) / (8 * LONG_GROUP) * LONG_GROUP;
  const unsigned g = unsigned(8 * (long_slots + (A.n_short_blocks + 7) / 8));
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (ctx->timing) DM_TRY(timing_events(ctx, &e0, &e1, 1));
  const R* ri = reinterpret_cast<const R*>(rin);
  R* ro = reinterpret_cast<R*>(out);
  hipStream_t st = ctx->stream;
  if (mode == MODE_UPDATE) launch_sweep<R, true, MODE_UPDATE>(st, g, e0, e1, A, ri, nullptr, ro, omega, T);
  else if (mode == MODE_EVAL) launch_sweep<R, true, MODE_EVAL>(st, g, e0, e1, A, ri, nullptr, ro, omega, T);
  else launch_sweep<R, true, MODE_BOUND>(st, g, e0, e1, A, ri, nullptr, ro, omega, T);
  DM_LAUNCH_CHECK(ctx);
  pend(ctx, mine, nblocks, bound_out);
  return DM_OK;
}

// sum the partials of the last launch whose bound has not been written yet
dm_status dual_flush(dm_ctx* ctx) {
  if (ctx->pend_out) {
    k_reduce_last<<<1, 256, 0, ctx->stream>>>(ctx->pend_partial, ctx->pend_n, ctx->pend_offset, ctx->pend_out);
    DM_LAUNCH_CHECK(ctx);
  }
  ctx->pend_out = nullptr;
  return DM_OK;
}

extern "C" dm_status dm_timing_enable(dm_ctx* ctx, int32_t enable) {
  if (!ctx) return DM_ERR_INVALID_ARG;
  ctx->timing = enable != 0;
  return DM_OK;
}

extern "C" dm_status dm_timing_read(dm_ctx* ctx, int64_t* sweeps, double* total_ms) {
  if (!ctx || !sweeps || !total_ms) return DM_ERR_INVALID_ARG;
  DM_HIP(ctx, hipSetDevice(ctx->device));
  DM_HIP(ctx, hipStreamSynchronize(ctx->stream));
  double tot = 0.0;
  for (size_t i = 0; i + 1 < ctx->ev_used; i += 2) {
    float ms = 0.0f;
    DM_HIP(ctx, hipEventElapsedTime(&ms, ctx->ev_pool[i], ctx->ev_pool[i + 1]));
    tot += ms;
  }
  *sweeps = ctx->ev_sweeps;
  *total_ms = tot;
  ctx->ev_used = 0;
  ctx->ev_sweeps = 0;
  return DM_OK;
}

#define DM_INSTANTIATE(R)                                                                                            \
  template dm_status records_import<R>(dm_ctx*, const R*, DArr<unsigned char>*);                                      \
  template dm_status cells_import<R>(dm_ctx*, const R*, CellState&, bool);                                            \
  template dm_status cells_export<R>(dm_ctx*, const R*, const R*, R*);                                                \
  template dm_status cells_vars<R>(dm_ctx*, const R*, const R*, R*, bool);                                            \
  template dm_status cells_rows<R>(dm_ctx*, int, const R*, const R*, R*, R, double*, const SweepExt*);                \
  template dm_status cells_iterate<R>(dm_ctx*, CellState&, int32_t, R, double*);                                     \
  template dm_status soft_sweep<R>(dm_ctx*, int, const unsigned char*, unsigned char*, R, R, double*);
DM_INSTANTIATE(float)
DM_INSTANTIATE(double)
#undef DM_INSTANTIATE

static dm_status check_solver(dm_ctx* ctx, int32_t msg_prec) {
  if (!ctx) return DM_ERR_INVALID_ARG;
  if (!ctx->has_space) return dm_fail(ctx, DM_ERR_STATE, "no product space built");
  if (!ctx->has_cost) return dm_fail(ctx, DM_ERR_STATE, "no costs built");
  if (msg_prec != DM_PREC_FP32 && msg_prec != DM_PREC_FP64)
    return dm_fail(ctx, DM_ERR_INVALID_ARG, "message precision must be FP32 or FP64");
  return DM_OK;
}

template <typename R>
static dm_status solve_impl(dm_ctx* ctx, int32_t iters, R omega, R T, R* lam, double* trace) {
  if (T > R(0)) {
    DM_TRY(records_import<R>(ctx, lam, ctx->rec));
    for (int32_t t = 0; t < iters; ++t)
      DM_TRY(soft_sweep<R>(ctx, MODE_UPDATE, ctx->rec[t & 1].p, ctx->rec[(t + 1) & 1].p, omega, T,
                           trace ? trace + t : nullptr));
    DM_TRY(dual_flush(ctx));
    return records_export<R>(ctx, ctx->rec[iters & 1].p, lam);
  }
  CellState& S = ctx->cells;
  DM_TRY(cells_import<R>(ctx, lam, S, false));
  DM_TRY(cells_iterate<R>(ctx, S, iters, omega, trace));
  const R* cells = S.cells<R>(0);
  if (hard_form<R>(ctx) == TWO_PASSES) {
    DM_TRY(cells_vars<R>(ctx, cells, S.costs<R>(), S.ts<R>(0), false));   // also sums the last bound
    return cells_export<R>(ctx, cells, S.ts<R>(0), lam);
  }
  if (ctx->nnz == 0) return DM_OK;
  const Summed<R> t{ctx->vpos.p, cells, S.costs<R>(), uint32_t(ctx->n_free)};
  const double* prev = ctx->pend_out ? ctx->pend_partial : nullptr;
  k_cell_export<R, Summed<R>><<<grid_for(ctx->nnz, 256) + (prev ? 1u : 0u), 256, 0, ctx->stream>>>(
      cells, t, ctx->ent_cell.p, ctx->cell_word.p, ctx->nnz, lam, prev, ctx->pend_n, ctx->pend_offset, ctx->pend_out);
  DM_LAUNCH_CHECK(ctx);
  ctx->pend_out = nullptr;
  return DM_OK;
}

extern "C" dm_status dm_dual_solve(dm_ctx* ctx, int32_t iters, double omega, double temperature,
                                   int32_t msg_prec, void* lambda, double* lb_trace) {
  DM_TRY(check_solver(ctx, msg_prec));
  ctx->err.clear();
  if (iters < 0 || (!lambda && ctx->nnz > 0))
    return dm_fail(ctx, DM_ERR_INVALID_ARG, "dm_dual_solve: bad arguments");
  if (!(omega > 0.0 && omega <= 1.0)) return dm_fail(ctx, DM_ERR_INVALID_ARG, "omega must be in (0, 1]");
  if (!(temperature >= 0.0)) return dm_fail(ctx, DM_ERR_INVALID_ARG, "temperature must be >= 0");
  DM_HIP(ctx, hipSetDevice(ctx->device));
  if (msg_prec == DM_PREC_FP32)
    return solve_impl<float>(ctx, iters, float(omega), float(temperature), static_cast<float*>(lambda), lb_trace);
  return solve_impl<double>(ctx, iters, omega, temperature, static_cast<double*>(lambda), lb_trace);
}

template <typename R>
static dm_status init_lambda(dm_ctx* ctx, R* lam) {
  if (ctx->nnz <= INIT_ENTRY_NNZ) {
    k_init_entry<R><<<grid_for(ctx->nnz, 256), 256, 0, ctx->stream>>>(ctx->rent_word.p, ctx->free_var.p, ctx->cost64.p,
                                                                      ctx->var_deg.p, ctx->nnz, lam);
    DM_LAUNCH_CHECK(ctx);
    return DM_OK;
  }
  DArr<R> share;
  DM_ALLOC(ctx, share, size_t(ctx->n_free));
  k_share<R><<<grid_for(ctx->n_free, 256), 256, 0, ctx->stream>>>(ctx->free_var.p, ctx->cost64.p, ctx->var_deg.p,
                                                                  ctx->n_free, share.p);
  k_init_lambda<R><<<grid_for(ctx->nnz, 256), 256, 0, ctx->stream>>>(ctx->rent_word.p, share.p, ctx->nnz, lam);
  DM_LAUNCH_CHECK(ctx);
  return DM_OK;   // the shares are freed in stream order
}

extern "C" dm_status dm_init_lambda(dm_ctx* ctx, int32_t msg_prec, void* lambda) {
  DM_TRY(check_solver(ctx, msg_prec));
  if (!lambda && ctx->nnz > 0) return dm_fail(ctx, DM_ERR_INVALID_ARG, "dm_init_lambda: NULL lambda");
  DM_HIP(ctx, hipSetDevice(ctx->device));
  if (ctx->nnz == 0) return DM_OK;
  if (msg_prec == DM_PREC_FP32) return init_lambda<float>(ctx, static_cast<float*>(lambda));
  return init_lambda<double>(ctx, static_cast<double*>(lambda));
}

template <typename R>
static dm_status bound_impl(dm_ctx* ctx, const R* lam, R T, double* out) {
  DM_ALLOC(ctx, ctx->scal, 16);
  if (T > R(0)) {
    DArr<unsigned char> bufs[2];
    DM_TRY(records_import<R>(ctx, lam, bufs));
    DM_TRY(soft_sweep<R>(ctx, MODE_BOUND, bufs[0].p, nullptr, R(0), T, ctx->scal.p));
    DM_TRY(dual_flush(ctx));
  } else {
    CellState S;
    DM_TRY(cells_import<R>(ctx, lam, S, false));
    DM_TRY(cells_vars<R>(ctx, S.cells<R>(0), S.costs<R>(), S.ts<R>(0), true));
    DM_TRY(cells_rows<R>(ctx, MODE_BOUND, S.cells<R>(0), S.ts<R>(0), static_cast<R*>(nullptr), R(0), ctx->scal.p,
                         nullptr));
    DM_TRY(dual_flush(ctx));
  }
  DM_HIP(ctx, hipMemcpyAsync(out, ctx->scal.p, sizeof(double), hipMemcpyDeviceToHost, ctx->stream));
  DM_HIP(ctx, hipStreamSynchronize(ctx->stream));
  return DM_OK;
}

extern "C" dm_status dm_lower_bound(dm_ctx* ctx, const void* lambda, double temperature, int32_t msg_prec,
                                    double* lb) {
  DM_TRY(check_solver(ctx, msg_prec));
  if ((!lambda && ctx->nnz > 0) || !lb) return dm_fail(ctx, DM_ERR_INVALID_ARG, "dm_lower_bound: NULL argument");
  if (!(temperature >= 0.0)) return dm_fail(ctx, DM_ERR_INVALID_ARG, "temperature must be >= 0");
  DM_HIP(ctx, hipSetDevice(ctx->device));
  if (msg_prec == DM_PREC_FP32)
    return bound_impl<float>(ctx, static_cast<const float*>(lambda), float(temperature), lb);
  return bound_impl<double>(ctx, static_cast<const double*>(lambda), temperature, lb);
}

extern "C" dm_status dm_workspace_query(const dm_ctx* ctx, int32_t stage, size_t* bytes) {
  if (!ctx || !bytes) return DM_ERR_INVALID_ARG;
  if (stage != DM_WS_SOLVE_FP32 && stage != DM_WS_SOLVE_FP64) return DM_ERR_INVALID_ARG;
  if (!ctx->has_space) return DM_ERR_STATE;
  *bytes = solver_layout(ctx, stage == DM_WS_SOLVE_FP32 ? 4 : 8).total;
  return DM_OK;
}

extern "C" dm_status dm_set_workspace(dm_ctx* ctx, int32_t stage, void* ptr, size_t bytes) {
  if (!ctx) return DM_ERR_INVALID_ARG;
  ctx->err.clear();
  if (stage != DM_WS_SOLVE_FP32 && stage != DM_WS_SOLVE_FP64)
    return dm_fail(ctx, DM_ERR_INVALID_ARG, "dm_set_workspace: unknown stage %d", stage);
  const int k = stage == DM_WS_SOLVE_FP32 ? 0 : 1;
  DM_HIP(ctx, hipSetDevice(ctx->device));
  DM_TRY(dual_flush(ctx));   // a pending bound may still read the old partials
  if (ptr) {
    if (reinterpret_cast<uintptr_t>(ptr) % 256 != 0)
      return dm_fail(ctx, DM_ERR_INVALID_ARG, "dm_set_workspace: the buffer must be 256-byte aligned");
    if (!ctx->has_space) return dm_fail(ctx, DM_ERR_STATE, "dm_set_workspace: no problem built");
    const size_t need = solver_layout(ctx, k == 0 ? 4 : 8).total;
    if (bytes < need)
      return dm_fail(ctx, DM_ERR_WORKSPACE, "dm_set_workspace: %zu bytes given, %zu needed", bytes, need);
  }
  // the solver's state moves: its own arrays (or views of the old buffer) go
  ctx->rec[0].release();
  ctx->rec[1].release();
  ctx->cells.release();
  ctx->partial.release();
  ctx->ws_ptr[k] = ptr;
  ctx->ws_bytes[k] = ptr ? bytes : 0;
  return DM_OK;
}
