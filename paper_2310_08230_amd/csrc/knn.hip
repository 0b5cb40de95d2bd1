// Descriptor distances and candidate pairs.
//
// d(m, n) = ||F_X(m) - F_Y(n)||_2 is the feature distance of Eq. (cost)
// (Sec. 4.2).  Two forms:
//  * BF16: descriptors rounded to BF16 once, squared distances
//    |a|^2 + |b|^2 - 2 a.b with the dot products from a BF16 MFMA GEMM
//    (FP32 accumulation) and the norms of the rounded vectors in FP32, so
//    the result is the distance of the rounded vectors up to FP32 rounding;
//  * FP32: sum of squared differences in FP32 (no cancellation).
// The candidates of a vertex are its K nearest vertices of the other shape,
// ordered by (squared distance, index).
#include <algorithm>
#include <cmath>
#include <mutex>

#include "dm_internal.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int TOPK_MAX = 4096;      // keys in the LDS table of one top-K block
constexpr int GEMM_KC = 128;        // K values per LDS stage of the distance GEMM
constexpr int GEMM_LDS_ROW = GEMM_KC + 8;   // bf16 per staged row (16-byte pad)

__device__ inline uint16_t f32_to_bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  uint32_t lsb = (u >> 16) & 1u;
  u += 0x7FFFu + lsb;
  return uint16_t(u >> 16);
}

__device__ inline float bf16_to_f32(uint16_t h) { return __uint_as_float(uint32_t(h) << 16); }

// Both descriptor sets in one launch, PREP_ROWS vertices per block: the rounded
// rows (zero padded to Dp values and to whole 64-row tiles), their FP32 norms
// and the check for values that are not finite.  The block reads and writes
// its rows coalesced and keeps them in LDS, where one thread per vertex sums
// the squares in order (a chain of Dp fused multiply-adds).  One thread per
// vertex straight from memory took 33 us per set at 1002 and 1502 vertices of
// 128 values (a wave's loads touched 64 lines each); this takes 6 for both.
// The FP32 form only checks.
constexpr int PREP_ROWS = 16;
constexpr int PREP_KC = 128;   // values per LDS stage

struct PrepSet {
  const float* F;
  int32_t nv, nvp;
  uint16_t* out;
  float* norm;
};

__global__ __launch_bounds__(256) void k_prep(PrepSet X, PrepSet Y, int32_t D, int32_t Dp, int* err) {
  __shared__ float sq[PREP_ROWS * (PREP_KC + 1)];
  const int32_t bx = (X.nvp + PREP_ROWS - 1) / PREP_ROWS;
  const PrepSet S = int32_t(blockIdx.x) < bx ? X : Y;
  const int32_t v0 = (int32_t(blockIdx.x) < bx ? int32_t(blockIdx.x) : int32_t(blockIdx.x) - bx) * PREP_ROWS;
  bool bad = false;
  float s = 0.0f;
  for (int32_t k0 = 0; k0 < Dp; k0 += PREP_KC) {
    const int32_t kc = min(PREP_KC, Dp - k0);
    for (int32_t i = threadIdx.x; i < PREP_ROWS * kc; i += 256) {
      const int32_t r = i / kc, c = i % kc, v = v0 + r, k = k0 + c;
      float f = 0.0f;
      if (v < S.nv && k < D) f = S.F[int64_t(v) * D + k];
      bad = bad || !isfinite(f);
      if (S.out && v < S.nvp) {
        const uint16_t h = f32_to_bf16_rne(f);
        S.out[int64_t(v) * Dp + k] = h;
        sq[r * (PREP_KC + 1) + c] = bf16_to_f32(h);
      }
    }
    __syncthreads();
    if (S.out && threadIdx.x < PREP_ROWS) {
      const float* row = sq + threadIdx.x * (PREP_KC + 1);
#pragma unroll 16
      for (int32_t c = 0; c < kc; ++c) s = fmaf(row[c], row[c], s);
    }
    __syncthreads();
  }
  if (S.out && threadIdx.x < PREP_ROWS && v0 + int32_t(threadIdx.x) < S.nvp) S.norm[v0 + threadIdx.x] = s;
  if (__ballot(bad) && (threadIdx.x & 63) == 0) atomicOr(err, 1);
}

// 64x64 output tile per 256-thread block; each wave owns a 32x32 quarter and
// runs the gfx950 v_mfma_f32_32x32x16_bf16 over K in steps of 16.  Operand
// layout of that instruction: lane l holds A[l%32][8*(l/32) .. +7] and
// B[8*(l/32) .. +7][l%32]; accumulator register r of lane l is
// C[8*(r/4) + 4*(l/32) + r%4][l%32].  The block stages its 64 rows of A and
// 64 rows of B (B = F_Y^T, so rows of F_Y), GEMM_KC values of K at a time, in
// LDS with coalesced 16-byte loads; the waves read their fragments from there
// (row stride padded by 16 bytes, so the 32 rows of a fragment read start in
// different banks).
__global__ __launch_bounds__(256) void k_gemm_bf16_dist(const uint16_t* A, const uint16_t* B,
                                                        const float* na, const float* nb, int32_t nva,
                                                        int32_t nvb, int32_t Dp, float* d2, float* d2t) {
  __shared__ __align__(16) uint16_t As[64 * GEMM_LDS_ROW];
  __shared__ __align__(16) uint16_t Bs[64 * GEMM_LDS_ROW];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int32_t mb = int32_t(blockIdx.y) * 64, nbk = int32_t(blockIdx.x) * 64;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  const int row = lane & 31, kg = (lane >> 5) * 8;
  f32x16 acc;
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
  // arrays are padded to multiples of 64 rows and Dp to a multiple of 16,
  // so every staged load stays in bounds
  for (int32_t k0 = 0; k0 < Dp; k0 += GEMM_KC) {
    const int kc = Dp - k0 < GEMM_KC ? int(Dp - k0) : GEMM_KC;
    const int pieces = kc / 8;   // 16-byte pieces per row
    __syncthreads();             // the previous stage has been read
    for (int idx = threadIdx.x; idx < 64 * pieces; idx += 256) {
      const int r = idx / pieces, c = (idx % pieces) * 8;
      *reinterpret_cast<uint4*>(As + r * GEMM_LDS_ROW + c) =
          *reinterpret_cast<const uint4*>(A + int64_t(mb + r) * Dp + k0 + c);
      *reinterpret_cast<uint4*>(Bs + r * GEMM_LDS_ROW + c) =
          *reinterpret_cast<const uint4*>(B + int64_t(nbk + r) * Dp + k0 + c);
    }
    __syncthreads();
    for (int k = 0; k < kc; k += 16) {
      const bf16x8 a = *reinterpret_cast<const bf16x8*>(As + (wm + row) * GEMM_LDS_ROW + k + kg);
      const bf16x8 b = *reinterpret_cast<const bf16x8*>(Bs + (wn + row) * GEMM_LDS_ROW + k + kg);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
    }
  }
  const int32_t m0 = mb + wm;
  const int32_t col = nbk + wn + (lane & 31);
  for (int r = 0; r < 16; ++r) {
    int32_t mrow = m0 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
    if (mrow < nva && col < nvb) {
      float v = na[mrow] + nb[col] - 2.0f * acc[r];
      v = v > 0.0f ? v : 0.0f;
      d2[int64_t(mrow) * nvb + col] = v;
      if (d2t) d2t[int64_t(col) * nva + mrow] = v;   // four neighbouring rows per lane
    }
  }
}

// 64x64 output tile per 256-thread block, 4x4 per thread, FP_KC values of K at
// a time from LDS; every distance sums its squared differences in the order of
// K.  A thread per pair straight from memory read 64 lines per load (candidates of
// 1200 x 1200 vertices of 128 values: 780 us so, 67 from tiles).
constexpr int FP_KC = 32;

__global__ __launch_bounds__(256) void k_dist_fp32(const float* FX, const float* FY, int32_t nvx, int32_t nvy,
                                                   int32_t D, float* d2, float* d2t) {
  __shared__ float As[64 * (FP_KC + 1)], Bs[64 * (FP_KC + 1)];
  const int32_t m0 = int32_t(blockIdx.y) * 64, n0 = int32_t(blockIdx.x) * 64;
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  float s[4][4] = {};
  for (int32_t k0 = 0; k0 < D; k0 += FP_KC) {
    __syncthreads();
    for (int i = threadIdx.x; i < 64 * FP_KC; i += 256) {
      const int r = i / FP_KC, c = i % FP_KC;
      const bool in = k0 + c < D;
      As[r * (FP_KC + 1) + c] = in && m0 + r < nvx ? FX[int64_t(m0 + r) * D + k0 + c] : 0.0f;
      Bs[r * (FP_KC + 1) + c] = in && n0 + r < nvy ? FY[int64_t(n0 + r) * D + k0 + c] : 0.0f;
    }
    __syncthreads();
    const int kc = D - k0 < FP_KC ? int(D - k0) : FP_KC;
    for (int k = 0; k < kc; ++k) {
      float a[4], b[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        a[u] = As[(ty + 16 * u) * (FP_KC + 1) + k];
        b[u] = Bs[(tx + 16 * u) * (FP_KC + 1) + k];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const float d = a[u] - b[w];
          s[u][w] = fmaf(d, d, s[u][w]);
        }
    }
  }
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const int32_t m = m0 + ty + 16 * u, n = n0 + tx + 16 * w;
      if (m < nvx && n < nvy) {
        d2[int64_t(m) * nvy + n] = s[u][w];
        if (d2t) d2t[int64_t(n) * nvx + m] = s[u][w];
      }
    }
}

__global__ void k_nonfinite(const float* a, int64_t n, int* err) {
  int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n && !isfinite(a[i])) atomicOr(err, 1);
}

// ascending bitonic sort of np2 keys (a power of two) in LDS by one block
__device__ void bitonic_lds(uint64_t* keys, int32_t np2) {
  for (int32_t size = 2; size <= np2; size <<= 1) {
    for (int32_t stride = size >> 1; stride > 0; stride >>= 1) {
      for (int32_t i = threadIdx.x; i < np2; i += blockDim.x) {
        int32_t j = i ^ stride;
        if (j > i) {
          bool up = (i & size) == 0;
          uint64_t a = keys[i], b = keys[j];
          if ((a > b) == up) {
            keys[i] = b;
            keys[j] = a;
          }
        }
      }
      __syncthreads();
    }
  }
}

// one block per query vertex, K > TOPK_MAX / 2 (then the row has at most
// TOPK_MAX keys): (squared distance, index) keys sorted whole in LDS, first K
// indices out.  dir 0: rows of d2 (X queries), 1: columns.
__global__ __launch_bounds__(256) void k_topk(const float* d2, int32_t nvx, int32_t nvy, int dir,
                                              int32_t K, int32_t* out, const int* err) {
  __shared__ uint64_t keys[TOPK_MAX];
  if (*err) return;   // a descriptor is not finite: nothing is written
  const int32_t q = blockIdx.x;
  const int32_t n = dir == 0 ? nvy : nvx;
  int32_t np2 = 1;
  while (np2 < n) np2 <<= 1;
  for (int32_t i = threadIdx.x; i < np2; i += blockDim.x) {
    uint64_t key = ~uint64_t(0);
    if (i < n) {
      const float v = dir == 0 ? d2[int64_t(q) * nvy + i] : d2[int64_t(i) * nvy + q];
      key = (uint64_t(__float_as_uint(v + 0.0f)) << 32) | uint32_t(i);
    }
    keys[i] = key;
  }
  __syncthreads();
  bitonic_lds(keys, np2);
  for (int32_t k = threadIdx.x; k < K; k += blockDim.x) out[int64_t(q) * K + k] = int32_t(keys[k] & 0xFFFFFFFFu);
}

// one block per query vertex of either shape, K <= TOPK_MAX / 2, any row
// length: the keys (squared distance bits << 32 | index; distances are >= 0,
// so the bits order like the values, and the index makes every key unique) are
// not stored.  A radix selection finds the K-th smallest key digit by digit
// (six digits of 11, 11, 10, 11, 11 and 10 bits, high to low): a histogram of
// the digit over the keys that share the digits found so far, and the digit
// whose cumulative count reaches the rank sought.  Once all keys with the
// digits found belong to the K smallest, the rest of the digits is not needed
// (the usual end, after the second or third: distances rarely tie).  The K
// keys are then gathered and sorted in LDS, so the result is the same ordered
// list as a full sort's first K.
// Rows of at most 256 * REG values stay in registers (a thread's own REG of
// them); longer ones (REG = 0) are read again for every digit.  Y queries read
// rows of the transposed distances where there is room for them (d2t), columns
// of d2 otherwise.  1002 and 1502 queries, K = 48: 85 us for two launches of six
// digits with the columns strided, 26 in one.
template <int REG>
__global__ __launch_bounds__(256) void k_topk_select(const float* d2, const float* d2t, int32_t nvx, int32_t nvy,
                                                     int32_t K, int32_t* out_xy, int32_t* out_yx, const int* err) {
  __shared__ uint32_t hist[2048];
  __shared__ uint32_t wsum[4];
  __shared__ uint64_t keys[TOPK_MAX / 2];
  __shared__ uint32_t sh_digit, sh_rank, sh_count, sh_all;
  if (*err) return;   // a descriptor is not finite: nothing is written
  const bool yq = int32_t(blockIdx.x) >= nvx;
  const int32_t q = yq ? int32_t(blockIdx.x) - nvx : int32_t(blockIdx.x);
  const int32_t n = yq ? nvx : nvy;
  const float* row = yq ? (d2t ? d2t + int64_t(q) * nvx : d2 + q) : d2 + int64_t(q) * nvy;
  const int64_t stride = yq && !d2t ? nvy : 1;
  int32_t* out = (yq ? out_yx : out_xy) + int64_t(q) * K;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  float reg[REG > 0 ? REG : 1];
  if constexpr (REG > 0) {
#pragma unroll
    for (int u = 0; u < REG; ++u) reg[u] = t + 256 * u < n ? row[int64_t(t + 256 * u) * stride] : 0.0f;
  }
  auto key = [&](int32_t i, float v) { return (uint64_t(__float_as_uint(v + 0.0f)) << 32) | uint32_t(i); };
  auto each = [&](auto f) {   // f(key) for every key of this thread
    if constexpr (REG > 0) {
#pragma unroll
      for (int u = 0; u < REG; ++u)
        if (t + 256 * u < n) f(key(t + 256 * u, reg[u]));
    } else {
      for (int32_t i = t; i < n; i += 256) f(key(i, row[int64_t(i) * stride]));
    }
  };
  uint64_t prefix = 0;   // the digits found so far, in place
  int known = 0;         // bits found so far
  uint32_t rank = uint32_t(K);   // 1-based rank sought among the keys with that prefix
  for (int pass = 0; pass < 6; ++pass) {   // uniform across the block
    const int width = pass % 3 == 2 ? 10 : 11;
    const int shift = 64 - known - width;
    const uint32_t mask = (1u << width) - 1u;
    for (int b = t; b < 2048; b += 256) hist[b] = 0u;
    __syncthreads();
    each([&](uint64_t k) {
      if (known == 0 || (k >> (64 - known)) == (prefix >> (64 - known)))
        atomicAdd(&hist[uint32_t(k >> shift) & mask], 1u);
    });
    __syncthreads();
    // counts of the eight bins of this thread, then an exclusive scan over
    // the 256 threads
    uint32_t bin[8], loc = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      bin[j] = hist[8 * t + j];
      loc += bin[j];
    }
    uint32_t incl = loc;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t add = __shfl_up(incl, off);
      if (lane >= off) incl += add;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    uint32_t below = incl - loc;   // keys in the bins before this thread's
    for (int w = 0; w < wave; ++w) below += wsum[w];
    if (below < rank && rank <= below + loc) {   // exactly one thread
      bool found = false;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        if (!found && rank <= below + bin[j]) {
          sh_digit = uint32_t(8 * t + j);
          sh_rank = rank - below;
          sh_all = rank - below == bin[j] ? 1u : 0u;
          found = true;
        }
        below += bin[j];
      }
    }
    __syncthreads();
    prefix |= uint64_t(sh_digit) << shift;
    rank = sh_rank;
    known += width;
    if (sh_all) {   // uniform: every key with this prefix is among the K smallest
      prefix |= (uint64_t(1) << shift) - 1u;
      break;
    }
    __syncthreads();
  }
  // exactly K keys are <= prefix
  if (t == 0) sh_count = 0u;
  __syncthreads();
  each([&](uint64_t k) {
    if (k <= prefix) {
      const uint32_t pos = atomicAdd(&sh_count, 1u);
      if (pos < uint32_t(TOPK_MAX / 2)) keys[pos] = k;   // exactly K < TOPK_MAX / 2 + 1 of them
    }
  });
  int32_t np2 = 1;
  while (np2 < K) np2 <<= 1;
  for (int32_t i = K + t; i < np2; i += 256) keys[i] = ~uint64_t(0);
  __syncthreads();
  bitonic_lds(keys, np2);
  for (int32_t k = t; k < K; k += 256) out[k] = int32_t(keys[k] & 0xFFFFFFFFu);
}

__global__ void k_zero_i32(int* p) { *p = 0; }

// Temporaries of one candidate computation, carved from one block of device
// memory: an error word, the squared distances d2 [nvx*nvy], with_t their
// transpose too, and, in the BF16 form, the rounded descriptors padded to 64
// rows and 8 columns with their norms.  Every piece starts on a 256-byte
// boundary.
struct KnnBufs {
  int* err = nullptr;
  float* d2 = nullptr;
  float* d2t = nullptr;
  uint16_t* A = nullptr;
  uint16_t* B = nullptr;
  float* na = nullptr;
  float* nb = nullptr;
};

inline size_t align256(size_t n) { return (n + 255) / 256 * 256; }

// bytes the temporaries need; with base set, the pieces' addresses in it
size_t knn_layout(int32_t nvx, int32_t nvy, int32_t D, int32_t prec, bool with_d2, bool with_t,
                  unsigned char* base, KnnBufs* out) {
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t at = off;
    off += align256(bytes);
    return base ? base + at : nullptr;
  };
  KnnBufs b;
  b.err = reinterpret_cast<int*>(take(sizeof(int)));
  if (with_d2) b.d2 = reinterpret_cast<float*>(take(sizeof(float) * size_t(nvx) * size_t(nvy)));
  if (with_t) b.d2t = reinterpret_cast<float*>(take(sizeof(float) * size_t(nvx) * size_t(nvy)));
  if (prec == DM_PREC_BF16) {
    const size_t Dp = size_t(D + 15) / 16 * 16;
    const size_t nxp = size_t(nvx + 63) / 64 * 64, nyp = size_t(nvy + 63) / 64 * 64;
    b.A = reinterpret_cast<uint16_t*>(take(sizeof(uint16_t) * nxp * Dp));
    b.B = reinterpret_cast<uint16_t*>(take(sizeof(uint16_t) * nyp * Dp));
    b.na = reinterpret_cast<float*>(take(sizeof(float) * nxp));
    b.nb = reinterpret_cast<float*>(take(sizeof(float) * nyp));
  }
  if (out) *out = b;
  return off;
}

// Scratch of the allocation-free entry point: one array per GPU, alive until
// the process ends.  Host code never passes the array's name to a kernel; it
// uses the device address taken once per device by knn_scratch_init.
constexpr size_t KNN_SCRATCH_BYTES = size_t(16) << 20;
static __device__ __align__(256) unsigned char scratch[KNN_SCRATCH_BYTES];

constexpr int KNN_MAX_DEVICES = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[KNN_MAX_DEVICES] = {};

// the check's word on its way to the host, and the wait for it (what was
// enqueued since runs on)
dm_status send_finite(dm_ctx* ctx, const int* err) {
  DM_HIP(ctx, hipMemcpyAsync(ctx->host_i32, err, sizeof(int), hipMemcpyDeviceToHost, ctx->stream));
  DM_HIP(ctx, hipEventRecord(ctx->landed, ctx->stream));
  return DM_OK;
}

dm_status wait_finite(dm_ctx* ctx) {
  DM_HIP(ctx, hipEventSynchronize(ctx->landed));
  if (ctx->host_i32[0]) return dm_fail(ctx, DM_ERR_NONFINITE, "non-finite descriptor");
  return DM_OK;
}

// the squared distances, enqueued; wait_finite tells whether all descriptors are finite
dm_status distances_into(dm_ctx* ctx, const float* FX, int32_t nvx, const float* FY, int32_t nvy, int32_t D,
                         int32_t prec, const KnnBufs& w, float* d2) {
  if (prec != DM_PREC_BF16 && prec != DM_PREC_FP32 && prec != DM_PREC_FP64)
    return dm_fail(ctx, DM_ERR_INVALID_ARG, "unknown precision %d", prec);
  hipStream_t st = ctx->stream;
  const bool bf = prec == DM_PREC_BF16;
  const int32_t Dp = bf ? (D + 15) / 16 * 16 : D;
  const int32_t nxp = bf ? (nvx + 63) / 64 * 64 : nvx, nyp = bf ? (nvy + 63) / 64 * 64 : nvy;
  const unsigned blocks = grid_for(nxp, PREP_ROWS) + grid_for(nyp, PREP_ROWS);
  k_zero_i32<<<1, 1, 0, st>>>(w.err);
  k_prep<<<blocks, 256, 0, st>>>(PrepSet{FX, nvx, nxp, w.A, w.na}, PrepSet{FY, nvy, nyp, w.B, w.nb}, D, Dp, w.err);
  DM_LAUNCH_CHECK(ctx);
  DM_TRY(send_finite(ctx, w.err));
  const dim3 grid(unsigned((nvy + 63) / 64), unsigned((nvx + 63) / 64));
  if (bf) k_gemm_bf16_dist<<<grid, 256, 0, st>>>(w.A, w.B, w.na, w.nb, nvx, nvy, Dp, d2, w.d2t);
  else k_dist_fp32<<<grid, 256, 0, st>>>(FX, FY, nvx, nvy, D, d2, w.d2t);
  DM_LAUNCH_CHECK(ctx);
  return DM_OK;
}

dm_status knn_check_args(dm_ctx* ctx, const char* name, const float* FX, int32_t nvx, const float* FY,
                         int32_t nvy, int32_t D, int32_t K, int32_t prec, const int32_t* cand_xy,
                         const int32_t* cand_yx) {
  if (!FX || !FY || !cand_xy || !cand_yx) return dm_fail(ctx, DM_ERR_INVALID_ARG, "%s: NULL argument", name);
  if (nvx < 1 || nvy < 1 || D < 1 || K < 1 || K > nvx || K > nvy ||
      ((nvx > TOPK_MAX || nvy > TOPK_MAX) && K > TOPK_MAX / 2) || nvx > (1 << 21) || nvy > (1 << 21))
    return dm_fail(ctx, DM_ERR_INVALID_ARG, "%s: nvx=%d nvy=%d D=%d K=%d out of range", name, nvx, nvy, D, K);
  if (prec != DM_PREC_BF16 && prec != DM_PREC_FP32 && prec != DM_PREC_FP64)
    return dm_fail(ctx, DM_ERR_INVALID_ARG, "%s: unknown precision %d", name, prec);
  return DM_OK;
}

// Distances into w.d2, then the K nearest both ways.  Everything is enqueued
// before the one wait, which is for the check of the descriptors alone; the
// selection writes nothing when the check fails.
dm_status knn_run(dm_ctx* ctx, const float* FX, int32_t nvx, const float* FY, int32_t nvy, int32_t D, int32_t K,
                  int32_t prec, int32_t* cand_xy, int32_t* cand_yx, const KnnBufs& w) {
  hipStream_t st = ctx->stream;
  DM_TRY(distances_into(ctx, FX, nvx, FY, nvy, D, prec, w, w.d2));
  if (K <= TOPK_MAX / 2) {
    const unsigned blocks = unsigned(nvx) + unsigned(nvy);
    if (std::max(nvx, nvy) <= 256 * 8)
      k_topk_select<8><<<blocks, 256, 0, st>>>(w.d2, w.d2t, nvx, nvy, K, cand_xy, cand_yx, w.err);
    else
      k_topk_select<0><<<blocks, 256, 0, st>>>(w.d2, w.d2t, nvx, nvy, K, cand_xy, cand_yx, w.err);
  } else {   // then both sides have at most TOPK_MAX vertices (checked above)
    k_topk<<<nvx, 256, 0, st>>>(w.d2, nvx, nvy, 0, K, cand_xy, w.err);
    k_topk<<<nvy, 256, 0, st>>>(w.d2, nvx, nvy, 1, K, cand_yx, w.err);
  }
  DM_LAUNCH_CHECK(ctx);
  return wait_finite(ctx);
}

}  // namespace

// device address of this GPU's scratch array, taken once per device with the
// device current (each GPU holds its own copy at its own address)
dm_status knn_scratch_init(dm_ctx* ctx) {
  const int dev = ctx->device;
  if (dev < 0 || dev >= KNN_MAX_DEVICES) return DM_OK;   // the allocation-free entry point refuses such devices
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[dev]) return DM_OK;
  void* ptr = nullptr;
  DM_HIP(ctx, hipSetDevice(dev));
  DM_HIP(ctx, hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
  if (!ptr) return dm_fail(ctx, DM_ERR_HIP, "no device address for the candidate scratch array");
  g_scratch_ptr[dev] = ptr;
  return DM_OK;
}

// both descriptor arrays flag one word, read back once
dm_status check_finite(dm_ctx* ctx, const float* a, int64_t na, const float* b, int64_t nb) {
  DArr<int> err;
  DM_ALLOC(ctx, err, 1);
  k_zero_i32<<<1, 1, 0, ctx->stream>>>(err.p);
  if (na > 0) k_nonfinite<<<grid_for(na, 256), 256, 0, ctx->stream>>>(a, na, err.p);
  if (nb > 0) k_nonfinite<<<grid_for(nb, 256), 256, 0, ctx->stream>>>(b, nb, err.p);
  DM_LAUNCH_CHECK(ctx);
  // nothing runs meanwhile: the plain wait is 12 us shorter than the event's
  int e = 0;
  DM_TRY(read_i32(ctx, err.p, &e));
  if (e) return dm_fail(ctx, DM_ERR_NONFINITE, "non-finite descriptor");
  return DM_OK;
}

dm_status knn_distances(dm_ctx* ctx, const float* FX, int32_t nvx, const float* FY, int32_t nvy,
                        int32_t D, int32_t prec, float* d2) {
  // the distances go to the caller's d2: the layout without its d2 piece
  DArr<unsigned char> ws;
  KnnBufs w;
  DM_ALLOC(ctx, ws, knn_layout(nvx, nvy, D, prec, false, false, nullptr, nullptr));
  knn_layout(nvx, nvy, D, prec, false, false, ws.p, &w);
  DM_TRY(distances_into(ctx, FX, nvx, FY, nvy, D, prec, w, d2));
  return wait_finite(ctx);
}

extern "C" dm_status dm_knn_candidates(dm_ctx* ctx, const float* FX, int32_t nvx, const float* FY,
                                       int32_t nvy, int32_t D, int32_t K, int32_t prec, int32_t* cand_xy,
                                       int32_t* cand_yx) {
  if (!ctx) return DM_ERR_INVALID_ARG;
  ctx->err.clear();
  DM_TRY(knn_check_args(ctx, "dm_knn_candidates", FX, nvx, FY, nvy, D, K, prec, cand_xy, cand_yx));
  DM_HIP(ctx, hipSetDevice(ctx->device));
  // the transposed distances where they are read and memory has room for both
  DArr<unsigned char> ws;
  KnnBufs w;
  bool with_t = K <= TOPK_MAX / 2;
  if (with_t && ws.resize(knn_layout(nvx, nvy, D, prec, true, true, nullptr, nullptr), ctx->stream, ctx->pool,
                          &ctx->cache) != hipSuccess) {
    (void)hipGetLastError();
    with_t = false;
  }
  if (!with_t) DM_ALLOC(ctx, ws, knn_layout(nvx, nvy, D, prec, true, false, nullptr, nullptr));
  knn_layout(nvx, nvy, D, prec, true, with_t, ws.p, &w);
  DM_TRY(knn_run(ctx, FX, nvx, FY, nvy, D, K, prec, cand_xy, cand_yx, w));
  return DM_OK;   // the temporaries are freed in stream order
}

extern "C" dm_status dm_knn_candidates_noalloc(dm_ctx* ctx, const float* FX, int32_t nvx, const float* FY,
                                               int32_t nvy, int32_t D, int32_t K, int32_t prec,
                                               int32_t* cand_xy, int32_t* cand_yx) {
  if (!ctx) return DM_ERR_INVALID_ARG;
  ctx->err.clear();
  DM_TRY(knn_check_args(ctx, "dm_knn_candidates_noalloc", FX, nvx, FY, nvy, D, K, prec, cand_xy, cand_yx));
  const size_t need = knn_layout(nvx, nvy, D, prec, true, false, nullptr, nullptr);
  if (need > KNN_SCRATCH_BYTES)
    return dm_fail(ctx, DM_ERR_WORKSPACE,
                   "dm_knn_candidates_noalloc: needs %zu bytes of scratch, the limit is %zu (nvx=%d nvy=%d D=%d)",
                   need, KNN_SCRATCH_BYTES, nvx, nvy, D);
  void* base = nullptr;
  {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (ctx->device >= 0 && ctx->device < KNN_MAX_DEVICES) base = g_scratch_ptr[ctx->device];
  }
  if (!base) return dm_fail(ctx, DM_ERR_STATE, "dm_knn_candidates_noalloc: no scratch address for device %d",
                            ctx->device);
  DM_HIP(ctx, hipSetDevice(ctx->device));
  KnnBufs w;
  // the transposed distances where they are read and the scratch has room for them
  const bool with_t =
      K <= TOPK_MAX / 2 && knn_layout(nvx, nvy, D, prec, true, true, nullptr, nullptr) <= KNN_SCRATCH_BYTES;
  knn_layout(nvx, nvy, D, prec, true, with_t, static_cast<unsigned char*>(base), &w);
  return knn_run(ctx, FX, nvx, FY, nvy, D, K, prec, cand_xy, cand_yx, w);
}
