// Launch layout of the row sweep (the row-parallel min-marginal sweep of
// Sec. 3.2 / Eq. (D), mapped onto the eight XCDs of the chip).
//
// Multipliers live in row order: every entry of the presolved rows owns one
// cell, and the cells of a row sit where the wave that sweeps the row reads
// them coalesced.  What crosses between rows is one value per variable (the
// correction that restores dual feasibility, see dual.hip), so the layout has
// two orders and an index each way:
//   * cells: short rows with b = 0 and few entries of each sign in 64-row
//     tiles (one lane per row), the other short rows in wave chunks (one lane
//     per entry), the projection rows with their entries in variable order.
//     cell_word names each cell's variable;
//   * variables: vpos names the (at most five) cells of each variable.
// Both orders follow the meshes: an element's key is the rank of its X
// element's owner face in the Morton order of the X face centroids (a face
// owns itself; an edge or a vertex is owned by its adjacent face of lowest
// rank), then the same rank on Y.  Variables are numbered by that key (the
// index v, against the canonical index i of the reduced problem: vperm[v] =
// i), rows are ordered by the smallest X rank and the smallest Y rank of their
// entries, so that 64 neighbouring rows share most of their variables, a
// wave's gathers fall into few cache lines, and each XCD, which takes a
// contiguous eighth of either order, holds nearly all of what it reads in its
// own L2 (2000/3000-face pair, both passes: 11 us more with the canonical order
// inside each X face; they take 108).  A generic problem without meshes keys a
// variable by its index.
#include <algorithm>
#include <climits>

#include "dm_internal.h"

namespace {

constexpr int PACK_SEG = 4096;    // entries per segment of the parallel chunk packing

// ---------------------------------------------------------------- keys
// bounding box of the vertices: out[0..2] minimum, out[3..5] maximum
__global__ __launch_bounds__(256) void k_bbox(const float* v, int32_t nv, float* out) {
  __shared__ float sh[6][256];
  float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (int32_t i = threadIdx.x; i < nv; i += 256)
    for (int k = 0; k < 3; ++k) {
      lo[k] = fminf(lo[k], v[3 * i + k]);
      hi[k] = fmaxf(hi[k], v[3 * i + k]);
    }
  for (int k = 0; k < 3; ++k) {
    sh[k][threadIdx.x] = lo[k];
    sh[3 + k][threadIdx.x] = hi[k];
  }
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (int(threadIdx.x) < o)
      for (int k = 0; k < 3; ++k) {
        sh[k][threadIdx.x] = fminf(sh[k][threadIdx.x], sh[k][threadIdx.x + o]);
        sh[3 + k][threadIdx.x] = fmaxf(sh[3 + k][threadIdx.x], sh[3 + k][threadIdx.x + o]);
      }
    __syncthreads();
  }
  if (threadIdx.x < 6) out[threadIdx.x] = sh[threadIdx.x][0];
}

__device__ inline uint32_t spread3(uint32_t x) {   // 10 bits -> every third bit of 30
  x &= 0x3FFu;
  x = (x | (x << 16)) & 0x030000FFu;
  x = (x | (x << 8)) & 0x0300F00Fu;
  x = (x | (x << 4)) & 0x030C30C3u;
  x = (x | (x << 2)) & 0x09249249u;
  return x;
}

// 30-bit Morton code of every face centroid on a 1024^3 grid over the box
__global__ void k_face_morton(const float* v, const int32_t* f, int32_t nf, const float* box, uint32_t* key,
                              int32_t* val) {
  const int32_t i = int32_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= nf) return;
  uint32_t q[3];
  for (int k = 0; k < 3; ++k) {
    const float c = (v[3 * f[3 * i] + k] + v[3 * f[3 * i + 1] + k] + v[3 * f[3 * i + 2] + k]) * (1.0f / 3.0f);
    const float ext = box[3 + k] - box[k];
    const float u = ext > 0.0f ? (c - box[k]) / ext : 0.0f;
    q[k] = uint32_t(fminf(fmaxf(u * 1024.0f, 0.0f), 1023.0f));
  }
  key[i] = spread3(q[0]) | (spread3(q[1]) << 1) | (spread3(q[2]) << 2);
  val[i] = i;
}

__global__ void k_rank_of(const int32_t* order, int32_t n, int32_t* rank) {
  const int32_t i = int32_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) rank[order[i]] = i;
}

// owner rank of every edge and vertex: the lowest rank of an adjacent face
__global__ void k_elem_rank(const int32_t* faces, const int32_t* face_edge, const int32_t* frank, int32_t nf,
                            int32_t* erank, int32_t* vrank) {
  const int32_t f = int32_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (f >= nf) return;
  const int32_t r = frank[f];
  for (int k = 0; k < 3; ++k) {
    atomicMin(&erank[face_edge[3 * f + k]], r);
    atomicMin(&vrank[faces[3 * f + k]], r);
  }
}

__global__ void k_fill_i32(int32_t* a, int64_t n, int32_t v) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) a[i] = v;
}

// key of every free variable (X rank of its element, then Y rank) as sort key
// and as table, with its index
__global__ void k_var_keys(const int32_t* free_var, const int32_t* code, const int32_t* xf, const int32_t* xe,
                           const int32_t* xv, const int32_t* yf, const int32_t* ye, const int32_t* yv, int ybits,
                           int64_t n, uint32_t* vkey, uint32_t* key, int32_t* val) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int4 c = reinterpret_cast<const int4*>(code)[free_var[i]];
  const int32_t xr = c.x == 0 ? xf[c.y] : (c.x == 1 ? xe[c.y] : xv[c.y]);
  const int32_t yc = c.z >> 3;
  const int32_t yr = yc == 0 ? yf[c.w] : (yc == 1 ? ye[c.w] : yv[c.w]);
  const uint32_t k = (uint32_t(xr) << ybits) | uint32_t(yr);
  vkey[i] = k;
  key[i] = k;
  val[i] = int32_t(i);
}

__global__ void k_iota2(uint32_t* a, int32_t* b, int64_t n) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  a[i] = uint32_t(i);
  b[i] = int32_t(i);
}

__global__ void k_var_order(const int32_t* vperm, const uint8_t* deg, int64_t n, int32_t* vinv, uint8_t* vdeg) {
  const int64_t v = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (v >= n) return;
  const int32_t i = vperm[v];
  vinv[i] = int32_t(v);
  vdeg[v] = deg[i];
}

// unused slots of every variable point at the zero cell
__global__ void k_unused_slots(const uint8_t* vdeg, int64_t n, uint32_t zero_cell, uint32_t* vpos) {
  const int64_t v = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (v >= n) return;
  for (int k = vdeg[v]; k < 5; ++k) vpos[size_t(k) * n + v] = zero_cell;
}

// entries per batch of loads in the one-thread-per-row kernels below (indices
// clamped to the row: no branch, all loads of a batch in flight together)
constexpr int ROW_BATCH = 8;

// Short rows: sort key (form, smallest X rank, smallest Y rank), sorted stably
// so that equal keys keep the row order.  Forms: 0 to 2 are the tiles
// (right-hand side 0 and at most TILE_HALF entries of each sign, the narrowest
// from form0 on), 3 the chunks.  count: rows of each tile form, entries of all
// of them.
__global__ __launch_bounds__(256) void k_short_keys(const int32_t* rrow_ptr, const int32_t* rrow_b,
                                                    const uint32_t* word, const uint32_t* vkey, int64_t n_short,
                                                    int ybits, int ydrop, int kbits, uint32_t form0, uint32_t* key,
                                                    int32_t* val, int32_t* count) {
  __shared__ int32_t sh[TILE_FORMS + 1];
  if (threadIdx.x <= TILE_FORMS) sh[threadIdx.x] = 0;
  __syncthreads();
  const int64_t j = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (j < n_short) {
    const uint32_t ymask = (1u << ybits) - 1u;
    const int32_t s = rrow_ptr[j], t = rrow_ptr[j + 1];
    int32_t nq = 0;
    uint32_t x = 0xFFFFFFFFu, y = 0xFFFFFFFFu;
    for (int32_t e0 = s; e0 < t; e0 += ROW_BATCH) {   // the loads of a batch go out together
      uint32_t w[ROW_BATCH], k[ROW_BATCH];
#pragma unroll
      for (int u = 0; u < ROW_BATCH; ++u) w[u] = word[e0 + u < t ? e0 + u : e0];
#pragma unroll
      for (int u = 0; u < ROW_BATCH; ++u) k[u] = vkey[w[u] & W_VAR_MASK];
#pragma unroll
      for (int u = 0; u < ROW_BATCH; ++u) {   // repeats of e0 change no minimum
        nq += (e0 + u < t && (w[u] & W_NEG)) ? 1 : 0;
        x = min(x, k[u] >> ybits);
        y = min(y, k[u] & ymask);
      }
    }
    const int32_t m = max(nq, (t - s) - nq);
    uint32_t form = rrow_b[j] != 0 ? uint32_t(TILE_FORMS) : form0;
    while (form < TILE_FORMS && m > TILE_HALF[form]) ++form;
    // chunks by the X rank alone: which rows share a chunk decides which of two
    // forms of the same minimum sweeps them
    key[j] = (form << kbits) | (x << (ybits - ydrop)) | (form < TILE_FORMS ? y >> ydrop : 0u);
    val[j] = int32_t(j);
    if (form < TILE_FORMS) {
      atomicAdd(&sh[form], 1);
      atomicAdd(&sh[TILE_FORMS], t - s);
    }
  }
  __syncthreads();
  if (threadIdx.x <= TILE_FORMS && sh[threadIdx.x]) atomicAdd(&count[threadIdx.x], sh[threadIdx.x]);
}

__device__ inline uint32_t cell_word_of(uint32_t w, const int32_t* vinv, const uint8_t* deg, int32_t* v) {
  const uint32_t i = w & W_VAR_MASK;
  *v = vinv[i];
  return uint32_t(*v) | (uint32_t(deg[i]) << CELL_DEG_SHIFT);
}

// Cells of the tile rows (rows perm[0 .. n), half H): pair j of lane l holds
// the row's j-th +1 and j-th -1 entry, each group in row order, at
// tile * 128 H + j * 128 + 2 l + sign.
__global__ void k_tile_fill(const int32_t* perm, int64_t n, int H, uint32_t cell0, const int32_t* rrow_ptr,
                            const uint32_t* word, const int32_t* vinv, const uint8_t* deg, int64_t n_free,
                            uint32_t* cell_word, uint32_t* ent_cell, uint32_t* vpos) {
  const int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const uint32_t base = cell0 + uint32_t(k / 64) * uint32_t(128 * H) + uint32_t(k % 64) * 2u;
  const int32_t j = perm[k];
  const int32_t s = rrow_ptr[j], t = rrow_ptr[j + 1];
  uint32_t np = 0, nq = 0;
  for (int32_t e0 = s; e0 < t; e0 += ROW_BATCH) {
    uint32_t w[ROW_BATCH], cw[ROW_BATCH];
    int32_t v[ROW_BATCH];
#pragma unroll
    for (int u = 0; u < ROW_BATCH; ++u) w[u] = word[e0 + u < t ? e0 + u : e0];
#pragma unroll
    for (int u = 0; u < ROW_BATCH; ++u) cw[u] = cell_word_of(w[u], vinv, deg, &v[u]);
#pragma unroll
    for (int u = 0; u < ROW_BATCH; ++u) {
      if (e0 + u >= t) continue;
      const uint32_t c = base + ((w[u] & W_NEG) ? 128u * nq++ + 1u : 128u * np++);
      cell_word[c] = cw[u];
      ent_cell[e0 + u] = c;
      vpos[size_t((w[u] >> W_SLOT_SHIFT) & 7u) * n_free + v[u]] = c;
    }
  }
}

// Order of the entries of every projection row, one block per row: a Y row's
// by the X rank of their elements, an X row's by the Y rank, in RANK_BINS bins
// (a bin takes 2^xdrop or 2^ydrop neighbouring ranks).  Count, scan and place
// in LDS; where entries of one bin land among themselves is left open, which
// no result depends on (a row's minimum is the same in any order, and equal
// minima are told apart by long_ent).  A radix sort of the same keys took
// 0.33 ms of the 2000/3000-face pair's build, this takes 0.03.
constexpr int RANK_BINS = 4096;

__global__ __launch_bounds__(256) void k_long_order(const int32_t* rrow_ptr, const int32_t* rrow_orig,
                                                    const uint32_t* word, const uint32_t* vkey, int64_t n_short,
                                                    int64_t first_y_full, int ybits, int xdrop, int ydrop,
                                                    int32_t* long_ent) {
  __shared__ int32_t bin[RANK_BINS];
  __shared__ int32_t wsum[4];
  const int64_t j = n_short + blockIdx.x;
  const int32_t e0 = rrow_ptr[n_short], s = rrow_ptr[j], t = rrow_ptr[j + 1];
  const bool yrow = rrow_orig[j] >= first_y_full;
  auto bin_of = [&](int32_t e) {
    const uint32_t k = vkey[word[e] & W_VAR_MASK];
    return yrow ? (k >> ybits) >> xdrop : (k & ((1u << ybits) - 1u)) >> ydrop;
  };
  for (int k = threadIdx.x; k < RANK_BINS; k += 256) bin[k] = 0;
  __syncthreads();
  for (int32_t e = s + int32_t(threadIdx.x); e < t; e += 256) atomicAdd(&bin[bin_of(e)], 1);
  __syncthreads();
  // exclusive scan: each thread its RANK_BINS / 256 bins, then the threads
  constexpr int PER = RANK_BINS / 256;
  int32_t c[PER], sum = 0;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    c[k] = bin[int(threadIdx.x) * PER + k];
    sum += c[k];
  }
  int32_t pre = sum;
  const int lane = int(threadIdx.x & 63), wave = int(threadIdx.x >> 6);
  for (int o = 1; o < 64; o <<= 1) {
    const int32_t u = __shfl_up(pre, o);
    if (lane >= o) pre += u;
  }
  if (lane == 63) wsum[wave] = pre;
  __syncthreads();
  int32_t at = s - e0 + pre - sum;
  for (int w = 0; w < wave; ++w) at += wsum[w];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    bin[int(threadIdx.x) * PER + k] = at;
    at += c[k];
  }
  __syncthreads();
  for (int32_t e = s + int32_t(threadIdx.x); e < t; e += 256) long_ent[atomicAdd(&bin[bin_of(e)], 1)] = e - e0;
}

// cells of the projection rows, row by row; long_ent (when given) is the order
// of their entries
__global__ void k_long_fill(const uint32_t* word, int64_t e0, int64_t nnz, const int32_t* long_ent, uint32_t cell0,
                            const int32_t* vinv, const uint8_t* deg, int64_t n_free, uint32_t* cell_word,
                            uint32_t* ent_cell, uint32_t* vpos) {
  const int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (p >= nnz - e0) return;
  const int64_t e = e0 + (long_ent ? long_ent[p] : p);
  const uint32_t w = word[e], c = cell0 + uint32_t(p);
  int32_t v;
  cell_word[c] = cell_word_of(w, vinv, deg, &v);
  ent_cell[e] = c;
  vpos[size_t((w >> W_SLOT_SHIFT) & 7u) * n_free + v] = c;
}

// long rows: sort key, Y projection rows (full row index rrow_orig at least
// first_y_full) first, each kind by the rank of its face (read off the row's
// first entry: all its elements have that face); *n_y counts the Y rows
__global__ void k_long_keys(const int32_t* rrow_ptr, const int32_t* rrow_orig, const uint32_t* word,
                            const uint32_t* vkey, int64_t n_short, int64_t n_long, int64_t first_y_full, int ybits,
                            int kbits, uint32_t* key, int32_t* val, int32_t* n_y) {
  const int64_t l = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (l >= n_long) return;
  const int64_t j = n_short + l;
  const uint32_t k = vkey[word[rrow_ptr[j]] & W_VAR_MASK];
  const bool y = rrow_orig[j] >= first_y_full;
  key[l] = y ? (k & ((1u << ybits) - 1u)) : ((1u << kbits) | (k >> ybits));
  val[l] = int32_t(l);
  if (y) atomicAdd(n_y, 1);
}

// first cell and length of the projection rows in launch order
__global__ void k_long_rows(const int32_t* perm, const int32_t* rrow_ptr, int64_t n_short, int64_t n_long,
                            uint32_t cell0, int2* row) {
  const int64_t l = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (l >= n_long) return;
  const int64_t j = n_short + perm[l];
  row[l] = make_int2(int32_t(cell0 + uint32_t(rrow_ptr[j] - rrow_ptr[n_short])), rrow_ptr[j + 1] - rrow_ptr[j]);
}

// ---------------------------------------------------------------- short rows left to the chunks
__global__ void k_perm_len(const int32_t* perm, const int32_t* rrow_ptr, const int32_t* rrow_b, int64_t n,
                           int32_t* len, int32_t* pb) {
  const int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const int32_t j = perm[k];
  len[k] = rrow_ptr[j + 1] - rrow_ptr[j];
  pb[k] = rrow_b[j];
}

__global__ void k_perm_entries(const int32_t* perm, const int32_t* rrow_ptr, const int32_t* prow_ptr, int64_t n,
                               int32_t* pent) {
  const int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const int32_t j = perm[k], s = rrow_ptr[j], o = prow_ptr[k], m = rrow_ptr[j + 1] - s;
  for (int32_t e = 0; e < m; ++e) pent[o + e] = s + e;
}

// Rows are packed greedily, in order, into wave chunks of at most 64 entries
// (one entry per lane, whole rows only).  The greedy walk runs in parallel
// over segments of PACK_SEG entries: segment j holds the rows whose first
// entry lies in [j*PACK_SEG, (j+1)*PACK_SEG).
__global__ void k_seg_rows(const int32_t* row_ptr, int64_t n_rows, int32_t n_seg, int32_t* seg_row) {
  int32_t j = int32_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (j > n_seg) return;
  if (j == n_seg) {
    seg_row[j] = int32_t(n_rows);
    return;
  }
  int64_t target = int64_t(j) * PACK_SEG;
  int64_t lo = 0, hi = n_rows;
  while (lo < hi) {
    int64_t mid = (lo + hi) >> 1;
    if (row_ptr[mid] < target) lo = mid + 1;
    else hi = mid;
  }
  seg_row[j] = int32_t(lo);
}

// One block per segment: the segment's row pointers are staged in LDS (a
// segment starts at most PACK_SEG / 2 rows, since every presolved row has at
// least two entries), then one thread walks them.  fill == 0: count the
// chunks of each segment; fill == 1: write their (first row, rows, first
// entry, entries) at the scanned offsets.
__global__ __launch_bounds__(256) void k_pack(const int32_t* seg_row, const int32_t* row_ptr, int32_t n_seg,
                                              int32_t* count, const int32_t* offset, int4* desc, int fill) {
  __shared__ int32_t rp[PACK_SEG / 2 + 1];
  const int32_t j = blockIdx.x;
  const int32_t rs = seg_row[j], nr = seg_row[j + 1] - rs;
  if (nr > PACK_SEG / 2) return;   // excluded by the caller's check
  for (int32_t i = threadIdx.x; i <= nr; i += blockDim.x) rp[i] = row_ptr[rs + i];
  __syncthreads();
  if (threadIdx.x != 0) return;
  int32_t r = 0, c = 0, o = fill ? offset[j] : 0;
  while (r < nr) {
    const int32_t q0 = r, e0 = rp[r];
    // extend the chunk while the next row still fits, eight row pointers per step
    for (;;) {
      int32_t v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = r + 1 + u <= nr ? rp[r + 1 + u] : INT32_MAX;
      int adv = 0;
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (adv == u && r + u < nr && v[u] - e0 <= 64) adv = u + 1;
      r += adv;
      if (adv < 8) break;
    }
    if (fill) desc[o + c] = make_int4(rs + q0, r - q0, e0, rp[r] - e0);
    ++c;
  }
  if (!fill) count[j] = c;
}

// per chunk, the positions (relative to its first entry) where its rows start
__global__ void k_chunk_mask(const int4* desc, const int32_t* row_ptr, int32_t n_chunks,
                             unsigned long long* mask) {
  const int32_t c = int32_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (c >= n_chunks) return;
  const int4 d = desc[c];
  unsigned long long m = 0ull;
  for (int32_t r = 0; r < d.y; ++r) m |= 1ull << (row_ptr[d.x + r] - d.z);
  mask[c] = m;
}

// Cells of every chunk: one wave per chunk, lane e its entry e; the sign mask
// and the right-hand side of each entry's row go beside them, so that a wave
// reads its entries without first reading the chunk descriptor.
__global__ __launch_bounds__(256) void k_chunk_fill(const int4* desc, const unsigned long long* mask,
                                                    const int32_t* pent, const int32_t* row_b, int32_t n_chunks,
                                                    uint32_t cell0, const uint32_t* word, const int32_t* vinv,
                                                    const uint8_t* deg, int64_t n_free, uint32_t* cell_word,
                                                    uint32_t* ent_cell, uint32_t* vpos, unsigned long long* neg,
                                                    int8_t* pb) {
  const int32_t c = int32_t(blockIdx.x) * 4 + int32_t(threadIdx.x >> 6);
  if (c >= n_chunks) return;   // uniform across the wave
  const int e = int(threadIdx.x & 63);
  const int4 d = desc[c];
  bool ng = false;
  int8_t b = 0;
  if (e < d.w) {
    const unsigned long long below = mask[c] & (e == 63 ? ~0ull : ((2ull << e) - 1ull));
    const int32_t src = pent[d.z + e];
    const uint32_t w = word[src], cell = cell0 + uint32_t(c) * 64u + uint32_t(e);
    int32_t v;
    cell_word[cell] = cell_word_of(w, vinv, deg, &v);
    ent_cell[src] = cell;
    vpos[size_t((w >> W_SLOT_SHIFT) & 7u) * n_free + v] = cell;
    b = int8_t(row_b[d.x + __popcll(below) - 1]);
    ng = (w & W_NEG) != 0;
  }
  const unsigned long long m = __ballot(ng);
  if (e == 0) neg[c] = m;
  pb[size_t(c) * 64 + e] = b;
}

// Morton rank of every face of a mesh and the owner ranks of its edges and vertices
dm_status mesh_ranks(dm_ctx* ctx, MeshDev& M, DArr<int32_t>& frank, DArr<int32_t>& erank, DArr<int32_t>& vrank) {
  hipStream_t st = ctx->stream;
  DArr<float> box;
  DArr<uint32_t> fkey;
  DArr<int32_t> forder;
  DM_ALLOC(ctx, box, 6);
  DM_ALLOC(ctx, fkey, size_t(M.nf));
  DM_ALLOC(ctx, forder, size_t(M.nf));
  DM_ALLOC(ctx, frank, size_t(M.nf));
  DM_ALLOC(ctx, erank, size_t(M.ne));
  DM_ALLOC(ctx, vrank, size_t(M.nv));
  k_bbox<<<1, 256, 0, st>>>(M.verts.p, M.nv, box.p);
  k_face_morton<<<grid_for(M.nf, 256), 256, 0, st>>>(M.verts.p, M.faces.p, M.nf, box.p, fkey.p, forder.p);
  DM_LAUNCH_CHECK(ctx);
  DM_TRY(sort_pairs_u32(ctx, fkey.p, forder.p, size_t(M.nf), 30));
  k_rank_of<<<grid_for(M.nf, 256), 256, 0, st>>>(forder.p, M.nf, frank.p);
  k_fill_i32<<<grid_for(M.ne, 256), 256, 0, st>>>(erank.p, M.ne, INT32_MAX);
  k_fill_i32<<<grid_for(M.nv, 256), 256, 0, st>>>(vrank.p, M.nv, INT32_MAX);
  k_elem_rank<<<grid_for(M.nf, 256), 256, 0, st>>>(M.faces.p, M.face_edge.p, frank.p, M.nf, erank.p, vrank.p);
  DM_LAUNCH_CHECK(ctx);
  return DM_OK;
}

// ---------------------------------------------------------------- order of the bound's terms
// A quasi-Newton search compares bounds.  Where the relaxation is tight these
// differ in their last bits only, so the order in which the rows' terms are
// added decides the steps that the search takes.  In FP64 the terms are therefore
// added in one order, whichever way the rows are launched: the one in which the
// earlier sweep over records dealt them to the eight XCDs, so that searches take
// the steps that they took with it.  The tile rows by their smallest X rank and
// row number, 256 to a block; the chunks, four to a block; the projection rows by
// (region, key), where the regions are the eighths of all entries in key order, an
// X row has the key of its face and the Y rows are dealt to the regions in turn.
// In FP32 the blocks' sums are added as launched: what the order changes there,
// the last bits of an FP64 sum, lies far below the terms' own rounding of 2^-24, and
// a step that hangs on it may change with the layout.
constexpr int NREG = 8;

// what needs no order yet, in one launch: vpos with the variables in canonical
// order, the row counts in variable order, the inverses of the two row orders,
// empty regions, and zeros in the places past the last row
__global__ void k_term_start(const uint32_t* vpos, const int32_t* vinv, const uint8_t* vdeg, int64_t n, uint32_t* cpos,
                             int32_t* deg, const int32_t* short_perm, int64_t n_short, int32_t* short_slot,
                             const int32_t* long_perm, int64_t n_long, int32_t* long_slot, int64_t n_terms,
                             double* terms, int32_t* bounds, uint32_t* arrived) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) {
    const int32_t v = vinv[i];
#pragma unroll
    for (int q = 0; q < 5; ++q) cpos[q * n + i] = vpos[q * n + v];
    deg[i] = vdeg[i];
  }
  if (i < n_short) short_slot[short_perm[i]] = int32_t(i);
  if (i < n_long) long_slot[long_perm[i]] = int32_t(i);
  if (i < n_terms) terms[i] = 0.0;
  if (i < 2 * NREG) bounds[i] = (i & 1) ? -2 : -1;
  if (i == 0) *arrived = 0u;
}

// pre[k]: entries of the variables of keys below k, for k = 0 .. nkeys, from
// their running sum in variable order
__global__ void k_key_prefix(const uint32_t* vkey, const int32_t* vperm, const int32_t* sum, int ybits, int64_t n,
                             int32_t nkeys, int32_t* pre) {
  const int64_t v = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (v > n) return;
  const int32_t hi = v < n ? int32_t(vkey[vperm[v]] >> ybits) : nkeys;
  int32_t lo = v > 0 ? int32_t(vkey[vperm[v - 1]] >> ybits) : -1;
  while (lo < hi) pre[++lo] = sum[v];
}

// region of a key: the eighth in which the middle of its own entries falls
__device__ inline int32_t key_region(const int32_t* pre, int32_t k, int64_t total) {
  const int64_t mid2 = int64_t(pre[k]) + pre[k + 1];
  const int64_t r = total > 0 ? (NREG * mid2) / (2 * total) : 0;
  return int32_t(r < 0 ? 0 : (r >= NREG ? NREG - 1 : r));
}

// first and last key of every region (bounds[2 r], bounds[2 r + 1]; k_term_start
// wrote -1 and -2); regions never decrease with the key
__global__ void k_region_keys(const int32_t* pre, int32_t nkeys, int64_t total, int32_t* bounds) {
  const int32_t k = int32_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (k >= nkeys) return;
  const int32_t r = key_region(pre, k, total);
  if (k == 0 || key_region(pre, k - 1, total) != r) bounds[2 * r] = k;
  if (k == nkeys - 1 || key_region(pre, k + 1, total) != r) bounds[2 * r + 1] = k;
}

// tile rows first (their place in cell order, slot, is below n_tile), by the
// smallest X rank of their entries
__global__ void k_term_keys(const int32_t* rrow_ptr, const uint32_t* word, const uint32_t* vkey, const int32_t* slot,
                            int64_t n_short, int64_t n_tile, int ybits, int kbits, uint32_t* key, int32_t* val) {
  const int64_t j = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (j >= n_short) return;
  const bool tile = slot[j] < n_tile;
  uint32_t m = tile ? 0xFFFFFFFFu : 0u;
  if (tile)
    for (int32_t e = rrow_ptr[j]; e < rrow_ptr[j + 1]; ++e) m = min(m, vkey[word[e] & W_VAR_MASK] >> ybits);
  if (rrow_ptr[j] == rrow_ptr[j + 1]) m = 0u;
  key[j] = (tile ? 0u : (1u << kbits)) | m;
  val[j] = int32_t(j);
}

// projection rows: (region, key); first_y_full as in k_long_keys, n_y Y rows,
// which are the last of the projection rows; a generic problem's rows all take
// their smallest key (one wave per row)
__global__ void k_term_long_keys(const int32_t* rrow_ptr, const int32_t* rrow_orig, const uint32_t* word,
                                 const uint32_t* vkey, int64_t n_short, int64_t n_long, int64_t first_y_full,
                                 int64_t n_y, int ybits, int kbits, const int32_t* pre, int64_t total,
                                 const int32_t* bounds, uint32_t* key, int32_t* val) {
  const int64_t l = int64_t(blockIdx.x) * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (l >= n_long) return;   // uniform across the wave
  const int64_t j = n_short + l;
  int32_t r, k;
  if (rrow_orig[j] < first_y_full) {
    uint32_t m = 0x7FFFFFFFu;
    for (int32_t e = rrow_ptr[j] + int32_t(threadIdx.x & 63); e < rrow_ptr[j + 1]; e += 64)
      m = min(m, vkey[word[e] & W_VAR_MASK] >> ybits);
    for (int off = 32; off > 0; off >>= 1) m = min(m, uint32_t(__shfl_xor(int(m), off)));
    k = m == 0x7FFFFFFFu ? 0 : int32_t(m);
    r = key_region(pre, k, total);
  } else {
    const int64_t o = l - (n_long - n_y);
    r = int32_t(o % NREG);
    const int64_t per = (n_y - r + NREG - 1) / NREG;   // Y rows of region r
    const int32_t lo = bounds[2 * r], hi = bounds[2 * r + 1];
    const int64_t span = hi >= lo ? int64_t(hi) - lo + 1 : 1;
    k = int32_t((hi >= lo ? lo : 0) + ((o / NREG) * span) / (per > 0 ? per : 1));
  }
  if ((threadIdx.x & 63) == 0) {
    key[l] = (uint32_t(r) << kbits) | uint32_t(k);
    val[l] = int32_t(l);
  }
}

// place[slot of the k-th row in order] = k: slot is the row's number in the
// order that the sweep counts in
__global__ void k_term_place(const int32_t* order, const int32_t* slot, int64_t n, int32_t* place) {
  const int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (k < n) place[slot[order[k]]] = int32_t(k);
}

// The same for few rows without the sort: one wave counts the rows before its
// own by (key, row number).  4000 rows 11 us, 16384 rows 92 us, the sort's
// dozen launches 150 us at either size.
constexpr int64_t RANK_BY_COUNT = 16384;

__global__ __launch_bounds__(256) void k_rank_place(const uint32_t* key, const int32_t* slot, int32_t n,
                                                    int32_t n_place, int32_t* place) {
  const int32_t j = int32_t(blockIdx.x) * 4 + int32_t(threadIdx.x >> 6);
  if (j >= n) return;   // uniform across the wave
  const uint32_t mine = key[j];
  int32_t before = 0;
  for (int32_t m = int32_t(threadIdx.x & 63); m < n; m += 64) {
    const uint32_t k = key[m];
    before += (k < mine || (k == mine && m < j)) ? 1 : 0;
  }
  for (int off = 32; off > 0; off >>= 1) before += __shfl_xor(before, off);
  if ((threadIdx.x & 63) == 0 && before < n_place) place[slot[j]] = before;
}

}  // namespace

// mean projection-row length above which a projection row gets a whole block
constexpr int64_t LONG_BLOCK_ROW = 512;

// largest X mesh: the size up to which the library answers for the layout
constexpr int32_t MAX_KEY_FACES = 16384;

dm_status sweep_layout(dm_ctx* ctx) {
  hipStream_t st = ctx->stream;
  const int64_t nfree = ctx->n_free, nr = ctx->n_rows, nshort = ctx->n_short, rnnz = ctx->nnz;
  const int64_t nlong = nr - nshort;
  const size_t nf1 = size_t(std::max<int64_t>(nfree, 1));
  const bool mesh = !ctx->generic && ctx->X.nf > 0;
  if (mesh && nfree > 0 && ctx->X.nf > MAX_KEY_FACES)
    return dm_fail(ctx, DM_ERR_WORKSPACE, "sweep layout: %d faces exceed %d key bins", ctx->X.nf, MAX_KEY_FACES);
  // ---- variable keys and the variable order; a product space has fewer than
  // 2^31 slots, so the two ranks of an element together fit 32 bits
  const int xbits = bits_for(mesh ? uint64_t(ctx->X.nf) : uint64_t(std::max<int64_t>(nfree, 1)));
  const int ybits = mesh ? bits_for(uint64_t(ctx->Y.nf)) : 0;
  DArr<uint32_t> vsort;
  DArr<uint32_t>& vkey = ctx->vkey;
  DM_ALLOC(ctx, vkey, nf1);
  ctx->has_bound_order = false;
  DM_ALLOC(ctx, ctx->vperm, nf1);
  DM_ALLOC(ctx, ctx->vinv, nf1);
  DM_ALLOC(ctx, ctx->vdeg, nf1);
  if (mesh) {
    DArr<int32_t> xf, xe, xv, yf, ye, yv;
    DM_TRY(mesh_ranks(ctx, ctx->X, xf, xe, xv));
    DM_TRY(mesh_ranks(ctx, ctx->Y, yf, ye, yv));
    DM_ALLOC(ctx, vsort, nf1);
    if (nfree > 0) {
      k_var_keys<<<grid_for(nfree, 256), 256, 0, st>>>(ctx->free_var.p, ctx->code.p, xf.p, xe.p, xv.p, yf.p, ye.p,
                                                       yv.p, ybits, nfree, vkey.p, vsort.p, ctx->vperm.p);
      DM_LAUNCH_CHECK(ctx);
      DM_TRY(sort_pairs_u32(ctx, vsort.p, ctx->vperm.p, size_t(nfree), xbits + ybits));
    }
  } else if (nfree > 0) {
    k_iota2<<<grid_for(nfree, 256), 256, 0, st>>>(vkey.p, ctx->vperm.p, nfree);
  }
  if (nfree > 0)
    k_var_order<<<grid_for(nfree, 256), 256, 0, st>>>(ctx->vperm.p, ctx->var_deg.p, nfree, ctx->vinv.p, ctx->vdeg.p);
  DM_LAUNCH_CHECK(ctx);

  // ---- order of the short rows and of the projection rows.  The low bits of
  // the Y rank are dropped where that saves the sort a pass (24 bits are three
  // passes); neighbouring ranks then keep the row order.
  const int full = xbits + ybits + 2;
  const int ydrop = full > 32 ? full - 32 : (full > 24 && full <= 26 && ybits > 2 ? full - 24 : 0);
  const int kbits = xbits + ybits - ydrop;
  DArr<uint32_t> skey, lkey;
  DArr<int32_t> count;
  DArr<int32_t>& perm = ctx->short_perm;
  DM_ALLOC(ctx, skey, size_t(std::max<int64_t>(nshort, 1)));
  DM_ALLOC(ctx, perm, size_t(std::max<int64_t>(nshort, 1)));
  DM_ALLOC(ctx, lkey, size_t(std::max<int64_t>(nlong, 1)));
  DM_ALLOC(ctx, ctx->long_perm, size_t(std::max<int64_t>(nlong, 1)));
  constexpr int NC = TILE_FORMS + 2;
  DM_ALLOC(ctx, count, NC);
  DM_HIP(ctx, hipMemsetAsync(count.p, 0, NC * sizeof(int32_t), st));
  if (nshort > 0) {
    // the narrowest tiles only where one workgroup may sweep the problem from LDS
    // and its arithmetic counts: rows of one place spread over more tiles cost
    // the variable pass cache lines (2000/3000-face pair 7 us more of 108
    // an iteration with them, 1000 faces 0.6 of 22)
    const uint32_t form0 = rnnz <= SMALL_NNZ[0] ? 0u : 1u;
    k_short_keys<<<grid_for(nshort, 256), 256, 0, st>>>(ctx->rrow_ptr.p, ctx->rrow_b.p, ctx->rent_word.p, vkey.p,
                                                        nshort, ybits, ydrop, kbits, form0, skey.p, perm.p, count.p);
    DM_LAUNCH_CHECK(ctx);
    DM_TRY(sort_pairs_u32(ctx, skey.p, perm.p, size_t(nshort), kbits + 2));
  }
  if (nlong > 0) {
    const int lbits = std::max(xbits, ybits);
    const int64_t first_y_full = mesh ? ctx->n_closed_full + ctx->X.nf : INT64_MAX;
    k_long_keys<<<grid_for(nlong, 256), 256, 0, st>>>(ctx->rrow_ptr.p, ctx->rrow_orig.p, ctx->rent_word.p, vkey.p,
                                                      nshort, nlong, first_y_full, ybits, lbits, lkey.p,
                                                      ctx->long_perm.p, count.p + TILE_FORMS + 1);
    DM_LAUNCH_CHECK(ctx);
    DM_TRY(sort_pairs_u32(ctx, lkey.p, ctx->long_perm.p, size_t(nlong), lbits + 1));
  }
  int32_t cnt[NC];
  {
    const int32_t* src[NC];
    for (int k = 0; k < NC; ++k) src[k] = count.p + k;
    DM_TRY(read_i32s(ctx, NC, src, cnt));
  }
  const int32_t* n_tile_rows = cnt;
  const int32_t nnz_chunk = int32_t(ctx->nnz_short) - cnt[TILE_FORMS];   // entries of the short rows left to the chunks
  ctx->n_long_y = cnt[TILE_FORMS + 1];
  ctx->long_wpr = (nlong > 0 && (rnnz - ctx->nnz_short) / nlong > LONG_BLOCK_ROW) ? 4 : 1;

  // ---- the chunks: the remaining short rows in key order, packed greedily
  int32_t form_row0[TILE_FORMS + 1] = {0};   // first row of each form in perm
  for (int f = 0; f < TILE_FORMS; ++f) form_row0[f + 1] = form_row0[f] + n_tile_rows[f];
  const int64_t nchr = nshort - form_row0[TILE_FORMS];
  const int32_t* cperm = perm.p + form_row0[TILE_FORMS];
  DArr<int32_t> plen, prow_ptr, pb, pent;
  int32_t n_chunks = 0;
  if (nchr > 0) {
    DM_ALLOC(ctx, plen, size_t(nchr));
    DM_ALLOC(ctx, pb, size_t(nchr));
    DM_ALLOC(ctx, prow_ptr, size_t(nchr) + 1);
    k_perm_len<<<grid_for(nchr, 256), 256, 0, st>>>(cperm, ctx->rrow_ptr.p, ctx->rrow_b.p, nchr, plen.p, pb.p);
    DM_LAUNCH_CHECK(ctx);
    DM_TRY(scan_i32(ctx, plen.p, prow_ptr.p, size_t(nchr)));
    DM_ALLOC(ctx, pent, size_t(std::max(nnz_chunk, 1)));
    k_perm_entries<<<grid_for(nchr, 256), 256, 0, st>>>(cperm, ctx->rrow_ptr.p, prow_ptr.p, nchr, pent.p);
    const int32_t n_seg = int32_t((int64_t(nnz_chunk) + PACK_SEG - 1) / PACK_SEG);
    DArr<int32_t> seg_row, seg_cnt, seg_off;
    DM_ALLOC(ctx, seg_row, size_t(n_seg) + 1);
    DM_ALLOC(ctx, seg_cnt, size_t(std::max(n_seg, 1)));
    DM_ALLOC(ctx, seg_off, size_t(n_seg) + 1);
    k_seg_rows<<<grid_for(n_seg + 1, 256), 256, 0, st>>>(prow_ptr.p, nchr, n_seg, seg_row.p);
    if (n_seg > 0)
      k_pack<<<unsigned(n_seg), 256, 0, st>>>(seg_row.p, prow_ptr.p, n_seg, seg_cnt.p, nullptr, nullptr, 0);
    DM_LAUNCH_CHECK(ctx);
    DM_TRY(scan_i32(ctx, seg_cnt.p, seg_off.p, size_t(n_seg)));
    DM_TRY(read_i32(ctx, seg_off.p + n_seg, &n_chunks));
    DM_ALLOC(ctx, ctx->chunk_desc, size_t(std::max(n_chunks, 1)));
    DM_ALLOC(ctx, ctx->chunk_mask, size_t(std::max(n_chunks, 1)));
    DM_ALLOC(ctx, ctx->chunk_neg, size_t(std::max(n_chunks, 1)));
    DM_ALLOC(ctx, ctx->chunk_b, size_t(std::max(n_chunks, 1)) * 64);
    if (n_seg > 0)
      k_pack<<<unsigned(n_seg), 256, 0, st>>>(seg_row.p, prow_ptr.p, n_seg, nullptr, seg_off.p, ctx->chunk_desc.p,
                                              1);
    if (n_chunks > 0)
      k_chunk_mask<<<grid_for(n_chunks, 256), 256, 0, st>>>(ctx->chunk_desc.p, prow_ptr.p, n_chunks,
                                                            ctx->chunk_mask.p);
    DM_LAUNCH_CHECK(ctx);
  }

  // ---- cells: tiles by form, chunks, projection rows, the zero cell
  ctx->n_chunks = n_chunks;
  int64_t chunk0 = 0;
  for (int f = 0; f < TILE_FORMS; ++f) {
    ctx->tile_rows[f] = n_tile_rows[f];
    ctx->n_tiles[f] = (n_tile_rows[f] + 63) / 64;
    ctx->tile_cell0[f] = chunk0;
    chunk0 += int64_t(ctx->n_tiles[f]) * 128 * TILE_HALF[f];
  }
  const int64_t long0 = chunk0 + int64_t(n_chunks) * 64;
  const int64_t ncell = long0 + (rnnz - ctx->nnz_short);
  if (ncell >= int64_t(CHUNK_PAD)) return dm_fail(ctx, DM_ERR_WORKSPACE, "sweep layout: too many cells");
  ctx->chunk_cell0 = chunk0;
  ctx->long_cell0 = long0;
  ctx->n_cells = ncell;
  DM_ALLOC(ctx, ctx->cell_word, size_t(std::max<int64_t>(ncell, 1)));
  DM_ALLOC(ctx, ctx->ent_cell, size_t(std::max<int64_t>(rnnz, 1)));
  DM_ALLOC(ctx, ctx->vpos, 5 * nf1);
  if (long0 > 0) DM_HIP(ctx, hipMemsetAsync(ctx->cell_word.p, 0xFF, sizeof(uint32_t) * size_t(long0), st));
  if (nfree > 0)
    k_unused_slots<<<grid_for(nfree, 256), 256, 0, st>>>(ctx->vdeg.p, nfree, uint32_t(ncell), ctx->vpos.p);
  for (int f = 0; f < TILE_FORMS; ++f)
    if (n_tile_rows[f] > 0)
      k_tile_fill<<<grid_for(n_tile_rows[f], 256), 256, 0, st>>>(
          perm.p + form_row0[f], n_tile_rows[f], TILE_HALF[f], uint32_t(ctx->tile_cell0[f]), ctx->rrow_ptr.p,
          ctx->rent_word.p, ctx->vinv.p, ctx->var_deg.p, nfree, ctx->cell_word.p, ctx->ent_cell.p, ctx->vpos.p);
  if (n_chunks > 0)
    k_chunk_fill<<<grid_for(n_chunks, 4), 256, 0, st>>>(ctx->chunk_desc.p, ctx->chunk_mask.p, pent.p, pb.p, n_chunks,
                                                        uint32_t(chunk0), ctx->rent_word.p, ctx->vinv.p,
                                                        ctx->var_deg.p, nfree, ctx->cell_word.p, ctx->ent_cell.p,
                                                        ctx->vpos.p, ctx->chunk_neg.p, ctx->chunk_b.p);
  // Entries of the projection rows in the order of the meshes: a Y row's
  // neighbouring cells then belong to neighbouring X elements, whose variables
  // the same XCD gathers at nearly the same time.  A generic problem's
  // variables are in the order of its rows as they are.
  const int64_t nl = rnnz - ctx->nnz_short;
  DM_ALLOC(ctx, ctx->long_row, size_t(std::max<int64_t>(nlong, 1)));
  if (nl > 0) {
    k_long_rows<<<grid_for(nlong, 256), 256, 0, st>>>(ctx->long_perm.p, ctx->rrow_ptr.p, nshort, nlong,
                                                      uint32_t(long0), ctx->long_row.p);
    if (mesh) {
      DM_ALLOC(ctx, ctx->long_ent, size_t(nl));
      const int bb = bits_for(uint64_t(RANK_BINS - 1));
      k_long_order<<<unsigned(nlong), 256, 0, st>>>(ctx->rrow_ptr.p, ctx->rrow_orig.p, ctx->rent_word.p, vkey.p, nshort,
                                                    ctx->n_closed_full + ctx->X.nf, ybits, std::max(0, xbits - bb),
                                                    std::max(0, ybits - bb), ctx->long_ent.p);
    } else {
      ctx->long_ent.release();
    }
    k_long_fill<<<grid_for(nl, 256), 256, 0, st>>>(ctx->rent_word.p, ctx->nnz_short, rnnz, ctx->long_ent.p,
                                                   uint32_t(long0), ctx->vinv.p, ctx->var_deg.p, nfree,
                                                   ctx->cell_word.p, ctx->ent_cell.p, ctx->vpos.p);
  }
  DM_LAUNCH_CHECK(ctx);
  return DM_OK;
}

// place[slot[row]] for the first n_place of n rows in order of (key, row number);
// order: the row numbers, and scratch
static dm_status place_rows(dm_ctx* ctx, uint32_t* key, int32_t* order, const int32_t* slot, int64_t n,
                            int64_t n_place, int bits, int32_t* place) {
  if (n <= RANK_BY_COUNT) {
    k_rank_place<<<grid_for(n, 4), 256, 0, ctx->stream>>>(key, slot, int32_t(n), int32_t(n_place), place);
  } else {
    DM_TRY(sort_pairs_u32(ctx, key, order, size_t(n), bits));
    k_term_place<<<grid_for(n_place, 256), 256, 0, ctx->stream>>>(order, slot, n_place, place);
  }
  DM_LAUNCH_CHECK(ctx);
  return DM_OK;
}

dm_status bound_order(dm_ctx* ctx) {
  if (ctx->has_bound_order) return DM_OK;
  hipStream_t st = ctx->stream;
  const int64_t nfree = ctx->n_free, nshort = ctx->n_short, nlong = ctx->n_rows - nshort, total = ctx->nnz;
  const bool mesh = !ctx->generic && ctx->X.nf > 0;
  const int32_t nkeys = mesh ? ctx->X.nf : int32_t(std::max<int64_t>(nfree, 1));
  const int ybits = mesh ? bits_for(uint64_t(ctx->Y.nf)) : 0, kbits = bits_for(uint64_t(nkeys));
  const int64_t ntile = int64_t(ctx->tile_rows[0]) + ctx->tile_rows[1] + ctx->tile_rows[2];
  ctx->term_tiles = int32_t((ntile + 255) / 256);
  ctx->term_chunks = (ctx->n_chunks + 3) / 4;
  const int32_t nb = ctx->term_tiles + ctx->term_chunks;
  DArr<unsigned char> tmp;
  uint32_t *skey = nullptr, *lkey = nullptr;
  int32_t *sorder = nullptr, *lorder = nullptr, *sslot = nullptr, *lslot = nullptr;
  int32_t *deg = nullptr, *wsum = nullptr, *pre = nullptr, *bounds = nullptr;
  {
    Slab k;
    k.add<double>(int64_t(nb) * 256 + nlong);
    k.add<double>(nb + nlong);
    k.add<int32_t>(ntile);
    k.add<int32_t>(nlong);
    k.add<uint32_t>(5 * nfree);
    k.add<uint32_t>(1);
    DM_ALLOC(ctx, ctx->term_mem, k.bytes);
    k.at = ctx->term_mem.p;
    ctx->terms = k.take<double>(int64_t(nb) * 256 + nlong);
    ctx->term_part = k.take<double>(nb + nlong);
    ctx->term_row = k.take<int32_t>(ntile);
    ctx->term_long = k.take<int32_t>(nlong);
    ctx->cpos = k.take<uint32_t>(5 * nfree);
    ctx->term_arrived = k.take<uint32_t>(1);
    Slab w;
    for (int q = 0; q < 3; ++q) w.add<int32_t>(nshort);
    for (int q = 0; q < 3; ++q) w.add<int32_t>(nlong);
    w.add<int32_t>(nfree);
    w.add<int32_t>(nfree + 1);
    w.add<int32_t>(nkeys + 1);
    w.add<int32_t>(2 * NREG);
    DM_ALLOC(ctx, tmp, w.bytes);
    w.at = tmp.p;
    skey = w.take<uint32_t>(nshort);
    sorder = w.take<int32_t>(nshort);
    sslot = w.take<int32_t>(nshort);
    lkey = w.take<uint32_t>(nlong);
    lorder = w.take<int32_t>(nlong);
    lslot = w.take<int32_t>(nlong);
    deg = w.take<int32_t>(nfree);
    wsum = w.take<int32_t>(nfree + 1);
    pre = w.take<int32_t>(nkeys + 1);
    bounds = w.take<int32_t>(2 * NREG);
  }
  const int64_t most = std::max({nfree, nshort, nlong, int64_t(nb) * 256, int64_t(2 * NREG)});
  k_term_start<<<grid_for(most, 256), 256, 0, st>>>(ctx->vpos.p, ctx->vinv.p, ctx->vdeg.p, nfree, ctx->cpos, deg,
                                                    ctx->short_perm.p, nshort, sslot, ctx->long_perm.p, nlong,
                                                    lslot, int64_t(nb) * 256, ctx->terms, bounds, ctx->term_arrived);
  DM_LAUNCH_CHECK(ctx);
  if (ntile > 0) {
    k_term_keys<<<grid_for(nshort, 256), 256, 0, st>>>(ctx->rrow_ptr.p, ctx->rent_word.p, ctx->vkey.p, sslot, nshort,
                                                       ntile, ybits, kbits, skey, sorder);
    DM_LAUNCH_CHECK(ctx);
    DM_TRY(place_rows(ctx, skey, sorder, sslot, nshort, ntile, kbits + 1, ctx->term_row));
  }
  if (nlong > 0) {
    DM_TRY(scan_i32(ctx, deg, wsum, size_t(nfree)));
    k_key_prefix<<<grid_for(nfree + 1, 256), 256, 0, st>>>(ctx->vkey.p, ctx->vperm.p, wsum, ybits, nfree, nkeys,
                                                           pre);
    k_region_keys<<<grid_for(nkeys, 256), 256, 0, st>>>(pre, nkeys, total, bounds);
    k_term_long_keys<<<grid_for(nlong, 4), 256, 0, st>>>(
        ctx->rrow_ptr.p, ctx->rrow_orig.p, ctx->rent_word.p, ctx->vkey.p, nshort, nlong,
        mesh ? ctx->n_closed_full + ctx->X.nf : INT64_MAX, ctx->n_long_y, ybits, kbits, pre, total, bounds, lkey,
        lorder);
    DM_LAUNCH_CHECK(ctx);
    DM_TRY(place_rows(ctx, lkey, lorder, lslot, nlong, nlong, kbits + 3, ctx->term_long));
  }
  DM_LAUNCH_CHECK(ctx);
  ctx->has_bound_order = true;
  return DM_OK;
}

TermSums term_sums(const dm_ctx* ctx) {
  TermSums T;
  T.terms = ctx->terms;
  T.n_blocks = ctx->term_tiles + ctx->term_chunks;
  T.n_long = int32_t(ctx->n_rows - ctx->n_short);
  T.rpb = 4 / ctx->long_wpr;
  T.n_long_blocks = (T.n_long + T.rpb - 1) / T.rpb;
  T.part = ctx->term_part;
  T.arrived = ctx->term_arrived;
  return T;
}
