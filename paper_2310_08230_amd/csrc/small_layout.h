// LDS of the one-workgroup form of the hard sweep (k_small in dual.hip), used by
// the kernel and by the host that sizes it: the cells with the zero cell, one
// residual per variable, and, where the problem has chunks, one slice per wave,
// which short_chunk_hard reads 16 bytes at a time.
#pragma once

#include <cstdint>

constexpr int CHUNK_SLICE = 192;   // reals of a wave's slice: three 64-value lists

// first real of the slices: the next 16-byte boundary
template <typename R>
constexpr int64_t small_slices_at(int64_t n_cells, int64_t n_vars) {
  constexpr int64_t V = 16 / int64_t(sizeof(R));
  return (n_cells + 1 + n_vars + V - 1) / V * V;
}

// reals in all
template <typename R>
constexpr int64_t small_reals(int64_t n_cells, int64_t n_vars, bool chunks, int64_t waves) {
  return chunks ? small_slices_at<R>(n_cells, n_vars) + waves * CHUNK_SLICE : n_cells + 1 + n_vars;
}
