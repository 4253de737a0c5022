// partials.h - how the reductions split their rows and items, and the work array of the learned
// preconditioner that follows from it (host arithmetic only).
#pragma once

#include <stdint.h>

#include <algorithm>

namespace sppc {

// Rows per partial sum of the column reductions: about 1024 blocks.  A block has 4 waves and few loads in
// flight each, so 256 blocks leave most of the bandwidth unused: residual of n = 1.17M, 8 columns 62 us with
// 286 blocks (3.6 TB/s), 34 us with 916; sum of squares 40 and 18.6 us.
inline int64_t cr_chunk(int64_t n) {
  int64_t c = (n / 1024 + 255) / 256 * 256;
  return c < 256 ? 256 : (c > 4096 ? 4096 : c);
}
inline int64_t cr_chunks(int64_t n) { return ((n > 0 ? n : 1) + cr_chunk(n) - 1) / cr_chunk(n); }

constexpr int MPNN_NPAR = 289;   // parameters of the network
constexpr int MPNN_SMALL = 1024; // doubles of its work array for values per sample

// rows per partial sum of the loss
inline int64_t ld_chunk(int64_t n) {
  const int64_t c = (n / 1024 + 63) / 64 * 64;
  return c < 64 ? 64 : c;
}
inline int64_t ld_chunks(int64_t n) { return (n + ld_chunk(n) - 1) / ld_chunk(n); }

// (row, sample) items per block of the gradient: enough blocks for 8 per CU, whole quarter tiles
inline int64_t grad_items(int64_t items) {
  const int64_t c = (items / 2048 + 63) / 64 * 64;
  return c < 64 ? 64 : c;
}
inline int64_t grad_blocks(int64_t items) { return (items + grad_items(items) - 1) / grad_items(items); }

// Doubles of the work array that an evaluation of S samples reaches: nine n x S blocks (fr | HF | u | hs |
// Hu | t | tJ | dO | HdO), the values per sample, and the partial sums of the largest of its reductions.
inline int64_t mpnn_work_used(int64_t n, int S) {
  const int64_t grad = grad_blocks(n * S) * MPNN_NPAR, cols = cr_chunks(n) * S, loss = 3 * ld_chunks(n) * S;
  return 9 * n * S + MPNN_SMALL + std::max({grad, cols, loss});
}

// Its size for any number of samples up to S (the array is kept from a larger evaluation for a smaller one).
// The gradient's blocks do not grow with the items everywhere: 2080 of 64 items at 133119 items (items / 2048
// is rounded down before it is rounded up to 64), 1040 of 128 at 133120.  So they enter by a bound that does.
inline int64_t mpnn_work_doubles(int64_t n, int S) {
  const int64_t grad = std::min<int64_t>((n * S + 63) / 64, 2080) * MPNN_NPAR;
  const int64_t cols = cr_chunks(n) * S, loss = 3 * ld_chunks(n) * S;
  return 9 * n * S + MPNN_SMALL + std::max({grad, cols, loss});
}

}  // namespace sppc
