// Launch geometry that depends on the caller's sizes alone (plain C++, checked on the host): a dimension
// of a grid has fewer than 2^32 work items, and at most 65535 blocks in y and z.  Kernels whose
// blocks follow a count that the caller chooses freely stride over it with a capped grid.
#pragma once
#include <cstdint>

namespace best {

constexpr int64_t kMaxGridItems = ((int64_t)1 << 32) - 1, kMaxGridYZ = 65535;

// Blocks of a strided launch over `blocks` blocks' worth of work.
inline int64_t capped_blocks(int64_t blocks, int threads) {
  const int64_t cap = kMaxGridItems / threads;
  return blocks < 1 ? 1 : blocks < cap ? blocks : cap;
}

// Projections per batch of the sliced Wasserstein distance of n draws: two key buffers of up to 2^23
// keys, which the last-level cache holds between the passes of a batch, and at most 2^16 projections (four
// to a block in y).
inline int64_t sliced_batch(int64_t n, int64_t n_proj) {
  int64_t p = ((int64_t)1 << 23) / n;
  if (p > (int64_t)1 << 16) p = (int64_t)1 << 16;
  if (p > n_proj) p = n_proj;
  return p < 1 ? 1 : p;
}

}  // namespace best
