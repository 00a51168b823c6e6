// Address arithmetic of the tiled GEMM over packed weights, free of HIP so that
// it is also compiled and enumerated on the host (tests/test_tile_plan.py).
#pragma once

namespace tandem {

// Byte offset, from the tile's first 32-row weight block, of the 1 KB fragment
// that DMA instruction f fetches for the 32-wide chunk kc: block f / 2 of the
// tile, k-step f % 2.  kfr: fragments per block (K / 16); blocks: blocks of the
// matrix from the tile's first one on.  A tile that reaches past the matrix
// fetches the last block again (its results are not stored).  The clamp is what
// keeps the load inside the matrix: the offset is the load's uniform one, which
// a raw buffer's range check does not cover.
constexpr int tile_weight_offset(int f, int kc, int kfr, int blocks) {
  const int b = (f >> 1) < blocks ? f >> 1 : blocks - 1;
  return (b * kfr + 2 * kc + (f & 1)) * 1024;
}

}  // namespace tandem
