// Address arithmetic of the tiled GEMM over packed weights and the choice between
// the prompt attentions, free of HIP so that they are also compiled and enumerated
// on the host (tests/test_tile_plan.py).
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

// Whether prompt rows (n_groups groups of at most 16 rows, the longest prompt ctx
// positions) take the attention whose four waves split the positions
// (attn_mfma_kernel) rather than the one with a wave per head over all of them
// (attn_prompt_kernel).  The first costs a launch about
// workgroups x gqa x hd x (0.9 + ctx / 2000) of the device's time, workgroups =
// n_kv n_groups: a fixed part per workgroup, merge and prologue, and the positions.
// The second is bound by its chain of ctx / 32 stages until the device is full.  Where
// the two meet, us per launch, first / second kernel:
//   hd 64, 4 of 16 heads per group: 1 x 512 rows 14.9 / 21.7, 1 x 2040 59 / 73,
//     2 x 2040 110 / 116, 4 x 2040 204 / 179, 4 x 128 11.9 / 11.9, 4 x 512 30.5 / 28.1,
//     8 x 128 15.0 / 12.5, 16 x 256 41.5 / 28.4
//   hd 128, 4 of 32: 1 x 128 12.7 / 14.1, 1 x 256 16.1 / 18.3, 1 x 512 29.1 / 27.1, 1 x 2040
//     182 / 142, 4 x 128 22.0 / 14.4
//   hd 128, 2 of 16: 1 x 512 19.5 / 25.7, 1 x 2040 100 / 117, 2 x 2040 191 / 199, 4 x 2040
//     369 / 347, 2 x 512 31.4 / 33.4, 4 x 256 25.8 / 22.2
//   hd 64, 8 of 16: 1 x 2040 60 / 80, 2 x 2040 109 / 132, 4 x 2040 200 / 208, 4 x 512
//     30.9 / 27.4
//   groups of one head, hd 128, 8 heads: 1 x 2040 55 / 117, 4 x 2040 195 / 321, 16 x 256
//     44.1 / 45.0 (the first throughout)
constexpr bool prompt_splits_positions(int n_cu, int n_kv, int gqa, int hd, int n_groups, int ctx) {
  return gqa == 1 || (double)n_kv * n_groups * gqa * hd * (0.9 + ctx / 2000.0) < (double)n_cu * ctx;
}

}  // namespace tandem
