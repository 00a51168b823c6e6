// Projection GEMMs of the decoder: C = A . W^T with W [out][in].
//
// bf16 models meet two MFMA kernels here (M > 128 rows, or weights without a
// packed copy; decode-sized M streams the packed weights, see k_stream.hip):
//   * gemm_tile_kernel, over the packed weights: the prefill and the wide
//     batches.  Described at the kernel.
//   * gemm_mfma_kernel, over the row-major weights: matrices without a packed
//     copy.  A holds the activations in split format (per 8 values: 8 bf16
//     high parts, then 8 bf16 low parts), so every weight fragment meets hi
//     and lo in two MFMAs: fp32-level activations, bf16 weights, fp32
//     accumulation.  One workgroup computes a BM x 128 output tile (BM in
//     {32, 64, 128}) over its slice of K, 64 k-values per chunk; 4 waves (8
//     when BM = 128) tile the 32 x 32 MFMA blocks.  Weight rows and
//     activation rows of each chunk stream into an NS-stage LDS ring with
//     global_load_lds_dwordx4 (no register staging); 16-byte pieces are
//     XOR-swizzled by row so the MFMA-layout reads spread over all banks.
// In both, all loads are issued unconditionally, the LDS reads are explicit
// ds_read_b128, and the only waits are compile-time vmcnt/lgkmcnt values plus
// a raw s_barrier: the compiler never sees a memory result it could over-wait
// for, so the ring stays full.  K may be split over the grid; the consuming
// kernel sums the partial tiles in a fixed order, keeping results bitwise
// reproducible.
//
// MFMA operand layout (32x32x16): lane l supplies row/column l % 32 and eight
// k-values of group l / 32; result element i of lane l is column l % 32 of
// row 8 (i / 4) + 4 (l / 32) + i % 4.  Any permutation of k that is the same
// for both operands gives the same dot product, so with row-major weights lane
// group g takes the k range [32 g, 32 g + 32) of each chunk, 8 values per k-step.
//
// fp32 path: a plain LDS-tiled VALU kernel (fp32 models, K not a multiple of 64).
#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "tile_plan.h"

namespace tandem {

namespace {

constexpr int BK = kGemmBK;        // k-values per chunk

__device__ __forceinline__ float silu(float x) { return x / (1.f + expf(-x)); }

template <int BMT, int NST, int NWT> struct GemmShape {
  static constexpr int NW = NWT;                      // waves per workgroup (4 or 8)
  static constexpr int BM = BMT;
  static constexpr int BN = 128;                      // weight rows per tile
  static constexpr int MB = BM / 32;                  // 32-row blocks
  static constexpr int WM = NW == 8 ? (MB >= 4 ? 4 : MB) : (MB >= 2 ? 2 : 1);   // waves along M
  static constexpr int WN = NW / WM;                  // waves along N
  static constexpr int MBW = MB / WM;                 // 32-row blocks per wave
  static constexpr int NBW = BN / 32 / WN;            // 32-column blocks per wave
  static constexpr int NS = NST;                      // ring stages
  static constexpr int PARTS = 2;                     // MFMA operand parts per activation (hi + lo)
  static constexpr int RB = BK * 2 * PARTS;           // bytes of one activation row per chunk
  static constexpr int NPC = RB / 16;                 // 16-byte pieces per activation row
  static constexpr int RPI = 64 / NPC;                // activation rows per 1 KB DMA instruction
  static constexpr int ASTAGE = BM * RB;              // bytes of one activation stage
  static constexpr int WSTAGE = BN * BK * 2;          // bytes of one weight stage
  static constexpr int STAGE = ASTAGE + WSTAGE;
  static constexpr int NA = BM / (RPI * NW);          // activation DMA instructions per wave per chunk
  static constexpr int NWD = BN / (8 * NW);           // weight DMA instructions per wave per chunk
  static constexpr int WAIT = (NS - 2) * (NA + NWD);  // vmcnt that leaves NS - 2 chunks in flight
  static constexpr int OUT_COLS = BN / 2;             // SwiGLU output columns per tile
  static_assert(NS * STAGE <= 160 * 1024, "LDS ring exceeds 160 KB");
  static_assert(NA >= 1 && NWD >= 1 && MBW >= 1 && NBW >= 1, "tile too small for the waves");
};

template <int BMT, int NST, int EPI, int NWT>
__global__ __launch_bounds__(64 * NWT) void gemm_mfma_kernel(
    const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, int M, int N, int K, int cps,
    float* __restrict__ out, int ldo, long split_stride) {
  using G = GemmShape<BMT, NST, NWT>;
  constexpr int PARTS = G::PARTS, NPC = G::NPC;
  __shared__ __attribute__((aligned(1024))) unsigned char ring[G::NS * G::STAGE];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 5, c32 = lane & 31;
  const int wm = wave / G::WN, wn = wave % G::WN;
  const int m0 = blockIdx.y * G::BM;
  const int nch = K / BK;
  const int kc0 = blockIdx.z * cps;
  const int nloc = min(cps, nch - kc0);
  if (nloc <= 0) return;

  // Global weight row of tile row t (0..BN-1).  SwiGLU tiles pair gate and up
  // rows inside every 32-row block: rows 32p .. 32p+15 are gate rows
  // j0 + 16p + c, rows 32p+16 .. 32p+31 the matching up rows; other tiles
  // hold BN consecutive rows.
  auto wrow_of = [&](int t) -> int {
    if (EPI == EPI_SWIGLU) {
      const int j = min(blockIdx.x * G::OUT_COLS + 16 * (t >> 5) + (t & 15), N - 1);
      return ((t >> 4) & 1) ? N + j : j;
    }
    return min(blockIdx.x * G::BN + t, N - 1);
  };

  // DMA sources.  Weight stage: instruction i of wave w covers tile rows
  // (BN/NW) w + 8i .. +8 (128 B each); lane -> row (lane >> 3), physical
  // piece lane & 7 holding logical piece (lane & 7) ^ ((row >> 1) & 7).
  const bf16_t* wsrc[G::NWD];
#pragma unroll
  for (int i = 0; i < G::NWD; ++i) {
    const int t = (G::BN / G::NW) * wave + 8 * i + (lane >> 3);
    const int lp = (lane & 7) ^ ((t >> 1) & 7);
    wsrc[i] = W + (size_t)wrow_of(t) * K + lp * 8;
  }
  // Activation stage: instruction i of wave w covers tile rows RPI (NW i + w) ..
  // +RPI - 1 (a row is NPC 16-byte pieces: split format 8 hi and 8 lo pieces,
  // fp16 8 pieces); physical piece lane % NPC holds logical piece
  // (lane % NPC) ^ (row % NPC).
  const bf16_t* asrc[G::NA];
#pragma unroll
  for (int i = 0; i < G::NA; ++i) {
    const int r = G::RPI * (G::NW * i + wave) + lane / NPC;
    const int lc = (lane % NPC) ^ (r % NPC);
    asrc[i] = A + (size_t)min(m0 + r, M - 1) * PARTS * (size_t)K + lc * 8;
  }
  unsigned char* const ring0 = ring;
  auto issue = [&](int it) {
    const int c = kc0 + min(it, nloc - 1);
    unsigned char* st = ring0 + (it % G::NS) * G::STAGE;
#pragma unroll
    for (int i = 0; i < G::NA; ++i)
      load_lds16(asrc[i] + (size_t)c * PARTS * BK, st + (G::NW * i + wave) * 1024);
#pragma unroll
    for (int i = 0; i < G::NWD; ++i)
      load_lds16_nt(wsrc[i] + (size_t)c * BK, st + G::ASTAGE + ((G::BN / G::NW) * wave + 8 * i) * 128);
  };

  f32x16_t acc[G::MBW][G::NBW];
#pragma unroll
  for (int mb = 0; mb < G::MBW; ++mb)
#pragma unroll
    for (int nb = 0; nb < G::NBW; ++nb) acc[mb][nb] = f32x16_t{};

  const uint32_t ring_addr = lds_addr_of(ring);
  struct Frags {
    u32x4_t a[G::MBW][PARTS];
    u32x4_t w[G::NBW];
  };
  // fragments of k-step j: k-group q of rows / columns c32 of each block
  auto read_frags = [&](uint32_t st, int j, Frags& f) {
    const int q = 4 * g + j;
#pragma unroll
    for (int mb = 0; mb < G::MBW; ++mb) {
      const int r = (wm * G::MBW + mb) * 32 + c32;
      const uint32_t rowa = st + (uint32_t)(r * G::RB);
#pragma unroll
      for (int part = 0; part < PARTS; ++part)
        f.a[mb][part] = lds_read16(rowa + (uint32_t)(((PARTS * q + part) ^ (r % NPC)) * 16));
    }
#pragma unroll
    for (int nb = 0; nb < G::NBW; ++nb) {
      const int t = (wn * G::NBW + nb) * 32 + c32;
      f.w[nb] = lds_read16(st + G::ASTAGE + (uint32_t)(t * 128 + ((q ^ ((t >> 1) & 7)) * 16)));
    }
  };
  auto fence = [&](Frags& f) {
#pragma unroll
    for (int mb = 0; mb < G::MBW; ++mb)
#pragma unroll
      for (int part = 0; part < PARTS; ++part) lds_fence_value(f.a[mb][part]);
#pragma unroll
    for (int nb = 0; nb < G::NBW; ++nb) lds_fence_value(f.w[nb]);
  };
  // split format: hi parts for every accumulator, then lo parts
  auto mfma_step = [&](const Frags& f) {
#pragma unroll
    for (int part = 0; part < PARTS; ++part)
#pragma unroll
      for (int mb = 0; mb < G::MBW; ++mb) {
#pragma unroll
        for (int nb = 0; nb < G::NBW; ++nb)
          acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, f.a[mb][part]),
                                                                __builtin_bit_cast(bf16x8_t, f.w[nb]), acc[mb][nb], 0, 0, 0);
      }
  };

#pragma unroll
  for (int s = 0; s < G::NS - 1; ++s) issue(s);
  for (int it = 0; it < nloc; ++it) {
    wait_vmcnt<G::WAIT>();          // this wave's loads of chunk it have landed
    lds_wait();                     // and its reads of chunk it - 1 are done
    __builtin_amdgcn_s_barrier();   // ... in every wave: chunk it is complete, stage it - 1 is free
    issue(it + G::NS - 1);
    const uint32_t st = ring_addr + (uint32_t)((it % G::NS) * G::STAGE);
    Frags f0, f1;
    read_frags(st, 0, f0);
    lds_wait();
    fence(f0);
    read_frags(st, 1, f1);          // next k-step in flight during this one
    mfma_step(f0);
    lds_wait();
    fence(f1);
    read_frags(st, 2, f0);
    mfma_step(f1);
    lds_wait();
    fence(f0);
    read_frags(st, 3, f1);
    mfma_step(f0);
    lds_wait();
    fence(f1);
    mfma_step(f1);
  }

  // epilogue: element i of lane l is row 8 (i / 4) + 4 g + i % 4, column c32
#pragma unroll
  for (int mb = 0; mb < G::MBW; ++mb) {
#pragma unroll
    for (int nb = 0; nb < G::NBW; ++nb) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int m = m0 + (wm * G::MBW + mb) * 32 + 8 * (i >> 2) + 4 * g + (i & 3);
        const float v = acc[mb][nb][i];
        if (EPI == EPI_SWIGLU) {
          // columns 0..15 of the block are gate values, 16..31 the matching up values
          const float up = __shfl_xor(v, 16, 64);
          const int j = blockIdx.x * G::OUT_COLS + 16 * (wn * G::NBW + nb) + (c32 & 15);
          if (m < M && c32 < 16 && j < N)
            split_store(reinterpret_cast<bf16_t*>(out) + (size_t)m * 2 * ldo, j, silu(v) * up);
        } else {
          const int n = blockIdx.x * G::BN + (wn * G::NBW + nb) * 32 + c32;
          if (m < M && n < N) out[blockIdx.z * split_stride + (size_t)m * ldo + n] = v;
        }
      }
    }
  }
}

// ------------------------------------------------------- packed, tiled
// C = A . W^T over the packed (MFMA-ordered) weights, more than 128 rows.
//
// One workgroup of 4 waves, one per SIMD, computes a BM x BN tile in chunks of
// 32 k-values (two MFMA k-steps).  What bounds it is the issue of a wave's own
// instructions: a vector-memory load takes 16 clocks of the compute unit's
// address path, so a wave that issues its whole chunk of loads at once stands
// still for 500 to 1000 clocks while the matrix cores idle.  Hence
//   * the loads of the chunk NS - 1 ahead go out one by one between the MFMAs;
//   * the fragments of the next k-step are read while the MFMAs of this one
//     run, across the chunk border too: the barrier for chunk c + 1 stands
//     before the last k-step of chunk c, whose MFMAs cover the first reads;
//   * a wave owns 128 x 128 results (fp16; 64 x 128 hi + lo), 0.5 KB of LDS
//     reads per MFMA, so that reads and DMA writes together take 3/4 of the
//     LDS cycles at the matrix cores' rate (a 64 x 128 fp16 wave tile, as
//     eight waves have it, takes all of them);
//   * results leave through LDS as whole 512-byte row pieces (64 separate
//     4-byte stores per block took as long as 130 MFMAs).
// Measured against the 8-wave kernel that issued its loads at the top of each
// 64-wide chunk (M = 8176, us): senior QKV 466 -> 381 (1.35 PFLOP/s of MFMA),
// O 333 -> 269, gate/up + SwiGLU 954 -> 721 (1.13 PFLOP/s), down 511 -> 423;
// 1024 rows of the small senior: gate/up 32 -> 25.5, down 23 -> 15.2.
// A 5-stage ring is no faster than 4 stages.  Rows past M lie outside the
// activations' descriptor by their per-lane offset and read as zeros; blocks past
// N repeat the last one.
template <int BM_, int BN_, int WM_, int NS_, bool A16> struct TileShape {
  static constexpr int NW = 4;                        // waves
  static constexpr int BM = BM_, BN = BN_;
  static constexpr int WM = WM_, WN = NW / WM;        // waves along M and N
  static constexpr int MBW = BM / 32 / WM;            // 32-row blocks per wave
  static constexpr int NBW = BN / 32 / WN;            // 32-column blocks per wave
  static constexpr int NS = NS_;                      // ring stages
  static constexpr int PARTS = A16 ? 1 : 2;           // MFMA operand parts per activation (fp16, or hi + lo)
  static constexpr int RB = 64 * PARTS;               // bytes of one activation row per chunk
  static constexpr int NPC = RB / 16;                 // 16-byte pieces per activation row
  static constexpr int RPI = 64 / NPC;                // activation rows per 1 KB DMA instruction
  static constexpr int ASTAGE = BM * RB, WSTAGE = BN * 64, STAGE = ASTAGE + WSTAGE;
  static constexpr int NA = ASTAGE / 1024 / NW;       // activation DMA instructions per wave per chunk
  static constexpr int NL = NA + WSTAGE / 1024 / NW;  // all DMA instructions per wave per chunk
  static constexpr int L1 = NL / 2, L0 = NL - L1;     // a chunk's loads go out in two k-steps
  static constexpr int NMF = MBW * NBW * PARTS;       // MFMAs per wave per k-step
  static constexpr int OST = NBW * 32 + 4;            // row stride (floats) of a wave's output block in LDS
  static constexpr int LDS = NS * STAGE > NW * 32 * OST * 4 ? NS * STAGE : NW * 32 * OST * 4;
  static_assert(LDS <= 160 * 1024, "LDS ring exceeds 160 KB");
  static_assert(NS >= 3 && NA >= 1 && NL > NA && (NS - 2) * NL < 64, "ring depth and wait counts");
};

// SWZ: tiles are dealt so that each XCD (workgroup id mod 8) takes one
// contiguous run of an order that walks groups of four tile rows column by
// column, which keeps a run's activation rows and weight columns in that XCD's
// L2; without it tiles go row by row.
template <int BM, int BN, int WM, int NS, int EPI, bool A16, int OCC, bool SWZ>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(OCC))) void gemm_tile_kernel(
    const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, int M, int N, int K, int cps,
    float* __restrict__ out, int ldo, long split_stride, int ntx, int nty) {
  using G = TileShape<BM, BN, WM, NS, A16>;
  constexpr int PARTS = G::PARTS, NPC = G::NPC, MBW = G::MBW, NBW = G::NBW, NL = G::NL, NW = G::NW;
  __shared__ __attribute__((aligned(1024))) unsigned char ring[G::LDS];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 5, c32 = lane & 31, wm = wave / G::WN, wn = wave % G::WN;
  const int tot = ntx * nty, bz = blockIdx.x / tot;
  int bx, by;
  {
    const int id = blockIdx.x % tot;
    if (SWZ) {
      const int q = tot / 8, r = tot % 8, x = id % 8;
      const int t = x * q + min(x, r) + id / 8;         // XCD x takes q + (x < r) tiles
      const int gi = t / (4 * ntx), gr = min(4, nty - 4 * gi), u = t - gi * 4 * ntx;
      by = 4 * gi + u % gr;
      bx = u / gr;
    } else {
      bx = id % ntx;
      by = id / ntx;
    }
  }
  const int m0 = by * BM, nch = K / 32, kc0 = bz * cps, nloc = min(cps, nch - kc0);
  if (nloc <= 0) return;
  const int lda = K * PARTS * 2, kfr = K / 16;            // bytes of an activation row, fragments of a weight block
  const int nblk = ((EPI == EPI_SWIGLU ? 2 * N : N) + 31) / 32, b0 = bx * (BN / 32);
  const __amdgpu_buffer_rsrc_t ar =
      buf_rsrc((const char*)A + (size_t)m0 * lda, (uint32_t)min(BM, M - m0) * (uint32_t)lda);
  const __amdgpu_buffer_rsrc_t wr =
      buf_rsrc((const char*)W + (size_t)b0 * kfr * 1024, (uint32_t)min(BN / 32, nblk - b0) * (uint32_t)kfr * 1024u);
  // XOR of an activation row's piece index: two rows (128-byte rows) or four
  // (64-byte rows) share the 256 bytes that all banks cover
  auto swz = [](int r) { return A16 ? (r >> 2) & 3 : r & 7; };
  int avoff[G::NA];
#pragma unroll
  for (int i = 0; i < G::NA; ++i) {
    const int r = G::RPI * (NW * i + wave) + lane / NPC;
    avoff[i] = r * lda + (((lane % NPC) ^ swz(r)) * 16);
  }
  // DMA instruction i of this wave for chunk c (clamped to the last one)
  auto load = [&](int c, int stage, int i) {
    unsigned char* st = ring + stage * G::STAGE;
    const int kc = kc0 + min(c, nloc - 1);
    if (i < G::NA) {
      buf_load_lds16(ar, st + (NW * i + wave) * 1024, avoff[i], kc * G::RB);
    } else {
      const int f = NW * (i - G::NA) + wave;
      buf_load_lds16(wr, st + G::ASTAGE + f * 1024, lane * 16, tile_weight_offset(f, kc, kfr, nblk - b0));
    }
  };
  f32x16_t acc[MBW][NBW];
#pragma unroll
  for (int a = 0; a < MBW; ++a)
#pragma unroll
    for (int b = 0; b < NBW; ++b) acc[a][b] = f32x16_t{};
  struct Frags {
    u32x4_t a[MBW][PARTS];
    u32x4_t w[NBW];
  };
  const uint32_t ring_addr = lds_addr_of(ring);
  uint32_t aaddr[2][PARTS];                               // of the wave's first row block, by k-step and part
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int p = 0; p < PARTS; ++p) {
      const int r = wm * MBW * 32 + c32;
      aaddr[j][p] = ring_addr + (uint32_t)(r * G::RB + (((PARTS * (2 * j + g) + p) ^ swz(r)) * 16));
    }
  const uint32_t waddr = ring_addr + G::ASTAGE + (uint32_t)(wn * NBW * 2048 + lane * 16);
  auto read = [&](int stage, int j, Frags& f) {
    const uint32_t so = stage * G::STAGE;
#pragma unroll
    for (int b = 0; b < NBW; ++b) f.w[b] = lds_read16(waddr + so + (uint32_t)(b * 2048 + j * 1024));
#pragma unroll
    for (int a = 0; a < MBW; ++a)
#pragma unroll
      for (int p = 0; p < PARTS; ++p) f.a[a][p] = lds_read16(aaddr[j][p] + so + (uint32_t)(a * 32 * G::RB));
  };
  // the fragments just read are complete
  auto landed = [&](Frags& f) {
    lds_wait();
#pragma unroll
    for (int a = 0; a < MBW; ++a)
#pragma unroll
      for (int p = 0; p < PARTS; ++p) lds_fence_value(f.a[a][p]);
#pragma unroll
    for (int b = 0; b < NBW; ++b) lds_fence_value(f.w[b]);
  };
  // the MFMAs of one k-step (weights first: the result is transposed, a lane
  // holds four consecutive columns of one row), with n loads of chunk c from
  // li0 on spread between them
  auto mfma_step = [&](Frags& f, int c, int stage, int li0, int n) {
    int mi = 0, li = 0;
#pragma unroll
    for (int p = 0; p < PARTS; ++p)
#pragma unroll
      for (int a = 0; a < MBW; ++a)
#pragma unroll
        for (int b = 0; b < NBW; ++b) {
          if (A16)
            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, f.w[b]),
                                                               __builtin_bit_cast(f16x8_t, f.a[a][p]), acc[a][b], 0, 0, 0);
          else
            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, f.w[b]),
                                                                __builtin_bit_cast(bf16x8_t, f.a[a][p]), acc[a][b], 0, 0, 0);
          ++mi;
#pragma unroll
          for (int rep = 0; rep < NL; ++rep)
            if (li < n && li * G::NMF < mi * n) {
              __builtin_amdgcn_sched_barrier(0);
              load(c, stage, li0 + li);
              ++li;
              __builtin_amdgcn_sched_barrier(0);
            }
        }
  };

#pragma unroll
  for (int d = 0; d < NS - 1; ++d)
#pragma unroll
    for (int i = 0; i < NL; ++i) load(d, d, i);
  Frags f0, f1;
  wait_vmcnt<(NS - 2) * NL>();
  __builtin_amdgcn_s_barrier();
  read(0, 0, f0);
  landed(f0);
  // Chunk c, stage u: k-step 0 carries the second half of the loads of chunk
  // c + NS - 2 (for c = 0 a repetition: the prologue issued them), then chunk
  // c + 1 has landed in every wave and stage c - 1 is free, and k-step 1
  // carries the first half of the loads of chunk c + NS - 1.
  for (int c0 = 0; c0 < nloc; c0 += NS) {
#pragma unroll
    for (int u = 0; u < NS; ++u) {
      if (u > 0 && c0 + u >= nloc) break;
      const int c = c0 + u;
      read(u, 1, f1);
      mfma_step(f0, c + NS - 2, (u + NS - 2) % NS, G::L0, G::L1);
      landed(f1);
      wait_vmcnt<(NS - 3) * NL>();
      __builtin_amdgcn_s_barrier();
      read((u + 1) % NS, 0, f0);
      mfma_step(f1, c + NS - 1, (u + NS - 1) % NS, 0, G::L0);
      landed(f0);
    }
  }
  wait_vmcnt<0>();
  __builtin_amdgcn_s_barrier();        // the ring is idle in every wave: its LDS takes the results

  // element 4 i + e of lane (g, c32) is row c32, column 8 i + 4 g + e of its block
  if (EPI == EPI_SWIGLU) {
    // columns 0 .. 15 of a block are gate values, 16 .. 31 the matching up
    // values (pair-interleaved packing): both in one lane
    constexpr int COLS = NBW * 16, ST = COLS + 8;
    static_assert(NW * 32 * ST * 2 <= G::LDS, "SwiGLU rows in LDS");
    uint16_t* sm = reinterpret_cast<uint16_t*>(ring) + wave * 32 * ST;
#pragma unroll
    for (int a = 0; a < MBW; ++a) {
      const int mrow = m0 + (wm * MBW + a) * 32;
#pragma unroll
      for (int b = 0; b < NBW; ++b)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          float y[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) y[e] = silu(acc[a][b][4 * i + e]) * acc[a][b][8 + 4 * i + e];
          if (A16) {
            *reinterpret_cast<uint2*>(sm + c32 * ST + b * 16 + 8 * i + 4 * g) =
                make_uint2((uint32_t)f2h(y[0]) | ((uint32_t)f2h(y[1]) << 16),
                           (uint32_t)f2h(y[2]) | ((uint32_t)f2h(y[3]) << 16));
          } else {
            const int m = mrow + c32, j = bx * (BN / 2) + wn * COLS + b * 16 + 8 * i + 4 * g;
            if (m < M && j < N) {
#pragma unroll
              for (int e = 0; e < 4; ++e) split_store(reinterpret_cast<bf16_t*>(out) + (size_t)m * 2 * ldo, j + e, y[e]);
            }
          }
        }
      if (!A16) continue;
      __builtin_amdgcn_wave_barrier();
      constexpr int LPR = COLS / 8;                       // lanes per row
#pragma unroll
      for (int r0 = 0; r0 < 32; r0 += 64 / LPR) {
        const int r = r0 + lane / LPR, cc = (lane % LPR) * 8;
        const uint4 v = *reinterpret_cast<const uint4*>(sm + r * ST + cc);
        const int m = mrow + r, j = bx * (BN / 2) + wn * COLS + cc;
        if (m < M && j < N) *reinterpret_cast<uint4*>(reinterpret_cast<uint16_t*>(out) + (size_t)m * ldo + j) = v;
      }
      __builtin_amdgcn_wave_barrier();
    }
  } else {
    constexpr int COLS = NBW * 32, ST = G::OST;
    float* sm = reinterpret_cast<float*>(ring) + wave * 32 * ST;
    const bool quads = N % 4 == 0 && ldo % 4 == 0;        // rows of whole, aligned float4
    float* o = out + (size_t)bz * split_stride;
#pragma unroll
    for (int a = 0; a < MBW; ++a) {
#pragma unroll
      for (int b = 0; b < NBW; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          *reinterpret_cast<float4*>(sm + c32 * ST + b * 32 + 8 * i + 4 * g) =
              make_float4(acc[a][b][4 * i], acc[a][b][4 * i + 1], acc[a][b][4 * i + 2], acc[a][b][4 * i + 3]);
      __builtin_amdgcn_wave_barrier();
      constexpr int LPR = COLS / 4;                       // lanes per row
#pragma unroll
      for (int r0 = 0; r0 < 32; r0 += 64 / LPR) {
        const int r = r0 + lane / LPR, cc = (lane % LPR) * 4;
        const float4 v = *reinterpret_cast<const float4*>(sm + r * ST + cc);
        const int m = m0 + (wm * MBW + a) * 32 + r, n = bx * BN + wn * COLS + cc;
        if (m >= M) continue;
        float* p = o + (size_t)m * ldo + n;
        if (quads) {
          if (n < N) *reinterpret_cast<float4*>(p) = v;
        } else {
          if (n < N) p[0] = v.x;
          if (n + 1 < N) p[1] = v.y;
          if (n + 2 < N) p[2] = v.z;
          if (n + 3 < N) p[3] = v.w;
        }
      }
      __builtin_amdgcn_wave_barrier();
    }
  }
}

// ---------------------------------------------------------------- VALU path
constexpr int kRowsMax = 32, kRowsMaxK = 1024;   // rows and K that gemm_rows_kernel takes

template <typename WT, bool SPLIT, int EPI>
__global__ __launch_bounds__(256) void gemm_valu_kernel(
    const void* __restrict__ Av, const WT* __restrict__ W, int M, int N, int K, int kper,
    float* __restrict__ out, int ldo, long split_stride) {
  // 32 x 32 output tile, 16 x 16 threads with 2 x 2 outputs each
  constexpr int T = 32;
  constexpr int NW = (EPI == EPI_SWIGLU) ? 2 : 1;
  __shared__ float As[T][T + 1];
  __shared__ float Ws[NW][T][T + 1];
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  const int m0 = blockIdx.y * T, n0 = blockIdx.x * T;
  const int kb = blockIdx.z * kper, ke = min(K, kb + kper);
  float acc[NW][2][2] = {};
  for (int k0 = kb; k0 < ke; k0 += T) {
    for (int e = threadIdx.x; e < T * T; e += 256) {
      const int r = e / T, c = e % T;
      const int m = m0 + r, k = k0 + c;
      float a = 0.f;
      if (m < M && k < ke) {
        if (SPLIT) a = split_load(reinterpret_cast<const bf16_t*>(Av) + (size_t)m * 2 * K, k);
        else a = reinterpret_cast<const float*>(Av)[(size_t)m * K + k];
      }
      As[r][c] = a;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const int n = n0 + r;
        const int row = n + w * N;
        Ws[w][r][c] = (n < N && k < ke) ? ld(W + (size_t)row * K + k) : 0.f;
      }
    }
    __syncthreads();
    for (int kk = 0; kk < T; ++kk) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const float a = As[ty * 2 + i][kk];
#pragma unroll
        for (int w = 0; w < NW; ++w)
#pragma unroll
          for (int jj = 0; jj < 2; ++jj) acc[w][i][jj] += a * Ws[w][tx * 2 + jj][kk];
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int jj = 0; jj < 2; ++jj) {
      const int m = m0 + ty * 2 + i, n = n0 + tx * 2 + jj;
      if (m >= M || n >= N) continue;
      if (EPI == EPI_SWIGLU)
        act_store<SPLIT>(out, m, ldo, n, silu(acc[0][i][jj]) * acc[NW - 1][i][jj]);
      else
        out[blockIdx.z * split_stride + (size_t)m * ldo + n] = acc[0][i][jj];
    }
}

// The same products of a float32 model for a few rows.  Every operand is on chip
// and a 32 x 32 tile spends its time on the round trips of its K loop and on rows
// that are not there, so the latency of one chain bounds it: here 32 lanes take
// two weight rows (SwiGLU: a gate row and its up row) and MR activation rows along
// K, 16 bytes per lane and load, all loads of 128 k-values in flight together, and
// add up over the lanes at the end.  No K slices: one partial for the consumer.
// Four rows of the 128-wide float32 pair: gate/up 10.5 -> 2.9 us, the other
// projections 5.3 -> 3.8; its rollout of 32 tokens 4.72 -> 4.51 ms.
template <int MR, int EPI>
__global__ __launch_bounds__(256) void gemm_rows_kernel(const float* __restrict__ A, const float* __restrict__ W,
                                                        int M, int N, int K, float* __restrict__ out, int ldo) {
  const int l = threadIdx.x & 31, pair = blockIdx.x * 8 + (threadIdx.x >> 5);
  const int m0 = blockIdx.y * MR;
  const int n_pairs = EPI == EPI_SWIGLU ? N : (N + 1) / 2;
  // a pair past the end repeats the last one (all lanes take part in the sums)
  const int pp = min(pair, n_pairs - 1);
  const int n0 = EPI == EPI_SWIGLU ? pp : 2 * pp;
  const int n1 = EPI == EPI_SWIGLU ? pp + N : min(2 * pp + 1, N - 1);
  const float* w0 = W + (size_t)n0 * K;
  const float* w1 = W + (size_t)n1 * K;
  const float* ar[MR];
#pragma unroll
  for (int m = 0; m < MR; ++m) ar[m] = A + (size_t)min(m0 + m, M - 1) * K;
  float acc0[MR] = {}, acc1[MR] = {};
#pragma unroll 2
  for (int k = 4 * l; k < K; k += 128) {
    const float4 x0 = *reinterpret_cast<const float4*>(w0 + k), x1 = *reinterpret_cast<const float4*>(w1 + k);
#pragma unroll
    for (int m = 0; m < MR; ++m) {
      const float4 y = *reinterpret_cast<const float4*>(ar[m] + k);
      acc0[m] += (y.x * x0.x + y.y * x0.y) + (y.z * x0.z + y.w * x0.w);
      acc1[m] += (y.x * x1.x + y.y * x1.y) + (y.z * x1.z + y.w * x1.w);
    }
  }
  // the sums over the 32 lanes: each exchange halves the rows a lane holds, so
  // at the end lane l has row l / (32 / MR) (the other exchanges add only)
  int have = MR;
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) {
    const bool hi = (l & o) != 0;
    if (have > 1) {
      have /= 2;
#pragma unroll
      for (int m = 0; m < MR / 2; ++m) {
        if (m >= have) break;
        const float s0 = hi ? acc0[m] : acc0[m + have], s1 = hi ? acc1[m] : acc1[m + have];
        acc0[m] = (hi ? acc0[m + have] : acc0[m]) + __shfl_xor(s0, o, 64);
        acc1[m] = (hi ? acc1[m + have] : acc1[m]) + __shfl_xor(s1, o, 64);
      }
    } else {
      acc0[0] += __shfl_xor(acc0[0], o, 64);
      acc1[0] += __shfl_xor(acc1[0], o, 64);
    }
  }
  const int m = m0 + l / (32 / MR);
  if (l % (32 / MR) != 0 || m >= M || pair >= n_pairs) return;
  if (EPI == EPI_SWIGLU) {
    out[(size_t)m * ldo + pair] = silu(acc0[0]) * acc1[0];
  } else {
    float* p = out + (size_t)m * ldo + 2 * pair;
    p[0] = acc0[0];
    if (2 * pair + 1 < N) p[1] = acc1[0];
  }
}

template <int BMT, int NST, int EPI>
hipError_t run_mfma(const GemmArgs& a, int S, int cps, hipStream_t st) {
  constexpr int NW = (BMT >= 128) ? 8 : 4;    // 128-row tiles: two waves per SIMD
  using G = GemmShape<BMT, NST, NW>;
  const int cols = (EPI == EPI_SWIGLU) ? G::OUT_COLS : G::BN;
  dim3 grid((a.N + cols - 1) / cols, (a.M + BMT - 1) / BMT, S);
  hipLaunchKernelGGL((gemm_mfma_kernel<BMT, NST, EPI, NW>), grid, dim3(64 * NW), 0, st, (const bf16_t*)a.A,
                     (const bf16_t*)a.W, a.M, a.N, a.K, cps, a.out, a.ldo, a.split_stride);
  return hipGetLastError();
}

template <int BM, int BN, int WM, int NS, int EPI, bool A16, int OCC, bool SWZ>
hipError_t run_tile(const GemmArgs& a, int S, int cps, hipStream_t st) {
  const int rows = EPI == EPI_SWIGLU ? 2 * a.N : a.N;
  const int ntx = (rows + BN - 1) / BN, nty = (a.M + BM - 1) / BM;
  hipLaunchKernelGGL((gemm_tile_kernel<BM, BN, WM, NS, EPI, A16, OCC, SWZ>), dim3((unsigned)ntx * nty * S), dim3(256), 0,
                     st, (const bf16_t*)a.A, (const bf16_t*)a.Wp, a.M, a.N, a.K, 2 * cps, a.out, a.ldo,
                     a.split_stride, ntx, nty);
  return hipGetLastError();
}

// Packed weights take the tile with the least estimated time: rounds of
// workgroups over the compute units times the time of a round, in units of
// 128 x 128 results per compute unit at the largest tile's rate.  A round of
// 128 x 256 fp16 tiles takes 2.2, one of 128 x 128 tiles (two workgroups per
// unit) 2.45, a half-filled one 1.67 (us for 256 x 256, 128 x 256 and
// 128 x 128, each launch on weights and activations that are in no cache:
// gate/up of 1024 small rows 29.2, 24.1, 28.8; down of 4056 small rows 91, 68,
// 47.5; LM head of 256 rows 32.4, 26.9, 34; in cache: down of 8176 rows 435,
// 423, 467).  The split format has half the columns per unit of work: QKV of
// 4056 small rows 29.1 in 128 x 256 tiles, 32.7 in 128 x 128.
template <int EPI>
hipError_t dispatch_tile(const GemmArgs& a, int S, int cps, hipStream_t st) {
  const int rows = EPI == EPI_SWIGLU ? 2 * a.N : a.N;
  auto tiles = [&](int bm, int bn) { return (long)((a.M + bm - 1) / bm) * ((rows + bn - 1) / bn) * S; };
  auto rounds = [](long t, long per) { return (double)((t + per - 1) / per); };
  const long t128 = tiles(128, 128), cu = a.n_cu;
  if (a.a16) {
    const double c128 = t128 <= cu ? 1.67 : 2.45 * rounds(t128, 2 * cu);
    const double cw = 2.2 * rounds(tiles(128, 256), cu), c256 = 4.0 * rounds(tiles(256, 256), cu);
    if (c256 <= cw && c256 <= c128) {
      // the XCD order pays where a tile reads much more than it writes (gate/up
      // of 8176 rows, K = 2560: 743 -> 721 us) or few tile rows share the
      // weights (LM head of 1024 rows: 85 -> 77); K = 1024 over many rows is
      // bound by its output, which leaves in order without it (75 against 79.5)
      if (a.K >= 2048 || a.M <= 1024) return run_tile<256, 256, 2, 4, EPI, true, 1, true>(a, S, cps, st);
      return run_tile<256, 256, 2, 4, EPI, true, 1, false>(a, S, cps, st);
    }
    if (cw < c128) return run_tile<128, 256, 1, 4, EPI, true, 1, true>(a, S, cps, st);
    return run_tile<128, 128, 2, 5, EPI, true, 2, true>(a, S, cps, st);
  }
  const double c128 = t128 <= cu ? 0.9 : 1.13 * rounds(t128, 2 * cu);
  if (rounds(tiles(128, 256), cu) < c128) return run_tile<128, 256, 2, 4, EPI, false, 1, true>(a, S, cps, st);
  // at most one 128 x 128 tile per compute unit: a deep ring where the K slice
  // has the chunks for it (QKV of 1024 small rows, 16 chunks: 13.7 -> 11.5 us;
  // O of 4056 rows, 32 chunks: 30.3 -> 24.2; O of 1024 rows, 8 chunks: 10.6, 12.4)
  if (t128 <= cu && 2 * cps >= 16) return run_tile<128, 128, 2, 6, EPI, false, 1, true>(a, S, cps, st);
  return run_tile<128, 128, 2, 3, EPI, false, 2, true>(a, S, cps, st);
}

template <int EPI>
hipError_t dispatch_mfma(const GemmArgs& a, int S, int cps, hipStream_t st) {
  // the tile kernel addresses a tile's activation rows with 32-bit offsets
  // (longer rows read the row-major weights; fp16 rows never are that long:
  // their gate/up matrix of 2 K rows has a packed copy, below 2^31 bytes)
  const bool tile = a.Wp && a.M > 64 && (size_t)256 * a.K * (a.a16 ? 2 : 4) < ((size_t)1 << 31);
  if (tile) return dispatch_tile<EPI>(a, S, cps, st);
  if (a.a16) return hipErrorInvalidValue;
  if (a.M <= 32) return run_mfma<32, 4, EPI>(a, S, cps, st);
  if (a.M <= 64) return run_mfma<64, 4, EPI>(a, S, cps, st);
  return run_mfma<128, 3, EPI>(a, S, cps, st);
}

template <typename WT, bool SPLIT>
hipError_t run_valu(const GemmArgs& a, int S, int kper, hipStream_t st) {
  dim3 grid((a.N + 31) / 32, (a.M + 31) / 32, S);
  if (a.epi == EPI_SWIGLU)
    hipLaunchKernelGGL((gemm_valu_kernel<WT, SPLIT, EPI_SWIGLU>), grid, dim3(256), 0, st, a.A,
                       (const WT*)a.W, a.M, a.N, a.K, kper, a.out, a.ldo, a.split_stride);
  else
    hipLaunchKernelGGL((gemm_valu_kernel<WT, SPLIT, EPI_PARTIAL>), grid, dim3(256), 0, st, a.A,
                       (const WT*)a.W, a.M, a.N, a.K, kper, a.out, a.ldo, a.split_stride);
  return hipGetLastError();
}

template <int MR>
hipError_t run_rows(const GemmArgs& a, hipStream_t st) {
  const int pairs = a.epi == EPI_SWIGLU ? a.N : (a.N + 1) / 2;
  const dim3 grid((pairs + 7) / 8, (a.M + MR - 1) / MR);
  if (a.epi == EPI_SWIGLU)
    hipLaunchKernelGGL((gemm_rows_kernel<MR, EPI_SWIGLU>), grid, dim3(256), 0, st, (const float*)a.A,
                       (const float*)a.W, a.M, a.N, a.K, a.out, a.ldo);
  else
    hipLaunchKernelGGL((gemm_rows_kernel<MR, EPI_PARTIAL>), grid, dim3(256), 0, st, (const float*)a.A,
                       (const float*)a.W, a.M, a.N, a.K, a.out, a.ldo);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm(const GemmArgs& a, int* splits_used, hipStream_t st) {
  if (a.M <= 0 || a.N <= 0) {
    if (splits_used) *splits_used = 0;
    return hipSuccess;
  }
  int S = a.epi == EPI_PARTIAL ? (a.splits < 1 ? 1 : a.splits) : 1;
  const bool mfma = (a.dt == DT_BF16) && (a.K % BK == 0);
  // packed weights take 128-row tiles (M > 64); fp16 activations need them
  if ((a.a16 && (!a.Wp || a.M <= 64)) || (a.Wp && (!mfma || (a.epi == EPI_SWIGLU && a.N % 16))))
    return hipErrorInvalidValue;
  if (mfma) {
    const int nch = a.K / BK;
    if (S > nch) S = nch;
    const int cps = (nch + S - 1) / S;
    S = (nch + cps - 1) / cps;
    if (splits_used) *splits_used = S;
    switch (a.epi) {
      case EPI_PARTIAL: return dispatch_mfma<EPI_PARTIAL>(a, S, cps, st);
      case EPI_STORE: return dispatch_mfma<EPI_STORE>(a, S, cps, st);
      default: return dispatch_mfma<EPI_SWIGLU>(a, S, cps, st);
    }
  }
  // A few rows of a float32 model whose rows of K are not long.  Steps of two layers
  // of d_model = ffn_dim = 1024 and a vocabulary of 32000 (d_model 512), us, tiles /
  // these rows: 1 row 394 / 149 (247 / 116), 4 rows 402 / 170 (252 / 135), 8 rows 408 /
  // 245 (257 / 183), 16 rows 426 / 273 (269 / 201), 32 rows 469 / 331 (298 / 234).  The
  // weights are read once per 8 rows, so the gain shrinks with the rows; more rows and
  // longer K were not measured and stay with the tiles.  Rows start 16-byte aligned
  // where K % 4 == 0.
  if (a.dt != DT_BF16 && a.M <= kRowsMax && a.K % 4 == 0 && a.K <= kRowsMaxK &&
      (((uintptr_t)a.A | (uintptr_t)a.W) & 15u) == 0) {
    if (splits_used) *splits_used = 1;
    return a.M <= 4 ? run_rows<4>(a, st) : run_rows<8>(a, st);
  }
  const int nk = (a.K + 31) / 32;
  if (S > nk) S = nk;
  const int kper = ((nk + S - 1) / S) * 32;
  S = (a.K + kper - 1) / kper;
  if (splits_used) *splits_used = S;
  if (a.dt == DT_BF16) return run_valu<bf16_t, true>(a, S, kper, st);
  return run_valu<float, false>(a, S, kper, st);
}

}  // namespace tandem
