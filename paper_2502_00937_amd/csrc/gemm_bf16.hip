// bf16 MFMA matrix product  C[M, N] = A[M, K] . W[N, K]^T  with fused epilogues.
//
// Both operands are K-contiguous, so a lane's 8 consecutive k values are one 16-byte
// load and map directly onto the v_mfma_f32_32x32x16_bf16 operand registers.
//
// Two kernels share the fragment layout and the epilogues; both move their operands global -> LDS
// directly (global_load_lds_dwordx4) and are described where they are defined:
// * gemm_bf16_pipe_kernel (most products, and the last rows of the other one's): one tile of 64 to 256 rows by 64 or
//   128 columns per workgroup, a ring of two to five 64-wide k-stages;
// * gemm_bf16_dma_kernel (products of many whole rounds of tiles): persistent, 256 x 256 tiles, eight waves of 128 x 64.
// Which of them, and which tile, a product takes is decided by the time that each is expected to need (launch_gemm_bf16).
// * LDS tiles are [row][64 bf16] with the 16-byte chunks XOR-swizzled by (row >> 1) & 7:
//   LDS serves a 16-byte-per-lane read 16 lanes at a time over 64 banks, and this
//   swizzle makes any 16 consecutive rows of one logical chunk hit 16 distinct bank groups.
// * The product is formed transposed (W fragment as the MFMA row operand), so a lane ends
//   up with four consecutive output columns of one token row per register quad.  The
//   epilogue adds bias, applies GELU / residual, converts, stages the 32 x TN block of a
//   wave through LDS and writes rows back with 16 bytes per lane.
// * Workgroup ids are dealt round-robin to the 8 XCDs; each XCD walks its own tiles in blocks
//   so the tiles in flight on one XCD share A and W slices in that XCD's L2.
#include <algorithm>
#include <type_traits>

#include "common.h"

namespace vitenc {

namespace {

constexpr int BK = 64;  // bf16 elements per k-step = 128 bytes = 8 chunks of 16 bytes
constexpr int GROUP_M = 4;  // row blocks that gemm_bf16_pipe_kernel walks together

// Epilogue of one wave.  acc[i][j] is a transposed 32x32 block: the lane holds token row
// row0 + 32i + (lane & 31); register 4jj + e holds output column ncol0 + 32j + 8jj + 4(lane >> 5) + e.
// prefetch() asks ahead of the k-loop for what finish() will need: the bias and, if AHEAD, the residual rows.  Loaded pass by
// pass behind the k-loop, each behind the store of the pass before it, the residual rows of a launch of one round were
// a chain of four to sixteen memory latencies: a launch of K = 64 took 3.5, 5.0 and 7.2 us on tiles of 64 x 64, 128 x 128 and
// 256 x 128, and takes 3.2, 4.5 and 6.3.  Where two workgroups share a unit the other one covers that, and the registers
// would cost a workgroup its place: there (AHEAD = false) a 32-row block's rows are asked for together in finish().
// finish() needs free LDS (all waves past their last tile read), in which each wave stages its own rows.
// Rows and columns past the matrix are read at a valid address and never stored.
template <int EPI, int FM, int FN, bool AHEAD>
struct WaveEpilogue {
  static constexpr bool RESID = EPI == EPI_BIAS_RESIDUAL;
  static constexpr int TN = FN * 32;
  static constexpr int LPR = TN / (RESID ? 4 : 8), RPI = 64 / LPR, PASSES = 32 / RPI;  // lanes per staged row (16 bytes each), rows per pass
  static constexpr int STAGE_ROW = TN * (RESID ? 4 : 2) + 16;                           // bytes per staged row (padded)
  f32x4 bias[RESID ? 1 : FN][RESID ? 1 : 4];
  f32x4 x[RESID && AHEAD ? FM : 1][RESID ? PASSES : 1];

  __device__ __forceinline__ void load_rows(const GemmArgs& a, int i, int row0, int col, int lane) {
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      const int row = min(row0 + i * 32 + p * RPI + lane / LPR, a.M - 1);
      x[AHEAD ? i : 0][p] = *(const f32x4*)(a.resid + (size_t)row * a.ldo + col);
    }
  }

  __device__ __forceinline__ void prefetch(const GemmArgs& a, int row0, int ncol0, int lane) {
    if constexpr (RESID) {
      const int col = min(ncol0 + lane % LPR * 4, a.N - 4);
      bias[0][0] = *(const f32x4*)(a.bias + col);
      if constexpr (AHEAD)
#pragma unroll
        for (int i = 0; i < FM; ++i) load_rows(a, i, row0, col, lane);
    } else {
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) bias[j][jj] = *(const f32x4*)(a.bias + ncol0 + j * 32 + jj * 8 + (lane >> 5) * 4);
    }
  }

  __device__ __forceinline__ void finish(const GemmArgs& a, f32x16 (&acc)[FM][FN], unsigned char* smem, int row0, int ncol0,
                                         int wave, int lane) {
    const int lrow = lane & 31, lk = lane >> 5;
    unsigned char* st = smem + wave * 32 * STAGE_ROW;
    if constexpr (EPI == EPI_PATCH) {
      // rows are (tile, patch); the residual stream row is tile*T + cls + patch and the position row is added
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        const int row = row0 + i * 32 + lrow;
        if (row >= a.M) continue;
        const int tile = row / a.patches, tok = a.cls + (row - tile * a.patches);
        float* xr = a.resid + ((size_t)tile * a.tokens + tok) * a.ldo;
        const float* pr = a.pos + (size_t)tok * a.ldo;
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
          for (int jj = 0; jj < 4; ++jj) {
            const int col = ncol0 + j * 32 + jj * 8 + lk * 4;
            if (col < a.N) {
              const f32x4 p = *(const f32x4*)(pr + col);
              f32x4 v;
#pragma unroll
              for (int e = 0; e < 4; ++e) v[e] = acc[i][j][jj * 4 + e] + bias[j][jj][e] + p[e];
              *(f32x4*)(xr + col) = v;
            }
          }
      }
    } else if constexpr (RESID) {
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        if constexpr (!AHEAD) load_rows(a, i, row0, min(ncol0 + lane % LPR * 4, a.N - 4), lane);
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
          for (int jj = 0; jj < 4; ++jj)
            *(f32x4*)(st + lrow * STAGE_ROW + (j * 32 + jj * 8 + lk * 4) * 4) =
                f32x4{acc[i][j][jj * 4], acc[i][j][jj * 4 + 1], acc[i][j][jj * 4 + 2], acc[i][j][jj * 4 + 3]};
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
          const int sr = p * RPI + lane / LPR, sc = lane % LPR * 4;
          const int row = row0 + i * 32 + sr, col = ncol0 + sc;
          const f32x4 v = *(const f32x4*)(st + sr * STAGE_ROW + sc * 4);
          if (row < a.M && col < a.N) *(f32x4*)(a.resid + (size_t)row * a.ldo + col) = x[AHEAD ? i : 0][p] + (v + bias[0][0]);
        }
        __builtin_amdgcn_wave_barrier();
      }
    } else {  // EPI_BIAS, EPI_BIAS_HEADS, EPI_BIAS_GELU: bf16 output
      float cs[FN][4];  // scale of each accumulator quad: the query columns' (see GemmArgs::q_cols), 1/2 ahead of GELU; the bias is scaled with it
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          cs[j][jj] = EPI == EPI_BIAS_GELU ? 0.5f : ncol0 + j * 32 + jj * 8 + lk * 4 < a.q_cols ? a.q_scale : 1.0f;
          bias[j][jj] *= cs[j][jj];
        }
      // EPI_BIAS_HEADS: heads of 64 or 128 columns stored one after the other, so the wave's TN columns lie inside
      // one head: a row stride and the offset of column ncol0, both wave-uniform
      const int hm_blk = EPI == EPI_BIAS_HEADS ? ncol0 / a.hm_dh : 0;
      const int rs = EPI == EPI_BIAS_HEADS ? a.hm_dh : a.ldo;
      const size_t col0_off =
          EPI == EPI_BIAS_HEADS ? (size_t)hm_blk * a.hm_rows * a.hm_dh + (ncol0 - hm_blk * a.hm_dh) : (size_t)ncol0;
#pragma unroll
      for (int i = 0; i < FM; ++i) {
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
          for (int jj = 0; jj < 4; ++jj) {
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              v[e] = fmaf(acc[i][j][jj * 4 + e], cs[j][jj], bias[j][jj][e]);
              if constexpr (EPI == EPI_BIAS_GELU) v[e] = gelu_fast_half(v[e]);
            }
            const u32x2 pk = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
            *(u32x2*)(st + lrow * STAGE_ROW + (j * 32 + jj * 8 + lk * 4) * 2) = pk;
          }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
          const int sr = p * RPI + lane / LPR, sc = lane % LPR * 8;
          const int row = row0 + i * 32 + sr, col = ncol0 + sc;
          const u32x4 v = *(const u32x4*)(st + sr * STAGE_ROW + sc * 2);
          if (row < a.M && col < a.N) *(u32x4*)((bf16_t*)a.out + (size_t)row * rs + col0_off + sc) = v;
        }
        __builtin_amdgcn_wave_barrier();
      }
    }
  }
};

// ---------------------------------------------------------------------------------------------
// Large-problem kernel: persistent, 256 x 256 tile, eight waves (two per SIMD), 128 x 64 per wave.
//
// The memory system, not the matrix cores, sets the pace of this product on gfx950.  A compute
// unit's L1 is filled in whole 128-byte lines: a probe that reads L2-resident rows in 64-byte
// pieces gets 70 GB/s per unit, in 128-byte pieces 135 GB/s.  A 256 x 256 tile needs 32 KiB per
// 32 k-values, which at full MFMA rate is 60 GB/s: affordable only when every line is asked for
// once.  Hence 64-wide k-stages (one 128-byte line per row) and the biggest tile the accumulators
// allow.
//
// * One workgroup per compute unit walks a list of tiles.  Operand tiles go global -> LDS directly
//   (global_load_lds_dwordx4: each lane supplies its own global offset, the wave writes 1 KiB of
//   consecutive LDS = 8 rows).  The stream of stages does not stop at tile boundaries, so the next
//   tile's first stages land while the current tile finishes and its epilogue runs; no launch gap, no
//   cold prologue per tile.
// * LDS is five units of 32 KiB: three stages of A, two of W.  A stage is multiplied in four 16-wide sub-steps, each
//   reading the next one's A fragments; the W fragments of all four are read in the first, so that W's unit is free
//   after a quarter of the stage (a barrier says so) and A's after three (the stage's sync, which also says that the next
//   stage has landed).  A unit's loads, two to a sub-step, thus have one and a half to two stages to land.  With two stages
//   of both operands, in which a load had half a stage, a wait on the slowest of them set the pace wherever the L2 missed:
//   51232 x 1280 x 5120 took 742 us and takes 668, 93312 x 4352 x 1152 917 and 878, 150020 x 1024 x 4096 1178 and 1115.
// * All of that only without branches: with run-time tests around the loads the same stages took 5 % longer than the two
//   of before, without them 2 to 10 % less (37 branches a stage).  Hence the STEADY form.
// * LDS rows are 128 bytes; the 16-byte chunk index is XORed with (row >> 1) & 7, which the lane
//   achieves by choosing which global chunk it loads, so any 16 consecutive rows of one logical
//   chunk fall on 16 distinct 16-byte bank groups of the 64 banks.
// * Tile order: the tile grid is cut into (8-row-block x 4-column-band) groups of 32 tiles, one per
//   compute unit of an XCD (a remainder of one or two tile columns is cut into 32 x 1 or 16 x 2
//   groups); consecutive groups along N go to consecutive XCDs, so the XCDs working at the same
//   time share A rows (first fetch fills the memory-side cache for the others) and the 32 units of
//   one XCD share both operands in its L2.
// * A wave's epilogue is staged (16 rows x 144 bytes) in the rows of A's dead unit that the wave itself refills next.
constexpr int D_BM = 256, D_BN = 256, D_BK = 64;
constexpr int D_ROW = D_BK * 2;                   // bytes per LDS row
constexpr int D_UNIT_BYTES = 256 * D_ROW;         // one operand's rows of a stage: 32 KiB
constexpr int D_LDS_BYTES = 5 * D_UNIT_BYTES;     // three units for A, two for W: all of the 160 KiB
constexpr int D_STAGING_ROW = 144;
static_assert(16 * D_STAGING_ROW <= 32 * D_ROW, "a wave stages its epilogue in the rows that it loads");
constexpr int D_GROUP_M = 8, D_GROUP_N = 4;

typedef const __attribute__((address_space(1))) void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

// Epilogue of one wave of the persistent kernel: same register layout as WaveEpilogue, but staged
// 16 rows at a time through the wave's private 16 x 144-byte LDS rows (`st`).
template <int EPI, bool STREAM_OUT, bool FULL>
__device__ __forceinline__ void wave_epilogue_p(const GemmArgs& a, f32x16 (&acc)[4][2], unsigned char* st, int row0,
                                                int ncol0, int lane) {
  constexpr int FM = 4, FN = 2;
  const int lrow = lane & 31, lk = lane >> 5;
  f32x4 bias[FN][4];  // per accumulator quad (the fp32 paths add their bias after the LDS round trip instead)
  if constexpr (EPI == EPI_BIAS || EPI == EPI_BIAS_GELU || EPI == EPI_BIAS_HEADS) {
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) bias[j][jj] = *(const f32x4*)(a.bias + ncol0 + j * 32 + jj * 8 + lk * 4);
  }

  if constexpr (EPI == EPI_PATCH) {
    // rows are (tile, patch); the residual stream row is tile * T + cls + patch, and that token's position row is
    // added.  Staged like the residual epilogue below (16 rows x 32 fp32 columns per piece, read back as 8 lanes
    // per row), so that the stream is written and the position table read in whole 128-byte row pieces; the row
    // mapping of a 32-row block is worked out once and serves both of its column blocks.
    const int sr0 = lane >> 3, sc = (lane & 7) * 4;
    f32x4 brow[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) brow[j] = *(const f32x4*)(a.bias + ncol0 + j * 32 + sc);
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      size_t dst_off[2][2], pos_off[2][2];  // [half][pass], in elements, of this lane's row
      bool ok[2][2];
#pragma unroll
      for (int half = 0; half < 2; ++half)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          const int row = row0 + i * 32 + half * 16 + p * 8 + sr0;
          ok[half][p] = FULL || row < a.M;
          const int rr = ok[half][p] ? row : 0;
          const int tile = rr / a.patches, tok = a.cls + (rr - tile * a.patches);
          dst_off[half][p] = ((size_t)tile * a.tokens + tok) * a.ldo;
          pos_off[half][p] = (size_t)tok * a.ldo;
        }
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const int col = ncol0 + j * 32 + sc;
        const bool col_ok = FULL || col < a.N;
        f32x4 posv[2][2];
#pragma unroll
        for (int half = 0; half < 2; ++half)
#pragma unroll
          for (int p = 0; p < 2; ++p)
            posv[half][p] = ok[half][p] && col_ok ? *(const f32x4*)(a.pos + pos_off[half][p] + col) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          if ((lrow >> 4) == half) {
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
              const f32x4 v = {acc[i][j][jj * 4], acc[i][j][jj * 4 + 1], acc[i][j][jj * 4 + 2], acc[i][j][jj * 4 + 3]};
              *(f32x4*)(st + (lrow & 15) * D_STAGING_ROW + (jj * 8 + lk * 4) * 4) = v;
            }
          }
          __builtin_amdgcn_wave_barrier();
#pragma unroll
          for (int p = 0; p < 2; ++p) {
            const f32x4 t = *(const f32x4*)(st + (p * 8 + sr0) * D_STAGING_ROW + sc * 4);
            if (ok[half][p] && col_ok) *(f32x4*)(a.resid + dst_off[half][p] + col) = posv[half][p] + (t + brow[j]);
          }
          __builtin_amdgcn_wave_barrier();
        }
      }
    }
  } else if constexpr (EPI == EPI_BIAS_RESIDUAL) {
    // Pieces of 16 rows x 32 fp32 columns (128 bytes + pad per staged row); a piece is read back
    // as 8 lanes per row, 8 rows per pass, and the bias is added there (one float4 per lane and column
    // block instead of one per accumulator quad).  The residual values of a 32 x 32 unit are loaded one
    // unit ahead; two, three and up to five units ahead (the registers of the next tile's first fragments
    // are free here, see the kernel) measured the same or slower: the epilogue is not bound by the latency
    // of these loads.  Addresses are a wave-uniform base (scalar arithmetic) plus a per-lane byte offset
    // that never changes; FULL tiles (all but the last row block and a ragged last column) carry no bounds
    // test.
    const int sr0 = lane >> 3, sc = (lane & 7) * 4;
    const uint32_t lane_off = (uint32_t)(sr0 * a.ldo + sc) * 4u;
    unsigned char* const tile_base = (unsigned char*)a.resid + ((size_t)row0 * a.ldo + ncol0) * 4;
    const int row_lim = a.M - row0 - sr0, col_lim = a.N - ncol0 - sc;  // valid: row offset < row_lim, col offset < col_lim
    auto x_ptr = [&](int i, int j, int half, int p) {
      return (float*)(tile_base + ((size_t)(i * 32 + half * 16 + p * 8) * a.ldo + j * 32) * 4 + lane_off);
    };
    auto x_ok = [&](int i, int j, int half, int p) {
      return FULL || (i * 32 + half * 16 + p * 8 < row_lim && j * 32 < col_lim);
    };
    f32x4 brow[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) brow[j] = *(const f32x4*)(a.bias + ncol0 + j * 32 + sc);
    f32x4 xin[2][2][2];  // [buffer][half][pass] of one unit
    auto load_unit = [&](int u, int buf) {  // unit u = i * FN + j
      const int i = u / FN, j = u % FN;
#pragma unroll
      for (int half = 0; half < 2; ++half)
#pragma unroll
        for (int p = 0; p < 2; ++p)
          xin[buf][half][p] = x_ok(i, j, half, p) ? *(const f32x4*)x_ptr(i, j, half, p) : f32x4{0.f, 0.f, 0.f, 0.f};
    };
    load_unit(0, 0);
#pragma unroll
    for (int u = 0; u < FM * FN; ++u) {
      const int i = u / FN, j = u % FN;
      if (u + 1 < FM * FN) load_unit(u + 1, (u + 1) & 1);
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        if ((lrow >> 4) == half) {
#pragma unroll
          for (int jj = 0; jj < 4; ++jj) {
            const f32x4 v = {acc[i][j][jj * 4], acc[i][j][jj * 4 + 1], acc[i][j][jj * 4 + 2], acc[i][j][jj * 4 + 3]};
            *(f32x4*)(st + (lrow & 15) * D_STAGING_ROW + (jj * 8 + lk * 4) * 4) = v;
          }
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          const f32x4 t = *(const f32x4*)(st + (p * 8 + sr0) * D_STAGING_ROW + sc * 4);
          if (x_ok(i, j, half, p)) *(f32x4*)x_ptr(i, j, half, p) = xin[u & 1][half][p] + (t + brow[j]);
        }
        __builtin_amdgcn_wave_barrier();
      }
    }
  } else {  // EPI_BIAS, EPI_BIAS_GELU: bf16 output, pieces of 16 rows x 64 columns (128 bytes + pad)
    // (storing the 8-byte register quads directly was measured slower than this LDS round trip)
    // Store addresses: wave-uniform base (scalar arithmetic) + a per-lane byte offset that never changes.
    float cs[FN][4];  // scale of each accumulator quad: the query columns' (see GemmArgs::q_cols), 1/2 ahead of GELU; the bias is scaled with it
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        cs[j][jj] = EPI == EPI_BIAS_GELU ? 0.5f : ncol0 + j * 32 + jj * 8 + lk * 4 < a.q_cols ? a.q_scale : 1.0f;
        bias[j][jj] *= cs[j][jj];
      }
    const int sc = (lane & 7) * 8;
    // EPI_BIAS_HEADS: heads of 64 or 128 columns stored one after the other, so the wave's 64 columns lie inside one
    // head: its rows are hm_dh elements apart and (row0, ncol0) sits at a wave-uniform address of its own
    const int rs = EPI == EPI_BIAS_HEADS ? a.hm_dh : a.ldo;
    const uint32_t lane_off = (uint32_t)((lane >> 3) * rs + sc) * 2u;
    const int hm_blk = EPI == EPI_BIAS_HEADS ? ncol0 / a.hm_dh : 0;
    unsigned char* const tile_base =
        (unsigned char*)a.out + (EPI == EPI_BIAS_HEADS ? ((size_t)hm_blk * a.hm_rows + row0) * a.hm_dh + (ncol0 - hm_blk * a.hm_dh)
                                                       : (size_t)row0 * a.ldo + ncol0) * 2;
    const int row_lim = a.M - row0 - (lane >> 3);
    const bool col_ok = ncol0 + sc < a.N;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      u32x2 pk[FN][4];  // all lanes convert once; the two half-wave passes below only move data
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            v[e] = fmaf(acc[i][j][jj * 4 + e], cs[j][jj], bias[j][jj][e]);
            if constexpr (EPI == EPI_BIAS_GELU) v[e] = gelu_fast_half(v[e]);
          }
          pk[j][jj] = u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
        }
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        if ((lrow >> 4) == half) {
#pragma unroll
          for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int jj = 0; jj < 4; ++jj)
              *(u32x2*)(st + (lrow & 15) * D_STAGING_ROW + (j * 32 + jj * 8 + lk * 4) * 2) = pk[j][jj];
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int p = 0; p < 2; ++p) {  // 8 lanes per row (8 bf16 each), 8 rows per pass
          const int sr = p * 8 + (lane >> 3);
          const u32x4 t = *(const u32x4*)(st + sr * D_STAGING_ROW + sc * 2);
          if (FULL || (i * 32 + half * 16 + p * 8 < row_lim && col_ok)) {
            u32x4* dst = (u32x4*)(tile_base + (size_t)(i * 32 + half * 16 + p * 8) * rs * 2 + lane_off);
            // STREAM_OUT: the output is larger than the memory-side cache; it passes through once and
            // would only displace the operands, so it is stored non-temporally (-1 % on the large encode
            // step).  Smaller outputs are what the next kernel finds in that cache; there the hint costs
            // 2-5 %.  (A compile-time flag: a run-time choice between the two stores gets merged into one
            // plain store.)  Whole 128-byte row pieces only: on the attention kernel's 8-byte stores the
            // hint cost 10 %.
            if constexpr (STREAM_OUT) __builtin_nontemporal_store(t, dst);
            else *dst = t;
          }
        }
        __builtin_amdgcn_wave_barrier();
      }
    }
  }
}

template <int EPI, bool STREAM_OUT>
__global__ __launch_bounds__(512) void gemm_bf16_dma_kernel(const GemmArgs a, int tiles_m, int tiles_n, int n_bands,
                                                            int groups_full, int narrow_w, int n_groups) {
  constexpr int FM = 4, FN = 2, TM = 128, TN = 64;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: keeps addresses in scalar registers
  const int wm = wave >> 2, wn = wave & 3;
  const int lrow = lane & 31, lk = lane >> 5;

  // ---- tile list of this workgroup: groups xcd, xcd + 8, ...; inside a group the unit's slot picks the tile
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;  // slot in [0, 32)
  const int sm = slot / D_GROUP_N, sn = slot % D_GROUP_N;
  auto tile_of = [&](int g, int& tm, int& tn) {  // false when the slot has no tile in group g
    if (g < groups_full) {  // 8 x 4 groups over the full-width column bands
      const int mblk = g / n_bands, band = g - mblk * n_bands;
      tm = mblk * D_GROUP_M + sm;
      tn = band * D_GROUP_N + sn;
    } else {  // the last one or two tile columns: 32 x 1 or 16 x 2 groups, so no slot idles
      tm = (g - groups_full) * (32 / narrow_w) + slot / narrow_w;
      tn = n_bands * D_GROUP_N + slot % narrow_w;
    }
    const bool ok = tm < tiles_m && tn < tiles_n;
    if (a.reverse) tm = tiles_m - 1 - tm;
    return ok;
  };
  auto next_group = [&](int g) {  // first group >= g (stride 8) in which this slot has a tile, or n_groups
    int tm, tn;
    while (g < n_groups && !tile_of(g, tm, tn)) g += 8;
    return g < n_groups ? g : n_groups;
  };

  // ---- loader addressing: one instruction fills 8 tile rows of 128 bytes (lane -> row lane/8, LDS
  //      chunk lane%8); wave w moves rows [32w, 32w + 32) of both operand tiles.  An address is a
  //      wave-uniform 64-bit base (scalar registers) plus a per-lane 32-bit byte offset that never
  //      changes.  The logical chunk that lands in LDS chunk c of row r is c ^ ((r >> 1) & 7); for
  //      row 32w + 8i + lane/8 that is (4 * (i & 1) + lane/16) & 7: two offset variants per operand.
  const int ld_row = wave * 32 + (lane >> 3);
  const int ld_chunk = (lane & 7) ^ (lane >> 4);
  const uint32_t offA0 = (uint32_t)(ld_row * a.lda + ld_chunk * 8) * 2u;
  const uint32_t offA1 = (uint32_t)(ld_row * a.lda + (ld_chunk ^ 4) * 8) * 2u;
  const uint32_t offW0 = (uint32_t)(ld_row * a.ldw + ld_chunk * 8) * 2u;
  const uint32_t offW1 = (uint32_t)(ld_row * a.ldw + (ld_chunk ^ 4) * 8) * 2u;
  const size_t a_step = (size_t)16 * a.lda, w_step = (size_t)16 * a.ldw;  // bytes per 8 rows
  // One direct-to-LDS instruction.  It is written as inline assembly so that the compiler's
  // wait-count insertion, which cannot know that the unit written here is never one being read,
  // does not fence every surrounding LDS read; completion is tracked by hand (the waits ahead of the
  // barriers).  M0 holds the LDS destination of lane 0; a scalar write of it needs one wait state ahead of
  // the load that reads it, which the compiler puts there for its own code but not inside an asm text.
  auto dma16 = [&](const unsigned char* gbase, uint32_t goff, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(goff), "s"(gbase) : "memory", "m0");
  };
  // load cursors, one per operand: the tile list position, the stage inside the tile, the tile's address at k = 0, the LDS
  // unit that is filled next
  const int KT = a.K / D_BK;
  const uint32_t lds_wave = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)smem + wave * 32 * D_ROW);  // (low 32 bits = LDS offset)
  struct Cursor { int g, kt; const unsigned char* base; uint32_t unit; };
  Cursor ca{next_group(xcd), 0, nullptr, 0}, cw = ca;
  auto set_tile = [&](Cursor& c, bool is_a) {
    int tm, tn;
    if (c.g < n_groups && tile_of(c.g, tm, tn))
      c.base = is_a ? (const unsigned char*)a.A + (size_t)tm * D_BM * a.lda * 2 : (const unsigned char*)a.W + (size_t)tn * D_BN * a.ldw * 2;
  };
  set_tile(ca, true);
  set_tile(cw, false);
  // instruction i of 4 (rows 32 wave + 8 i ..) of the operand's next stage
  auto load_a = [&](int i) { dma16(ca.base + i * a_step, (i & 1) ? offA1 : offA0, lds_wave + ca.unit + i * 8 * D_ROW); };
  auto load_w = [&](int i) {
    dma16(cw.base + i * w_step, (i & 1) ? offW1 : offW0, lds_wave + 3 * D_UNIT_BYTES + cw.unit + i * 8 * D_ROW);
  };
  auto advance = [&](Cursor& c, bool is_a) {
    c.unit = c.unit + D_UNIT_BYTES == (is_a ? 3u : 2u) * D_UNIT_BYTES ? 0 : c.unit + D_UNIT_BYTES;
    c.base += D_ROW;
    if (++c.kt == KT) {
      c.kt = 0;
      c.g = next_group(c.g + 8);
      set_tile(c, is_a);
    }
  };

  // ---- fragment addressing: row*128 + ((2ks + lk) ^ ((row >> 1) & 7)) * 16, row = 32-aligned base + lrow;
  //      with pos0 = lk ^ sw the chunk of sub-step ks is pos0 ^ 2ks, i.e. the byte offset XOR (ks << 5)
  const int sw = (lrow >> 1) & 7;
  const uint32_t fa_off = (uint32_t)((wm * TM + lrow) * D_ROW + ((lk ^ sw) << 4));
  const uint32_t fb_off = (uint32_t)(3 * D_UNIT_BYTES + (wn * TN + lrow) * D_ROW + ((lk ^ sw) << 4));

  f32x16 acc[FM][FN];
  bf16x8 fa0[FM], fa1[FM], fb[4][FN];  // A fragments of even / odd sub-steps, W fragments of all four
  uint32_t ua = 0, uw = 0;             // byte offsets of the stage being multiplied in A's and in W's units
  auto rd_a = [&](uint32_t unit, int ks, int i) {
    return *(const bf16x8*)(smem + unit + (fa_off ^ (uint32_t)(ks << 5)) + i * 32 * D_ROW);
  };
  auto rd_b = [&](uint32_t unit, int ks, int j) {
    return *(const bf16x8*)(smem + unit + (fb_off ^ (uint32_t)(ks << 5)) + j * 32 * D_ROW);
  };
  auto mm = [&](int i, const bf16x8& x, const bf16x8 (&w)[FN]) {
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[j], x, acc[i][j], 0, 0, 0);
  };

  // ---- how many k-stages this workgroup multiplies in total
  int n_my_tiles = 0;
  for (int g = next_group(xcd); g < n_groups; g = next_group(g + 8)) ++n_my_tiles;
  const int total_stages = n_my_tiles * KT;
  int stage = 0;  // the one being multiplied

  // One 64-wide k-stage.  On entry fa0 / fb[0] hold the fragments of its sub-step 0.
  //   sub-step 0: the W fragments of the other three sub-steps are read, and A's of the next;
  //   barrier:    every wave has its W fragments, W's unit is dead: it takes W of stage + 2 (one load per MFMA pair);
  //   sub-step 2: reads the last A fragments;
  //   sync:       stage + 1 has landed for every wave (A and W of stage + 2 may be in flight), A's unit is dead: it takes A
  //               of stage + 3, in sub-step 3, which reads the next stage's first fragments.
  // last = a tile's last stage: the loads of A wait until the epilogue has used the unit; in the residual kernel the next
  // tile's first fragments are read behind the epilogue, too, which needs their registers for residual values.
  bool pend_a = false;  // the second half of A's loads is still to be issued
  // STEADY: no tile end, and the stages whose loads go out exist: no branch but the cursors'
  auto k_stage = [&](auto steady_tag, const bool last) {
    constexpr bool STEADY = decltype(steady_tag)::value;
    const uint32_t una = ua + D_UNIT_BYTES == 3u * D_UNIT_BYTES ? 0 : ua + D_UNIT_BYTES, unw = uw ^ D_UNIT_BYTES;
    const bool more_w = STEADY || stage + 2 < total_stages, more_a = STEADY || (stage + 3 < total_stages && !last);
    const bool ahead = STEADY || (stage + 1 < total_stages && !(last && EPI == EPI_BIAS_RESIDUAL)), pend = STEADY || pend_a;
    fa1[0] = rd_a(ua, 1, 0); fb[1][0] = rd_b(uw, 1, 0); fb[1][1] = rd_b(uw, 1, 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      mm(i, fa0[i], fb[0]);
      if (i + 1 < FM) fa1[i + 1] = rd_a(ua, 1, i + 1);
      if (i < 2) { fb[2 + i][0] = rd_b(uw, 2 + i, 0); fb[2 + i][1] = rd_b(uw, 2 + i, 1); }
      if ((i & 1) && pend) load_a(2 + (i >> 1));
      __builtin_amdgcn_sched_barrier(0);
    }
    if (pend) advance(ca, true);
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      mm(i, fa1[i], fb[1]);
      fa0[i] = rd_a(ua, 2, i);
      if (i == 0) {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0xC27F);  // lgkmcnt(2): the last reads of fa1 and of fa0 so far came behind those of fb
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
      }
      if ((i & 1) && more_w) load_w(i >> 1);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < FM; ++i) fa1[i] = rd_a(ua, 3, i);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      mm(i, fa0[i], fb[2]);
      if (!(i & 1) && more_w) load_w(2 + (i >> 1));
      __builtin_amdgcn_sched_barrier(0);
    }
    if (more_w) advance(cw, false);
    if (more_w) __builtin_amdgcn_s_waitcnt(0x0078);  // vmcnt(8) lgkmcnt(0)
    else __builtin_amdgcn_s_waitcnt(0x0070);         // vmcnt(0) lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    if (ahead) { fb[0][0] = rd_b(unw, 0, 0); fb[0][1] = rd_b(unw, 0, 1); fa0[0] = rd_a(una, 0, 0); }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      mm(i, fa1[i], fb[3]);
      if (ahead && i + 1 < FM) fa0[i + 1] = rd_a(una, 0, i + 1);
      if ((i & 1) && more_a) load_a(i >> 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (!STEADY) pend_a = more_a;
    ua = una;
    uw = unw;
    ++stage;
  };

  // ---- prologue: A of three stages, W of two, in the order in which the stages above would have asked for them
#pragma unroll
  for (int st = 0; st < 3; ++st) {
    if (st < total_stages) {
#pragma unroll
      for (int i = 0; i < (st < 2 ? 4 : 2); ++i) load_a(i);
      if (st < 2) advance(ca, true);
      else pend_a = true;
    }
    if (st < 2 && st < total_stages) {
#pragma unroll
      for (int i = 0; i < 4; ++i) load_w(i);
      advance(cw, false);
    }
  }
  if (total_stages > 0) {
    if (total_stages >= 3) __builtin_amdgcn_s_waitcnt(0x007A);  // vmcnt(10): stage 0 has landed
    else __builtin_amdgcn_s_waitcnt(0x0070);
    __builtin_amdgcn_s_barrier();
    fb[0][0] = rd_b(0, 0, 0); fb[0][1] = rd_b(0, 0, 1);
#pragma unroll
    for (int i = 0; i < FM; ++i) fa0[i] = rd_a(0, 0, i);
  }

  int stamp_i = 0;  // measurement aid: tiles of this workgroup stamped so far
  for (int g_c = next_group(xcd); g_c < n_groups; g_c = next_group(g_c + 8)) {
    int tm, tn;
    tile_of(g_c, tm, tn);
    // measurement aid (off unless the host asked for it): constant-rate clock at the tile's start, after its
    // k-loop and after its epilogue, and the shader clocks the tile took
    unsigned long long stamp_t0 = 0, stamp_t1 = 0, stamp_c0 = 0;
    if (a.tile_stamps) { stamp_t0 = wall_clock64(); stamp_c0 = __builtin_readcyclecounter(); }
    const int row0 = tm * D_BM + wm * TM, ncol0 = tn * D_BN + wn * TN;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    constexpr bool RESID = EPI == EPI_BIAS_RESIDUAL;
    unsigned char* staging = smem;
    const int steady = pend_a ? min(KT - 1, total_stages - 3 - stage) : 0;
    int kt = 0;
    for (; kt < steady; ++kt) k_stage(std::true_type{}, false);
    for (; kt < KT; ++kt) {
      if (kt == KT - 1) staging = smem + ua + wave * 32 * D_ROW;  // A's unit of the last stage: dead behind its sync, refilled below
      k_stage(std::false_type{}, kt == KT - 1);
    }
    if constexpr (RESID) {  // the fragment registers are dead across the epilogue: say so
#pragma unroll
      for (int i = 0; i < FM; ++i) fa0[i] = bf16x8{};
      fb[0][0] = bf16x8{}; fb[0][1] = bf16x8{};
    }
    asm volatile("" ::: "memory");  // keep the epilogue's loads below the k-loop
    if (a.tile_stamps) stamp_t1 = wall_clock64();
    // a wave's 128 x 64 block lies wholly inside the matrix for all but the last row block / a ragged last column
    if (row0 + TM <= a.M && ncol0 + TN <= a.N)
      wave_epilogue_p<EPI, STREAM_OUT, true>(a, acc, staging, row0, ncol0, lane);
    else
      wave_epilogue_p<EPI, STREAM_OUT, false>(a, acc, staging, row0, ncol0, lane);
    if (stage + 2 < total_stages) {  // the loads of A that the last stage held back: into the rows that only this wave has staged in
      __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
      load_a(0);
      load_a(1);
      pend_a = true;
    }
    if constexpr (RESID) {  // the next tile's first fragments (its first stage landed before the last sync)
      if (stage < total_stages) {
        fb[0][0] = rd_b(uw, 0, 0); fb[0][1] = rd_b(uw, 0, 1);
#pragma unroll
        for (int i = 0; i < FM; ++i) fa0[i] = rd_a(ua, 0, i);
      }
    }
    if (a.tile_stamps) {
      asm volatile("" ::: "memory");
      const unsigned long long stamp_t2 = wall_clock64();
      if (tid == 0 && stamp_i < kTileStampSlots) {
        unsigned long long* d = a.tile_stamps + ((size_t)blockIdx.x * kTileStampSlots + stamp_i) * 4;
        d[0] = stamp_t0; d[1] = stamp_t1; d[2] = stamp_t2;
        d[3] = __builtin_readcyclecounter() - stamp_c0 + 1;  // never 0: marks the slot as written
      }
      ++stamp_i;
    }
  }
}

// ---------------------------------------------------------------------------------------------
// One BM x BN tile per workgroup, WM x WN waves of BM/WM x BN/WN, operands global -> LDS directly into a ring of NS 64-wide
// k-stages.  A stage is multiplied in groups of G 16-wide sub-steps; a group's fragments are read while the group before it
// is multiplied, into the other of two register sets.  Ahead of a stage's last group one wait + barrier establishes that
// the next stage has landed for every wave and that nobody reads this one's LDS any more; from there on the loads of the
// stage that takes its place go out, one after every few MFMAs, for as long as it takes to come round to the next barrier.
// What bounds it: alone on its unit (few workgroups) a stage takes 1.3 to 1.5 times its MFMAs, or its loads at 64 bytes
// per clock if those are more (64 x 64: 0.18 us a stage against 0.11); with all units at work the shader clock falls under
// the power cap (a 256 x 128 stage 0.53 us with 24 workgroups, 0.75 with 224, the same with every operand in the L2).  Its
// predecessor read all of a stage's fragments and then multiplied, and issued a stage's loads back to back, so that loads,
// reads and MFMAs added up: fc2 of 577 rows (1024 x 4096, 160 tiles of 64 x 64) 19.2 us, now 14.5; of 1154 rows 26.1 and
// 19.9; out-proj of 577 rows 7.6 and 6.1.
// Beyond one round of tiles their height decides: a product of 4616 x 1024 x 4096 took 61 us on tiles of 128 x 128 (296 of
// them on 256 units) and takes 44 on 200 of 192 x 128.  Hence heights of 64 to 256 rows, chosen by pipe_time below.
// Tiles are dealt to the XCDs in eight runs of equal length (workgroup id mod 8 = XCD) of an order that walks four row blocks
// at a time, column by column: an XCD's tiles share A and W rows in its L2, and none has a tile more than another, which
// the former cut into rectangles could not give (5103 x 1152 x 4352 on tiles of 192 x 128: 85 us so, 54 in runs; groups
// of eight row blocks are up to 3 % slower).
// A token's k-steps are added in the same order in every variant, and as in the persistent kernel.

// vmcnt(N) lgkmcnt(0): N of this wave's vector-memory operations may be in flight, none of its LDS operations
template <int N>
__device__ __forceinline__ void wait_loads() {
  static_assert(N >= 0 && N < 64, "vmcnt has six bits");
  __builtin_amdgcn_s_waitcnt(0x0070 | (N & 15) | ((N >> 4) << 14));
}

// n / d and the remainder, both wave-uniform, for 0 <= n < 2^31 and d > 0: a quarter of the instructions of the division
__device__ __forceinline__ int div_uniform(int n, int d, int& rem) {
  const float inv = __builtin_amdgcn_rcpf((float)d);
  int c = (int)((float)n * inv);  // off by at most n / d * 2^-22 + 1
  rem = n - c * d;
  const int more = (int)((float)rem * inv);  // by at most 1
  c += more;
  rem -= more * d;
  if (rem < 0) { --c; rem += d; }
  if (rem >= d) { ++c; rem -= d; }
  rem = __builtin_amdgcn_readfirstlane(rem);
  return __builtin_amdgcn_readfirstlane(c);
}

template <int EPI, int NS, int BM, int BN, int WM, int WN, int G>
__global__ __launch_bounds__(WM * WN * 64) void gemm_bf16_pipe_kernel(const GemmArgs a, int tiles_m, int tiles_n, int n_tiles) {
  constexpr int STAGE = (BM + BN) * D_ROW, NW = WM * WN, TM = BM / WM, TN = BN / WN, FM = TM / 32, FN = TN / 32;
  constexpr int LA = BM / 8 / NW, LW = BN / 8 / NW, LOADS = LA + LW;  // direct-to-LDS instructions per wave and stage, 8 rows each
  static_assert(LA * NW * 8 == BM && LW * NW * 8 == BN && FM * 32 * WM == BM && FN * 32 * WN == BN, "whole pieces and blocks");
  static_assert(256 % BN == 0 && 64 % TN == 0, "W rows are padded to 256; the epilogue's lanes share a row evenly");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

  // ---- tile assignment: XCD x takes n_tiles / 8 tiles, one more if x < n_tiles % 8
  const int xcd = blockIdx.x & 7, q = blockIdx.x >> 3;
  const int per = n_tiles >> 3, more = n_tiles & 7;
  if (q >= per + (xcd < more ? 1 : 0)) return;
  int rem, r;
  const int group = div_uniform(xcd * per + min(xcd, more) + q, GROUP_M * tiles_n, rem);
  const int tile_n = div_uniform(rem, min(GROUP_M, tiles_m - group * GROUP_M), r);
  const int m0 = (group * GROUP_M + r) * BM, n0 = tile_n * BN;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int lrow = lane & 31, lk = lane >> 5;

  // ---- loader: an instruction fills 8 rows of 128 bytes (a piece); the chunk that lands in LDS chunk c of row r is
  //      c ^ ((r >> 1) & 7).  Rows of A past the matrix are its last row again: tile heights need not divide the padding.
  const int ld_chunk = (lane & 7) ^ (lane >> 4);
  uint32_t offA[LA], offW[LW];
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    const int p = wave * LA + i;
    offA[i] = (uint32_t)(min(p * 8 + (lane >> 3), a.M - 1 - m0) * a.lda + (ld_chunk ^ (4 * (p & 1))) * 8) * 2u;
  }
#pragma unroll
  for (int i = 0; i < LW; ++i) {
    const int p = wave * LW + i;
    offW[i] = (uint32_t)((p * 8 + (lane >> 3)) * a.ldw + (ld_chunk ^ (4 * (p & 1))) * 8) * 2u;
  }
  const unsigned char* const baseA = (const unsigned char*)a.A + (size_t)m0 * a.lda * 2;
  const unsigned char* const baseW = (const unsigned char*)a.W + (size_t)n0 * a.ldw * 2;
  const uint32_t lds0 = (uint32_t)(uintptr_t)smem;  // low 32 bits of a generic LDS pointer = LDS offset
  auto dma16 = [&](const unsigned char* gbase, uint32_t goff, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(goff), "s"(gbase) : "memory", "m0");
  };
  auto issue = [&](int slot, int kt, int i) {  // instruction i of stage kt into the ring slot at byte `slot`
    const uint32_t st = __builtin_amdgcn_readfirstlane(lds0 + slot);
    if (i < LA) dma16(baseA + kt * D_ROW, offA[i], st + (wave * LA + i) * 8 * D_ROW);
    else dma16(baseW + kt * D_ROW, offW[i - LA], st + (BM + (wave * LW + i - LA) * 8) * D_ROW);
  };

  // ---- the first NS stages (of a shorter product: its last one again, so that the waits can count them), and behind
  //      the first of them what the epilogue will need
  const int KT = a.K / D_BK;
#pragma unroll
  for (int i = 0; i < LOADS; ++i) issue(0, 0, i);
  WaveEpilogue<EPI, FM, FN, (NS > 2)> epilogue;
  epilogue.prefetch(a, m0 + wm * TM, n0 + wn * TN, lane);
  asm volatile("" ::: "memory");  // keep those loads here
#pragma unroll
  for (int s = 1; s < NS; ++s)
#pragma unroll
    for (int i = 0; i < LOADS; ++i) issue(s * STAGE, min(s, KT - 1), i);

  // ---- fragments: group g of a stage is read into set g & 1
  const int sw = (lrow >> 1) & 7;
  const uint32_t fa_off = (uint32_t)((wm * TM + lrow) * D_ROW + ((lk ^ sw) << 4));
  const uint32_t fb_off = (uint32_t)((BM + wn * TN + lrow) * D_ROW + ((lk ^ sw) << 4));
  f32x16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  constexpr int NG = 4 / G, NMG = G * FM * FN, SLOTS = 4 * FM * FN;  // groups, MFMAs of a group and of a stage
  static_assert(NG % 2 == 0, "a stage's first group is read into the same set every time");
  bf16x8 fa[2][G][FM], fb[2][G][FN];
  auto read = [&](int set, int slot, int g) {
#pragma unroll
    for (int ks = 0; ks < G; ++ks) {
#pragma unroll
      for (int j = 0; j < FN; ++j) fb[set][ks][j] = *(const bf16x8*)(smem + slot + (fb_off ^ (uint32_t)((g * G + ks) << 5)) + j * 32 * D_ROW);
#pragma unroll
      for (int i = 0; i < FM; ++i) fa[set][ks][i] = *(const bf16x8*)(smem + slot + (fa_off ^ (uint32_t)((g * G + ks) << 5)) + i * 32 * D_ROW);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // the MFMAs of a set; with LOAD, instruction l of stage kt follows the MFMA l * SLOTS / LOADS places behind the barrier
  // (the set's first one is `first` places behind it)
  auto mul = [&](auto load_tag, int set, int slot, int kt, int first) {
    constexpr bool LOAD = decltype(load_tag)::value;
#pragma unroll
    for (int m = 0; m < NMG; ++m) {
      const int ks = m / (FM * FN), i = m / FN % FM, j = m % FN;
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[set][ks][j], fa[set][ks][i], acc[i][j], 0, 0, 0);
      if constexpr (LOAD) {
#pragma unroll
        for (int l = 0; l < LOADS; ++l)
          if (l * SLOTS / LOADS == first + m) issue(slot, kt, l);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  const std::true_type T{};
  const std::false_type F{};
  wait_loads<(NS - 1) * LOADS>();  // (the epilogue's loads are older than those that may be in flight here)
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  int cur = 0;  // byte offset of the slot being multiplied
  read(0, 0, 0);
#pragma unroll
  for (int g = 0; g + 1 < NG; ++g) {
    read((g + 1) & 1, cur, g + 1);
    mul(F, g & 1, 0, 0, 0);
  }
  // From barrier to barrier: the last group of stage kt, then all but the last of stage kt + 1.  (The loads are behind a
  // compile-time flag: a branch around them made the compiler copy all accumulators twice a stage.)
  auto step = [&](auto load_tag, int kt) {
    const int nxt = cur + STAGE == NS * STAGE ? 0 : cur + STAGE;
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    read(0, nxt, 0);
    mul(load_tag, 1, cur, kt + NS, 0);
#pragma unroll
    for (int g = 0; g + 1 < NG; ++g) {
      read((g + 1) & 1, nxt, g + 1);
      mul(load_tag, g & 1, cur, kt + NS, (g + 1) * NMG);
    }
    cur = nxt;
  };
  int kt = 0;
  for (; kt < KT - NS; ++kt) {
    wait_loads<(NS - 2) * LOADS>();  // stage kt + 1 has landed; stages kt + 2 .. kt + NS - 1 may be in flight
    step(T, kt);
  }
  for (; kt < KT - 1; ++kt) {
    const int newer = KT - 2 - kt;  // stages behind kt + 1, at most NS - 2
    if (NS >= 5 && newer >= 3) wait_loads<NS >= 5 ? 3 * LOADS : 0>();
    else if (NS >= 4 && newer >= 2) wait_loads<NS >= 4 ? 2 * LOADS : 0>();
    else if (NS >= 3 && newer >= 1) wait_loads<NS >= 3 ? LOADS : 0>();
    else wait_loads<0>();
    step(F, kt);
  }
  mul(F, 1, 0, 0, 0);
  wait_loads<0>();  // (a product of fewer than NS stages may still be loading)
  __builtin_amdgcn_s_barrier();
  epilogue.finish(a, acc, smem, m0 + wm * TM, n0 + wn * TN, wave, lane);
}

template <int NS, int BM, int BN, int WM, int WN, int G>
hipError_t launch_pipe_as(const GemmArgs& a, hipStream_t s) {
  const int tiles_m = (a.M + BM - 1) / BM, tiles_n = (a.N + BN - 1) / BN;
  const long n_tiles = (long)tiles_m * tiles_n, grid = (n_tiles + 7) / 8 * 8;
  if (grid > 0x7fffffffL) return hipErrorInvalidValue;
  constexpr int lds = NS * (BM + BN) * D_ROW;
  static_assert(NS >= 2 && NS <= 5 && lds <= 160 * 1024, "the waits of the last stages; a unit's LDS");
  static_assert(WM * WN * 32 * (BN / WN * 4 + 16) <= lds, "epilogue staging must fit in the ring");
#define VIT_LAUNCH(EPI)                                                                                            \
  do {                                                                                                             \
    auto kfn = gemm_bf16_pipe_kernel<EPI, NS, BM, BN, WM, WN, G>;                                                  \
    static LdsLimitOnce lds_limit;                                                                                 \
    if (hipError_t e = lds_limit.ensure((const void*)kfn, lds); e != hipSuccess) return e;                         \
    hipLaunchKernelGGL(kfn, dim3((unsigned)grid), dim3(WM * WN * 64), lds, s, a, tiles_m, tiles_n, (int)n_tiles);  \
  } while (0)
  switch (a.epilogue) {
    case EPI_BIAS: VIT_LAUNCH(EPI_BIAS); break;
    case EPI_BIAS_HEADS: VIT_LAUNCH(EPI_BIAS_HEADS); break;
    case EPI_BIAS_GELU: VIT_LAUNCH(EPI_BIAS_GELU); break;
    case EPI_BIAS_RESIDUAL: VIT_LAUNCH(EPI_BIAS_RESIDUAL); break;
    case EPI_PATCH: VIT_LAUNCH(EPI_PATCH); break;
    default: return hipErrorInvalidValue;
  }
#undef VIT_LAUNCH
  return hipGetLastError();
}

// The time that a product is expected to take, in us.  A round is one tile (or, where two workgroups share a unit, two) on
// each of 256 units; a stage takes `alone` with few units at work and `full` with all of them (the clock falls), and a
// round has a fixed time of its own and an epilogue by its kind: bias, bias + GELU, residual or patch rows.  Fitted to
// the times of 20 encoder products (out-proj, QKV, fc1 and fc2 at widths of 768, 1024, 1152, 1280 and 3200, so 768 to
// 12 800 columns and stages of 12 to 200) at 18 sizes each of 197 to 160 000 rows, weighted towards the tiles that are near
// the best one.  bench.py --product-times times every form on the products of nine encoders of 384 to 3200 columns, four of them
// not among those: the form chosen is on average 0.9 % slower than the best of the ten there, 0.9 and 0.8 % at 26 other numbers of rows
// and at five other widths.  (Two launches of the choice that this one replaced, by numbers of tiles alone and with 256 x 256, 128 x
// 128, 64 x 128 and 64 x 64 to choose from, took 13 % longer.)
// Patch rows have epilogues of their own, fitted to the patch embeddings of four encoders (1024 to 3200 columns) at 1 to 260 tiles
// of pixels: on the one-tile kernel they take 1.5 to 2.5 times a residual's, on the persistent one less than that.  Priced as
// residual rows, products of many rounds stayed on the one-tile kernel (149760 x 1024 x 640: 477 us, 294 on the persistent
// one); with these the tile chosen is on average 1 % slower than the best of the ten.
struct TileTime { int bm, bn, per_unit; float alone, full, fixed, epilogue[4]; };
constexpr float LAUNCH_US = 1.8f;
constexpr TileTime PIPE_TILES[] = {
    {64, 64, 2, 0.191f, 0.389f, 1.6f, {0.0f, 0.0f, 0.1f, 1.0f}},
    {64, 128, 1, 0.204f, 0.331f, 2.1f, {0.0f, 0.0f, 0.2f, 2.4f}},
    {96, 128, 1, 0.319f, 0.415f, 1.4f, {0.0f, 1.1f, 2.0f, 5.0f}},
    {128, 128, 1, 0.310f, 0.500f, 1.7f, {0.0f, 0.6f, 2.7f, 7.1f}},
    {160, 128, 1, 0.284f, 0.605f, 2.5f, {0.0f, 1.3f, 4.4f, 7.5f}},
    {192, 128, 1, 0.315f, 0.707f, 1.8f, {0.0f, 1.1f, 5.1f, 10.2f}},
    {256, 128, 1, 0.312f, 0.880f, 2.7f, {0.0f, 1.2f, 6.9f, 13.3f}},
    {160, 128, 2, 0.759f, 1.142f, 0.0f, {1.1f, 2.0f, 5.0f, 8.2f}},
    {192, 128, 2, 0.768f, 1.278f, 0.0f, {1.6f, 2.5f, 6.2f, 10.1f}},
};
constexpr int PIPE_TILE_COUNT = sizeof(PIPE_TILES) / sizeof(PIPE_TILES[0]);
static_assert(PIPE_TILE_COUNT == PRODUCT_PERSISTENT, "forms are numbered tiles first");

int epilogue_kind(int epilogue) {
  return epilogue == EPI_BIAS_GELU ? 1 : epilogue == EPI_BIAS_RESIDUAL ? 2 : epilogue == EPI_PATCH ? 3 : 0;
}

float pipe_time(const TileTime& t, int kind, long M, long N, int stages) {
  const long n = ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn), cap = 256L * t.per_unit;
  auto round = [&](long c) {
    if (t.per_unit == 1) {
      const float u = c / 256.0f;
      return t.fixed + stages * (t.alone + (t.full - t.alone) * u) + t.epilogue[kind] * (0.3f + 0.7f * u);
    }
    if (c <= 256) return t.fixed + stages * t.alone + t.epilogue[kind] * (0.3f + 0.7f * c / 256.0f);
    const float u = (c - 256) / 256.0f;
    return t.fixed + stages * (t.alone + (t.full - t.alone) * (0.85f + 0.15f * u)) + t.epilogue[kind] * (1.0f + u);
  };
  return LAUNCH_US + (n / cap) * round(cap) + (n % cap ? round(n % cap) : 0.0f);
}

struct PipeChoice { int tile; float us; };
PipeChoice best_pipe(int kind, long M, long N, int stages) {
  PipeChoice best{0, pipe_time(PIPE_TILES[0], kind, M, N, stages)};
  for (int i = 1; i < PIPE_TILE_COUNT; ++i) {
    const float us = pipe_time(PIPE_TILES[i], kind, M, N, stages);
    if (us < best.us) best = {i, us};
  }
  // Operand and output that the memory-side cache cannot hold together slow all tiles down where the persistent kernel stays as
  // it was: 384 columns of K = 768 with position rows, 86 550 rows 84.5 us on tiles and 83.5 on the persistent kernel, 98 000
  // rows 110.6 and 89.0; 512 of K = 2048 with residual, 51 232 rows 145 and 132, 57 700 rows 160 and 137.  With 0.06 us a MB the
  // form chosen is on average 0.5 % slower than the best of the ten from 15 000 rows on, without it 1.0 %.
  const double bytes = (double)M * (stages * (BK * 2) + N * (kind < 2 ? 2 : 4));
  if (bytes > 256.0 * 1024 * 1024) best.us += (float)(0.06e-6 * bytes);
  return best;
}

hipError_t launch_pipe(const GemmArgs& a, int tile, hipStream_t s) {
  // The longer a product of few 64 x 64 tiles, the more of its stages wait for weights that no unit has read yet: a fifth
  // stage is worth 5 to 9 % from K = 4096 on (fc2 of 577 rows, 1024 x 4096, 15.0 us and 13.9; of 729 rows, 1152 x 4352, 19.9
  // and 18.3; 577 rows, 1280 x 5120, 23.3 and 20.5), nothing at K = 3072 and below, and it costs products of two workgroups to
  // a unit 2 to 4 % (QKV of 577 rows 9.4 and 9.7).
  const bool long_alone = a.K >= 4096 && (long)((a.M + 63) / 64) * ((a.N + 63) / 64) <= 256;
  switch (tile) {
    case 0: return long_alone ? launch_pipe_as<5, 64, 64, 2, 2, 2>(a, s) : launch_pipe_as<4, 64, 64, 2, 2, 2>(a, s);
    case 1: return launch_pipe_as<4, 64, 128, 2, 4, 2>(a, s);
    case 2: return launch_pipe_as<4, 96, 128, 1, 4, 1>(a, s);
    case 3: return launch_pipe_as<4, 128, 128, 2, 4, 1>(a, s);
    case 4: return launch_pipe_as<4, 160, 128, 1, 4, 1>(a, s);
    case 5: return launch_pipe_as<3, 192, 128, 2, 4, 1>(a, s);
    case 6: return launch_pipe_as<3, 256, 128, 4, 2, 1>(a, s);
    case 7: return launch_pipe_as<2, 160, 128, 1, 4, 1>(a, s);
    case 8: return launch_pipe_as<2, 192, 128, 2, 2, 1>(a, s);
    default: break;
  }
  return hipErrorInvalidValue;
}

// The persistent kernel's walk: column bands of four tiles; a remainder of one or two tile columns gets its own group shape (a
// remainder of three is a band with one idle column).  An XCD takes every eighth group, so a round is eight groups.
struct Walk { int tiles_m, tiles_n, narrow_w, n_bands, groups_full, n_groups; };
Walk persistent_walk(long M, long N) {
  Walk w;
  w.tiles_m = (int)((M + D_BM - 1) / D_BM);
  w.tiles_n = (int)((N + D_BN - 1) / D_BN);
  const int rem = w.tiles_n % D_GROUP_N;
  w.narrow_w = rem == 3 ? 0 : rem;
  w.n_bands = w.tiles_n / D_GROUP_N + (rem == 3 ? 1 : 0);
  w.groups_full = ((w.tiles_m + D_GROUP_M - 1) / D_GROUP_M) * w.n_bands;
  w.n_groups = w.groups_full + (w.narrow_w ? (w.tiles_m + 32 / w.narrow_w - 1) / (32 / w.narrow_w) : 0);
  return w;
}

constexpr TileTime PERSISTENT_TILE = {256, 256, 1, 0.675f, 1.513f, 4.5f, {4.3f, 7.2f, 17.2f, 14.2f}};
constexpr float NARROW_GROUP = 0.11f;  // what the groups of a remainder's columns take longer than those of a band
float persistent_time(int kind, long M, long N, int stages) {
  const Walk w = persistent_walk(M, N);
  const int rounds = (w.n_groups + 7) / 8;
  const float u = (float)w.tiles_m * w.tiles_n / (256.0f * rounds), narrow = (float)(w.n_groups - w.groups_full) / w.n_groups;
  const TileTime& t = PERSISTENT_TILE;
  return LAUNCH_US + t.fixed + rounds * (stages * (t.alone + (t.full - t.alone) * u) + t.epilogue[kind]) * (1.0f + NARROW_GROUP * narrow);
}

constexpr int PERSISTENT_GRID = 8 * D_GROUP_M * D_GROUP_N;  // one workgroup per compute unit: 8 XCDs x 32 slots

// compute units of the current device, looked up once per device
hipError_t compute_units(int* units) {
  static std::atomic<int> of_device[64];
  int dev = 0;
  if (hipError_t e = hipGetDevice(&dev); e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  *units = of_device[dev].load(std::memory_order_relaxed);
  if (*units == 0) {
    if (hipError_t e = hipDeviceGetAttribute(units, hipDeviceAttributeMultiprocessorCount, dev); e != hipSuccess) return e;
    of_device[dev].store(*units, std::memory_order_relaxed);
  }
  return hipSuccess;
}

hipError_t launch_dma(const GemmArgs& a, hipStream_t s) {
  const Walk w = persistent_walk(a.M, a.N);
#define VIT_LAUNCH(EPI, STREAM)                                                                                      \
  do {                                                                                                               \
    auto kfn = gemm_bf16_dma_kernel<EPI, STREAM>;                                                                    \
    static LdsLimitOnce lds_limit;                                                                                   \
    if (hipError_t e = lds_limit.ensure((const void*)kfn, D_LDS_BYTES); e != hipSuccess) return e;                   \
    hipLaunchKernelGGL(kfn, dim3(PERSISTENT_GRID), dim3(512), D_LDS_BYTES, s, a, w.tiles_m, w.tiles_n, w.n_bands,    \
                       w.groups_full, w.narrow_w, w.n_groups);                                                       \
  } while (0)
  switch (a.epilogue) {
    case EPI_BIAS:
      if (a.stream_out) VIT_LAUNCH(EPI_BIAS, true);
      else VIT_LAUNCH(EPI_BIAS, false);
      break;
    case EPI_BIAS_HEADS:
      if (a.stream_out) VIT_LAUNCH(EPI_BIAS_HEADS, true);
      else VIT_LAUNCH(EPI_BIAS_HEADS, false);
      break;
    case EPI_BIAS_GELU:
      if (a.stream_out) VIT_LAUNCH(EPI_BIAS_GELU, true);
      else VIT_LAUNCH(EPI_BIAS_GELU, false);
      break;
    case EPI_BIAS_RESIDUAL: VIT_LAUNCH(EPI_BIAS_RESIDUAL, false); break;
    case EPI_PATCH: VIT_LAUNCH(EPI_PATCH, false); break;
    default: return hipErrorInvalidValue;
  }
#undef VIT_LAUNCH
  return hipGetLastError();
}

}  // namespace

int gemm_row_pad() { return 256; }

// Which kernels a product takes.  kind as in TileTime::epilogue.
ProductPlan plan_product(int epilogue, long M, long N, int K, int units, bool reverse) {
  const int kind = epilogue_kind(epilogue), stages = K / BK;
  const PipeChoice pipe = best_pipe(kind, M, N, stages);
  ProductPlan plan{pipe.tile, 0, 0, pipe.us};
  // The unit count is a performance assumption only (no workgroup waits for another): a device with fewer of them takes
  // one workgroup per tile.
  if (units < PERSISTENT_GRID) return plan;
  const float whole = persistent_time(kind, M, N, stages);
  if (whole < plan.us) plan = {PRODUCT_PERSISTENT, 0, 0, whole};
  // A product one column band wide (1, 2 or 4 tile columns) is walked in rounds of 256 / tiles_n row blocks, one tile per
  // unit.  Where the last round leaves most units idle for a whole tile time, its rows go to the other kernel in a second
  // launch (fc2 of 20195 x 1024 x 4096: 174 us so, 216 without).  All kernels give a row the same bits, so where the cut
  // falls does not show in the result.  It is made at the end that the walk reaches last.
  const int tiles_m = (int)((M + D_BM - 1) / D_BM), tiles_n = (int)((N + D_BN - 1) / D_BN);
  if (epilogue != EPI_PATCH && (tiles_n == 1 || tiles_n == 2 || tiles_n == 4)) {
    const int per_round = 256 / tiles_n, tail_blocks = tiles_m % per_round;
    if (tail_blocks > 0 && tiles_m > per_round) {
      const long main_rows = (long)(tiles_m - tail_blocks) * D_BM;
      const float us = persistent_time(kind, main_rows, N, stages) + best_pipe(kind, M - main_rows, N, stages).us;
      if (us < plan.us) {
        const long rest = reverse ? (long)tail_blocks * D_BM : M - main_rows;  // (walked in reverse, the persistent kernel takes
                                                                               //  the last rows, ragged row block included)
        plan = {PRODUCT_PERSISTENT, (int)rest, best_pipe(kind, rest, N, stages).tile, us};
      }
    }
  }
  return plan;
}

hipError_t launch_gemm_bf16(const GemmArgs& a, hipStream_t s, int form) {
  if (a.M <= 0 || a.N <= 0) return hipSuccess;
  // 16-byte epilogue accesses need 8-element aligned columns and leading dimensions
  if (a.K <= 0 || a.K % BK != 0 || a.lda % 8 != 0 || a.ldw % 8 != 0 || a.ldo % 8 != 0 || a.N % 8 != 0)
    return hipErrorInvalidValue;
  // head-by-head output: heads of 64 or 128 columns (a wave's column block never straddles two)
  if (a.epilogue == EPI_BIAS_HEADS && (a.hm_dh <= 0 || a.hm_dh % 64 != 0 || a.hm_rows < (size_t)a.M)) return hipErrorInvalidValue;
  if (form >= 0) return form == PRODUCT_PERSISTENT ? launch_dma(a, s) : launch_pipe(a, form, s);
  int units = 0;
  if (hipError_t e = compute_units(&units); e != hipSuccess) return e;
  const ProductPlan plan = plan_product(a.epilogue, a.M, a.N, a.K, units, a.reverse != 0);
  if (plan.rest_rows > 0) {
    auto rows_from = [&](int row0, int rows) {
      GemmArgs b = a;
      b.M = rows;
      b.A = (const unsigned char*)a.A + (size_t)row0 * a.lda * 2;
      if (a.out) b.out = (unsigned char*)a.out + (size_t)row0 * (a.epilogue == EPI_BIAS_HEADS ? a.hm_dh : a.ldo) * 2;  // a row's stride
      if (a.resid) b.resid = a.resid + (size_t)row0 * a.ldo;
      return b;
    };
    const int cut = a.reverse ? plan.rest_rows : a.M - plan.rest_rows;
    const GemmArgs lower = rows_from(0, cut), upper = rows_from(cut, a.M - cut);
    if (hipError_t e = launch_dma(a.reverse ? upper : lower, s); e != hipSuccess) return e;
    return launch_pipe(a.reverse ? lower : upper, plan.rest_form, s);
  }
  return plan.form == PRODUCT_PERSISTENT ? launch_dma(a, s) : launch_pipe(a, plan.form, s);
}

}  // namespace vitenc
