// fp32 arithmetic mode: matrix product and attention on the fp32 matrix instruction (products and sums in fp32
// throughout).  This mode exists for exact-arithmetic parity runs on small encoders.
//
// Both kernels cut their contraction over the four waves of a workgroup and add the four partial results in LDS in a
// fixed order: the shapes of this mode are a few hundred rows by a few hundred columns, so what bounds them is the
// length of one wave's chain of dependent steps, not the rate of any unit.  Operands go from global memory straight to
// registers (v_mfma_f32_32x32x2_f32 takes one fp32 value per lane and takes 64 clocks: the L1 delivers faster than
// that), several k-blocks ahead; no LDS is written before the final sum.
#include "common.h"

namespace vitenc {

namespace {

// C[M, N] = A[M, K] . W[N, K]^T, tile 32 F x 32 F.  Wave w takes k-values [16w, 16w + 16) of every 64: two chunks of 8,
// of which a lane half takes 4 consecutive values each (one 16-byte load per 32 rows).  The product is formed
// transposed, so a lane holds four consecutive columns of one row per register quad.  A row's sums are formed in the
// same order whatever F is, so a token does not depend on the tile size its launch took.
// Operand rows are padded by the host so tile loads never leave the buffers.
// DEPTH k-blocks are in flight per wave, and a unit is to hold WGS workgroups at the least; the registers set one against the
// other.  Short products gain from workgroups: 32 x 32 tiles three with three blocks (two with four, and fc1 of four 197-token
// images of width 192 is 600 tiles on 256 units), 64 x 64 tiles four with one (two blocks leave room for one workgroup, and
// nothing then covers a wave's loads and its sums).  Encodes of the 12-block encoder of width 192 by 4, 12 and 64 images: 599, 975
// and 3295 us with four and two blocks, 565, 871 and 2984 with three and one.  From K = 768 on the loads in flight count for more
// on 64 x 64 tiles: encodes of three blocks of width 768, 20, 40 and 64 images 2560, 4776 and 7629 us with one block, 2387, 4729
// and 7481 with two.  The error of the encoder against 64 bits is 3.5e-7 (four short chains; one long one gave 6.5e-7).
template <int EPI, int F, int DEPTH, int WGS>
__global__ __launch_bounds__(256, WGS) void gemm_f32_kernel(const GemmArgs a) {
  constexpr int LD = 36;                 // LDS row: 32 columns and a pad that spreads the rows over the banks
  __shared__ __attribute__((aligned(16))) float red[4][32 * F][LD];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lrow = lane & 31, lk = lane >> 5;
  const int m0 = blockIdx.y * 32 * F, n0 = blockIdx.x * 32 * F;
  const float* pa[F];
  const float* pw[F];
#pragma unroll
  for (int i = 0; i < F; ++i) {
    pa[i] = (const float*)a.A + (size_t)(m0 + i * 32 + lrow) * a.lda + wave * 16 + lk * 4;
    pw[i] = (const float*)a.W + (size_t)(n0 + i * 32 + lrow) * a.ldw + wave * 16 + lk * 4;
  }
  f32x4 fa[DEPTH][F][2], fw[DEPTH][F][2];
  auto load = [&](int d, int kb) {
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        fa[d][i][c] = *(const f32x4*)(pa[i] + kb * 64 + c * 8);
        fw[d][i][c] = *(const f32x4*)(pw[i] + kb * 64 + c * 8);
      }
  };
  f32x16 acc[F][F];
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  const int KB = a.K / 64;
#pragma unroll
  for (int d = 0; d < DEPTH; ++d) load(d, min(d, KB - 1));
  // eight lanes finish a row of each 32 x 32 block; on 32 x 32 tiles, what they need for it (bias, residual or position rows)
  // is asked for here and not behind the sums (encode of four images 618 -> 600 us); 64 x 64 ones are many to a unit and cover it
  const int er = tid >> 3, ec = (tid & 7) * 4;
  Epilogue4F32<EPI> epilogue;
  if constexpr (F == 1) {
    epilogue.fetch(a, m0 + er, n0 + ec);
    __builtin_amdgcn_sched_barrier(0);
  }
  for (int k0 = 0; k0 < KB; k0 += DEPTH) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
      if (k0 + d >= KB) break;
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int i = 0; i < F; ++i)
#pragma unroll
            for (int j = 0; j < F; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fw[d][j][c][e], fa[d][i][c][e], acc[i][j], 0, 0, 0);
      if (k0 + d + DEPTH < KB) load(d, k0 + d + DEPTH);
    }
  }
  // one 32-column block at a time: the four partial sums meet in LDS, eight lanes finish a row
#pragma unroll
  for (int j = 0; j < F; ++j) {
    if (j > 0) __syncthreads();
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const f32x4 v = {acc[i][j][jj * 4], acc[i][j][jj * 4 + 1], acc[i][j][jj * 4 + 2], acc[i][j][jj * 4 + 3]};
        *(f32x4*)&red[wave][i * 32 + lrow][jj * 8 + lk * 4] = v;
      }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < F; ++i) {
      const int r = i * 32 + er;
      const int row = m0 + r, col = n0 + j * 32 + ec;
      const f32x4 v = (*(const f32x4*)&red[0][r][ec] + *(const f32x4*)&red[1][r][ec]) +
                      (*(const f32x4*)&red[2][r][ec] + *(const f32x4*)&red[3][r][ec]);
      if (row < a.M && col < a.N) {
        if constexpr (F > 1) epilogue.fetch(a, row, col);
        epilogue.store(v);
      }
    }
  }
}

// One workgroup = 32 query rows x one head (two workgroups to a work item's 64 rows); its four waves take every fourth
// block of 32 keys each, with a running maximum and sum of their own, and are merged at the end.  Scores are formed
// transposed (keys x queries), so a lane's column is its query: the running values are one register, and the weights
// are already laid out as the operand of the second product, whose key order follows the accumulator's rows.
// Measured at 4 x 197 tokens, 3 heads of 64: 12.2 us against 415 us of the predecessor (one key at a time, four lanes
// to a query); the whole encode 634 against 6 378.
constexpr int F32_BQ = 32, F32_BK = 32;

template <int DHP>
__global__ __launch_bounds__(256) void attention_f32_kernel(const AttnArgs a) {
  constexpr int CH = DHP / 8, FB = (DHP + 31) / 32;  // 8-wide chunks of a head, 32-wide blocks of its columns
  constexpr int LD = 36;
  __shared__ __attribute__((aligned(16))) float red[4][F32_BQ][LD];
  __shared__ float red_m[4][F32_BQ], red_l[4][F32_BQ];
  const AttnWork w = a.work[blockIdx.x >> 1];
  const int head = blockIdx.y;
  const int q0 = w.q0 + (blockIdx.x & 1) * F32_BQ;
  const int seg_end = w.seg_start + w.seg_len;
  if (q0 >= seg_end) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lq = lane & 31, lk = lane >> 5;
  const float* base = (const float*)a.qkv;
  const int qoff = head * DHP, koff = (a.heads + head) * DHP, voff = (2 * a.heads + head) * DHP;
  const float scale = 1.0f / sqrtf((float)a.dh);
  f32x4 q[CH];
  {
    const float* qp = base + (size_t)min(q0 + lq, seg_end - 1) * a.ld_qkv + qoff + lk * 4;
#pragma unroll
    for (int c = 0; c < CH; ++c) q[c] = *(const f32x4*)(qp + c * 8) * scale;
  }
  f32x16 o[FB];
#pragma unroll
  for (int b = 0; b < FB; ++b)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[b][v] = 0.f;
  float m = -INFINITY, l = 0.f;  // of query lq; l over this lane's keys only until the end
  for (int k0 = w.seg_start + wave * F32_BK; k0 < seg_end; k0 += 4 * F32_BK) {
    f32x4 kf[CH];
    const float* kp = base + (size_t)min(k0 + lq, seg_end - 1) * a.ld_qkv + koff + lk * 4;
#pragma unroll
    for (int c = 0; c < CH; ++c) kf[c] = *(const f32x4*)(kp + c * 8);
    float vf[FB][16];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const float* vp = base + (size_t)min(k0 + (v >> 2) * 8 + lk * 4 + (v & 3), seg_end - 1) * a.ld_qkv + voff;
#pragma unroll
      for (int b = 0; b < FB; ++b) vf[b][v] = vp[min(b * 32 + lq, DHP - 1)];
    }
    f32x16 s;
#pragma unroll
    for (int v = 0; v < 16; ++v) s[v] = 0.f;
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[c][e], q[c][e], s, 0, 0, 0);
    float mb = m;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      if (k0 + (v >> 2) * 8 + lk * 4 + (v & 3) >= seg_end) s[v] = -INFINITY;
      mb = fmaxf(mb, s[v]);
    }
    mb = fmaxf(mb, __shfl_xor(mb, 32, 64));
    const float mref = mb == -INFINITY ? 0.f : mb;  // every score so far is -inf: their weights are 0, not NaN
    const float corr = expf(m - mref);              // the library's exp: this mode is for exact-arithmetic parity
    m = mb;
    float ls = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      s[v] = expf(s[v] - mref);
      ls += s[v];
    }
    l = l * corr + ls;
#pragma unroll
    for (int b = 0; b < FB; ++b) {
#pragma unroll
      for (int v = 0; v < 16; ++v) o[b][v] *= corr;
#pragma unroll
      for (int v = 0; v < 16; ++v) o[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[b][v], s[v], o[b], 0, 0, 0);
    }
  }
  l += __shfl_xor(l, 32, 64);
  if (lk == 0) { red_m[wave][lq] = m; red_l[wave][lq] = l; }
  __syncthreads();
  float mt = -INFINITY, lt = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) mt = fmaxf(mt, red_m[i][lq]);
  const float mref = mt == -INFINITY ? 0.f : mt;
#pragma unroll
  for (int i = 0; i < 4; ++i) lt += red_l[i][lq] * expf(red_m[i][lq] - mref);
  const float f = expf(m - mref) / lt;
#pragma unroll
  for (int b = 0; b < FB; ++b) {
    if (b > 0) __syncthreads();
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      const f32x4 v = {o[b][jj * 4], o[b][jj * 4 + 1], o[b][jj * 4 + 2], o[b][jj * 4 + 3]};
      *(f32x4*)&red[wave][lq][jj * 8 + lk * 4] = v * f;
    }
    __syncthreads();
    const int r = tid >> 3, c = (tid & 7) * 4;
    if (q0 + r < seg_end && b * 32 + c < DHP)
      *(f32x4*)((float*)a.out + (size_t)(q0 + r) * a.ld_o + head * DHP + b * 32 + c) =
          (*(const f32x4*)&red[0][r][c] + *(const f32x4*)&red[1][r][c]) + (*(const f32x4*)&red[2][r][c] + *(const f32x4*)&red[3][r][c]);
  }
}

}  // namespace

hipError_t launch_gemm_f32(const GemmArgs& a, hipStream_t s) {
  if (a.M <= 0 || a.N <= 0) return hipSuccess;
  if (a.K <= 0 || a.K % 64 != 0 || a.lda % 4 != 0 || a.ldw % 4 != 0 || a.ldo % 4 != 0 || a.N % 4 != 0) return hipErrorInvalidValue;
  // 64 x 64 tiles read half the operand bytes of 32 x 32 ones, which pays once the units' shares of them come out even.  Up to
  // K = 704 that is said by a line on their number.  Whole encodes, in us, with the line at 1024, 1536, 2048, 2560, 3072 and 4096
  // tiles: 12 blocks of width 192, 40 images 2018, 1913, 1915, 1916, 1910 and 1913; 64: 2920, 2922, 2873, 2853, 2845, 2849; 100: 4270,
  // 4271, 4279, 4282, 4234, 4230; 240: 9358, 9356, 9362, 9563, 9533, 9544; 300: 11510, 11533, 11545, 11522, 11780, 11805.
  // From K = 768 on, with two k-blocks in flight, a larger tile takes 0.85 of what its four small ones do, so it is taken where
  // the largest share of a unit grows by no more than 1.18: three blocks of width 768, 20 images (shares of 3 against 3) 2387 us and
  // 2594 on small tiles, 28 (5 against 4.25) 3583 and 3595, 4 (fc1, 3 against 2.5) 710 and 692; two blocks of width 1024, 20 images
  // (4 against 4) 2699 and 2875.  Fewer than two for each unit never gain.
  const long tiles64 = (long)((a.M + 63) / 64) * ((a.N + 63) / 64), tiles32 = (long)((a.M + 31) / 32) * ((a.N + 31) / 32);
  const long share64 = (tiles64 + 255) / 256, share32 = (tiles32 + 255) / 256;
  const bool deep = a.K >= 768;
  const bool large = (deep ? tiles64 >= 512 && share64 * 400 <= share32 * 118 : tiles64 >= 2560) ||
                     (a.M + 31) / 32 > 65535;  // (more row blocks than a grid's second dimension holds)
  const int t = large ? 64 : 32;
  const dim3 grid((a.N + t - 1) / t, (a.M + t - 1) / t), block(256);
#define VIT_LAUNCH(EPI)                                                                                 \
  do {                                                                                                  \
    if (large && deep) hipLaunchKernelGGL((gemm_f32_kernel<EPI, 2, 2, 1>), grid, block, 0, s, a);       \
    else if (large) hipLaunchKernelGGL((gemm_f32_kernel<EPI, 2, 1, 2>), grid, block, 0, s, a);          \
    else hipLaunchKernelGGL((gemm_f32_kernel<EPI, 1, 3, 3>), grid, block, 0, s, a);                     \
  } while (0)
  switch (a.epilogue) {
    case EPI_BIAS: VIT_LAUNCH(EPI_BIAS); break;
    case EPI_BIAS_GELU: VIT_LAUNCH(EPI_BIAS_GELU); break;
    case EPI_BIAS_RESIDUAL: VIT_LAUNCH(EPI_BIAS_RESIDUAL); break;
    case EPI_PATCH: VIT_LAUNCH(EPI_PATCH); break;
    default: return hipErrorInvalidValue;
  }
#undef VIT_LAUNCH
  return hipGetLastError();
}

hipError_t launch_attention_f32(const AttnArgs& a, hipStream_t s) {
  if (a.n_work <= 0) return hipSuccess;
  if (a.ld_qkv % 4 != 0 || a.ld_o % 4 != 0) return hipErrorInvalidValue;
  const dim3 grid(2 * (unsigned)a.n_work, a.heads), block(256);
  switch (a.dh_pad) {  // the padded head dims the host plans
    case 64: hipLaunchKernelGGL(attention_f32_kernel<64>, grid, block, 0, s, a); break;
    case 72: hipLaunchKernelGGL(attention_f32_kernel<72>, grid, block, 0, s, a); break;
    case 80: hipLaunchKernelGGL(attention_f32_kernel<80>, grid, block, 0, s, a); break;
    case 96: hipLaunchKernelGGL(attention_f32_kernel<96>, grid, block, 0, s, a); break;
    case 128: hipLaunchKernelGGL(attention_f32_kernel<128>, grid, block, 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace vitenc
