// Image preprocessing on the GPU (paper Sec. 2, "Image Preprocessing": resize, rescale, normalise,
// segment into tiles): one 8-bit interleaved image in, the encoder's fp32 [tile, C, S, S] pixels out.
// Bound by HBM: C bytes read per source pixel (the four taps of neighbouring outputs share cache
// lines), 4C bytes written per output pixel.
#include "../../include/vitenc.h"

#include <hip/hip_runtime.h>

#include <cmath>

namespace vitenc {
vit_status_t set_error(vit_status_t st, const char* fmt, ...);  // vitenc_api.hip: message for vit_last_error()
}
using vitenc::set_error;

namespace {

struct PrepArgs {
  const unsigned char* img;
  float* out;
  int H, W, C, S, rows, cols, thumb;
  float tile_y, tile_x, thumb_y, thumb_x;  // source pixels per canvas pixel: of the tiles' canvas, of the thumbnail's
  float scale[4], shift[4];  // out = tap * scale[c] + shift[c]: 1/(255 std) and -mean/std
};

// Source taps of output coordinate o on an axis resized from n_in to n_out pixels (pixel centres at
// half-integers, coordinate clamped below at 0, last pixel repeated above).
__device__ __forceinline__ void taps(int o, float ratio, int n_in, int& i0, int& i1, float& w) {
  float src = ((float)o + 0.5f) * ratio - 0.5f;
  src = fmaxf(src, 0.f);
  i0 = min((int)src, n_in - 1);
  i1 = min(i0 + 1, n_in - 1);
  w = src - (float)i0;
}

// Canvas coordinates of the first pixel of a thread's run, and the source pixels per canvas pixel; the thumbnail (if any) is
// the last tile.
struct Place { int oy, ox; float ratio_y, ratio_x; };
__device__ __forceinline__ Place place(const PrepArgs& a, int tile, int y, int x) {
  if (tile < a.rows * a.cols) {  // a tile of the (rows*S) x (cols*S) canvas
    const int ty = tile / a.cols, tx = tile - ty * a.cols;
    return {ty * a.S + y, tx * a.S + x, a.tile_y, a.tile_x};
  }
  return {y, x, a.thumb_y, a.thumb_x};  // the whole image at S x S
}

__device__ __forceinline__ float blend(float p00, float p01, float p10, float p11, float wx, float wy, float scale, float shift) {
  const float top = p00 + (p01 - p00) * wx, bot = p10 + (p11 - p10) * wx;
  return (top + (bot - top) * wy) * scale + shift;
}

// One thread per output pixel (x fastest, so a wave writes 256 contiguous bytes per channel plane); grid.y = tile index.
// For tile sides that are no multiple of 4 and images under 8 bytes.
__global__ __launch_bounds__(256) void preprocess_kernel(const PrepArgs a) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= a.S * a.S) return;
  const int y = idx / a.S, x = idx - y * a.S;
  const int tile = blockIdx.y;
  const Place pl = place(a, tile, y, x);
  int y0, y1, x0, x1;
  float wy, wx;
  taps(pl.oy, pl.ratio_y, a.H, y0, y1, wy);
  taps(pl.ox, pl.ratio_x, a.W, x0, x1, wx);
  const unsigned char* r0 = a.img + (size_t)y0 * a.W * a.C;
  const unsigned char* r1 = a.img + (size_t)y1 * a.W * a.C;
  float* o = a.out + ((size_t)tile * a.C * a.S + y) * a.S + x;
  for (int c = 0; c < a.C; ++c)
    o[(size_t)c * a.S * a.S] = blend(r0[x0 * a.C + c], r0[x1 * a.C + c], r1[x0 * a.C + c], r1[x1 * a.C + c], wx, wy, a.scale[c], a.shift[c]);
}

// Four neighbouring output pixels per thread.  A pixel's two horizontal taps are neighbours in the interleaved image, at
// most 8 bytes together: one 8-byte load (any alignment) per pixel and row in place of 4 C single bytes, and 16-byte
// stores.  What bounds it then are vector instructions, so the taps' places in their window are constants: at the right edge,
// where the second tap is the first one again, it is the next bytes (whatever they are) with weight 0; and only a window
// that would reach past the image's last byte starts earlier and is shifted down.  An 896 x 896 image to 4 tiles of 448 and
// a thumbnail (14.5 MB moved) takes 5.6 us, launch included, on shifted taps 5.8.
template <int C>
__global__ __launch_bounds__(256) void preprocess_quad_kernel(const PrepArgs a) {
  const int idx = (blockIdx.x * 256 + threadIdx.x) * 4;
  if (idx >= a.S * a.S) return;
  // idx / S: the quotient of a float reciprocal is off by at most one below 2^22 rows
  int y = (int)((float)idx * __builtin_amdgcn_rcpf((float)a.S)), x = idx - y * a.S;
  if (x < 0) { --y; x += a.S; }
  if (x >= a.S) { ++y; x -= a.S; }
  const int tile = blockIdx.y;
  const Place pl = place(a, tile, y, x);
  int y0, y1;
  float wy;
  taps(pl.oy, pl.ratio_y, a.H, y0, y1, wy);
  const size_t last = (size_t)a.H * a.W * C - 8;  // the last place an 8-byte window may start
  const size_t row0 = (size_t)y0 * a.W * C, row1 = (size_t)y1 * a.W * C;
  uint64_t q[2][4];
  float wx[4];
  uint32_t at[4];  // byte of the first tap in its row
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    int x0, x1;
    taps(pl.ox + i, pl.ratio_x, a.W, x0, x1, wx[i]);
    if (x1 == x0) wx[i] = 0.f;
    at[i] = (uint32_t)x0 * C;
  }
  const unsigned char* const rows[2] = {a.img + row0, a.img + row1};
  if (row1 + at[3] <= last) {  // (neither the rows nor the taps of a run ever go back)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int r = 0; r < 2; ++r) __builtin_memcpy(&q[r][i], rows[r] + at[i], 8);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const size_t want = (r ? row1 : row0) + at[i], from = want < last ? want : last;
        __builtin_memcpy(&q[r][i], a.img + from, 8);
        q[r][i] >>= (want - from) * 8;
      }
  }
  float* const o = a.out + ((size_t)tile * C * a.S + y) * a.S + x;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    float4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      auto byte = [](uint64_t w, int n) { return (float)(uint8_t)((uint32_t)(n < 4 ? w : w >> 32) >> (8 * (n & 3))); };
      (&v.x)[i] = blend(byte(q[0][i], c), byte(q[0][i], C + c), byte(q[1][i], c), byte(q[1][i], C + c), wx[i], wy, a.scale[c], a.shift[c]);
    }
    *(float4*)(o + (size_t)c * a.S * a.S) = v;
  }
}

}  // namespace

extern "C" vit_status_t vit_preprocess_tiles(const uint8_t* image, int32_t height, int32_t width, int32_t channels,
                                             int32_t tile_size, int32_t grid_rows, int32_t grid_cols,
                                             int32_t thumbnail, const float* mean, const float* std_,
                                             float* out_pixels, size_t out_capacity_bytes, void* stream) {
  if (!image || !mean || !std_ || !out_pixels) return set_error(VIT_EINVAL, "vit_preprocess_tiles: NULL argument");
  if (height <= 0 || width <= 0 || channels <= 0 || channels > 4 || tile_size <= 0 || grid_rows <= 0 || grid_cols <= 0)
    return set_error(VIT_EINVAL, "vit_preprocess_tiles: sizes must be positive and channels <= 4");
  if ((int64_t)grid_rows * grid_cols + 1 > 65535 || (int64_t)tile_size * tile_size > (int64_t)1 << 30 ||
      (int64_t)height * width * channels > (int64_t)1 << 40 || (int64_t)width * channels > INT32_MAX)
    return set_error(VIT_EINVAL, "vit_preprocess_tiles: at most 65534 tiles of at most 2^30 pixels, image rows below 2^31 bytes");
  PrepArgs a;
  for (int c = 0; c < channels; ++c) {
    if (!(std_[c] > 0.f) || !std::isfinite(std_[c]) || !std::isfinite(mean[c]))
      return set_error(VIT_EINVAL, "vit_preprocess_tiles: std must be positive, mean and std finite");
    a.scale[c] = 1.0f / (255.0f * std_[c]);
    a.shift[c] = -mean[c] / std_[c];
  }
  const int n_tiles = grid_rows * grid_cols + (thumbnail ? 1 : 0);
  const size_t need = (size_t)n_tiles * channels * tile_size * tile_size * sizeof(float);
  if (out_capacity_bytes < need)
    return set_error(VIT_ECAPACITY, "vit_preprocess_tiles: out_pixels holds %zu bytes, %zu needed", out_capacity_bytes, need);
  a.img = image; a.out = out_pixels;
  a.H = height; a.W = width; a.C = channels; a.S = tile_size; a.rows = grid_rows; a.cols = grid_cols;
  a.thumb = thumbnail ? 1 : 0;
  a.tile_y = (float)height / (float)((int64_t)grid_rows * tile_size);
  a.tile_x = (float)width / (float)((int64_t)grid_cols * tile_size);
  a.thumb_y = (float)height / (float)tile_size; a.thumb_x = (float)width / (float)tile_size;
  // Rows of 4 pixels need a side that is a multiple of 4 (a run then lies in one row, 16-byte aligned in every plane if the
  // buffer is); everything else takes the general kernel.
  const bool quad = tile_size % 4 == 0 && ((uintptr_t)out_pixels & 15) == 0 && (int64_t)height * width * channels >= 8;
  const int64_t threads = (int64_t)tile_size * tile_size / (quad ? 4 : 1);
  const dim3 grid((unsigned)((threads + 255) / 256), (unsigned)n_tiles), block(256);
  hipStream_t s = (hipStream_t)stream;
  if (!quad) hipLaunchKernelGGL(preprocess_kernel, grid, block, 0, s, a);
  else if (channels == 1) hipLaunchKernelGGL(preprocess_quad_kernel<1>, grid, block, 0, s, a);
  else if (channels == 2) hipLaunchKernelGGL(preprocess_quad_kernel<2>, grid, block, 0, s, a);
  else if (channels == 3) hipLaunchKernelGGL(preprocess_quad_kernel<3>, grid, block, 0, s, a);
  else hipLaunchKernelGGL(preprocess_quad_kernel<4>, grid, block, 0, s, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return set_error(VIT_EDEVICE, "vit_preprocess_tiles: launch: %s", hipGetErrorString(e));
  return VIT_OK;
}
