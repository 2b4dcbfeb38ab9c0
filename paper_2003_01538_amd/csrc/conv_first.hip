// The first layer of a VGG-type network and its max pool in one kernel:
// 3x3 / 1 / p1 convolution of the transformed image (3 channels stored as 4)
// to 64 channels, bias, ReLU, then 2x2 / 2 max pool; only the pooled tensor
// is written.
//
// The two layers are bound by memory: at 224 x 224 the unpooled tensor is 16
// times the input and four times the pooled one, and was written and read
// again (B = 32: 411 MB of the 475 MB that both launches moved).  The
// reduction has 36 terms, so one 32x32x16 step covers four filter taps and
// three steps the filter; the weights (six fragments) stay in registers.
//
// A lane owns one pooling window, whose four conv pixels read a 4x4 patch of
// the image: its operand for patch row r is that row's four pixels (two per
// half wave, two 8-byte loads straight from the image), loaded once for all
// four conv pixels.  Each of these takes three of the four rows, with weight
// fragments whose columns are shifted by the pixel's dx (zero where the
// filter does not reach): 24 MFMAs for 128 conv pixels, as many as with
// operands gathered per conv pixel, for a fifth of the loads.  The max over
// the window is then a max over accumulators.  It commutes with the rounding
// (both are monotone), so the result is that of the two layers up to the order
// of the 36 terms of a sum.
//
// VGG-11's first layer, 32 images of 224 x 224: 31 us (2 TB/s) against 124 +
// 43 us in two launches, each measured alone with events around it.  Bound
// by the latency of the patch loads: two waves a SIMD, one run ahead.
#include "common.hpp"
#include "device.hpp"
#include "lds_dma.hpp"

#include <algorithm>

namespace fs {

namespace {

typedef unsigned int v2u __attribute__((ext_vector_type(2)));

constexpr uint32_t COL_OOB = 0x40000000u;  // added to a row's offset: past every image, whose bytes are below 2^29

// A wave takes a run of 32 windows, then the one `waves` runs further on.
__global__ void __launch_bounds__(256, 2) k_conv_first_pool(ConvArgs a, int waves) {
  const int lane = threadIdx.x & 63, fq = lane >> 5;
  const int wave = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int Hp = a.H / 2, Wp = a.W / 2, total = a.B * Hp * Wp;
  const int z = blockIdx.y;

  const __amdgpu_buffer_rsrc_t rx =
      rsrc(reinterpret_cast<const uint16_t*>(a.x) + z * a.x_mstride, (uint32_t)((int64_t)a.B * a.H * a.W * 8));
  const __amdgpu_buffer_rsrc_t ry =
      rsrc(reinterpret_cast<const uint16_t*>(a.y) + z * a.y_mstride, (uint32_t)((int64_t)total * 128));
  const uint16_t* __restrict__ w = reinterpret_cast<const uint16_t*>(a.w) + z * a.w_mstride;

  // weight fragments (filter row ky, shift dx, block j): channel 32 j +
  // (lane & 31), patch columns 2 fq and 2 fq + 1, so filter columns kx - dx
  bf16x8 wf[3][2][2];
#pragma unroll
  for (int ky = 0; ky < 3; ++ky)
#pragma unroll
    for (int dx = 0; dx < 2; ++dx)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        v2u h[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int kx = 2 * fq + i - dx;
          h[i] = v2u{0, 0};
          if ((unsigned)kx < 3u)
            h[i] = *reinterpret_cast<const v2u*>(w + (j * 32 + (lane & 31)) * a.Kp + (ky * 3 + kx) * 4);
        }
        wf[ky][dx][j] = __builtin_bit_cast(bf16x8, v4u{h[0][0], h[0][1], h[1][0], h[1][1]});
      }
  floatx4 bias[2][4];  // of the channels this lane accumulates
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      bias[j][g] = *reinterpret_cast<const floatx4*>(a.bias + z * a.b_mstride + j * 32 + 8 * g + 4 * fq);

  // this lane's window: pooled row `row` (over all images), `py` in its image, column px
  const int step = waves * 32, step_px = step % Wp, step_row = step / Wp, step_py = step_row % Hp;
  int t = wave * 32 + (lane & 31);
  int row = t / Wp, px = t - row * Wp, py = row % Hp;

  auto load = [&](v2u (&v)[4][2]) {  // patch row r, columns 2 fq and 2 fq + 1
    const int x = 2 * px - 1 + 2 * fq;
    const uint32_t c0 = x >= 0 ? (uint32_t)(x * 8) : COL_OOB, c1 = x + 1 < a.W ? (uint32_t)(x * 8 + 8) : COL_OOB;
    const bool in = t < total;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const bool ok = in && (r > 0 || py > 0) && (r < 3 || py < Hp - 1);
      const uint32_t ro = ok ? (uint32_t)((2 * row + r - 1) * a.W * 8) : OOB;
      v[r][0] = __builtin_bit_cast(v2u, __builtin_amdgcn_raw_buffer_load_b64(rx, ro + c0, 0, 0));
      v[r][1] = __builtin_bit_cast(v2u, __builtin_amdgcn_raw_buffer_load_b64(rx, ro + c1, 0, 0));
    }
  };
  const uint32_t low = fq ? 0u : ~0u;  // columns 0 and 1 of the patch
  v2u cur[4][2], nxt[4][2];
  load(cur);
  for (int t0 = wave * 32; t0 < total; t0 += step) {
    const uint32_t yo = t < total ? (uint32_t)((t * 64 + 8 * fq) * 2) : OOB;
    t += step;
    px += step_px;
    row += step_row;
    py += step_py;
    if (px >= Wp) {
      px -= Wp;
      ++row;
      ++py;
    }
    if (py >= Hp) py -= Hp;
    load(nxt);  // past the last window: nothing is read
    // the column that the pixels of shift dx do not read is cleared: it meets
    // a zero weight, but zero times a pixel that is not finite is not zero
    bf16x8 f[2][4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      f[0][r] = __builtin_bit_cast(bf16x8, v4u{cur[r][0][0], cur[r][0][1], cur[r][1][0] & low, cur[r][1][1] & low});
      f[1][r] = __builtin_bit_cast(bf16x8, v4u{cur[r][0][0] & ~low, cur[r][0][1] & ~low, cur[r][1][0], cur[r][1][1]});
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      floatx16 acc[2][2];
#pragma unroll
      for (int dy = 0; dy < 2; ++dy)
#pragma unroll
        for (int dx = 0; dx < 2; ++dx) {
#pragma unroll
          for (int e = 0; e < 16; ++e) acc[dy][dx][e] = 0.f;
#pragma unroll
          for (int ky = 0; ky < 3; ++ky)
            acc[dy][dx] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[ky][dx][j], f[dx][dy + ky], acc[dy][dx], 0, 0, 0);
        }
      float v[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const float b = bias[j][e >> 2][e & 3];
        v[e] = fmaxf(fmaxf(fmaxf(fmaxf(acc[0][0][e] + b, acc[0][1][e] + b), acc[1][0][e] + b), acc[1][1][e] + b), 0.f);
      }
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        float o[8];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[g * 8 + r]), __float_as_uint(v[g * 8 + 4 + r]),
                                                           false, false);
          o[r] = __uint_as_float(sw[0]);
          o[4 + r] = __uint_as_float(sw[1]);
        }
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, f8_to_bf8(o)), ry, yo + j * 64 + g * 32, 0, 0);
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      cur[r][0] = nxt[r][0];
      cur[r][1] = nxt[r][1];
    }
  }
}

}  // namespace

bool conv_first_pool_ok(const ConvArgs& a) {
  return a.Cin == 4 && a.kh == 3 && a.kw == 3 && a.stride == 1 && a.pad == 1 && a.relu && !a.res && !a.x2 &&
         a.Cout == 64 && a.Kp >= 36 && a.H % 2 == 0 && a.W % 2 == 0 &&
         (int64_t)a.B * a.H * a.W * 32 < (int64_t(1) << 31);
}

// Two waves a SIMD (the fragments, a block's accumulators and two patches
// fill their registers), each with the same number of runs.
void launch_conv_first_pool(const ConvArgs& a, int num_cus, hipStream_t s) {
  const int runs = (a.B * (a.H / 2) * (a.W / 2) + 31) / 32;
  const int per = (runs * a.Z + num_cus * 8 - 1) / (num_cus * 8);
  const int blocks = ((runs + per - 1) / per + 3) / 4;
  hipLaunchKernelGGL(k_conv_first_pool, dim3(blocks, a.Z), dim3(256), 0, s, a, blocks * 4);
}

}  // namespace fs
