// fp32 convolution as an implicit GEMM on the matrix cores
// (v_mfma_f32_32x32x2_f32), operands fed to LDS by direct loads.
//
// Bound: the fp32 matrix rate (154 TFLOP/s in a large product on this card),
// 64 FLOP per SIMD and clock, so a 32x32x32 step holds a SIMD for 1024
// cycles; operand traffic is small beside that (32 bytes per clock and CU at
// the smallest tile).  What cost the kernel before this one its time was the
// staging through registers (a full wait for global memory at every barrier),
// 4-byte LDS reads, and too few tiles: 64x32 tiles leave 336 workgroups for
// the 7x7x512 layers at eight images, 1.3 rounds on 256 CUs.
//
// LDS rows are 32 floats of one pixel or one output channel (128 bytes, eight
// 16-byte chunks, swizzled like the bf16 kernels').  A chunk of the input is
// four channels of one filter tap, so the tap is a per-lane quantity and any
// Cin that is a multiple of 4 fits (the first layer's three channels are
// padded to four).  An operand read takes 16 bytes, four K values, per lane:
// the k-th MFMA of a group multiplies the k-th of them in both operands, so
// one read serves four MFMAs.  Per output the sum runs over the K-tiles in
// order, inside a tile over e = 0..3 for each 8-wide group.
//
// G = WM x WN waves share a tile ring and meet once per K-tile; KS such groups
// split the reduction (contiguous runs of K-tiles), their sums added through
// LDS in group order, so that layers with few tiles still fill the chip.  With
// G = 1 a wave's ring is its own and the loop has no barrier.  Every group
// runs the same number of steps and every step issues the same loads (past
// the end: out of range, zeros), so waits are constants.
#include "common.hpp"
#include "device.hpp"
#include "lds_dma.hpp"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace fs {

namespace {

constexpr int F32_BK = 32;            // floats per K-tile row (128 bytes)
constexpr int F32_BLK = 1024 + 64;    // LDS bytes of a 4-channel group column of a 32x32 partial block (padded)

// One direct load: 64 lanes x 16 bytes from base + voff + soff to lds.
__device__ __forceinline__ void load16_lds(const void* base, uint32_t bytes, char* lds, uint32_t voff, int soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc(base, bytes), (lds_void*)lds, 16, voff, soff, 0, 0);
}

// UNI: Cin is a multiple of 32, so a K-tile lies in one filter tap: the tap and
// the channel are scalars that the loads take as their scalar offset, and a
// lane's own part (is the tap inside the image?) changes with the tap only.
// The fp32 MFMAs run on the same units as ordinary vector instructions, which
// therefore take their time from them, whichever wave issues them: with the tap
// worked out per lane and K-tile (75 vector instructions to 16 MFMAs) the
// matrix rate stopped at 100 TFLOP/s on every tile shape.
//
// WIDE: a filter of 2^24 values, or one that spans 2^23 pixels, which the 24-bit
// products and fdiv_small of the general form do not cover.
enum { F32_GEN, F32_UNI, F32_WIDE };
template <int FM, int FN, int WM, int WN, int KS, int STAGES, int FORM>
__global__ void __launch_bounds__(64 * WM * WN * KS) k_conv_f32(ConvArgs a) {
  constexpr bool UNI = FORM == F32_UNI;
  constexpr int G = WM * WN, NW = G * KS;
  constexpr int BM = 32 * FM * WM, BN = 32 * FN * WN;
  constexpr int AP = BM / 8 / G, BP = BN / 8 / G, LPT = AP + BP;  // load instructions per wave and K-tile
  static_assert(AP * 8 * G == BM && BP * 8 * G == BN && STAGES >= 2, "tile");
  constexpr int STAGE = (BM + BN) * ROW, RING = STAGES * STAGE;
  constexpr int RED = KS > 1 ? NW * FM * FN * 4 * F32_BLK : 0;
  constexpr int SMEM = KS * RING > RED ? KS * RING : RED;
  __shared__ __attribute__((aligned(1024))) char smem[SMEM];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ks = wave / G, wg = wave - ks * G, wm = wg / WN, wn = wg - wm * WN;
  const int lr = lane >> 3, fr = lane & 31, fq = lane >> 5;
  char* const ring = smem + ks * RING;

  const int tiles_m = (a.M + BM - 1) / BM, tiles_n = (a.Cout + BN - 1) / BN;
  const int id = xcd_remap(blockIdx.x, tiles_m * tiles_n * a.Z);
  const int z = id / (tiles_m * tiles_n), t = id - z * (tiles_m * tiles_n);
  const int mt = t / tiles_n, m0 = mt * BM, n0 = (t - mt * tiles_n) * BN;

  // UNI: the input seen from `shift` bytes before its start, so that the
  // offset of a pixel's top-left tap is never negative (a tap outside the
  // image is out of range by a select, not by its address)
  const uint32_t shift = UNI ? (uint32_t)(a.pad * (a.W + 1) * a.Cin * 4) : 0u;
  const char* const xbase = reinterpret_cast<const char*>(reinterpret_cast<const float*>(a.x) + z * a.x_mstride) - shift;
  const uint32_t xbytes = (uint32_t)((int64_t)a.B * a.H * a.W * a.Cin * 4) + shift;
  const float* const wbase = reinterpret_cast<const float*>(a.w) + z * a.w_mstride;
  const uint32_t wbytes = (uint32_t)((int64_t)a.Cout * a.Kp * 4);

  // ---- this lane's rows: load instruction i fills rows 8 (i G + wg) .. +8 of
  // the tile; chunk (lane & 7) of a row holds logical chunk (lane & 7) ^ swz(row)
  const int HoWo = a.Ho * a.Wo;
  const bool small_m = a.M < (1 << 22) - 4096;
  const float inv_howo = 1.0f / (float)HoWo, inv_wo = 1.0f / (float)a.Wo;
  int a_off[AP], a_iy[AP], a_ix[AP];  // a_off: bytes (UNI: with this lane's chunk and the shift) or elements
#pragma unroll
  for (int i = 0; i < AP; ++i) {
    const int blk = i * G + wg, m = m0 + blk * 8 + lr;
    const int b = small_m ? fdiv_small(m, inv_howo) : m / HoWo, r = m - b * HoWo;
    const int oy = small_m ? fdiv_small(r, inv_wo) : r / a.Wo, ox = r - oy * a.Wo;
    a_iy[i] = m < a.M ? oy * a.stride - a.pad : -(1 << 28);
    a_ix[i] = ox * a.stride - a.pad;
    a_off[i] = ((b * a.H + oy * a.stride - a.pad) * a.W + a_ix[i]) * a.Cin;
    if (UNI) a_off[i] = a_off[i] * 4 + (int)shift + (((lane & 7) ^ lr ^ (blk & 1)) << 4);
  }
  uint32_t b_off[BP];
#pragma unroll
  for (int i = 0; i < BP; ++i) {
    const int blk = i * G + wg, n = n0 + blk * 8 + lr;
    b_off[i] = n < a.Cout ? (uint32_t)(((int64_t)n * a.Kp + (((lane & 7) ^ lr ^ (blk & 1)) << 2)) * 4) : OOB;
  }

  // K-tiles of this group; every group runs n_steps
  const int nk = (a.K + F32_BK - 1) / F32_BK, n_steps = (nk + KS - 1) / KS;
  int u = ks * n_steps;                                  // the next one to load
  const int u_end = min(nk, u + n_steps);
  // UNI: its tap and channel
  int ky = 0, kx = 0, ci = 0;
  uint32_t a_cur[AP];
  auto set_tap = [&]() {
#pragma unroll
    for (int i = 0; i < AP; ++i) {
      const bool ok = (unsigned)(a_iy[i] + ky) < (unsigned)a.H && (unsigned)(a_ix[i] + kx) < (unsigned)a.W;
      a_cur[i] = ok ? (uint32_t)a_off[i] : OOB;
    }
  };
  if constexpr (UNI) {
    const int k0 = u * F32_BK, tap = __builtin_amdgcn_readfirstlane(k0 / a.Cin);
    ci = k0 - tap * a.Cin;
    ky = __builtin_amdgcn_readfirstlane(tap / a.kw);
    kx = tap - ky * a.kw;
    set_tap();
  }
  const int cpt = a.Cin >> 2, taps = a.kh * a.kw;  // 16-byte chunks per tap
  const float inv_cpt = 1.0f / (float)cpt, inv_kw = 1.0f / (float)a.kw;
  auto issue = [&](char* base) {
    // past the group's end: empty buffers, zeros
    const bool live = u < u_end;  // wave-uniform
    const uint32_t xb = live ? xbytes : 0u, wb = live ? wbytes : 0u;
    if constexpr (UNI) {
      const int soff = __builtin_amdgcn_readfirstlane(((ky * a.W + kx) * a.Cin + ci) * 4);
#pragma unroll
      for (int i = 0; i < AP; ++i)
        load16_lds(xbase, xb, base + (i * G + wg) * 1024, a_cur[i], soff);
    } else {
      // input offset of this lane's chunk for rows of even and of odd blocks
      int dy[2], dx[2], dof[2];
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const int gch = u * 8 + ((lane & 7) ^ lr ^ p);
        int tap, ty, tx;
        if constexpr (FORM == F32_WIDE) {
          tap = gch / cpt;
          ty = tap / a.kw;
          tx = tap - ty * a.kw;
          dof[p] = (int)(((uint32_t)ty * a.W + tx) * a.Cin + ((gch - tap * cpt) << 2));
        } else {
          tap = fdiv_small(gch, inv_cpt);
          ty = fdiv_small(tap, inv_kw);
          tx = tap - __mul24(ty, a.kw);
          dof[p] = __mul24(__mul24(ty, a.W) + tx, a.Cin) + ((gch - __mul24(tap, cpt)) << 2);
        }
        dy[p] = tap < taps ? ty : -(1 << 28);  // past the filter: outside the image
        dx[p] = tx;
      }
#pragma unroll
      for (int i = 0; i < AP; ++i) {
        const int p = G % 2 ? i & 1 : wg & 1;
        const bool ok = (unsigned)(a_iy[i] + dy[p]) < (unsigned)a.H && (unsigned)(a_ix[i] + dx[p]) < (unsigned)a.W;
        const uint32_t keep = 0u - (uint32_t)ok;
        const uint32_t off = ((uint32_t)(a_off[i] + dof[p]) * 4u & keep) | (OOB & ~keep);
        load16_lds(xbase, xb, base + (i * G + wg) * 1024, off, 0);
      }
    }
#pragma unroll
    for (int i = 0; i < BP; ++i)
      load16_lds(wbase, wb, base + BM * ROW + (i * G + wg) * 1024, b_off[i],
                 __builtin_amdgcn_readfirstlane(live ? u * (F32_BK * 4) : 0));
    ++u;
    if constexpr (UNI) {
      ci += F32_BK;
      if (ci == a.Cin) {  // wave-uniform
        ci = 0;
        if (++kx == a.kw) {
          kx = 0;
          ++ky;
        }
        set_tap();
      }
    }
  };

  floatx16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  // operand addresses of the four 8-wide groups of a K-tile, in stage 0
  const int sw = swz(fr);  // 32-row blocks repeat the swizzle
  const char *As[4], *Bs[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int c = ((2 * s + fq) ^ sw) << 4;
    As[s] = ring + (wm * FM * 32 + fr) * ROW + c;
    Bs[s] = ring + (BM + wn * FN * 32 + fr) * ROW + c;
  }
  auto compute = [&](auto stc) {
    constexpr int o = decltype(stc)::value * STAGE;
    floatx4 av[4][FM], bv[4][FN];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
#pragma unroll
      for (int i = 0; i < FM; ++i) av[s][i] = *reinterpret_cast<const floatx4*>(As[s] + o + i * 32 * ROW);
#pragma unroll
      for (int j = 0; j < FN; ++j) bv[s][j] = *reinterpret_cast<const floatx4*>(Bs[s] + o + j * 32 * ROW);
    }
    __builtin_amdgcn_sched_barrier(0);  // the reads first, or the compiler puts each before its MFMAs with a wait
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(bv[s][j][e], av[s][i][e], acc[i][j], 0, 0, 0);
  };

#pragma unroll
  for (int s = 0; s < STAGES - 1; ++s) issue(ring + s * STAGE);
  for (int i = 0; i < n_steps; i += STAGES)
    static_for<0, STAGES>([&](auto sc) {  // the ring's positions by name
      constexpr int s = decltype(sc)::value;
      if (i + s < n_steps) {
        wait_vmcnt<(STAGES - 2) * LPT>();
        if constexpr (G > 1) {
          wait_lgkm0();  // this wave's operand reads of the stage that is filled next
          wg_barrier();
        }
        issue(ring + (s + STAGES - 1) % STAGES * STAGE);
        compute(sc);
      }
    });

  // ---- bias, residual, ReLU.  D[n][m]: lane l holds pixel l % 32 and channels
  // 8 g + 4 (l / 32) + r: four consecutive ones, one 16-byte store per g.  With
  // one group, pieces outside the layer read zeros and store nothing instead of
  // being skipped, so that a lane's loads are all in flight together.
  const uint32_t obytes = (uint32_t)((int64_t)a.M * a.Cout * 4);
  const bool has_res = a.res != nullptr;
  const float* __restrict__ bias = a.bias + z * a.b_mstride;
  const __amdgpu_buffer_rsrc_t rb = rsrc(bias, (uint32_t)a.Cout * 4u);
  const __amdgpu_buffer_rsrc_t rres =
      has_res ? rsrc(reinterpret_cast<const float*>(a.res) + z * a.res_mstride, obytes) : rsrc(a.y, 0u);
  const __amdgpu_buffer_rsrc_t ry = rsrc(reinterpret_cast<float*>(a.y) + z * a.y_mstride, obytes);
  auto load4 = [&](const __amdgpu_buffer_rsrc_t& r, uint32_t o) {
    return __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(r, o, 0, 0));
  };
  auto out_off = [&](int m, int n) {
    return m < a.M && n < a.Cout ? (uint32_t)(((int64_t)m * a.Cout + n) * 4) : OOB;
  };
  auto finish = [&](floatx4 v, floatx4 b, floatx4 r, uint32_t o) {
    v += b;
    if (has_res) v += r;
    if (a.relu)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = v[e] > 0.f ? v[e] : 0.f;
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, v), ry, o, 0, 0);
  };
  if constexpr (KS == 1) {
    uint32_t o[FM][FN][4];
    floatx4 bv[FN][4], rv[FM][FN][4];
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int gg = 0; gg < 4; ++gg) {
        const int n = n0 + (wn * FN + j) * 32 + 8 * gg + 4 * fq;
        bv[j][gg] = load4(rb, (uint32_t)n * 4u);
#pragma unroll
        for (int i = 0; i < FM; ++i) {
          o[i][j][gg] = out_off(m0 + (wm * FM + i) * 32 + fr, n);
          rv[i][j][gg] = has_res ? load4(rres, o[i][j][gg]) : floatx4{0.f, 0.f, 0.f, 0.f};
        }
      }
    wait_vmcnt<0>();  // also the out-of-range loads past the last tile, before the workgroup leaves its LDS
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int gg = 0; gg < 4; ++gg)
          finish(floatx4{acc[i][j][gg * 4], acc[i][j][gg * 4 + 1], acc[i][j][gg * 4 + 2], acc[i][j][gg * 4 + 3]},
                 bv[j][gg], rv[i][j][gg], o[i][j][gg]);
  } else {
    static_assert(KS == 1 || G == 1, "split groups are single waves");
    wait_vmcnt<0>();  // the out-of-range loads past the last tile land before the LDS is reused
    wg_barrier();
    constexpr int WAVE = FM * FN * 4 * F32_BLK;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int gg = 0; gg < 4; ++gg)
          *reinterpret_cast<floatx4*>(smem + wave * WAVE + ((i * FN + j) * 4 + gg) * F32_BLK + lane * 16) =
              floatx4{acc[i][j][gg * 4], acc[i][j][gg * 4 + 1], acc[i][j][gg * 4 + 2], acc[i][j][gg * 4 + 3]};
    wait_lgkm0();
    wg_barrier();
    // one item = one pixel x 4 channels; eight consecutive items are a pixel's 32 channels
    for (int it = tid; it < FM * FN * 256; it += 64 * NW) {
      const int blk = it >> 8, px = (it >> 3) & 31, c4 = it & 7;
      const int m = m0 + (blk / FN) * 32 + px, n = n0 + (blk % FN) * 32 + c4 * 4;
      if (m >= a.M || n >= a.Cout) continue;
      const char* src = smem + (blk * 4 + (c4 >> 1)) * F32_BLK + ((c4 & 1) * 32 + px) * 16;
      floatx4 v = *reinterpret_cast<const floatx4*>(src);
#pragma unroll
      for (int k = 1; k < KS; ++k) v += *reinterpret_cast<const floatx4*>(src + k * WAVE);
      const uint32_t o = out_off(m, n);
      finish(v, *reinterpret_cast<const floatx4*>(bias + n), has_res ? load4(rres, o) : floatx4{0.f, 0.f, 0.f, 0.f}, o);
    }
  }
}

}  // namespace

bool conv_f32_ok(const ConvArgs& a) {
  return !a.x2 && a.split == 1 && a.Cin % 4 == 0 && a.Cout % 8 == 0 && a.Kp % F32_BK == 0;
}

void launch_conv_f32(const ConvArgs& a, int bm, int bn, int ks, hipStream_t s) {
  const int tiles = ((a.M + bm - 1) / bm) * ((a.Cout + bn - 1) / bn) * a.Z;
  const bool uni = a.Cin % F32_BK == 0 &&
                   ((int64_t)a.B * a.H * a.W + a.pad * (a.W + 1)) * a.Cin * 4 < (1ll << 31);
  const bool wide = (int64_t)a.kh * a.kw * a.Cin / 4 + 64 >= (1 << 22) || (int64_t)a.kh * a.W + a.kw >= (1 << 23);
#define FS_FORM(FMv, FNv, WMv, WNv, KSv, Sv, FORMv)                                                            \
  hipLaunchKernelGGL((k_conv_f32<FMv, FNv, WMv, WNv, KSv, Sv, FORMv>), dim3(tiles), dim3(64 * WMv * WNv * KSv), \
                     0, s, a)
#define FS_F32(FMv, FNv, WMv, WNv, KSv, Sv)                                         \
  if (bm == 32 * FMv * WMv && bn == 32 * FNv * WNv && ks == KSv) {                  \
    if (uni)                                                                        \
      FS_FORM(FMv, FNv, WMv, WNv, KSv, Sv, F32_UNI);                                \
    else if (wide)                                                                  \
      FS_FORM(FMv, FNv, WMv, WNv, KSv, Sv, F32_WIDE);                               \
    else                                                                            \
      FS_FORM(FMv, FNv, WMv, WNv, KSv, Sv, F32_GEN);                                \
    return;                                                                         \
  }
  FS_F32(1, 1, 2, 2, 1, 3) FS_F32(1, 1, 1, 1, 4, 2) FS_F32(1, 1, 1, 1, 8, 2) FS_F32(1, 1, 2, 1, 1, 2) FS_F32(1, 1, 4, 1, 1, 2)
#undef FS_F32
#undef FS_FORM
}

// The tile of a layer: 64x64 (0), 32x32 with the reduction over four (1) or
// eight waves (2), or, for layers whose channels would leave 64 columns half
// empty, 64x32 (3) and 128x32 (4) with the waves along the pixels.  Time in us of
// a layer on each: a + b q + (c q + d) ceil(n) + f n, with q K-tiles per wave and
// n workgroups per CU (at least one); coefficients fitted (non-negative, least
// squares of the relative error, 3 to 7 % rms) to back-to-back launches of every
// tile on 283 layers: 3 to 256 channels in, 8 to 256 out, 1x1 to 5x5, maps of 4 to
// 56, B = 1 to 64, one to three models.  The tile it names is 0.6 % slower than the
// fastest of the five on average and 9 % at most.  Without the narrow tiles
// layers of few channels lost up to half their speed to empty columns: 3x3,
// 3 -> 16 on 32x32, B = 64, three models, 24.7 us on 64x64 against 14.7 on 128x32;
// 1x1, 64 -> 24 on 32x32, B = 64, two models, 17.7 against 11.0.  With channels to
// fill them wider tiles win: 56x56x64, B = 8, three models, 53.7 on 64x64 against
// 78 on 32x32 over four waves; 14x14x256 77 against 56.2; one image, 7x7x512 82.6
// against 25.4 over four and 22.3 over eight.  Shape and batch decide alone (the
// 256 CUs are the chip's), so a result's bits never depend on timing.
struct F32Cost {
  int bm, bn, ks;
  double a, b, c, d, f;
};
static const F32Cost kF32Cost[] = {
    {64, 64, 1, 2.30, 0.13, 0.45, 1.15, 0.},      {32, 32, 4, 1.97, 0.12, 0.51, 0.48, 0.71},
    {32, 32, 8, 1.10, 0.01, 1.00, 2.57, 0.05},    {64, 32, 1, 2.76, 0.37, 0.24, 0.57, 0.},
    {128, 32, 1, 2.26, 0.21, 0.45, 1.10, 0.},
};

int conv_f32_tile(const ConvArgs& a) {
  const int nk = (a.K + F32_BK - 1) / F32_BK;
  int best = 0;
  double best_us = 1e300;
  for (int i = 0; i < (int)(sizeof(kF32Cost) / sizeof(F32Cost)); ++i) {
    const F32Cost& t = kF32Cost[i];
    const double tiles = (double)((a.M + t.bm - 1) / t.bm) * ((a.Cout + t.bn - 1) / t.bn) * a.Z;
    const double n = std::max(1.0, tiles / 256), q = (nk + t.ks - 1) / t.ks;
    const double us = t.a + t.b * q + (t.c * q + t.d) * std::ceil(n) + t.f * n;
    if (us < best_us) {
      best_us = us;
      best = i;
    }
  }
  return best;
}

}  // namespace fs
