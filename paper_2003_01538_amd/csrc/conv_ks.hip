// Convolution for layers with few output tiles (small batches, late layers),
// bf16: the waves of a workgroup split the REDUCTION of one output tile.
//
// At a small batch the other bf16 kernels give each workgroup a whole
// reduction: the 7x7x512 3x3 layer at one image is 12 workgroups of 72
// K-tiles, one after the other, and takes 33 us at any batch up to 32, the
// latency of 72 dependent fetches.  Here a workgroup owns a tile of 32 FM
// output pixels x 32 NB channels and its KS x NB waves each run a contiguous
// KS-th of the K-tiles, with their fp32 sums added through LDS in wave order
// at the end.  The serial chain is KS times shorter, no partial sum leaves
// the CU, and no second launch finishes it.
//
// Input: all channels of the input pixels that the tile reads are staged in
// LDS once, by direct loads, with one barrier; the waves then run without
// meeting until the end.  For a 3x3 filter those pixels are ONE run of the
// flattened [B*H*W] pixel index, from the first output's top-left tap to the
// last output's bottom-right one (a run of BM + 2W + 2 for stride 1): each
// LDS row is one pixel's 64-channel chunk (128 bytes), there are no padding
// rows, and a tap outside the image reads a row of zeros instead.  For
// stride 2 the run's even pixels come first, then the odd ones, so that
// consecutive outputs still read consecutive rows (the swizzle's condition
// for conflict-free operand reads).  For a 1x1 filter, and for a projection
// shortcut's input, the rows are the tile's own pixels.
//
// Weights: each wave streams its own K-tiles straight into registers, RING
// K-tiles ahead, from the fragment-ordered copy (one 1 KB load per k16
// step); where only packed rows exist (the allocation-free entry point) it
// loads 8 rows x 128 bytes per instruction and turns them through 4 KB of LDS
// that belong to the wave alone, or reads 32 rows as they lie where there is
// no LDS left.  The operand values, the K order within a wave and the order of
// the waves' sums are the same on every route, so the bits are.
#include "common.hpp"
#include "device.hpp"
#include "lds_dma.hpp"

#include <algorithm>
#include <cmath>

namespace fs {

namespace {

constexpr int KS_BLK = 1024 + 64;  // LDS bytes of one 8-channel group of a 32x32 partial block (padded: 16-byte reads of 4 groups x 4 pixels hit distinct banks)

constexpr int KS_WAVES = 8; // waves of a workgroup: KS along the reduction x NB along the channels
constexpr int KS_PASS = 2;   // 32-pixel blocks whose partial sums are in LDS at a time

struct KsGeom {
  int rows;   // LDS rows per 64-channel chunk of the main input (multiple of 8)
  int half;   // stride 2: rows of even pixels (the odd ones follow)
  int off2;   // LDS byte offset of the projection shortcut's rows
  int zero;   // ... of the row of zeros
  int wbuf;   // ... of the waves' weight buffers (4 KB each; packed-row weights only)
  int mt, nt; // tiles along M and N
};

extern __shared__ __attribute__((aligned(1024))) char ks_smem[];

// WT: where the weights come from: the fragment-ordered copy, packed rows turned
// through LDS, or packed rows read as they lie (32 rows per load, slower, where
// the input leaves no LDS to turn them).
enum { W_FRAG, W_TURN, W_ROWS };

template <int FM, int KS, int NB, int RING, int WPS, int WT>
__global__ void __launch_bounds__(64 * KS * NB, WPS) k_conv_ks(ConvArgs a, KsGeom g) {
  static_assert(KS * NB == KS_WAVES, "waves");
  constexpr int NW = KS_WAVES, BM = 32 * FM, BN = 32 * NB;
  char* const sm = ks_smem;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ks = wave / NB, nb = wave - ks * NB;
  const int lr = lane >> 3, fr = lane & 31, fq = lane >> 5;

  // M tiles fastest, XCD-contiguous: an XCD's workgroups share few weights
  const int id = xcd_remap(blockIdx.x, g.mt * g.nt * a.Z);
  const int mt = id % g.mt, nz = id / g.mt;
  const int z = nz / g.nt, n0 = (nz - z * g.nt) * BN, m0 = mt * BM;

  const int HoWo = a.Ho * a.Wo, W = a.W, S = a.stride, pad = a.pad;
  const float inv_howo = 1.0f / (float)HoWo, inv_wo = 1.0f / (float)a.Wo;
  const bool k1 = a.kh == 1;
  const int CH = a.Cin / BK;
  const int npix = a.B * a.H * W;

  const __amdgpu_buffer_rsrc_t rx =
      rsrc(reinterpret_cast<const uint16_t*>(a.x) + z * a.x_mstride, (uint32_t)((int64_t)npix * a.Cin * 2));
  const __amdgpu_buffer_rsrc_t rw =
      WT == W_FRAG ? rsrc(reinterpret_cast<const uint16_t*>(a.wf) + z * a.wf_mstride, (uint32_t)((int64_t)a.Cout * a.Kp * 2))
         : rsrc(reinterpret_cast<const uint16_t*>(a.w) + z * a.w_mstride, (uint32_t)((int64_t)a.Cout * a.Kp * 2));

  // first pixel of the run (the top-left tap of output m0; may lie before the tensor)
  int p0;
  {
    const int b = m0 / HoWo, r = m0 - b * HoWo, oy = r / a.Wo, ox = r - oy * a.Wo;
    p0 = (b * a.H + oy * S) * W + ox * S - pad * (W + 1);
  }

  // ---- input rows into LDS: instruction v fills rows 8 (v % nrb) .. +8 of chunk v / nrb
  {
    const int nrb = g.rows >> 3, total = nrb * CH;
    int rb = wave, cc = 0;
    for (int v = wave; v < total; v += NW, rb += NW) {
      while (rb >= nrb) {
        rb -= nrb;
        ++cc;
      }
      const int r = rb * 8 + lr;
      int p;
      if (k1) {
        const int m = m0 + r;
        const int b = fdiv_small(m, inv_howo), q = m - b * HoWo, oy = fdiv_small(q, inv_wo), ox = q - oy * a.Wo;
        p = m < a.M ? (b * a.H + oy * S) * W + ox * S : -1;
      } else {
        p = p0 + (S == 1 ? r : (r < g.half ? 2 * r : 2 * (r - g.half) + 1));
      }
      const int lc = (lane & 7) ^ swz(r);
      const uint32_t off =
          (unsigned)p < (unsigned)npix ? (uint32_t)(((int64_t)p * a.Cin + cc * BK + lc * 8) * 2) : OOB;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_void*)(sm + v * 1024), 16, off, 0, 0, 0);
    }
  }
  const int CH2 = a.x2 ? a.Cin2 / BK : 0;
  if (CH2) {  // the projection shortcut's input: the tile's own pixels
    const __amdgpu_buffer_rsrc_t rx2 = rsrc(reinterpret_cast<const uint16_t*>(a.x2) + z * a.x2_mstride,
                                            (uint32_t)((int64_t)a.B * a.H2 * a.W2 * a.Cin2 * 2));
    for (int v = wave; v < CH2 * (BM / 8); v += NW) {
      const int cc = v / (BM / 8), r = (v - cc * (BM / 8)) * 8 + lr, m = m0 + r;
      const int b = fdiv_small(m, inv_howo), q = m - b * HoWo, oy = fdiv_small(q, inv_wo), ox = q - oy * a.Wo;
      const int lc = (lane & 7) ^ swz(r);
      const uint32_t off =
          m < a.M ? (uint32_t)(((((int64_t)b * a.H2 + oy * a.stride2) * a.W2 + ox * a.stride2) * a.Cin2 + cc * BK + lc * 8) * 2)
                  : OOB;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rx2, (lds_void*)(sm + g.off2 + v * 1024), 16, off, 0, 0, 0);
    }
  }
  if (!k1 && tid < 8) *reinterpret_cast<uint4*>(sm + g.zero + tid * 16) = uint4{0, 0, 0, 0};

  // ---- this wave's K-tiles and its weights
  const int nk1 = a.kh * a.kw * CH, nk = nk1 + CH2;
  const int u0 = ks * nk / KS, u1 = (ks + 1) * nk / KS;
  const int nw = n0 + nb * 32;
  const uint32_t wbase = WT == W_FRAG   ? (uint32_t)((int64_t)(nw / 32) * (a.Kp / 16) * 1024 + lane * 16)
                         : WT == W_TURN ? (uint32_t)(((int64_t)(nw + lr) * a.Kp + (lane & 7) * 8) * 2)
                                        : (uint32_t)(((int64_t)(nw + fr) * a.Kp + fq * 8) * 2);
  const uint32_t wstep = WT == W_FRAG ? 1024u : WT == W_TURN ? (uint32_t)a.Kp * 16 : 32u;  // load to load: k16 steps, or 8 packed rows
  auto load_w = [&](int u, uint4 (&v)[4]) {
    // past this wave's range: out of range, so that every step issues the same loads
    const uint32_t b = u < u1 ? wbase + (uint32_t)u * (WT == W_FRAG ? 4096u : 128u) : OOB;
#pragma unroll
    for (int s = 0; s < 4; ++s)
      v[s] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rw, b + wstep * s, 0, 0));
  };

  // ---- this lane's pixels: run position of the centre tap, top-left input coordinates
  int q0[FM], iy0[FM], ix0[FM];
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int m = m0 + i * 32 + fr;
    const int b = fdiv_small(m, inv_howo), r = m - b * HoWo, oy = fdiv_small(r, inv_wo), ox = r - oy * a.Wo;
    // past M: never inside the image (a 1x1 filter's rows past M hold zeros themselves)
    iy0[i] = m < a.M || k1 ? oy * S - pad : -(1 << 28);
    ix0[i] = ox * S - pad;
    q0[i] = k1 ? i * 32 + fr : (b * a.H + oy * S) * W + ox * S - pad * (W + 1) - p0;
  }
  const int sh = k1 ? 0 : S - 1;  // stride 2: row = j / 2, + half for odd j

  floatx16 acc[FM];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;

  // position of a K-tile: filter row and column, 64-channel chunk (scalars,
  // advanced one K-tile at a time; past the filter: the shortcut's chunk)
  int ky, kx, cc;
  {
    const int tap = u0 / CH;
    cc = u0 - tap * CH;
    ky = tap / a.kw;
    kx = tap - ky * a.kw;
    if (u0 >= nk1) cc = u0 - nk1;
  }
  // LDS address of this lane's first operand (k16 step 0) of block i; step s
  // is at address ^ (s << 5), since rows are 128 bytes and chunks are swizzled by XOR
  int ad[FM];
  auto address = [&](int u) {
    if (u < nk1) {  // wave-uniform
      const int cbase = cc * g.rows * ROW, dq = k1 ? 0 : ky * W + kx;
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        const int j = q0[i] + dq, row = (j >> sh) + (j & sh) * g.half;
        const bool ok = (unsigned)(iy0[i] + ky) < (unsigned)a.H && (unsigned)(ix0[i] + kx) < (unsigned)W;
        const int keep = 0 - (int)ok;  // a bitwise blend: the compiler branched around a select
        ad[i] = (((cbase + row * ROW) & keep) | (g.zero & ~keep)) + ((fq ^ swz(row)) << 4);
      }
    } else {
      const int cbase = g.off2 + cc * BM * ROW;
#pragma unroll
      for (int i = 0; i < FM; ++i) ad[i] = cbase + (i * 32 + fr) * ROW + ((fq ^ swz(i * 32 + fr)) << 4);
    }
  };
  auto advance = [&](int u) {  // to K-tile u
    if (++cc == CH && u <= nk1) {
      cc = 0;
      if (++kx == a.kw) {
        kx = 0;
        ++ky;
      }
    }
  };
  auto read_half = [&](int h, bf16x8 (&f)[2][FM]) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int i = 0; i < FM; ++i) f[s][i] = *reinterpret_cast<const bf16x8*>(sm + (ad[i] ^ ((2 * h + s) << 5)));
  };
  auto mma_half = [&](const bf16x8 (&f)[2][FM], const bf16x8& b0, const bf16x8& b1) {
#pragma unroll
    for (int i = 0; i < FM; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b0, f[0][i], acc[i], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < FM; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b1, f[1][i], acc[i], 0, 0, 0);
  };

  uint4 wr[RING][4];
#pragma unroll
  for (int d = 0; d < RING; ++d) load_w(u0 + d, wr[d]);
  wait_vmcnt<4 * RING>();  // the input rows landed; the weights may be in flight
  wait_lgkm0();            // ...and the zeros
  wg_barrier();
  // Each half K-tile's operands are read while the other half's MFMAs run
  // (reading them where they are used left a wave waiting for LDS four times
  // per K-tile, with one other wave on its SIMD to fill in).
  bf16x8 fa[2][FM], fb[2][FM];
  address(u0);
  read_half(0, fa);
  auto k_tile = [&](int u, const uint4 (&wv)[4]) {
    bf16x8 bw[4];
    if constexpr (WT != W_TURN) {
#pragma unroll
      for (int s = 0; s < 4; ++s) bw[s] = __builtin_bit_cast(bf16x8, wv[s]);
    } else {  // rows of 8 x 128 bytes -> fragments, through this wave's own LDS (in order within the wave)
      char* const wb = sm + g.wbuf + wave * 4096;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int r = s * 8 + lr;
        *reinterpret_cast<uint4*>(wb + r * ROW + (((lane & 7) ^ swz(r)) << 4)) = wv[s];
      }
      __asm__ __volatile__("" ::: "memory");
#pragma unroll
      for (int s = 0; s < 4; ++s)  // after the writes above: one wave's LDS operations run in order
        bw[s] = *reinterpret_cast<const bf16x8*>(wb + fr * ROW + (((2 * s + fq) ^ swz(fr)) << 4));
    }
    read_half(1, fb);
    __builtin_amdgcn_sched_barrier(0);
    mma_half(fa, bw[0], bw[1]);
    if (u + 1 < u1) {
      advance(u + 1);
      address(u + 1);
    }
    read_half(0, fa);  // the next K-tile's (after the last one: read again, unused)
    __builtin_amdgcn_sched_barrier(0);
    mma_half(fb, bw[2], bw[3]);
  };
  // whole rings first: no path skips a load in the loop, so that the
  // compiler's waits leave the younger ones in flight
  int u = u0;
  for (; u + RING <= u1; u += RING) {
#pragma unroll
    for (int d = 0; d < RING; ++d) {
      k_tile(u + d, wr[d]);
      load_w(u + d + RING, wr[d]);
    }
  }
#pragma unroll
  for (int d = 0; d < RING - 1; ++d)
    if (u + d < u1) k_tile(u + d, wr[d]);

  // ---- the waves' sums through LDS, KS_PASS 32-pixel blocks at a time.
  // D[n][m]: lane l holds pixel l % 32 and channels 8 g + 4 (l / 32) + r, one
  // 16-byte piece per (block, g).  Then one item = one pixel x 8 channels:
  // the KS sums in order, bias, residual, ReLU, one 16-byte store (4 NB items
  // make a pixel's 64 NB bytes)
  const float* __restrict__ bias = a.bias + z * a.b_mstride;
  const uint32_t obytes = (uint32_t)((int64_t)a.M * a.Cout * 2);
  const bool has_res = a.res != nullptr;
  const __amdgpu_buffer_rsrc_t rres =
      has_res ? rsrc(reinterpret_cast<const uint16_t*>(a.res) + z * a.res_mstride, obytes) : rsrc(a.y, 0u);
  const __amdgpu_buffer_rsrc_t ry = rsrc(reinterpret_cast<uint16_t*>(a.y) + z * a.y_mstride, obytes);
  constexpr int PB = FM < KS_PASS ? FM : KS_PASS;  // blocks per pass
  constexpr int WAVE = PB * 4 * KS_BLK;            // LDS bytes per wave
#pragma unroll
  for (int i0 = 0; i0 < FM; i0 += PB) {
    wait_lgkm0();
    wg_barrier();  // every wave has read its last operands, or the last pass's sums
#pragma unroll
    for (int i = i0; i < FM && i < i0 + PB; ++i)
#pragma unroll
      for (int gg = 0; gg < 4; ++gg)
        *reinterpret_cast<float4*>(sm + wave * WAVE + ((i - i0) * 4 + gg) * KS_BLK + lane * 16) =
            make_float4(acc[i][gg * 4], acc[i][gg * 4 + 1], acc[i][gg * 4 + 2], acc[i][gg * 4 + 3]);
    wait_lgkm0();
    wg_barrier();
    for (int it = tid; it < (FM - i0 < PB ? FM - i0 : PB) * 32 * 4 * NB; it += 64 * NW) {
      const int c8 = it % (4 * NB), px = it / (4 * NB), m = m0 + i0 * 32 + px, n = n0 + c8 * 8;
      if (m >= a.M) continue;
      const uint32_t o = (uint32_t)(((int64_t)m * a.Cout + n) * 2);
      const uint4 rv = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rres, o, 0, 0));  // zeros without one
      const float4 b0 = *reinterpret_cast<const float4*>(bias + n), b1 = *reinterpret_cast<const float4*>(bias + n + 4);
      const char* src = sm + (c8 >> 2) * WAVE + ((px >> 5) * 4 + (c8 & 3)) * KS_BLK + (px & 31) * 16;
      float v[8];
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        const char* s = src + k * NB * WAVE;
        const float4 lo = *reinterpret_cast<const float4*>(s), hi = *reinterpret_cast<const float4*>(s + 512);
        if (k == 0) {
          v[0] = lo.x; v[1] = lo.y; v[2] = lo.z; v[3] = lo.w;
          v[4] = hi.x; v[5] = hi.y; v[6] = hi.z; v[7] = hi.w;
        } else {
          v[0] += lo.x; v[1] += lo.y; v[2] += lo.z; v[3] += lo.w;
          v[4] += hi.x; v[5] += hi.y; v[6] += hi.z; v[7] += hi.w;
        }
      }
      v[0] += b0.x; v[1] += b0.y; v[2] += b0.z; v[3] += b0.w;
      v[4] += b1.x; v[5] += b1.y; v[6] += b1.z; v[7] += b1.w;
      if (has_res) {
        float rr[8];
        bf8_to_f8(rv, rr);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += rr[e];
      }
      if (a.relu)
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = v[e] > 0.f ? v[e] : 0.f;
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, f8_to_bf8(v)), ry, o, 0, 0);
    }
  }
}

// LDS plan of a layer for tiles of bm pixels; *lds = bytes needed.  packed:
// with the buffers that turn packed weight rows.
KsGeom ks_geom(const ConvArgs& a, int bm, int bn, bool packed, size_t* lds) {
  KsGeom g{};
  g.mt = (a.M + bm - 1) / bm;
  g.nt = a.Cout / bn;
  int64_t need = bm;  // a 1x1 filter reads the tile's own pixels
  if (a.kh == 3) {
    // an upper bound over every tile: a step to the next output moves `stride`
    // pixels, the end of an output row stride (W - Wo) more, the end of an
    // image (H - stride Ho) W more (never positive for stride 2)
    const int64_t steps = bm - 1, rows = (steps + a.Wo - 1) / a.Wo, imgs = (steps + a.Ho * a.Wo - 1) / (a.Ho * a.Wo);
    need = a.stride * steps + rows * a.stride * (a.W - a.Wo) +
           imgs * std::max(0, a.H - a.stride * a.Ho) * (int64_t)a.W + 2 * (a.W + 1) + 1;
  }
  g.half = a.stride == 2 ? (int)((need + 1) / 2) : 0;
  const int64_t nr = a.stride == 2 && a.kh == 3 ? 2 * (int64_t)g.half : need;
  g.rows = (int)((nr + 7) / 8 * 8);
  const int64_t CH = a.Cin / BK, CH2 = a.x2 ? a.Cin2 / BK : 0;
  int64_t off = CH * g.rows * ROW;
  g.off2 = (int)std::min<int64_t>(off, INT32_MAX);
  off += CH2 * bm * ROW;
  g.zero = (int)std::min<int64_t>(off, INT32_MAX);
  if (a.kh == 3) off += ROW;
  if (packed) {
    off = (off + 1023) / 1024 * 1024;
    g.wbuf = (int)std::min<int64_t>(off, INT32_MAX);
    off += (int64_t)KS_WAVES * 4096;
  }
  *lds = (size_t)std::max<int64_t>(off, (int64_t)KS_WAVES * std::min(bm / 32, KS_PASS) * 4 * KS_BLK);
  return g;
}

constexpr size_t KS_LDS = 160 * 1024;

}  // namespace

// Layers the kernel can run: 3x3 (pad 1) or 1x1 (pad 0) filters of stride 1
// or 2 on whole 64-channel chunks, whole channel blocks, and the tile's
// input in LDS.
bool conv_ks_ok(const ConvArgs& a, int bm, int bn) {
  if (a.kh != a.kw || !((a.kh == 3 && a.pad == 1) || (a.kh == 1 && a.pad == 0)) || a.stride < 1 || a.stride > 2)
    return false;
  if (a.Cin % BK || a.Cout % bn || (a.x2 && !a.wf)) return false;
  const int K1 = a.kh * a.kw * a.Cin;
  if (a.x2 ? (a.Cin2 % BK || a.K1 != K1 || a.K != K1 + a.Cin2 || (a.Ho - 1) * a.stride2 >= a.H2 ||
              (a.Wo - 1) * a.stride2 >= a.W2 || (int64_t)a.B * a.H2 * a.W2 * a.Cin2 * 2 >= (1ll << 31))
           : a.K != K1)
    return false;
  if (a.K != a.Kp || (a.Ho - 1) * a.stride - a.pad >= a.H || (a.Wo - 1) * a.stride - a.pad >= a.W) return false;
  if ((int64_t)a.M * a.Cout * 2 >= (1ll << 31)) return false;
  if ((int64_t)a.M + 4096 >= (1 << 22) || a.K / BK >= (1 << 22)) return false;  // fdiv_small range
  if ((int64_t)a.B * a.H * a.W * a.Cin * 2 >= (1ll << 31) || (int64_t)a.Cout * a.Kp * 2 >= (1ll << 31)) return false;
  if (a.K / BK < KS_WAVES / (bn / 32)) return false;  // every wave has a K-tile
  size_t lds = 0;
  ks_geom(a, bm, bn, false, &lds);  // packed rows that find no LDS to be turned in are read as they lie
  return lds <= KS_LDS;
}

void launch_conv_ks(const ConvArgs& a_in, int bm, int bn, hipStream_t s) {
  ConvArgs a = a_in;  // outputs are always finished here
  a.split = 1;
  a.partial = nullptr;
  size_t lds = 0;
  KsGeom g = ks_geom(a, bm, bn, !a.wf, &lds);
  const bool rows = lds > KS_LDS;  // no room to turn packed rows
  if (rows) g = ks_geom(a, bm, bn, false, &lds);
  const dim3 grid((unsigned)(g.mt * g.nt * a.Z)), block(64 * KS_WAVES);
  // the turned weights take registers: a shorter ring
#define FS_KS(FMv, KSv, NBv, RINGv, WPSv)                                                               \
  if (bm == 32 * FMv && bn == 32 * NBv) {                                                               \
    if (a.wf)                                                                                           \
      hipLaunchKernelGGL((k_conv_ks<FMv, KSv, NBv, RINGv, WPSv, W_FRAG>), grid, block, lds, s, a, g);   \
    else if (rows)                                                                                      \
      hipLaunchKernelGGL((k_conv_ks<FMv, KSv, NBv, RINGv, WPSv, W_ROWS>), grid, block, lds, s, a, g);   \
    else                                                                                                \
      hipLaunchKernelGGL((k_conv_ks<FMv, KSv, NBv, 2, WPSv, W_TURN>), grid, block, lds, s, a, g);       \
    return;                                                                                             \
  }
  FS_KS(1, 8, 1, 4, 4) FS_KS(1, 4, 2, 4, 4) FS_KS(2, 4, 2, 2, 4) FS_KS(2, 2, 4, 2, 4) FS_KS(3, 2, 4, 3, 2)
#undef FS_KS
}

// The tiles of the rule below: pixels, channels, waves along the reduction,
// whether registers let two workgroups share a CU, the most workgroups per CU at
// which the tile was the fastest kernel anywhere, and the time in us with
// fragment-ordered weights and with packed rows turned through LDS,
//   a + (b q + c + l lds / 80 KB + r residual) f,
// q: K-tiles per wave, f: 1 for up to one workgroup a CU; beyond that, for n of
// them, one * ceil(n) where LDS holds one at a time, else max(two, slope n).
// rows: packed rows read as they lie take that many times as long as fragments.
struct KsCost {
  double a, b, c, l, one, two, slope, r;
};
struct KsTile {
  int bm, bn, ks, pair;
  double most;
  KsCost frag, turn;
  double rows;
};
static const KsTile kKsTiles[] = {
    {32, 32, 8, 1, 3, {2.96, 0.22, 0.77, 2.06, 1.20, 1.79, 1.11, 0.18}, {3.11, 0.42, 0.00, 2.56, 1.11, 2.17, 1.42, 0.00}, 1.70},
    {32, 64, 4, 1, 2, {3.07, 0.23, 0.60, 2.12, 1.14, 1.88, 1.17, 0.04}, {3.19, 0.41, 0.00, 2.38, 1.10, 2.15, 1.31, 0.00}, 2.00},
    {64, 64, 4, 1, 2, {3.01, 0.34, 0.25, 2.10, 1.21, 1.66, 1.10, 0.09}, {2.74, 0.57, 0.00, 2.54, 1.12, 1.60, 1.15, 0.00}, 1.45},
    {64, 128, 2, 1, 2, {2.94, 0.35, 0.61, 2.05, 1.16, 1.77, 1.16, 0.10}, {3.05, 0.59, 0.00, 2.52, 1.06, 1.81, 1.22, 0.00}, 1.70},
    {96, 128, 2, 0, 2, {1.38, 0.50, 2.48, 2.67, 1.05, 1.39, 1.15, 0.42}, {1.00, 0.71, 2.37, 3.05, 1.01, 2.24, 1.15, 0.31}, 1.40},
};

// Estimated time (us) of the layer on a tile, with the weights in the form that
// the layer has them in; *rounds: more than one workgroup a CU.
static double ks_estimate(const ConvArgs& a, const KsTile& t, double cus, bool* rounds) {
  size_t lds = 0;
  const KsGeom g = ks_geom(a, t.bm, t.bn, false, &lds);
  const double n = (double)g.mt * g.nt * a.Z / cus;
  *rounds = n > 1;
  if (n > t.most) return 1e30;
  bool turn = false;
  if (!a.wf) {
    size_t with = 0;
    ks_geom(a, t.bm, t.bn, true, &with);
    turn = with <= KS_LDS;
  }
  const KsCost& c = turn ? t.turn : t.frag;
  const int nk = a.K / BK, per_cu = std::min(t.pair ? 2 : 1, (int)(KS_LDS / lds));
  const double wg = (nk + t.ks - 1) / t.ks * c.b + c.c + c.l * (double)lds / (80 * 1024) + (a.res ? c.r : 0.0);
  const double us = c.a + wg * (n <= 1 ? 1.0 : per_cu == 1 ? c.one * std::ceil(n) : std::max(c.two, c.slope * n));
  return a.wf || turn ? us : us * t.rows;
}

// The time below which this kernel is taken: that of the kernel that runs the
// layer otherwise, less what the estimates may be off.  An ensemble's implicit
// GEMM runs in the fastest of twenty timed tiles, of which nine are estimated;
// short reductions leave little to split (1x1, 512 -> 128 on 28x28, B = 14 to 22,
// packed: 7.9 us against 8.6).
static double ks_limit(const ConvArgs& a, double cus) {
  const double nk = a.K / BK;
  if (conv_hs_chosen(a)) {
    auto per_cu = [&](int bm) { return std::max(1.0, (double)((a.M + bm - 1) / bm) * (a.Cout / 128) * a.Z / cus); };
    // the register-weight tiles' patch, nearly: their rows, a partial one at
    // either end, the rows above and below, and the rows between two images
    auto fits = [&](int bm) { return (bm / a.W + 4) * (a.W + 2) <= 320; };
    const double n = per_cu(128), n96 = per_cu(96), n160 = per_cu(160);
    const double hs = 1.91 + (0.387 * nk + 2.31) * std::ceil(n) + (1.87 + (a.res ? 0.10 : 0.0)) * n;
    if (!a.wf) return 0.97 * hs;
    const double e96 = 3.10 + 0.032 * nk + (0.144 * nk + 1.33) * std::ceil(n96) + (0.154 * nk + 1.50) * n96;
    const double e160 = 2.26 + 0.137 * nk + 0.137 * nk * std::ceil(n160) + (0.311 * nk + 7.28) * n160;
    double us = a.x2 ? e96 : hs;  // a projection shortcut runs in the register-weight form only
    if (fits(96)) us = std::min(us, e96);
    if (fits(160)) us = std::min(us, e160);
    return 0.97 * us;
  }
  if (conv_halo_ok(a, 4, 56, 64))
    return 4.6 + 4.1 * std::ceil((double)a.B * ((a.Ho + 3) / 4) * (a.Cout / 64) * a.Z / cus);
  ConvArgs d = a;
  d.split = conv_split(BF16, a, (int)cus);
  double us = 0;
  conv_dma_pick(d, (int)cus, &us);
  if (d.split > 1) us += 3.0 + (double)d.split * a.M * a.Cout * a.Z * 8 / 6.5e6;  // the completion: partial sums out and in
  return (a.wf || nk <= 8 ? 0.91 : 0.97) * us;
}

// Which of this kernel's tiles runs the layer, or -1: the one that is estimated
// fastest, if that beats the kernel that runs the layer otherwise, with the
// weights in the form the layer has them in.  The estimates were fitted to
// back-to-back launches of every tile and of every other kernel in both forms
// on 820 layers: 64 to 2048 channels, 3x3 and 1x1, stride 1 and 2, maps of 3 to
// 117, B = 1 to 48, one to five models.  The rule is 0.3 % slower there than the
// fastest kernel on average, and nowhere more than 3 % slower than the kernel
// that ran the layer otherwise at its fastest tile (packed rows: against that
// kernel at the tile it gets, with two of 192 layers 0.3 and 0.8 us slower).  Measured (us, this kernel against the other):
// 7x7x512 3x3, three models, B = 1 / 8 / 16: 7.3 / 12.4 / 17.6 against 26.3 / 32.4 /
// 32.5; 14x14x256 B = 1 / 8: 6.1 / 11.3 against 15.9 / 16.6; 28x28x128 to 256
// stride 2 (split over workgroups), B = 8 / 16: 9.3 / 12.7 against 16.9 / 22.5.
// The others win with more tiles (14x14x256 B = 32 24.6 against 26.4; 28x28x128
// to 256 stride 2 17.3 against 24.0), where rounds of workgroups fill a CU's LDS
// one at a time (14x14x512, B = 12, five models, 51 against 64), where the
// reduction is two K-tiles (1x1, 128 -> 512 on 28x28, 4.4 against 5.3), and with
// packed rows that find no LDS to be turned in (28x28x512, B = 10, 40 against 73).
// It depends on the shape and the batch only (256 CUs, the chip's), never on
// timing, so a result's bits do not vary from run to run.
int conv_ks_pick(const ConvArgs& a_in, int* bm, int* bn) {
  constexpr double cus = 256;
  ConvArgs a = a_in;
  a.split = 1;  // the caller's split is the implicit GEMM's
  double best = 1e30, us = 1e30;
  int pick = -1;
  for (int i = 0; i < (int)(sizeof(kKsTiles) / sizeof(KsTile)); ++i) {
    if (!conv_ks_ok(a, kKsTiles[i].bm, kKsTiles[i].bn)) continue;
    bool rounds = false;
    const double e = ks_estimate(a, kKsTiles[i], cus, &rounds);
    // of nearly equal tiles the larger one: more workgroups cost more than the
    // estimate where their weights are not in L2 again when a launch starts
    // (14x14x256, B = 32, among the layers of a network: 64x64 15.4 us, 64x128
    // 14.4, in a loop 12.5 and 12.4) or have to be turned (16x16x256, B = 24: 18.9
    // and 16.1)
    const double key = rounds ? 1.05 * e : e;
    if (key < best) {
      best = key;
      us = e;
      pick = i;
    }
  }
  if (pick < 0 || us >= ks_limit(a, cus)) return -1;
  *bm = kKsTiles[pick].bm;
  *bn = kKsTiles[pick].bn;
  return pick;
}

}  // namespace fs
