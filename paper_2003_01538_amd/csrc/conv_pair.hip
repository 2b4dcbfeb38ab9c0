// Two 1x1 convolutions in one launch: a bottleneck block's widening conv
// (bias, residual or projection shortcut, ReLU) and the narrowing conv (bias,
// ReLU) of the block after it, which reads the first one's output.
//
// Both are bound by memory: of the traffic of the two launches (64 -> 256
// channels with a residual, then 256 -> 64: 896 channels per pixel) more than a quarter
// is the wide tensor, written by the first and read again by the second.  It
// still has to be written - the block after next takes it as its residual -
// but need not be read: the MFMA leaves a lane eight consecutive channels of
// one pixel, which, rounded to bf16 for the store, are exactly the operand
// the same lane owes the second product.  So no LDS and no barrier lies
// between the two.
//
// A wave owns 32 pixels: their narrow input stays in registers (NKM + NKP
// fragments of 16 channels: main part and projection shortcut), so do the
// second conv's accumulators (NB2 blocks of 32 channels).  The wide
// dimension is walked in chunks of 32 * CN channels; per chunk both convs'
// weights come through a two-stage LDS ring in MFMA fragment order (one
// conflict-free 1 KB read per fragment), shared by the four waves, and the
// residual one chunk ahead into registers.
//
// Per chunk the operand reads run four fragments ahead of their MFMAs
// (scheduling groups; two ahead, as the compiler orders them, the 256 -> 1024
// -> 256 pair takes 387 us instead of 373) and the residual loads are kept at
// the chunk's start.
//
// Five models at B = 256, against the two launches: 56x56, 64 -> 256 -> 64
// 1035 us (4.96 TB/s) against 1002 + 487; -> 128 1164 against 998 + 645;
// 28x28, 128 -> 512 -> 128 560 (4.6 TB/s) against 600 + 274, with the
// projection shortcut 632 against 610 + 284, -> 256 696 against 597 + 390;
// 14x14, 256 -> 1024 -> 256 373 against 353 + 167.  The first are bound by
// memory; the last by the LDS and L2 reads of its weights (1 MB per 128
// pixels), which more pixels per wave would halve, but its accumulators
// and input already fill the registers of two waves a SIMD.
//
// Each sum runs over its reduction in steps of 16 in ascending order, as in
// the implicit GEMM kernel, and the wide values are rounded to bf16 before
// they are used: the results are those of the two launches, bit for bit.
#include "common.hpp"
#include "device.hpp"
#include "lds_dma.hpp"

#include <algorithm>

namespace fs {

namespace {

constexpr int PM = 128;      // pixels per workgroup
constexpr int MAXN1 = 1024;  // widest first conv

template <int NKM, int NKP, int NB2, int CN, int OCC>
__global__ void __launch_bounds__(256, OCC) k_conv_pair(ConvArgs a, ConvArgs d) {
  constexpr int NK = NKM + NKP;
  constexpr bool RES = NKP == 0;
  constexpr int W1 = CN * NK, W2 = NB2 * 2 * CN;  // 1 KB weight fragments per chunk
  constexpr int LPW = (W1 + W2) / 4;              // DMA instructions per wave and chunk
  constexpr int STAGE = (W1 + W2) * 1024;
  constexpr int AHEAD = 4;  // weight fragments read ahead of their MFMA
  static_assert(W1 % 4 == 0 && W2 % 4 == 0, "fragments divide over the waves");
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  // Read as floatx4 below: before a read of LDS that it cannot tell from the
  // direct loads by type, the compiler waits for every one in flight.
  __shared__ __attribute__((aligned(16))) float sb1[MAXN1 + NB2 * 32];
  float* const sb2 = sb1 + MAXN1;

  const int tid = threadIdx.x, lane = tid & 63, fq = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tiles = (a.M + PM - 1) / PM;
  const int id = xcd_remap(blockIdx.x, tiles * a.Z);
  const int z = id / tiles, m0 = (id - z * tiles) * PM;
  const int m = m0 + wave * 32 + (lane & 31);
  const bool in = m < a.M;

  const __amdgpu_buffer_rsrc_t rx =
      rsrc(reinterpret_cast<const uint16_t*>(a.x) + z * a.x_mstride, (uint32_t)((int64_t)a.M * a.Cin * 2));
  const __amdgpu_buffer_rsrc_t rx2 =
      rsrc(NKP ? reinterpret_cast<const uint16_t*>(a.x2) + z * a.x2_mstride : reinterpret_cast<const uint16_t*>(a.x),
           NKP ? (uint32_t)((int64_t)a.B * a.H2 * a.W2 * a.Cin2 * 2) : 0u);
  const __amdgpu_buffer_rsrc_t rw1 =
      rsrc(reinterpret_cast<const uint16_t*>(a.wf) + z * a.wf_mstride, (uint32_t)((int64_t)a.Cout * a.Kp * 2));
  const __amdgpu_buffer_rsrc_t rw2 =
      rsrc(reinterpret_cast<const uint16_t*>(d.wf) + z * d.wf_mstride, (uint32_t)((int64_t)d.Cout * d.Kp * 2));
  const __amdgpu_buffer_rsrc_t ry =
      rsrc(reinterpret_cast<const uint16_t*>(a.y) + z * a.y_mstride, (uint32_t)((int64_t)a.M * a.Cout * 2));
  const __amdgpu_buffer_rsrc_t rt =
      rsrc(reinterpret_cast<const uint16_t*>(d.y) + z * d.y_mstride, (uint32_t)((int64_t)d.M * d.Cout * 2));
  // without a residual every read of it is out of range: zeros
  const __amdgpu_buffer_rsrc_t rr =
      rsrc(a.res ? reinterpret_cast<const uint16_t*>(a.res) + z * a.res_mstride : reinterpret_cast<const uint16_t*>(a.x),
           a.res ? (uint32_t)((int64_t)a.M * a.Cout * 2) : 0u);

  // this lane's narrow input: channels 16 s + 8 fq .. + 7 of its pixel
  bf16x8 hf[NK];
  const uint32_t h_off = in ? (uint32_t)(((int64_t)m * a.Cin + 8 * fq) * 2) : OOB;
#pragma unroll
  for (int s = 0; s < NKM; ++s)
    hf[s] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rx, h_off + s * 32, 0, 0));
  if constexpr (NKP > 0) {
    const int HoWo = a.Ho * a.Wo;
    const int b = m / HoWo, r = m - b * HoWo, oy = r / a.Wo, ox = r - oy * a.Wo;
    const uint32_t p_off =
        in ? (uint32_t)(((((int64_t)b * a.H2 + oy * a.stride2) * a.W2 + ox * a.stride2) * a.Cin2 + 8 * fq) * 2) : OOB;
#pragma unroll
    for (int s = 0; s < NKP; ++s)
      hf[NKM + s] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rx2, p_off + s * 32, 0, 0));
  }
  for (int i = tid; i < a.Cout; i += 256) sb1[i] = a.bias[z * a.b_mstride + i];
  for (int i = tid; i < d.Cout; i += 256) sb2[i] = d.bias[z * d.b_mstride + i];

  // chunk c's weights: fragments (block c CN + i, step s) of the first conv,
  // in memory as they lie in LDS, then (block j, steps 2 CN c ..) of the second
  const uint32_t w2_blk = (uint32_t)(d.Kp / 16) * 1024u;
  auto issue = [&](int c, int stage) {
#pragma unroll
    for (int u = 0; u < LPW; ++u) {
      const int f = u * 4 + wave;
      char* dst = smem + stage * STAGE + f * 1024;
      if (u * 4 < W1) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rw1, (lds_void*)dst, 16, lane * 16, (c * W1 + f) * 1024, 0, 0);
      } else {
        const int g = f - W1, j = g / (2 * CN), t = g - j * (2 * CN);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rw2, (lds_void*)dst, 16, lane * 16,
                                                 j * w2_blk + (c * 2 * CN + t) * 1024, 0, 0);
      }
    }
  };
  const uint32_t y_off = in ? (uint32_t)(((int64_t)m * a.Cout + 8 * fq) * 2) : OOB;
  const uint32_t r_off = a.res ? y_off : OOB;

  floatx16 acc2[NB2];
#pragma unroll
  for (int j = 0; j < NB2; ++j)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc2[j][e] = 0.f;

  v4u ra[RES ? 2 * CN : 1], rb[RES ? 2 * CN : 1];  // residual of the even and of the odd chunks
  const int NC = a.Cout / (32 * CN);

  // one chunk with its residual rc; `more`: the next one's weights and
  // residual (into rn) are issued first
  auto chunk = [&](int c, auto& rc, auto& rn, auto more) {
    const int stage = c & 1;
    wait_lgkm0();
    wg_barrier();  // chunk c is in LDS; every wave is done with chunk c - 1
    if constexpr (decltype(more)::value) {
      issue(c + 1, stage ^ 1);
      __asm__ __volatile__("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (RES)
#pragma unroll
        for (int i = 0; i < 2 * CN; ++i)
          rn[i] = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(rr, r_off + i * 32, (c + 1) * 64 * CN, 0));
      __builtin_amdgcn_sched_barrier(0);
    }
    const char* wl = smem + stage * STAGE + lane * 16;
    floatx16 acc[CN];
#pragma unroll
    for (int i = 0; i < CN; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
#pragma unroll
    for (int s = 0; s < NK; ++s)
#pragma unroll
      for (int i = 0; i < CN; ++i)
        acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(wl + (i * NK + s) * 1024),
                                                         hf[s], acc[i], 0, 0, 0);
    floatx4 bv[CN][4];
#pragma unroll
    for (int i = 0; i < CN; ++i)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        bv[i][g] = *reinterpret_cast<const floatx4*>(sb1 + (c * CN + i) * 32 + 16 * (g >> 1) + 8 * fq + 4 * (g & 1));
    __builtin_amdgcn_sched_group_barrier(0x100, AHEAD, 0);
#pragma unroll
    for (int s = 0; s < CN * NK; ++s) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x100, 4 * CN, 0);
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 yf[2 * CN];
#pragma unroll
    for (int i = 0; i < CN; ++i)
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        float v[8];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[i][g * 8 + r]),
                                                           __float_as_uint(acc[i][g * 8 + 4 + r]), false, false);
          v[r] = __uint_as_float(sw[0]);
          v[4 + r] = __uint_as_float(sw[1]);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += bv[i][2 * g + (e >> 2)][e & 3];
        if constexpr (RES) {
          float q[8];
          bf8_to_f8(__builtin_bit_cast(uint4, rc[i * 2 + g]), q);
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] += q[e];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = v[e] > 0.f ? v[e] : 0.f;
        const uint4 o = f8_to_bf8(v);
        yf[i * 2 + g] = __builtin_bit_cast(bf16x8, o);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, o), ry, y_off + (i * 2 + g) * 32, c * 64 * CN, 0);
      }
#pragma unroll
    for (int t = 0; t < 2 * CN; ++t)
#pragma unroll
      for (int j = 0; j < NB2; ++j)
        acc2[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            *reinterpret_cast<const bf16x8*>(wl + (W1 + j * 2 * CN + t) * 1024), yf[t], acc2[j], 0, 0, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, AHEAD, 1);
#pragma unroll
    for (int s = 0; s < W2; ++s) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 1);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 1);
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  issue(0, 0);
  __asm__ __volatile__("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (RES)
#pragma unroll
    for (int i = 0; i < 2 * CN; ++i)
      ra[i] = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(rr, r_off + i * 32, 0, 0));
  // a wave's loads of chunk c's weights are followed by its residual loads
  // of chunk c and, from the second chunk on, its stores of chunk c - 1
  // (2 CN each; rows past M store out of range, so the count is the same for
  // every wave)
  constexpr int NR = RES ? 2 * CN : 0;
  wait_vmcnt<NR>();
  chunk(0, ra, rb, std::true_type{});
  for (int c = 1; c < NC - 1; c += 2) {  // NC is even
    wait_vmcnt<NR + 2 * CN>();
    chunk(c, rb, ra, std::true_type{});
    wait_vmcnt<NR + 2 * CN>();
    chunk(c + 1, ra, rb, std::true_type{});
  }
  wait_vmcnt<NR + 2 * CN>();
  chunk(NC - 1, rb, ra, std::false_type{});

  const uint32_t t_off = in ? (uint32_t)(((int64_t)m * d.Cout + 8 * fq) * 2) : OOB;
#pragma unroll
  for (int j = 0; j < NB2; ++j)
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      float v[8];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc2[j][g * 8 + r]),
                                                         __float_as_uint(acc2[j][g * 8 + 4 + r]), false, false);
        v[r] = __uint_as_float(sw[0]);
        v[4 + r] = __uint_as_float(sw[1]);
      }
      const float* bp = sb2 + j * 32 + 16 * g + 8 * fq;
      const float4 b0 = *reinterpret_cast<const float4*>(bp), b1 = *reinterpret_cast<const float4*>(bp + 4);
      v[0] += b0.x; v[1] += b0.y; v[2] += b0.z; v[3] += b0.w;
      v[4] += b1.x; v[5] += b1.y; v[6] += b1.z; v[7] += b1.w;
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = v[e] > 0.f ? v[e] : 0.f;
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, f8_to_bf8(v)), rt, t_off + (j * 2 + g) * 32, 0, 0);
    }
}

// The instances: fragments of the main input and of the projection shortcut,
// blocks of 32 outputs of the second conv, blocks of the wide dimension per
// chunk (two where the ring then leaves room for two workgroups a CU).
template <int NKM, int NKP, int NB2, int CN, int OCC>
void launch_t(const ConvArgs& a, const ConvArgs& d, hipStream_t s) {
  const int lds = 2 * (CN * (NKM + NKP) + NB2 * 2 * CN) * 1024;
  const int tiles = (a.M + PM - 1) / PM;
  hipLaunchKernelGGL((k_conv_pair<NKM, NKP, NB2, CN, OCC>), dim3(tiles * a.Z), dim3(256), lds, s, a, d);
}

struct Pair {
  int nkm, nkp, nb2;
  void (*fn)(const ConvArgs&, const ConvArgs&, hipStream_t);
};
const Pair kPairs[] = {
    {4, 4, 2, launch_t<4, 4, 2, 2, 3>},   {4, 0, 2, launch_t<4, 0, 2, 2, 3>},   {4, 0, 4, launch_t<4, 0, 4, 2, 2>},
    {8, 16, 4, launch_t<8, 16, 4, 1, 2>}, {8, 0, 4, launch_t<8, 0, 4, 2, 2>},   {8, 0, 8, launch_t<8, 0, 8, 1, 2>},
    {16, 0, 8, launch_t<16, 0, 8, 1, 2>},
};

const Pair* pair_of(const ConvArgs& a, const ConvArgs& d) {
  for (const Pair& p : kPairs)
    if (p.nkm * 16 == a.Cin && p.nkp * 16 == (a.x2 ? a.Cin2 : 0) && p.nb2 * 32 == d.Cout) return &p;
  return nullptr;
}

}  // namespace

// Whether the two layers have the form the kernel takes: shapes only, so a
// plan may ask before the weights are laid out.
bool conv_pair_ok(const ConvArgs& a, const ConvArgs& d) {
  auto plain = [](const ConvArgs& c) {
    return c.kh == 1 && c.kw == 1 && c.stride == 1 && c.pad == 0 && c.relu && c.H == c.Ho && c.W == c.Wo;
  };
  if (!plain(a) || !plain(d) || d.x2 || d.res || (a.x2 && a.res)) return false;
  if (d.Cin != a.Cout || d.M != a.M || d.Z != a.Z || d.Kp != d.Cin) return false;
  if (a.Kp != a.Cin + (a.x2 ? a.Cin2 : 0) || (a.x2 && a.K1 != a.Cin)) return false;
  if (a.Cout % 128 || a.Cout > MAXN1) return false;
  const int64_t lim = int64_t(1) << 31;
  if ((int64_t)a.M * a.Cout * 2 >= lim || (a.x2 && (int64_t)a.B * a.H2 * a.W2 * a.Cin2 * 2 >= lim)) return false;
  return pair_of(a, d) != nullptr;
}

// One launch from three workgroups for every four CUs on.  A workgroup walks
// the whole wide dimension by itself, so below that the launch takes the time
// of one walk however few there are (1024 channels wide: 48 us at 49
// workgroups, where the two launches take 17 + 14 us; at 196 they take 50 us or
// more: 512 wide, 25 to 32 us against 22 + 14, 31 against 21 + 20).
bool conv_pair_chosen(const ConvArgs& a, const ConvArgs& d, int num_cus) {
  return a.wf && d.wf && conv_pair_ok(a, d) && (int64_t)((a.M + PM - 1) / PM) * a.Z * 4 >= (int64_t)num_cus * 3;
}

void launch_conv_pair(const ConvArgs& a, const ConvArgs& d, hipStream_t s) { pair_of(a, d)->fn(a, d, s); }

}  // namespace fs
