// 3x3 stride-1 convolution (forward and input gradient) of wide bf16 layers: contraction channels a
// multiple of 128, output channels a multiple of 128.
//
// The generic wide kernel stages the pixel operand once per tap and synchronises per chunk of 64-128
// contraction values; with one or two tiles per compute unit its phases (loads, LDS, matrix
// instructions) then add up instead of overlapping. Here a workgroup stages the rows of its 128
// pixels plus the W + 1 neighbours on each side for a slice of 128 channels ONCE, and contracts all
// nine taps from them: a ninth of the staging (and of the on-load batch norm), one barrier per 1152
// contraction values, and between barriers the eight waves run freely.
//
//   pixel operand:  flat rows m0 - W - 1 .. m0 + 127 + W + 1 of one slice, row pitch 272 bytes (the
//                   fragment reads of consecutive lanes fall into distinct banks), two buffers; a tap is a row
//                   shift, and a lane whose neighbour lies outside the image reads the zero row at LDS
//                   address 0 instead (address AND a sign-extended bit of its tap mask)
//   weight operand: fragments straight from the packed operand into the registers of the wave that uses
//                   them, a ring of three steps, no wave loads what another one loads
//   waves:          BN/64 (64 channels each) x KG parts of every slice's k-steps; a wave holds all 128
//                   pixels x 64 channels = eight accumulators of mfma_f32_32x32x16_bf16. The KG parts meet in
//                   LDS as fp32 tiles, added in a fixed order.
//
// What bounds it (time stamps, 256 -> 256 channels at 14x14, two minibatches of 32): of 21 us in the kernel
// 3.4 are the cold start up to the first slice in LDS, 14 the loop (9.7 of them matrix instructions; waves of
// 128 x 32, which read twice as much from LDS per matrix instruction, took 1 us more), 3.5 the parts meeting,
// the stores and the statistics. BN = 64 where 128-channel tiles would leave compute units
// idle. Two minibatches with on-load batch norm 30.8 (the generic wide kernel) -> 22.0 us, input
// gradient of one 19.2 -> 16.6 us. With the 98 statistics rows of its input added here, instead of by a launch of 4.5 us before it
// (WideRows), the forward launch takes 2.6 us more.
#include "ddg_conv_wide.h"

namespace ddg {

namespace halo {
constexpr int BM = 128, CS = 128;
constexpr int PITCH = CS * 2 + 16;
constexpr int NU = 6;                                 // 16-byte units a thread stages per slice
constexpr int ROWS = NU * 512 / (CS / 8);             // 192 staged rows: 128 + 2*(W + 1) at most
constexpr int BUF = ROWS * PITCH;
constexpr int WMAX = (ROWS - BM) / 2 - 1;             // 31
constexpr int TAB = PITCH + 2 * BUF;                  // XFORM: scale and shift of the input channels
constexpr int ICMAX = 2048;
constexpr int orow(int BN) { return BN * 4 + 16; }    // bytes per pixel of an fp32 tile
constexpr int lds_bytes(int BN) { return (256 / BN) * BM * orow(BN); }   // KG/2 tiles of 128 x BN
static_assert(TAB + 2 * ICMAX * 4 <= lds_bytes(128) && TAB + 2 * ICMAX * 4 <= lds_bytes(64), "staging fits beside the table");
}

template <int STATS, bool XFORM, int BN>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void conv_halo_kernel(ConvWideArgs a) {
  using namespace halo;
  constexpr int NCH = BN / 64, KG = 8 / NCH, KPW = 8 / KG;   // channel groups, parts of a slice, k16-steps per wave and tap
  constexpr int SPR = 3 * KPW;                               // steps per kernel row
  constexpr int RING = 3;                                    // steps whose weight fragments are in flight
  constexpr int OROW = orow(BN);
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  const int wn = wave % NCH, kg = wave / NCH;
  const bool second = blockIdx.z != 0;
  const bf16_t* __restrict__ g_in = second ? a.in_b : a.in;
  bf16_t* __restrict__ g_out = second ? a.out_b : a.out;
  float* __restrict__ g_stat = second ? a.stat_partial_b : a.stat_partial;
  const float* __restrict__ g_scale = second ? a.scale_b : a.scale;
  const float* __restrict__ g_shift = second ? a.shift_b : a.shift;
  const int m0 = blockIdx.x * BM, c0 = blockIdx.y * BN;
  const int OCB = a.OC >> 4, nsl = a.IC / CS;
  const int nrows = BM + 2 * a.W + 2;

  // ---- staging: unit tid + q*512 = row (tid>>4) + 32*q, 16-byte chunk tid&15
  const int pc = tid & 15;
  auto row_off = [&](int q) __attribute__((always_inline)) {   // byte offset of row q's first channel of this chunk
    int r = (tid >> 4) + 32 * q;
    r = r < nrows ? r : nrows - 1;
    int m = m0 - a.W - 1 + r;
    m = m < 0 ? 0 : (m < a.M ? m : a.M - 1);       // neighbours that do not exist: any row, never used
    return ((unsigned)m * a.IC + pc * 8) * 2u;
  };
  const int sdst = PITCH + (tid >> 4) * PITCH + pc * 16;
  float* tab = reinterpret_cast<float*>(smem + TAB);
  const wide_rsrc_t rin = wide_rsrc(g_in, (size_t)a.M * a.IC * 2), rw = wide_rsrc(a.wpack, (size_t)9 * a.IC * a.OC * 2);

  // ---- weights: lane = channel l32 of 32, k-octet `half` of a 16-value step; two fragments per step
  const unsigned wlane = ((l32 >> 4) * 64 + half * 16 + (l32 & 15)) * 16;   // bytes
  const unsigned wbase = ((c0 >> 4) + wn * 4) * 1024 + (KPW == 2 ? kg : kg >> 1) * OCB * 1024 + (KPW == 2 ? 0 : (kg & 1) * 512);
  const unsigned tapstep = (a.IC >> 5) * OCB * 1024, slstep = 4 * OCB * 1024;   // bytes per tap, per slice
  uint4 w[RING][2];
  // k16-step s of a kernel row whose weights start at byte offset `base`: tap s / KPW of the row, step s % KPW of the wave's part
#define DDG_HALO_W(slot, s, base)                                                    \
  {                                                                                  \
    const unsigned so = (base) + (unsigned)((s) / KPW) * tapstep + ((s) % KPW) * 512; \
    w[slot][0] = wide_load(rw, wlane, so);                                           \
    w[slot][1] = wide_load(rw, wlane, so + 2048);                                    \
  }

  // everything slice 0 needs is requested at once (its scale and shift directly, the table in LDS serves the
  // later slices); index arithmetic while that is in flight
  const bool from_rows = XFORM && a.rows.partial != nullptr;
  const BnRows rows = second ? a.rows_b : a.rows;
  WideRows<512> sums;
  if (XFORM && from_rows) sums.request(rows, a.IC);
  uint4 first[NU];
#pragma unroll
  for (int q = 0; q < NU; ++q) first[q] = wide_load(rin, row_off(q), 0);
  float sc0[8], sh0[8];
  if (XFORM && !from_rows) {
#pragma unroll
    for (int e = 0; e < 8; e += 4) {
      *reinterpret_cast<float4*>(&sc0[e]) = *reinterpret_cast<const float4*>(g_scale + pc * 8 + e);
      *reinterpret_cast<float4*>(&sh0[e]) = *reinterpret_cast<const float4*>(g_shift + pc * 8 + e);
    }
    for (int c = tid; c < a.IC; c += 512) { tab[c] = g_scale[c]; tab[a.IC + c] = g_shift[c]; }
  }
#pragma unroll
  for (int s = 0; s < RING - 1; ++s) DDG_HALO_W(s, s, wbase)
  if (tid < PITCH / 16) *reinterpret_cast<uint4*>(smem + tid * 16) = make_uint4(0, 0, 0, 0);

  // ---- pixels a lane multiplies: i*32 + l32; bit t: tap t lies inside the image
  int bofs[4];
  int taps[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int p = i * 32 + l32, m = m0 + p < a.M ? m0 + p : a.M - 1;
    const int rem = m % a.HW, h = rem / a.W, x = rem - h * a.W;
    bofs[i] = PITCH + (p + a.W + 1) * PITCH;
    taps[i] = 0;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      const int hh = h + t / 3 - 1, ww = x + t % 3 - 1;
      taps[i] |= (int)((hh >= 0 && hh < a.H && ww >= 0 && ww < a.W ? 1u : 0u) << t);
    }
  }
  const int kofs = kg * KPW * 32 + half * 16;      // byte offset of the wave's first k-step in a row

  if (XFORM && from_rows) {
    sums.finish(rows, a.IC, tab, reinterpret_cast<double*>(smem + PITCH + BUF), blockIdx.x == 0 && blockIdx.y == 0);   // (the other buffer is free)
#pragma unroll
    for (int e = 0; e < 8; e += 4) {
      *reinterpret_cast<float4*>(&sc0[e]) = *reinterpret_cast<const float4*>(&tab[pc * 8 + e]);
      *reinterpret_cast<float4*>(&sh0[e]) = *reinterpret_cast<const float4*>(&tab[a.IC + pc * 8 + e]);
    }
  }
#pragma unroll
  for (int q = 0; q < NU; ++q)
    *reinterpret_cast<uint4*>(smem + sdst + q * 32 * PITCH) = XFORM ? wide_act(first[q], sc0, sh0) : first[q];
  __syncthreads();

  f32x16_t acc[2][4];                              // [32 channels][32 pixels]
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[j][i][e] = 0.f;

  // A trip is one row of the kernel: three taps. The schedule within a trip is spelled out (the compiler, left
  // alone, reads one fragment, waits for it and multiplies): step s requests the pixel fragments of step
  // s+1 and the weights of step s+2, then multiplies. A third of the next slice goes into the other
  // buffer at the end of a trip (free since the barrier that ended slice sl-1), requested one trip
  // earlier; after the last slice that slice is stored once more, into a buffer that nothing reads.
  uint4 f[2][4];
#define DDG_HALO_F(dst, s)                                                           \
  {                                                                                  \
    const int tap = row * 3 + (s) / KPW, sh = ((row - 1) * a.W + (s) / KPW - 1) * PITCH + bufo; /* uniform */ \
    _Pragma("unroll") for (int i = 0; i < 4; ++i) {                                  \
      const int in = __builtin_amdgcn_sbfe(taps[i], tap, 1);                         \
      dst[i] = *reinterpret_cast<const uint4*>(smem + (((bofs[i] + sh) & in) + kofs) + (s) % KPW * 32); \
    }                                                                                \
  }
  uint4 p[2];                                      // this trip's third of the next slice
#pragma unroll
  for (int q = 0; q < 2; ++q) p[q] = wide_load(rin, row_off(q), nsl > 1 ? CS * 2 : 0);
  for (int sl = 0; sl < nsl; ++sl) {
    const int bufo = (sl & 1) * BUF, nxt = sl + 1 < nsl ? sl + 1 : nsl - 1;
#pragma unroll 1
    for (int row = 0; row < 3; ++row) {
      const unsigned wcur = wbase + sl * slstep + row * 3 * tapstep;
      const unsigned wnext = row < 2 ? wcur + 3 * tapstep : wbase + nxt * slstep;
      const int nr = row < 2 ? row + 1 : 0, ns = row < 2 ? nxt : (sl + 2 < nsl ? sl + 2 : nsl - 1);
      uint4 pn[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) pn[q] = wide_load(rin, row_off(2 * nr + q), ns * (CS * 2));
      DDG_HALO_F(f[0], 0)
#pragma unroll
      for (int s = 0; s < SPR; ++s) {
        if (s + 2 < SPR) DDG_HALO_W((s + 2) % RING, s + 2, wcur)
        else DDG_HALO_W((s + 2) % RING, (s + 2) % SPR, wnext)
        if (s + 1 < SPR) DDG_HALO_F(f[(s + 1) & 1], s + 1)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, w[s % RING][j]),
                                                                __builtin_bit_cast(bf16x8_t, f[s & 1][i]), acc[j][i], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
      unsigned char* P = smem + sdst + (BUF - bufo) + row * 64 * PITCH;
      if (XFORM) {
        const int c = nxt * CS + pc * 8;
        float sc[8], sh[8];
        *reinterpret_cast<float4*>(&sc[0]) = *reinterpret_cast<const float4*>(&tab[c]);
        *reinterpret_cast<float4*>(&sc[4]) = *reinterpret_cast<const float4*>(&tab[c + 4]);
        *reinterpret_cast<float4*>(&sh[0]) = *reinterpret_cast<const float4*>(&tab[a.IC + c]);
        *reinterpret_cast<float4*>(&sh[4]) = *reinterpret_cast<const float4*>(&tab[a.IC + c + 4]);
        p[0] = wide_act(p[0], sc, sh); p[1] = wide_act(p[1], sc, sh);
      }
      *reinterpret_cast<uint4*>(P) = p[0];
      *reinterpret_cast<uint4*>(P + 32 * PITCH) = p[1];
      p[0] = pn[0]; p[1] = pn[1];
    }
    __syncthreads();
  }
#undef DDG_HALO_F
#undef DDG_HALO_W

  // what the epilogue reads from memory is requested before the parts meet
  constexpr int CPT = BN / 8, RPP = 512 / CPT, NP = BM / RPP;   // threads per pixel, pixels per pass, passes
  const int oc = tid % CPT, prow = tid / CPT;
  WideTail<STATS> tail;
  typename WideTail<STATS>::Ops ops[NP];
  tail.init(a, c0 + oc * 8);
#pragma unroll
  for (int q = 0; q < NP; ++q) {
    const int m = m0 + prow + q * RPP;
    tail.fetch(a, (size_t)(m < a.M ? m : a.M - 1) * a.OC + c0 + oc * 8, ops[q]);
  }
  // ---- the KG parts as fp32 tiles [KG/2][128 pixels][BN channels]: the upper half of the parts stores, the
  // lower half adds. Accumulator register r of a lane: pixel i*32 + l32, channel (r/4)*8 + half*4 + r%4
  {
    unsigned char* T = smem + (kg % (KG / 2)) * (BM * OROW) + l32 * OROW + (wn * 64 + half * 4) * 4;
    if (kg >= KG / 2) {
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            *reinterpret_cast<f32x4_t*>(T + i * 32 * OROW + j * 128 + q * 32) =
                f32x4_t{acc[j][i][q * 4], acc[j][i][q * 4 + 1], acc[j][i][q * 4 + 2], acc[j][i][q * 4 + 3]};
    }
    __syncthreads();
    if (kg < KG / 2) {
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            f32x4_t* d = reinterpret_cast<f32x4_t*>(T + i * 32 * OROW + j * 128 + q * 32);
            *d = *d + f32x4_t{acc[j][i][q * 4], acc[j][i][q * 4 + 1], acc[j][i][q * 4 + 2], acc[j][i][q * 4 + 3]};
          }
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NP; ++q) {
    const int row = prow + q * RPP, m = m0 + row;
    if (m < a.M) {
      const unsigned char* T = smem + row * OROW + oc * 32;
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = 0.f;
#pragma unroll
      for (int k = 0; k < KG / 2; ++k) {
        const f32x4_t lo = *reinterpret_cast<const f32x4_t*>(T + k * (BM * OROW));
        const f32x4_t hi = *reinterpret_cast<const f32x4_t*>(T + k * (BM * OROW) + 16);
#pragma unroll
        for (int e = 0; e < 4; ++e) { v[e] += lo[e]; v[4 + e] += hi[e]; }
      }
      tail.finish(a, g_out, (size_t)m * a.OC + c0 + oc * 8, ops[q], v);
    }
  }
  if (STATS) {
    __syncthreads();                               // the fp32 tiles have been read
    tail.template store_row<BN>(reinterpret_cast<float*>(smem), g_stat + (size_t)blockIdx.x * 2 * a.OC, a.OC, c0);
  }
}

bool conv_halo_ok(int IC, int W, int R) { return R == 3 && IC % halo::CS == 0 && IC <= halo::ICMAX && W <= halo::WMAX; }
int conv_halo_rows(int M) { return (M + halo::BM - 1) / halo::BM; }

template <int STATS, bool XFORM, int BN>
static hipError_t halo_run(const ConvWideArgs& a, int sets, hipStream_t s) {
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&conv_halo_kernel<STATS, XFORM, BN>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, halo::lds_bytes(BN));
  if (attr != hipSuccess) return attr;
  DDG_LAUNCH((conv_halo_kernel<STATS, XFORM, BN>), dim3(conv_halo_rows(a.M), a.OC / BN, sets), dim3(512), halo::lds_bytes(BN), s, a);
  return hipGetLastError();
}

template <int BN>
static hipError_t halo_dispatch(const ConvWideArgs& a, int sets, int stats, bool xform, hipStream_t s) {
  if (stats == 2) return xform ? hipErrorInvalidValue : halo_run<2, false, BN>(a, sets, s);
  if (stats == 1) return xform ? halo_run<1, true, BN>(a, sets, s) : halo_run<1, false, BN>(a, sets, s);
  return xform ? halo_run<0, true, BN>(a, sets, s) : halo_run<0, false, BN>(a, sets, s);
}

hipError_t conv_halo_launch(const ConvWideArgs& a, int sets, int stats, bool xform, hipStream_t s) {
  if (!conv_halo_ok(a.IC, a.W, a.R) || a.OC % 128 != 0) return hipErrorInvalidValue;
  // 128-channel tiles only where 64-channel tiles would need a second round on the 256 compute units
  const bool wide = (size_t)conv_halo_rows(a.M) * (a.OC / 64) * sets > 256;
  return wide ? halo_dispatch<128>(a, sets, stats, xform, s) : halo_dispatch<64>(a, sets, stats, xform, s);
}

}  // namespace ddg
