// 1x1 convolution (forward and input gradient) of wide bf16 layers with 128 or 256 contraction channels and a multiple
// of 128 output channels: the expanding layers of a bottleneck block.
//
// Such a layer moves about as many bytes as it multiplies in the time (256 -> 1024 channels, 12544 pixels: 32 MB, 6.6
// GFLOP), and with 64-pixel tiles of their own every workgroup spent most of its life starting and ending. Here the
// weights of 128 output channels stay in registers (a wave: 32 channels x all contraction channels) and the workgroup
// walks over pixels, 64 at a time: the next 64 on their way to registers and the ones after the barrier in the other of
// two LDS buffers while these are multiplied.
//
//   grid:   (pixel groups) x (minibatches) x OC/128 workgroups, at most one per compute unit; the groups share the
//           64-pixel tiles evenly. Workgroups are numbered so that those of one pixel group run on one XCD and find
//           its rows in that L2. One or two statistics rows per pixel group (6272 pixels x 1024 channels: 2*14 for two
//           minibatches, 2*25 for one, where 64-pixel tiles of their own had 98).
//   waves:  4 (32 channels) x 2 (32 pixels), mfma_f32_32x32x16_bf16 with channels as rows. Which channel feeds which row
//           is free, and here lane half h is given channels h*16 .. h*16 + 15, so that a lane's accumulator is 16
//           consecutive channels of one pixel. It goes through LDS (two buffers) so that memory sees 256 bytes per pixel:
//           finished straight from the accumulators, in 16-byte pieces of 32 pixels, the epilogue alone took longer
//           than the whole launch takes now (input gradient 37.6 us).
//   order:  one barrier per 64 pixels. Between two of them tile t is multiplied, tile t-1 finished and stored (what its
//           epilogue reads was requested a tile earlier), tile t+1 put into LDS and tile t+2 requested.
//   sums:   a thread adds the values of eight tiles at most in fp32 (16 additions); from there on, over the threads and
//           over the tiles, everything is added in fp64. A row of several tiles is a larger sum, which fp32 rounds more than
//           rows of a tile each: it is kept in two rows, the sum and what rounding it to fp32 leaves (readers add
//           rows in fp64). So the statistics are no less exact than with a row per 64 pixels, however many pixels there are:
//           against 64 bits, values of a normal distribution, 7 tiles a row: sums 0.3, sums of squares 0.4, of
//           products 0.6 times that error; 43 tiles 0.3, 0.4, 0.6 (in one fp32 row: 3.8, 0.5, 0.9 and 11, 2.8, 1.6).
//
// 256 -> 1024 channels: two minibatches of 6272 pixels with on-load batch norm 22.4 (64-pixel tiles) -> 17.2 us, input
// gradient of one with the sums of the layer below 21.5 -> 17.4; sums in fp64 0.5 more and the same. What bounds it: of the forward launch 3.9 us are start and
// end, the seven tiles 1.9 us each, of which matrix instructions with their fragment reads 0.7, finishing 0.6 and
// staging 0.5: the parts add, two waves a SIMD hide little of each other. The input gradient waits for the three
// tensors of its epilogue (8 us without them). Tried: two tiles in flight (the same), one wave of each SIMD finishing
// before it multiplies (18.1), matrix and vector instructions interleaved by hand (17.8), the activation
// stored by a launch of its own (15.9 and a 6.6 us launch). Since then the forward launch also adds the statistics rows of its
// input (WideRows): 1.6 us more, for a finalise launch of 4.5 before it.
#include "ddg_conv_wide.h"

namespace ddg {

namespace point {
constexpr int BM = 64;
constexpr int pitch(int K) { return K * 2 + 16; }              // bytes per staged pixel: the fragment reads of consecutive lanes fall into distinct banks
constexpr int opitch(int stats) { return stats == 1 ? 128 * 2 + 16 : 128 * 4 + 16; }   // bytes per pixel of a finished tile: as stored, or fp32 where something is added to it
constexpr int RED = 32 * 128 * 4;                              // where sums of the 32 pixel classes meet
constexpr int lds_bytes(int K, int stats) { return 2 * BM * (pitch(K) + opitch(stats)) + (stats ? RED : 0); }
static_assert(512 * 32 + 2 * 256 * 4 <= 2 * BM * opitch(1), "sums and table of the on-load batch norm");
constexpr int CHAIN = 8;                                       // tiles whose values a thread adds in fp32 (a power of two)
}

template <int STATS, bool XFORM, int K>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void conv_point_kernel(ConvWideArgs a, int groups, bool rests) {
  using namespace point;
  constexpr int PITCH = pitch(K), BUF = BM * PITCH, UPR = K / 8, NU = BM * UPR / 512, RPP = 512 / UPR, KS = K / 16;
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  const int wn = wave & 3, wp = wave >> 2;
  const int nct = a.OC >> 7, ntiles = (a.M + BM - 1) / BM;
  int V;
  {
    const int T = gridDim.x, L = blockIdx.x, xcd = L & 7, q = T >> 3, r = T & 7;
    V = xcd * q + (xcd < r ? xcd : r) + (L >> 3);
  }
  const int c0 = (V % nct) * 128;
  int grp = V / nct;
  const bool second = grp >= groups;
  if (second) grp -= groups;
  const int t0 = grp * ntiles / groups, t1 = (grp + 1) * ntiles / groups;
  const bf16_t* __restrict__ g_in = second ? a.in_b : a.in;
  bf16_t* __restrict__ g_out = second ? a.out_b : a.out;
  float* __restrict__ g_stat = second ? a.stat_partial_b : a.stat_partial;
  const float* __restrict__ g_scale = second ? a.scale_b : a.scale;
  const float* __restrict__ g_shift = second ? a.shift_b : a.shift;

  // ---- staging: unit tid + q*512 of a tile = pixel prow + q*RPP, 16-byte chunk pc
  const int pc = tid % UPR, prow = tid / UPR;
  const wide_rsrc_t rin = wide_rsrc(g_in, (size_t)a.M * K * 2), rw = wide_rsrc(a.wpack, (size_t)K * a.OC * 2);
  unsigned src = (unsigned)(t0 * BM + prow) * (K * 2) + pc * 16;
  int left = t1 - t0, mrow = t0 * BM + prow;
  struct Tile { uint4 u[NU]; };
  auto issue = [&](Tile& st) __attribute__((always_inline)) {           // (rows past the tensor and tiles past the group's: zeros, never used)
#pragma unroll
    for (int q = 0; q < NU; ++q) st.u[q] = wide_load(rin, left > 0 && mrow + q * RPP < a.M ? src + q * RPP * (K * 2) : NOWHERE, 0);
    src += BM * K * 2; mrow += BM; --left;
  };
  const bool from_rows = XFORM && a.rows.partial != nullptr;
  const BnRows rows = second ? a.rows_b : a.rows;
  WideRows<512> sums;
  if (XFORM && from_rows) sums.request(rows, K);
  Tile sa;
  issue(sa);
  float sc[8], sh[8];
  if (XFORM && !from_rows) {
#pragma unroll
    for (int e = 0; e < 8; e += 4) {
      *reinterpret_cast<float4*>(&sc[e]) = *reinterpret_cast<const float4*>(g_scale + pc * 8 + e);
      *reinterpret_cast<float4*>(&sh[e]) = *reinterpret_cast<const float4*>(g_shift + pc * 8 + e);
    }
  }
  // ---- weights: matrix row l32 holds channel (l32 >> 2 & 1)*16 + (l32 >> 3)*4 + (l32 & 3) of the wave's 32
  bf16x8_t w[KS];
  {
    const unsigned wl = (((l32 >> 2) & 1) * 64 + half * 16 + (l32 >> 3) * 4 + (l32 & 3)) * 16 + ((c0 >> 4) + wn * 2) * 1024;
    const unsigned kstep = (a.OC >> 4) * 1024;
#pragma unroll
    for (int s = 0; s < KS; ++s) w[s] = __builtin_bit_cast(bf16x8_t, wide_load(rw, wl, (s >> 1) * kstep + (s & 1) * 512));
  }
  if (XFORM && from_rows) {          // (where the finished tiles go later)
    unsigned char* lds = smem + 2 * BUF;
    float* tab = reinterpret_cast<float*>(lds + 512 * 32);
    sums.finish(rows, K, tab, reinterpret_cast<double*>(lds), grp == 0 && c0 == 0);
#pragma unroll
    for (int e = 0; e < 8; e += 4) {
      *reinterpret_cast<float4*>(&sc[e]) = *reinterpret_cast<const float4*>(&tab[pc * 8 + e]);
      *reinterpret_cast<float4*>(&sh[e]) = *reinterpret_cast<const float4*>(&tab[K + pc * 8 + e]);
    }
  }
  auto stash = [&](const Tile& st, int buf) __attribute__((always_inline)) {
    unsigned char* P = smem + buf * BUF + prow * PITCH + pc * 16;
#pragma unroll
    for (int q = 0; q < NU; ++q) *reinterpret_cast<uint4*>(P + q * RPP * PITCH) = XFORM ? wide_act(st.u[q], sc, sh) : st.u[q];
  };
  stash(sa, 0);
  issue(sa);
  __syncthreads();

  // ---- epilogue: thread = pixels orow and orow + 32 of a tile, channels oc*8 .. +7
  constexpr int OP = opitch(STATS), OBUF = BM * OP;
  unsigned char* outb = smem + 2 * BUF;
  const int oc = tid & 15, orow = tid >> 4;
  WideTail<STATS> tail;
  typename WideTail<STATS>::Ops ops[2] = {};
  const wide_rsrc_t rout = wide_rsrc(g_out, (size_t)a.M * a.OC * 2);
  tail.init(a, c0 + oc * 8);
  auto fetch = [&](int t) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int m = t * BM + orow + 32 * q;
      tail.fetch(a, (size_t)(m < a.M ? m : a.M - 1) * a.OC + c0 + oc * 8, ops[q]);
    }
  };
  auto finish = [&](int t) __attribute__((always_inline)) {     // (tile t0 - 1: nothing)
    const unsigned char* T = outb + ((t - t0) & 1) * OBUF + orow * OP;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int m = t * BM + orow + 32 * q;
      float v[8];
      if (STATS == 1) {
        Store<bf16_t>::unpack_vec(*reinterpret_cast<const uint4*>(T + q * 32 * OP + oc * 16), v);
      } else {
        *reinterpret_cast<float4*>(&v[0]) = *reinterpret_cast<const float4*>(T + q * 32 * OP + oc * 32);
        *reinterpret_cast<float4*>(&v[4]) = *reinterpret_cast<const float4*>(T + q * 32 * OP + oc * 32 + 16);
      }
      const bool ok = t >= t0 && m < a.M;
      const uint4 o = tail.result(a, ops[q], v, ok);
      wide_store(rout, o, ok ? (unsigned)m * (unsigned)(a.OC * 2) + (c0 + oc * 8) * 2 : NOWHERE);
    }
  };
  // the threads' sums so far, by thread: channel tid & 127, pixel classes (tid >> 7)*8 .. +7
  double tot[2] = {0.0, 0.0};
  unsigned char* redb = smem + 2 * (BUF + OBUF);
  auto gather = [&]() __attribute__((always_inline)) {
    float* red = reinterpret_cast<float*>(redb);
#pragma unroll
    for (int w = 0; w < 2; ++w) {
      float (&v)[8] = w ? tail.ssq : tail.ssum;
#pragma unroll
      for (int e = 0; e < 8; e += 4) *reinterpret_cast<float4*>(&red[orow * 128 + oc * 8 + e]) = make_float4(v[e], v[e + 1], v[e + 2], v[e + 3]);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = 0.f;
      __syncthreads();
#pragma unroll
      for (int r = 0; r < 8; ++r) tot[w] += (double)red[((tid >> 7) * 8 + r) * 128 + (tid & 127)];
      __syncthreads();
    }
  };
  const int frag = (wp * 32 + l32) * PITCH + half * 16;
  const int odst = (wp * 32 + l32) * OP + (wn * 32 + half * 16) * (STATS == 1 ? 2 : 4);
  for (int t = t0; t < t1; ++t) {
    f32x16_t acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    const unsigned char* B = smem + ((t - t0) & 1) * BUF + frag;
#pragma unroll
    for (int s = 0; s < KS; ++s)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[s], *reinterpret_cast<const bf16x8_t*>(B + s * 32), acc, 0, 0, 0);
    finish(t - 1);
    if (STATS && ((t - t0) & (CHAIN - 1)) == CHAIN - 1) gather();
    fetch(t);
    stash(sa, (t + 1 - t0) & 1);                   // (free since the barrier that ended tile t-1)
    issue(sa);
    // register r of a lane: pixel wp*32 + l32, channel wn*32 + half*16 + r
    unsigned char* O = outb + ((t - t0) & 1) * OBUF + odst;
    if (STATS == 1) {
#pragma unroll
      for (int p = 0; p < 2; ++p)
        *reinterpret_cast<uint4*>(O + p * 16) =
            make_uint4(Store<bf16_t>::pack2(acc[p * 8], acc[p * 8 + 1]), Store<bf16_t>::pack2(acc[p * 8 + 2], acc[p * 8 + 3]),
                       Store<bf16_t>::pack2(acc[p * 8 + 4], acc[p * 8 + 5]), Store<bf16_t>::pack2(acc[p * 8 + 6], acc[p * 8 + 7]));
    } else {
#pragma unroll
      for (int p = 0; p < 4; ++p)
        *reinterpret_cast<f32x4_t*>(O + p * 16) = f32x4_t{acc[p * 4], acc[p * 4 + 1], acc[p * 4 + 2], acc[p * 4 + 3]};
    }
    __syncthreads();
  }
  finish(t1 - 1);
  if (STATS) {
    gather();
    double* red = reinterpret_cast<double*>(redb);         // [quarter of the classes][2][128]
#pragma unroll
    for (int w = 0; w < 2; ++w) red[((tid >> 7) * 2 + w) * 128 + (tid & 127)] = tot[w];
    __syncthreads();
    if (tid < 256) {
      const double t = (red[tid] + red[256 + tid]) + (red[512 + tid] + red[768 + tid]);
      const size_t at = (size_t)(tid >> 7) * a.OC + c0 + (tid & 127);
      const float sum = (float)t, rest = (float)(t - (double)sum);
      g_stat[(size_t)grp * 2 * a.OC + at] = sum;
      // (an infinite sum has no rest)
      if (rests) g_stat[(size_t)(groups + grp) * 2 * a.OC + at] = fabsf(rest) <= 3.4e38f ? rest : 0.f;
    }
  }
}

bool conv_point_ok(int IC, int R) { return R == 1 && (IC == 128 || IC == 256); }
// Pixel groups per minibatch: as many as keep the launch at one workgroup per compute unit, and no more than share the
// longest group's tiles.
int conv_point_groups(int M, int OC, int sets) {
  const int tiles = (M + point::BM - 1) / point::BM;
  int g = 256 / ((OC / 128) * sets);
  g = g < 1 ? 1 : g > tiles ? tiles : g;
  const int most = (tiles + g - 1) / g;
  return (tiles + most - 1) / most;
}
int conv_point_rows(int M, int OC, int sets) {     // (a group of one tile rounds its sum as a row per tile always has been)
  const int groups = conv_point_groups(M, OC, sets);
  return groups < (M + point::BM - 1) / point::BM ? 2 * groups : groups;
}

template <int STATS, bool XFORM, int K>
static hipError_t point_run(const ConvWideArgs& a, int sets, hipStream_t s) {
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&conv_point_kernel<STATS, XFORM, K>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, point::lds_bytes(K, STATS));
  if (attr != hipSuccess) return attr;
  static_assert(point::lds_bytes(K, STATS) <= 160 * 1024, "one compute unit's LDS");
  const int groups = conv_point_groups(a.M, a.OC, sets);
  DDG_LAUNCH((conv_point_kernel<STATS, XFORM, K>), dim3(groups * sets * (a.OC / 128)), dim3(512), point::lds_bytes(K, STATS), s, a, groups,
             conv_point_rows(a.M, a.OC, sets) > groups);
  return hipGetLastError();
}

template <int K>
static hipError_t point_dispatch(const ConvWideArgs& a, int sets, int stats, bool xform, hipStream_t s) {
  if (stats == 2) return xform ? hipErrorInvalidValue : point_run<2, false, K>(a, sets, s);
  if (stats == 1) return xform ? point_run<1, true, K>(a, sets, s) : point_run<1, false, K>(a, sets, s);
  return xform ? hipErrorInvalidValue : point_run<0, false, K>(a, sets, s);    // (a forward pass always keeps its statistics)
}

hipError_t conv_point_launch(const ConvWideArgs& a, int sets, int stats, bool xform, hipStream_t s) {
  if (!conv_point_ok(a.IC, a.R) || a.OC % 128 != 0) return hipErrorInvalidValue;
  return a.IC == 256 ? point_dispatch<256>(a, sets, stats, xform, s) : point_dispatch<128>(a, sets, stats, xform, s);
}

}  // namespace ddg
