// First 1x1 layer of a bottleneck block (IC -> OC channels, IC a power of two from 256 to 2048, OC = 128 or 256; one or both
// minibatches of a training forward pass) that forms its own input: y = relu(bn(z) + x), the output of the block before, from that block's last convolution output z
// and its input x, and stores it.
//
// As a pass of its own the normalise-add-ReLU of a wide block moves three tensors and the convolution reads the result
// again. Here a workgroup owns 64 pixels and ALL output channels, so that every element is formed once:
//
//   waves 8-11: z and x, 16-byte loads four chunks of 64 channels ahead (64 KB in flight a workgroup; the launch is bound by
//             memory), form y, store it and leave it in LDS. Loads complete in order, so a wave that also waited for weights from
//             L2 would wait for everything it had requested from memory before them (29.6 us)
//   batch norm: the workgroup adds the producer's statistics rows itself (fp64; 32 sums at most, in as
//             many rows or, behind conv_point_kernel, twice as many), so there is no launch in between; workgroup 0 stores the vectors
//   pixels:   a chunk at a time through two LDS buffers, one barrier a chunk
//   weights:  fragments straight from the packed operand into the registers of the wave that uses them, two chunks ahead
//   waves 0-7: OC/32 (32 channels) x 256/OC (32 or 64 pixels) with mfma_f32_32x32x16_bf16, rows fed as in conv_point_kernel
//
// Bottleneck stage of 23 blocks, batch 32, 1024 -> 256 at 14x14, two minibatches (77 MB moved): 26.9 us, for 14.8 (normalise-add-
// ReLU) + 16.8 (conv_wide_kernel); a training step 4.39 -> 4.25 ms. Workgroups that all start at the same columns: 29.0. Every
// wave loading both kinds of operand: 29.6. With a rest beside each sum, 28 rows instead of 14, it takes
// 1.7 us more (2.6 with 8 rows in flight instead of 16). Without the sums' prologue it would take 3 us less, without multiplying 2, without
// loading z and x 8; weights four chunks ahead do not fit the registers (spills: 32.4).
#include "ddg_conv_wide.h"

namespace ddg {

namespace form {
constexpr int BM = 64, CK = 64, DEPTH = 4;
constexpr int PITCH = CK * 2 + 16, BUF = BM * PITCH;
constexpr int ICMAX = 2048, SUMS_MAX = 32;
constexpr int opitch(int OC) { return OC * 2 + 16; }
constexpr int max3(int a, int b, int c) { return a > b ? (a > c ? a : c) : (b > c ? b : c); }
// the table of scales and shifts; then the chunks, later the finished tile, later the sums per row class
constexpr int lds_bytes(int OC, int IC) { return IC * 8 + max3(2 * BUF, BM * opitch(OC), 2 * OC * (4096 / OC) * 4); }
}

template <int OC>
__global__ __launch_bounds__(768) __attribute__((amdgpu_waves_per_eu(3, 3))) void conv_form_kernel(ConvWideArgs a, FormSet f0, FormSet f1) {
  using namespace form;
  constexpr int NCG = OC / 32, NPG = 8 / NCG, NI = BM / NPG / 32;   // channel groups, pixel groups, 32-pixel blocks of a wave
  constexpr int KS = CK / 16;
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  const int wn = wave % NCG, wp = wave / NCG;
  const bool second = blockIdx.z != 0;
  const FormSet& f = second ? f1 : f0;
  bf16_t* __restrict__ g_out = second ? a.out_b : a.out;
  float* __restrict__ g_stat = second ? a.stat_partial_b : a.stat_partial;
  const int m0 = blockIdx.x * BM, IC = a.IC, nch = IC / CK;
  float* s_sc = reinterpret_cast<float*>(smem);
  float* s_sh = s_sc + IC;
  unsigned char* pix = smem + IC * 8;

  // ---- waves 8-11: pixels pr and pr + 32 of a chunk, channels pc*8 ..
  const bool producer = wave >= 8;
  const int pt = tid & 255, pc = pt & 7, pr = pt >> 3;
  const size_t bytes = (size_t)a.M * IC * 2;
  const wide_rsrc_t rz = wide_rsrc(f.z, bytes), rr = wide_rsrc(f.res, bytes), ry = wide_rsrc(f.y, bytes);
  const wide_rsrc_t rw = wide_rsrc(a.wpack, (size_t)IC * OC * 2);
  // The chunk that workgroup b starts with: rows of IC channels are a multiple of 512 bytes apart, so workgroups that all read
  // the same columns of their rows would all be at the same few memory channels.
  const int rot = (int)(blockIdx.x + blockIdx.x / 8);
  auto turned = [&](int chunk) __attribute__((always_inline)) { return (chunk + rot) & (nch - 1); };
  auto at = [&](int chunk, int q) __attribute__((always_inline)) {   // byte offset of the thread's unit q of a chunk
    const int m = m0 + pr + 32 * q;
    return m < a.M && chunk < nch ? ((unsigned)m * IC + pc * 8 + turned(chunk) * CK) * 2u : NOWHERE;
  };
  uint4 zq[DEPTH][2], rq[DEPTH][2];
  // ---- weights: matrix row l32 holds channel (l32 >> 2 & 1)*16 + (l32 >> 3)*4 + (l32 & 3) of the wave's 32
  const unsigned wl = (((l32 >> 2) & 1) * 64 + half * 16 + (l32 >> 3) * 4 + (l32 & 3)) * 16 + wn * 2048;
  constexpr unsigned kstep = (OC / 16) * 1024;                   // bytes per 32 contraction channels of the operand
  bf16x8_t w[2][KS];
#define DDG_FORM_W(slot, chunk)                                                       \
  {                                                                                   \
    _Pragma("unroll") for (int s = 0; s < KS; ++s)                                    \
      w[slot][s] = __builtin_bit_cast(bf16x8_t, wide_load(rw, wl, (turned(chunk) * (CK / 32) + (s >> 1)) * kstep + (s & 1) * 512)); \
  }
  if (producer) {
#pragma unroll
    for (int j = 0; j < DEPTH; ++j)
#pragma unroll
      for (int q = 0; q < 2; ++q) { zq[j][q] = wide_load(rz, at(j, q), 0); rq[j][q] = wide_load(rr, at(j, q), 0); }
  } else {
    DDG_FORM_W(0, 0)
    DDG_FORM_W(1, 1)
    // scale and shift of all input channels, here because the other waves' registers are full of z and x: 16 rows in flight
    for (int c = tid * 2; c < IC; c += 1024) {
      constexpr int RU = 16;
      const float2 gm = *reinterpret_cast<const float2*>(f.rows.gamma + c), bt = *reinterpret_cast<const float2*>(f.rows.beta + c);
      double s0 = 0.0, s1 = 0.0, q0 = 0.0, q1 = 0.0;
      for (int r0 = 0; r0 < f.rows.rows; r0 += RU) {
        float2 sv[RU], qv[RU];
#pragma unroll
        for (int r = 0; r < RU; ++r) {
          const float* p = f.rows.partial + (size_t)(r0 + r < f.rows.rows ? r0 + r : f.rows.rows - 1) * 2 * IC + c;
          sv[r] = *reinterpret_cast<const float2*>(p);
          qv[r] = *reinterpret_cast<const float2*>(p + IC);
        }
#pragma unroll
        for (int r = 0; r < RU; ++r) {
          const bool on = r0 + r < f.rows.rows;
          s0 += (double)(on ? sv[r].x : 0.f); s1 += (double)(on ? sv[r].y : 0.f);
          q0 += (double)(on ? qv[r].x : 0.f); q1 += (double)(on ? qv[r].y : 0.f);
        }
      }
      auto put = [&](int ch, double t1, double t2, float gamma, float beta) __attribute__((always_inline)) {
        const double mu = t1 * f.rows.inv_count;
        double var = t2 * f.rows.inv_count - mu * mu;
        if (var < 0.0) var = 0.0;
        const float is = (float)rsqrt(var + (double)f.rows.eps), sc = gamma * is, sh = beta - (float)mu * sc;
        s_sc[ch] = sc; s_sh[ch] = sh;
        if (blockIdx.x == 0) { f.rows.mean[ch] = (float)mu; f.rows.invstd[ch] = is; f.rows.scale[ch] = sc; f.rows.shift[ch] = sh; }
      };
      put(c, s0, q0, gm.x, bt.x);
      put(c + 1, s1, q1, gm.y, bt.y);
    }
  }
  __syncthreads();

  f32x16_t acc[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
  const int dst = pr * PITCH + pc * 16, frag = (wp * NI * 32 + l32) * PITCH + half * 16;
  // chunk `chunk` from its registers (slot j) into LDS and memory; the chunk DEPTH later requested into them
#define DDG_FORM_CHUNK(j, chunk)                                                                              \
  {                                                                                                           \
    const int c = turned(chunk) * CK + pc * 8;                                                                      \
    float sc[8], sh[8];                                                                                       \
    *reinterpret_cast<float4*>(&sc[0]) = *reinterpret_cast<const float4*>(&s_sc[c]);                          \
    *reinterpret_cast<float4*>(&sc[4]) = *reinterpret_cast<const float4*>(&s_sc[c + 4]);                      \
    *reinterpret_cast<float4*>(&sh[0]) = *reinterpret_cast<const float4*>(&s_sh[c]);                          \
    *reinterpret_cast<float4*>(&sh[4]) = *reinterpret_cast<const float4*>(&s_sh[c + 4]);                      \
    _Pragma("unroll") for (int q = 0; q < 2; ++q) {                                                           \
      float v[8], r[8];                                                                                       \
      Store<bf16_t>::unpack_vec(zq[j][q], v);                                                                 \
      Store<bf16_t>::unpack_vec(rq[j][q], r);                                                                 \
      _Pragma("unroll") for (int e = 0; e < 8; ++e) { const float t = v[e] * sc[e] + sh[e] + r[e]; v[e] = t > 0.f ? t : 0.f; } \
      uint4 o;                                                                                                \
      o.x = Store<bf16_t>::pack2(v[0], v[1]); o.y = Store<bf16_t>::pack2(v[2], v[3]);                         \
      o.z = Store<bf16_t>::pack2(v[4], v[5]); o.w = Store<bf16_t>::pack2(v[6], v[7]);                         \
      *reinterpret_cast<uint4*>(pix + ((j) & 1) * BUF + dst + q * 32 * PITCH) = o;                            \
      wide_store(ry, o, at(chunk, q));                                                                        \
      zq[j][q] = wide_load(rz, at((chunk) + DEPTH, q), 0);       /* (past the end: zeros, never used) */      \
      rq[j][q] = wide_load(rr, at((chunk) + DEPTH, q), 0);                                                    \
    }                                                                                                         \
  }
  // Both kinds of waves pass the same barriers: one here, one per chunk. Between two of them chunk n is multiplied and chunk
  // n+1 put into the other buffer.
  if (producer) {
    DDG_FORM_CHUNK(0, 0)
    __syncthreads();
    for (int cb = 0; cb < nch; cb += DEPTH) {
#pragma unroll
      for (int j = 0; j < DEPTH; ++j) {
        if (cb + j + 1 < nch) DDG_FORM_CHUNK((j + 1) % DEPTH, cb + j + 1)
        __syncthreads();
      }
    }
  } else {
    __syncthreads();
    for (int cb = 0; cb < nch; cb += DEPTH) {
#pragma unroll
      for (int j = 0; j < DEPTH; ++j) {
        const unsigned char* B = pix + (j & 1) * BUF + frag;
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
          for (int i = 0; i < NI; ++i)
            acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[j & 1][s], *reinterpret_cast<const bf16x8_t*>(B + i * 32 * PITCH + s * 32), acc[i], 0, 0, 0);
        const int nw = cb + j + 2 < nch ? cb + j + 2 : nch - 1;  // (past the end: the last chunk, never used)
        DDG_FORM_W(j & 1, nw)
        __syncthreads();
      }
    }
  }
#undef DDG_FORM_CHUNK
#undef DDG_FORM_W

  // ---- epilogue: register r of a lane holds pixel (wp*NI + i)*32 + l32, channel wn*32 + half*16 + r
  constexpr int OP = opitch(OC), CPT = OC / 8, RPP = 512 / CPT, NP = BM / RPP;   // threads per pixel, pixels per pass, passes
  if (!producer) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      unsigned char* O = pix + ((wp * NI + i) * 32 + l32) * OP + (wn * 32 + half * 16) * 2;
#pragma unroll
      for (int p = 0; p < 2; ++p)
        *reinterpret_cast<uint4*>(O + p * 16) =
            make_uint4(Store<bf16_t>::pack2(acc[i][p * 8], acc[i][p * 8 + 1]), Store<bf16_t>::pack2(acc[i][p * 8 + 2], acc[i][p * 8 + 3]),
                       Store<bf16_t>::pack2(acc[i][p * 8 + 4], acc[i][p * 8 + 5]), Store<bf16_t>::pack2(acc[i][p * 8 + 6], acc[i][p * 8 + 7]));
    }
  }
  __syncthreads();
  // thread (of the first 512) = pixels prow + q*RPP, channels oc*8 ..; sums of the stored values over its pixels
  const int oc = tid % CPT, prow = (tid & 511) / CPT;
  float sum[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) sum[e] = 0.f;
  if (!producer) {
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      const int row = prow + q * RPP, m = m0 + row;
      if (m < a.M) {
        const uint4 o = *reinterpret_cast<const uint4*>(pix + row * OP + oc * 16);
        float r[8];
        Store<bf16_t>::unpack_vec(o, r);
#pragma unroll
        for (int e = 0; e < 8; ++e) { sum[e] += r[e]; sum[8 + e] += r[e] * r[e]; }
        *reinterpret_cast<uint4*>(g_out + (size_t)m * OC + oc * 8) = o;
      }
    }
  }
  __syncthreads();                                 // the tile has been read
  float* red = reinterpret_cast<float*>(pix);      // [row class][2][OC]
  if (!producer) {
#pragma unroll
    for (int e = 0; e < 16; e += 4)
      *reinterpret_cast<float4*>(&red[(prow * 2 + e / 8) * OC + oc * 8 + e % 8]) = make_float4(sum[e], sum[e + 1], sum[e + 2], sum[e + 3]);
  }
  __syncthreads();
  if (tid < 2 * OC) {                              // the row classes in order
    float t = 0.f;
#pragma unroll
    for (int r = 0; r < RPP; ++r) t += red[r * 2 * OC + tid];
    g_stat[(size_t)blockIdx.x * 2 * OC + tid] = t;
  }
}

bool conv_form_ok(int IC, int OC, int R, int sums) {
  return R == 1 && (OC == 128 || OC == 256) && IC % (form::CK * form::DEPTH) == 0 && (IC & (IC - 1)) == 0 && IC <= form::ICMAX && sums >= 1 && sums <= form::SUMS_MAX;
}

template <int OC>
static hipError_t form_run(const ConvWideArgs& a, const FormSet& f0, const FormSet& f1, int sets, hipStream_t s) {
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&conv_form_kernel<OC>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, form::lds_bytes(OC, form::ICMAX));
  if (attr != hipSuccess) return attr;
  DDG_LAUNCH((conv_form_kernel<OC>), dim3((a.M + form::BM - 1) / form::BM, 1, sets), dim3(768), form::lds_bytes(OC, a.IC), s, a, f0, f1);
  return hipGetLastError();
}

hipError_t conv_form_launch(const FormSet& f0, const FormSet* f1, const void* wpack, void* out, float* stat_partial, void* out_b, float* stat_partial_b,
                            int N, int H, int W, int IC, int OC, hipStream_t s) {
  const size_t M = (size_t)N * H * W;
  auto sums = [](const FormSet& f) { return (f.rows.rows + 1) / 2; };   // (at least: each may have a rest)
  if (!conv_form_ok(IC, OC, 1, sums(f0)) || (f1 && !conv_form_ok(IC, OC, 1, sums(*f1)))) return hipErrorInvalidValue;
  if (M * (size_t)(IC > OC ? IC : OC) >= ((size_t)1 << 31)) return hipErrorInvalidValue;   // 32-bit byte offsets inside
  ConvWideArgs a{};
  a.wpack = (const bf16_t*)wpack; a.out = (bf16_t*)out; a.stat_partial = stat_partial; a.out_b = (bf16_t*)out_b; a.stat_partial_b = stat_partial_b;
  a.M = (int)M; a.H = H; a.W = W; a.HW = H * W; a.IC = IC; a.OC = OC; a.R = 1;
  const FormSet& b = f1 ? *f1 : f0;
  return OC == 128 ? form_run<128>(a, f0, b, f1 ? 2 : 1, s) : form_run<256>(a, f0, b, f1 ? 2 : 1, s);
}

}  // namespace ddg
