// Implicit-GEMM convolution (forward and input-gradient) on CDNA4 matrix cores.
//
// GEMM view: rows = output channels (weights operand), columns = output pixels
// (activation operand), contraction = (tap, input channel). Each wave owns
// MB pixel-blocks x NB channel-blocks of 16x16 accumulators; a lane's accumulator
// registers are 4 consecutive channels of one pixel, so the result is stored NHWC
// with one 8/16-byte store per lane. Activation fragments are gathered straight
// from the NHWC tensor (one 16-byte load of 8 bf16 or 4 fp32 channels of one tap),
// which makes the im2col matrix implicit; zero padding, stride and the
// divisibility test of the input-gradient are folded into the gather predicate.
//
// The forward variant also accumulates per-channel sum and sum of squares of the
// stored outputs (batch-norm statistics) and writes one partial row per workgroup
// in a fixed order, so the statistics are deterministic.
#include "ddg_device.h"
#include "ddg_kernels.h"
#include "ddg_wgrad_vec.h"
#include "ddg_update.h"
#include <cstdlib>

namespace ddg {

// Keeps a loaded fragment alive at the point of its use whatever the predicate says: without it
// the compiler moves the load back under the predicate, which makes it a branch, and every
// branch around a load ends in a wait for all loads in flight.
__device__ __forceinline__ void keep_frag(uint4& f) { asm volatile("" : "+v"(f.x), "+v"(f.y), "+v"(f.z), "+v"(f.w)); }
__device__ __forceinline__ void keep_frag(float4& f) { asm volatile("" : "+v"(f.x), "+v"(f.y), "+v"(f.z), "+v"(f.w)); }

// VEC: the contraction channel count is a multiple of the fragment width (every layer but a
// 3-channel stem): gathers are whole fragments and none of them is conditional.
// Two convolutions of the same tile shape may share a launch (a stage's first 3x3 layer and its projection, which read the
// same input): blockIdx.z = convolution * minibatches + minibatch. A launch that waits for the one before costs 4-5 us
// whatever it does, and these are 5-7 us.
struct ConvPair { ConvArgs c[2]; };

// k-steps whose loads are requested together. The small tiles are those of launches with few waves (conv_plan): such a wave has its SIMD
// nearly to itself and waited for every k-step's loads. 16 -> 16 channels, fp32, 2 x 256 pixels: 6.3 -> 4.3 us; ResNet-20 on 24x24 images, fp32, batch
// 64, 16 iterations 10.9 -> 9.5 ms, 87 fp32 pipelines of two to five modules (20 to 32 wide, batch 16 to 256) 0.938 of the time with a step at a time; bf16:
// conv_plan. Launches with other waves to run would lose their places.
template <typename T, int MB, int NB, bool VEC>
constexpr int conv_batch() { return !VEC ? 1 : Mma<T>::KV == 8 ? (MB * NB <= 2 ? 5 : 1) : (MB * NB == 1 ? 9 : 1); }

// bx of gx, by: this workgroup's index among those that walk over the pixels, its group of channel blocks.
template <typename T, int MB, int NB, bool DGRAD, bool VEC, int KB = conv_batch<T, MB, NB, VEC>()>
__device__ __forceinline__ void conv_mfma_body(const ConvArgs& a, bool second, int bx, int by, int gx) {
  using M_ = Mma<T>;
  using S_ = Store<T>;
  constexpr int KV = M_::KV;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l16 = lane & 15, lg = lane >> 4;
  const int cb0 = by * NB;
  const int OCB = a.OC >> 4;
  // second: the second minibatch of a two-group launch (same weights, own tensors)
  const T* __restrict__ in = reinterpret_cast<const T*>(second ? a.in_b : a.in);
  const T* __restrict__ wp = reinterpret_cast<const T*>(a.wpack);
  T* __restrict__ out = reinterpret_cast<T*>(second ? a.out_b : a.out);
  float* __restrict__ stat_partial = second ? a.stat_partial_b : a.stat_partial;
  const T* __restrict__ addg = reinterpret_cast<const T*>(a.add_g);
  const T* __restrict__ addm = reinterpret_cast<const T*>(a.add_mask);
  const int tiles = (a.M + 16 * MB - 1) / (16 * MB);
  const int ohow = a.OH * a.OW;
  const int cpmask = (1 << a.log2cp) - 1;
  const int sshift = a.stride - 1;  // stride is 1 or 2

  float ssum[NB][4], ssq[NB][4];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int j = 0; j < 4; ++j) { ssum[nb][j] = 0.f; ssq[nb][j] = 0.f; }

  for (int tile = bx * 4 + wave; tile < tiles; tile += gx * 4) {
    int pn[MB], ph[MB], pw[MB];
    bool pv[MB];
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const int m = (tile * MB + i) * 16 + l16;
      pv[i] = m < a.M;
      const int mm = pv[i] ? m : 0;
      const int n = mm / ohow;
      const int rem = mm - n * ohow;
      const int oh = rem / a.OW;
      const int ow = rem - oh * a.OW;
      pn[i] = n;
      if (DGRAD) { ph[i] = oh + a.pad; pw[i] = ow + a.pad; }
      else { ph[i] = oh * a.stride - a.pad; pw[i] = ow * a.stride - a.pad; }
    }
    f32x4_t acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[i][nb] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    // what k-step ks multiplies; a padded or masked position reads the tensor's first elements instead (dropped below)
    auto request = [&](int ks, typename M_::frag_t (&wf)[NB], typename M_::frag_t (&ld)[MB], bool (&okv)[MB]) __attribute__((always_inline)) {
      const int kidx = (ks * 4 + lg) * KV;
      const int tap = kidx >> a.log2cp;
      const int c0 = kidx & cpmask;
      const int r = (a.R == 3) ? tap / 3 : 0;
      const int s = (a.R == 3) ? tap - r * 3 : tap;
      const bool tap_ok = (tap < a.ntaps) && (c0 < a.IC);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        wf[nb] = M_::load(wp + ((size_t)(ks * OCB + cb0 + nb) * 64 + lane) * KV);
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        int ih, iw;
        bool ok = tap_ok && pv[i];
        if (DGRAD) {
          const int th = ph[i] - r, tw = pw[i] - s;
          ok = ok && th >= 0 && tw >= 0 && ((th | tw) & sshift) == 0;
          ih = th >> sshift; iw = tw >> sshift;
          ok = ok && ih < a.IH && iw < a.IW;
        } else {
          ih = ph[i] + r; iw = pw[i] + s;
          ok = ok && ih >= 0 && ih < a.IH && iw >= 0 && iw < a.IW;
        }
        okv[i] = ok;
        if (VEC) {
          const unsigned off = ok ? (unsigned)((pn[i] * a.IH + ih) * a.IW + iw) * (unsigned)a.IC + (unsigned)c0 : 0u;   // (32 bits: the host checks)
          ld[i] = M_::load(in + off);
        } else {
          ld[i] = M_::zero();
          if (ok) {
            const T* p = in + ((size_t)(pn[i] * a.IH + ih) * a.IW + iw) * a.IC + c0;
            if constexpr (KV == 8) {
              // contraction channels not a multiple of 8 (3-channel images): element gather
              uint32_t e[8];
#pragma unroll
              for (int j = 0; j < 8; ++j) e[j] = (c0 + j < a.IC) ? (uint32_t)reinterpret_cast<const uint16_t*>(p)[j] : 0u;
              ld[i] = make_uint4(e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16));
            } else {
              const float* pf = reinterpret_cast<const float*>(p);
              ld[i] = make_float4(pf[0], c0 + 1 < a.IC ? pf[1] : 0.f, c0 + 2 < a.IC ? pf[2] : 0.f, c0 + 3 < a.IC ? pf[3] : 0.f);
            }
          }
        }
      }
    };
    // KB k-steps are requested together (past the last one: that one again, not multiplied)
    for (int k0 = 0; k0 < a.ksteps; k0 += KB) {
      typename M_::frag_t wf[KB][NB], ld[KB][MB];
      bool okv[KB][MB];
#pragma unroll
      for (int k = 0; k < KB; ++k) request(KB == 1 || k0 + k < a.ksteps ? k0 + k : a.ksteps - 1, wf[k], ld[k], okv[k]);
#pragma unroll
      for (int k = 0; k < KB; ++k) {
        if (KB > 1 && k0 + k >= a.ksteps) break;
#pragma unroll
        for (int i = 0; i < MB; ++i) {
          typename M_::frag_t af = ld[k][i];
          if (VEC) {
            keep_frag(af);
            if (!okv[k][i]) af = M_::zero();
          }
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) acc[i][nb] = M_::mma(wf[k][nb], af, acc[i][nb]);
        }
      }
    }

    // epilogue: lane = pixel l16 of block i, channels (cb0+nb)*16 + lg*4 .. +3
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const int m = (tile * MB + i) * 16 + l16;
      if (!pv[i]) continue;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const size_t idx = (size_t)m * a.OC + (cb0 + nb) * 16 + lg * 4;
        float v[4] = {acc[i][nb][0], acc[i][nb][1], acc[i][nb][2], acc[i][nb][3]};
        if (addg) {
          float g[4];
          S_::load4(addg + idx, g);
          if (addm) {
            float mk[4];
            S_::load4(addm + idx, mk);
#pragma unroll
            for (int j = 0; j < 4; ++j) g[j] = (mk[j] > 0.f) ? g[j] : 0.f;
          }
#pragma unroll
          for (int j = 0; j < 4; ++j) v[j] += g[j];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          v[j] = S_::round(v[j]);
          ssum[nb][j] += v[j];
          ssq[nb][j] += v[j] * v[j];
        }
        S_::store4(out + idx, v[0], v[1], v[2], v[3]);
      }
    }
  }

  if (stat_partial) {
    __shared__ float red[4][2][NB * 16];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float s1 = row_sum16(ssum[nb][j]), s2 = row_sum16(ssq[nb][j]);
        if (l16 == 0) {
          red[wave][0][nb * 16 + lg * 4 + j] = s1;
          red[wave][1][nb * 16 + lg * 4 + j] = s2;
        }
      }
    __syncthreads();
    if (threadIdx.x < 2 * NB * 16) {
      const int which = threadIdx.x / (NB * 16), c = threadIdx.x % (NB * 16);
      const float t = ((red[0][which][c] + red[1][which][c]) + red[2][which][c]) + red[3][which][c];
      stat_partial[((size_t)bx * 2 + which) * a.OC + cb0 * 16 + c] = t;
    }
  }
}

template <typename T, int MB, int NB, bool DGRAD, bool VEC, int KB = conv_batch<T, MB, NB, VEC>()>
__global__ __launch_bounds__(256) void conv_mfma_kernel(ConvPair ab, int sets) {
  const int conv = (int)blockIdx.z >= sets ? 1 : 0;
  conv_mfma_body<T, MB, NB, DGRAD, VEC, KB>(ab.c[conv], (int)blockIdx.z != conv * sets, blockIdx.x, blockIdx.y, gridDim.x);
}

// Weight gradient (vector gathers) and input gradient of a layer in one launch: both need its dz and nothing of each
// other, and a launch that waits for the one before costs 4-5 us whatever it does (bwd_generic_ok: how large a layer may be).
template <typename T, int MB, int NB>
__global__ __launch_bounds__(256) void bwd_generic_kernel(WgradArgs w, ConvArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int b = blockIdx.x, nw = w.msplit * (w.Cout / 16);      // (column group slowest, as in a launch of its own)
  if (b < nw * w.jgroups) wgrad_vec_body<T>(w, smem, b % nw % w.msplit, b % nw / w.msplit, b / nw);
  else conv_mfma_body<T, MB, NB, true, true>(a, false, (b - nw * w.jgroups) % a.grid_x, (b - nw * w.jgroups) / a.grid_x, a.grid_x);
}

// Input gradient of a stride-2 convolution (the first block of a stage and its projection). A pixel of the
// input meets only the taps of its parity: 1, 2, 2 or 4 of the nine (1 or none of a 1x1 kernel's one),
// and the kernel above multiplied zeros for the rest and waited for a gather per tap. Here a wave owns
// 16*MB pixels of ONE parity class: its taps are known at compile time, its source pixels are
// neighbours in memory, and a tap's fragments are requested while the tap before is multiplied. The sums
// keep their order (a skipped tap added zero), so results are bit-identical.
// Bound by memory and latency. 3x3 and 1x1 launch together, in a running pipeline: fp32 batch 128, 32 -> 16 channels
// 56 -> 26 us, 64 -> 32 channels 36 -> 18 us.
// PROJ: the launch also carries the gradient that comes through the projection (a.proj_in, a.proj_wpack: a 1x1 kernel, so
// only pixels of even row and column receive any): rounded as a tensor of its own would be, then added. One launch of
// 5 us and a tensor written and read less per stage.
// CPT: k-steps per tap (contraction channels / KSTEP). PR, PC: parity of the pixel's row and column.
template <typename T, int MB, int NB, int CPT, int R, int PR, int PC, bool PROJ>
__device__ __forceinline__ void dgrad_s2_tile(const ConvArgs& a, int tile, int cb0) {
  using M_ = Mma<T>;
  using S_ = Store<T>;
  typedef typename M_::frag_t frag_t;
  constexpr int KV = M_::KV;
  constexpr int NR = R == 3 ? 1 + PR : 1 - PR, NS = R == 3 ? 1 + PC : 1 - PC, NT = NR * NS;   // taps of this class
  const int lane = threadIdx.x & 63, l16 = lane & 15, lg = lane >> 4;
  const int OCB = a.OC >> 4;
  const T* __restrict__ in = reinterpret_cast<const T*>(a.in);
  const T* __restrict__ wp = reinterpret_cast<const T*>(a.wpack);
  T* __restrict__ out = reinterpret_cast<T*>(a.out);
  const T* __restrict__ addg = reinterpret_cast<const T*>(a.add_g);
  const T* __restrict__ addm = reinterpret_cast<const T*>(a.add_mask);
  const int hc = (a.OH + 1 - PR) >> 1, wc = (a.OW + 1 - PC) >> 1, hwc = hc * wc, mc = a.N * hwc;

  int pn[MB], pi[MB], pj[MB];
  bool pv[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    const int p = (tile * MB + i) * 16 + l16;
    pv[i] = p < mc;
    const int pp = pv[i] ? p : 0;
    pn[i] = pp / hwc;
    const int rem = pp - pn[i] * hwc;
    pi[i] = rem / wc; pj[i] = rem - pi[i] * wc;
  }
  f32x4_t acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[i][nb] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  frag_t wf[2][CPT][NB], xf[2][CPT][MB];
  bool ok[2][MB];
  // tap t of the class: kernel row r, column s; source pixel (pi + dh, pj + dw)
#define DDG_S2_TAP(t, set)                                                                         \
  {                                                                                                \
    constexpr int NS1 = NS > 0 ? NS : 1;                                                           \
    const int tr = (t) / NS1, ts = (t) % NS1;                                                      \
    const int r = R == 3 ? (PR ? 2 * tr : 1) : 0, sc = R == 3 ? (PC ? 2 * ts : 1) : 0;             \
    const int dh = R == 3 && PR ? 1 - tr : 0, dw = R == 3 && PC ? 1 - ts : 0;                      \
    _Pragma("unroll") for (int i = 0; i < MB; ++i) {                                               \
      const int ih = pi[i] + dh, iw = pj[i] + dw;                                                  \
      ok[set][i] = pv[i] && ih < a.IH && iw < a.IW;                                                \
      const unsigned off = ok[set][i] ? (unsigned)((pn[i] * a.IH + ih) * a.IW + iw) * (unsigned)a.IC : 0u; \
      _Pragma("unroll") for (int c = 0; c < CPT; ++c)                                              \
        xf[set][c][i] = M_::load(in + (off + (unsigned)((c * 4 + lg) * KV)));                      \
    }                                                                                              \
    _Pragma("unroll") for (int c = 0; c < CPT; ++c)                                                \
      _Pragma("unroll") for (int nb = 0; nb < NB; ++nb)                                            \
        wf[set][c][nb] = M_::load(wp + ((size_t)(((r * R + sc) * CPT + c) * OCB + cb0 + nb) * 64 + lane) * KV); \
  }
  constexpr bool PRJ = PROJ && PR == 0 && PC == 0;
  frag_t pw[PRJ ? CPT : 1][NB], px[PRJ ? CPT : 1][MB];
  if constexpr (PRJ) {     // source pixel (pi, pj), which exists
    const T* __restrict__ pin = reinterpret_cast<const T*>(a.proj_in);
    const T* __restrict__ pwp = reinterpret_cast<const T*>(a.proj_wpack);
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
#pragma unroll
      for (int i = 0; i < MB; ++i)
        px[c][i] = M_::load(pin + ((unsigned)((pn[i] * a.IH + pi[i]) * a.IW + pj[i]) * (unsigned)a.IC + (unsigned)((c * 4 + lg) * KV)));
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) pw[c][nb] = M_::load(pwp + ((size_t)(c * OCB + cb0 + nb) * 64 + lane) * KV);
    }
  }
  if constexpr (NT > 0) DDG_S2_TAP(0, 0)
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if (t + 1 < NT) DDG_S2_TAP(t + 1, (t + 1) & 1)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int c = 0; c < CPT; ++c)
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        frag_t f = xf[t & 1][c][i];
        keep_frag(f);
        if (!ok[t & 1][i]) f = M_::zero();
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[i][nb] = M_::mma(wf[t & 1][c][nb], f, acc[i][nb]);
      }
  }
#undef DDG_S2_TAP
  f32x4_t pacc[PRJ ? MB : 1][NB];
  if constexpr (PRJ) {
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        pacc[i][nb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < CPT; ++c) pacc[i][nb] = M_::mma(pw[c][nb], pv[i] ? px[c][i] : M_::zero(), pacc[i][nb]);
      }
  }

#pragma unroll
  for (int i = 0; i < MB; ++i) {
    if (!pv[i]) continue;
    const size_t m = ((size_t)pn[i] * a.OH + 2 * pi[i] + PR) * a.OW + 2 * pj[i] + PC;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const size_t idx = m * a.OC + (cb0 + nb) * 16 + lg * 4;
      float v[4] = {acc[i][nb][0], acc[i][nb][1], acc[i][nb][2], acc[i][nb][3]};
      if (PROJ) {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] += PRJ ? S_::round(pacc[PRJ ? i : 0][nb][j]) : 0.f;
      }
      if (addg) {
        float g[4];
        S_::load4(addg + idx, g);
        if (addm) {
          float mk[4];
          S_::load4(addm + idx, mk);
#pragma unroll
          for (int j = 0; j < 4; ++j) g[j] = (mk[j] > 0.f) ? g[j] : 0.f;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] += g[j];
      }
      S_::store4(out + idx, S_::round(v[0]), S_::round(v[1]), S_::round(v[2]), S_::round(v[3]));
    }
  }
}

// one wave per tile; the classes with most taps first
struct S2Tiles { int t11, t10, t01, t00; };
template <typename T, int MB, int NB, int CPT, int R, bool PROJ>
__global__ __launch_bounds__(256) void conv_dgrad_s2_kernel(ConvArgs a, S2Tiles t) {
  int tile = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int cb0 = blockIdx.y * NB;
  if (tile < t.t11) { dgrad_s2_tile<T, MB, NB, CPT, R, 1, 1, PROJ>(a, tile, cb0); return; }
  tile -= t.t11;
  if (tile < t.t10) { dgrad_s2_tile<T, MB, NB, CPT, R, 1, 0, PROJ>(a, tile, cb0); return; }
  tile -= t.t10;
  if (tile < t.t01) { dgrad_s2_tile<T, MB, NB, CPT, R, 0, 1, PROJ>(a, tile, cb0); return; }
  tile -= t.t01;
  if (tile < t.t00) dgrad_s2_tile<T, MB, NB, CPT, R, 0, 0, PROJ>(a, tile, cb0);
}

// Covered: whole k-steps per tap (1, 2 or 4 of them: 32-128 channels in bf16, 16-64 in fp32). Two pixel blocks per
// wave once that leaves a wave per SIMD; 32 output channels per wave in bf16 (its matrix instructions are
// cheap, the gathers are not), 16 in fp32.
bool conv_dgrad_s2_ok(const ConvArgs& a) {
  const int kstep = a.dtype == BF16 ? Mma<bf16_t>::KSTEP : Mma<float>::KSTEP;
  if (!a.dgrad || a.stride != 2 || a.stat_partial || a.in_b || (a.R != 1 && a.R != 3) || a.pad != (a.R == 3 ? 1 : 0)) return false;
  if (a.IC % kstep != 0 || (1 << a.log2cp) != a.IC || a.IH != (a.OH + 1) / 2 || a.IW != (a.OW + 1) / 2) return false;
  const int cpt = a.IC / kstep;
  return cpt == 1 || cpt == 2 || cpt == 4;
}

template <typename T>
static bool conv_dgrad_s2_launch(const ConvArgs& a, hipStream_t s) {
  constexpr int KSTEP = Mma<T>::KSTEP;
  if (!conv_dgrad_s2_ok(a)) return false;
  const int cpt = a.IC / KSTEP;
  const int nb = KSTEP == 32 && (a.OC / 16) % 2 == 0 ? 2 : 1, gy = a.OC / 16 / nb;
  const int mb = (size_t)a.M / 32 * gy >= 1024 ? 2 : 1;
  const int h0 = (a.OH + 1) / 2, h1 = a.OH / 2, w0 = (a.OW + 1) / 2, w1 = a.OW / 2;
  auto tiles = [&](int h, int w) { return (a.N * h * w + 16 * mb - 1) / (16 * mb); };
  const S2Tiles t{tiles(h1, w1), tiles(h1, w0), tiles(h0, w1), tiles(h0, w0)};
  const dim3 grid((t.t11 + t.t10 + t.t01 + t.t00 + 3) / 4, gy), block(256);
#define DDG_S2_CASE(MB_, NB_, CPT_)                                                                              \
  if (mb == MB_ && nb == NB_ && cpt == CPT_) {                                                                   \
    if (a.R == 3 && a.proj_in) DDG_LAUNCH((conv_dgrad_s2_kernel<T, MB_, NB_, CPT_, 3, true>), grid, block, 0, s, a, t); \
    else if (a.R == 3) DDG_LAUNCH((conv_dgrad_s2_kernel<T, MB_, NB_, CPT_, 3, false>), grid, block, 0, s, a, t); \
    else DDG_LAUNCH((conv_dgrad_s2_kernel<T, MB_, NB_, CPT_, 1, false>), grid, block, 0, s, a, t);               \
    return true;                                                                                                 \
  }
  DDG_S2_CASE(1, 1, 1) DDG_S2_CASE(1, 1, 2) DDG_S2_CASE(1, 1, 4)
  DDG_S2_CASE(2, 1, 1) DDG_S2_CASE(2, 1, 2) DDG_S2_CASE(2, 1, 4)
  if constexpr (KSTEP == 32) {
    DDG_S2_CASE(1, 2, 1) DDG_S2_CASE(1, 2, 2) DDG_S2_CASE(1, 2, 4)
    DDG_S2_CASE(2, 2, 1) DDG_S2_CASE(2, 2, 2) DDG_S2_CASE(2, 2, 4)
  }
#undef DDG_S2_CASE
  return false;
}

static int ceil_log2(int v) {
  int l = 0;
  while ((1 << l) < v) ++l;
  return l;
}

size_t conv_wpack_elems(int kchannels, int nchannels, int R, int dtype, int* log2cp, int* ksteps) {
  const int kv = mma_kv(dtype);
  int l2 = ceil_log2(kchannels);
  while ((1 << l2) < kv) ++l2;
  const int K = R * R * (1 << l2);
  const int kstep = 4 * kv;
  const int ks = (K + kstep - 1) / kstep;
  if (log2cp) *log2cp = l2;
  if (ksteps) *ksteps = ks;
  return (size_t)ks * (nchannels / 16) * 64 * kv;
}

void conv_plan(ConvArgs& a) {
  const int ocb = a.OC / 16;
  if (ocb % 4 == 0) { a.nb = 4; a.mb = 2; }
  else if (ocb % 2 == 0) { a.nb = 2; a.mb = 2; }
  else { a.nb = 1; a.mb = 4; }
  auto waves = [&](int mb, int nb) { return (long)((a.M + 16 * mb - 1) / (16 * mb)) * (ocb / nb); };
  if (a.dtype == BF16) {
    // a launch of few waves is over when its longest one is: smaller tiles. Forward, fewer channels only: a tile's pixels are those whose statistics a
    // thread adds in fp32, and fewer of them would be another order of sums. ResNet-20, bf16, 16 iterations with wide tiles everywhere, so, and with
    // fewer pixels forward as well: 28x28 images, batch 8 8.84 / 7.50 / 7.22 ms, batch 64 9.77 / 8.79 / 8.64; 32x32, batch 37 4.21 / 4.16 / 4.12.
    if (waves(a.mb, a.nb) < 512) {
      a.nb = 1;
      if (a.dgrad) a.mb = waves(2, 1) < 512 ? 1 : 2;
    }
  } else {
    // fp32 matrix instructions are 16 times slower per flop than bf16 ones: a wave's tile is
    // what bounds the launch, so tiles shrink until there are about two per SIMD
    a.nb = 1; a.mb = 4;
    while (a.mb > 1 && waves(a.mb, 1) < 2048) a.mb /= 2;
  }
  const int gy = ocb / a.nb;
  const int tiles = (a.M + 16 * a.mb - 1) / (16 * a.mb);
  int gx = (tiles + 3) / 4;
  const int cap = 512 / gy > 1 ? 512 / gy : 1;   // also the number of statistics rows
  if (gx > cap) gx = cap;
  if (gx < 1) gx = 1;
  a.grid_x = gx;
}

template <typename T>
static hipError_t conv_dispatch(const ConvArgs& a, const ConvArgs* other, hipStream_t s) {
  const int sets = a.in_b ? 2 : 1;
  dim3 grid(a.grid_x, (a.OC / 16) / a.nb, other ? 2 * sets : sets), block(256);
  const ConvPair ab{{a, other ? *other : a}};
  const bool vec = a.IC % Mma<T>::KV == 0;
  if constexpr (Mma<T>::KV == 4) {
    // A stage's first convolutions of many waves, a k-step at a time: with nine their waves hold 108 registers instead of 40 and what other modules run
    // beside them waits. Networks of ResNet's kind at 32x32, 8 to 32 layers, two or three modules, batch 104 to 136, 77 pipelines: nine everywhere
    // is 1 to 2 % slower than one everywhere in 15 of them, at batch 116 to 128 above all; with this line none is (the worst 0.8 %), and the means are equal. 372 pipelines
    // in all, of one to five modules: 0.06 % shorter with the line, the 88 of one module 0.1 % longer. Stride 1 has no line: it would cost networks at 24x24 and 28x28 1 %
    // in the mean and up to 5 (ResNet-56, batch 64).
    const long waves = (long)a.grid_x * 4 * grid.y * grid.z;
    if (a.mb == 1 && vec && !a.dgrad && a.stride == 2 && waves > 2048) {
      DDG_LAUNCH((conv_mfma_kernel<T, 1, 1, false, true, 1>), grid, block, 0, s, ab, sets);
      return hipGetLastError();
    }
  }
#define DDG_CONV_CASE(MB_, NB_)                                                                   \
  if (a.mb == MB_ && a.nb == NB_) {                                                               \
    if (vec) {                                                                                    \
      if (a.dgrad) DDG_LAUNCH((conv_mfma_kernel<T, MB_, NB_, true, true>), grid, block, 0, s, ab, sets);   \
      else DDG_LAUNCH((conv_mfma_kernel<T, MB_, NB_, false, true>), grid, block, 0, s, ab, sets);          \
    } else {                                                                                      \
      if (a.dgrad) DDG_LAUNCH((conv_mfma_kernel<T, MB_, NB_, true, false>), grid, block, 0, s, ab, sets);  \
      else DDG_LAUNCH((conv_mfma_kernel<T, MB_, NB_, false, false>), grid, block, 0, s, ab, sets);         \
    }                                                                                             \
    return hipGetLastError();                                                                     \
  }
  DDG_CONV_CASE(4, 1)
  DDG_CONV_CASE(2, 1)
  DDG_CONV_CASE(1, 1)
  DDG_CONV_CASE(2, 2)
  DDG_CONV_CASE(2, 4)
#undef DDG_CONV_CASE
  return hipErrorInvalidValue;
}

bool conv_shares_launch(const ConvArgs& a, const ConvArgs& b) {
  return !a.dgrad && !b.dgrad && a.dtype == b.dtype && a.M == b.M && a.IC == b.IC && a.OC == b.OC && a.mb == b.mb && a.nb == b.nb &&
         a.grid_x == b.grid_x;
}

hipError_t conv_launch(const ConvArgs& a, hipStream_t s, const ConvArgs* other) {
  // the gathers form 32-bit element offsets
  if ((size_t)a.N * a.IH * a.IW * a.IC >= ((size_t)1 << 32)) return hipErrorInvalidValue;
  if (other) {
    if (!conv_shares_launch(a, *other) || (a.in_b != nullptr) != (other->in_b != nullptr)) return hipErrorInvalidValue;
    return a.dtype == BF16 ? conv_dispatch<bf16_t>(a, other, s) : conv_dispatch<float>(a, other, s);
  }
  if (a.dtype == BF16 ? conv_dgrad_s2_launch<bf16_t>(a, s) : conv_dgrad_s2_launch<float>(a, s)) return hipGetLastError();
  if (a.proj_in) return hipErrorInvalidValue;   // (the caller asks conv_dgrad_s2_ok)
  if (stem_conv_ok(a)) return stem_conv_launch(a, s);
  return a.dtype == BF16 ? conv_dispatch<bf16_t>(a, nullptr, s) : conv_dispatch<float>(a, nullptr, s);
}

// Alone on the chip the shared launch is 2 to 26 us faster at every size (modules of 4 basic blocks with 16-64 channels at 7-28 wide
// images, batch 32 to 512, and of 2 bottlenecks of 256 to 2048 channels in fp32, batch 1 to 16: 1 to 20 % of a step), and in bf16 pipelines up to
// 7 %. In fp32 it holds the chip's places longer at the weight gradient's registers and LDS (three workgroups a compute unit), and what other
// modules would have run beside it waits: two launches above 3 << 20 gradient values. 48 fp32 pipelines of two to four modules, 20 to 28 wide
// images, batch 64 to 512, time against two launches everywhere: 0.973, without the line 0.980; of these from batch 256 on 0.993 and 1.005.
// Twelve of one module: 0.949 without the line, so it does not hold there (`alone`).
bool bwd_generic_ok(const WgradArgs& w, const ConvArgs& a, bool alone) {
  if (w.dtype != BF16 && !alone && (size_t)w.M * w.Cout > (size_t)3 << 20) return false;
  return w.vec && a.dgrad && !a.proj_in && w.dtype == a.dtype && a.IC % mma_kv(a.dtype) == 0 && !conv_dgrad_s2_ok(a);
}

template <typename T>
static hipError_t bwd_generic_dispatch(const WgradArgs& w, const ConvArgs& a, hipStream_t s) {
  const dim3 grid(w.msplit * (w.Cout / 16) * w.jgroups + a.grid_x * (a.OC / 16 / a.nb));
#define DDG_BWD_CASE(MB_, NB_)                                                                    \
  if (a.mb == MB_ && a.nb == NB_) {                                                               \
    DDG_LAUNCH((bwd_generic_kernel<T, MB_, NB_>), grid, dim3(256), WGV_LDS, s, w, a);             \
    return hipGetLastError();                                                                     \
  }
  DDG_BWD_CASE(4, 1) DDG_BWD_CASE(2, 1) DDG_BWD_CASE(1, 1)
  if constexpr (Mma<T>::KV == 8) { DDG_BWD_CASE(2, 2) DDG_BWD_CASE(2, 4) }
#undef DDG_BWD_CASE
  return hipErrorInvalidValue;
}

hipError_t bwd_generic_launch(const WgradArgs& w, const ConvArgs& a, hipStream_t s) {
  if (!bwd_generic_ok(w, a, true) || a.stat_partial || a.in_b) return hipErrorInvalidValue;
  // 32-bit element offsets inside
  if ((size_t)w.N * w.H * w.W * w.Cin >= ((size_t)1 << 32) || (size_t)w.M * w.Cout >= ((size_t)1 << 32)) return hipErrorInvalidValue;
  return a.dtype == BF16 ? bwd_generic_dispatch<bf16_t>(w, a, s) : bwd_generic_dispatch<float>(w, a, s);
}

// wpack[((ks*OCB + cb)*64 + lane)*KV + j] = W-element for row cb*16+lane%16 and
// contraction index k = (ks*4 + lane/16)*KV + j -> (tap = k >> log2cp, channel = k & (CP-1)).
template <typename T>
__global__ void pack_weights_kernel(const float* __restrict__ W, T* __restrict__ wpack, int Cout,
                                    int Cin, int R, int dgrad, int log2cp, int ksteps, int OCB) {
  constexpr int KV = Mma<T>::KV;
  const size_t total = (size_t)ksteps * OCB * 64 * KV;
  const int kc = dgrad ? Cout : Cin;   // contraction channels
  const int nc = dgrad ? Cin : Cout;   // output channels
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
    const int j = (int)(i % KV);
    const int lane = (int)((i / KV) % 64);
    const int cb = (int)((i / (KV * 64)) % OCB);
    const int ks = (int)(i / ((size_t)KV * 64 * OCB));
    const int k = (ks * 4 + lane / 16) * KV + j;
    const int tap = k >> log2cp, c = k & ((1 << log2cp) - 1);
    const int n = cb * 16 + (lane & 15);
    float v = 0.f;
    if (tap < R * R && c < kc && n < nc) {
      int r = tap / R, s = tap % R;
      if (dgrad == 2) { r = R - 1 - r; s = R - 1 - s; }   // taps mirrored: the input-gradient as a plain correlation
      const int co = dgrad ? c : n, ci = dgrad ? n : c;
      v = W[(((size_t)co * Cin + ci) * R + r) * R + s];
    }
    Store<T>::store1(wpack + i, v);
  }
}

template <typename T>
__global__ __launch_bounds__(256) void pack_all_kernel(const PackDesc* __restrict__ descs) {
  constexpr int KV = Mma<T>::KV;
  const PackDesc d = descs[blockIdx.y];
  const int kc = d.mode ? d.Cout : d.Cin, nc = d.mode ? d.Cin : d.Cout, RR = d.R * d.R;
  T* wpack = reinterpret_cast<T*>(d.wpack);
  // A thread forms one lane's fragment: KV consecutive k of one row, i.e. KV channels of one tap (a
  // tap's channels are padded to a multiple of KV), all requested together, one 16-byte store.
  // (An element per thread, stored two bytes at a time: 109 us for 23 bottleneck blocks; now 84.)
  for (unsigned f = blockIdx.x * blockDim.x + threadIdx.x; f < d.total / KV; f += gridDim.x * blockDim.x) {
    const int lane = (int)(f & 63);
    const int cb = (int)((f >> 6) % (unsigned)d.OCB);
    const int ks = (int)((f >> 6) / (unsigned)d.OCB);
    const int k = (ks * 4 + lane / 16) * KV;
    const int tap = k >> d.log2cp, c = k & ((1 << d.log2cp) - 1);
    const int n = cb * 16 + (lane & 15);
    const int ts = d.mode == 2 ? RR - 1 - tap : tap;      // mirrored taps
    const size_t step = (size_t)(d.mode ? d.Cin : 1) * RR;
    const size_t base = d.mode ? ((size_t)c * d.Cin + n) * RR + ts : ((size_t)n * d.Cin + c) * RR + ts;
    float v[KV];
#pragma unroll
    for (int j = 0; j < KV; ++j) v[j] = (tap < RR && c + j < kc && n < nc) ? d.W[base + j * step] : 0.f;
    Store<T>::store_vec(wpack + (size_t)f * KV, v);
  }
}

hipError_t pack_all_launch(const PackDesc* dev_descs, int n, int dtype, hipStream_t s, unsigned max_total) {
  if (n <= 0) return hipSuccess;
  // workgroups per operand: a fragment per thread of the largest one, at most 256
  const unsigned per = 256u * (unsigned)mma_kv(dtype);
  unsigned bx = (max_total + per - 1) / per;
  bx = bx < 1 ? 16 : (bx > 256 ? 256 : bx);
  if (dtype == BF16) DDG_LAUNCH(pack_all_kernel<bf16_t>, dim3(bx, n), dim3(256), 0, s, dev_descs);
  else DDG_LAUNCH(pack_all_kernel<float>, dim3(bx, n), dim3(256), 0, s, dev_descs);
  return hipGetLastError();
}

// Update and repacking of a small module in one launch: a thread updates a weight in memory order (momentum SGD
// or Adam) and stores the new value where it stands in the two packed
// operands (their padding never changes). Two or three dependent launches of about 5 us each become one (ResNet-20
// fp32 14.32 -> 14.18 ms, bf16 batch 37 6.32 -> 6.22 ms for 16 iterations; a 430 thousand parameter module of
// ResNet-110 even). The stores are scattered, so the line lies where a module's operands stop fitting an XCD's
// 4 MiB L2 with room (UPDATE_PACK_MAX parameters): larger ones go through update_tiles_kernel.
// blockIdx.y: a segment of the parameter vector, `conv` weights (maybe none) followed by `plain` values.
template <typename T, bool ADAM>
__global__ __launch_bounds__(256) void update_pack_kernel(const UpdDesc* __restrict__ descs, UpdArgs a) {
  const UpdDesc d = descs[blockIdx.y];
  UpdStep<ADAM> u;
  u.init(a, gridDim.x * gridDim.y);
  const unsigned n = d.conv + d.plain, RR = (unsigned)(d.R * d.R);
  for (unsigned i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
    const float wn = u.step(a, d.off + i, a.g[d.off + i]);
    if (i >= d.conv) continue;
    const unsigned t = RR == 9 ? i / 9u : i, tap = RR == 9 ? i - t * 9u : 0u;
    const unsigned co = t / d.Cin, ci = t - co * d.Cin;
    upd_pack<T>(d, co, ci, tap, wn);
  }
}

hipError_t update_pack_launch(const UpdDesc* dev_descs, int n, unsigned max_len, const UpdArgs& a, int dtype, bool adam, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  unsigned gx = (max_len + 255) / 256;
  gx = gx < 1 ? 1 : (gx > 64 ? 64 : gx);
  const dim3 grid(gx, n), block(256);
  if (dtype == BF16) {
    if (adam) DDG_LAUNCH((update_pack_kernel<bf16_t, true>), grid, block, 0, s, dev_descs, a);
    else DDG_LAUNCH((update_pack_kernel<bf16_t, false>), grid, block, 0, s, dev_descs, a);
  } else {
    if (adam) DDG_LAUNCH((update_pack_kernel<float, true>), grid, block, 0, s, dev_descs, a);
    else DDG_LAUNCH((update_pack_kernel<float, false>), grid, block, 0, s, dev_descs, a);
  }
  return hipGetLastError();
}

// Update and repacking of a large module (more than UPDATE_PACK_MAX parameters) in one launch, bound by memory: 20 bytes a
// parameter for momentum SGD (28 for Adam) and 4 for two bf16 operands. A workgroup updates a tile of 32 output channels x
// `cols` input channels x all taps with 16-byte accesses in memory order (cols: about 1.1 KB of a row: 32 at 3x3, up to 256
// at 1x1), leaves the new values in LDS and writes from there the fragments of both operands that the tile makes up, 1 KB
// stores a wave. A pass of its own over the weights gathered every fragment from memory, each cache line once per tap
// (25.6 M parameters of 23 bottleneck blocks, 614 MB: 77 + 88 us for the update and that pass, now 102, 6.0 TB/s).
// Layers without whole fragments in a tile (fewer than 32 channels) and values that are no conv weights go element by element.
namespace updt {
constexpr int ROWS = 32, ROWMAX = 288, LDS_FLOATS = ROWS * (ROWMAX + 1);
}
template <typename T, bool ADAM>
__global__ __launch_bounds__(256) void update_tiles_kernel(const UpdDesc* __restrict__ descs, UpdArgs a) {
  using namespace updt;
  constexpr int KV = Mma<T>::KV, KB = 4 * KV, U = 3;
  __shared__ float tile[LDS_FLOATS];
  const UpdDesc d = descs[blockIdx.y];
  UpdStep<ADAM> u;
  u.init(a, gridDim.x * gridDim.y);
  const unsigned RR = (unsigned)(d.R * d.R), tid = threadIdx.x;
  const unsigned first = d.cols ? d.conv : 0;              // element by element from here on
  for (unsigned i = first + blockIdx.x * 256 + tid; i < d.conv + d.plain; i += gridDim.x * 256) {
    const float wn = u.step(a, d.off + i, a.g[d.off + i]);
    if (i >= d.conv) continue;
    const unsigned t = RR == 9 ? i / 9u : i, tap = RR == 9 ? i - t * 9u : 0u;
    const unsigned co = t / d.Cin, ci = t - co * d.Cin;
    upd_pack<T>(d, co, ci, tap, wn);
  }
  if (!d.cols) return;
  const unsigned rowlen = d.Cin * RR, len = d.cols * RR, pitch = len + 1, nu = len / 4;
  const unsigned tcols = d.Cin / d.cols, ntiles = d.conv / (ROWS * len), units = ROWS * nu;
  const unsigned lane = tid & 63, wave = tid >> 6, r16 = lane & 15, kk = (lane >> 4) * KV;
  for (unsigned tl = blockIdx.x; tl < ntiles; tl += gridDim.x) {
    const unsigned co0 = tl / tcols * ROWS, ci0 = (tl % tcols) * d.cols;
    const size_t base = d.off + (size_t)co0 * rowlen + ci0 * RR;
    for (unsigned q0 = tid; q0 < units; q0 += 256 * U) {
      float4 w[U], v[U], m2[U], g[U];
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const unsigned q = q0 + k * 256 < units ? q0 + k * 256 : q0, r = q / nu;
        const size_t e = base + (size_t)r * rowlen + (q - r * nu) * 4;
        w[k] = *reinterpret_cast<const float4*>(a.w + e);
        v[k] = *reinterpret_cast<const float4*>(a.v + e);
        g[k] = *reinterpret_cast<const float4*>(a.g + e);
        if (ADAM) m2[k] = *reinterpret_cast<const float4*>(a.m2 + e);
        else m2[k] = make_float4(0.f, 0.f, 0.f, 0.f);
      }
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const unsigned q = q0 + k * 256;
        if (q >= units) break;
        const unsigned r = q / nu, c = (q - r * nu) * 4;
        const size_t e = base + (size_t)r * rowlen + c;
        w[k].x = u.calc(a, w[k].x, g[k].x, v[k].x, m2[k].x);
        w[k].y = u.calc(a, w[k].y, g[k].y, v[k].y, m2[k].y);
        w[k].z = u.calc(a, w[k].z, g[k].z, v[k].z, m2[k].z);
        w[k].w = u.calc(a, w[k].w, g[k].w, v[k].w, m2[k].w);
        *reinterpret_cast<float4*>(a.w + e) = w[k];
        *reinterpret_cast<float4*>(a.v + e) = v[k];
        if (ADAM) *reinterpret_cast<float4*>(a.m2 + e) = m2[k];
        float* t = tile + r * pitch + c;
        t[0] = w[k].x; t[1] = w[k].y; t[2] = w[k].z; t[3] = w[k].w;
      }
    }
    __syncthreads();
    // fragments: 16 rows x KB contraction channels of one tap. Forward operand: rows are output channels, input gradient: input
    // channels (pitch is odd, so the 16 rows of either fall into distinct banks)
    const unsigned kf = d.cols / KB, nf = 2 * kf * RR, kd = ROWS / KB, nd = d.pack_d ? d.cols / 16 * kd * RR : 0;
    for (unsigned b = wave; b < nf + nd; b += 4) {
      const bool fwd = b < nf;
      const unsigned x = fwd ? b : b - nf, tap = x % RR, y = x / RR, per = fwd ? kf : kd, k0 = y % per * KB, n0 = y / per * 16;
      const float* src = fwd ? tile + (n0 + r16) * pitch + (k0 + kk) * RR + tap : tile + (k0 + kk) * pitch + (n0 + r16) * RR + tap;
      const unsigned stride = fwd ? RR : pitch;
      float o[KV];
#pragma unroll
      for (int j = 0; j < KV; ++j) o[j] = src[j * stride];
      const unsigned k = fwd ? (tap << d.l2f) + ci0 + k0 : ((d.mirror ? RR - 1 - tap : tap) << d.l2d) + co0 + k0;
      const unsigned cb = (fwd ? co0 : ci0) / 16 + n0 / 16;
      Store<T>::store_vec(reinterpret_cast<T*>(fwd ? d.pack_f : d.pack_d) + ((size_t)(k / KB * (fwd ? d.ocb_f : d.ocb_d) + cb) * 64 + lane) * KV, o);
    }
    __syncthreads();                                       // the tile has been read
  }
}

unsigned update_tile_cols(unsigned Cin, unsigned Cout, int R, size_t off) {
  if (Cin % 32 || Cout % 32 || (R != 1 && R != 3) || off % 4) return 0;
  const unsigned most = R == 3 ? 32u : 256u;               // of a row: at most ROWMAX values
  return Cin < most ? Cin : Cin % most ? 32u : most;
}

hipError_t update_tiles_launch(const UpdDesc* dev_descs, int n, unsigned max_len, const UpdArgs& a, int dtype, bool adam, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  // workgroups per segment: a tile (about 9000 values) each of the largest one, at most 128
  unsigned gx = (max_len + 8191) / 8192;
  gx = gx < 1 ? 1 : (gx > 128 ? 128 : gx);
  const dim3 grid(gx, n), block(256);
  if (dtype == BF16) {
    if (adam) DDG_LAUNCH((update_tiles_kernel<bf16_t, true>), grid, block, 0, s, dev_descs, a);
    else DDG_LAUNCH((update_tiles_kernel<bf16_t, false>), grid, block, 0, s, dev_descs, a);
  } else {
    if (adam) DDG_LAUNCH((update_tiles_kernel<float, true>), grid, block, 0, s, dev_descs, a);
    else DDG_LAUNCH((update_tiles_kernel<float, false>), grid, block, 0, s, dev_descs, a);
  }
  return hipGetLastError();
}

hipError_t pack_weights_launch(const float* W, void* wpack, int Cout, int Cin, int R, int dgrad,
                               int dtype, hipStream_t s) {
  int log2cp, ksteps;
  const int kc = dgrad ? Cout : Cin, nc = dgrad ? Cin : Cout;
  const size_t total = conv_wpack_elems(kc, nc, R, dtype, &log2cp, &ksteps);
  int grid = (int)((total + 255) / 256);
  if (grid > 1024) grid = 1024;
  if (dtype == BF16)
    DDG_LAUNCH(pack_weights_kernel<bf16_t>, dim3(grid), dim3(256), 0, s, W,
                       reinterpret_cast<bf16_t*>(wpack), Cout, Cin, R, dgrad, log2cp, ksteps, nc / 16);
  else
    DDG_LAUNCH(pack_weights_kernel<float>, dim3(grid), dim3(256), 0, s, W,
                       reinterpret_cast<float*>(wpack), Cout, Cin, R, dgrad, log2cp, ksteps, nc / 16);
  return hipGetLastError();
}

}  // namespace ddg
