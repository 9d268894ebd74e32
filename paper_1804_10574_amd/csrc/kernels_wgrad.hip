// Weight-gradient convolution: dW[co][tap][ci] = sum over pixels m of dz[m][co] * x[pix(m,tap)][ci].
//
// The contraction runs over pixels, which are the slow index of both NHWC operands, so
// this version feeds the fp32 matrix-core atom (one element per lane, no transposition
// needed): rows = output channels, columns = (tap, input channel), k = 4 pixels per
// instruction. bf16 tensors are widened on load; products of bf16 values are exact in fp32.
// Work is split over pixel ranges; each workgroup writes one partial tile and a second
// kernel adds the partials in a fixed order (no atomics: results are reproducible).
#include "ddg_device.h"
#include "ddg_kernels.h"
#include "ddg_wgrad_vec.h"
#include "ddg_update.h"
#include <cstdlib>
#include <type_traits>

namespace ddg {

constexpr int WG_NJ = 9;  // column blocks (16 wide) per wave at most

// NJ: column blocks per wave, 3 for the stem (3 channels padded to 4, 36 columns; with 9 two thirds of the
// gathers and matrix instructions were padding). As in the kernel below nothing in the loop is conditional and
// the loads of step st+3 are requested before step st is multiplied. Stem, 3 -> 16 channels, in a running
// pipeline: bf16 batch 256 60 -> 25 us, fp32 batch 128 24 -> 13 us. (Stems of 3 channels run in stem_wgrad_kernel since, where a
// workgroup's pixels fit LDS; wide rows and more than 0.4 to 1.5 M pixels come here.)
template <typename T, int NJ>
__global__ __launch_bounds__(256) void wgrad_mfma_kernel(WgradArgs a) {
  using S_ = Store<T>;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l16 = lane & 15, lg = lane >> 4;
  const int cob = blockIdx.y;
  const int jb0 = blockIdx.z * WG_NJ;
  const T* __restrict__ x = reinterpret_cast<const T*>(a.x);
  const T* __restrict__ dz = reinterpret_cast<const T*>(a.dz);
  const int cpmask = (1 << a.log2cp) - 1;
  const int ntaps = a.R * a.R;

  // per-lane column descriptors: column j -> (tap, ci)
  int jr[NJ], js[NJ], jc[NJ];
  bool jv[NJ];
#pragma unroll
  for (int b = 0; b < NJ; ++b) {
    const int j = (jb0 + b) * 16 + l16;
    const int tap = j >> a.log2cp;
    jc[b] = j & cpmask;
    jr[b] = tap / a.R - a.pad;
    js[b] = tap % a.R - a.pad;
    jv[b] = (jb0 + b) < a.JB && tap < ntaps && jc[b] < a.Cin;
  }
  f32x4_t acc[NJ];
#pragma unroll
  for (int b = 0; b < NJ; ++b) acc[b] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const int pq = a.P * a.Q;
  const bool fdiv = a.M < (1 << 22);
  const float inv_pq = 1.0f / (float)pq, inv_q = 1.0f / (float)a.Q;
  long m0 = ((long)blockIdx.x * 4 + wave) * (long)a.steps * 4;
  struct StepRegs { float dv; float xv[NJ]; unsigned ok; };   // ok bit b: column block b valid, bit 31: pixel valid
  auto issue = [&](StepRegs& r, int st) __attribute__((always_inline)) {
    const long m = m0 + (long)st * 4 + lg;
    const bool mv = st < a.steps && m < a.M;
    const int mm = mv ? (int)m : 0;
    // (small non-negative integers divide exactly through fp32; an integer division costs as
    // much as the step's matrix instructions)
    const int n = fdiv ? (int)(((float)mm + 0.5f) * inv_pq) : mm / pq;
    const int rem = mm - n * pq;
    const int p = fdiv ? (int)(((float)rem + 0.5f) * inv_q) : rem / a.Q;
    const int q = rem - p * a.Q;
    r.dv = S_::load1(dz + (size_t)mm * a.Cout + cob * 16 + l16);
    const int ihb = p * a.stride, iwb = q * a.stride;
    unsigned okb = mv ? 0x80000000u : 0u;
#pragma unroll
    for (int b = 0; b < NJ; ++b) {
      const int ih = ihb + jr[b], iw = iwb + js[b];
      const bool ok = mv && jv[b] && ih >= 0 && ih < a.H && iw >= 0 && iw < a.W;
      r.xv[b] = S_::load1(x + (ok ? ((size_t)(n * a.H + ih) * a.W + iw) * a.Cin + jc[b] : (size_t)0));
      okb |= (ok ? 1u : 0u) << b;
    }
    r.ok = okb;
  };
  auto contract = [&](StepRegs& r) __attribute__((always_inline)) {
    asm volatile("" : "+v"(r.dv));      // (keeps the load where it is, see below)
    const float dv = (r.ok >> 31) ? r.dv : 0.f;
#pragma unroll
    for (int b = 0; b < NJ; ++b) {
      asm volatile("" : "+v"(r.xv[b]));
      acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(dv, (r.ok >> b) & 1u ? r.xv[b] : 0.f, acc[b], 0, 0, 0);
    }
  };
  StepRegs rs[4];      // four sets, used in turn (a step past the end is masked: it adds zeros)
#pragma unroll
  for (int u = 0; u < 3; ++u) issue(rs[u], u);
  for (int st = 0; st < a.steps; st += 4) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      issue(rs[(u + 3) & 3], st + u + 3);
      __builtin_amdgcn_sched_barrier(0);
      contract(rs[u]);
    }
  }

  // sum the four waves in a fixed order, then write the partial tile
  __shared__ float red[4][NJ][16][17];
#pragma unroll
  for (int b = 0; b < NJ; ++b)
#pragma unroll
    for (int i = 0; i < 4; ++i) red[wave][b][lg * 4 + i][l16] = acc[b][i];
  __syncthreads();
  const int Jp = a.JB * 16;
  for (int e = threadIdx.x; e < NJ * 256; e += 256) {
    const int b = e >> 8, row = (e >> 4) & 15, col = e & 15;
    if (jb0 + b >= a.JB) continue;
    const float t = ((red[0][b][row][col] + red[1][b][row][col]) + red[2][b][row][col]) + red[3][b][row][col];
    a.partial[((size_t)blockIdx.x * a.Cout + cob * 16 + row) * Jp + (jb0 + b) * 16 + col] = t;
  }
}

template <typename T>
__global__ __launch_bounds__(256) void wgrad_mfma_vec_kernel(WgradArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  wgrad_vec_body<T>(a, smem, blockIdx.x, blockIdx.y, blockIdx.z);
}

// dW[co][ci][r][s] = sum over splits (in order) of partial[split][co][tap*CP + ci]
__global__ __launch_bounds__(256) void wgrad_reduce_kernel(WgradArgs a) {
  const int Jp = a.JB * 16;
  const int total = a.Cout * Jp;
  // 16 threads share one output: each sums a strided subset, then a fixed-order tree
  __shared__ float red[16][17];
  const int sub = threadIdx.x & 15, loc = threadIdx.x >> 4;
  const int e = blockIdx.x * 16 + loc;
  float s = 0.f;
  if (e < total)
    for (int sp = sub; sp < a.msplit; sp += 16) s += a.partial[(size_t)sp * total + e];
  red[loc][sub] = s;
  __syncthreads();
  if (sub == 0 && e < total) {
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) t += red[loc][i];
    const int co = e / Jp, j = e - co * Jp;
    const int tap = j >> a.log2cp, ci = j & ((1 << a.log2cp) - 1);
    if (tap < a.R * a.R && ci < a.Cin) {
      const int r = tap / a.R, sx = tap % a.R;
      a.dW[(((size_t)co * a.Cin + ci) * a.R + r) * a.R + sx] = t;
    }
  }
}

// All layers of a module in one launch: blockIdx.y picks the layer. The rows of an output are added in four
// classes rc = 0 .. 3 (rows rc, rc+4, ... in increasing order), the classes then in order.
//
// Many rows (the narrow layers: up to 128 rows of a few thousand outputs): a workgroup covers 64 groups of 4
// outputs, one thread per class with 8 loads in flight (a wave reads 1 KiB of one row).
//
// Few rows (RED_FEW; most wide layers: one row to eight of up to 590 thousand outputs): a thread adds all rows of its
// outputs with every load in flight, a workgroup covers 1024 outputs (1x1: stored as they come) or one output
// channel (3x3: through LDS into the [ci][r][s] order, so that memory sees whole lines instead of four bytes in every
// 36). 23 bottleneck blocks with the 7 to 16 rows of layers in launches of their own, 1.15 GB: 297 -> 251 us; with the 2 rows (6 in the
// last launch) of layers that share one, 0.2 GB, 52 us, four loads instead of sixteen.
constexpr int RED_FEW = 16, RED_J_MAX = 9 * 512;

__host__ __device__ static inline bool red_few(int rows, int Cout, int Cin, int R, int Jp) {
  return rows <= RED_FEW && Jp == R * R * Cin && (R == 1 ? Cout * Jp % 1024 == 0 : Jp <= RED_J_MAX);
}

__global__ __launch_bounds__(256) void wgrad_reduce_all_kernel(const WredDesc* __restrict__ descs) {
  const WredDesc d = descs[blockIdx.y];
  const int total4 = d.Cout * d.Jp / 4;
  __shared__ float4 red[RED_J_MAX / 4];
  if (red_few(d.rows, d.Cout, d.Cin, d.R, d.Jp)) {
    const int per = d.R == 1 ? 256 : d.Jp / 4;     // groups of 4 outputs of this workgroup
    if ((int)blockIdx.x * per >= total4) return;
    float* out = d.dW + (size_t)blockIdx.x * per * 4;
    float* tr = reinterpret_cast<float*>(red);
    for (int k = threadIdx.x; k < per; k += 256) {
      const float4* __restrict__ p = reinterpret_cast<const float4*>(d.partial) + (size_t)blockIdx.x * per + k;
      float4 v[RED_FEW];
      if (d.rows <= 4) {
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = p[(size_t)(r < d.rows ? r : d.rows - 1) * total4];
      } else {
#pragma unroll
        for (int r = 0; r < RED_FEW; ++r) v[r] = p[(size_t)(r < d.rows ? r : d.rows - 1) * total4];
      }
      float4 c[4];
#pragma unroll
      for (int rc = 0; rc < 4; ++rc) c[rc] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int r = 0; r < RED_FEW; ++r)
        if (r < d.rows) { c[r & 3].x += v[r].x; c[r & 3].y += v[r].y; c[r & 3].z += v[r].z; c[r & 3].w += v[r].w; }
      const float4 t = make_float4(((c[0].x + c[1].x) + c[2].x) + c[3].x, ((c[0].y + c[1].y) + c[2].y) + c[3].y,
                                   ((c[0].z + c[1].z) + c[2].z) + c[3].z, ((c[0].w + c[1].w) + c[2].w) + c[3].w);
      if (d.R == 1) {
        float* q = out + (size_t)k * 4;
        q[0] = t.x; q[1] = t.y; q[2] = t.z; q[3] = t.w;
      } else {
        const int j = k * 4, tap = j >> d.log2cp, ci = j & ((1 << d.log2cp) - 1);
        tr[ci * 9 + tap] = t.x; tr[(ci + 1) * 9 + tap] = t.y; tr[(ci + 2) * 9 + tap] = t.z; tr[(ci + 3) * 9 + tap] = t.w;
      }
    }
    if (d.R != 1) {
      __syncthreads();
      for (int k = threadIdx.x; k < d.Jp; k += 256) out[k] = tr[k];
    }
    return;
  }
  if ((int)blockIdx.x * 64 >= total4) return;
  const int cl = threadIdx.x & 63, rc = threadIdx.x >> 6;
  const int col = blockIdx.x * 64 + cl;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  if (col < total4) {
    const float4* __restrict__ p = reinterpret_cast<const float4*>(d.partial) + col;
    for (int r0 = rc; r0 < d.rows; r0 += 32) {
      float4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int r = r0 + 4 * u;
        v[u] = r < d.rows ? p[(size_t)r * total4] : make_float4(0.f, 0.f, 0.f, 0.f);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) { s.x += v[u].x; s.y += v[u].y; s.z += v[u].z; s.w += v[u].w; }
    }
  }
  red[rc * 64 + cl] = s;
  __syncthreads();
  if (rc == 0 && col < total4) {
    const float4 a0 = red[cl], a1 = red[64 + cl], a2 = red[128 + cl], a3 = red[192 + cl];
    const float t[4] = {((a0.x + a1.x) + a2.x) + a3.x, ((a0.y + a1.y) + a2.y) + a3.y,
                        ((a0.z + a1.z) + a2.z) + a3.z, ((a0.w + a1.w) + a2.w) + a3.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = col * 4 + i;
      const int co = e / d.Jp, j = e - co * d.Jp;
      const int tap = j >> d.log2cp, ci = j & ((1 << d.log2cp) - 1);
      if (tap < d.R * d.R && ci < d.Cin) {
        const int r = tap / d.R, sx = tap % d.R;
        d.dW[(((size_t)co * d.Cin + ci) * d.R + r) * d.R + sx] = t[i];
      }
    }
  }
}

// Adding up, update and repacking of a small module in one launch (see update_pack_kernel), for callers whose update follows
// at once: a weight's sum is applied by the thread that formed it, the gradient vector is written but not read again, and a
// launch in the chain goes. blockIdx.y: a segment of the parameter vector. A layer: its sums as above (same order), then one
// workgroup for batch-norm scales and shifts, whose gradients are complete. The head: a workgroup per class, which forms
// the class's gradient as head_wgrad_kernel does.
template <typename T, bool ADAM>
__global__ __launch_bounds__(256) void reduce_update_kernel(const WredDesc* __restrict__ wdescs, const UpdDesc* __restrict__ udescs, int nlayers,
                                                            UpdArgs a, HeadSums h) {
  UpdStep<ADAM> u;
  u.init(a, gridDim.x * gridDim.y);
  const UpdDesc ud = udescs[blockIdx.y];
  float* g = const_cast<float*>(a.g);
  const int tid = threadIdx.x;
  __shared__ float4 red[RED_J_MAX / 4];
  float* redf = reinterpret_cast<float*>(red);
  if ((int)blockIdx.y >= nlayers) {               // the head: dfcw[j][:] = sum_n dlogits[n][j] * pooled[n][:], dfcb[j], loss
    const int j = blockIdx.x, C = h.C;
    if (j >= h.classes) return;
    float b = 0.f, l = 0.f;
    for (int n = tid; n < h.N; n += 256) {
      b += h.dlogits[(size_t)n * h.classes + j];
      if (j == 0) l += h.loss_n[n];
    }
    redf[256 + tid] = b; redf[512 + tid] = l;
    const int cpt = C < 256 ? C : 256, groups = 256 / cpt;
    const int cl = tid % cpt, gr = tid / cpt;
    for (int c0 = 0; c0 < C; c0 += cpt) {
      const int c = c0 + cl;
      float t = 0.f;
      if (gr < groups && c < C) {
#pragma unroll 16
        for (int n = gr; n < h.N; n += groups) t += h.dlogits[(size_t)n * h.classes + j] * h.pooled[(size_t)n * C + c];
      }
      redf[tid] = t;
      __syncthreads();
      if (gr == 0 && c < C) {
        float q = 0.f;
        for (int k = 0; k < groups; ++k) q += redf[k * cpt + cl];
        const size_t e = ud.off + (size_t)j * C + c;
        g[e] = q;
        u.step(a, e, q);
      }
      __syncthreads();
    }
    const int terms = h.N < 256 ? h.N : 256;
    if (tid == 0) {
      float t = 0.f;
#pragma unroll 16
      for (int q = 0; q < terms; ++q) t += redf[256 + q];
      const size_t e = ud.off + (size_t)h.classes * C + j;
      g[e] = t;
      u.step(a, e, t);
    }
    if (tid == 64 && j == 0 && h.loss_out) {
      float t = 0.f;
#pragma unroll 16
      for (int q = 0; q < terms; ++q) t += redf[512 + q];
      *h.loss_out = t / (float)h.N;
    }
    return;
  }
  const WredDesc d = wdescs[blockIdx.y];
  const int total4 = d.Cout * d.Jp / 4;
  const bool few = red_few(d.rows, d.Cout, d.Cin, d.R, d.Jp);
  const int per = few ? (d.R == 1 ? 256 : d.Jp / 4) : 64;      // groups of 4 outputs of a workgroup
  const int nb = (total4 + per - 1) / per;
  if ((int)blockIdx.x > nb) return;
  if ((int)blockIdx.x == nb) {
    for (unsigned i = tid; i < ud.plain; i += 256) u.step(a, ud.off + ud.conv + i, a.g[ud.off + ud.conv + i]);
    return;
  }
  const int RR = d.R * d.R;
  auto apply = [&](int co, int ci, int tap, float s) __attribute__((always_inline)) {
    const size_t e = ud.off + ((size_t)co * d.Cin + ci) * RR + tap;
    g[e] = s;
    upd_pack<T>(ud, co, ci, tap, u.step(a, e, s));
  };
  if (few) {
    for (int k = tid; k < per; k += 256) {
      const float4* __restrict__ p = reinterpret_cast<const float4*>(d.partial) + (size_t)blockIdx.x * per + k;
      float4 v[RED_FEW];
#pragma unroll
      for (int r = 0; r < RED_FEW; ++r) v[r] = p[(size_t)(r < d.rows ? r : d.rows - 1) * total4];
      float4 c[4];
#pragma unroll
      for (int rc = 0; rc < 4; ++rc) c[rc] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int r = 0; r < RED_FEW; ++r)
        if (r < d.rows) { c[r & 3].x += v[r].x; c[r & 3].y += v[r].y; c[r & 3].z += v[r].z; c[r & 3].w += v[r].w; }
      const float t[4] = {((c[0].x + c[1].x) + c[2].x) + c[3].x, ((c[0].y + c[1].y) + c[2].y) + c[3].y,
                          ((c[0].z + c[1].z) + c[2].z) + c[3].z, ((c[0].w + c[1].w) + c[2].w) + c[3].w};
      const int j = k * 4, tap = RR == 9 ? j >> d.log2cp : 0, ci = RR == 9 ? j & ((1 << d.log2cp) - 1) : j;
#pragma unroll
      for (int i = 0; i < 4; ++i) redf[(ci + i) * RR + tap] = t[i];
    }
    __syncthreads();
    // in the order of the parameter vector: 3x3, one output channel; 1x1, 1024 consecutive weights
    for (int k = tid; k < per * 4; k += 256) {
      const int e = (int)blockIdx.x * per * 4 + k, q = RR == 9 ? k / 9 : 0;
      if (RR == 9) apply(blockIdx.x, q, k - q * 9, redf[k]);
      else apply(e / d.Cin, e % d.Cin, 0, redf[k]);
    }
    return;
  }
  const int cl = tid & 63, rc = tid >> 6;
  const int col = blockIdx.x * 64 + cl;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  // rows of a class, 8 or 16 in flight: with 128 rows two trips instead of four (ResNet-20, fp32, batch 128, 16 iterations 12.24 -> 12.14 ms); with 37
  // rows the longer trip is 1 % of ResNet-20 at batch 37 slower than two short ones
  auto add = [&](auto in_flight) __attribute__((always_inline)) {
    constexpr int U = decltype(in_flight)::value;
    const float4* __restrict__ p = reinterpret_cast<const float4*>(d.partial) + col;
    for (int r0 = rc; r0 < d.rows; r0 += 4 * U) {
      float4 v[U];
#pragma unroll
      for (int q = 0; q < U; ++q) {
        const int r = r0 + 4 * q;
        v[q] = r < d.rows ? p[(size_t)r * total4] : make_float4(0.f, 0.f, 0.f, 0.f);
      }
#pragma unroll
      for (int q = 0; q < U; ++q) { s.x += v[q].x; s.y += v[q].y; s.z += v[q].z; s.w += v[q].w; }
    }
  };
  if (col < total4) {
    if (d.rows > 64) add(std::integral_constant<int, 16>{});
    else add(std::integral_constant<int, 8>{});
  }
  red[rc * 64 + cl] = s;
  __syncthreads();
  const int e = (int)blockIdx.x * 256 + tid;      // one output per thread
  if (e < total4 * 4) {
    const float t = ((redf[tid] + redf[256 + tid]) + redf[512 + tid]) + redf[768 + tid];
    const int co = e / d.Jp, j = e - co * d.Jp;
    const int tap = j >> d.log2cp, ci = j & ((1 << d.log2cp) - 1);
    if (tap < RR && ci < d.Cin) apply(co, ci, tap, t);
  }
}

hipError_t reduce_update_launch(const WredDesc* wdescs, const UpdDesc* udescs, int nlayers, int max_blocks, const UpdArgs& a, const HeadSums* head,
                                int dtype, bool adam, hipStream_t s) {
  int gx = nlayers > 0 ? max_blocks + 1 : 0;      // and the batch-norm values' workgroup
  if (head && head->classes > gx) gx = head->classes;
  const int gy = nlayers + (head ? 1 : 0);
  if (gx <= 0 || gy <= 0) return hipSuccess;
  const dim3 grid(gx, gy), block(256);
  const HeadSums h = head ? *head : HeadSums{};
  if (dtype == BF16) {
    if (adam) DDG_LAUNCH((reduce_update_kernel<bf16_t, true>), grid, block, 0, s, wdescs, udescs, nlayers, a, h);
    else DDG_LAUNCH((reduce_update_kernel<bf16_t, false>), grid, block, 0, s, wdescs, udescs, nlayers, a, h);
  } else {
    if (adam) DDG_LAUNCH((reduce_update_kernel<float, true>), grid, block, 0, s, wdescs, udescs, nlayers, a, h);
    else DDG_LAUNCH((reduce_update_kernel<float, false>), grid, block, 0, s, wdescs, udescs, nlayers, a, h);
  }
  return hipGetLastError();
}

int wgrad_reduce_blocks(const WredDesc& d) {
  const int total4 = d.Cout * d.Jp / 4;
  if (red_few(d.rows, d.Cout, d.Cin, d.R, d.Jp)) return d.R == 1 ? total4 / 256 : d.Cout;
  return (total4 + 63) / 64;
}

hipError_t wgrad_reduce_all_launch(const WredDesc* dev_descs, int n, int max_blocks, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  DDG_LAUNCH(wgrad_reduce_all_kernel, dim3(max_blocks > 0 ? max_blocks : 1, n), dim3(256), 0, s, dev_descs);
  return hipGetLastError();
}

void wgrad_plan(WgradArgs& a) {
  int l2 = 0;
  while ((1 << l2) < a.Cin) ++l2;
  a.log2cp = l2;
  a.J = a.R * a.R * (1 << l2);
  a.JB = (a.J + 15) / 16;
  a.vec = (a.Cin % 4 == 0) ? 1 : 0;       // the kernel with 4-channel gathers
  a.jgroups = a.vec ? (a.JB * 16 + 64 * WGV_NG - 1) / (64 * WGV_NG) : (a.JB + WG_NJ - 1) / WG_NJ;
  const int tiles = (a.Cout / 16) * a.jgroups;
  int want = 512 / tiles;                // workgroups over the pixel range (two per compute unit; more only add partial tiles)
  if (const char* e = getenv("DDG_TUNE_WGRAD_GENERIC_WGS")) {   // timing experiments, within [64, 4096]
    const int v = atoi(e);
    if (v >= 64 && v <= 4096) want = v / tiles;
  }
  if (want < 1) want = 1;
  const long quads = ((long)a.M + 3) / 4;  // 4-pixel steps in total
  long steps = (quads + (long)want * 4 - 1) / ((long)want * 4);
  if (steps < 8) steps = 8;
  a.steps = (int)steps;
  a.msplit = (int)((quads + steps * 4 - 1) / (steps * 4));
  if (a.msplit < 1) a.msplit = 1;
}

size_t wgrad_partial_elems(const WgradArgs& a) { return (size_t)a.msplit * a.Cout * a.JB * 16; }

hipError_t wgrad_launch(const WgradArgs& a, hipStream_t s) {
  dim3 grid(a.msplit, a.Cout / 16, a.jgroups), block(256);
  if (a.vec) {
    if (a.Cin % 4 != 0) return hipErrorInvalidValue;
    // 32-bit element offsets inside
    if ((size_t)a.N * a.H * a.W * a.Cin >= ((size_t)1 << 32) || (size_t)a.M * a.Cout >= ((size_t)1 << 32)) return hipErrorInvalidValue;
    if (a.dtype == BF16) DDG_LAUNCH(wgrad_mfma_vec_kernel<bf16_t>, grid, block, WGV_LDS, s, a);
    else DDG_LAUNCH(wgrad_mfma_vec_kernel<float>, grid, block, WGV_LDS, s, a);
    return hipGetLastError();
  }
  if (stem_wgrad_ok(a)) return stem_wgrad_launch(a, s);
  if (a.JB <= 3) {
    if (a.dtype == BF16) DDG_LAUNCH((wgrad_mfma_kernel<bf16_t, 3>), grid, block, 0, s, a);
    else DDG_LAUNCH((wgrad_mfma_kernel<float, 3>), grid, block, 0, s, a);
  } else {
    if (a.dtype == BF16) DDG_LAUNCH((wgrad_mfma_kernel<bf16_t, WG_NJ>), grid, block, 0, s, a);
    else DDG_LAUNCH((wgrad_mfma_kernel<float, WG_NJ>), grid, block, 0, s, a);
  }
  return hipGetLastError();
}

hipError_t wgrad_reduce_launch(const WgradArgs& a, hipStream_t s) {
  const int total = a.Cout * a.JB * 16;
  DDG_LAUNCH(wgrad_reduce_kernel, dim3((total + 15) / 16), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace ddg
