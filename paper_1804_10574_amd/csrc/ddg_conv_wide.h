// What the GEMM-class kernels of the wide bf16 layers share: their arguments, 16-byte loads and the on-load transform.
// WideTail is the epilogue of conv_halo_kernel; conv_wide_kernel has its own (64-pixel tiles, its own thread layout) with the
// same rounding points, masks and statistics: a change of a rule in one belongs in the other.
#pragma once
#include "ddg_device.h"
#include "ddg_kernels.h"

namespace ddg {

struct ConvWideArgs {
  const bf16_t* in;        // [M][IC]
  const bf16_t* wpack;     // [k-step][OC/16][64][8], k = tap*IC + channel
  bf16_t* out;             // [M][OC]
  float* stat_partial;     // [rows][2][OC] or null
  const bf16_t* add_g;     // optional: out += add_g (where add_mask > 0, if given)
  const bf16_t* add_mask;
  const float* scale;      // optional (XFORM kernels): the conv input is relu(in*scale + shift), per input channel
  const float* shift;
  // STATS = 2 (input gradient): the outputs are an error gradient v; with the ReLU mask of the
  // layer below applied, g = (bmask*bmscale + bmshift > 0) ? v : 0 (bmask null: g = v), the rows
  // hold sum g and sum g*xhat of that layer's BN (xhat = (bz - bmean)*binvstd): its
  // bn_bwd_reduce pass comes for free. stat_partial receives the rows, and the stored output is
  // g (the mask is applied here, once; readers take the gradient as already masked).
  const bf16_t* bmask; const float* bmscale; const float* bmshift;
  const bf16_t* bz; const float* bmean; const float* binvstd;
  // optional second minibatch (blockIdx.z = 1; forward only): same weights, its own tensors
  const bf16_t* in_b; bf16_t* out_b; float* stat_partial_b; const float* scale_b; const float* shift_b;
  // optional, in place of scale and shift (halo and point kernels): the statistics rows they derive from, of either minibatch
  BnRows rows, rows_b;
  int M, H, W, HW, IC, OC, R;
};

// Scale and shift of C input channels from the producer's statistics rows, by a workgroup of NT threads, into LDS (tab: C scales, then C shifts):
// a launch of its own for it is 4.5 us of latency in the chain between two convolutions. Every workgroup adds the same rows in the same
// order (fp64), one of each minibatch stores the vectors. A thread owns one 16-byte column group and every S-th row, U of them in flight.
template <int NT> struct WideRows {
  static constexpr int U = 14;
  float4 v[U];
  wide_rsrc_t res;
  unsigned at, step;
  __device__ __forceinline__ void request(const BnRows& r, int C) {
    const int cols4 = C >> 1;
    // rows past the last: zeros. Their distance is in the lane's offset, which is checked against the resource's size; what the check does with the
    // uniform offset is not documented, and with few rows that alone passed the end.
    res = wide_rsrc(r.partial, (size_t)r.rows * C * 8);
    at = threadIdx.x * 16; step = NT / cols4 * cols4 * 16;
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = __builtin_bit_cast(float4, wide_load(res, at + u * step, 0));
  }
  // part: NT * 32 bytes of LDS. Ends with a barrier.
  __device__ __forceinline__ void finish(const BnRows& r, int C, float* tab, double* part, bool write) {
    const int cols4 = C >> 1, S = NT / cols4, tid = threadIdx.x;
    double t[4] = {0.0, 0.0, 0.0, 0.0};
    for (int left = r.rows - S * U;; left -= S * U) {
      at += U * step;
      if (left > 0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          t[0] += (double)v[u].x; t[1] += (double)v[u].y; t[2] += (double)v[u].z; t[3] += (double)v[u].w;
          v[u] = __builtin_bit_cast(float4, wide_load(res, at + u * step, 0));
        }
      } else {
#pragma unroll
        for (int u = 0; u < U; ++u) { t[0] += (double)v[u].x; t[1] += (double)v[u].y; t[2] += (double)v[u].z; t[3] += (double)v[u].w; }
        break;
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) part[tid * 4 + j] = t[j];
    __syncthreads();
    for (int c = tid; c < C; c += NT) {
      double t1 = 0.0, t2 = 0.0;
      for (int q = 0; q < S; ++q) { t1 += part[q * 2 * C + c]; t2 += part[q * 2 * C + C + c]; }
      const double mu = t1 * r.inv_count;
      double var = t2 * r.inv_count - mu * mu;
      if (var < 0.0) var = 0.0;
      const float is = (float)rsqrt(var + (double)r.eps), sc = r.gamma[c] * is, sh = r.beta[c] - (float)mu * sc;
      tab[c] = sc; tab[C + c] = sh;
      if (write) { r.mean[c] = (float)mu; r.invstd[c] = is; r.scale[c] = sc; r.shift[c] = sh; }
    }
    __syncthreads();
  }
};
constexpr int WIDE_ROWS_CMAX = 256;

// relu(v*sc + sh) of eight bf16 values, rounded back to bf16
__device__ __forceinline__ uint4 wide_act(uint4 v, const float* sc, const float* sh) {
  float f[8];
  Store<bf16_t>::unpack_vec(v, f);
#pragma unroll
  for (int e = 0; e < 8; ++e) { const float t = f[e] * sc[e] + sh[e]; f[e] = t > 0.f ? t : 0.f; }
  uint4 o;
  o.x = Store<bf16_t>::pack2(f[0], f[1]); o.y = Store<bf16_t>::pack2(f[2], f[3]);
  o.z = Store<bf16_t>::pack2(f[4], f[5]); o.w = Store<bf16_t>::pack2(f[6], f[7]);
  return o;
}

// Epilogue of a thread: per-channel sums over the pixels it stores (8 channels), and what one
// 8-channel group of one pixel needs from memory. `fetch` requests it, `finish` uses it, so that the
// requests can be made before a barrier.
template <int STATS> struct WideTail {
  float ssum[8], ssq[8];
  float bmu[8], bis[8], bms[8], bmh[8];   // STATS = 2: constants of the BN below, this thread's 8 channels
  struct Ops { uint4 g, gm, z, mk; };

  __device__ __forceinline__ void init(const ConvWideArgs& a, int c) {
#pragma unroll
    for (int e = 0; e < 8; ++e) { ssum[e] = 0.f; ssq[e] = 0.f; }
    if (STATS == 2) {
      auto ld8 = [&](const float* p, float (&d)[8], float dflt) __attribute__((always_inline)) {
        float4 lo = make_float4(dflt, dflt, dflt, dflt), hi = lo;
        if (p) { lo = *reinterpret_cast<const float4*>(p + c); hi = *reinterpret_cast<const float4*>(p + c + 4); }
        d[0] = lo.x; d[1] = lo.y; d[2] = lo.z; d[3] = lo.w; d[4] = hi.x; d[5] = hi.y; d[6] = hi.z; d[7] = hi.w;
      };
      ld8(a.bmean, bmu, 0.f); ld8(a.binvstd, bis, 1.f);
      ld8(a.bmscale, bms, 1.f); ld8(a.bmscale ? a.bmshift : nullptr, bmh, 0.f);
    }
  }
  // idx: element offset of the 8 channels (always inside the tensor; a pixel past the end is fetched
  // from the last one and not used)
  __device__ __forceinline__ void fetch(const ConvWideArgs& a, size_t idx, Ops& o) const {
    if (a.add_g) {
      o.g = *reinterpret_cast<const uint4*>(a.add_g + idx);
      if (a.add_mask) o.gm = *reinterpret_cast<const uint4*>(a.add_mask + idx);
    }
    if (STATS == 2) {
      o.z = *reinterpret_cast<const uint4*>(a.bz + idx);
      if (a.bmask && a.bmask != a.bz) o.mk = *reinterpret_cast<const uint4*>(a.bmask + idx);
    }
  }
  __device__ __forceinline__ void finish(const ConvWideArgs& a, bf16_t* out, size_t idx, const Ops& o, float (&v)[8]) {
    *reinterpret_cast<uint4*>(out + idx) = result(a, o, v, true);
  }
  // The eight values to store, their sums taken; zeros, and nothing added to the sums, unless `valid` (no branch).
  __device__ __forceinline__ uint4 result(const ConvWideArgs& a, const Ops& o, float (&v)[8], bool valid) {
    if (a.add_g) {
      float g[8];
      Store<bf16_t>::unpack_vec(o.g, g);
      if (a.add_mask) {
        float mk[8];
        Store<bf16_t>::unpack_vec(o.gm, mk);
#pragma unroll
        for (int e = 0; e < 8; ++e) g[e] = mk[e] > 0.f ? g[e] : 0.f;
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] += g[e];
    }
    uint4 q;
    q.x = Store<bf16_t>::pack2(v[0], v[1]); q.y = Store<bf16_t>::pack2(v[2], v[3]);
    q.z = Store<bf16_t>::pack2(v[4], v[5]); q.w = Store<bf16_t>::pack2(v[6], v[7]);
    q.x = valid ? q.x : 0u; q.y = valid ? q.y : 0u; q.z = valid ? q.z : 0u; q.w = valid ? q.w : 0u;
    if (STATS == 1) {
      float r[8];
      Store<bf16_t>::unpack_vec(q, r);            // the values as stored
#pragma unroll
      for (int e = 0; e < 8; ++e) { ssum[e] += r[e]; ssq[e] += r[e] * r[e]; }
    }
    if (STATS == 2) {
      // the gradient leaves this kernel already multiplied by the ReLU mask of the layer below
      // (every reader of it applies that mask first, so it is applied once, here)
      float r[8], zz[8], mk[8];
      Store<bf16_t>::unpack_vec(q, r);
      Store<bf16_t>::unpack_vec(o.z, zz);
      Store<bf16_t>::unpack_vec(a.bmask && a.bmask != a.bz ? o.mk : o.z, mk);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float g = (!a.bmask || mk[e] * bms[e] + bmh[e] > 0.f) ? r[e] : 0.f;
        r[e] = g;
        ssum[e] += g;
        ssq[e] += g * ((zz[e] - bmu[e]) * bis[e]);
      }
      q.x = Store<bf16_t>::pack2(r[0], r[1]); q.y = Store<bf16_t>::pack2(r[2], r[3]);   // (exact: bf16 values or zeros)
      q.z = Store<bf16_t>::pack2(r[4], r[5]); q.w = Store<bf16_t>::pack2(r[6], r[7]);
    }
    return q;
  }
  // Adds the 512 threads' sums per channel in a fixed order and stores the workgroup's row. Thread
  // tid holds channels (tid % (BN/8))*8 ..; red: LDS scratch of 2*BN*(4096/BN + 512/(2*BN)) floats,
  // free when this is called by every thread.
  template <int BN> __device__ __forceinline__ void store_row(float* red, float* row, int OC, int c0) const {
    constexpr int CPT = BN / 8, CLS = 512 / CPT, PARTS = 512 / (2 * BN);   // row classes, parts of them
    const int tid = threadIdx.x, oc = tid % CPT, cls = tid / CPT;
#pragma unroll
    for (int e = 0; e < 8; e += 4) {
      *reinterpret_cast<float4*>(&red[(cls * 2 + 0) * BN + oc * 8 + e]) = make_float4(ssum[e], ssum[e + 1], ssum[e + 2], ssum[e + 3]);
      *reinterpret_cast<float4*>(&red[(cls * 2 + 1) * BN + oc * 8 + e]) = make_float4(ssq[e], ssq[e + 1], ssq[e + 2], ssq[e + 3]);
    }
    __syncthreads();
    const int col = tid % (2 * BN), part = tid / (2 * BN);
    float s = 0.f;
#pragma unroll
    for (int r = 0; r < CLS / PARTS; ++r) s += red[(part * (CLS / PARTS) + r) * 2 * BN + col];
    float* red2 = red + CLS * 2 * BN;
    red2[part * 2 * BN + col] = s;
    __syncthreads();
    if (tid < 2 * BN) {
      float t = 0.f;
#pragma unroll
      for (int p = 0; p < PARTS; ++p) t += red2[p * 2 * BN + tid];
      row[(size_t)(tid / BN) * OC + c0 + tid % BN] = t;
    }
  }
};

// 3x3 layers with contraction channels and image rows that the halo kernel covers (kernels_conv_halo.hip)
bool conv_halo_ok(int IC, int W, int R);
int conv_halo_rows(int M);
hipError_t conv_halo_launch(const ConvWideArgs& a, int sets, int stats, bool xform, hipStream_t s);
// 1x1 layers with few contraction channels (kernels_conv_point.hip)
bool conv_point_ok(int IC, int R);
int conv_point_groups(int M, int OC, int sets);      // sums a launch forms per channel and minibatch
int conv_point_rows(int M, int OC, int sets);        // rows they take: one each, or two
hipError_t conv_point_launch(const ConvWideArgs& a, int sets, int stats, bool xform, hipStream_t s);

}  // namespace ddg
