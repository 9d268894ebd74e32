// Per-channel batch-norm quantities computed from per-workgroup partial rows by the kernel
// that CONSUMES them: every workgroup adds the rows [rows][2][C] in the same fixed order
// (so all get bit-identical values), keeps the result in LDS, and workgroup 0 also writes
// it to memory for later kernels. This removes a tiny, latency-bound finalise launch from
// the dependency chain between a producer and its consumer. Used for C <= 64, where the
// rows are a few tens of KB and stay in L2; wider layers use the finalise kernels.
#pragma once
#include "ddg_device.h"
#include "ddg_kernels.h"

namespace ddg {

constexpr int STATS_CMAX = 64;

// 256 threads, C a compile-time constant in {16, 32, 64}. f(c, t1, t2) runs once per channel (in
// thread c) with the two column sums. A row is 2*C floats; a thread owns one 16-byte column
// group and every NSL-th row, keeps its loads in flight together (unconditional: a row past the end
// reads as zeros) and adds its rows in order (fp32, like the rows
// themselves). The NSL row slices of a column are then combined in a fixed order in
// fp64 in two short steps (four values per thread, then 256/(2C) per column), all unrolled.
// This sits in the prologue of nearly every training kernel, where latency is all that counts: the rows and the
// per-channel parameters are requested (request()) before anything else a kernel loads and added up (reduce()) when its other
// loads are on their way; loads return in order, so rows requested behind a tile would wait for it. The fp64 part
// multiplies by 1/count and takes one rsqrt instead of two divisions, a square root and a division.
template <int C>
struct StatRows {
  static_assert(C == 16 || C == 32 || C == 64, "channel count");
  static constexpr int NCOL4 = C / 2;            // float4 groups per row (2*C/4)
  static constexpr int NSL = 256 / NCOL4;        // row slices: 32, 16, 8
  static constexpr int G = 256 / (2 * C);        // second-step groups per column: 8, 4, 2 (NSL == 4*G)
  static constexpr int U = C == 64 ? 12 : 8;     // loads in flight: all rows of the usual launches (256, 128, 96)
  float4 v[U];

  __device__ __forceinline__ void load(const float* __restrict__ partial, int rows, int r0) {
    const wide_rsrc_t res = wide_rsrc(partial, (size_t)rows * (NCOL4 * 16));
#pragma unroll
    for (int u = 0; u < U; ++u) {
      v[u] = __builtin_bit_cast(float4, wide_load(res, (unsigned)((r0 + u * NSL) * NCOL4 + threadIdx.x % NCOL4) * 16, 0));
    }
  }
  __device__ __forceinline__ void request(const float* __restrict__ partial, int rows) { load(partial, rows, threadIdx.x / NCOL4); }

  __device__ __forceinline__ void add(float4& acc) const {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      acc.x += v[u].x; acc.y += v[u].y; acc.z += v[u].z; acc.w += v[u].w;
    }
  }
  // (Rows beyond the first U of a thread are loaded at the top of their own trip. As a loop that loads at its end for the next trip
  // the same sums held U more vectors in registers: bn_apply_kernel 112 instead of 64, conv3x3_tiled_kernel<16, 32, 1, RES> 142
  // instead of 116.)
  template <typename F>
  __device__ __forceinline__ void reduce(const float* __restrict__ partial, int rows, F f) {
    __shared__ float4 sh[256];
    __shared__ double sh2[256];
    const int tid = threadIdx.x;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    add(acc);
    for (int r0 = tid / NCOL4 + NSL * U; r0 < rows; r0 += NSL * U) { load(partial, rows, r0); add(acc); }
    sh[tid] = acc;
    __syncthreads();
    {
      // thread (column col of 2C, group g): slices g*4 .. g*4+3
      const float* shf = reinterpret_cast<const float*>(sh);
      const int col = tid % (2 * C), g = tid / (2 * C);
      double t = 0.0;
#pragma unroll
      for (int k = 0; k < 4; ++k) t += (double)shf[((g * 4 + k) * NCOL4) * 4 + col];
      sh2[g * (2 * C) + col] = t;
    }
    __syncthreads();
    if (tid < C) {
      double t1 = 0.0, t2 = 0.0;
#pragma unroll
      for (int g = 0; g < G; ++g) { t1 += sh2[g * (2 * C) + tid]; t2 += sh2[g * (2 * C) + C + tid]; }
      f(tid, t1, t2);
    }
    __syncthreads();
  }
};

// Forward statistics -> scale = gamma*invstd, shift = beta - mean*scale in LDS (s_scale, s_shift);
// workgroup 0 (write != 0) also stores mean, invstd, scale, shift.
template <int C>
struct BnFwdRows {
  StatRows<C> r;
  float gamma, beta;
  __device__ __forceinline__ void request(const BnRows& p) {
    r.request(p.partial, p.rows);
    const int tc = threadIdx.x < C ? threadIdx.x : 0;
    gamma = p.gamma[tc]; beta = p.beta[tc];
  }
  __device__ __forceinline__ void finish(const BnRows& p, float* s_scale, float* s_shift, bool write) {
    r.reduce(p.partial, p.rows, [&](int c, double t1, double t2) {
      const double mu = t1 * p.inv_count;
      double var = t2 * p.inv_count - mu * mu;
      if (var < 0.0) var = 0.0;
      const float is = (float)rsqrt(var + (double)p.eps);
      const float sc = gamma * is;
      const float sh = beta - (float)mu * sc;
      s_scale[c] = sc; s_shift[c] = sh;
      if (write) { p.mean[c] = (float)mu; p.invstd[c] = is; p.scale[c] = sc; p.shift[c] = sh; }
    });
  }
};
template <int C>
__device__ __forceinline__ void bn_fwd_from_rows(const BnRows& p, float* s_scale, float* s_shift, bool write) {
  BnFwdRows<C> r;
  r.request(p);
  r.finish(p, s_scale, s_shift, write);
}

// Backward sums (sum g, sum g*xhat) -> coefficients of dz = A*g + B*z + C0 in LDS (s_coef[3][C]);
// workgroup 0 also stores dgamma, dbeta.
template <int C>
struct BnBwdFromRows {
  StatRows<C> r;
  float gamma, invstd, mean;
  __device__ __forceinline__ void request(const BnBwdRows& p) {
    r.request(p.partial, p.rows);
    const int tc = threadIdx.x < C ? threadIdx.x : 0;
    gamma = p.gamma[tc]; invstd = p.invstd[tc]; mean = p.mean[tc];
  }
  __device__ __forceinline__ void finish(const BnBwdRows& p, float* s_coef, bool write) {
    r.reduce(p.partial, p.rows, [&](int c, double db, double dg) {
      const double g = gamma, is = invstd, mu = mean;
      const double A = g * is, B = -A * is * (dg * p.inv_count), C0 = -A * (db * p.inv_count) - B * mu;
      s_coef[c] = (float)A; s_coef[C + c] = (float)B; s_coef[2 * C + c] = (float)C0;
      if (write) { p.dgamma[c] = (float)dg; p.dbeta[c] = (float)db; }
    });
  }
};
template <int C>
__device__ __forceinline__ void bn_bwd_from_rows(const BnBwdRows& p, float* s_coef, bool write) {
  BnBwdFromRows<C> r;
  r.request(p);
  r.finish(p, s_coef, write);
}

// Run-time channel count (16, 32 or 64; the host checks): one of the three instances.
__device__ __forceinline__ void bn_fwd_from_rows_rt(const BnRows& p, int C, float* s_scale, float* s_shift, bool write) {
  if (C == 16) bn_fwd_from_rows<16>(p, s_scale, s_shift, write);
  else if (C == 32) bn_fwd_from_rows<32>(p, s_scale, s_shift, write);
  else bn_fwd_from_rows<64>(p, s_scale, s_shift, write);
}
__device__ __forceinline__ void bn_bwd_from_rows_rt(const BnBwdRows& p, int C, float* s_coef, bool write) {
  if (C == 16) bn_bwd_from_rows<16>(p, s_coef, write);
  else if (C == 32) bn_bwd_from_rows<32>(p, s_coef, write);
  else bn_bwd_from_rows<64>(p, s_coef, write);
}

}  // namespace ddg
