// Batch norm of layers with more than 64 channels: the partial rows [rows][2][C] a convolution's
// epilogue wrote become per-channel values either in the elementwise kernel that consumes them
// (a few rows: no launch between producer and consumer) or in a finalise kernel of their own
// (many rows, or a consumer that needs every channel at once).
//
// The elementwise kernels own 64 channels x a run of pixels per workgroup, so a workgroup adds up
// 64 of the C channels only. What bounds them: memory (3 tensors), and the row reads, which
// cost (pixel groups) * rows * 2 * C * 4 bytes of L2 traffic for the launch: it grows with the square of
// the pixel count, hence a line at WIDE_ROWS_MAX rows. In pixels that is 8192 behind conv_wide_kernel (a row per 64
// pixels) and 16384 behind conv_halo_kernel (a row per 128); behind conv_point_kernel, whose rows a launch's width bounds, it is
// reached by 256 channels or fewer only (more than 8192 pixels). The generic convolution (fp32) writes at most 512 rows, by its
// grid. Two blocks 512-128-128-512 at 28x28, a step, finalised here against in a launch of its own: 6272 pixels 291
// against 314 us; behind the halo kernel alone 8624 pixels 361.1 against 363.2, 12544 408 against 409, 14112 430.0
// against 427.0, 15680 453 against 450: even at about 100 rows, 1 % behind at 128.
// 23 bottleneck blocks at 14x14, batch 32, with 98 rows, per launch: normalise-add-ReLU of two 6272 x 1024
// minibatches 28.3 -> 16.4 us against a finalise launch and bn_apply_pair_kernel (conv_form_kernel does it now for all blocks but
// the last); BN backward of 6272 x 256 9.8 -> 5.6 us, of 6272 x 1024 12.0 -> 9.6 us (a launch that depends on the one before costs 4.7 us whatever it does).
#include "ddg_device.h"
#include "ddg_kernels.h"

namespace ddg {

namespace {

constexpr int WIDE_ROWS_MAX = 128;

// Column sums of 64 channels, in fp64, by 256 threads: f(c, sum, second sum) runs in thread c < 64.
// A thread owns one 16-byte column group of 32 (16 of the sums, 16 of the second sums) and every 8th
// row; 13 rows are requested together and unconditionally (a row past the end repeats the last and counts as
// zero), which covers 104 rows in one memory round trip.
template <typename F>
__device__ __forceinline__ void reduce_rows_64ch(const float* __restrict__ partial, int rows, int C, int c0, F f) {
  constexpr int U = 13;
  __shared__ double sh[8][128];
  const int tid = threadIdx.x, col = tid & 31, slice = tid >> 5;
  const float* p = partial + (size_t)(col >> 4) * C + c0 + (col & 15) * 4;
  const size_t rstride = (size_t)2 * C;
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
  for (int r0 = slice; r0 < rows; r0 += 8 * U) {
    float4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = r0 + u * 8;
      v[u] = *reinterpret_cast<const float4*>(p + (size_t)(r < rows ? r : rows - 1) * rstride);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = r0 + u * 8 < rows;
      a0 += (double)(in ? v[u].x : 0.f); a1 += (double)(in ? v[u].y : 0.f);
      a2 += (double)(in ? v[u].z : 0.f); a3 += (double)(in ? v[u].w : 0.f);
    }
  }
  double* d = &sh[slice][col * 4];
  d[0] = a0; d[1] = a1; d[2] = a2; d[3] = a3;
  __syncthreads();
  if (tid < 64) {
    double t1 = 0.0, t2 = 0.0;
#pragma unroll
    for (int s = 0; s < 8; ++s) { t1 += sh[s][tid]; t2 += sh[s][64 + tid]; }
    f(tid, t1, t2);
  }
  __syncthreads();
}

__device__ __forceinline__ void fwd_values(double t1, double t2, double inv_count, float eps, float gamma, float beta,
                                           float* mean, float* invstd, float* scale, float* shift) {
  const double mu = t1 * inv_count;
  double var = t2 * inv_count - mu * mu;
  if (var < 0.0) var = 0.0;
  const float is = (float)rsqrt(var + (double)eps);
  const float sc = gamma * is;
  *mean = (float)mu; *invstd = is; *scale = sc; *shift = beta - (float)mu * sc;
}

// scale and shift of channels c0 .. c0+63 into LDS; `write`: this workgroup also stores the vectors
__device__ __forceinline__ void wide_fwd_from_rows(const BnRows& p, int C, int c0, float* s_scale, float* s_shift, bool write) {
  const int tc = c0 + (threadIdx.x & 63);
  const float gamma = p.gamma[tc], beta = p.beta[tc];
  reduce_rows_64ch(p.partial, p.rows, C, c0, [&](int c, double t1, double t2) {
    float mu, is, sc, sh;
    fwd_values(t1, t2, p.inv_count, p.eps, gamma, beta, &mu, &is, &sc, &sh);
    s_scale[c] = sc; s_shift[c] = sh;
    if (write) { p.mean[tc] = mu; p.invstd[tc] = is; p.scale[tc] = sc; p.shift[tc] = sh; }
  });
}

}  // namespace

// ---------------------------------------------------------------------------------
// y = [relu](z*scale + shift + shortcut), shortcut = res, res*rscale+rshift (rrows), or nothing.
// blockIdx: x pixel group of U passes, y 64-channel group, z minibatch.
// ---------------------------------------------------------------------------------
template <typename T, int U, bool RES, bool RROWS>
__global__ __launch_bounds__(256) void bn_apply_wide_kernel(BnApplySet s0, BnApplySet s1, int M, int C, int relu) {
  constexpr int V = Store<T>::VEC, LPR = 64 / V, PPP = 256 / LPR;   // threads per pixel, pixels per pass
  typedef typename Store<T>::vec_t vec_t;
  const BnApplySet& q = blockIdx.z ? s1 : s0;
  const T* z = reinterpret_cast<const T*>(q.z);
  const T* res = reinterpret_cast<const T*>(q.res);
  T* y = reinterpret_cast<T*>(q.y);
  const int c0 = blockIdx.y * 64, cl = (threadIdx.x % LPR) * V;
  const int p0 = blockIdx.x * (PPP * U) + threadIdx.x / LPR;
  vec_t zq[U], rq[RES ? U : 1];
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const int p = p0 + j * PPP;
    const size_t o = (size_t)(p < M ? p : M - 1) * C + c0 + cl;
    zq[j] = *reinterpret_cast<const vec_t*>(z + o);
    if (RES) rq[j] = *reinterpret_cast<const vec_t*>(res + o);
  }
  __shared__ float s_sc[64], s_sh[64], s_rs[64], s_rh[64];
  wide_fwd_from_rows(q.zrows, C, c0, s_sc, s_sh, blockIdx.x == 0);
  if (RROWS) wide_fwd_from_rows(q.rrows, C, c0, s_rs, s_rh, blockIdx.x == 0);
  float sc[V], sh[V], rs[V], rh[V];
#pragma unroll
  for (int e = 0; e < V; ++e) {
    sc[e] = s_sc[cl + e]; sh[e] = s_sh[cl + e];
    if (RROWS) { rs[e] = s_rs[cl + e]; rh[e] = s_rh[cl + e]; }
  }
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const int p = p0 + j * PPP;
    if (p >= M) continue;
    float v[V];
    Store<T>::unpack_vec(zq[j], v);
#pragma unroll
    for (int e = 0; e < V; ++e) v[e] = v[e] * sc[e] + sh[e];
    if (RES) {
      float r[V];
      Store<T>::unpack_vec(rq[j], r);
#pragma unroll
      for (int e = 0; e < V; ++e) v[e] += RROWS ? r[e] * rs[e] + rh[e] : r[e];
    }
    if (relu) {
#pragma unroll
      for (int e = 0; e < V; ++e) v[e] = v[e] > 0.f ? v[e] : 0.f;
    }
    Store<T>::store_vec(y + (size_t)p * C + c0 + cl, v);
  }
}

// Passes per workgroup: as many as leave two workgroups per compute unit.
template <typename T>
static int wide_passes(int M, int C, int sets, int umax) {
  constexpr int PPP = 256 / (64 / Store<T>::VEC);
  int u = umax;
  while (u > 1 && (size_t)((M + PPP * u - 1) / (PPP * u)) * (C / 64) * sets < 512) u >>= 1;
  return u;
}

bool bn_rows_wide_ok(int rows, int C) { return C > 64 && C % 64 == 0 && rows > 0 && rows <= WIDE_ROWS_MAX; }

template <typename T, int U>
static void bn_apply_wide_dispatch(const BnApplySet& a, const BnApplySet& b, int sets, int M, int C, int relu, hipStream_t s) {
  constexpr int PPP = 256 / (64 / Store<T>::VEC);
  const dim3 grid((M + PPP * U - 1) / (PPP * U), C / 64, sets);
  if (a.rrows.partial) DDG_LAUNCH((bn_apply_wide_kernel<T, U, true, true>), grid, dim3(256), 0, s, a, b, M, C, relu);
  else if (a.res) DDG_LAUNCH((bn_apply_wide_kernel<T, U, true, false>), grid, dim3(256), 0, s, a, b, M, C, relu);
  else DDG_LAUNCH((bn_apply_wide_kernel<T, U, false, false>), grid, dim3(256), 0, s, a, b, M, C, relu);
}

template <typename T>
static void bn_apply_wide_type(const BnApplySet& a, const BnApplySet& b, int sets, int M, int C, int relu, hipStream_t s) {
  switch (wide_passes<T>(M, C, sets, 8)) {
    case 8: bn_apply_wide_dispatch<T, 8>(a, b, sets, M, C, relu, s); break;
    case 4: bn_apply_wide_dispatch<T, 4>(a, b, sets, M, C, relu, s); break;
    case 2: bn_apply_wide_dispatch<T, 2>(a, b, sets, M, C, relu, s); break;
    default: bn_apply_wide_dispatch<T, 1>(a, b, sets, M, C, relu, s);
  }
}

hipError_t bn_apply_wide_launch(const BnApplySet& a, const BnApplySet* b, int M, int C, int relu, int dtype, hipStream_t s) {
  if (!bn_rows_wide_ok(a.zrows.rows, C) || !a.zrows.partial) return hipErrorInvalidValue;
  if (a.rrows.partial && (!a.res || !bn_rows_wide_ok(a.rrows.rows, C))) return hipErrorInvalidValue;
  if (dtype == BF16) bn_apply_wide_type<bf16_t>(a, b ? *b : a, b ? 2 : 1, M, C, relu, s);
  else bn_apply_wide_type<float>(a, b ? *b : a, b ? 2 : 1, M, C, relu, s);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// dz = A*g + B*z + C0, g = dy where the ReLU was active (mask as in bn_bwd_reduce_launch); the
// coefficients come from the rows of (sum g, sum g*xhat).
// ---------------------------------------------------------------------------------
template <typename T, int U, bool MASK>
__global__ __launch_bounds__(256) void bn_bwd_apply_wide_kernel(const T* __restrict__ dy, const T* __restrict__ mask,
                                                                const float* __restrict__ mscale,
                                                                const float* __restrict__ mshift,
                                                                const T* __restrict__ z, BnBwdRows rows,
                                                                T* __restrict__ dz, int M, int C) {
  constexpr int V = Store<T>::VEC, LPR = 64 / V, PPP = 256 / LPR;
  typedef typename Store<T>::vec_t vec_t;
  const int c0 = blockIdx.y * 64, cl = (threadIdx.x % LPR) * V;
  const int p0 = blockIdx.x * (PPP * U) + threadIdx.x / LPR;
  vec_t gq[U], zq[U], mq[MASK ? U : 1];
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const int p = p0 + j * PPP;
    const size_t o = (size_t)(p < M ? p : M - 1) * C + c0 + cl;
    gq[j] = *reinterpret_cast<const vec_t*>(dy + o);
    zq[j] = *reinterpret_cast<const vec_t*>(z + o);
    if (MASK) mq[j] = *reinterpret_cast<const vec_t*>(mask + o);
  }
  __shared__ float s_co[3 * 64];
  {
    const int tc = c0 + (threadIdx.x & 63);
    const double g = rows.gamma[tc], is = rows.invstd[tc], mu = rows.mean[tc];
    const bool write = blockIdx.x == 0;
    reduce_rows_64ch(rows.partial, rows.rows, C, c0, [&](int c, double db, double dg) {
      const double A = g * is, B = -A * is * (dg * rows.inv_count), C0 = -A * (db * rows.inv_count) - B * mu;
      s_co[c] = (float)A; s_co[64 + c] = (float)B; s_co[128 + c] = (float)C0;
      if (write) { rows.dgamma[tc] = (float)dg; rows.dbeta[tc] = (float)db; }
    });
  }
  float A[V], B[V], C0[V], ms[V], mh[V];
#pragma unroll
  for (int e = 0; e < V; ++e) {
    A[e] = s_co[cl + e]; B[e] = s_co[64 + cl + e]; C0[e] = s_co[128 + cl + e];
    if (MASK) { ms[e] = mscale ? mscale[c0 + cl + e] : 1.f; mh[e] = mscale ? mshift[c0 + cl + e] : 0.f; }
  }
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const int p = p0 + j * PPP;
    if (p >= M) continue;
    float g[V], zz[V];
    Store<T>::unpack_vec(gq[j], g);
    Store<T>::unpack_vec(zq[j], zz);
    if (MASK) {
      float mk[V];
      Store<T>::unpack_vec(mq[j], mk);
#pragma unroll
      for (int e = 0; e < V; ++e) g[e] = (mk[e] * ms[e] + mh[e]) > 0.f ? g[e] : 0.f;
    }
#pragma unroll
    for (int e = 0; e < V; ++e) g[e] = A[e] * g[e] + (B[e] * zz[e] + C0[e]);
    Store<T>::store_vec(dz + (size_t)p * C + c0 + cl, g);
  }
}

template <typename T, int U>
static void bn_bwd_apply_wide_dispatch(const void* dy, const void* mask, const float* mscale, const float* mshift, const void* z,
                                       const BnBwdRows& rows, void* dz, int M, int C, hipStream_t s) {
  constexpr int PPP = 256 / (64 / Store<T>::VEC);
  const dim3 grid((M + PPP * U - 1) / (PPP * U), C / 64);
  if (mask)
    DDG_LAUNCH((bn_bwd_apply_wide_kernel<T, U, true>), grid, dim3(256), 0, s, (const T*)dy, (const T*)mask, mscale, mshift,
               (const T*)z, rows, (T*)dz, M, C);
  else
    DDG_LAUNCH((bn_bwd_apply_wide_kernel<T, U, false>), grid, dim3(256), 0, s, (const T*)dy, (const T*)nullptr, nullptr,
               nullptr, (const T*)z, rows, (T*)dz, M, C);
}

template <typename T>
static void bn_bwd_apply_wide_type(const void* dy, const void* mask, const float* mscale, const float* mshift, const void* z,
                                   const BnBwdRows& rows, void* dz, int M, int C, hipStream_t s) {
  switch (wide_passes<T>(M, C, 1, 4)) {
    case 4: bn_bwd_apply_wide_dispatch<T, 4>(dy, mask, mscale, mshift, z, rows, dz, M, C, s); break;
    case 2: bn_bwd_apply_wide_dispatch<T, 2>(dy, mask, mscale, mshift, z, rows, dz, M, C, s); break;
    default: bn_bwd_apply_wide_dispatch<T, 1>(dy, mask, mscale, mshift, z, rows, dz, M, C, s);
  }
}

hipError_t bn_bwd_apply_wide_launch(const void* dy, const void* mask, const float* mscale, const float* mshift, const void* z,
                                    const BnBwdRows& rows, void* dz, int M, int C, int dtype, hipStream_t s) {
  if (!bn_rows_wide_ok(rows.rows, C) || !rows.partial) return hipErrorInvalidValue;
  if (dtype == BF16) bn_bwd_apply_wide_type<bf16_t>(dy, mask, mscale, mshift, z, rows, dz, M, C, s);
  else bn_bwd_apply_wide_type<float>(dy, mask, mscale, mshift, z, rows, dz, M, C, s);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// Finalise kernels: one workgroup per 16 channels. A thread owns one 16-byte column group of 8 and
// every 32nd row, four rows requested together; everything is added in fp64 in a fixed order. All
// latency: parameters are requested before the rows, one rsqrt and no division at the end.
// ---------------------------------------------------------------------------------
template <typename F>
__device__ __forceinline__ void reduce_rows_16ch(const float* __restrict__ partial, int rows, int C, int c0, F f) {
  constexpr int U = 4;
  __shared__ double sh[32][32], sh2[8][32];
  const int tid = threadIdx.x, col = tid & 7, slice = tid >> 3;
  const float* p = partial + (size_t)(col >> 2) * C + c0 + (col & 3) * 4;
  const size_t rstride = (size_t)2 * C;
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
  for (int r0 = slice; r0 < rows; r0 += 32 * U) {
    float4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = r0 + u * 32;
      v[u] = *reinterpret_cast<const float4*>(p + (size_t)(r < rows ? r : rows - 1) * rstride);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = r0 + u * 32 < rows;
      a0 += (double)(in ? v[u].x : 0.f); a1 += (double)(in ? v[u].y : 0.f);
      a2 += (double)(in ? v[u].z : 0.f); a3 += (double)(in ? v[u].w : 0.f);
    }
  }
  double* d = &sh[slice][col * 4];
  d[0] = a0; d[1] = a1; d[2] = a2; d[3] = a3;
  __syncthreads();
  {
    const int k = tid & 31, g = tid >> 5;
    sh2[g][k] = (sh[g * 4][k] + sh[g * 4 + 1][k]) + (sh[g * 4 + 2][k] + sh[g * 4 + 3][k]);
  }
  __syncthreads();
  if (tid < 16) {
    double t1 = 0.0, t2 = 0.0;
#pragma unroll
    for (int g = 0; g < 8; ++g) { t1 += sh2[g][tid]; t2 += sh2[g][16 + tid]; }
    f(tid, t1, t2);
  }
}

__global__ __launch_bounds__(256) void bn_finalize_kernel(const float* __restrict__ partial, int rows, int C,
                                                         const float* __restrict__ gamma, const float* __restrict__ beta,
                                                         double inv_count, float eps, float* mean, float* invstd,
                                                         float* scale, float* shift, const float* __restrict__ partial_b,
                                                         float* mean_b) {
  if (blockIdx.y) {   // the second set of rows and vectors
    partial = partial_b; mean = mean_b; invstd = mean_b + C; scale = mean_b + 2 * C; shift = mean_b + 3 * C;
  }
  const int c0 = blockIdx.x * 16, tc = c0 + (threadIdx.x & 15);
  const float g = gamma[tc], b = beta[tc];
  reduce_rows_16ch(partial, rows, C, c0, [&](int, double t1, double t2) {
    fwd_values(t1, t2, inv_count, eps, g, b, &mean[tc], &invstd[tc], &scale[tc], &shift[tc]);
  });
}

hipError_t bn_finalize_launch(const float* partial, int rows, int C, const float* gamma,
                              const float* beta, float count, float eps, float* mean, float* invstd,
                              float* scale, float* shift, hipStream_t s, const float* partial_b, float* mean_b) {
  if (C % 16 != 0) return hipErrorInvalidValue;
  DDG_LAUNCH(bn_finalize_kernel, dim3(C / 16, partial_b ? 2 : 1), dim3(256), 0, s, partial, rows, C, gamma,
             beta, 1.0 / (double)count, eps, mean, invstd, scale, shift, partial_b, mean_b);
  return hipGetLastError();
}

// dbeta = sum g, dgamma = sum g*xhat; dz = A*g + B*z + C0 with
//   A = gamma*invstd, B = -gamma*invstd^2*dgamma/m, C0 = -gamma*invstd*dbeta/m - B*mean
__global__ __launch_bounds__(256) void bn_bwd_finalize_kernel(const float* __restrict__ partial, int rows, int C,
                                                             const float* __restrict__ gamma,
                                                             const float* __restrict__ mean,
                                                             const float* __restrict__ invstd, double inv_count,
                                                             float* dgamma, float* dbeta, float* coef) {
  const int c0 = blockIdx.x * 16, tc = c0 + (threadIdx.x & 15);
  const double g = gamma[tc], is = invstd[tc], mu = mean[tc];
  reduce_rows_16ch(partial, rows, C, c0, [&](int, double db, double dg) {
    const double A = g * is, B = -A * is * (dg * inv_count), C0 = -A * (db * inv_count) - B * mu;
    dbeta[tc] = (float)db; dgamma[tc] = (float)dg;
    coef[tc] = (float)A; coef[C + tc] = (float)B; coef[2 * C + tc] = (float)C0;
  });
}

hipError_t bn_bwd_finalize_launch(const float* partial, int rows, int C, const float* gamma,
                                  const float* mean, const float* invstd, float count, float* dgamma,
                                  float* dbeta, float* coef, hipStream_t s) {
  if (C % 16 != 0) return hipErrorInvalidValue;
  DDG_LAUNCH(bn_bwd_finalize_kernel, dim3(C / 16), dim3(256), 0, s, partial, rows, C, gamma,
             mean, invstd, 1.0 / (double)count, dgamma, dbeta, coef);
  return hipGetLastError();
}

}  // namespace ddg
