// Bandwidth-bound kernels: batch-norm apply / backward, the head
// (global average pool, linear, softmax cross-entropy), momentum SGD, copies.
//
// Tensors are NHWC, so a thread that walks the tensor with a stride that is a
// multiple of the channel count always sees the same channels: per-channel
// coefficients live in registers and every access is a 16-byte vector.
// Reductions write per-workgroup partial rows that a finalise kernel adds in a
// fixed order in double precision (deterministic, no atomics).
#include "ddg_device.h"
#include "ddg_kernels.h"
#include "ddg_stats.h"
#include "ddg_bn_reduce.h"

namespace ddg {

// ---------------------------------------------------------------------------------
// y = [relu](z*scale + shift + shortcut), shortcut = res*rscale+rshift, res, or nothing
// ---------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void bn_apply_kernel(const T* __restrict__ z, const float* __restrict__ scale,
                                                       const float* __restrict__ shift, BnRows zrows,
                                                       const T* __restrict__ res,
                                                       const float* __restrict__ rscale,
                                                       const float* __restrict__ rshift, BnRows rrows,
                                                       T* __restrict__ y, size_t nvec, int C, int relu) {
  constexpr int V = Store<T>::VEC;
  const size_t stride = (size_t)gridDim.x * blockDim.x;  // host makes stride*V a multiple of C
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int c0 = (int)((i * V) % C);
  __shared__ float s_sc[STATS_CMAX], s_sh[STATS_CMAX], s_rs[STATS_CMAX], s_rh[STATS_CMAX];
  if (zrows.partial) { bn_fwd_from_rows_rt(zrows, C, s_sc, s_sh, blockIdx.x == 0); scale = s_sc; shift = s_sh; }
  if (rrows.partial) { bn_fwd_from_rows_rt(rrows, C, s_rs, s_rh, blockIdx.x == 0); rscale = s_rs; rshift = s_rh; }
  float sc[V], sh[V], rs[V], rh[V];
#pragma unroll
  for (int j = 0; j < V; ++j) {
    sc[j] = scale[c0 + j]; sh[j] = shift[c0 + j];
    rs[j] = rscale ? rscale[c0 + j] : 1.f;
    rh[j] = rshift ? rshift[c0 + j] : 0.f;
  }
  for (; i < nvec; i += stride) {
    float v[V];
    Store<T>::load_vec(z + i * V, v);
#pragma unroll
    for (int j = 0; j < V; ++j) v[j] = v[j] * sc[j] + sh[j];
    if (res) {
      float r[V];
      Store<T>::load_vec(res + i * V, r);
#pragma unroll
      for (int j = 0; j < V; ++j) v[j] += r[j] * rs[j] + rh[j];
    }
    if (relu) {
#pragma unroll
      for (int j = 0; j < V; ++j) v[j] = v[j] > 0.f ? v[j] : 0.f;
    }
    Store<T>::store_vec(y + i * V, v);
  }
}

// grid such that (grid*256*V) % C == 0 and the tensor is covered a few times over
static int elem_grid(size_t nvec, int C, int V, int max_blocks) {
  size_t blocks = (nvec + 255) / 256;
  if (blocks > (size_t)max_blocks) blocks = max_blocks;
  // 256*V elements per block; need blocks*256*V % C == 0
  int per = 256 * V;
  int need = 1;
  while ((size_t)need * per % C != 0) ++need;  // C <= 256*V*need, small loop
  blocks = ((blocks + need - 1) / need) * need;
  return (int)blocks;
}

// Same operation for the common case 256*V % C == 0 (a thread's channels are the same for all
// its vectors). A workgroup owns 256*U consecutive vectors; every thread issues all its loads
// first, the per-channel vectors are derived from the partial rows while those are in flight,
// and nothing loops: with U = 4 a thread keeps 128 bytes in flight, which is what it takes to
// approach the memory system's bandwidth with two workgroups per compute unit. ROWS: some vectors come
// from partial rows; without (wider layers) the kernel carries neither that code's LDS nor its
// registers (two 6272 x 1024 bf16 minibatches: 23.6 us with them, 20 us without).
template <typename T, int U, bool ROWS>
__global__ __launch_bounds__(256) void bn_apply_chunk_kernel(const T* __restrict__ z, const float* __restrict__ scale,
                                                             const float* __restrict__ shift, BnRows zrows,
                                                             const T* __restrict__ res,
                                                             const float* __restrict__ rscale,
                                                             const float* __restrict__ rshift, BnRows rrows,
                                                             T* __restrict__ y, size_t nvec, int C, int relu) {
  constexpr int V = Store<T>::VEC;
  typedef typename Store<T>::vec_t vec_t;
  const size_t base = (size_t)blockIdx.x * (256 * U) + threadIdx.x;
  const int c0 = (int)((threadIdx.x * V) % C);
  vec_t zq[U], rq[U];
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const size_t i = base + (size_t)j * 256;
    if (i < nvec) {
      zq[j] = *reinterpret_cast<const vec_t*>(z + i * V);
      if (res) rq[j] = *reinterpret_cast<const vec_t*>(res + i * V);
    }
  }
  if constexpr (ROWS) {
    __shared__ float s_sc[STATS_CMAX], s_sh[STATS_CMAX], s_rs[STATS_CMAX], s_rh[STATS_CMAX];
    if (zrows.partial) { bn_fwd_from_rows_rt(zrows, C, s_sc, s_sh, blockIdx.x == 0); scale = s_sc; shift = s_sh; }
    if (rrows.partial) { bn_fwd_from_rows_rt(rrows, C, s_rs, s_rh, blockIdx.x == 0); rscale = s_rs; rshift = s_rh; }
  }
  float sc[V], sh[V], rs[V], rh[V];
#pragma unroll
  for (int j = 0; j < V; ++j) {
    sc[j] = scale[c0 + j]; sh[j] = shift[c0 + j];
    rs[j] = rscale ? rscale[c0 + j] : 1.f;
    rh[j] = rshift ? rshift[c0 + j] : 0.f;
  }
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const size_t i = base + (size_t)j * 256;
    if (i >= nvec) continue;
    float v[V];
    Store<T>::unpack_vec(zq[j], v);
#pragma unroll
    for (int e = 0; e < V; ++e) v[e] = v[e] * sc[e] + sh[e];
    if (res) {
      float r[V];
      Store<T>::unpack_vec(rq[j], r);
#pragma unroll
      for (int e = 0; e < V; ++e) v[e] += r[e] * rs[e] + rh[e];
    }
    if (relu) {
#pragma unroll
      for (int e = 0; e < V; ++e) v[e] = v[e] > 0.f ? v[e] : 0.f;
    }
    Store<T>::store_vec(y + i * V, v);
  }
}

// Two minibatches of one layer per launch: blockIdx.y selects the set of pointers.
template <typename T, int U, bool ROWS>
__global__ __launch_bounds__(256) void bn_apply_pair_kernel(BnApplySet s0, BnApplySet s1, size_t nvec, int C, int relu) {
  constexpr int V = Store<T>::VEC;
  typedef typename Store<T>::vec_t vec_t;
  const BnApplySet& q = blockIdx.y ? s1 : s0;
  const T* z = reinterpret_cast<const T*>(q.z);
  const T* res = reinterpret_cast<const T*>(q.res);
  T* y = reinterpret_cast<T*>(q.y);
  const float *scale = q.scale, *shift = q.shift, *rscale = q.rscale, *rshift = q.rshift;
  const size_t base = (size_t)blockIdx.x * (256 * U) + threadIdx.x;
  const int c0 = (int)((threadIdx.x * V) % C);
  vec_t zq[U], rq[U];
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const size_t i = base + (size_t)j * 256;
    if (i < nvec) {
      zq[j] = *reinterpret_cast<const vec_t*>(z + i * V);
      if (res) rq[j] = *reinterpret_cast<const vec_t*>(res + i * V);
    }
  }
  if constexpr (ROWS) {
    __shared__ float s_sc[STATS_CMAX], s_sh[STATS_CMAX], s_rs[STATS_CMAX], s_rh[STATS_CMAX];
    if (q.zrows.partial) { bn_fwd_from_rows_rt(q.zrows, C, s_sc, s_sh, blockIdx.x == 0); scale = s_sc; shift = s_sh; }
    if (q.rrows.partial) { bn_fwd_from_rows_rt(q.rrows, C, s_rs, s_rh, blockIdx.x == 0); rscale = s_rs; rshift = s_rh; }
  }
  float sc[V], sh[V], rs[V], rh[V];
#pragma unroll
  for (int j = 0; j < V; ++j) {
    sc[j] = scale[c0 + j]; sh[j] = shift[c0 + j];
    rs[j] = rscale ? rscale[c0 + j] : 1.f;
    rh[j] = rshift ? rshift[c0 + j] : 0.f;
  }
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const size_t i = base + (size_t)j * 256;
    if (i >= nvec) continue;
    float v[V];
    Store<T>::unpack_vec(zq[j], v);
#pragma unroll
    for (int e = 0; e < V; ++e) v[e] = v[e] * sc[e] + sh[e];
    if (res) {
      float r[V];
      Store<T>::unpack_vec(rq[j], r);
#pragma unroll
      for (int e = 0; e < V; ++e) v[e] += r[e] * rs[e] + rh[e];
    }
    if (relu) {
#pragma unroll
      for (int e = 0; e < V; ++e) v[e] = v[e] > 0.f ? v[e] : 0.f;
    }
    Store<T>::store_vec(y + i * V, v);
  }
}

template <typename T, bool ROWS>
static void bn_apply_pair_dispatch(const BnApplySet& a, const BnApplySet& b, size_t nvec, int C, int relu, hipStream_t s) {
  if (nvec >= (size_t)512 * 1024)
    DDG_LAUNCH((bn_apply_pair_kernel<T, 4, ROWS>), dim3((unsigned)((nvec + 1023) / 1024), 2), dim3(256), 0, s, a, b, nvec, C, relu);
  else if (nvec >= (size_t)512 * 512)
    DDG_LAUNCH((bn_apply_pair_kernel<T, 2, ROWS>), dim3((unsigned)((nvec + 511) / 512), 2), dim3(256), 0, s, a, b, nvec, C, relu);
  else
    DDG_LAUNCH((bn_apply_pair_kernel<T, 1, ROWS>), dim3((unsigned)((nvec + 255) / 256), 2), dim3(256), 0, s, a, b, nvec, C, relu);
}

bool bn_apply_pair_launch(const BnApplySet& a, const BnApplySet& b, size_t elems, int C, int relu, int dtype,
                          hipStream_t s, hipError_t* err) {
  const int V = dtype == BF16 ? 8 : 4;
  if ((256 * V) % C != 0) return false;
  // the same kind of work in both sets (the kernel decides per set, the shapes must agree)
  const bool rows = a.zrows.partial || a.rrows.partial;
  if (dtype == BF16) {
    if (rows) bn_apply_pair_dispatch<bf16_t, true>(a, b, elems / 8, C, relu, s);
    else bn_apply_pair_dispatch<bf16_t, false>(a, b, elems / 8, C, relu, s);
  } else {
    if (rows) bn_apply_pair_dispatch<float, true>(a, b, elems / 4, C, relu, s);
    else bn_apply_pair_dispatch<float, false>(a, b, elems / 4, C, relu, s);
  }
  *err = hipGetLastError();
  return true;
}

template <typename T, bool ROWS>
static void bn_apply_chunk_dispatch(const T* z, const float* scale, const float* shift, const BnRows& zr, const T* res,
                                    const float* rscale, const float* rshift, const BnRows& rr, T* y, size_t nvec, int C,
                                    int relu, hipStream_t s) {
  // 4 vectors per thread once that still leaves two workgroups per compute unit
  if (nvec >= (size_t)512 * 1024) {
    DDG_LAUNCH((bn_apply_chunk_kernel<T, 4, ROWS>), dim3((unsigned)((nvec + 1023) / 1024)), dim3(256), 0, s, z, scale, shift, zr,
               res, rscale, rshift, rr, y, nvec, C, relu);
  } else if (nvec >= (size_t)512 * 512) {
    DDG_LAUNCH((bn_apply_chunk_kernel<T, 2, ROWS>), dim3((unsigned)((nvec + 511) / 512)), dim3(256), 0, s, z, scale, shift, zr,
               res, rscale, rshift, rr, y, nvec, C, relu);
  } else {
    DDG_LAUNCH((bn_apply_chunk_kernel<T, 1, ROWS>), dim3((unsigned)((nvec + 255) / 256)), dim3(256), 0, s, z, scale, shift, zr,
               res, rscale, rshift, rr, y, nvec, C, relu);
  }
}

template <typename T>
static void bn_apply_dispatch(const T* z, const float* scale, const float* shift, const BnRows& zr, const T* res,
                              const float* rscale, const float* rshift, const BnRows& rr, T* y, size_t nvec, int C,
                              int relu, bool rows, hipStream_t s) {
  constexpr int V = Store<T>::VEC;
  if ((256 * V) % C != 0) {
    // a thread's channels change from vector to vector: grid-stride kernel
    const int maxb = rows ? 512 : 2048;
    DDG_LAUNCH(bn_apply_kernel<T>, dim3(elem_grid(nvec, C, V, maxb)), dim3(256), 0, s, z, scale, shift, zr, res, rscale,
               rshift, rr, y, nvec, C, relu);
    return;
  }
  if (rows) bn_apply_chunk_dispatch<T, true>(z, scale, shift, zr, res, rscale, rshift, rr, y, nvec, C, relu, s);
  else bn_apply_chunk_dispatch<T, false>(z, scale, shift, zr, res, rscale, rshift, rr, y, nvec, C, relu, s);
}

hipError_t bn_apply_launch(const void* z, const float* scale, const float* shift, const BnRows* zrows,
                           const void* res, const float* rscale, const float* rshift, const BnRows* rrows,
                           void* y, size_t elems, int C, int relu, int dtype, hipStream_t s) {
  const BnRows zr = zrows ? *zrows : BnRows{}, rr = rrows ? *rrows : BnRows{};
  const bool rows = zrows || rrows;
  if (dtype == BF16)
    bn_apply_dispatch<bf16_t>((const bf16_t*)z, scale, shift, zr, (const bf16_t*)res, rscale, rshift, rr, (bf16_t*)y,
                              elems / 8, C, relu, rows, s);
  else
    bn_apply_dispatch<float>((const float*)z, scale, shift, zr, (const float*)res, rscale, rshift, rr, (float*)y,
                             elems / 4, C, relu, rows, s);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// BN backward, pass 1: g = dy masked by (mask > 0); partial sums of g and g*xhat.
// ---------------------------------------------------------------------------------
// blockIdx.y: one of two layers of the same shape (the last layer of a stage's first block and its projection).
template <typename T>
__global__ __launch_bounds__(256) void bn_bwd_reduce_kernel(BnBwdSet q0, BnBwdSet q1, size_t nvec, int C) {
  bn_bwd_reduce_body<T>(blockIdx.y ? q1 : q0, nvec, C, blockIdx.x, gridDim.x);
}

// When C > 256*V a block covers only part of the channels; the other entries of its
// partial row must read as zero, so the row buffer is cleared by the finalise contract:
// rows are written completely only if 256*V % C == 0 or C % (256*V) == 0 handled below.
int bn_bwd_grid(size_t elems, int C, int dtype) {
  const int V = dtype == BF16 ? 8 : 4;
  return elem_grid(elems / V, C, V, 256);
}

template <typename T>
__global__ void zero_f32_kernel(float* p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0.f;
}

hipError_t bn_bwd_reduce_launch(const BnBwdSet& q, const BnBwdSet* other, size_t elems, int C, int dtype, hipStream_t s) {
  const int V = dtype == BF16 ? 8 : 4;
  const int grid = bn_bwd_grid(elems, C, dtype);
  if (C > 256 * V) {  // a block's row is only partly written: clear the rows first
    const size_t n = (size_t)grid * 2 * C;
    DDG_LAUNCH(zero_f32_kernel<float>, dim3(256), dim3(256), 0, s, q.partial, n);
    if (other) DDG_LAUNCH(zero_f32_kernel<float>, dim3(256), dim3(256), 0, s, other->partial, n);
  }
  const BnBwdSet& o = other ? *other : q;
  if (dtype == BF16) DDG_LAUNCH(bn_bwd_reduce_kernel<bf16_t>, dim3(grid, other ? 2 : 1), dim3(256), 0, s, q, o, elems / 8, C);
  else DDG_LAUNCH(bn_bwd_reduce_kernel<float>, dim3(grid, other ? 2 : 1), dim3(256), 0, s, q, o, elems / 4, C);
  return hipGetLastError();
}

// dz = A*g + B*z + C0 (coefficients from bn_bwd_finalize_launch, or derived from the rows)
// blockIdx.y: one of two layers of the same shape
template <typename T>
__global__ __launch_bounds__(256) void bn_bwd_apply_kernel(BnBwdSet q0, BnBwdSet q1, size_t nvec, int C) {
  const BnBwdSet& q = blockIdx.y ? q1 : q0;
  const T* __restrict__ dy = reinterpret_cast<const T*>(q.dy);
  const T* __restrict__ mask = reinterpret_cast<const T*>(q.mask);
  const float* __restrict__ mscale = q.mscale;
  const float* __restrict__ mshift = q.mshift;
  const T* __restrict__ z = reinterpret_cast<const T*>(q.z);
  const float* coef = q.coef;
  const BnBwdRows rows = q.rows;
  T* __restrict__ dz = reinterpret_cast<T*>(q.dz);
  constexpr int V = Store<T>::VEC;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int c0 = (int)((i * V) % C);
  __shared__ float s_coef[3 * STATS_CMAX];
  if (rows.partial) { bn_bwd_from_rows_rt(rows, C, s_coef, blockIdx.x == 0); coef = s_coef; }
  float A[V], B[V], C0[V], ms[V], mh[V];
#pragma unroll
  for (int j = 0; j < V; ++j) {
    A[j] = coef[c0 + j]; B[j] = coef[C + c0 + j]; C0[j] = coef[2 * C + c0 + j];
    ms[j] = mscale ? mscale[c0 + j] : 1.f; mh[j] = mscale ? mshift[c0 + j] : 0.f;
  }
  for (; i < nvec; i += stride) {
    float g[V], zz[V];
    Store<T>::load_vec(dy + i * V, g);
    Store<T>::load_vec(z + i * V, zz);
    if (mask) {
      float mk[V];
      Store<T>::load_vec(mask + i * V, mk);
#pragma unroll
      for (int j = 0; j < V; ++j) g[j] = (mk[j] * ms[j] + mh[j]) > 0.f ? g[j] : 0.f;
    }
#pragma unroll
    for (int j = 0; j < V; ++j) g[j] = A[j] * g[j] + (B[j] * zz[j] + C0[j]);
    Store<T>::store_vec(dz + i * V, g);
  }
}

// The same operation without a loop, for final coefficients and 256*V % C == 0 (a thread's
// channels are the same for all its vectors): a workgroup owns 256*U consecutive vectors, a
// thread requests all its tensor data first and its per-channel constants (16-byte loads) while
// that is in flight.
template <typename T, int U>
__global__ __launch_bounds__(256) void bn_bwd_apply_chunk_kernel(const T* __restrict__ dy, const T* __restrict__ mask,
                                                                 const float* __restrict__ mscale,
                                                                 const float* __restrict__ mshift,
                                                                 const T* __restrict__ z, const float* __restrict__ coef,
                                                                 T* __restrict__ dz, size_t nvec, int C) {
  constexpr int V = Store<T>::VEC;
  typedef typename Store<T>::vec_t vec_t;
  const size_t base = (size_t)blockIdx.x * (256 * U) + threadIdx.x;
  const int c0 = (int)((threadIdx.x * V) % C);
  vec_t gq[U], zq[U], mq[U];
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const size_t i = base + (size_t)j * 256;
    if (i < nvec) {
      gq[j] = *reinterpret_cast<const vec_t*>(dy + i * V);
      zq[j] = *reinterpret_cast<const vec_t*>(z + i * V);
      if (mask && mask != z) mq[j] = *reinterpret_cast<const vec_t*>(mask + i * V);
    }
  }
  float A[V], B[V], C0[V], ms[V], mh[V];
#pragma unroll
  for (int j = 0; j < V; j += 4) {
    *reinterpret_cast<float4*>(&A[j]) = *reinterpret_cast<const float4*>(coef + c0 + j);
    *reinterpret_cast<float4*>(&B[j]) = *reinterpret_cast<const float4*>(coef + C + c0 + j);
    *reinterpret_cast<float4*>(&C0[j]) = *reinterpret_cast<const float4*>(coef + 2 * C + c0 + j);
    if (mscale) {
      *reinterpret_cast<float4*>(&ms[j]) = *reinterpret_cast<const float4*>(mscale + c0 + j);
      *reinterpret_cast<float4*>(&mh[j]) = *reinterpret_cast<const float4*>(mshift + c0 + j);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) { ms[j + e] = 1.f; mh[j + e] = 0.f; }
    }
  }
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const size_t i = base + (size_t)j * 256;
    if (i >= nvec) continue;
    float g[V], zz[V];
    Store<T>::unpack_vec(gq[j], g);
    Store<T>::unpack_vec(zq[j], zz);
    if (mask) {
      float mk[V];
      Store<T>::unpack_vec(mask != z ? mq[j] : zq[j], mk);
#pragma unroll
      for (int e = 0; e < V; ++e) g[e] = (mk[e] * ms[e] + mh[e]) > 0.f ? g[e] : 0.f;
    }
#pragma unroll
    for (int e = 0; e < V; ++e) g[e] = A[e] * g[e] + (B[e] * zz[e] + C0[e]);
    Store<T>::store_vec(dz + i * V, g);
  }
}

template <typename T>
static bool bn_bwd_apply_chunked(const T* dy, const T* mask, const float* mscale, const float* mshift, const T* z,
                                 const float* coef, T* dz, size_t nvec, int C, hipStream_t s) {
  constexpr int V = Store<T>::VEC;
  // final coefficients, a thread's channels fixed, 16-byte aligned per-channel vectors
  if (!coef || (256 * V) % C != 0 || C % 4 != 0) return false;
  if (((uintptr_t)coef | (uintptr_t)mscale | (uintptr_t)mshift) & 15u) return false;
  if (nvec >= (size_t)512 * 1024)
    DDG_LAUNCH((bn_bwd_apply_chunk_kernel<T, 2>), dim3((unsigned)((nvec + 511) / 512)), dim3(256), 0, s, dy, mask, mscale,
               mshift, z, coef, dz, nvec, C);
  else
    DDG_LAUNCH((bn_bwd_apply_chunk_kernel<T, 1>), dim3((unsigned)((nvec + 255) / 256)), dim3(256), 0, s, dy, mask, mscale,
               mshift, z, coef, dz, nvec, C);
  return true;
}

hipError_t bn_bwd_apply_launch(const BnBwdSet& q, const BnBwdSet* other, size_t elems, int C, int dtype, hipStream_t s) {
  const bool rows = q.rows.partial != nullptr;
  if (other && (other->rows.partial != nullptr) != rows) return hipErrorInvalidValue;
  const int maxb = rows ? 512 : 2048;
  if (!rows && !other) {
    const bool done = dtype == BF16
        ? bn_bwd_apply_chunked<bf16_t>((const bf16_t*)q.dy, (const bf16_t*)q.mask, q.mscale, q.mshift, (const bf16_t*)q.z, q.coef,
                                       (bf16_t*)q.dz, elems / 8, C, s)
        : bn_bwd_apply_chunked<float>((const float*)q.dy, (const float*)q.mask, q.mscale, q.mshift, (const float*)q.z, q.coef,
                                      (float*)q.dz, elems / 4, C, s);
    if (done) return hipGetLastError();
  }
  const BnBwdSet& o = other ? *other : q;
  const int V = dtype == BF16 ? 8 : 4;
  const dim3 grid(elem_grid(elems / V, C, V, maxb), other ? 2 : 1);
  if (dtype == BF16) DDG_LAUNCH(bn_bwd_apply_kernel<bf16_t>, grid, dim3(256), 0, s, q, o, elems / 8, C);
  else DDG_LAUNCH(bn_bwd_apply_kernel<float>, grid, dim3(256), 0, s, q, o, elems / 4, C);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// Running batch-norm estimates (for evaluation) of all layers of a module (see forward_tail_kernel):
//   rmean <- (1-rho)*rmean + rho*mean,  rvar <- (1-rho)*rvar + rho*var*m/(m-1)
// with the batch statistics of the forward pass that just ran (var = 1/invstd^2 - eps), and
// the per-channel vectors the evaluation forward normalises with:
//   escale = gamma/sqrt(rvar + eps),  eshift = beta - rmean*escale.
// ---------------------------------------------------------------------------------
__device__ __forceinline__ void running_update_body(const RunDesc& d, float rho, int c) {
  if (c >= d.C) return;
  const float is = d.invstd[c];
  const float var = 1.f / (is * is) - d.eps;
  d.rmean[c] = (1.f - rho) * d.rmean[c] + rho * d.mean[c];
  d.rvar[c] = (1.f - rho) * d.rvar[c] + rho * (var * d.count / (d.count - 1.f));
}

__global__ __launch_bounds__(256) void eval_vectors_kernel(const RunDesc* __restrict__ descs) {
  const RunDesc d = descs[blockIdx.y];
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= d.C) return;
  const float sc = d.gamma[c] / sqrtf(d.rvar[c] + d.eps);
  d.escale[c] = sc;
  d.eshift[c] = d.beta[c] - d.rmean[c] * sc;
}

hipError_t eval_vectors_launch(const RunDesc* dev_descs, int n, int max_c, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  DDG_LAUNCH(eval_vectors_kernel, dim3((max_c + 255) / 256, n), dim3(256), 0, s, dev_descs);
  return hipGetLastError();
}

// Sum / maximum over a workgroup of four waves in a fixed order; every thread gets the result. sh: 4
// floats of LDS that no other step uses between two barriers.
__device__ __forceinline__ float block_sum(float v, float* sh) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  return ((sh[0] + sh[1]) + sh[2]) + sh[3];
}
__device__ __forceinline__ float block_max(float v, float* sh) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  return fmaxf(fmaxf(sh[0], sh[1]), fmaxf(sh[2], sh[3]));
}

// mean of the per-sample losses (evaluation; training gets it from head_wgrad_kernel)
__global__ __launch_bounds__(256) void loss_mean_kernel(const float* __restrict__ loss_n, int N, float* __restrict__ out) {
  __shared__ float sh[4];
  float l = 0.f;
  for (int n = threadIdx.x; n < N; n += 256) l += loss_n[n];
  l = block_sum(l, sh);
  if (threadIdx.x == 0) *out = l / (float)N;
}

// ---------------------------------------------------------------------------------
// Head. Small: N x C x classes is a few hundred thousand operations, so what it costs is the length
// of its chains of loads and sums. Operands are brought to LDS in one round trip (STAGED: wherever they fit),
// and the sums run there in plain ascending order.
// ---------------------------------------------------------------------------------
constexpr size_t HEAD_LDS_MAX = (size_t)96 << 10;

// Per sample (one workgroup of 256 threads): global average pool, logits, stable softmax, loss,
// dlogits = (p - onehot)/N, and dh = dlogits * fcw / HW broadcast over the pixels.
// Dynamic LDS: 2*C + 2*classes + 256 floats, and with STAGED the classifier, rows of C + 1 floats.
template <typename T, bool STAGED>
__global__ __launch_bounds__(256) void head_sample_kernel(const T* __restrict__ h, const float* __restrict__ fcw,
                                                          const float* __restrict__ fcb,
                                                          const int32_t* __restrict__ labels,
                                                          float* __restrict__ pooled, float* __restrict__ dlogits,
                                                          float* __restrict__ loss_n, T* __restrict__ dh, int N,
                                                          int HW, int C, int classes, float* __restrict__ logits_out) {
  extern __shared__ float sm[];
  __shared__ float s_w[4];
  float* s_pool = sm;               // [C]
  float* s_dh = sm + C;             // [C]
  float* s_lg = sm + 2 * C;         // [classes]
  float* s_dl = s_lg + classes;     // [classes]
  float* s_red = s_dl + classes;    // [256]
  float* s_fc = s_red + 256;        // STAGED: [classes][C + 1]
  const int n = blockIdx.x, tid = threadIdx.x;
  if (STAGED) {
    const int total = classes * C;
#pragma unroll 8
    for (int e = tid; e < total; e += 256) s_fc[e + e / C] = fcw[e];
  }
  auto weight = [&](int j, int c) __attribute__((always_inline)) { return STAGED ? s_fc[j * (C + 1) + c] : fcw[(size_t)j * C + c]; };
  // pool: thread (channel lane cl, pixel class g); pixel classes are added in order afterwards
  const int cpt = C < 256 ? C : 256, groups = 256 / cpt;
  const int cl = tid % cpt, g = tid / cpt;
  for (int c0 = 0; c0 < C; c0 += cpt) {
    const int c = c0 + cl;
    float a = 0.f;
    if (g < groups && c < C) {
      const T* p = h + (size_t)n * HW * C + c;
#pragma unroll 16
      for (int i = g; i < HW; i += groups) a += Store<T>::load1(p + (size_t)i * C);
    }
    s_red[tid] = a;
    __syncthreads();
    if (g == 0 && c < C) {
      float t = 0.f;
      for (int q = 0; q < groups; ++q) t += s_red[q * cpt + cl];
      t /= (float)HW;
      s_pool[c] = t;
      pooled[(size_t)n * C + c] = t;
    }
    __syncthreads();
  }
  // logits
  for (int j = tid; j < classes; j += 256) {
    float a = fcb[j];
#pragma unroll 16
    for (int c = 0; c < C; ++c) a += weight(j, c) * s_pool[c];
    s_lg[j] = a;
    if (logits_out) logits_out[(size_t)n * classes + j] = a;
  }
  __syncthreads();
  float mx = s_lg[0];
  for (int j = tid; j < classes; j += 256) mx = fmaxf(mx, s_lg[j]);
  mx = block_max(mx, s_w);
  for (int j = tid; j < classes; j += 256) s_dl[j] = expf(s_lg[j] - mx);
  __syncthreads();
  float den = 0.f;
#pragma unroll 16
  for (int j = 0; j < classes; ++j) den += s_dl[j];
  // a label outside [0, classes) has no class to point at: that sample's loss (and with it the
  // mean loss) is NaN, so the caller sees it, and nothing outside the logits is read
  const int y = labels[n];
  const bool y_ok = (unsigned)y < (unsigned)classes;
  __syncthreads();
  for (int j = tid; j < classes; j += 256) {
    const float d = (s_dl[j] / den - (j == y ? 1.f : 0.f)) / (float)N;
    s_dl[j] = d;
    dlogits[(size_t)n * classes + j] = d;
  }
  if (tid == 0) loss_n[n] = y_ok ? -(s_lg[y] - mx - logf(den)) : __builtin_nanf("");
  if (!dh) return;
  __syncthreads();
  for (int c = tid; c < C; c += 256) {
    float a = 0.f;
#pragma unroll 16
    for (int j = 0; j < classes; ++j) a += s_dl[j] * weight(j, c);
    s_dh[c] = Store<T>::round(a / (float)HW);
  }
  __syncthreads();
  // broadcast over the pixels, 4 channels per store
  const int c4n = C / 4;
  for (int e = tid; e < HW * c4n; e += 256) {
    const int i = e / c4n, c = (e - i * c4n) * 4;
    Store<T>::store4(dh + ((size_t)n * HW + i) * C + c, s_dh[c], s_dh[c + 1], s_dh[c + 2], s_dh[c + 3]);
  }
}

// One workgroup of 1024 threads per class j: dfcw[j][:] = sum_n dlogits[n][j] * pooled[n][:],
// dfcb[j]; thread (channel lane, sample class g) of the first 256 adds samples g, g+groups, ... in order,
// then the classes are added in order. Workgroup 0 also writes the mean loss. STAGED: dynamic LDS
// holds [N][C] of pooled and [N] of dlogits.
template <bool STAGED>
__global__ __launch_bounds__(1024) void head_wgrad_kernel(const float* __restrict__ pooled,
                                                          const float* __restrict__ dlogits,
                                                          const float* __restrict__ loss_n, float* __restrict__ dfcw,
                                                          float* __restrict__ dfcb, float* loss_out, int N, int C,
                                                          int classes) {
  extern __shared__ float sm[];
  __shared__ float s_red[256], s_b[256], s_l[256];
  const int j = blockIdx.x, tid = threadIdx.x;
  float* s_pool = sm;
  float* s_dl = sm + (size_t)N * C;
  if (STAGED) {
    for (int n = tid; n < N; n += 1024) s_dl[n] = dlogits[(size_t)n * classes + j];
    const float4* p4 = reinterpret_cast<const float4*>(pooled);
#pragma unroll 8
    for (int e = tid; e < N * C / 4; e += 1024) reinterpret_cast<float4*>(s_pool)[e] = p4[e];
  }
  // 256 partial sums over samples of the bias gradient (and the mean loss)
  if (tid < 256) {
    float a = 0.f, l = 0.f;
    for (int n = tid; n < N; n += 256) {
      a += dlogits[(size_t)n * classes + j];
      if (j == 0) l += loss_n[n];
    }
    s_b[tid] = a; s_l[tid] = l;
  }
  __syncthreads();
  const int cpt = C < 256 ? C : 256, groups = 256 / cpt;
  const int cl = tid % cpt, g = tid / cpt;
  for (int c0 = 0; c0 < C; c0 += cpt) {
    const int c = c0 + cl;
    float a = 0.f;
    if (tid < 256 && g < groups && c < C) {
#pragma unroll 16
      for (int n = g; n < N; n += groups)
        a += (STAGED ? s_dl[n] : dlogits[(size_t)n * classes + j]) * (STAGED ? s_pool[n * C + c] : pooled[(size_t)n * C + c]);
    }
    if (tid < 256) s_red[tid] = a;
    __syncthreads();
    if (tid < 256 && g == 0 && c < C) {
      float t = 0.f;
      for (int q = 0; q < groups; ++q) t += s_red[q * cpt + cl];
      dfcw[(size_t)j * C + c] = t;
    }
    __syncthreads();
  }
  // added in order by one thread each, beside the sums above's last stores
  const int terms = N < 256 ? N : 256;
  if (tid == 256) {
    float t = 0.f;
#pragma unroll 16
    for (int q = 0; q < terms; ++q) t += s_b[q];
    dfcb[j] = t;
  }
  if (tid == 320 && j == 0 && loss_out) {
    float t = 0.f;
#pragma unroll 16
    for (int q = 0; q < terms; ++q) t += s_l[q];
    *loss_out = t / (float)N;
  }
}

template <bool STAGED>
static hipError_t head_wgrad_run(const HeadArgs& a, size_t lds, hipStream_t s) {
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&head_wgrad_kernel<STAGED>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)HEAD_LDS_MAX);
  if (attr != hipSuccess) return attr;
  DDG_LAUNCH(head_wgrad_kernel<STAGED>, dim3(a.classes), dim3(1024), lds, s, a.pooled, a.dlogits, a.loss_n, a.dfcw, a.dfcb,
             a.loss_out, a.N, a.C, a.classes);
  return hipGetLastError();
}

template <typename T, bool STAGED>
static hipError_t head_sample_run(const HeadArgs& a, size_t lds, hipStream_t s) {
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&head_sample_kernel<T, STAGED>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)HEAD_LDS_MAX);
  if (attr != hipSuccess) return attr;
  DDG_LAUNCH((head_sample_kernel<T, STAGED>), dim3(a.N), dim3(256), lds, s, (const T*)a.h, a.fcw, a.fcb, a.labels,
             a.pooled, a.dlogits, a.loss_n, (T*)a.dh, a.N, a.HW, a.C, a.classes, a.logits_out);
  return hipGetLastError();
}

template <typename T>
static hipError_t head_sample_any(const HeadArgs& a, hipStream_t s) {
  const size_t lds = (size_t)(2 * a.C + 2 * a.classes + 256) * sizeof(float);
  const size_t with_fc = lds + (size_t)a.classes * (a.C + 1) * sizeof(float);
  return with_fc <= HEAD_LDS_MAX ? head_sample_run<T, true>(a, with_fc, s) : head_sample_run<T, false>(a, lds, s);
}

hipError_t head_launch(const HeadArgs& a, hipStream_t s) {
  if (a.C % 4 != 0) return hipErrorInvalidValue;
  hipError_t e = a.dtype == BF16 ? head_sample_any<bf16_t>(a, s) : head_sample_any<float>(a, s);
  if (e != hipSuccess) return e;
  if (a.sums_later) return hipGetLastError();
  if (!a.dfcw) {   // evaluation: no gradients; the mean loss if asked for
    if (a.loss_out) DDG_LAUNCH(loss_mean_kernel, dim3(1), dim3(256), 0, s, a.loss_n, a.N, a.loss_out);
    return hipGetLastError();
  }
  const size_t lds = (size_t)a.N * (a.C + 1) * sizeof(float);
  return lds + 3 * 256 * sizeof(float) <= HEAD_LDS_MAX ? head_wgrad_run<true>(a, lds, s) : head_wgrad_run<false>(a, 0, s);
}

// beta1^n and beta2^n of Adam's next update.
__global__ void adam_advance_kernel(double* pw, double b1, double b2) { pw[0] *= b1; pw[1] *= b2; }

hipError_t adam_advance_launch(double* pw, float b1, float b2, hipStream_t s) {
  DDG_LAUNCH(adam_advance_kernel, dim3(1), dim3(1), 0, s, pw, (double)b1, (double)b2);
  return hipGetLastError();
}

__global__ void set_scalar_kernel(float* dst, float v) { *dst = v; }

hipError_t set_scalar_launch(float* dst, float v, hipStream_t s) {
  DDG_LAUNCH(set_scalar_kernel, dim3(1), dim3(1), 0, s, dst, v);
  return hipGetLastError();
}

__device__ __forceinline__ void copy_body(const uint4* __restrict__ src, uint4* __restrict__ dst, size_t bytes, unsigned block, unsigned blocks) {
  const size_t nvec = bytes / 16;
  for (size_t i = (size_t)block * 256 + threadIdx.x; i < nvec; i += (size_t)blocks * 256) dst[i] = src[i];
  if (block == 0)
    for (size_t b = nvec * 16 + threadIdx.x; b < bytes; b += 256)
      reinterpret_cast<unsigned char*>(dst)[b] = reinterpret_cast<const unsigned char*>(src)[b];
}
__global__ __launch_bounds__(256) void copy_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, size_t bytes) {
  copy_body(src, dst, bytes, blockIdx.x, gridDim.x);
}
// What ends a training forward pass, in one launch: the running estimates (the first n*per workgroups) and the copy of the
// module's input into its ring (the rest). Neither needs the other; each was a launch of 4 to 5 us that a stream waits for
// (16 iterations, one of the two launches saved: 4 images in fp32 3.73 -> 3.66 ms, ResNet-20 bf16 batch 37 4.98 -> 4.91).
__global__ __launch_bounds__(256) void forward_tail_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, size_t bytes,
                                                           const RunDesc* __restrict__ descs, int n, int per, float rho) {
  const int b = blockIdx.x, first = n * per;
  if (b < first) running_update_body(descs[b / per], rho, b % per * 256 + threadIdx.x);
  else copy_body(src, dst, bytes, b - first, gridDim.x - first);
}

static int copy_grid(size_t bytes) {
  const size_t g = (bytes / 16 + 255) / 256;
  return g < 1 ? 1 : g > 2048 ? 2048 : (int)g;
}

hipError_t forward_tail_launch(const void* src, void* dst, size_t bytes, const RunDesc* dev_descs, int n, int max_c, float rho, hipStream_t s) {
  const int per = (max_c + 255) / 256, grid = n * per + (src ? copy_grid(bytes) : 0);
  if (grid <= 0) return hipSuccess;
  DDG_LAUNCH(forward_tail_kernel, dim3(grid), dim3(256), 0, s, (const uint4*)src, (uint4*)dst, bytes, dev_descs, n, per, rho);
  return hipGetLastError();
}

hipError_t copy_launch(const void* src, void* dst, size_t bytes, hipStream_t s) {
  DDG_LAUNCH(copy_kernel, dim3(copy_grid(bytes)), dim3(256), 0, s, (const uint4*)src, (uint4*)dst, bytes);
  return hipGetLastError();
}

template <typename T>
__global__ void to_f32_kernel(const T* __restrict__ src, float* __restrict__ dst, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    dst[i] = Store<T>::load1(src + i);
}

hipError_t to_f32_launch(const void* src, float* dst, size_t elems, int dtype, hipStream_t s) {
  int grid = (int)((elems + 255) / 256);
  if (grid > 2048) grid = 2048;
  if (grid < 1) grid = 1;
  if (dtype == BF16) DDG_LAUNCH(to_f32_kernel<bf16_t>, dim3(grid), dim3(256), 0, s, (const bf16_t*)src, dst, elems);
  else DDG_LAUNCH(to_f32_kernel<float>, dim3(grid), dim3(256), 0, s, (const float*)src, dst, elems);
  return hipGetLastError();
}

}  // namespace ddg
