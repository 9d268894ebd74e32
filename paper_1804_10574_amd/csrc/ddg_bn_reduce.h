// Sums of the batch-norm backward (g = dy masked, partial sums of g and g*xhat), 256 threads; a header so that a launch that
// carries several kinds of work can include it.
#pragma once
#include "ddg_device.h"
#include "ddg_kernels.h"

namespace ddg {

// bx of gx: this workgroup's index among those that walk over the tensor (one partial row each).
template <typename T>
__device__ __forceinline__ void bn_bwd_reduce_body(const BnBwdSet& q, size_t nvec, int C, int bx, int gx) {
  const T* __restrict__ dy = reinterpret_cast<const T*>(q.dy);
  const T* __restrict__ mask = reinterpret_cast<const T*>(q.mask);
  const float* __restrict__ mscale = q.mscale;
  const float* __restrict__ mshift = q.mshift;
  const T* __restrict__ z = reinterpret_cast<const T*>(q.z);
  const float* __restrict__ mean = q.mean;
  const float* __restrict__ invstd = q.invstd;
  float* __restrict__ partial = q.partial;
  constexpr int V = Store<T>::VEC;
  const size_t stride = (size_t)gx * 256;
  size_t i = (size_t)bx * 256 + threadIdx.x;
  const int c0 = (int)((i * V) % C);
  float mu[V], is[V], s1[V], s2[V], ms[V], mh[V];
#pragma unroll
  for (int j = 0; j < V; ++j) {
    mu[j] = mean[c0 + j]; is[j] = invstd[c0 + j]; s1[j] = 0.f; s2[j] = 0.f;
    ms[j] = mscale ? mscale[c0 + j] : 1.f; mh[j] = mscale ? mshift[c0 + j] : 0.f;
  }
  // four vectors per trip, all requested before any is used (the sums keep their order)
  typedef typename Store<T>::vec_t vec_t;
  constexpr int U = 4;
  const bool own_mask = mask && mask != z;
  for (; i < nvec; i += U * stride) {
    vec_t gq[U], zq[U], mq[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const size_t iu = i + u * stride;
      if (iu < nvec) {
        gq[u] = *reinterpret_cast<const vec_t*>(dy + iu * V);
        zq[u] = *reinterpret_cast<const vec_t*>(z + iu * V);
        if (own_mask) mq[u] = *reinterpret_cast<const vec_t*>(mask + iu * V);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (i + u * stride >= nvec) continue;
      float g[V], zz[V];
      Store<T>::unpack_vec(gq[u], g);
      Store<T>::unpack_vec(zq[u], zz);
      if (mask) {
        float mk[V];
        Store<T>::unpack_vec(own_mask ? mq[u] : zq[u], mk);
#pragma unroll
        for (int j = 0; j < V; ++j) g[j] = (mk[j] * ms[j] + mh[j]) > 0.f ? g[j] : 0.f;
      }
#pragma unroll
      for (int j = 0; j < V; ++j) {
        s1[j] += g[j];
        s2[j] += g[j] * ((zz[j] - mu[j]) * is[j]);
      }
    }
  }
  // Threads with equal (threadIdx.x*V) % C hold the same channels; their sums are added in thread
  // order, one thread per sum. (Two threads that added all sums of 128 rows were most of this kernel for
  // 16 channels: 11.3 -> 7.2 us at 37 x 32 x 32 x 16 in a running
  // pipeline.)
  const int per = C / V < 256 ? C / V : 256;  // distinct channel vectors among the block's threads
  __shared__ float red[2][256][V + 1];
#pragma unroll
  for (int j = 0; j < V; ++j) { red[0][threadIdx.x][j] = s1[j]; red[1][threadIdx.x][j] = s2[j]; }
  __syncthreads();
  // sum e of 2 * per * V: (which, channel vector, element); block b, thread t covers channels ((b*256+t)*V) % C
  const int nper = per * V, rows = 256 / per;
  for (int e = threadIdx.x; e < 2 * nper; e += 256) {
    const int which = e / nper, k = e - which * nper, t0 = k / V, j = k - t0 * V;
    float t = 0.f;
#pragma unroll 16
    for (int r = 0; r < rows; ++r) t += red[which][r * per + t0][j];
    const int cb = (int)((((size_t)bx * 256 + t0) * V) % C);
    partial[((size_t)bx * 2 + which) * C + cb + j] = t;
  }
}

}  // namespace ddg
