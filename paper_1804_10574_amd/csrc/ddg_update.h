// Optimizer step of one parameter (momentum SGD or Adam, the formulas of sgd_kernel / adam_kernel) and its place in a layer's
// packed operands; shared by the launches that update.
#pragma once
#include "ddg_device.h"
#include "ddg_kernels.h"

namespace ddg {

// What every workgroup needs before its first parameter. Adam: pw holds beta1^n, beta2^n; every workgroup uses the powers of
// this update, and the last one to have read them (pw_readers counts, `workgroups` in all) stores them.
template <bool ADAM> struct UpdStep {
  float lr, c1, c2;
  __device__ __forceinline__ void init(const UpdArgs& a, unsigned workgroups) {
    lr = a.lr_dev ? *a.lr_dev : a.lr;
    c1 = 1.f; c2 = 1.f;
    if (ADAM) {
      const double p1 = a.pw[0] * a.b1d, p2 = a.pw[1] * a.b2d;
      c1 = (float)(1.0 - p1); c2 = (float)(1.0 - p2);
      __shared__ unsigned s_seen;
      asm volatile("" ::"v"(c1), "v"(c2));            // (read before it is counted)
      __syncthreads();
      if (threadIdx.x == 0) s_seen = atomicAdd(a.pw_readers, 1u);
      __syncthreads();
      if (threadIdx.x == 0 && s_seen + 1 == workgroups) {
        a.pw[0] = p1; a.pw[1] = p2;
        *a.pw_readers = 0u;
      }
    }
  }
  // parameter e with gradient g -> its new value, stored
  __device__ __forceinline__ float step(const UpdArgs& a, size_t e, float g) const {
    const float wi = a.w[e];
    float wn;
    if (ADAM) {
      const float gi = g + a.wd * wi;
      const float mi = a.b1 * a.v[e] + (1.f - a.b1) * gi;
      const float vi = a.b2 * a.m2[e] + (1.f - a.b2) * gi * gi;
      a.v[e] = mi; a.m2[e] = vi;
      wn = wi - lr * (mi / c1) / (sqrtf(vi / c2) + a.eps);
    } else {
      const float vi = a.mu * a.v[e] + (g + a.wd * wi);
      a.v[e] = vi;
      wn = wi - lr * vi;
    }
    a.w[e] = wn;
    return wn;
  }
};

// The new value of weight (co, ci, tap) of a layer where it stands in the two packed operands (their padding never changes).
template <typename T>
__device__ __forceinline__ void upd_pack(const UpdDesc& d, unsigned co, unsigned ci, unsigned tap, float wn) {
  constexpr int KV = Mma<T>::KV;
  const unsigned RR = (unsigned)(d.R * d.R);
  auto at = [&](unsigned k, unsigned row, unsigned ocb) __attribute__((always_inline)) {
    return (((k / (4 * KV)) * ocb + (row >> 4)) * 64 + (k / KV % 4) * 16 + (row & 15)) * KV + k % KV;
  };
  Store<T>::store1(reinterpret_cast<T*>(d.pack_f) + at((tap << d.l2f) + ci, co, d.ocb_f), wn);
  if (d.pack_d)
    Store<T>::store1(reinterpret_cast<T*>(d.pack_d) + at(((d.mirror ? RR - 1 - tap : tap) << d.l2d) + co, ci, d.ocb_d), wn);
}

}  // namespace ddg
