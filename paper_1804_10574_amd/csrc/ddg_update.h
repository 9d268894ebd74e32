// Optimizer step of one parameter (momentum SGD or Adam) and its place in a layer's
// packed operands; shared by the launches that update.
#pragma once
#include "ddg_device.h"
#include "ddg_kernels.h"

namespace ddg {

// What every workgroup needs before its first parameter. Adam: pw holds beta1^n, beta2^n; every workgroup uses the powers of
// this update, and the last one to have read them (pw_readers counts, `workgroups` in all) stores them. Without pw_readers a
// launch before (adam_advance_launch) has moved them to this update.
template <bool ADAM> struct UpdStep {
  float lr, c1, c2;
  __device__ __forceinline__ void init(const UpdArgs& a, unsigned workgroups) {
    lr = a.lr_dev ? *a.lr_dev : a.lr;
    c1 = 1.f; c2 = 1.f;
    if (ADAM) {
      const double p1 = a.pw_readers ? a.pw[0] * a.b1d : a.pw[0], p2 = a.pw_readers ? a.pw[1] * a.b2d : a.pw[1];
      c1 = (float)(1.0 - p1); c2 = (float)(1.0 - p2);
      if (!a.pw_readers) return;
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
  // new value of a parameter w with gradient g and optimizer state v, m2 (moved)
  __device__ __forceinline__ float calc(const UpdArgs& a, float wi, float g, float& v, float& m2) const {
    if (ADAM) {
      const float gi = g + a.wd * wi;
      const float mi = a.b1 * v + (1.f - a.b1) * gi;
      const float vi = a.b2 * m2 + (1.f - a.b2) * gi * gi;
      v = mi; m2 = vi;
      return wi - lr * (mi / c1) / (sqrtf(vi / c2) + a.eps);
    }
    const float vi = a.mu * v + (g + a.wd * wi);
    v = vi;
    return wi - lr * vi;
  }
  // parameter e with gradient g -> its new value, stored
  __device__ __forceinline__ float step(const UpdArgs& a, size_t e, float g) const {
    float v = a.v[e], m2 = ADAM ? a.m2[e] : 0.f;
    const float wn = calc(a, a.w[e], g, v, m2);
    a.v[e] = v;
    if (ADAM) a.m2[e] = m2;
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
