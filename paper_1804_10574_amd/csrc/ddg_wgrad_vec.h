// Weight-gradient kernel body with vector gathers (see kernels_wgrad.hip for the contraction); a header so that a launch that
// carries several kinds of work can include it.
#pragma once
#include "ddg_device.h"
#include "ddg_kernels.h"

namespace ddg {

// The same contraction with 16-byte (fp32) / 8-byte (bf16) gathers of x, for layers whose input
// channel count is a multiple of 4: a lane loads 4 consecutive channels of one (pixel, tap) and
// feeds them to 4 instructions, so the 16 columns of instruction e of group G are the columns
// ((G*16 + lane%16)*4 + e) of the (tap, channel) index: a permutation of the columns that only
// the write-out has to know. One load per 4 instructions instead of one per instruction.
constexpr int WGV_NG = 3;  // groups of 64 columns per wave

constexpr int WGV_LDS = 4 * WGV_NG * 4 * 16 * 17 * 4;   // bytes of LDS the body uses: the four waves' tiles meet there

// bx, by, bz: pixel slice, 16-channel block of the output channels, column group.
template <typename T>
__device__ __forceinline__ void wgrad_vec_body(const WgradArgs& a, unsigned char* smem, int bx, int by, int bz) {
  using S_ = Store<T>;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l16 = lane & 15, lg = lane >> 4;
  const int cob = by;
  const int g0 = bz * WGV_NG;
  const T* __restrict__ x = reinterpret_cast<const T*>(a.x);
  const T* __restrict__ dz = reinterpret_cast<const T*>(a.dz);
  const int cpmask = (1 << a.log2cp) - 1;
  const int ntaps = a.R * a.R;
  const int Jp = a.JB * 16;

  int jr[WGV_NG], js[WGV_NG], jc[WGV_NG];
  bool jv[WGV_NG];
#pragma unroll
  for (int g = 0; g < WGV_NG; ++g) {
    const int j = ((g0 + g) * 16 + l16) * 4;      // first of the lane's 4 columns (same tap: 4 divides the padded channel count)
    const int tap = j >> a.log2cp;
    jc[g] = j & cpmask;
    jr[g] = tap / a.R - a.pad;
    js[g] = tap % a.R - a.pad;
    jv[g] = j < Jp && tap < ntaps && jc[g] < a.Cin;
  }
  f32x4_t acc[WGV_NG][4];
#pragma unroll
  for (int g = 0; g < WGV_NG; ++g)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[g][e] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const int pq = a.P * a.Q;
  const bool fdiv = a.M < (1 << 22);
  const float inv_pq = 1.0f / (float)pq, inv_q = 1.0f / (float)a.Q;
  long m0 = ((long)bx * 4 + wave) * (long)a.steps * 4;
  // Nothing in the loop is conditional (a masked position loads element 0 and contributes a
  // zero), and the loads of step st+1 are requested before the matrix instructions of step st (three steps
  // ahead: no faster, 8 steps of 12 fp32 instructions and their addresses are what the launch costs).
  struct StepRegs { float dv; float xq[WGV_NG][4]; unsigned ok; };   // ok bit g: group g valid, bit 31: pixel valid
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
    r.dv = S_::load1(dz + ((unsigned)mm * (unsigned)a.Cout + (unsigned)(cob * 16 + l16)));
    const int ihb = p * a.stride, iwb = q * a.stride;
    unsigned okb = mv ? 0x80000000u : 0u;
#pragma unroll
    for (int g = 0; g < WGV_NG; ++g) {
      const int ih = ihb + jr[g], iw = iwb + js[g];
      const bool ok = mv && jv[g] && ih >= 0 && ih < a.H && iw >= 0 && iw < a.W;
      const unsigned off = ok ? (unsigned)((n * a.H + ih) * a.W + iw) * (unsigned)a.Cin + (unsigned)jc[g] : 0u;   // (32 bits: the host checks)
      S_::load4(x + off, r.xq[g]);
      okb |= (ok ? 1u : 0u) << g;
    }
    r.ok = okb;
  };
  auto contract = [&](StepRegs& r) __attribute__((always_inline)) {
    // (the empty statements keep the loads where they are: left to itself the compiler moves a
    // load under its predicate, and a branch around a load ends in a wait for every load in flight)
    asm volatile("" : "+v"(r.dv));
    const float dv = (r.ok >> 31) ? r.dv : 0.f;
#pragma unroll
    for (int g = 0; g < WGV_NG; ++g) {
      asm volatile("" : "+v"(r.xq[g][0]), "+v"(r.xq[g][1]), "+v"(r.xq[g][2]), "+v"(r.xq[g][3]));
      const bool ok = (r.ok >> g) & 1u;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        acc[g][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(dv, ok ? r.xq[g][e] : 0.f, acc[g][e], 0, 0, 0);
    }
  };
  StepRegs ra, rb;     // two sets, used in turn (a step past the end is masked: it adds zeros)
  issue(ra, 0);
  for (int st = 0; st < a.steps; st += 2) {
    issue(rb, st + 1);
    contract(ra);
    issue(ra, st + 2);
    contract(rb);
  }

  // sum the four waves in a fixed order, then write the partial tile (columns back in order)
  float (*red)[WGV_NG * 4][16][17] = reinterpret_cast<float (*)[WGV_NG * 4][16][17]>(smem);
#pragma unroll
  for (int g = 0; g < WGV_NG; ++g)
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < 4; ++i) red[wave][g * 4 + e][lg * 4 + i][l16] = acc[g][e][i];
  __syncthreads();
  for (int t = threadIdx.x; t < WGV_NG * 16 * 64; t += 256) {
    const int jj = t & 63, row = (t >> 6) & 15, g = t >> 10;
    const int col = jj >> 2, e = jj & 3, b = g * 4 + e;
    const int j = (g0 + g) * 64 + jj;
    if (j >= Jp) continue;
    const float v = ((red[0][b][row][col] + red[1][b][row][col]) + red[2][b][row][col]) + red[3][b][row][col];
    a.partial[((size_t)bx * a.Cout + cob * 16 + row) * Jp + j] = v;
  }
}

}  // namespace ddg
