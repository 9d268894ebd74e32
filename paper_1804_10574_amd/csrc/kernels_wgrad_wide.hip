// Weight gradient of wide bf16 layers (1x1 and 3x3, stride 1; input and output channels
// multiples of 128): the companion of conv_wide_kernel.
//
//   dW[co][tap][ci] = sum over pixels p of dz[p][co] * x[pix(p, tap)][ci]
//
// A GEMM whose contraction index, the pixel, is the slow index of both NHWC operands. A
// workgroup owns a 128 (co) x 128 (ci) tile of one tap and a slice of the pixels; it stages
// 64 pixels of both operands per step exactly as they lie in memory ([pixel][128 channels],
// row stride 288 bytes) and takes MFMA fragments out of LDS with the transposing read of
// gfx950 (ds_read_b64_tr_b16: a lane ends up with 8 consecutive pixels of one channel). A tap
// is a shifted pixel row with zeros outside the image. Global loads of the next two steps are in
// flight while a step is contracted: with one step ahead the loop ran at the memory latency, 1.2 us a
// step, whatever its size. 6272 pixels: 1024 x 256 channels 14.4 -> 12.5 us, 256 x 256 3x3 23.9 -> 19.9 us.
//
// Eight waves as 2 (pixel halves of a step) x 2 (co) x 2 (ci), 64 x 64 each = 16 accumulator
// tiles of mfma_f32_16x16x32_bf16; the two pixel halves meet in LDS at the end, so a workgroup
// writes one tile for twice the matrix work in flight. The pixel slices (split-K) give the
// launch enough workgroups; each writes an fp32 partial tile [split][co][tap*Cin + ci], which
// wgrad_reduce_all_kernel adds in a fixed order (deterministic). The partial tiles are what
// this kernel costs in memory traffic (64 KB per workgroup, written here and read by the
// reduction), hence one workgroup of eight waves per compute unit rather than two of four.
#include "ddg_conv_wide.h"
#include <cstdlib>

namespace ddg {

struct WgradWideArgs {
  const bf16_t* x;       // [M][Cin]
  const bf16_t* dz;      // [M][Cout]
  const float* scale;    // optional per-channel transform of x: relu(x*scale+shift)
  const float* shift;
  float* partial;        // [splits][Cout][J], J = taps*Cin
  int M, H, W, HW, Cin, Cout, R, J;
  int nsplits;           // pixel slices: slice i covers 64-pixel steps [i*nsteps/nsplits, (i+1)*nsteps/nsplits)
  int nsteps;            // ceil(M/64)
  int cit, taps;         // Cin/128, R*R: tile index = (cot*taps + tap)*cit + ci tile
  int by_xcd;            // 1: workgroups are renumbered so that a pixel slice stays on one XCD
};

namespace wgw {
constexpr int BP = 64;                     // pixels per step
constexpr int ROW = 256 + 32;              // bytes per staged pixel (128 channels), 32 modulo 128
constexpr int OPB = BP * ROW;              // one operand, one buffer: 18432
constexpr int BUF = 2 * OPB;
constexpr int LDS = 2 * BUF;               // 73728
}

typedef short wtr4_t __attribute__((ext_vector_type(4)));
// 8-pixel fragment of one channel per lane: two transposing reads 4 pixels apart
__device__ __forceinline__ uint4 wide_frag_tr(const unsigned char* p) {
  typedef wtr4_t __attribute__((address_space(3))) * lds_ptr_t;
  const wtr4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(p));
  const wtr4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(p + 4 * wgw::ROW));
  const uint2 l = __builtin_bit_cast(uint2, lo), h = __builtin_bit_cast(uint2, hi);
  return make_uint4(l.x, l.y, h.x, h.y);
}

// A thread's share of one step on its way to LDS: rows prow and prow + 32 of dz and x, and which of them exist
// (bits 0, 1: the dz rows lie inside the tensor; bits 2, 3: the x rows lie inside the image).
struct WgwSet { uint4 z0, z1, x0, x1; unsigned in; };

template <int R, bool XFORM>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void wgrad_wide_kernel(WgradWideArgs a) {
  using namespace wgw;
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lg = lane >> 4;
  const int wa = wave & 1, wb = (wave >> 1) & 1;     // co half, ci half
  const int kg = wave >> 2;                          // pixels 32*kg .. 32*kg + 31 of every step
  // Workgroups go to the 8 XCDs round-robin in launch order. All tiles of one pixel slice read
  // the same rows of x and dz, so the (slice, tile) pairs are numbered slice-major and XCD j is
  // given the j-th eighth of that sequence: the rows of a slice then come from memory once into
  // one XCD's L2 (two at a boundary) and every other tile finds them there.
  int tile = blockIdx.x, split = blockIdx.y;
  if (a.by_xcd) {
    const int T = gridDim.x * gridDim.y, L = blockIdx.x + gridDim.x * blockIdx.y;
    const int xcd = L & 7, q = T >> 3, r = T & 7;
    const int V = xcd * q + (xcd < r ? xcd : r) + (L >> 3);   // XCD j holds q (+1 if j < r) workgroups
    split = V / (int)gridDim.x;
    tile = V - split * (int)gridDim.x;
  }
  const int cit = tile % a.cit;
  const int tap = (tile / a.cit) % (R * R);
  const int cot = tile / (a.cit * R * R);
  const int co0 = cot * 128, ci0 = cit * 128;
  const int dr = R == 3 ? tap / 3 - 1 : 0, ds = R == 3 ? tap % 3 - 1 : 0;
  const int s0 = split * a.nsteps / a.nsplits;
  const int s1 = (split + 1) * a.nsteps / a.nsplits;

  // staging map: 16-byte unit tid + q*512 of a 64 x 128 tile = pixel (tid>>4) + 32*q, chunk tid&15
  const int ch = tid & 15, prow = tid >> 4;
  const wide_rsrc_t rz = wide_rsrc(a.dz, (size_t)a.M * a.Cout * 2), rx = wide_rsrc(a.x, (size_t)a.M * a.Cin * 2);
  const unsigned zc = (co0 + ch * 8) * 2, xc = (ci0 + ch * 8) * 2;
  // small non-negative integers divide exactly through fp32 (the host checks M < 2^22)
  const float inv_hw = 1.0f / (float)a.HW, inv_w = 1.0f / (float)a.W;
  // No load is conditional, so that the compiler's wait counts leave the newest sets in flight: a row that
  // does not exist loads the last one (a tap outside the image its own pixel) and is zeroed on the
  // way to LDS. A step past the slice repeats its last one (never used).
  auto issue = [&](WgwSet& r, int step) __attribute__((always_inline)) {
    const int st = step < s1 ? step : s1 - 1;
    r.in = 0;
    auto row = [&](int q, uint4& zq, uint4& xq) __attribute__((always_inline)) {
      const int m = st * BP + prow + 32 * q, mc = m < a.M ? m : a.M - 1;
      bool in = m < a.M;
      r.in |= (in ? 1u : 0u) << q;
      int mx = mc;
      if (R == 3) {
        const int n = (int)(((float)mc + 0.5f) * inv_hw);
        const int rem = mc - n * a.HW;
        const int hh = (int)(((float)rem + 0.5f) * inv_w);
        const int h = hh + dr, w = rem - hh * a.W + ds;
        in = in && h >= 0 && h < a.H && w >= 0 && w < a.W;
        mx = in ? mc + dr * a.W + ds : mc;
      }
      r.in |= (in ? 4u : 0u) << q;
      zq = wide_load(rz, (unsigned)mc * (unsigned)(a.Cout * 2) + zc, 0);
      xq = wide_load(rx, (unsigned)mx * (unsigned)(a.Cin * 2) + xc, 0);
    };
    row(0, r.z0, r.x0);
    row(1, r.z1, r.x1);
  };
  // per-channel constants of this thread's 8 input channels (the same in every step)
  float tsc[8], tsh[8];
  if (XFORM) {
#pragma unroll
    for (int e = 0; e < 8; ++e) { tsc[e] = a.scale[ci0 + ch * 8 + e]; tsh[e] = a.shift[ci0 + ch * 8 + e]; }
  }
  auto keep = [](uint4 v, unsigned in) __attribute__((always_inline)) {   // (all bits, or zero)
    const unsigned k = in ? 0xffffffffu : 0u;
    return make_uint4(v.x & k, v.y & k, v.z & k, v.w & k);
  };
  auto stash = [&](WgwSet r, int bufo) __attribute__((always_inline)) {
    unsigned char* Z = smem + bufo + prow * ROW + ch * 16;
    unsigned char* X = Z + OPB;
    *reinterpret_cast<uint4*>(Z) = keep(r.z0, r.in & 1u);
    *reinterpret_cast<uint4*>(Z + 32 * ROW) = keep(r.z1, r.in & 2u);
    if (XFORM) { r.x0 = wide_act(r.x0, tsc, tsh); r.x1 = wide_act(r.x1, tsc, tsh); }
    // a pixel outside the image or past the end is zero after the transform
    *reinterpret_cast<uint4*>(X) = keep(r.x0, r.in & 4u);
    *reinterpret_cast<uint4*>(X + 32 * ROW) = keep(r.x1, r.in & 8u);
  };

  f32x4_t acc[4][4];                                 // [co block][ci block]: rows = ci, columns = co
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // fragment address of (k-step 0, channel block 0): lane s of a 16-lane block points at
  // channels 4*(s%4).. of pixel lg*8 + s/4; the second read is 4 pixels further
  const int frag = (lg * 8 + (l16 >> 2)) * ROW + (l16 & 3) * 8;
  const int zoff = frag + wa * 128 + kg * 32 * ROW;   // + i*32 (channel block)
  const int xoff = OPB + frag + wb * 128 + kg * 32 * ROW;
  auto contract = [&](int bufo) __attribute__((always_inline)) {
    const unsigned char* B = smem + bufo;
    uint4 zf[4], xf[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) zf[i] = wide_frag_tr(B + zoff + i * 32);
#pragma unroll
    for (int j = 0; j < 4; ++j) xf[j] = wide_frag_tr(B + xoff + j * 32);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = Mma<bf16_t>::mma(xf[j], zf[i], acc[i][j]);
  };

  // Two sets: at the top of step s the buffer s & 1 holds step s, one set holds step s+1, and the other, free
  // since step s was stored, takes step s+2. The body is written out twice so that both are named variables.
  WgwSet ra, rb;
  issue(ra, s0);          // (the host gives every slice at least one step)
  issue(rb, s0 + 1);
  stash(ra, 0);
  __syncthreads();
#define DDG_WGW_STEP(s, rfree, rnext)                                     \
  {                                                                       \
    const int bufo = ((s) - s0) & 1 ? BUF : 0;                            \
    issue(rfree, (s) + 2);                                                \
    __builtin_amdgcn_sched_barrier(0);                                    \
    contract(bufo);                                                       \
    __builtin_amdgcn_sched_barrier(0);                                    \
    stash(rnext, BUF - bufo);                                             \
    __syncthreads();                                                      \
  }
  for (int s = s0; s < s1; s += 2) {
    DDG_WGW_STEP(s, ra, rb)
    if (s + 1 >= s1) break;
    DDG_WGW_STEP(s + 1, rb, ra)
  }
#undef DDG_WGW_STEP

  // The two pixel halves meet through LDS (the staging buffers are free after the loop's last barrier): a wave
  // keeps two of its four co blocks, hands over the other two and adds what its partner hands over, so
  // that all eight waves store. [wave][block][ci block][lane] of 16 bytes, 64 KB.
  {
    f32x4_t* ex = reinterpret_cast<f32x4_t*>(smem) + wave * 512 + lane;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) ex[(i * 4 + j) * 64] = kg ? acc[i][j] : acc[2 + i][j];
    __syncthreads();
    const f32x4_t* got = reinterpret_cast<const f32x4_t*>(smem) + (wave ^ 4) * 512 + lane;
    // lane (l16, lg) of blocks (i, j) holds co = co0 + (wa*4 + i)*16 + l16, ci = ci0 + (wb*4 + j)*16 + lg*4 + e
    float* dst = a.partial + ((size_t)split * a.Cout + co0 + wa * 64 + kg * 32 + l16) * a.J + (size_t)tap * a.Cin + ci0 + wb * 64 + lg * 4;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        *reinterpret_cast<f32x4_t*>(dst + (size_t)(i * 16) * a.J + j * 16) = (kg ? acc[2 + i][j] : acc[i][j]) + got[(i * 4 + j) * 64];
  }
}

bool wgrad_wide_ok(int Cin, int Cout, int R, int stride, int dtype) {
  if (dtype != BF16 || stride != 1 || (R != 1 && R != 3)) return false;
  if (Cin < 128 || (Cin & (Cin - 1)) != 0) return false;   // power of two: the partial tile's column is tap*Cin + ci
  return Cout % 128 == 0;
}

// Number of pixel slices (= partial tiles per output element) for a layer: enough workgroups to
// fill the GPU (one of eight waves per compute unit), at least 2 steps of 64 pixels each.
// DDG_TUNE_WGRAD_WIDE_WGS overrides the target workgroup count within [64, 2048].
int wgrad_wide_splits(int M, int Cin, int Cout, int R) {
  int target = 256;
  if (const char* e = getenv("DDG_TUNE_WGRAD_WIDE_WGS")) {
    const int v = atoi(e);
    if (v >= 64 && v <= 2048) target = v;
  }
  const int tiles = (Cout / 128) * (Cin / 128) * R * R;
  const int nsteps = (M + wgw::BP - 1) / wgw::BP;
  int splits = target / tiles;      // never more workgroups than the target: one past what fits at once costs a whole extra round
  if (splits > nsteps / 2) splits = nsteps / 2;
  return splits < 1 ? 1 : splits;
}

template <int R, bool XFORM>
static hipError_t wgrad_wide_run(const WgradWideArgs& a, dim3 grid, hipStream_t s) {
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&wgrad_wide_kernel<R, XFORM>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, wgw::LDS);
  if (attr != hipSuccess) return attr;
  DDG_LAUNCH((wgrad_wide_kernel<R, XFORM>), grid, dim3(512), wgw::LDS, s, a);
  return hipGetLastError();
}

hipError_t wgrad_wide_launch(const void* x, const void* dz, float* partial, int N, int H, int W, int Cin, int Cout,
                             int R, int splits, hipStream_t s, const float* scale, const float* shift) {
  if (!wgrad_wide_ok(Cin, Cout, R, 1, BF16) || splits < 1) return hipErrorInvalidValue;
  if ((size_t)N * H * W >= ((size_t)1 << 22)) return hipErrorInvalidValue;   // pixel indices divide through fp32 inside
  if ((size_t)N * H * W * (Cin > Cout ? Cin : Cout) >= ((size_t)1 << 31)) return hipErrorInvalidValue;   // 32-bit byte offsets (the forward launch has the same limit)
  WgradWideArgs a{};
  a.x = (const bf16_t*)x; a.dz = (const bf16_t*)dz; a.partial = partial; a.scale = scale; a.shift = shift;
  a.M = N * H * W; a.H = H; a.W = W; a.HW = H * W; a.Cin = Cin; a.Cout = Cout; a.R = R; a.J = R * R * Cin;
  a.nsteps = (a.M + wgw::BP - 1) / wgw::BP;
  if (splits > a.nsteps) return hipErrorInvalidValue;   // an empty slice
  a.nsplits = splits;
  a.by_xcd = getenv("DDG_NO_WGRAD_XCD") ? 0 : 1;
  a.cit = Cin / 128; a.taps = R * R;
  const dim3 grid((Cout / 128) * a.taps * a.cit, splits);
  if (R == 3) return scale ? wgrad_wide_run<3, true>(a, grid, s) : wgrad_wide_run<3, false>(a, grid, s);
  return scale ? wgrad_wide_run<1, true>(a, grid, s) : wgrad_wide_run<1, false>(a, grid, s);
}

}  // namespace ddg
