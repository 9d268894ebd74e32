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
// is a shifted pixel row; where the neighbour lies outside the image both rows are zero, which the
// buffer loads give without an instruction (an offset past the tensor's end).
//
// Several layers share a launch. One layer of 6272 pixels is 16 or 36 tiles: to fill the chip alone it had
// to be cut into 7-16 slices of 6-14 steps, and start-up, the tiles' partial sums (64 KB a workgroup, written
// here and read again by the reduction) and the last wave cost more than the contraction: 45 us for the
// three layers of a bottleneck block, 1.15 GB of partial sums for 23 blocks. With layers collected until
// their tiles fill the 512 places of the chip, slices are as long as SLICE_MAX allows: 25 us a block, 0.2 GB
// (2548 pixels: 37 -> 12 us; 6272 pixels at 28x28, 512-128-512: 29 -> 9 us; 441 at 7x7, 2048-512-2048: 31 -> 21 us).
//
// Eight waves as 2 (pixel halves of a step) x 2 (co) x 2 (ci), 64 x 64 each = four accumulators of
// mfma_f32_32x32x16_bf16 (16x16x32 runs at little more than half the rate); the two pixel halves meet in LDS
// at the end. 128 registers and 72 KB of LDS: two workgroups a compute unit, one of which multiplies while
// the other waits for its rows (one workgroup with two steps in flight: 34 against 27 us). What bounds it: the
// LDS port. With the loads taken out of the loop 16 of 25 us are left, the transposing reads of 64 KB a step at about
// 64 bytes a clock and the stores of 32 KB; 6 us are matrix instructions.
#include "ddg_conv_wide.h"

namespace ddg {

struct WgwLayer {
  const bf16_t* x;       // [M][Cin]
  const bf16_t* dz;      // [M][Cout]
  const float* scale;    // optional per-channel transform of x: relu(x*scale+shift)
  const float* shift;
  float* partial;        // [splits][Cout][taps*Cin]
  int M, H, W, Cin, Cout, R, splits, wg0;   // wg0: first workgroup of the layer
};
struct WgwArgs { WgwLayer l[WGRAD_WIDE_LAYERS]; int n; };

namespace wgw {
constexpr int BP = 64;                     // pixels per step
constexpr int ROW = 256 + 32;              // bytes per staged pixel (128 channels), 32 modulo 128
constexpr int OPB = BP * ROW;              // one operand, one buffer: 18432
constexpr int BUF = 2 * OPB;
constexpr int LDS = 2 * BUF;               // 73728
constexpr int PLACES = 512;                // workgroups that run at the same time: two per compute unit
constexpr int SLICE_MAX = 49;              // steps an accumulator runs through: the fp32 sums get no longer than a layer of
                                           // 144 tiles on its own (512 channels 3x3, 3136 pixels) has always had them
constexpr unsigned NOWHERE = 0xfffffff0u;  // past the end of any tensor: the load gives zeros
}

typedef short wtr4_t __attribute__((ext_vector_type(4)));
// 8-pixel fragment of one channel per lane: two transposing reads 4 pixels apart
__device__ __forceinline__ bf16x8_t wide_frag_tr(const unsigned char* p) {
  typedef wtr4_t __attribute__((address_space(3))) * lds_ptr_t;
  const wtr4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(p));
  const wtr4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(p + 4 * wgw::ROW));
  const uint2 l = __builtin_bit_cast(uint2, lo), h = __builtin_bit_cast(uint2, hi);
  return __builtin_bit_cast(bf16x8_t, make_uint4(l.x, l.y, h.x, h.y));
}

// A thread's share of one step on its way to LDS: rows prow and prow + 32 of dz and x.
struct WgwSet { uint4 z0, z1, x0, x1; };

__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4, 4))) void wgrad_wide_kernel(WgwArgs args) {
  using namespace wgw;
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, l32 = lane & 31, half = lane >> 5;
  const int wa = wave & 1, wb = (wave >> 1) & 1;     // co half, ci half
  const int kg = wave >> 2;                          // pixels 32*kg .. 32*kg + 31 of every step
  // Workgroups go to the 8 XCDs round-robin in launch order. All tiles of one pixel slice read
  // the same rows of x and dz, so the (layer, slice, tile) triples are numbered in that order and XCD j is
  // given the j-th eighth of that sequence: the rows of a slice then come from memory once into
  // one XCD's L2 (two at a boundary) and every other tile finds them there.
  int V;
  {
    const int T = gridDim.x, L = blockIdx.x, xcd = L & 7, q = T >> 3, r = T & 7;
    V = xcd * q + (xcd < r ? xcd : r) + (L >> 3);    // XCD j holds q (+1 if j < r) workgroups
  }
  int li = 0;
  while (li + 1 < args.n && V >= args.l[li + 1].wg0) ++li;
  const WgwLayer a = args.l[li];
  V -= a.wg0;
  const int ncit = a.Cin >> 7, taps = a.R * a.R, tiles = (a.Cout >> 7) * taps * ncit;
  const int split = V / tiles, tile = V - split * tiles;
  const int cit = tile % ncit, tap = (tile / ncit) % taps, cot = tile / (ncit * taps);
  const int co0 = cot * 128, ci0 = cit * 128;
  const bool r3 = a.R == 3;
  const int dr = r3 ? tap / 3 - 1 : 0, ds = r3 ? tap % 3 - 1 : 0;
  const int nsteps = (a.M + BP - 1) / BP;
  const int s0 = split * nsteps / a.splits, s1 = (split + 1) * nsteps / a.splits;
  const int m_end = s1 * BP < a.M ? s1 * BP : a.M;

  // staging map: 16-byte unit tid + q*512 of a 64 x 128 tile = pixel (tid>>4) + 32*q, chunk tid&15
  const int ch = tid & 15, prow = tid >> 4;
  const unsigned zst = a.Cout * 2, xst = a.Cin * 2;
  const wide_rsrc_t rz = wide_rsrc(a.dz, (size_t)a.M * zst), rx = wide_rsrc(a.x, (size_t)a.M * xst);
  // pixel, image row and column, and byte offsets of the thread's two rows in the step that is requested next
  int m0 = s0 * BP + prow, h0, w0, h1, w1;
  unsigned zo = (unsigned)m0 * zst + (co0 + ch * 8) * 2, xo = (unsigned)(m0 + dr * a.W + ds) * xst + (ci0 + ch * 8) * 2;
  {
    const int HW = a.H * a.W, r0 = m0 % HW, r1 = (m0 + 32) % HW;
    h0 = r0 / a.W; w0 = r0 - h0 * a.W; h1 = r1 / a.W; w1 = r1 - h1 * a.W;
  }
  const int dh = (BP / a.W) % a.H, dw = BP % a.W;
  auto issue = [&](WgwSet& r) __attribute__((always_inline)) {
    bool i0 = m0 < m_end, i1 = m0 + 32 < m_end;
    if (r3) {
      i0 = i0 && (unsigned)(h0 + dr) < (unsigned)a.H && (unsigned)(w0 + ds) < (unsigned)a.W;
      i1 = i1 && (unsigned)(h1 + dr) < (unsigned)a.H && (unsigned)(w1 + ds) < (unsigned)a.W;
      w0 += dw; h0 += dh; if (w0 >= a.W) { w0 -= a.W; ++h0; } if (h0 >= a.H) h0 -= a.H;
      w1 += dw; h1 += dh; if (w1 >= a.W) { w1 -= a.W; ++h1; } if (h1 >= a.H) h1 -= a.H;
    }
    r.z0 = wide_load(rz, i0 ? zo : NOWHERE, 0);
    r.x0 = wide_load(rx, i0 ? xo : NOWHERE, 0);
    r.z1 = wide_load(rz, i1 ? zo + 32 * zst : NOWHERE, 0);
    r.x1 = wide_load(rx, i1 ? xo + 32 * xst : NOWHERE, 0);
    m0 += BP; zo += BP * zst; xo += BP * xst;
  };
  // per-channel constants of this thread's 8 input channels (the same in every step)
  const bool xform = a.scale != nullptr;
  float tsc[8], tsh[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) { tsc[e] = 0.f; tsh[e] = 0.f; }
  if (xform) {
#pragma unroll
    for (int e = 0; e < 8; ++e) { tsc[e] = a.scale[ci0 + ch * 8 + e]; tsh[e] = a.shift[ci0 + ch * 8 + e]; }
  }
  // (a row that does not exist is relu(shift) after the transform; its dz row is zero)
  auto stash = [&](WgwSet r, int bufo) __attribute__((always_inline)) {
    unsigned char* Z = smem + bufo + prow * ROW + ch * 16;
    unsigned char* X = Z + OPB;
    *reinterpret_cast<uint4*>(Z) = r.z0;
    *reinterpret_cast<uint4*>(Z + 32 * ROW) = r.z1;
    if (xform) { r.x0 = wide_act(r.x0, tsc, tsh); r.x1 = wide_act(r.x1, tsc, tsh); }
    *reinterpret_cast<uint4*>(X) = r.x0;
    *reinterpret_cast<uint4*>(X + 32 * ROW) = r.x1;
  };

  f32x16_t acc[2][2];                                // [co block][ci block]: rows = ci, columns = co
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  // fragment address of (k-step 0, block 0): a group of 16 lanes takes 16 channels (groups 0, 2 the first, 1, 3 the
  // second half of a block) of 8 pixels (groups 0, 1 the first, 2, 3 the second eight); within it lane s points at
  // channels 4*(s%4).. of pixel s/4, the second read is 4 pixels further
  const int frag = (half * 8 + (l16 >> 2)) * ROW + ((lane >> 4) & 1) * 32 + (l16 & 3) * 8;
  const int zoff = frag + wa * 128 + kg * 32 * ROW;   // + i*64 (channel block)
  const int xoff = OPB + frag + wb * 128 + kg * 32 * ROW;
  auto contract = [&](int bufo) __attribute__((always_inline)) {
    const unsigned char* B = smem + bufo;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      bf16x8_t zf[2], xf[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) zf[i] = wide_frag_tr(B + zoff + i * 64 + k * 16 * ROW);
#pragma unroll
      for (int j = 0; j < 2; ++j) xf[j] = wide_frag_tr(B + xoff + j * 64 + k * 16 * ROW);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf[j], zf[i], acc[i][j], 0, 0, 0);
    }
  };

  // (the host gives every slice at least one step; the step requested last is stored and never multiplied)
  WgwSet ra;
  issue(ra);
  stash(ra, 0);
  __syncthreads();
  for (int s = s0; s < s1; ++s) {
    const int bufo = (s - s0) & 1 ? BUF : 0;
    issue(ra);
    __builtin_amdgcn_sched_barrier(0);
    contract(bufo);
    __builtin_amdgcn_sched_barrier(0);
    stash(ra, BUF - bufo);
    __syncthreads();
  }

  // The two pixel halves meet through LDS (the staging buffers are free after the loop's last barrier): a wave
  // keeps one of its two co blocks, hands over the other and adds what its partner hands over, so
  // that all eight waves store. [wave][ci block, quarter][lane] of 16 bytes, 64 KB.
  auto quarter = [&](const f32x16_t& v, int q) __attribute__((always_inline)) {
    return f32x4_t{v[q * 4], v[q * 4 + 1], v[q * 4 + 2], v[q * 4 + 3]};
  };
  f32x4_t* ex = reinterpret_cast<f32x4_t*>(smem) + wave * 512 + lane;
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) ex[(j * 4 + q) * 64] = kg ? quarter(acc[0][j], q) : quarter(acc[1][j], q);
  __syncthreads();
  const f32x4_t* got = reinterpret_cast<const f32x4_t*>(smem) + (wave ^ 4) * 512 + lane;
  // register q*4 + e of a lane holds co = l32 of the block, ci = q*8 + half*4 + e of the block
  const int J = taps * a.Cin;
  float* dst = a.partial + ((size_t)split * a.Cout + co0 + wa * 64 + kg * 32 + l32) * J + (size_t)tap * a.Cin + ci0 + wb * 64 + half * 4;
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<f32x4_t*>(dst + j * 32 + q * 8) = (kg ? quarter(acc[1][j], q) : quarter(acc[0][j], q)) + got[(j * 4 + q) * 64];
}

bool wgrad_wide_ok(int Cin, int Cout, int R, int stride, int dtype) {
  if (dtype != BF16 || stride != 1 || (R != 1 && R != 3)) return false;
  if (Cin < 128 || (Cin & (Cin - 1)) != 0) return false;   // power of two: the partial tile's column is tap*Cin + ci
  return Cout % 128 == 0;
}

// Layers join a launch, in the order of the backward pass, while their workgroups fit the chip at once; a launch that
// leaves places free (the last one, or a layer that fills it alone) cuts its layers into more slices, of at least two
// steps each.
void wgrad_wide_plan(std::vector<WgradWidePlan>& layers) {
  using namespace wgw;
  auto tiles = [](const WgradWidePlan& l) { return (l.Cout / 128) * (l.Cin / 128) * l.R * l.R; };
  auto nsteps = [](const WgradWidePlan& l) { return (l.M + BP - 1) / BP; };
  for (WgradWidePlan& l : layers) l.splits = (nsteps(l) + SLICE_MAX - 1) / SLICE_MAX;
  for (size_t first = 0; first < layers.size();) {
    long wgs = 0;
    size_t end = first;
    while (end < layers.size() && end - first < (size_t)WGRAD_WIDE_LAYERS &&
           (end == first || wgs + (long)tiles(layers[end]) * layers[end].splits <= PLACES)) {
      wgs += (long)tiles(layers[end]) * layers[end].splits;
      ++end;
    }
    const int more = wgs < PLACES ? (int)(PLACES / wgs) : 1;
    for (size_t i = first; i < end; ++i) {
      WgradWidePlan& l = layers[i];
      const int most = nsteps(l) / 2 > 1 ? nsteps(l) / 2 : 1;
      if (l.splits * more <= most) l.splits *= more;
      else if (l.splits < most) l.splits = most;
      l.launch = i + 1 == end;
    }
    first = end;
  }
}

hipError_t wgrad_wide_launch(const WgradWideLayer* layers, int n, hipStream_t s) {
  if (n < 1 || n > WGRAD_WIDE_LAYERS) return hipErrorInvalidValue;
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&wgrad_wide_kernel),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, wgw::LDS);
  if (attr != hipSuccess) return attr;
  WgwArgs a{};
  size_t wgs = 0;
  for (int i = 0; i < n; ++i) {
    const WgradWideLayer& q = layers[i];
    const size_t M = (size_t)q.N * q.H * q.W;
    if (!wgrad_wide_ok(q.Cin, q.Cout, q.R, 1, BF16) || q.splits < 1) return hipErrorInvalidValue;
    if (M * (q.Cin > q.Cout ? q.Cin : q.Cout) >= ((size_t)1 << 31)) return hipErrorInvalidValue;   // 32-bit byte offsets (the forward launch has the same limit)
    if ((size_t)q.splits > (M + wgw::BP - 1) / wgw::BP) return hipErrorInvalidValue;   // an empty slice
    WgwLayer& d = a.l[i];
    d.x = (const bf16_t*)q.x; d.dz = (const bf16_t*)q.dz; d.scale = q.scale; d.shift = q.shift; d.partial = q.partial;
    d.M = (int)M; d.H = q.H; d.W = q.W; d.Cin = q.Cin; d.Cout = q.Cout; d.R = q.R; d.splits = q.splits; d.wg0 = (int)wgs;
    wgs += (size_t)(q.Cout / 128) * (q.Cin / 128) * q.R * q.R * q.splits;
  }
  if (wgs >= ((size_t)1 << 31)) return hipErrorInvalidValue;
  a.n = n;
  DDG_LAUNCH(wgrad_wide_kernel, dim3((unsigned)wgs), dim3(512), wgw::LDS, s, a);
  return hipGetLastError();
}

}  // namespace ddg
