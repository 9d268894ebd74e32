// Weight gradient of wide bf16 layers (1x1 and 3x3, stride 1; input and output channels
// multiples of 128): the companion of conv_wide_kernel.
//
//   dW[co][tap][ci] = sum over pixels p of dz[p][co] * x[pix(p, tap)][ci]
//
// A GEMM whose contraction index, the pixel, is the slow index of both NHWC operands. A
// workgroup owns a 128 (co) x 128 (ci) tile of one tap and a slice of the pixels; it stages
// 64 pixels of both operands per step exactly as they lie in memory ([pixel][128 channels],
// the 64-byte quarters of a row turned by the pixel modulo 4) and takes MFMA fragments out of LDS with the transposing read of
// gfx950 (ds_read_b64_tr_b16: a lane ends up with 8 consecutive pixels of one channel). A tap
// is a shifted pixel row; where the neighbour lies outside the image both rows are zero, which the
// buffer loads give without an instruction (an offset past the tensor's end).
//
// Several layers share a launch. One layer of 6272 pixels is 16 or 36 tiles: to fill the chip alone it had
// to be cut into 7-16 slices of 6-14 steps, and start-up, the tiles' partial sums (64 KB a workgroup, written
// here and read again by the reduction) and the last wave cost more than the contraction: 45 us for the
// three layers of a bottleneck block, 1.15 GB of partial sums for 23 blocks. With layers collected until
// their tiles fill the 512 places of the chip, slices are as long as SLICE_MAX allows: 27 us a block, 0.2 GB.
//
// The sums. A matrix instruction rounds its accumulator once per 16 pixels, and over a slice of 49 steps that adds up: 1.9e-7
// of the gradient (2-norm, against 64 bits) where slices of 6 steps had 8.6e-8. So an accumulator runs over two steps only
// (one, in slices of up to 8 steps) and is then added to a second one, and what this addition rounds off is what the
// accumulator starts from again: 6.1e-8, whatever the length of the slice. Slices of one or two steps
// add up the halves of their steps apart, four roundings each. Never a larger error than with a layer on its own in 256
// workgroups (88 sets of layers, 1 to 784 steps). Folding costs 3 of the 27 us, and every step instead of every second
// one 2.7 more; every third one would save 0.7 but is 6.9e-8, more than slices of 2 or 3 steps had at 2548 pixels.
//
// Four waves as 2 (co) x 2 (ci), 64 x 64 each = four accumulators of mfma_f32_32x32x16_bf16 (16x16x32 runs at little more
// than half the rate) and their sums, 256 registers; 64 KB of LDS: two workgroups a compute unit, one of which multiplies
// while the other waits for its rows. Eight waves, which halve the pixels of a step between them, have room for one set of
// accumulators only (21.9 us a block, before what follows).
//
// Rows of 288 bytes made a transposing read 4.4 cycles of the LDS port instead of 2.6; turned rows of 256 do not. A load was
// requested one contraction before its use; now, between the matrix instructions of the step before, a whole step. Kernel
// size and activation are constants in the loop, the slice's end is the resource's end. A launch of 512 workgroups (23
// blocks at 14x14, batch 32): 90.1 us; LDS rows 86.8, a step ahead 84.0, constants 81.7, the same bits. What bounds it:
// vector instructions, 62 % of the cycles (112 a step fold, 112 form the activation, 40 find the neighbours of 3x3 layers);
// matrix instructions are 28 %, and the two add up to nearly all of the time.
#include "ddg_conv_wide.h"
#include <algorithm>
#include <cstdlib>
#include <type_traits>

namespace ddg {

struct WgwLayer {
  const bf16_t* x;       // [M][Cin]
  const bf16_t* dz;      // [M][Cout]
  const float* scale;    // optional per-channel transform of x: relu(x*scale+shift)
  const float* shift;
  float* partial;        // [splits][Cout][taps*Cin]
  int M, H, W, Cin, Cout, R, splits, wg0;   // wg0: first workgroup of the layer
};
struct WgwArgs { WgwLayer l[WGRAD_WIDE_LAYERS]; int n, by_xcd; };

namespace wgw {
constexpr int BP = 64;                     // pixels per step
constexpr int ROW = 256;                   // bytes per staged pixel (128 channels)
constexpr int OPB = BP * ROW;              // one operand, one buffer: 16384
constexpr int BUF = 2 * OPB;
constexpr int LDS = 2 * BUF;               // 65536
constexpr int PLACES = 512;                // workgroups that run at the same time: two per compute unit
constexpr int SLICE_MAX = 49;              // steps of a slice, unless its layer alone fills the chip
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

// A thread's share of one step on its way to LDS: rows prow, prow + 16, .. (unit q: row prow + 16*q) of dz and x.
struct WgwSet { uint4 z[4], x[4]; };

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void wgrad_wide_kernel(WgwArgs args) {
  using namespace wgw;
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, l32 = lane & 31, half = lane >> 5;
  const int wa = wave & 1, wb = wave >> 1;           // co half, ci half
  // Workgroups go to the 8 XCDs round-robin in launch order. All tiles of one pixel slice read
  // the same rows of x and dz, so the (layer, slice, tile) triples are numbered in that order and XCD j is
  // given the j-th eighth of that sequence: the rows of a slice then come from memory once into
  // one XCD's L2 (two at a boundary) and every other tile finds them there.
  int V = blockIdx.x;
  if (args.by_xcd) {
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

  // staging map: 16-byte unit tid + q*256 of a 64 x 128 tile = pixel (tid>>4) + 16*q, chunk tid&15
  const int ch = tid & 15, prow = tid >> 4;
  // Resources cover the rows of the slice, those of x shifted by the tap (49 steps, so offsets stay small whatever the tensor's
  // size): rows past the slice cost no instruction, rows outside the image get an offset past the end.
  const unsigned zst = a.Cout * 2, xst = a.Cin * 2;
  const int first = s0 * BP, rows = m_end - first;
  const wide_rsrc_t rz = wide_rsrc(a.dz + (size_t)first * a.Cout, (size_t)rows * zst);
  const wide_rsrc_t rx = wide_rsrc(a.x + ((ptrdiff_t)first + dr * a.W + ds) * a.Cin, (size_t)rows * xst);
  // the neighbour of pixel `rem` of the image, in column w, is inside it where rem - lo < span and w != edge
  const unsigned HW = a.H * a.W, lo = dr < 0 ? a.W : 0, span = HW - (dr != 0 ? a.W : 0);
  const unsigned edge = ds < 0 ? 0u : ds > 0 ? a.W - 1u : ~0u;
  const unsigned drem = 16 % HW, dw = 16 % (unsigned)a.W;        // 16 pixels further
  // per-channel constants of this thread's 8 input channels (the same in every step)
  const bool xform = a.scale != nullptr;
  float tsc[8], tsh[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) { tsc[e] = 0.f; tsh[e] = 0.f; }
  if (xform) {
#pragma unroll
    for (int e = 0; e < 8; ++e) { tsc[e] = a.scale[ci0 + ch * 8 + e]; tsh[e] = a.shift[ci0 + ch * 8 + e]; }
  }
  // fragment address of (k-step 0, block 0): a group of 16 lanes takes 16 channels (groups 0, 2 the first, 1, 3 the
  // second half of a block) of 8 pixels (groups 0, 1 the first, 2, 3 the second eight); within it lane s points at
  // channels 4*(s%4).. of pixel s/4, the second read is 4 pixels further. All pixels of a lane are s/4 modulo 4
  const int frag = (half * 8 + (l16 >> 2)) * ROW + ((lane >> 4) & 1) * 32 + (l16 & 3) * 8, turn = (l16 >> 2) * 64;
  const int zoff = frag + (wa * 128 ^ turn);         // ^ i*64 (channel block)
  const int xoff = OPB + frag + (wb * 128 ^ turn);

  f32x16_t acc[2][2], sum[2][2];                     // [co block][ci block]: rows = ci, columns = co
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) sum[i][j][e] = 0.f;
  const int period = s1 - s0 <= 8 ? 1 : 2;

  // One pass over the slice. HOW 0: acc takes all; 1: acc takes the first half of every step, sum the second; 2: acc takes all
  // and is folded into sum every `period` steps. taps3, act: r3 and xform, as constants where the time goes (a
  // branch per unit would end the block that the scheduler interleaves).
  auto run = [&](auto how, auto taps3, auto act) __attribute__((always_inline)) {
    constexpr int HOW = decltype(how)::value;
    // image pixel and column, and byte offsets of the thread's unit that is requested next
    unsigned rem = (unsigned)(first + prow) % HW, w = rem % (unsigned)a.W;
    unsigned zo = prow * zst + (co0 + ch * 8) * 2, xo = prow * xst + (ci0 + ch * 8) * 2;
    WgwSet r;
    auto issue = [&](int q) __attribute__((always_inline)) {   // the units in turn
      if (taps3) {
        const bool in = (rem - lo < span) & (w != edge);
        r.z[q] = wide_load(rz, in ? zo : NOWHERE, 0);
        r.x[q] = wide_load(rx, in ? xo : NOWHERE, 0);
        const unsigned r1 = rem + drem, w1 = w + dw, r2 = r1 - HW, w2 = w1 - a.W;    // (wrapped around zero unless past the end)
        rem = r1 < r2 ? r1 : r2; w = w1 < w2 ? w1 : w2;
      } else {
        r.z[q] = wide_load(rz, zo, 0);
        r.x[q] = wide_load(rx, xo, 0);
      }
      zo += 16 * zst; xo += 16 * xst;
    };
    // (a row that does not exist is relu(shift) after the transform; its dz row is zero)
    auto stash = [&](int q, int bufo) __attribute__((always_inline)) {
      unsigned char* Z = smem + bufo + q * 16 * ROW + prow * ROW + (ch * 16 ^ (prow & 3) * 64);
      *reinterpret_cast<uint4*>(Z) = r.z[q];
      *reinterpret_cast<uint4*>(Z + OPB) = act ? wide_act(r.x[q], tsc, tsh) : r.x[q];
    };
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    // sum += acc; acc = what that addition rounded off (exactly where |sum| >= |acc|, else to a rounding of acc)
    auto fold = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const float t = acc[i][j][e], m = sum[i][j][e], s = m + t, d = s - m;
            acc[i][j][e] = t - d;
            sum[i][j][e] = s;
          }
    };
    // Step `s` out of the buffer at bufo. Beside the matrix instructions of 16 pixels, a unit of the next step goes from its
    // registers to the other buffer (free since the barrier that ended the step before) and the unit of the step after
    // that is requested into them: a load has a whole step to arrive.
    auto step = [&](int bufo) __attribute__((always_inline)) {
      const unsigned char* B = smem + bufo;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        bf16x8_t zf[2], xf[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) zf[i] = wide_frag_tr(B + (zoff ^ i * 64) + k * 16 * ROW);
#pragma unroll
        for (int j = 0; j < 2; ++j) xf[j] = wide_frag_tr(B + (xoff ^ j * 64) + k * 16 * ROW);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            f32x16_t& c = HOW == 1 && k >= 2 ? sum[i][j] : acc[i][j];
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf[j], zf[i], c, 0, 0, 0);
          }
        stash(k, BUF - bufo);
        issue(k);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    // (the host gives every slice at least one step; the step requested last is stored and never multiplied)
#pragma unroll
    for (int q = 0; q < 4; ++q) issue(q);
#pragma unroll
    for (int q = 0; q < 4; ++q) { stash(q, 0); issue(q); }
    __syncthreads();
    for (int s = s0; s < s1; ++s) {
      step((s - s0) & 1 ? BUF : 0);
      if (HOW == 2 && ((s - s0) & (period - 1)) == period - 1) fold();
      __syncthreads();
    }
  };
  using std::integral_constant;
  using std::bool_constant;
  if (s1 - s0 <= 2) run(integral_constant<int, 1>{}, r3, xform);
  else if (r3 && xform) run(integral_constant<int, 2>{}, bool_constant<true>{}, bool_constant<true>{});
  else if (r3) run(integral_constant<int, 2>{}, bool_constant<true>{}, bool_constant<false>{});
  else if (xform) run(integral_constant<int, 2>{}, bool_constant<false>{}, bool_constant<true>{});
  else run(integral_constant<int, 2>{}, bool_constant<false>{}, bool_constant<false>{});
  // Folding an infinity leaves no number in acc. If any element of the tile ends as none, the slice is added up plainly,
  // which supplies those elements: infinities come out as infinities.
  int bad = 0;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        sum[i][j][e] += acc[i][j][e];
        bad |= sum[i][j][e] == sum[i][j][e] ? 0 : 1;
      }
  if (s1 - s0 > 2 && __syncthreads_or(bad)) {
    run(integral_constant<int, 0>{}, r3, xform);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) sum[i][j][e] = sum[i][j][e] == sum[i][j][e] ? sum[i][j][e] : acc[i][j][e];
  }

  // register q*4 + e of a lane holds co = l32 of the block, ci = q*8 + half*4 + e of the block
  const int J = taps * a.Cin;
  float* dst = a.partial + ((size_t)split * a.Cout + co0 + wa * 64 + l32) * J + (size_t)tap * a.Cin + ci0 + wb * 64 + half * 4;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<f32x4_t*>(dst + (size_t)(i * 32) * J + j * 32 + q * 8) =
            f32x4_t{sum[i][j][q * 4], sum[i][j][q * 4 + 1], sum[i][j][q * 4 + 2], sum[i][j][q * 4 + 3]};
}

bool wgrad_wide_ok(int Cin, int Cout, int R, int stride, int dtype) {
  if (dtype != BF16 || stride != 1 || (R != 1 && R != 3)) return false;
  if (Cin < 128 || (Cin & (Cin - 1)) != 0) return false;   // power of two: the partial tile's column is tap*Cin + ci
  return Cout % 128 == 0;
}

// Layers join a launch, in the order of the backward pass, while their workgroups fit the chip at once; a launch that
// leaves places free (the last one, or a layer that fills it alone) cuts its layers into more slices, of at least two
// steps each, and no more than fill 256 places by themselves: the reduction rounds too, and the partial sums of all 512 are
// what it would show (512 -> 128 channels, 380 steps in 126 slices 1.2e-7, in 64 1.0e-7).
void wgrad_wide_plan(std::vector<WgradWidePlan>& layers) {
  using namespace wgw;
  int places = PLACES;
  if (const char* e = getenv("DDG_TUNE_WGRAD_WIDE_WGS")) {   // timing experiments, within [64, 2048]
    const int v = atoi(e);
    if (v >= 64 && v <= 2048) places = v;
  }
  auto tiles = [](const WgradWidePlan& l) { return (l.Cout / 128) * (l.Cin / 128) * l.R * l.R; };
  auto nsteps = [](const WgradWidePlan& l) { return (l.M + BP - 1) / BP; };
  for (WgradWidePlan& l : layers) l.splits = (nsteps(l) + SLICE_MAX - 1) / SLICE_MAX;
  for (size_t first = 0; first < layers.size();) {
    long wgs = 0;
    size_t end = first;
    while (end < layers.size() && end - first < (size_t)WGRAD_WIDE_LAYERS &&
           (end == first || wgs + (long)tiles(layers[end]) * layers[end].splits <= places)) {
      wgs += (long)tiles(layers[end]) * layers[end].splits;
      ++end;
    }
    const int more = wgs < places ? (int)(places / wgs) : 1;
    for (size_t i = first; i < end; ++i) {
      WgradWidePlan& l = layers[i];
      const int most = std::max(std::min(places / 2 / tiles(l), nsteps(l) / 2), 1);
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
  a.by_xcd = getenv("DDG_NO_WGRAD_XCD") ? 0 : 1;
  DDG_LAUNCH(wgrad_wide_kernel, dim3((unsigned)wgs), dim3(256), wgw::LDS, s, a);
  return hipGetLastError();
}

}  // namespace ddg
