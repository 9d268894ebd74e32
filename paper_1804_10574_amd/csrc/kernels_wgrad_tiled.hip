// Weight gradient of a 3x3, stride-1, pad-1 convolution on the bf16 matrix cores,
// for the CIFAR-shaped layers (16/32/64 channels, feature maps 32/16/8 wide).
//
//   dW[co][tap][ci] = sum over pixels m of dz[m][co] * a[pix(m,tap)][ci]
//
// The contraction index is the pixel, which is the slow index of both NHWC operands, while an
// MFMA lane wants 8 consecutive contraction values of one channel. gfx950 can transpose on the
// way out of LDS (ds_read_b64_tr_b16: in every block of 16 lanes, lane s supplies the address
// of 4 consecutive 16-bit values, and lane i receives value i%4 of lanes i/4, i/4+4, i/4+8,
// i/4+12). So both operands are staged exactly as they lie in memory, [pixel][channel] with
// 16-byte writes; lane s of a block points at channels 4*(s%4).. of pixel P + s/4, lane i gets
// channel i of pixels P..P+3, and two such reads make one 8-pixel fragment. A tap is a shifted
// pixel address into the halo tile: the im2col matrix never exists and nothing is shifted in
// registers. The pixel stride in LDS is 32 or 96 bytes modulo 128, which spreads the four
// pixels of a 16-lane block over all banks.
//
// The activation a can be produced on the fly from the saved conv output:
// a = relu(z*scale + shift) is applied while staging (scale == nullptr: use x as stored).
//
// The error gradient dz can likewise be formed while staging: with dy given, the kernel applies
// the ReLU mask and the batch-norm backward formula dz = A*g + B*z + C0 (coefficients final, or
// derived from the partial rows of the BN-backward sums), uses dz for the contraction and
// writes it out once for the input-gradient kernel that follows: no separate apply pass.
//
// A workgroup walks over tiles of 8 image rows, keeps its accumulators in registers across
// tiles (the next tile's global loads are in flight meanwhile), and writes one partial tile at
// the end; wgrad_reduce_all_kernel adds the partials in a fixed order (deterministic).
#include "ddg_wgrad_tiled.h"
#include <cstdlib>

namespace ddg {

template <int CIN, int COUT, int W, int S = 1, int R = 3>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu((CIN == 32 || S == 2) ? 2 : 3))) void wgrad_tiled_kernel(WgradTiledArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  wgrad_tiled_body<CIN, COUT, W, true, S, R>(a, smem, blockIdx.x, blockIdx.y, gridDim.x);
}

// The three weight gradients of a stage's first block, which do not depend on each other: the stride-2 3x3 layer, the
// projection, and the second layer, whose dz is in memory. One launch instead of three of 5-8 us, each of which
// left most of the chip idle (ResNet-20 bf16, 37 images, with the two input gradients in one launch: 380 -> 329 us an iteration).
template <int CIN, int W>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void wgrad_down_kernel(WgradTiledArgs a3, WgradTiledArgs a1, WgradTiledArgs a2,
                                                                                               int g3, int g1, int rows2) {
  extern __shared__ __align__(16) unsigned char smem[];
  static_assert(WgradTiledCfg<CIN, 2 * CIN, W, 2, 3>::OT == 1 && WgradTiledCfg<CIN, 2 * CIN, W, 2, 1>::OT == 1, "one slice of the input channels");
  const int b = blockIdx.x;
  if (b < g3) wgrad_tiled_body<CIN, 2 * CIN, W, true, 2, 3>(a3, smem, b, 0, g3);
  else if (b < g3 + g1) wgrad_tiled_body<CIN, 2 * CIN, W, true, 2, 1>(a1, smem, b - g3, 0, g1);
  else wgrad_tiled_body<2 * CIN, 2 * CIN, W, false>(a2, smem, (b - g3 - g1) % rows2, (b - g3 - g1) / rows2, rows2);
}

template <int CIN, int W>
static hipError_t wgrad_down_run(const WgradTiledArgs& a3, const WgradTiledArgs& a1, const WgradTiledArgs& a2, int g3, int g1, int rows2, hipStream_t s) {
  using C2 = WgradTiledCfg<2 * CIN, 2 * CIN, W>;
  constexpr int l3 = WgradTiledCfg<CIN, 2 * CIN, W, 2, 3>::LDS, l1 = WgradTiledCfg<CIN, 2 * CIN, W, 2, 1>::LDS;
  constexpr int lds = l3 > l1 ? (l3 > C2::LDS ? l3 : C2::LDS) : (l1 > C2::LDS ? l1 : C2::LDS);
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&wgrad_down_kernel<CIN, W>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (attr != hipSuccess) return attr;
  DDG_LAUNCH((wgrad_down_kernel<CIN, W>), dim3(g3 + g1 + rows2 * C2::OT), dim3(256), lds, s, a3, a1, a2, g3, g1, rows2);
  return hipGetLastError();
}

template <int CIN, int COUT, int W, int S = 1, int R = 3>
static hipError_t wgrad_tiled_launch_t(const WgradTiledArgs& a, int grid_x, hipStream_t s) {
  using Cfg = WgradTiledCfg<CIN, COUT, W, S, R>;
  const size_t lds = (size_t)Cfg::LDS;
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&wgrad_tiled_kernel<CIN, COUT, W, S, R>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  DDG_LAUNCH((wgrad_tiled_kernel<CIN, COUT, W, S, R>), dim3(grid_x, Cfg::OT), dim3(256), lds, s, a);
  return hipGetLastError();
}

// The layers between two stages: 3x3 stride 2 and the 1x1 stride-2 projection, Cout = 2*Cin,
// from 32x32 (16 channels) or 16x16 (32 channels) inputs.
static bool wgrad_tiled_stride2(int H, int W, int Cin, int Cout, int R, int stride) {
  return stride == 2 && (R == 3 || R == 1) && Cout == 2 * Cin && ((Cin == 16 && W == 32) || (Cin == 32 && W == 16)) &&
         H % 16 == 0;
}

// Returns the number of partial rows (grid.x) the tiled kernel will use for this shape, or 0
// if the shape is not covered (then the generic kernel is used).
int wgrad_tiled_rows(int N, int H, int W, int Cin, int Cout, int R, int stride, int dtype) {
  if (dtype == F32) return wgrad_tiled_f32_rows(N, H, W, Cin, Cout, R, stride);
  if (dtype == BF16 && wgrad_tiled_stride2(H, W, Cin, Cout, R, stride)) {
    const int tiles = N * (H / 2 / 8);
    const int want = 64;
    return want < tiles ? want : tiles;
  }
  if (dtype != BF16 || R != 3 || stride != 1 || Cin != Cout) return 0;
  if (!((Cin == 16 && W == 32) || (Cin == 32 && W == 16) || (Cin == 64 && W == 8))) return 0;
  if (H % 8 != 0) return 0;
  const int tiles = N * (H / 8);
  int want = (Cin == 16) ? 128 : (Cin == 32 ? 64 : 16);
  if (const char* e = getenv("DDG_TUNE_WGRAD_ROWS")) {   // override within [8, 1024]
    const int v = atoi(e);
    if (v >= 8 && v <= 1024) want = v;
  }
  const char* name = Cin == 16 ? "DDG_TUNE_WGRAD_ROWS_C16" : (Cin == 32 ? "DDG_TUNE_WGRAD_ROWS_C32" : "DDG_TUNE_WGRAD_ROWS_C64");
  if (const char* e = getenv(name)) {                    // per-shape override within [8, 256]
    const int v = atoi(e);
    if (v >= 8 && v <= 256) want = v;
  }
  if (want > tiles) want = tiles;
  return want;
}

hipError_t wgrad_tiled_launch(const void* x, const float* scale, const float* shift, const void* dz,
                              const WgradFuse* fuse, float* partial, int N, int H, int W, int C, int rows,
                              hipStream_t s, int Cout, int R, int stride) {
  if (Cout == 0) Cout = C;
  WgradTiledArgs a{};
  a.x = (const bf16_t*)x; a.scale = scale; a.shift = shift; a.dz = (const bf16_t*)dz; a.partial = partial;
  if (fuse) {
    a.dy = (const bf16_t*)fuse->dy; a.mask = (const bf16_t*)fuse->mask; a.mscale = fuse->mscale; a.mshift = fuse->mshift;
    a.zc = (const bf16_t*)fuse->z; a.coef = fuse->coef; a.dz_out = (bf16_t*)fuse->dz_out;
    if (fuse->rows) a.rows = *fuse->rows;
  }
  if (wgrad_tiled_stride2(H, W, C, Cout, R, stride)) {
    a.N = N; a.H = H / 2; a.W = W / 2; a.tiles = N * (a.H / 8);     // output geometry
    if (rows < 1 || rows > a.tiles) return hipErrorInvalidValue;
    if (C == 16 && R == 3) return wgrad_tiled_launch_t<16, 32, 16, 2, 3>(a, rows, s);
    if (C == 16 && R == 1) return wgrad_tiled_launch_t<16, 32, 16, 2, 1>(a, rows, s);
    if (C == 32 && R == 3) return wgrad_tiled_launch_t<32, 64, 8, 2, 3>(a, rows, s);
    if (C == 32 && R == 1) return wgrad_tiled_launch_t<32, 64, 8, 2, 1>(a, rows, s);
    return hipErrorInvalidValue;
  }
  if (Cout != C || R != 3 || stride != 1) return hipErrorInvalidValue;
  a.N = N; a.H = H; a.W = W; a.tiles = N * (H / 8);
  if (C == 16 && W == 32) return wgrad_tiled_launch_t<16, 16, 32>(a, rows, s);
  if (C == 32 && W == 16) return wgrad_tiled_launch_t<32, 32, 16>(a, rows, s);
  if (C == 64 && W == 8) return wgrad_tiled_launch_t<64, 64, 8>(a, rows, s);
  return hipErrorInvalidValue;
}

hipError_t wgrad_down_launch(const void* x, int N, int H, int W, int C, const WgradFuse& f3, float* partial3, int rows3,
                             const WgradFuse& f1, float* partial1, int rows1, const WgradPair& second, hipStream_t s) {
  if (!wgrad_tiled_stride2(H, W, C, 2 * C, 3, 2) || !f3.rows || !f1.rows) return hipErrorInvalidValue;
  const int tiles = N * (H / 2 / 8);
  if (rows3 < 1 || rows3 > tiles || rows1 < 1 || rows1 > tiles || second.rows < 1 || second.rows > tiles) return hipErrorInvalidValue;
  auto args = [&](const WgradFuse& f, float* partial) {
    WgradTiledArgs a{};
    a.x = (const bf16_t*)x; a.partial = partial;
    a.dy = (const bf16_t*)f.dy; a.mask = (const bf16_t*)f.mask; a.mscale = f.mscale; a.mshift = f.mshift;
    a.zc = (const bf16_t*)f.z; a.rows = *f.rows; a.dz_out = (bf16_t*)f.dz_out;
    a.N = N; a.H = H / 2; a.W = W / 2; a.tiles = tiles;
    return a;
  };
  const WgradTiledArgs a3 = args(f3, partial3), a1 = args(f1, partial1);
  WgradTiledArgs a2{};
  a2.x = (const bf16_t*)second.x; a2.scale = second.scale; a2.shift = second.shift; a2.dz = (const bf16_t*)second.dz;
  a2.partial = second.partial; a2.N = N; a2.H = H / 2; a2.W = W / 2; a2.tiles = tiles;
  return C == 16 ? wgrad_down_run<16, 16>(a3, a1, a2, rows3, rows1, second.rows, s)
                 : wgrad_down_run<32, 8>(a3, a1, a2, rows3, rows1, second.rows, s);
}

}  // namespace ddg
