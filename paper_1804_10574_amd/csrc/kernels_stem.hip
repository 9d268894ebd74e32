// First layer of a network: 3x3, stride 1, 1 to 4 input channels in bf16 and 1 to 3 in fp32 (four are a whole fragment of the generic kernel
// there), rows up to 223 or 127 wide by the tile (stem_conv_ok); weight gradient: 3 channels (four have the kernel with vector gathers, fewer other columns), and as many
// pixels a workgroup as 48 KB of LDS hold: 1.5 M in all at 16 output channels, 0.38 M at 64 (32 wide). Others run in the generic kernels.
//
// With so few channels a fragment of the implicit GEMM is one tap of one pixel, 6 or 12 bytes at an address of its own, and the generic kernels
// spent their time on vector instructions: pixel indexes, bounds and element gathers for every tap of every pixel (61 and 111 a matrix
// instruction and step). Here a workgroup stages the pixels it needs once, 16 bytes each, in LDS: output pixels are consecutive, so tap
// (r, s) of pixel m is flat pixel m + (r-1)*W + (s-1), whatever the image's size; taps outside the image read a pixel of zeros. Tiles, order of sums
// and statistics rows are those of the generic kernels: results are the same bit for bit.
#include "ddg_device.h"
#include "ddg_kernels.h"

namespace ddg {

namespace stem {
constexpr int NPX = 2;                      // pixels a thread stages
constexpr int SLOTS = NPX * 256 + 1;        // and a pixel of zeros, first
constexpr size_t WG_LDS_MAX = 48 * 1024;   // (what a launch may ask for without an attribute)

// Row and column of a pixel in its image: exact by fp32 for indexes below 2^22 (an integer division costs as much as a step).
struct Place {
  int hw, W; bool fdiv; float inv_hw, inv_w;
  __device__ __forceinline__ Place(int H, int W_, int M) : hw(H * W_), W(W_), fdiv(M < (1 << 22)), inv_hw(1.0f / (float)(H * W_)), inv_w(1.0f / (float)W_) {}
  __device__ __forceinline__ void of(int m, int& h, int& w) const {
    const int n = fdiv ? (int)(((float)m + 0.5f) * inv_hw) : m / hw;
    const int rem = m - n * hw;
    h = fdiv ? (int)(((float)rem + 0.5f) * inv_w) : rem / W;
    w = rem - h * W;
  }
};

// NE channels of a pixel (those past C: any)
template <typename T, int NE>
__device__ __forceinline__ void load_pixel(const T* __restrict__ in, int m, int M, int C, T (&e)[NE]) {
  const T* p = in + (size_t)(m < 0 ? 0 : m < M ? m : M - 1) * C;
#pragma unroll
  for (int j = 0; j < NE; ++j) e[j] = p[j < C ? j : C - 1];
}
}

// Forward: a wave owns MB pixel blocks x NB channel blocks; k-step ks of a lane is tap ks*4 + lane/16.
template <typename T, int MB, int NB>
__global__ __launch_bounds__(256) void stem_conv_kernel(ConvArgs a) {
  using M_ = Mma<T>;
  using S_ = Store<T>;
  typedef typename M_::frag_t frag_t;
  constexpr int KV = M_::KV, NE = 4, P = 64 * MB;
  __shared__ __align__(16) unsigned char px[stem::SLOTS * 16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, lg = lane >> 4;
  const int cb0 = blockIdx.y * NB, OCB = a.OC >> 4, W = a.IW;
  const bool second = blockIdx.z != 0;
  const T* __restrict__ in = reinterpret_cast<const T*>(second ? a.in_b : a.in);
  const T* __restrict__ wp = reinterpret_cast<const T*>(a.wpack);
  T* __restrict__ out = reinterpret_cast<T*>(second ? a.out_b : a.out);
  float* __restrict__ stat_partial = second ? a.stat_partial_b : a.stat_partial;
  const int tiles = (a.M + 16 * MB - 1) / (16 * MB), need = P + 2 * W + 2;
  const stem::Place place(a.OH, a.OW, a.M);

  // what the next trip stages, on its way
  T e[stem::NPX][NE];
  auto request = [&](int m0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < stem::NPX; ++u) stem::load_pixel<T, NE>(in, m0 - W - 1 + tid + u * 256, a.M, a.IC, e[u]);
  };
  int tile0 = blockIdx.x * 4;
  if (tile0 < tiles) request(tile0 * MB * 16);
  frag_t wf[3][NB];
#pragma unroll
  for (int ks = 0; ks < 3; ++ks)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) wf[ks][nb] = M_::load(wp + ((size_t)(ks * OCB + cb0 + nb) * 64 + lane) * KV);
  // this lane's taps: byte offset from the centre pixel, and where they stand (tap 9 and beyond: zero weights)
  int koff[3], kr[3], kc[3];
#pragma unroll
  for (int ks = 0; ks < 3; ++ks) {
    const int tap = ks * 4 + lg;
    kr[ks] = tap < 9 ? tap / 3 - 1 : 1 << 20; kc[ks] = tap < 9 ? tap % 3 - 1 : 0;
    koff[ks] = tap < 9 ? (kr[ks] * W + kc[ks]) * 16 : 0;
  }
  if (tid == 0) *reinterpret_cast<uint4*>(px) = make_uint4(0, 0, 0, 0);
  float ssum[NB][4], ssq[NB][4];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int j = 0; j < 4; ++j) { ssum[nb][j] = 0.f; ssq[nb][j] = 0.f; }

  for (; tile0 < tiles; tile0 += gridDim.x * 4) {
    const int m0 = tile0 * MB * 16;
    __syncthreads();                       // the pixels of the trip before have been read
#pragma unroll
    for (int u = 0; u < stem::NPX; ++u) {
      const int s = tid + u * 256;
      uint32_t f[NE];                      // the elements' bits
#pragma unroll
      for (int j = 0; j < NE; ++j) {
        if constexpr (KV == 4) f[j] = __float_as_uint(e[u][j]);
        else f[j] = e[u][j].v;
        if (j >= a.IC) f[j] = 0u;
      }
      const uint4 q = KV == 4 ? make_uint4(f[0], f[1], f[2], f[3]) : make_uint4(f[0] | f[1] << 16, f[2] | f[3] << 16, 0u, 0u);
      if (s < need) *reinterpret_cast<uint4*>(px + (s + 1) * 16) = q;
    }
    __syncthreads();
    request((tile0 + gridDim.x * 4) * MB * 16);
    frag_t x[MB][3];
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const int b = (wave * MB + i) * 16 + l16;
      int h, w;
      place.of(m0 + b < a.M ? m0 + b : 0, h, w);
#pragma unroll
      for (int ks = 0; ks < 3; ++ks) {
        const bool ok = (unsigned)(h + kr[ks]) < (unsigned)a.IH && (unsigned)(w + kc[ks]) < (unsigned)W;
        x[i][ks] = *reinterpret_cast<const frag_t*>(px + (ok ? (b + W + 2) * 16 + koff[ks] : 0));
      }
    }
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const int m = m0 + (wave * MB + i) * 16 + l16;
      f32x4_t acc[NB];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        acc[nb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 3; ++ks) acc[nb] = M_::mma(wf[ks][nb], x[i][ks], acc[nb]);
      }
      if (m >= a.M) continue;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        float v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          v[j] = S_::round(acc[nb][j]);
          ssum[nb][j] += v[j];
          ssq[nb][j] += v[j] * v[j];
        }
        S_::store4(out + (size_t)m * a.OC + (cb0 + nb) * 16 + lg * 4, v[0], v[1], v[2], v[3]);
      }
    }
  }
  if (stat_partial) {
    __shared__ float red[4][2][NB * 16];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float s1 = row_sum16(ssum[nb][j]), s2 = row_sum16(ssq[nb][j]);
        if (l16 == 0) { red[wave][0][nb * 16 + lg * 4 + j] = s1; red[wave][1][nb * 16 + lg * 4 + j] = s2; }
      }
    __syncthreads();
    if (tid < 2 * NB * 16) {
      const int which = tid / (NB * 16), c = tid % (NB * 16);
      stat_partial[((size_t)blockIdx.x * 2 + which) * a.OC + cb0 * 16 + c] = ((red[0][which][c] + red[1][which][c]) + red[2][which][c]) + red[3][which][c];
    }
  }
}

bool stem_conv_ok(const ConvArgs& a) {
  return !a.dgrad && a.R == 3 && a.stride == 1 && a.pad == 1 && a.IC <= 4 && a.IC % mma_kv(a.dtype) != 0 && a.ksteps == 3 && !a.add_g &&
         64 * a.mb + 2 * a.IW + 2 <= stem::NPX * 256;
}
hipError_t stem_conv_launch(const ConvArgs& a, hipStream_t s) {
  if (!stem_conv_ok(a)) return hipErrorInvalidValue;
  const dim3 grid(a.grid_x, (a.OC / 16) / a.nb, a.in_b ? 2 : 1), block(256);
#define DDG_STEM_CASE(T_, MB_, NB_)                                               \
  if (a.mb == MB_ && a.nb == NB_) {                                               \
    DDG_LAUNCH((stem_conv_kernel<T_, MB_, NB_>), grid, block, 0, s, a);           \
    return hipGetLastError();                                                     \
  }
  if (a.dtype == BF16) {
    DDG_STEM_CASE(bf16_t, 4, 1) DDG_STEM_CASE(bf16_t, 2, 1) DDG_STEM_CASE(bf16_t, 2, 2) DDG_STEM_CASE(bf16_t, 2, 4)
  } else {
    DDG_STEM_CASE(float, 4, 1) DDG_STEM_CASE(float, 2, 1) DDG_STEM_CASE(float, 1, 1)
  }
#undef DDG_STEM_CASE
  return hipErrorInvalidValue;
}

// Weight gradient (the contraction of wgrad_mfma_kernel: k = 4 pixels an instruction, columns = tap * 4 + channel): the workgroup's
// 16 * steps pixels and their neighbours are staged once, so a step's operand is an LDS read per column block. dz is requested three steps ahead.
template <typename T>
__global__ __launch_bounds__(256) void stem_wgrad_kernel(WgradArgs a) {
  using S_ = Store<T>;
  constexpr int NJ = 3;
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, lg = lane >> 4;
  const int cob = blockIdx.y, W = a.W;
  const T* __restrict__ x = reinterpret_cast<const T*>(a.x);
  const T* __restrict__ dz = reinterpret_cast<const T*>(a.dz);
  const long first = (long)blockIdx.x * 16 * a.steps;
  const int need = 16 * a.steps + 2 * W + 2;

  const long m0 = first + (long)wave * a.steps * 4;
  auto issue = [&](float& r, int st) __attribute__((always_inline)) {
    const long m = m0 + (long)st * 4 + lg;
    r = S_::load1(dz + (size_t)(st < a.steps && m < a.M ? m : 0) * a.Cout + cob * 16 + l16);
  };
  float dv[4];
#pragma unroll
  for (int u = 0; u < 3; ++u) issue(dv[u], u);

  for (int s0 = tid; s0 < need; s0 += 4 * 256) {
    T e[4][4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const long m = first - W - 1 + s0 + u * 256;
      stem::load_pixel<T, 4>(x, m < a.M ? (int)m : a.M - 1, a.M, a.Cin, e[u]);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int s = s0 + u * 256;
      if (s < need)
        *reinterpret_cast<float4*>(smem + (s + 1) * 16) = make_float4(S_::load1(&e[u][0]), S_::load1(&e[u][1]), S_::load1(&e[u][2]), S_::load1(&e[u][3]));
    }
  }
  if (tid == 0) *reinterpret_cast<uint4*>(smem) = make_uint4(0, 0, 0, 0);

  int jr[NJ], js[NJ], joff[NJ];          // this lane's columns: tap row and column, byte offset from the centre pixel
#pragma unroll
  for (int b = 0; b < NJ; ++b) {
    const int j = b * 16 + l16, tap = j >> 2, c = j & 3;
    const bool on = tap < 9 && c < a.Cin;
    jr[b] = on ? tap / 3 - 1 : 1 << 20; js[b] = on ? tap % 3 - 1 : 0;
    joff[b] = on ? (jr[b] * W + js[b]) * 16 + c * 4 : 0;
  }
  f32x4_t acc[NJ];
#pragma unroll
  for (int b = 0; b < NJ; ++b) acc[b] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const stem::Place place(a.P, a.Q, a.M);
  __syncthreads();
  for (int st = 0; st < a.steps; st += 4) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      issue(dv[(u + 3) & 3], st + u + 3);
      const long m = m0 + (long)(st + u) * 4 + lg;
      const bool mv = st + u < a.steps && m < a.M;
      int h, w;
      place.of(mv ? (int)m : 0, h, w);
      const int centre = (int)(m - first + W + 2) * 16;
      float xv[NJ];
#pragma unroll
      for (int b = 0; b < NJ; ++b) {
        const bool ok = mv && (unsigned)(h + jr[b]) < (unsigned)a.H && (unsigned)(w + js[b]) < (unsigned)W;
        xv[b] = *reinterpret_cast<const float*>(smem + (ok ? centre + joff[b] : 0));
      }
      asm volatile("" : "+v"(dv[u]));      // (keeps the load where it is)
      const float d = mv ? dv[u] : 0.f;
#pragma unroll
      for (int b = 0; b < NJ; ++b) acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(d, xv[b], acc[b], 0, 0, 0);
    }
  }
  __syncthreads();                          // the pixels have been read
  float (*red)[NJ][16][17] = reinterpret_cast<float (*)[NJ][16][17]>(smem);
#pragma unroll
  for (int b = 0; b < NJ; ++b)
#pragma unroll
    for (int i = 0; i < 4; ++i) red[wave][b][lg * 4 + i][l16] = acc[b][i];
  __syncthreads();
  const int Jp = a.JB * 16;
  for (int e = tid; e < NJ * 256; e += 256) {
    const int b = e >> 8, row = (e >> 4) & 15, col = e & 15;
    a.partial[((size_t)blockIdx.x * a.Cout + cob * 16 + row) * Jp + b * 16 + col] = ((red[0][b][row][col] + red[1][b][row][col]) + red[2][b][row][col]) + red[3][b][row][col];
  }
}

static size_t stem_wgrad_lds(const WgradArgs& a) {
  const size_t px = ((size_t)16 * a.steps + 2 * a.W + 3) * 16, red = (size_t)4 * 3 * 16 * 17 * 4;
  return px > red ? px : red;
}
bool stem_wgrad_ok(const WgradArgs& a) {
  return !a.vec && a.R == 3 && a.stride == 1 && a.pad == 1 && a.Cin <= 4 && a.log2cp == 2 && a.JB == 3 && a.jgroups == 1 && stem_wgrad_lds(a) <= stem::WG_LDS_MAX;
}
hipError_t stem_wgrad_launch(const WgradArgs& a, hipStream_t s) {
  if (!stem_wgrad_ok(a)) return hipErrorInvalidValue;
  const dim3 grid(a.msplit, a.Cout / 16), block(256);
  if (a.dtype == BF16) DDG_LAUNCH(stem_wgrad_kernel<bf16_t>, grid, block, stem_wgrad_lds(a), s, a);
  else DDG_LAUNCH(stem_wgrad_kernel<float>, grid, block, stem_wgrad_lds(a), s, a);
  return hipGetLastError();
}

}  // namespace ddg
