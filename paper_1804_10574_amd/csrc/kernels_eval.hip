// Evaluation forward of the CIFAR-shaped networks. With running estimates a batch norm is a fixed
// affine map, so nothing has to be known about the whole minibatch between two layers, and one
// workgroup can take an image (or a strip of its rows) through many layers without leaving its
// compute unit: activations stay in LDS, weights come from L2 in fragment order, and memory sees
// the network's input and output only.
//
// What bounds it: a layer of one image is 4.7 MFLOP on one compute unit, about 1 us of matrix and
// LDS time in bf16, against 10-13 us for the per-layer launch of a whole minibatch of 256 and 6-7
// us for the smallest one (the launch, its weights and its halo loads are then all there is).
// Measured, whole call: ResNet-110, batch 256, bf16 1394 -> 214 us (1.4-1.7 us per layer); the 32-channel group of
// ResNet-56, batch 100, bf16 134 -> 29 us; ResNet-20, one image, fp32 227 -> 100 us.
//
// Two ways of cutting the work, chosen by eval_plan() below:
//   whole images: all blocks of a module in one launch, one image per workgroup (bf16);
//   strips: one residual block per launch, TH output rows per workgroup, the rows of the halo
//           recomputed (fp32, whose matrix rate makes an image 10-18 us per layer on one unit, so
//           that one image has to be spread over several; bf16 modules whose buffers, each at its largest over the blocks,
//           exceed LDS: large images, and deep networks in one module from 32x32 on (ResNet-110: its table of scales and shifts
//           alone is 32 KB); and bf16 where a few large images would leave most compute units idle). Strips are no slower than
//           the per-layer kernels either: the blocks of ResNet-110 in one module, batch 37, 501 -> 339 us, batch 1 459 -> 323. As whole images
//           those of ResNet-20 take 42 us at batch 256 and 38 at batch 1, 95 and 55 in strips (calls one after the other).
//
// Buffers: three LDS regions of NHWC pixels with a zero border (row and column -1 and H / W). An identity block reads x, writes
// o = relu(bn1(conv1 x)), then adds relu(bn2(conv2 o) + x)
// back into x in place (an output pixel needs x at that pixel only). A block between stages writes
// its output to the third region, and the regions change roles.
//
// Pitch: bf16 pixels of 32 and 64 channels have GAP bytes between them, and there is a kernel for either GAP. 32: pixels are an
// odd multiple of 32 bytes apart and rows continue that where a block of 16 pixels spans two, so that
// fragment reads have no bank conflicts (4 cycles each; 8-12 with pixels an odd multiple of 16 bytes apart). 16: more fits,
// larger images as a whole (three identity blocks of 32 channels to 29x29 instead of 26x26, of 64 to 18x18 instead of 17x17) and higher strips with
// fewer halo rows. fp32, where the matrix instructions hide the reads: 16, whose conflicts cost less than those of the stores with 32, 1-3 %.
//
// Eight waves; a wave holds the weight fragments of one layer in registers (two sets: the next
// layer's are requested before the current one is contracted) and walks over 16-pixel blocks:
//   16 channels: every wave all channels, 8 pixel groups;  32 channels: one channel block and 4 pixel groups (with both
//   blocks in every wave a layer's weights enter the compute unit eight times, 147 KB at 64 bytes a cycle), but with GAP 16, which
//   larger maps take, both and 8 groups: half the reads of LDS per matrix instruction (24x24, 3 blocks, 256 images:
//   31 us instead of 39 with one block each and of 36 with GAP 32);
//   64 channels: 4 channel blocks x 2 halves of the contraction (a layer's weights, 73 KB in bf16,
//   then enter the compute unit once; the halves meet in LDS).
// Rounding points are those of the per-layer kernels: the conv output and the activations are
// rounded to the storage type, sums are fp32.
#include "ddg_device.h"
#include "ddg_kernels.h"
#include <type_traits>

namespace ddg {

namespace ev {

constexpr int NT = 512;
constexpr size_t LDS_MAX = 160 * 1024;
constexpr int RED_BYTES = 2 * 8 * 2 * 64 * 16;   // exchange of the contraction halves, double-buffered
constexpr int DUMP_BYTES = 64 * 16;               // where lanes without a pixel write

// The layer table is in memory, so the compiler cannot see that the pointers in it are global ones, and
// the LDS regions change roles at run time: without help it makes flat accesses of both kinds, which
// wait for both memories. Pointers from the table are cast to the global address space, LDS is
// addressed by byte offsets from its start.
#define EV_GLOBAL __attribute__((address_space(1)))
template <typename V> __device__ __forceinline__ V load16(const void* p) {
  static_assert(sizeof(V) == 16, "16-byte vectors");
  return __builtin_bit_cast(V, *(const EV_GLOBAL u32x4_t*)(uintptr_t)p);
}
__device__ __forceinline__ float load_f(const float* p) { return *(const EV_GLOBAL float*)(uintptr_t)p; }
__device__ __forceinline__ unsigned char* lds() {
  extern __shared__ __align__(16) unsigned char smem[];
  return smem;
}

// bytes of a pixel of ch channels (of esz bytes; `gap`: as above), and of a buffer row of W pixels and their border
__host__ __device__ constexpr int pix_bytes_of(int ch, int esz, int gap) { return ch * esz <= 16 ? 16 : esz == 4 ? ch * 4 + 16 : ch == 16 ? 32 : ch * 2 + gap; }
template <typename T, int GAP> __host__ __device__ constexpr int pix_bytes(int ch) { return pix_bytes_of(ch, (int)sizeof(T), GAP); }
__host__ __device__ constexpr int row_bytes(int W, int pix) { return W % 16 == 0 || pix % 32 != 0 ? (W + 2) * pix : W * pix + (2 * pix + 255) / 256 * 256; }

struct Args {
  const EvalBlockDesc* blocks; int nb;   // the blocks this launch runs
  const EvalConvDesc* convs; int nconv;  // and their convolutions
  const void* in; void* out;
  int N, H, W, C;          // input of the first block (C: real channels)
  unsigned off1, off2, red_off, tab_off, dump_off;   // LDS offsets: second and third region, exchange area, scale / shift table
};
// A launch of one block in strips of TH output rows. Its convolutions come with the arguments: from a table in memory a workgroup would
// fetch the table, then the pointers, then what they point at.
struct StripArgs {
  EvalConvDesc conv[3];
  const void* in; void* out;
  int H, W, C, stride;     // input of the block (C: real channels)
  int TH, strips;
  unsigned off1, off2, red_off, tab_off;
};

// One convolution layer shape: CIN -> COUT, R x R, stride S, NCB channel blocks and 1/KS of the
// contraction per wave, U pixel blocks in flight.
template <typename T, int GAP, int CIN, int COUT, int R, int S, int NCB, int KS, int U>
struct Conv {
  typedef typename Mma<T>::frag_t frag_t;
  static constexpr int KV = Mma<T>::KV, KSTEP = Mma<T>::KSTEP, PIX = pix_bytes<T, GAP>(CIN);
  static constexpr int KSTEPS = (R * R * CIN + KSTEP - 1) / KSTEP, KPW = KSTEPS / KS;
  // Lanes of the last k-step past the last tap (16 channels in bf16, the stem) multiply zero weights; what they
  // read has to be zero as well, or an infinite activation becomes NaN in every channel: the buffer's first
  // pixel, which is border.
  static constexpr bool RAGGED = R * R * CIN % KSTEP != 0;
  static_assert(!RAGGED || KS == 1, "the last k-step is the last of every wave");
  static constexpr int NCB_ = NCB, KS_ = KS, U_ = U, OCB = COUT / 16, CBG = OCB / NCB, PG = 8 / (CBG * KS), PAD = R / 2;
  static_assert(KSTEPS % KS == 0 && OCB % NCB == 0 && 8 % (CBG * KS) == 0 && (KS == 1 || (PG == 1 && NCB == 1 && U % 2 == 0)), "wave layout");

  struct Wts { frag_t w[NCB][KPW]; float4 sc[NCB], sh[NCB]; };

  // this wave's place: channel-block group, half of the contraction, pixel group
  __device__ static __forceinline__ int cbg(int wave) { return wave % CBG; }
  __device__ static __forceinline__ int kh(int wave) { return KS == 1 ? 0 : (wave / CBG) % KS; }
  __device__ static __forceinline__ int pg(int wave) { return wave / (CBG * KS); }

  // weights from memory
  __device__ static __forceinline__ void load_weights(const EvalConvDesc& d, Wts& r, int wave, int lane) {
    const T* w = reinterpret_cast<const T*>(d.w);
#pragma unroll
    for (int b = 0; b < NCB; ++b)
#pragma unroll
      for (int ks = 0; ks < KPW; ++ks)
        r.w[b][ks] = load16<frag_t>(w + ((size_t)((kh(wave) * KPW + ks) * OCB + cbg(wave) * NCB + b) * 64 + lane) * KV);
  }
  // scale and shift ([COUT] each) from the LDS table
  __device__ static __forceinline__ void load_affine(const EvalConvDesc& d, int tab, Wts& r, int wave, int lane) {
    const float* sc = reinterpret_cast<const float*>(lds() + tab) + d.toff;
#pragma unroll
    for (int b = 0; b < NCB; ++b) {
      const int c = (cbg(wave) * NCB + b) * 16 + (lane >> 4) * 4;
      r.sc[b] = *reinterpret_cast<const float4*>(sc + c);
      r.sh[b] = *reinterpret_cast<const float4*>(sc + COUT + c);
    }
  }
  __device__ static __forceinline__ void load(const EvalConvDesc& d, int tab, Wts& r, int wave, int lane) {
    load_weights(d, r, wave, lane);
    load_affine(d, tab, r, wave, lane);
  }
  // per-lane LDS offset of k-step ks relative to the top left tap of an output pixel (RB: bytes of a
  // row of the source buffer)
  __device__ static __forceinline__ void addresses(int (&ka)[KPW], int wave, int lane, int RB) {
#pragma unroll
    for (int ks = 0; ks < KPW; ++ks) {
      const int k = ((kh(wave) * KPW + ks) * 4 + (lane >> 4)) * KV;
      const int tap = k / CIN, c0 = k % CIN;
      ka[ks] = tap < R * R ? (tap / R) * RB + (tap % R) * PIX + c0 * (int)sizeof(T) : 0;
    }
  }
  template <int V>
  __device__ static __forceinline__ void contract(int src, const int (&pa)[U], const int (&ka)[KPW], const Wts& wt, f32x4_t (&acc)[NCB][U]) {
#pragma unroll
    for (int ks = 0; ks < KPW; ++ks) {
      frag_t x[V];
#pragma unroll
      for (int u = 0; u < V; ++u) {
        const bool past = RAGGED && ks == KPW - 1 && (ks * 4 + (int)(threadIdx.x & 63) / 16) * KV >= R * R * CIN;
        x[u] = *reinterpret_cast<const frag_t*>(lds() + src + (past ? 0 : pa[u] + ka[ks]));
      }
#pragma unroll
      for (int b = 0; b < NCB; ++b)
#pragma unroll
        for (int u = 0; u < V; ++u) acc[b][u] = Mma<T>::mma(wt.w[b][ks], x[u], acc[b][u]);
    }
  }
  // The halves of the contraction meet: each wave hands U/2 pixel blocks over and finishes the others,
  // which end up in acc[0 .. U/2) (blocks 0 .. U/2-1 in the first half's waves, the rest in the second's).
  __device__ static __forceinline__ void exchange(f32x4_t (&acc)[U], int red, int& flip, int wave, int lane) {
    constexpr int E = U / 2 > 0 ? U / 2 : 1;
    f32x4_t* ex = reinterpret_cast<f32x4_t*>(lds() + red) + flip * (8 * E * 64);
    flip ^= 1;
    const int h = kh(wave), cb = cbg(wave);
#pragma unroll
    for (int i = 0; i < U / 2; ++i) ex[((cb * 2 + h) * E + i) * 64 + lane] = h == 0 ? acc[U / 2 + i] : acc[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < U / 2; ++i) acc[i] = (h == 0 ? acc[i] : acc[U / 2 + i]) + ex[((cb * 2 + (1 - h)) * E + i) * 64 + lane];
  }
  // Output rows [lo, hi) of W columns from the source buffer (its first row is image row srow0, RB
  // bytes a row). f(acc, channel block index, row, col, valid) once per 16-pixel block and channel block.
  template <typename F>
  __device__ static __forceinline__ void pass(int src, int srow0, int RB, int lo, int hi, int W,
                                              const int (&ka)[KPW], const Wts& wt, int red, int& flip,
                                              int wave, int lane, F f) {
    const int npx = (hi - lo) * W, npb = (npx + 15) >> 4;
    const float invW = 1.0f / (float)W;
    for (int g0 = pg(wave); g0 < npb; g0 += PG * U) {
      int row[U], col[U], pa[U];
      bool ok[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int p = (g0 + u * PG) * 16 + (lane & 15);
        ok[u] = p < npx;
        const int pc = ok[u] ? p : npx - 1;
        const int q = (int)(((float)pc + 0.5f) * invW);     // exact: pc < 2^16
        row[u] = lo + q; col[u] = pc - q * W;
        pa[u] = (row[u] * S - PAD - srow0) * RB + (col[u] * S - PAD + 1) * PIX;
      }
      f32x4_t acc[NCB][U];
#pragma unroll
      for (int b = 0; b < NCB; ++b)
#pragma unroll
        for (int u = 0; u < U; ++u) acc[b][u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      // (fp32 matrix instructions are worth a branch that leaves out a second block that does not exist)
      const bool all = sizeof(T) == 2 || U == 1 || g0 + (U - 1) * PG < npb;
      if (all) contract<U>(src, pa, ka, wt, acc);
      else contract<U == 1 ? 1 : U - 1>(src, pa, ka, wt, acc);
      if (KS == 1) {
#pragma unroll
        for (int b = 0; b < NCB; ++b)
#pragma unroll
          for (int u = 0; u < U; ++u) f(acc[b][u], b, row[u], col[u], ok[u]);
      } else {
        // the halves of the contraction meet: each wave hands two pixel blocks over and finishes two
        exchange(acc[0], red, flip, wave, lane);
        const int h = kh(wave);
#pragma unroll
        for (int i = 0; i < U / 2; ++i)
          f(acc[0][i], 0, h == 0 ? row[i] : row[U / 2 + i], h == 0 ? col[i] : col[U / 2 + i], h == 0 ? ok[i] : ok[U / 2 + i]);
      }
    }
  }
};

template <typename T, int GAP, int C> struct Same;       // 3x3, stride 1, C -> C
template <int GAP> struct Same<bf16_t, GAP, 16> { typedef Conv<bf16_t, GAP, 16, 16, 3, 1, 1, 1, 4> type; };
template <int GAP> struct Same<bf16_t, GAP, 32> { typedef Conv<bf16_t, GAP, 32, 32, 3, 1, GAP == 32 ? 1 : 2, 1, GAP == 32 ? 4 : 2> type; };
template <int GAP> struct Same<bf16_t, GAP, 64> { typedef Conv<bf16_t, GAP, 64, 64, 3, 1, 1, 2, 4> type; };
template <int GAP> struct Same<float, GAP, 16> { typedef Conv<float, GAP, 16, 16, 3, 1, 1, 1, 1> type; };
template <int GAP> struct Same<float, GAP, 32> { typedef Conv<float, GAP, 32, 32, 3, 1, 1, 1, 1> type; };
template <int GAP> struct Same<float, GAP, 64> { typedef Conv<float, GAP, 64, 64, 3, 1, 1, 2, 2> type; };
template <typename T, int GAP, int C> struct Down;       // 3x3, stride 2, C -> 2C
template <int GAP> struct Down<bf16_t, GAP, 16> { typedef Conv<bf16_t, GAP, 16, 32, 3, 2, 2, 1, 2> type; };
template <int GAP> struct Down<bf16_t, GAP, 32> { typedef Conv<bf16_t, GAP, 32, 64, 3, 2, 1, 1, 2> type; };
template <int GAP> struct Down<float, GAP, 16> { typedef Conv<float, GAP, 16, 32, 3, 2, 1, 1, 1> type; };
template <int GAP> struct Down<float, GAP, 32> { typedef Conv<float, GAP, 32, 64, 3, 2, 1, 1, 1> type; };

// The thread's index, as a value the compiler does not know: the lane-dependent addresses of a stage are then computed where the
// stage begins. Otherwise those of all stages are hoisted to the start of the kernel, and spilled.
template <typename T> __device__ __forceinline__ int own_tid() {
  int t = threadIdx.x;
  if (sizeof(T) == 2) asm volatile("" : "+v"(t));
  return t;
}

// what a workgroup holds between blocks
struct Bufs {
  int x, o, y;     // LDS offsets
  int row0;        // image row of buffer row 0 of x
  int H, W;        // of x
};

template <typename T>
__device__ __forceinline__ void zero(int p, int bytes) {
  for (int i = threadIdx.x * 16; i < bytes; i += NT * 16) *reinterpret_cast<uint4*>(lds() + p + i) = make_uint4(0, 0, 0, 0);
}

// z (as stored) * scale + shift of four channels
__device__ __forceinline__ void as_stored(const f32x4_t& a, float (&v)[4], bf16_t) {
  const uint32_t p = Store<bf16_t>::pack2(a[0], a[1]), q = Store<bf16_t>::pack2(a[2], a[3]);
  v[0] = __uint_as_float(p << 16); v[1] = __uint_as_float(p & 0xffff0000u);
  v[2] = __uint_as_float(q << 16); v[3] = __uint_as_float(q & 0xffff0000u);
}
__device__ __forceinline__ void as_stored(const f32x4_t& a, float (&v)[4], float) { v[0] = a[0]; v[1] = a[1]; v[2] = a[2]; v[3] = a[3]; }
template <typename T>
__device__ __forceinline__ void affine(const f32x4_t& a, const float4& sc, const float4& sh, float (&v)[4]) {
  as_stored(a, v, T{});
  v[0] = v[0] * sc.x + sh.x; v[1] = v[1] * sc.y + sh.y; v[2] = v[2] * sc.z + sh.z; v[3] = v[3] * sc.w + sh.w;
}
template <typename T>
__device__ __forceinline__ void store_relu(int p, const float (&v)[4]) {
  Store<T>::store4(reinterpret_cast<T*>(lds() + p), fmaxf(v[0], 0.f), fmaxf(v[1], 0.f), fmaxf(v[2], 0.f), fmaxf(v[3], 0.f));
}

// Lane l of an accumulator pair (two pixel blocks, rounded to bf16) holds channels 4*(l/16) .. +3 of pixel l%16 of either
// block. Swapping rows of 16 lanes gives every lane 8 channels of one pixel: channels 8*(l/32) .. +7, pixel l%16 of the
// first block (l/16 even) or the second (odd), so that LDS sees 16-byte accesses instead of twice as many of 8.
__device__ __forceinline__ uint4 pair_rows(const f32x4_t& a, const f32x4_t& b) {
  const auto lo = __builtin_amdgcn_permlane16_swap(Store<bf16_t>::pack2(a[0], a[1]), Store<bf16_t>::pack2(b[0], b[1]), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(Store<bf16_t>::pack2(a[2], a[3]), Store<bf16_t>::pack2(b[2], b[3]), false, false);
  return make_uint4(lo[0], hi[0], lo[1], hi[1]);
}

// Identity blocks on whole images of the usual size, 512 / C pixels wide and high (bf16). A wave owns NB pixel blocks
// below each other (a block is 16 pixels: half a row, a row, or two rows of 8) and walks down the input rows: what it reads
// of a row serves every output row that the row is a tap of, 26 / 18 / 27 fragment reads a layer instead of 40 / 36 / 36 with
// a tap at a time, which is most of the LDS time that bounds a layer. All addresses are one per-lane register and an
// instruction immediate. Fragments are requested D rows ahead, and finished pairs of blocks are normalised and stored
// between the matrix instructions of the next row. Eight waves:
//   16 channels: half a row x 8 rows. A k-step (32) is two taps: columns -1 and 0 of a row; column 1 of a row and the
//                next; column 1 of the last row alone (the other lanes read border and multiply zero weights);
//   32 channels: one channel block x 4 rows; a k-step is a tap;
//   64 channels: one channel block x half of the input channels, all four blocks; the halves meet in LDS.
template <int GAP, int C>
__device__ __forceinline__ void identity_square(const EvalConvDesc* cv, int tab, int count, Bufs& B, int red, int& flip) {
  typedef bf16_t T;
  typedef typename Same<T, GAP, C>::type K;
  typedef Mma<T>::frag_t frag_t;
  constexpr int PIX = K::PIX, W = 512 / C, RB = row_bytes(W, PIX), OCB = C / 16;
  constexpr int BLK = C == 64 ? 2 : 1, NB = C == 16 ? 8 : 4, NT = NB * BLK + 3 - BLK;   // rows of a block, blocks of a wave, row positions it reads
  constexpr int NW = C == 16 ? 5 : 9, D = 3, F = C == 64 ? 2 : NB;                     // weight fragments; blocks a wave finishes
  const int tid = own_tid<T>(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lg = lane >> 4;
  const int cb = C == 16 ? 0 : C == 32 ? wave & 1 : wave & 3, half = C == 64 ? wave >> 2 : 0;      // channel block; half of the contraction
  const int row0 = C == 64 ? 0 : (wave >> 1) * NB;
  const int base = C == 16 ? row0 * RB + ((wave & 1) * 16 + l16) * PIX : C == 32 ? row0 * RB + l16 * PIX : (l16 >> 3) * RB + (l16 & 7) * PIX;
  // fragment k of row position t at ka[k] + t * RB
  int ka[3];
  if (C == 16) {
    ka[0] = base + (lg >> 1) * PIX + (lg & 1) * 16;
    ka[1] = base + 2 * PIX + (lg >> 1) * RB + (lg & 1) * 16;
    ka[2] = lg < 2 ? base + 2 * PIX + lg * 16 : 0;           // (column -1 of every row is border)
  } else {
#pragma unroll
    for (int k = 0; k < 3; ++k) ka[k] = base + k * PIX + half * 64 + lg * 16;
  }
  const int c0 = cb * 16 + (lane >> 5) * 8;                  // this lane's 8 channels, and where it finishes a pair of blocks
  const int da = base + RB + PIX + c0 * (int)sizeof(T) + (lg & 1) * BLK * RB + (C == 64 ? half * 2 * BLK * RB : 0);
  // Weights are requested a layer ahead, their address (from the table in memory) two.
  struct Wts { frag_t w[NW]; } w1, w2;
  int wo[NW];                                                // element offsets in the packed operand [k-step][channel block][lane][8]
#pragma unroll
  for (int k = 0; k < NW; ++k) {
    const int tap = k < 3 ? k * 3 + (lg >> 1) : k == 3 ? (lg >> 1) * 3 + 2 : 8 + (lg >> 1);        // (16 channels; tap 9: zeros)
    wo[k] = C == 16 ? ((tap >> 1) * 64 + ((tap & 1) * 2 + (lg & 1)) * 16 + l16) * 8 : (((C == 64 ? k * 2 + half : k) * OCB + cb) * 64 + lane) * 8;
  }
  uint64_t wp = reinterpret_cast<uint64_t>(cv[0].w);
  auto load = [&](Wts& r, int next) __attribute__((always_inline)) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)wp), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(wp >> 32));
    const uint64_t u = (uint64_t)hi << 32 | lo;
#pragma unroll
    for (int k = 0; k < NW; ++k) r.w[k] = load16<frag_t>(reinterpret_cast<const T*>(u) + wo[k]);
    if (next < 2 * count) wp = reinterpret_cast<uint64_t>(cv[next].w);
  };
  int st = tab + (cv[0].toff + c0) * 4;                      // scale and shift of the layer's channels, 2 * C floats a layer
  load(w1, 1);
  // one layer: dst = relu(bn(conv(src)) [+ dst])
  auto layer = [&](int src, const Wts& wt, int dst, auto add) __attribute__((always_inline)) {
    constexpr bool ADD = decltype(add)::value;
    f32x4_t acc[NB];
    frag_t x[D][3];
    uint4 r[F / 2];
    auto request = [&](int t) __attribute__((always_inline)) {
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (C != 16 || k == 0 || (k == 1 && t < NB) || (k == 2 && t >= 2)) x[t % D][k] = *reinterpret_cast<const frag_t*>(lds() + src + ka[k] + t * RB);
    };
#pragma unroll
    for (int t = 0; t < D; ++t) request(t);
    float sc[8], sh[8];
    Store<float>::load4(reinterpret_cast<const float*>(lds() + st), *reinterpret_cast<float(*)[4]>(&sc[0]));
    Store<float>::load4(reinterpret_cast<const float*>(lds() + st + 16), *reinterpret_cast<float(*)[4]>(&sc[4]));
    Store<float>::load4(reinterpret_cast<const float*>(lds() + st + 4 * C), *reinterpret_cast<float(*)[4]>(&sh[0]));
    Store<float>::load4(reinterpret_cast<const float*>(lds() + st + 4 * C + 16), *reinterpret_cast<float(*)[4]>(&sh[4]));
    st += 8 * C;
#pragma unroll
    for (int i = 0; i < F / 2; ++i)
      if (ADD) r[i] = *reinterpret_cast<const uint4*>(lds() + dst + da + i * 2 * BLK * RB);
    auto finish = [&](int i) __attribute__((always_inline)) {   // blocks 2 * i and 2 * i + 1
      float v[8], q[8];
      Store<T>::unpack_vec(pair_rows(acc[2 * i], acc[2 * i + 1]), v);
      if (ADD) Store<T>::unpack_vec(r[i], q);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        v[e] = v[e] * sc[e] + sh[e];
        if (ADD) v[e] += q[e];
        v[e] = fmaxf(v[e], 0.f);
      }
      Store<T>::store_vec(reinterpret_cast<T*>(lds() + dst + da + i * 2 * BLK * RB), v);
    };
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      __builtin_amdgcn_sched_barrier(0);
      // the blocks this row position is tap row dy of
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int dy = 0; dy < 3; ++dy) {
          const int b = (t - dy) / BLK;
          if (t < dy || (t - dy) % BLK != 0 || b >= NB) continue;
          if (C == 16 && ((k == 1 && dy != 0) || (k == 2 && dy != 2))) continue;
          acc[b] = Mma<T>::mma(wt.w[C == 16 ? (k == 0 ? dy : 2 + k) : dy * 3 + k], x[t % D][k], acc[b]);
        }
      if (t + D < NT) request(t + D);
      const int last = t - 1 - 2;      // the position before completed block last / BLK
      if (C != 64 && last >= 0 && last % 2 == 1) {
        finish(last / 2);
#pragma unroll
        for (int k = 0; k < 9; ++k) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // a matrix instruction,
          __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);   // five vector instructions of the pair before
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (C == 64) K::exchange(acc, red, flip, wave, lane);
    finish(F / 2 - 1);
  };
  for (int i = 0; i < count; ++i) {
    load(w2, 2 * i + 2);
    layer(B.x, w1, B.o, std::false_type{});
    __syncthreads();
    if (i + 1 < count) load(w1, 2 * i + 3);
    layer(B.o, w2, B.x, std::true_type{});
    __syncthreads();
  }
}

// Identity blocks on whole images whose pixel blocks fit G groups per wave: every address of a layer
// is the same for all layers of the run (both buffers start at image row -1), so a lane computes its
// pixels' offsets once. Lanes past the last pixel write to `dump`.
template <typename T, int GAP, int C, int G>
__device__ __forceinline__ void identity_images(const EvalConvDesc* cv, int tab, int count, Bufs& B, int red, int dump, int& flip) {
  typedef typename Same<T, GAP, C>::type K;
  constexpr int PIX = K::PIX, U = K::U_, NCB = K::NCB_, F = K::KS_ == 1 ? U : U / 2;   // F: pixel blocks a wave finishes per group
  const int tid = own_tid<T>(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int W = B.W, RB = row_bytes(W, PIX), npx = B.H * W;
  int ka[K::KPW];
  K::addresses(ka, wave, lane, RB);
  const int centre = RB + PIX + (K::cbg(wave) * NCB * 16 + (lane >> 4) * 4) * (int)sizeof(T);
  int pa[G][U], da[G][F];
  const float invW = 1.0f / (float)W;
#pragma unroll
  for (int g = 0; g < G; ++g) {
    int ok[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int p = ((g * U + u) * K::PG + K::pg(wave)) * 16 + (lane & 15), pc = p < npx ? p : npx - 1;
      const int q = (int)(((float)pc + 0.5f) * invW);
      pa[g][u] = q * RB + (pc - q * W) * PIX;
      ok[u] = p < npx ? pa[g][u] + centre : -1;
    }
#pragma unroll
    for (int i = 0; i < F; ++i) da[g][i] = (K::KS_ == 1 || K::kh(wave) == 0) ? ok[i] : ok[U - F + i];
  }
  typename K::Wts w1, w2;
  K::load(cv[0], tab, w1, wave, lane);
  auto layer = [&](int src, const typename K::Wts& wt, int g, f32x4_t (&acc)[NCB][U]) __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < NCB; ++b)
#pragma unroll
      for (int u = 0; u < U; ++u) acc[b][u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    K::template contract<U>(src, pa[g], ka, wt, acc);
    if (K::KS_ == 2) K::exchange(acc[0], red, flip, wave, lane);
  };
  for (int i = 0; i < count; ++i) {
    K::load(cv[2 * i + 1], tab, w2, wave, lane);
#pragma unroll
    for (int g = 0; g < G; ++g) {
      f32x4_t acc[NCB][U];
      layer(B.x, w1, g, acc);
#pragma unroll
      for (int b = 0; b < NCB; ++b)
#pragma unroll
        for (int u = 0; u < F; ++u) {
          float v[4];
          affine<T>(acc[b][u], w1.sc[b], w1.sh[b], v);
          store_relu<T>(da[g][u] >= 0 ? B.o + da[g][u] + b * 16 * (int)sizeof(T) : dump + lane * 16, v);
        }
    }
    __syncthreads();
    if (i + 1 < count) K::load(cv[2 * i + 2], tab, w1, wave, lane);
#pragma unroll
    for (int g = 0; g < G; ++g) {
      f32x4_t acc[NCB][U];
      layer(B.o, w2, g, acc);
#pragma unroll
      for (int b = 0; b < NCB; ++b)
#pragma unroll
        for (int u = 0; u < F; ++u) {
          float v[4], r[4];
          const int p = da[g][u] >= 0 ? B.x + da[g][u] + b * 16 * (int)sizeof(T) : dump + lane * 16;
          affine<T>(acc[b][u], w2.sc[b], w2.sh[b], v);
          Store<T>::load4(reinterpret_cast<const T*>(lds() + p), r);
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] += r[e];
          store_relu<T>(p, v);
        }
    }
    __syncthreads();
  }
}

// `count` identity blocks of C channels, output rows [lo, hi) (all rows when count > 1). pre() is what has to be done before the
// first contraction, with both layers' weights on their way; it is followed by a barrier. last(v, row, channel, pixel, valid) takes
// four channels of an output pixel of the last block (of every block when count > 1).
template <typename T, int GAP, int C, typename Pre, typename Last>
__device__ __forceinline__ void identity_run(const EvalConvDesc* cv, int tab, int count, Bufs& B, int lo, int hi, int red, int& flip, Pre pre, Last last) {
  typedef typename Same<T, GAP, C>::type K;
  constexpr int PIX = K::PIX;
  const int tid = own_tid<T>(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int W = B.W, RB = row_bytes(W, PIX);
  const int olo = lo > 0 ? lo - 1 : 0, ohi = hi < B.H ? hi + 1 : B.H;
  const int orow0 = lo - 1;
  const int cq = K::cbg(wave) * K::NCB_ * 16 + (lane >> 4) * 4;
  typename K::Wts w1, w2;
  K::load_weights(cv[0], w1, wave, lane);
  K::load_weights(cv[1], w2, wave, lane);
  int ka[K::KPW];
  K::addresses(ka, wave, lane, RB);
  pre();
  __syncthreads();
  K::load_affine(cv[0], tab, w1, wave, lane);
  for (int i = 0; i < count; ++i) {
    if (i > 0) K::load_weights(cv[2 * i + 1], w2, wave, lane);
    K::load_affine(cv[2 * i + 1], tab, w2, wave, lane);
    K::pass(B.x, B.row0, RB, olo, ohi, W, ka, w1, red, flip, wave, lane,
            [&](const f32x4_t& acc, int b, int row, int col, bool ok) __attribute__((always_inline)) {
              float v[4];
              affine<T>(acc, w1.sc[b], w1.sh[b], v);
              if (ok) store_relu<T>(B.o + (row - orow0) * RB + (col + 1) * PIX + (cq + b * 16) * (int)sizeof(T), v);
            });
    __syncthreads();
    if (i + 1 < count) K::load(cv[2 * i + 2], tab, w1, wave, lane);
    K::pass(B.o, orow0, RB, lo, hi, W, ka, w2, red, flip, wave, lane,
            [&](const f32x4_t& acc, int b, int row, int col, bool ok) __attribute__((always_inline)) {
              float v[4], r[4];
              affine<T>(acc, w2.sc[b], w2.sh[b], v);
              const int p = B.x + (row - B.row0) * RB + (col + 1) * PIX + (cq + b * 16) * (int)sizeof(T);
              Store<T>::load4(reinterpret_cast<const T*>(lds() + p), r);
#pragma unroll
              for (int e = 0; e < 4; ++e) v[e] += r[e];
              last(v, cq + b * 16, row, col, p, ok);
            });
    if (i + 1 < count) __syncthreads();
  }
}

// A block between stages: C -> 2C channels, stride 2, 1x1 projection on the shortcut (pre, last: as above)
template <typename T, int GAP, int C, typename Pre, typename Last>
__device__ __forceinline__ void down_block(const EvalConvDesc* cv, int tab, const Bufs& B, int lo, int hi, int Ho, int Wo, int red, int& flip, Pre pre, Last last) {
  typedef typename Down<T, GAP, C>::type K1;
  typedef typename Same<T, GAP, 2 * C>::type K2;
  typedef Conv<T, GAP, C, 2 * C, 1, 2, K2::NCB_, 1, 1> KP;    // (only its weight layout: same channel blocks as K2)
  const int tid = own_tid<T>(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int RB = row_bytes(B.W, K1::PIX), RBo = row_bytes(Wo, K2::PIX);
  const int olo = lo > 0 ? lo - 1 : 0, ohi = hi < Ho ? hi + 1 : Ho;
  const int orow0 = lo - 1;
  typename K1::Wts w1;
  typename K2::Wts w2;
  K1::load_weights(cv[0], w1, wave, lane);
  K2::load_weights(cv[1], w2, wave, lane);
  zero<T>(B.o, (hi - lo + 2) * RBo);
  pre();
  __syncthreads();
  K1::load_affine(cv[0], tab, w1, wave, lane);
  {
    int ka[K1::KPW];
    K1::addresses(ka, wave, lane, RB);
    const int cq = K1::cbg(wave) * K1::NCB_ * 16 + (lane >> 4) * 4;
    K1::pass(B.x, B.row0, RB, olo, ohi, Wo, ka, w1, red, flip, wave, lane,
             [&](const f32x4_t& acc, int b, int row, int col, bool ok) __attribute__((always_inline)) {
               float v[4];
               affine<T>(acc, w1.sc[b], w1.sh[b], v);
               if (ok) store_relu<T>(B.o + (row - orow0) * RBo + (col + 1) * K2::PIX + (cq + b * 16) * (int)sizeof(T), v);
             });
  }
  // the projection: every wave the channel blocks it finishes, the whole contraction
  const int cg = K2::cbg(wave), cq = cg * K2::NCB_ * 16 + (lane >> 4) * 4;
  typename KP::frag_t wp[K2::NCB_][KP::KPW];
  float4 psc[K2::NCB_], psh[K2::NCB_];
#pragma unroll
  for (int b = 0; b < K2::NCB_; ++b) {
#pragma unroll
    for (int ks = 0; ks < KP::KPW; ++ks)
      wp[b][ks] = load16<typename KP::frag_t>(reinterpret_cast<const T*>(cv[2].w) +
                                              ((size_t)(ks * KP::OCB + cg * K2::NCB_ + b) * 64 + lane) * KP::KV);
    psc[b] = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(lds() + tab) + cv[2].toff + cq + b * 16);
    psh[b] = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(lds() + tab) + cv[2].toff + 2 * C + cq + b * 16);
  }
  K2::load_affine(cv[1], tab, w2, wave, lane);
  __syncthreads();
  {
    int ka[K2::KPW], kp[KP::KPW];
    K2::addresses(ka, wave, lane, RBo);
#pragma unroll
    for (int ks = 0; ks < KP::KPW; ++ks) {
      const int k = (ks * 4 + (lane >> 4)) * KP::KV;
      kp[ks] = k < C ? k * (int)sizeof(T) : -1;          // (past the last channel: the buffer's first pixel, border)
    }
    K2::pass(B.o, orow0, RBo, lo, hi, Wo, ka, w2, red, flip, wave, lane,
             [&](const f32x4_t& acc, int b, int row, int col, bool ok) __attribute__((always_inline)) {
               const int xp = (row * 2 - B.row0) * RB + (col * 2 + 1) * K1::PIX;
               f32x4_t pa = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
               for (int ks = 0; ks < KP::KPW; ++ks)
                 pa = Mma<T>::mma(wp[b][ks], *reinterpret_cast<const typename KP::frag_t*>(lds() + B.x + (kp[ks] < 0 ? 0 : xp + kp[ks])), pa);
               float v[4], r[4];
               affine<T>(acc, w2.sc[b], w2.sh[b], v);
               affine<T>(pa, psc[b], psh[b], r);
#pragma unroll
               for (int e = 0; e < 4; ++e) v[e] += r[e];
               last(v, cq + b * 16, row, col, B.y + (row - orow0) * RBo + (col + 1) * K2::PIX + (cq + b * 16) * (int)sizeof(T), ok);
             });
  }
}

// rows [row0, row0 + rows) of an image with C channels into a buffer with a zero border
template <typename T>
__device__ __forceinline__ void load_rows(int buf, const T* img, int row0, int rows, int H, int W, int C, int pix) {
  constexpr int V = Store<T>::VEC;
  const int cpp = pix / 16, per_row = row_bytes(W, pix) / 16, total = rows * per_row;   // 16-byte chunks, padding included
  const int ch = C / V;
  for (int i = threadIdx.x; i < total; i += NT) {
    const int r = i / per_row, e = i - r * per_row, px = e / cpp, k = e - px * cpp;
    const int h = row0 + r, w = px - 1;
    uint4 q = make_uint4(0, 0, 0, 0);
    if (k < ch && h >= 0 && h < H && w >= 0 && w < W)
      q = *reinterpret_cast<const uint4*>(img + ((size_t)h * W + w) * C + k * V);
    *reinterpret_cast<uint4*>(lds() + buf + i * 16) = q;
  }
}
// the network input: up to KV channels per pixel, one 16-byte chunk each
template <typename T>
__device__ __forceinline__ void load_rows_stem(int buf, const T* img, int row0, int rows, int H, int W, int C) {
  constexpr int V = Store<T>::VEC;
  const int per_row = row_bytes(W, 16) / 16, total = rows * per_row;
  for (int i = threadIdx.x; i < total; i += NT) {
    const int r = i / per_row, w = i - r * per_row - 1, h = row0 + r;
    float f[V];
#pragma unroll
    for (int e = 0; e < V; ++e) f[e] = 0.f;
    if (h >= 0 && h < H && w >= 0 && w < W)
#pragma unroll
      for (int e = 0; e < V; ++e) if (e < C) f[e] = Store<T>::load1(img + ((size_t)h * W + w) * C + e);
    Store<T>::store_vec(reinterpret_cast<T*>(lds() + buf + i * 16), f);
  }
}

// the blocks of a launch, an image per workgroup
template <typename T, int GAP>
__global__ __launch_bounds__(NT) void eval_blocks_kernel(Args a) {
  const int n = blockIdx.x;
  const int tid = threadIdx.x;
  const int red = (int)a.red_off;
  int flip = 0;
  Bufs B;
  B.x = 0; B.o = (int)a.off1; B.y = (int)a.off2;
  B.H = a.H; B.W = a.W;
  int C = a.C;
  const T* img = reinterpret_cast<const T*>(a.in) + (size_t)n * a.H * a.W * a.C;
  const EvalBlockDesc& b0 = a.blocks[0];
  const int Ho0 = (a.H - 1) / (b0.kind == EVAL_DOWN ? 2 : b0.stride) + 1;
  B.row0 = -1;
  {
    const int rows = (Ho0 - 1) * (b0.kind == EVAL_DOWN ? 2 : b0.stride) + 3;
    if (b0.kind == EVAL_STEM) {
      load_rows_stem<T>(B.o, img, B.row0, rows, a.H, a.W, a.C);
    } else {
      load_rows<T>(B.x, img, B.row0, rows, a.H, a.W, a.C, pix_bytes<T, GAP>(a.C));
      if (b0.kind == EVAL_IDENTITY) zero<T>(B.o, (a.H + 2) * row_bytes(a.W, pix_bytes<T, GAP>(a.C)));
    }
  }
  // scale and shift of every batch norm of the launch, a wave per layer and four layers at a time
  float* const tab0 = reinterpret_cast<float*>(lds() + a.tab_off);
  const int tab = (int)a.tab_off - 4 * a.convs[0].toff;
  {
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int c0 = wave; c0 < a.nconv; c0 += 32) {
      float g[4], be[4], rm[4], rv[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int ci = c0 + k * 8 < a.nconv ? c0 + k * 8 : c0;
        const EvalConvDesc& d = a.convs[ci];
        const int c = lane < d.cout ? lane : 0;
        g[k] = load_f(d.gamma + c); be[k] = load_f(d.beta + c); rm[k] = load_f(d.rmean + c); rv[k] = load_f(d.rvar + c);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (c0 + k * 8 >= a.nconv) break;
        const EvalConvDesc& d = a.convs[c0 + k * 8];
        const float sc = g[k] / sqrtf(rv[k] + d.eps);
        if (lane < d.cout) {
          tab0[d.toff - a.convs[0].toff + lane] = sc;
          tab0[d.toff - a.convs[0].toff + d.cout + lane] = be[k] - rm[k] * sc;
        }
      }
    }
  }
  int bi = 0;
  if (b0.kind == EVAL_STEM) {
    typedef Conv<T, GAP, Mma<T>::KV, 16, 3, 1, 1, 1, 2> K1;
    typedef Conv<T, GAP, Mma<T>::KV, 16, 3, 2, 1, 1, 2> K2;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int Wo = (a.W - 1) / b0.stride + 1, srow0 = B.row0;
    constexpr int PIX = pix_bytes<T, GAP>(16);
    const int RBo = row_bytes(Wo, PIX), RBi = row_bytes(a.W, K1::PIX);
    zero<T>(B.x, (Ho0 + 2) * RBo);
    typename K1::Wts w;
    __syncthreads();
    K1::load(a.convs[0], tab, w, wave, lane);
    int ka[K1::KPW];
    K1::addresses(ka, wave, lane, RBi);
    __syncthreads();
    auto put = [&](const f32x4_t& acc, int b, int row, int col, bool ok) __attribute__((always_inline)) {
      float v[4];
      affine<T>(acc, w.sc[b], w.sh[b], v);
      if (ok) store_relu<T>(B.x + (row - B.row0) * RBo + (col + 1) * PIX + (lane >> 4) * 4 * (int)sizeof(T), v);
    };
    if (b0.stride == 1) {
      K1::pass(B.o, srow0, RBi, 0, Ho0, Wo, ka, w, red, flip, wave, lane, put);
    } else {
      typename K2::Wts v2;
#pragma unroll
      for (int k = 0; k < K2::KPW; ++k) v2.w[0][k] = w.w[0][k];
      K2::pass(B.o, srow0, RBi, 0, Ho0, Wo, ka, v2, red, flip, wave, lane, put);
    }
    B.H = Ho0; B.W = Wo; C = 16;
    __syncthreads();
    bi = 1;
    if (bi < a.nb) zero<T>(B.o, (B.H + 2) * row_bytes(B.W, PIX));   // (the input image was there)
  }
  __syncthreads();
  auto none = [] {};
  auto in_lds = [](float (&v)[4], int, int, int, int p, bool ok) __attribute__((always_inline)) { if (ok) store_relu<T>(p, v); };
  while (bi < a.nb) {
    const EvalConvDesc* cv = a.convs + (a.blocks[bi].conv0 - a.blocks[0].conv0);
    if (a.blocks[bi].kind == EVAL_IDENTITY) {
      int cnt = 1;
      while (bi + cnt < a.nb && a.blocks[bi + cnt].kind == EVAL_IDENTITY) ++cnt;
      const int npx = B.H * B.W;
      const bool square = B.W == 512 / C && B.H == B.W;
      if (C == 16) {
        if (square) identity_square<GAP, 16>(cv, tab, cnt, B, red, flip);
        else if (npx <= 1024) identity_images<T, GAP, 16, 2>(cv, tab, cnt, B, red, (int)a.dump_off, flip);
        else identity_run<T, GAP, 16>(cv, tab, cnt, B, 0, B.H, red, flip, none, in_lds);
      } else if (C == 32) {
        if (square) identity_square<GAP, 32>(cv, tab, cnt, B, red, flip);
        else if (npx <= 256) identity_images<T, GAP, 32, 1>(cv, tab, cnt, B, red, (int)a.dump_off, flip);
        else identity_run<T, GAP, 32>(cv, tab, cnt, B, 0, B.H, red, flip, none, in_lds);
      } else {
        if (square) identity_square<GAP, 64>(cv, tab, cnt, B, red, flip);
        else if (npx <= 64) identity_images<T, GAP, 64, 1>(cv, tab, cnt, B, red, (int)a.dump_off, flip);
        else identity_run<T, GAP, 64>(cv, tab, cnt, B, 0, B.H, red, flip, none, in_lds);
      }
      __syncthreads();
      bi += cnt;
    } else {
      const int Ho = (B.H - 1) / 2 + 1, Wo = (B.W - 1) / 2 + 1;
      zero<T>(B.y, (Ho + 2) * row_bytes(Wo, pix_bytes<T, GAP>(2 * C)));
      if (C == 16) down_block<T, GAP, 16>(cv, tab, B, 0, Ho, Ho, Wo, red, flip, none, in_lds);
      else down_block<T, GAP, 32>(cv, tab, B, 0, Ho, Ho, Wo, red, flip, none, in_lds);
      __syncthreads();
      const int t = B.x; B.x = B.y; B.y = t;
      B.H = Ho; B.W = Wo;
      C *= 2;
      ++bi;
    }
  }
  // the image's output
  constexpr int V = Store<T>::VEC;
  const int ch = C / V, pix = pix_bytes<T, GAP>(C), RB = row_bytes(B.W, pix), per_row = B.W * ch, total = B.H * per_row;
  T* out = reinterpret_cast<T*>(a.out) + (size_t)n * B.H * B.W * C;
  for (int i = tid; i < total; i += NT) {
    const int r = i / per_row, e = i - r * per_row, px = e / ch, k = e - px * ch;
    *reinterpret_cast<uint4*>(out + (size_t)i * V) =
        *reinterpret_cast<const uint4*>(lds() + B.x + (r + 1) * RB + (px + 1) * pix + k * 16);
  }
}

// One block in strips. A workgroup runs 3-10 us, most of it waiting for memory, so everything it reads is requested before anything is
// waited for: batch-norm vectors, the first rows, the weights of both layers. KIND and C (input channels; stem: none) at
// compile time: the code of one kind of block is a tenth of that of all of them.
template <typename T, int GAP, int KIND, int C>
__global__ __launch_bounds__(NT) void eval_strip_kernel(StripArgs a) {
  constexpr int V = Store<T>::VEC, NCONV = KIND == EVAL_STEM ? 1 : KIND == EVAL_IDENTITY ? 2 : 3, CO = KIND == EVAL_STEM ? 16 : KIND == EVAL_IDENTITY ? C : 2 * C;
  const int n = blockIdx.x / a.strips, st = blockIdx.x - n * a.strips;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int red = (int)a.red_off;
  int flip = 0;
  Bufs B;
  B.x = 0; B.o = (int)a.off1; B.y = (int)a.off2;
  B.H = a.H; B.W = a.W;
  const T* img = reinterpret_cast<const T*>(a.in) + (size_t)n * a.H * a.W * a.C;
  // output rows of this workgroup, and the input rows they need
  const int s0 = KIND == EVAL_DOWN ? 2 : KIND == EVAL_STEM ? a.stride : 1;
  const int Ho = (a.H - 1) / s0 + 1, Wo = (a.W - 1) / s0 + 1;
  const int lo = st * a.TH, hi = lo + a.TH < Ho ? lo + a.TH : Ho;
  const int olo = KIND == EVAL_STEM ? lo : (lo > 0 ? lo - 1 : 0), ohi = KIND == EVAL_STEM ? hi : (hi < Ho ? hi + 1 : Ho);
  B.row0 = olo * s0 - 1;
  const int rows = (ohi - 1) * s0 + 2 - B.row0;
  // ---- batch norms: a wave per convolution
  float g = 0.f, be = 0.f, rm = 0.f, rv = 0.f;
  const EvalConvDesc& mine = a.conv[wave < NCONV ? wave : 0];
  const int mc = lane < mine.cout ? lane : 0;
  if (wave < NCONV) { g = load_f(mine.gamma + mc); be = load_f(mine.beta + mc); rm = load_f(mine.rmean + mc); rv = load_f(mine.rvar + mc); }
  // ---- input rows, zero border and padding between pixels included: 16-byte chunks of LDS, U of a thread at a time
  constexpr int U = 4;
  uint4 q[U];
  constexpr int PIXI = KIND == EVAL_STEM ? 16 : pix_bytes<T, GAP>(C);
  const int per_row = row_bytes(a.W, PIXI) / 16, total = rows * per_row;
  const wide_rsrc_t ri = wide_rsrc(img, (size_t)a.H * a.W * a.C * sizeof(T));
  auto request = [&](int i0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * NT, r = i / per_row, e = i - r * per_row, h = B.row0 + r;
      const int w = e / (PIXI / 16) - 1, k = e % (PIXI / 16);
      const bool in = i < total && h >= 0 && h < a.H && w >= 0 && w < a.W;
      if (KIND == EVAL_STEM) {        // up to V channels of a pixel
        float f[V];
#pragma unroll
        for (int c = 0; c < V; ++c) f[c] = in && c < a.C ? Store<T>::load1(img + ((size_t)h * a.W + w) * a.C + c) : 0.f;
        if (sizeof(T) == 4) q[u] = make_uint4(__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3]));
        else q[u] = make_uint4(Store<bf16_t>::pack2(f[0], f[1]), Store<bf16_t>::pack2(f[2], f[3]), 0u, 0u);
      } else {
        q[u] = wide_load(ri, in && k < C / V ? (unsigned)((h * a.W + w) * C + k * V) * (unsigned)sizeof(T) : NOWHERE, 0);
      }
    }
  };
  const int dst = KIND == EVAL_STEM ? B.o : B.x;
  if (KIND != EVAL_STEM) request(tid);
  const int tab = (int)a.tab_off - 4 * a.conv[0].toff;
  auto pre = [&]() __attribute__((always_inline)) {
    if (KIND == EVAL_IDENTITY) zero<T>(B.o, (hi - lo + 2) * row_bytes(a.W, PIXI));
    if (wave < NCONV && lane < mine.cout) {
      float* t = reinterpret_cast<float*>(lds() + tab) + mine.toff;
      const float sc = g / sqrtf(rv + mine.eps);
      t[lane] = sc; t[mine.cout + lane] = be - rm * sc;
    }
    for (int i0 = tid; i0 < total; i0 += U * NT) {
      if (KIND == EVAL_STEM || i0 != tid) request(i0);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (i0 + u * NT < total) *reinterpret_cast<uint4*>(lds() + dst + (i0 + u * NT) * 16) = q[u];
    }
  };
  T* out = reinterpret_cast<T*>(a.out) + (size_t)n * Ho * Wo * CO;
  auto last = [&](float (&v)[4], int c, int row, int col, int, bool ok) __attribute__((always_inline)) {
    if (ok) Store<T>::store4(out + ((size_t)row * Wo + col) * CO + c, fmaxf(v[0], 0.f), fmaxf(v[1], 0.f), fmaxf(v[2], 0.f), fmaxf(v[3], 0.f));
  };
  if constexpr (KIND == EVAL_IDENTITY) {
    identity_run<T, GAP, C>(a.conv, tab, 1, B, lo, hi, red, flip, pre, last);
  } else if constexpr (KIND == EVAL_DOWN) {
    down_block<T, GAP, C>(a.conv, tab, B, lo, hi, Ho, Wo, red, flip, pre, last);
  } else {
    typedef Conv<T, GAP, Mma<T>::KV, 16, 3, 1, 1, 1, 2> K1;
    typedef Conv<T, GAP, Mma<T>::KV, 16, 3, 2, 1, 1, 2> K2;
    typename K1::Wts w;
    K1::load_weights(a.conv[0], w, wave, lane);
    const int RBi = row_bytes(a.W, K1::PIX);
    int ka[K1::KPW];
    K1::addresses(ka, wave, lane, RBi);
    pre();
    __syncthreads();
    K1::load_affine(a.conv[0], tab, w, wave, lane);
    auto put = [&](const f32x4_t& acc, int b, int row, int col, bool ok) __attribute__((always_inline)) {
      float v[4];
      affine<T>(acc, w.sc[b], w.sh[b], v);
      last(v, (lane >> 4) * 4, row, col, 0, ok);
    };
    if (a.stride == 1) {
      K1::pass(B.o, B.row0, RBi, lo, hi, Wo, ka, w, red, flip, wave, lane, put);
    } else {
      typename K2::Wts v2;
#pragma unroll
      for (int k = 0; k < K2::KPW; ++k) v2.w[0][k] = w.w[0][k];
      K2::pass(B.o, B.row0, RBi, lo, hi, Wo, ka, v2, red, flip, wave, lane, put);
    }
  }
}

}  // namespace ev

// LDS of a launch over `kinds`/`chans` (nb blocks) on H x W images with TH output rows per workgroup. (Strips store from the accumulators, so a
// strip of a stem or of a block between stages does not use the region that is counted for its output.)
static void eval_lds(const EvalBlockShape* b, int nb, int H, int W, int TH, int strips, int dtype, int gap, EvalLaunch* l) {
  const size_t esz = dtype_size(dtype);
  auto row = [&](int w, int c) -> size_t { return ev::row_bytes(w, ev::pix_bytes_of(c, (int)esz, gap)); };   // bytes of a row of w pixels
  size_t need[3] = {0, 0, 0};     // regions A, B, C
  int xi = 0, yi = 2;             // which region holds x, which is free
  auto want = [&](int region, size_t bytes) { if (bytes > need[region]) need[region] = bytes; };
  auto rows = [&](int r, int h) -> size_t { return strips > 1 && r < h + 2 ? r : h + 2; };
  bool exch = false;
  size_t tab = 0;                 // scale and shift of every convolution
  int h = H, w = W;
  for (int i = 0; i < nb; ++i) {
    if (b[i].kind == EVAL_STEM) {
      want(1, rows((TH - 1) * b[i].stride + 3, h) * ev::row_bytes(w, 16));
      h = (h - 1) / b[i].stride + 1; w = (w - 1) / b[i].stride + 1;
      want(0, rows(TH + 2, h) * row(w, 16));
      if (nb > 1) want(1, (size_t)(h + 2) * row(w, 16));
    } else if (b[i].kind == EVAL_IDENTITY) {
      want(xi, rows(TH + 4, h) * row(w, b[i].c));
      want(1, rows(TH + 2, h) * row(w, b[i].c));
      if (b[i].c == 64) exch = true;
    } else {
      want(xi, rows((TH + 1) * 2 + 3, h) * row(w, b[i].c));
      h = (h - 1) / 2 + 1; w = (w - 1) / 2 + 1;
      want(1, rows(TH + 2, h) * row(w, 2 * b[i].c));
      want(yi, rows(TH + 2, h) * row(w, 2 * b[i].c));
      int t = xi; xi = yi; yi = t;
      if (2 * b[i].c == 64) exch = true;
    }
  }
  for (int i = 0; i < nb; ++i)
    tab += 8 * (size_t)(b[i].kind == EVAL_STEM ? 16 : b[i].kind == EVAL_IDENTITY ? 2 * b[i].c : 6 * b[i].c);
  l->off1 = (unsigned)need[0];
  l->off2 = (unsigned)(need[0] + need[1]);
  l->red_off = (unsigned)(need[0] + need[1] + need[2]);
  l->tab_off = l->red_off + (exch ? ev::RED_BYTES : 0);
  l->dump_off = l->tab_off + (unsigned)tab;
  l->lds = l->dump_off + ev::DUMP_BYTES;
  l->gap = gap;
}

bool eval_block_ok(int kind, int c) {
  if (kind == EVAL_STEM) return c >= 1 && c <= 4;
  if (kind == EVAL_IDENTITY) return c == 16 || c == 32 || c == 64;
  return kind == EVAL_DOWN && (c == 16 || c == 32);
}

// Estimated time of a bf16 launch of N images, us: 2 for the launch, 0.15 per MB in and out, and per round over 256 compute units
// (registers: one workgroup per unit) 2, 1 per layer, 0.04 per KB of a workgroup's rows in and out, and for every 16 pixels of a
// layer what `per` says, in whole groups of a workgroup's waves. Fitted to 1752 measured evaluations (maps 8 to 64 wide, 1 to 256 images,
// one to three blocks, both pitches, whole images and strips), when a strip's workgroup still fetched what it reads piece by piece. Whole images it meets within 10 % rms;
// strips now take 21 % less than it says in the mean. Over 711 evaluations (the same range, stems, blocks between stages and ResNet-20 too) the cut that
// it chooses takes 1.7 % longer than the best of the four in the mean, more than 10 % longer in 47: whole images in place of strips, the worst 3 blocks
// of 16 channels, 40x40, 64 images, 29 us instead of 20.
static double eval_cost(const EvalBlockShape* b, const EvalLaunch& l, int N) {
  const bool wide = l.gap == 32;
  double layers = 0.0, matrix = 0.0;
  int h = l.H, w = l.W, co = 0;
  for (int i = 0; i < l.count; ++i) {
    const int s = b[i].kind == EVAL_DOWN ? 2 : b[i].stride;
    h = (h - 1) / s + 1; w = (w - 1) / s + 1;
    co = b[i].kind == EVAL_STEM ? 16 : b[i].kind == EVAL_DOWN ? 2 * b[i].c : b[i].c;
    const bool whole = l.strips == 1, square = whole && w == 512 / co && h == w && b[i].kind == EVAL_IDENTITY;
    const double per = co == 16 ? (square ? 0.008 : 0.023) : co == 32 ? (!wide ? 0.050 : whole && h * w <= 256 ? 0.035 : 0.064)
                                : square ? (wide ? 0.19 : 0.30) : wide ? 0.365 : 0.40;
    const double each = co == 32 && !wide ? 1.5 : 1.0;     // (both channel blocks in every wave: twice the weights)
    auto groups = [&](int r) { const int pb = (r * w + 15) / 16, g = co == 64 ? 4 : co == 32 ? 16 : 8; return (pb + g - 1) / g * g; };
    const int th = whole ? h : l.TH, r1 = whole || th + 2 > h ? h : th + 2;
    if (b[i].kind != EVAL_STEM) { layers += each; matrix += groups(r1) * per; }
    layers += each; matrix += groups(th) * per;
  }
  const int s0 = b[0].kind == EVAL_DOWN ? 2 : b[0].stride, cin = b[0].kind == EVAL_STEM ? 3 : b[0].c;
  const double in = 2.0 * l.H * l.W * cin * (l.strips > 1 ? 1.0 + 4.0 / (l.TH * s0) : 1.0), out = 2.0 * h * w * co;
  const double rounds = (double)(((size_t)N * l.strips + 255) / 256);
  return 2.0 + 0.15e-6 * N * (in + out) + rounds * (2.0 + layers + 0.04e-3 * (in + out) / l.strips + matrix);
}

// How a module's blocks are cut into launches: all blocks at once, whole images (bf16, if the buffers fit LDS), or one
// block per launch in strips of the height that minimises
//   rounds over 256 compute units x (2 us + the strip's matrix time, halo rows included)
// (2 us: loads, barriers and epilogues of a block; of 84 fp32 evaluations of one block, 7 to 48 wide, 1 to 256 images, two take more than 5 % longer than
// the best height, of 84 in bf16 22, 3.4 % in the mean). bf16: in either of two pitches, whichever of the four
// eval_cost() finds shortest. us a call, strips of 32 / 16 bytes between pixels, whole images of 32 / 16 (-: does not fit):
//   3 blocks of 32 channels, 28x28, 256 images  59 / 58 / - / 37       3 blocks, 24x24, 256 images  52 / 48 / 34 / 30
//   3 blocks of 64 channels, 14x14, 256 images  59 / 70 / 45 / 56      3 blocks, 14x14, 37 images  30 / 31 / 41 / 52
//   1 block of 16 channels, 48x48: 8 images 6 in strips, 19 whole; 256 images 23, 23      3 blocks, 256 images 69, 44
bool eval_plan(const EvalBlockShape* b, int nb, int N, int H, int W, int dtype, EvalPlan* out) {
  for (int i = 0; i < nb; ++i)
    if (!eval_block_ok(b[i].kind, b[i].c) || (i > 0 && b[i].kind == EVAL_STEM)) return false;
  if (nb < 1 || H * W >= 65536) return false;
  out->launches.clear();
  out->whole = EvalLaunch{};
  auto convs = [&](int lo, int hi) { int c = 0; for (int i = lo; i < hi; ++i) c += b[i].kind == EVAL_STEM ? 1 : b[i].kind == EVAL_IDENTITY ? 2 : 3; return c; };
  double whole_t = 1e30, strips_t = 0.0;
  for (int gap = 32; dtype == BF16 && gap >= 16; gap -= 16) {
    EvalLaunch l{};
    l.first = 0; l.count = nb; l.H = H; l.W = W; l.TH = H; l.strips = 1;
    eval_lds(b, nb, H, W, H, 1, dtype, gap, &l);
    l.conv0 = 0; l.nconv = convs(0, nb);
    if (l.lds > ev::LDS_MAX) continue;
    const double t = eval_cost(b, l, N);
    if (t < whole_t) { whole_t = t; out->whole = l; }
  }
  // matrix-core FLOP per second of one compute unit
  const double rate = dtype == BF16 ? 4.0e12 : 0.5e12;
  int h = H, w = W;
  for (int i = 0; i < nb; ++i) {
    const int s = b[i].kind == EVAL_DOWN ? 2 : (b[i].kind == EVAL_STEM ? b[i].stride : 1);
    const int ho = (h - 1) / s + 1, wo = (w - 1) / s + 1;
    const int co = b[i].kind == EVAL_STEM ? 16 : (b[i].kind == EVAL_DOWN ? 2 * b[i].c : b[i].c);
    const double f2 = 2.0 * 9 * co * co, f1 = b[i].kind == EVAL_STEM ? 0.0 : 2.0 * 9 * co * b[i].c;
    EvalLaunch pick{};
    double pick_t = 1e30;
    for (int gap = dtype == BF16 ? 32 : 16; gap >= 16; gap -= 16) {
      EvalLaunch best{};
      double best_t = 1e30;
      for (int th = 1; th <= ho; ++th) {
        if (th > 8 && th < ho && th % 4 != 0) continue;
        EvalLaunch l{};
        l.first = i; l.count = 1; l.H = h; l.W = w; l.TH = th; l.strips = (ho + th - 1) / th;
        eval_lds(b + i, 1, h, w, th, l.strips, dtype, gap, &l);
        if (l.lds > ev::LDS_MAX) continue;
        // 16-pixel blocks, walked in groups of a workgroup's 8 waves (64 channels: 4 blocks together)
        auto blocks = [&](int r) { const int pb = (r * wo + 15) / 16, g = co == 16 ? 8 : co == 32 ? 4 : dtype == BF16 ? 4 : 1; return (pb + g - 1) / g * g; };
        const int r1 = th + 2 < ho ? th + 2 : ho;
        const double flop = 16.0 * (blocks(r1) * f1 + blocks(th) * f2);   // whole groups of pixel blocks
        const double rounds = ((size_t)N * l.strips + 255) / 256;
        const double t = rounds * (2e-6 + flop / rate);
        if (t < best_t) { best_t = t; best = l; }
      }
      if (best_t >= 1e30) continue;
      const double t = dtype == BF16 ? eval_cost(b + i, best, N) : best_t;
      if (t < pick_t) { pick_t = t; pick = best; }
    }
    if (pick_t >= 1e30) { strips_t = 1e30; break; }
    pick.conv0 = convs(0, i); pick.nconv = convs(i, i + 1);
    out->launches.push_back(pick);
    strips_t += pick_t;
    h = ho; w = wo;
  }
  if (out->whole.count && whole_t <= strips_t) out->launches.assign(1, out->whole);
  return out->whole.count || strips_t < 1e30;
}

namespace ev {
template <typename T, int GAP, int KIND, int C>
static hipError_t strip_run(const StripArgs& a, unsigned grid, size_t lds, hipStream_t s) {
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&eval_strip_kernel<T, GAP, KIND, C>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS_MAX);
  if (attr != hipSuccess) return attr;
  DDG_LAUNCH((eval_strip_kernel<T, GAP, KIND, C>), dim3(grid), dim3(NT), lds, s, a);
  return hipGetLastError();
}
template <typename T, int GAP>
static hipError_t strip_launch(int kind, const StripArgs& a, unsigned grid, size_t lds, hipStream_t s) {
  if (kind == EVAL_STEM) return strip_run<T, GAP, EVAL_STEM, 0>(a, grid, lds, s);
  if (kind == EVAL_DOWN) return a.C == 16 ? strip_run<T, GAP, EVAL_DOWN, 16>(a, grid, lds, s) : strip_run<T, GAP, EVAL_DOWN, 32>(a, grid, lds, s);
  return a.C == 16 ? strip_run<T, GAP, EVAL_IDENTITY, 16>(a, grid, lds, s) : a.C == 32 ? strip_run<T, GAP, EVAL_IDENTITY, 32>(a, grid, lds, s)
                                                                                       : strip_run<T, GAP, EVAL_IDENTITY, 64>(a, grid, lds, s);
}
}

hipError_t eval_blocks_launch(const EvalTables& t, const EvalLaunch& l, const void* in, void* out, int N, int C, int dtype, hipStream_t s) {
  if (!t.dev_blocks || !t.dev_convs || !t.blocks || !t.convs || l.nconv < 1 || N < 1 || l.count < 1 || l.lds > ev::LDS_MAX || (l.strips > 1 && l.count != 1))
    return hipErrorInvalidValue;
  if (l.strips > 1 || dtype == F32) {      // (fp32: always strips, if only one)
    const EvalBlockDesc& b = t.blocks[l.first];
    if (l.count != 1 || l.nconv > 3 || !eval_block_ok(b.kind, C)) return hipErrorInvalidValue;
    if ((size_t)l.H * l.W * C * dtype_size(dtype) >= ((size_t)1 << 31)) return hipErrorInvalidValue;   // 32-bit byte offsets inside an image
    ev::StripArgs a{};
    for (int i = 0; i < l.nconv; ++i) a.conv[i] = t.convs[l.conv0 + i];
    a.in = in; a.out = out; a.H = l.H; a.W = l.W; a.C = C; a.stride = b.stride; a.TH = l.TH; a.strips = l.strips;
    a.off1 = l.off1; a.off2 = l.off2; a.red_off = l.red_off; a.tab_off = l.tab_off;
    const unsigned grid = (unsigned)(N * l.strips);
    return dtype == F32 ? ev::strip_launch<float, 16>(b.kind, a, grid, l.lds, s) : l.gap == 16 ? ev::strip_launch<bf16_t, 16>(b.kind, a, grid, l.lds, s)
                                                                                               : ev::strip_launch<bf16_t, 32>(b.kind, a, grid, l.lds, s);
  }
  ev::Args a{};
  a.blocks = t.dev_blocks + l.first; a.nb = l.count; a.in = in; a.out = out; a.N = N; a.H = l.H; a.W = l.W; a.C = C;
  a.off1 = l.off1; a.off2 = l.off2; a.red_off = l.red_off;
  a.convs = t.dev_convs + l.conv0; a.nconv = l.nconv; a.tab_off = l.tab_off; a.dump_off = l.dump_off;
  typedef void (*Kernel)(ev::Args);
  static const Kernel kernels[2] = {ev::eval_blocks_kernel<bf16_t, 16>, ev::eval_blocks_kernel<bf16_t, 32>};
  const int which = l.gap == 16 ? 0 : 1;
  static bool attr_set[2] = {false, false};
  if (!attr_set[which]) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernels[which]), hipFuncAttributeMaxDynamicSharedMemorySize, (int)ev::LDS_MAX);
    if (e != hipSuccess) return e;
    attr_set[which] = true;
  }
  DDG_LAUNCH(kernels[which], dim3((unsigned)N), dim3(ev::NT), l.lds, s, a);
  return hipGetLastError();
}

}  // namespace ddg
