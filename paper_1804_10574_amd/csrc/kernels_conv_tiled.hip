// 3x3, stride-1, pad-1 convolution (forward and input-gradient) for the CIFAR layer shapes:
// C = Cin = Cout in {16, 32, 64} on feature maps W = 32, 16, 8 wide, bf16 operands.
//
// A workgroup stages the (8+2) x (W+2) halo tile of the input once in LDS (NHWC, pixels and rows
// padded so that the fragment reads have no bank conflicts); the nine taps are
// then shifted LDS addresses: the im2col matrix never exists. While staging, the input can be
// turned into the activation it stands for, a = relu(x*scale + shift) (batch-norm + ReLU of
// the previous layer), so that activation is never written to memory. Zero padding is
// applied after that transform.
//
// Each wave owns 4 pixel-blocks x 1 output-channel block (16x16 MFMA tiles) and keeps its
// slice of the weights in registers for the whole kernel; a workgroup walks over several
// tiles, prefetching the next tile's global loads during the MFMA phase. The epilogue stores
// NHWC, optionally adds a (masked) shortcut gradient, and accumulates batch-norm statistics
// (sum, sum of squares of the stored values) in registers; one partial row per workgroup.
#include "ddg_device.h"
#include "ddg_kernels.h"
#include "ddg_stats.h"
#include "ddg_bn_reduce.h"
#include "ddg_wgrad_tiled.h"
#include <cstdlib>

namespace ddg {

struct ConvTiledArgs {
  const bf16_t* in;        // [N,H,W,C]
  const bf16_t* res;       // optional (RES kernels): input = relu(in*scale+shift + res), same layout
  bf16_t* y_out;           // optional (RES kernels): that input is also stored here (tile rows only)
  const float* scale;      // optional input transform relu(in*scale+shift)
  const float* shift;
  BnRows in_rows;          // in_rows.partial != null: scale/shift come from these partial rows
  const bf16_t* wpack;     // packed operand [ks][C/16][64][8]
  bf16_t* out;             // [N,H,W,C]
  ConvStat st;             // epilogue statistics: partial rows [grid][2][C]
  const bf16_t* add_g;     // optional epilogue term, same layout as out
  const bf16_t* add_mask;  // add_g counts only where add_mask > 0
  // XF_APPLY kernels: `in` is dy, the gradient w.r.t. the ReLU output after a batch norm, and the
  // convolved tensor is dz = A*g + B*bz + C0 with g = dy where bmask*bmscale+bmshift > 0 (bmask
  // null: g = dy); A, B, C0 derive from the partial rows `brows` of that BN's backward sums.
  // dz is formed while staging and also stored to dz_out (tile rows only).
  const bf16_t* bz; const bf16_t* bmask; const float* bmscale; const float* bmshift;
  BnBwdRows brows; bf16_t* dz_out;
  int N, H;                // N counts the images of all groups
  int tiles;               // N * H/8
  ImgOf img;               // tile -> image
  // groups 2: the batch is two independent minibatches laid end to end (batch-norm
  // statistics are per minibatch). A workgroup works on one group only: workgroups
  // [g*grid/groups, (g+1)*grid/groups) take group g, write that group's statistics rows
  // (rows are indexed by workgroup), and use that group's input transform: in_rows.partial and
  // st.partial advance by rows*2*C per group, the per-channel vectors by vec_stride floats.
  int groups;
  int vec_stride;
};

template <int C, int W>
struct ConvTiledCfg {
  static constexpr int TH = 8, ROWS = TH + 2, WC = W + 2;
  // Bytes per staged pixel and per tile row. A 16-byte fragment read takes 4 cycles if the 16 lanes it serves together
  // (0-3, 12-15, 20-27, and so on) touch 16 different 16-byte groups of 256 bytes, else 8 or 12. Pixels an odd multiple of 32
  // bytes apart do that; where a block of 16 pixels spans two rows (8 wide), the rows have to be a multiple of 256 apart too.
  static constexpr int PIX = C == 16 ? 32 : C * 2 + 32;
  static constexpr int ROWB = W == 8 ? (WC * PIX + 255) / 256 * 256 : WC * PIX;
  static constexpr int TILE_BYTES = ROWS * ROWB, LDS_BYTES = TILE_BYTES + 16;
  static constexpr int CH = C / 8;                       // 16-byte chunks per pixel
  static constexpr int NCHUNK = ROWS * WC * CH;          // chunks per tile (halo columns included)
  static constexpr int PER_THREAD = (NCHUNK + 255) / 256;
  static constexpr int KSTEPS = (9 * C + 31) / 32;
  static constexpr int PG = W / 8;                       // waves along the pixel dimension
  static constexpr int COB = C / 16;
};

// Waves per SIMD the register allocation aims for (more co-resident workgroups when several
// streams run): the largest value each variant reaches without spilling.
// What staging does to the loaded input: nothing or relu(in*scale+shift) (decided at run time),
// the residual-block output relu(in*scale+shift + res), or the batch-norm backward formula
// (XF_APPLY: the ReLU mask is the BN's own conv output bz; XF_APPLY_MASK: a separate tensor).
enum { XF_PLAIN = 0, XF_RES = 1, XF_APPLY = 2, XF_APPLY_MASK = 3 };

constexpr int conv_tiled_waves(int C, int MODE, int XF) {
  return C == 64 ? (MODE == 2 && XF >= XF_APPLY ? 1 : 2)
                 : (((C == 32 && (XF != XF_PLAIN || MODE == 2)) || (C == 16 && XF >= XF_APPLY && MODE == 2)) ? 2 : 3);
}

// MODE is the epilogue's statistics mode, fixed at compile time: 0 none, 1 sum / sum of squares
// of the stored output (forward), 2 the BN-backward sums of the layer below (input gradient).
//
// Instruction count matters as much as bytes here (a wave64 VALU instruction occupies its SIMD
// for four cycles, and these kernels run a few microseconds): the staging map of a thread is
// computed once, LDS fragment addresses are one per-lane register per k-step plus an
// instruction immediate per pixel block, fragment reads are unconditional 16-byte reads, the
// tensors the epilogue needs are requested before the MFMA phase, and fp32 -> bf16 uses the
// packed hardware conversion.
// RES: the input is the output of the residual block before, y = relu(in*scale+shift + res),
// formed while staging and written to y_out by the workgroup that owns the rows.
// bidx of gdim: this workgroup's index in the launch (or in the part of a launch this work has).
template <int C, int W, int MODE, int XF>
__device__ __forceinline__ void conv3x3_tiled_body(const ConvTiledArgs& a, unsigned char* tile, int bidx, int gdim) {
  using Cfg = ConvTiledCfg<C, W>;
  constexpr bool RES = XF == XF_RES, APPLY = XF == XF_APPLY || XF == XF_APPLY_MASK;
  constexpr int TH = Cfg::TH, WC = Cfg::WC, PIX = Cfg::PIX, ROWB = Cfg::ROWB, CH = Cfg::CH, NCHUNK = Cfg::NCHUNK;
  constexpr int PT = Cfg::PER_THREAD, KSTEPS = Cfg::KSTEPS, PG = Cfg::PG, COB = Cfg::COB;
  constexpr bool RAGGED_K = (9 * C) % 32 != 0;   // the last k-step runs past tap 8 for some lanes

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, lg = lane >> 4;
  const int pgrp = wave % PG, cb = wave / PG;
  // this workgroup's group (one of at most two), its index among the group's workgroups, the group's tile range
  const int g1 = gdim >> (a.groups - 1);
  const int grp = bidx >= g1 ? 1 : 0, bl = bidx - grp * g1;
  const int tiles_g = a.tiles >> (a.groups - 1), t_end = (grp + 1) * tiles_g;

  // what the on-load transform waits for is requested before everything else
  BnFwdRows<C> fwd;
  BnBwdFromRows<C> bwd;
  BnRows in_rows = a.in_rows;
  float bms = 1.f, bmh = 0.f;
  const int vo = grp * a.vec_stride;
  if (APPLY) {
    bwd.request(a.brows);
    if (a.bmscale && tid < C) { bms = a.bmscale[tid]; bmh = a.bmshift[tid]; }
  } else if (in_rows.partial) {
    in_rows.partial += (size_t)grp * in_rows.rows * 2 * C;
    in_rows.mean += vo; in_rows.invstd += vo; in_rows.scale += vo; in_rows.shift += vo;
    fwd.request(in_rows);
  } else if (a.scale && tid < C) {
    bms = a.scale[vo + tid]; bmh = a.shift[vo + tid];
  }

  float below[4] = {0.f, 1.f, 1.f, 0.f};   // mode 2: constants of the BN below (mean, invstd, mask scale, mask shift)
  if (MODE == 2 && tid < C) {
    below[0] = a.st.zmean[tid]; below[1] = a.st.zinvstd[tid];
    if (a.st.mscale) { below[2] = a.st.mscale[tid]; below[3] = a.st.mshift[tid]; }
  }

  // ---- staging map (the same for every tile): chunk v = tid + i*256 -> halo pixel, 8 channels
  const int my_ch = tid % CH;
  unsigned goff[PT];   // byte offset of the chunk from column 0 of the tile's first halo row
  unsigned out = 0;    // 3 bits per chunk: in the first / the last halo row, in a pad column (or no chunk)
  unsigned own = 0;    // bit i: chunk i lies in the tile's own rows, which this workgroup stores
  int loff[PT];        // LDS byte offset (no chunk: behind the tile)
#pragma unroll
  for (int i = 0; i < PT; ++i) {
    const int v = tid + i * 256;
    const int px = v / CH;
    const int rr = px / WC, cc = px - rr * WC;
    const bool col_ok = v < NCHUNK && cc >= 1 && cc <= W;
    out |= ((rr == 0 ? 1u : 0u) | (rr == TH + 1 ? 2u : 0u) | (col_ok ? 0u : 4u)) << (3 * i);
    own |= (col_ok && rr >= 1 && rr <= TH ? 1u : 0u) << i;
    goff[i] = (unsigned)((rr * W + cc - 1) * C + my_ch * 8) * 2;
    loff[i] = v < NCHUNK ? rr * ROWB + cc * PIX + my_ch * 16 : Cfg::TILE_BYTES;
  }
  uint4 stage[PT], stage2[(RES || APPLY) ? PT : 1], stage3[XF == XF_APPLY_MASK ? PT : 1];
  // element offset of column 0 of tile t's first halo row (it may lie before the tensor, where nothing is loaded), and which
  // chunks of it lie outside the image
  auto tile_at = [&](int t, unsigned& outside) {
    const int n = a.img.of(t), r0 = (t - n * a.img.d) * TH;
    outside = 4u | (r0 == 0 ? 1u : 0u) | (r0 + TH == a.H ? 2u : 0u);
    return ((ptrdiff_t)(n * a.H + r0) - 1) * (W * C);
  };
  auto resource = [&](const bf16_t* p, ptrdiff_t at, bool any = true) { return wide_rsrc(p + at, any ? (TH + 2) * W * C * 2 : 0); };
  auto issue_loads = [&](int t) {     // (a tile past the last: loads that fetch nothing, so that their number is the same)
    unsigned outside;
    const ptrdiff_t at = tile_at(t, outside);
    const bool any = t < t_end;
    const wide_rsrc_t r1 = resource(a.in, at, any);
    const wide_rsrc_t r2 = resource(RES ? a.res : APPLY ? a.bz : a.in, at, any), r3 = resource(XF == XF_APPLY_MASK ? a.bmask : a.in, at, any);
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      const unsigned o = (out & (outside << (3 * i))) ? NOWHERE : goff[i];
      stage[i] = __builtin_bit_cast(uint4, wide_load(r1, o, 0));
      if (RES || APPLY) stage2[i] = __builtin_bit_cast(uint4, wide_load(r2, o, 0));
      if (XF == XF_APPLY_MASK) stage3[i] = __builtin_bit_cast(uint4, wide_load(r3, o, 0));
    }
  };
  // ---- this wave's weights: KSTEPS fragments of its output-channel block (before the tile: with the tile they have arrived too,
  // so the loop never waits for them)
  uint4 wf[KSTEPS];
#pragma unroll
  for (int ks = 0; ks < KSTEPS; ++ks)
    wf[ks] = *reinterpret_cast<const uint4*>(a.wpack + ((size_t)(ks * COB + cb) * 64 + lane) * 8);

  int t = grp * tiles_g + bl;
  issue_loads(t);

  // ---- LDS fragment addresses: lane part + k-step part in a register, pixel block as immediate
  // pixel of block i, lane l16: pt = (pgrp*4 + i)*16 + l16; its row/column split is additive in i
  const int ptl = pgrp * 64 + l16;
  const int lane_base = (ptl / W) * ROWB + (ptl % W) * PIX;
  int kaddr[KSTEPS];
  bool klast_ok = true;
#pragma unroll
  for (int ks = 0; ks < KSTEPS; ++ks) {
    const int kidx = (ks * 4 + lg) * 8;
    const int tap = kidx / C, c0 = kidx % C;
    const bool ok = tap < 9;
    if (ks == KSTEPS - 1) klast_ok = ok;
    const int tp = ok ? tap : 0;
    kaddr[ks] = lane_base + (tp / 3) * ROWB + (tp % 3) * PIX + c0 * 2;
  }

  // ---- per-channel transform of the input (while the first tile's loads are in flight); the
  // vectors stay in LDS and a thread reads its 8 channels when it stages (registers are scarce)
  const bool xform = !APPLY && (a.scale != nullptr || a.in_rows.partial != nullptr);
  __shared__ __align__(16) float s_sc[APPLY ? 4 : C], s_sh[APPLY ? 4 : C];
  // XF_APPLY: A, B, C0 of the formula, then the mask's scale and shift
  __shared__ __align__(16) float s_coef[APPLY ? 5 * C : 4];
  if (APPLY) {
    if (tid < C) { s_coef[3 * C + tid] = bms; s_coef[4 * C + tid] = bmh; }
    bwd.finish(a.brows, s_coef, bidx == 0);   // ends with a barrier
  } else if (in_rows.partial) {
    fwd.finish(in_rows, s_sc, s_sh, bl == 0);
  } else if (a.scale) {
    if (tid < C) { s_sc[tid] = bms; s_sh[tid] = bmh; }
    __syncthreads();
  }
  auto write_stage = [&](int t) {
    unsigned outside;
    const ptrdiff_t at = tile_at(t, outside);
    auto ld8 = [&](const float* p, float (&d)[8]) {
      *reinterpret_cast<float4*>(&d[0]) = *reinterpret_cast<const float4*>(p + my_ch * 8);
      *reinterpret_cast<float4*>(&d[4]) = *reinterpret_cast<const float4*>(p + my_ch * 8 + 4);
    };
    float k0[8], k1[8], k2[8], m0[8], m1[8];      // this thread's channels: A, B, C0, the mask's scale and shift; or scale and shift
    wide_rsrc_t ro;
    if (APPLY) {
      ld8(&s_coef[0], k0); ld8(&s_coef[C], k1); ld8(&s_coef[2 * C], k2);
      if (C != 64) { ld8(&s_coef[3 * C], m0); ld8(&s_coef[4 * C], m1); }   // (64 channels: no registers for these)
      ro = resource(a.dz_out, at);
    } else if (xform) {
      ld8(s_sc, k0); ld8(s_sh, k1);
      if (RES) ro = a.y_out ? resource(a.y_out, at) : wide_rsrc(nullptr, 0);
    }
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      uint4 q = stage[i];
      if (APPLY || xform) {
        float g[8], zz[8];
        Store<bf16_t>::unpack_vec(q, g);
        if (APPLY) {
          Store<bf16_t>::unpack_vec(stage2[i], zz);
          if (a.bmask) {
            float mk[8];
            Store<bf16_t>::unpack_vec(XF == XF_APPLY_MASK ? stage3[i] : stage2[i], mk);
            if (C == 64) { ld8(&s_coef[3 * C], m0); ld8(&s_coef[4 * C], m1); }
#pragma unroll
            for (int j = 0; j < 8; ++j) g[j] = (mk[j] * m0[j] + m1[j]) > 0.f ? g[j] : 0.f;
          }
#pragma unroll
          for (int j = 0; j < 8; ++j) g[j] = k0[j] * g[j] + (k1[j] * zz[j] + k2[j]);
        } else {
          if (RES) Store<bf16_t>::unpack_vec(stage2[i], zz);
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            g[j] = g[j] * k0[j] + k1[j];
            if (RES) g[j] += zz[j];
            g[j] = fmaxf(g[j], 0.f);
          }
        }
        // zero padding comes after the transform
        const bool in = !(out & (outside << (3 * i)));
        q.x = in ? Store<bf16_t>::pack2(g[0], g[1]) : 0u; q.y = in ? Store<bf16_t>::pack2(g[2], g[3]) : 0u;
        q.z = in ? Store<bf16_t>::pack2(g[4], g[5]) : 0u; q.w = in ? Store<bf16_t>::pack2(g[6], g[7]) : 0u;
        if (APPLY || RES) wide_store(ro, q, (own >> i) & 1u ? goff[i] : NOWHERE);
      }
      *reinterpret_cast<uint4*>(tile + loff[i]) = q;
    }
  };

  float ssum[4] = {0.f, 0.f, 0.f, 0.f}, ssq[4] = {0.f, 0.f, 0.f, 0.f};
  // mode 2: per-channel constants of the BN below (mean, invstd, mask scale, mask shift) in LDS;
  // a lane reads those of its 4 channels in the epilogue
  __shared__ __align__(16) float s_below[MODE == 2 ? 4 * C : 4];
  const bf16_t* st_mask = reinterpret_cast<const bf16_t*>(a.st.mask);
  const bf16_t* st_z = reinterpret_cast<const bf16_t*>(a.st.z);
  const bool two_tensors = MODE == 2 && st_z != st_mask;
  const bool add = MODE != 1 && a.add_g != nullptr;   // (a shortcut gradient is added to gradients only)
  if (MODE == 2) {
    if (tid < C) { s_below[tid] = below[0]; s_below[C + tid] = below[1]; s_below[2 * C + tid] = below[2]; s_below[3 * C + tid] = below[3]; }
    // (made visible by the barriers of the tile loop before any epilogue runs)
  }
  // (the weights' wait, which comes before the first tile's: inside the loop it would be one for all loads in flight, every time)
#pragma unroll
  for (int ks = 0; ks < KSTEPS; ++ks) asm volatile("" : "+v"(wf[ks].x), "+v"(wf[ks].y), "+v"(wf[ks].z), "+v"(wf[ks].w));
  // output element offset of (block 0, this lane) inside a tile; block i adds i*16*C
  const int out_lane = ptl * C + cb * 16 + lg * 4;

  for (; t < t_end; t += g1) {
    __syncthreads();            // the previous tile has been consumed
    write_stage(t);
    __syncthreads();
    // what the epilogue reads, requested now, and before the next tile: loads return in order, so behind that tile's they were there no
    // sooner than it was (ResNet-110, batch 256: 29.07 -> 28.88 ms per 16 iterations, ResNet-56, batch 128: 10.61 -> 10.54; requested a tile ahead,
    // beside the tile's own loads: 29.29 and 10.76)
    const int n = a.img.of(t), r0 = (t - n * a.img.d) * TH;
    const unsigned obase = (unsigned)((n * a.H + r0) * W) * C + out_lane;
    uint2 eg[4], em[4], ek[4], ez[4];
    if (add) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        eg[i] = *reinterpret_cast<const uint2*>(a.add_g + obase + i * 16 * C);
        if (a.add_mask) em[i] = *reinterpret_cast<const uint2*>(a.add_mask + obase + i * 16 * C);
      }
    }
    if (MODE == 2) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        ek[i] = *reinterpret_cast<const uint2*>(st_mask + obase + i * 16 * C);
        if (two_tensors) ez[i] = *reinterpret_cast<const uint2*>(st_z + obase + i * 16 * C);
      }
    }

    issue_loads(t + g1);               // in flight during the MFMA phase

    f32x4_t acc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) {
      const unsigned char* kp = tile + kaddr[ks];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int blk = ((i * 16) / W) * ROWB + ((i * 16) % W) * PIX;   // constant after unrolling
        uint4 af = *reinterpret_cast<const uint4*>(kp + blk);
        if (RAGGED_K && ks == KSTEPS - 1 && !klast_ok) af = make_uint4(0, 0, 0, 0);
        acc[i] = Mma<bf16_t>::mma(wf[ks], af, acc[i]);
      }
    }

    // epilogue: lane = pixel l16 of block i, channels cb*16 + lg*4 .. +3
    auto lo = [](uint32_t u) { return __uint_as_float(u << 16); };
    auto hi = [](uint32_t u) { return __uint_as_float(u & 0xffff0000u); };
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float v[4] = {acc[i][0], acc[i][1], acc[i][2], acc[i][3]};
      if (add) {
        float g[4] = {lo(eg[i].x), hi(eg[i].x), lo(eg[i].y), hi(eg[i].y)};
        if (a.add_mask) {
          const float mk[4] = {lo(em[i].x), hi(em[i].x), lo(em[i].y), hi(em[i].y)};
#pragma unroll
          for (int j = 0; j < 4; ++j) g[j] = (mk[j] > 0.f) ? g[j] : 0.f;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] += g[j];
      }
      uint2 o;
      o.x = Store<bf16_t>::pack2(v[0], v[1]); o.y = Store<bf16_t>::pack2(v[2], v[3]);
      float bmu[4], bis[4], zz[4];
      if (MODE == 2) {
        // the gradient leaves this kernel already multiplied by the ReLU mask of the layer below
        // (every reader of it applies that mask first, so it is applied once, here)
        const float mk[4] = {lo(ek[i].x), hi(ek[i].x), lo(ek[i].y), hi(ek[i].y)};
        const int cq = cb * 16 + lg * 4;
        const float4 bmu4 = *reinterpret_cast<const float4*>(&s_below[cq]);
        const float4 bis4 = *reinterpret_cast<const float4*>(&s_below[C + cq]);
        const float4 bms4 = *reinterpret_cast<const float4*>(&s_below[2 * C + cq]);
        const float4 bmh4 = *reinterpret_cast<const float4*>(&s_below[3 * C + cq]);
        bmu[0] = bmu4.x; bmu[1] = bmu4.y; bmu[2] = bmu4.z; bmu[3] = bmu4.w;
        bis[0] = bis4.x; bis[1] = bis4.y; bis[2] = bis4.z; bis[3] = bis4.w;
        const float bms[4] = {bms4.x, bms4.y, bms4.z, bms4.w}, bmh[4] = {bmh4.x, bmh4.y, bmh4.z, bmh4.w};
        if (two_tensors) { zz[0] = lo(ez[i].x); zz[1] = hi(ez[i].x); zz[2] = lo(ez[i].y); zz[3] = hi(ez[i].y); }
        else { zz[0] = mk[0]; zz[1] = mk[1]; zz[2] = mk[2]; zz[3] = mk[3]; }
        const uint32_t k0 = (mk[0] * bms[0] + bmh[0]) > 0.f ? 0x0000ffffu : 0u;
        const uint32_t k1 = (mk[1] * bms[1] + bmh[1]) > 0.f ? 0xffff0000u : 0u;
        const uint32_t k2 = (mk[2] * bms[2] + bmh[2]) > 0.f ? 0x0000ffffu : 0u;
        const uint32_t k3 = (mk[3] * bms[3] + bmh[3]) > 0.f ? 0xffff0000u : 0u;
        o.x &= k0 | k1; o.y &= k2 | k3;
      }
      *reinterpret_cast<uint2*>(a.out + obase + i * 16 * C) = o;
      if (MODE != 0) {
        const float r[4] = {lo(o.x), hi(o.x), lo(o.y), hi(o.y)};   // the values as stored
        if (MODE == 1) {
#pragma unroll
          for (int j = 0; j < 4; ++j) { ssum[j] += r[j]; ssq[j] += r[j] * r[j]; }
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            ssum[j] += r[j];
            ssq[j] += r[j] * ((zz[j] - bmu[j]) * bis[j]);
          }
        }
      }
    }
  }

  if (MODE != 0) {
    // channel cb*16 + lg*4 + j: sum over the 16 pixel lanes, then over the PG waves of this cb
    __shared__ float red[4][2][16];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float s1 = row_sum16(ssum[j]), s2 = row_sum16(ssq[j]);
      if (l16 == 0) { red[wave][0][lg * 4 + j] = s1; red[wave][1][lg * 4 + j] = s2; }
    }
    __syncthreads();
    if (tid < 2 * C) {
      const int which = tid / C, c = tid % C;
      const int cbb = c / 16, cl = c % 16;
      float s = 0.f;
#pragma unroll
      for (int g = 0; g < PG; ++g) s += red[cbb * PG + g][which][cl];
      a.st.partial[((size_t)bidx * 2 + which) * C + c] = s;
    }
  }
}

template <int C, int W, int MODE, int XF = XF_PLAIN>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(conv_tiled_waves(C, MODE, XF)))) void conv3x3_tiled_kernel(ConvTiledArgs a) {
  extern __shared__ __align__(16) unsigned char tile[];
  conv3x3_tiled_body<C, W, MODE, XF>(a, tile, blockIdx.x, gridDim.x);
}

// Two independent pieces of backward work of one shape in one launch (a launch costs a few
// microseconds of dispatch whatever it carries): the first conv_grid workgroups run the
// input-gradient kernel of a unit (which forms its dz while staging), the others the plain weight
// gradient of the unit above it, whose dz the launch before has stored.
template <int C, int W, int MODE, int XF>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(conv_tiled_waves(C, MODE, XF)))) void bwd_pair_kernel(ConvTiledArgs ca, WgradTiledArgs wa, int conv_grid, int wg_rows) {
  extern __shared__ __align__(16) unsigned char tile[];
  const int b = blockIdx.x;
  if (b < conv_grid) {
    conv3x3_tiled_body<C, W, MODE, XF>(ca, tile, b, conv_grid);
  } else {
    const int v = b - conv_grid;
    wgrad_tiled_body<C, C, W, false>(wa, tile, v % wg_rows, v / wg_rows, wg_rows);
  }
}

// The input gradient of the second layer of a stage's first block: beside it the sums of the block's projection, which wait for
// the same gradient, and the plain weight gradient of the unit above.
template <int C, int W, int XF>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(conv_tiled_waves(C, 2, XF)))) void bwd_down_kernel(ConvTiledArgs ca, WgradTiledArgs wa, BnReduceRide rd, int conv_grid, int wg_rows, int wg_blocks) {
  extern __shared__ __align__(16) unsigned char tile[];
  const int b = blockIdx.x;
  if (b < conv_grid) {
    conv3x3_tiled_body<C, W, 2, XF>(ca, tile, b, conv_grid);
  } else if (b < conv_grid + wg_blocks) {
    const int v = b - conv_grid;
    wgrad_tiled_body<C, C, W, false>(wa, tile, v % wg_rows, v / wg_rows, wg_rows);
  } else {
    bn_bwd_reduce_body<bf16_t>(rd.q, rd.elems / 8, C, b - conv_grid - wg_blocks, rd.grid);
  }
}

// Workgroups per launch for a layer with C channels (and so the number of partial statistics
// rows the launch writes). Every workgroup loads its wave's weights and adds up the rows of the
// layer before, so on the small feature maps fewer, longer-running workgroups mean less L2
// traffic. DDG_TUNE_CONV_GRID_C16/_C32/_C64 override the defaults within [32, 2048].
static int conv_tiled_cap(int C) {
  int cap = C == 16 ? 256 : (C == 32 ? 128 : 96);   // (measured: c64 flat between 64 and 96, worse at 48 and at 128+)
  const char* name = C == 16 ? "DDG_TUNE_CONV_GRID_C16" : (C == 32 ? "DDG_TUNE_CONV_GRID_C32" : "DDG_TUNE_CONV_GRID_C64");
  if (const char* e = getenv(name)) {
    const int v = atoi(e);
    if (v >= 32 && v <= 2048) cap = v;
  }
  return cap;
}

// No launch uses more workgroups than this (sizes row buffers).
int conv_tiled_max_grid() {
  int m = conv_tiled_cap(16);
  if (conv_tiled_cap(32) > m) m = conv_tiled_cap(32);
  if (conv_tiled_cap(64) > m) m = conv_tiled_cap(64);
  return m;
}

int conv_tiled_grid(int N, int H, int W, int Cin, int Cout, int R, int stride, int dtype) {
  if (dtype == F32) return conv_tiled_f32_grid(N, H, W, Cin, Cout, R, stride);
  if (dtype != BF16 || R != 3 || stride != 1 || Cin != Cout) return 0;
  if (!((Cin == 16 && W == 32) || (Cin == 32 && W == 16) || (Cin == 64 && W == 8))) return 0;
  if (H % 8 != 0) return 0;
  const int tiles = N * (H / 8);
  const int cap = conv_tiled_cap(Cin);
  return tiles < cap ? tiles : cap;
}

template <int C, int W>
static hipError_t conv_tiled_launch_t(const ConvTiledArgs& a, int grid, hipStream_t s, const WgradTiledArgs* wa, int wg_rows, const BnReduceRide* ride) {
  using Cfg = ConvTiledCfg<C, W>;
  if (ride) {
    using WCfg = WgradTiledCfg<C, C, W>;
    if (!wa || !a.bz || a.st.mode != 2 || a.scale || a.in_rows.partial || !a.brows.partial || !a.dz_out || C == 16 || ride->C != C || ride->grid < 1)
      return hipErrorInvalidValue;
    constexpr int lds = Cfg::LDS_BYTES > WCfg::LDS ? Cfg::LDS_BYTES : WCfg::LDS;
    if constexpr (C != 16) {
      const int wgb = wg_rows * WCfg::OT;
      const dim3 g(grid + wgb + ride->grid);
      if (a.bmask && a.bmask != a.bz) DDG_LAUNCH((bwd_down_kernel<C, W, XF_APPLY_MASK>), g, dim3(256), lds, s, a, *wa, *ride, grid, wg_rows, wgb);
      else DDG_LAUNCH((bwd_down_kernel<C, W, XF_APPLY>), g, dim3(256), lds, s, a, *wa, *ride, grid, wg_rows, wgb);
    }
    return hipGetLastError();
  }
  if (wa) {
    using WCfg = WgradTiledCfg<C, C, W>;
    if (!a.bz || a.st.mode == 1 || a.scale || a.in_rows.partial || !a.brows.partial || !a.dz_out || wg_rows < 1)
      return hipErrorInvalidValue;
    constexpr int lds = Cfg::LDS_BYTES > WCfg::LDS ? Cfg::LDS_BYTES : WCfg::LDS;
    static_assert(lds <= 48 * 1024, "dynamic LDS within the default limit");
    const bool own_mask = a.bmask && a.bmask != a.bz;
    const dim3 g(grid + wg_rows * WCfg::OT);
    if (a.st.mode == 2) {
      if (own_mask) DDG_LAUNCH((bwd_pair_kernel<C, W, 2, XF_APPLY_MASK>), g, dim3(256), lds, s, a, *wa, grid, wg_rows);
      else DDG_LAUNCH((bwd_pair_kernel<C, W, 2, XF_APPLY>), g, dim3(256), lds, s, a, *wa, grid, wg_rows);
    } else {
      if (own_mask) DDG_LAUNCH((bwd_pair_kernel<C, W, 0, XF_APPLY_MASK>), g, dim3(256), lds, s, a, *wa, grid, wg_rows);
      else DDG_LAUNCH((bwd_pair_kernel<C, W, 0, XF_APPLY>), g, dim3(256), lds, s, a, *wa, grid, wg_rows);
    }
    return hipGetLastError();
  }
  if (a.res) {
    if (a.st.mode != 1 || !(a.scale || a.in_rows.partial)) return hipErrorInvalidValue;
    DDG_LAUNCH((conv3x3_tiled_kernel<C, W, 1, XF_RES>), dim3(grid), dim3(256), Cfg::LDS_BYTES, s, a);
  } else if (a.bz) {
    // input-gradient kernel that applies the batch-norm backward formula to its input
    if (a.st.mode == 1 || a.scale || a.in_rows.partial || !a.brows.partial || !a.dz_out) return hipErrorInvalidValue;
    const bool own_mask = a.bmask && a.bmask != a.bz;
    if (a.st.mode == 2) {
      if (own_mask) DDG_LAUNCH((conv3x3_tiled_kernel<C, W, 2, XF_APPLY_MASK>), dim3(grid), dim3(256), Cfg::LDS_BYTES, s, a);
      else DDG_LAUNCH((conv3x3_tiled_kernel<C, W, 2, XF_APPLY>), dim3(grid), dim3(256), Cfg::LDS_BYTES, s, a);
    } else {
      if (own_mask) DDG_LAUNCH((conv3x3_tiled_kernel<C, W, 0, XF_APPLY_MASK>), dim3(grid), dim3(256), Cfg::LDS_BYTES, s, a);
      else DDG_LAUNCH((conv3x3_tiled_kernel<C, W, 0, XF_APPLY>), dim3(grid), dim3(256), Cfg::LDS_BYTES, s, a);
    }
  } else if (a.st.mode == 1) DDG_LAUNCH((conv3x3_tiled_kernel<C, W, 1>), dim3(grid), dim3(256), Cfg::LDS_BYTES, s, a);
  else if (a.st.mode == 2) DDG_LAUNCH((conv3x3_tiled_kernel<C, W, 2>), dim3(grid), dim3(256), Cfg::LDS_BYTES, s, a);
  else DDG_LAUNCH((conv3x3_tiled_kernel<C, W, 0>), dim3(grid), dim3(256), Cfg::LDS_BYTES, s, a);
  return hipGetLastError();
}

hipError_t conv_tiled_launch(const void* in, const float* scale, const float* shift, const BnRows* in_rows,
                             const void* wpack, void* out, const ConvStat& st, const void* add_g,
                             const void* add_mask, int N, int H, int W, int C, int grid, hipStream_t s,
                             const void* res, void* y_out, int groups, int vec_stride, const WgradFuse* apply,
                             const WgradPair* pair, const BnReduceRide* ride) {
  if (groups < 1 || N % groups != 0 || grid % groups != 0) return hipErrorInvalidValue;
  if (groups > 2 || (groups > 1 && st.mode != 1) || (st.mode == 1 && add_g)) return hipErrorInvalidValue;   // two groups: forward only
  ConvTiledArgs a{};
  if (apply) {
    if (groups != 1 || res || !apply->rows) return hipErrorInvalidValue;
    if (apply->dy != in) return hipErrorInvalidValue;   // the gradient is the conv input
    a.bz = (const bf16_t*)apply->z; a.bmask = (const bf16_t*)apply->mask; a.bmscale = apply->mscale;
    a.bmshift = apply->mshift; a.brows = *apply->rows; a.dz_out = (bf16_t*)apply->dz_out;
  }
  a.groups = groups; a.vec_stride = vec_stride;
  a.in = (const bf16_t*)in; a.scale = scale; a.shift = shift; a.wpack = (const bf16_t*)wpack;
  a.res = (const bf16_t*)res; a.y_out = (bf16_t*)y_out;
  if (in_rows) a.in_rows = *in_rows; else a.in_rows = BnRows{};
  a.out = (bf16_t*)out; a.st = st; a.add_g = (const bf16_t*)add_g;
  a.add_mask = (const bf16_t*)add_mask; a.N = N; a.H = H; a.tiles = N * (H / 8); a.img = ImgOf::make(H / 8, a.tiles);
  if ((size_t)N * H * W * C >= ((size_t)1 << 31)) return hipErrorInvalidValue;   // 32-bit element offsets inside
  WgradTiledArgs wa{};
  if (pair) {
    if (!apply || pair->rows < 1 || pair->rows > N * (H / 8)) return hipErrorInvalidValue;
    wa.x = (const bf16_t*)pair->x; wa.scale = pair->scale; wa.shift = pair->shift; wa.dz = (const bf16_t*)pair->dz;
    wa.partial = pair->partial; wa.N = N; wa.H = H; wa.W = W; wa.tiles = N * (H / 8);
  }
  const WgradTiledArgs* wp = pair ? &wa : nullptr;
  const int wr = pair ? pair->rows : 0;
  if (C == 16 && W == 32) return conv_tiled_launch_t<16, 32>(a, grid, s, wp, wr, ride);
  if (C == 32 && W == 16) return conv_tiled_launch_t<32, 16>(a, grid, s, wp, wr, ride);
  if (C == 64 && W == 8) return conv_tiled_launch_t<64, 8>(a, grid, s, wp, wr, ride);
  return hipErrorInvalidValue;
}

}  // namespace ddg
