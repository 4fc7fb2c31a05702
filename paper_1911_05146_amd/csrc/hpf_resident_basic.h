// Where an image of a run of basic blocks lies: in the registers of the eight waves of a work-group and on a canvas in LDS
// (kernels_resident_basic.hip), and the 3x3 convolutions that read a canvas.
#pragma once
#include <type_traits>

#include "hpf_resident_reg.h"

namespace hpf {
namespace {

template <int C>
struct Geo {
  static constexpr int NC = C, IMG = C == 16 ? 32 : C == 32 ? 16 : 8, P = IMG * IMG;
  static constexpr int CG = C == 64 ? 2 : 1, NPW = RG_NW / CG;          // waves per tile, waves along the pixels
  static constexpr int PTW = P / 16 / NPW, NTW = C / 16 / CG;           // pixel tiles and channel tiles per wave
  static constexpr int CW = IMG + 2, MS = C + 8;                        // canvas row and pixel pitch (elements)
  static constexpr int NPX = PTW * 16;
  // tile j of a wave in the canvas, from its first one
  static constexpr int tile_off(int j) { return C == 16 ? ((j >> 1) * CW + (j & 1) * 16) * MS : j * CW * MS; }
  using W = WStage<C, (9 * C + 31) / 32 * 32>;
  static constexpr int CANVAS = CW * CW * MS * 2;                       // bytes
};

// 3x3 convolution from the canvas.  src: tap (0, 0) of the lane's pixel of the wave's first tile (+ fk; 16 channels: + (fq & 1)*8); FLIP: the
// data gradient (taps mirrored).  w: the staged matrix at the wave's first channel tile, + lane*8.  zero: eight zeros (of the border).
// third(integral_constant 0 ... 2) runs at the start, after one and after two thirds of the contraction: the next matrix' loads.
template <int C, bool FLIP, class THIRD>
__device__ __forceinline__ void conv3x3(const bf16_t* src, const bf16_t* zero, const bf16_t* w, int fq, floatx4 (&acc)[Geo<C>::PTW][Geo<C>::NTW], THIRD&& third) {
  auto thirds = [&](int i) {
    if (i == 0) third(std::integral_constant<int, 0>{});
    else if (i == 1) third(std::integral_constant<int, 1>{});
    else third(std::integral_constant<int, 2>{});
  };
  using G = Geo<C>;
  constexpr int MS = G::MS, CW = G::CW;
  if constexpr (C == 16) {   // packed weights [16][160], k = tap*16 + c, zero beyond tap 8: lane groups 0-1 take the even tap of a step, 2-3 the odd one.
    // The odd half of the last step has no tap: zeros, not another tap's values times the zero weights (0 * infinity)
#pragma unroll
    for (int st = 0; st < 5; ++st) {
      if (st % 2 == 0) thirds(st / 2);
      constexpr int last = 8;
      const int ta = 2 * st, tb = 2 * st + 1 > last ? last : 2 * st + 1;
      const int oa = FLIP ? (2 - ta / 3) * CW + 2 - ta % 3 : ta / 3 * CW + ta % 3, ob = FLIP ? (2 - tb / 3) * CW + 2 - tb % 3 : tb / 3 * CW + tb % 3;
      const bf16_t* q = src + (fq < 2 ? oa : ob) * MS;
      const bf16x8 wf = G::W::get(w, st, 0);
#pragma unroll
      for (int j = 0; j < G::PTW; ++j) {
        const bf16_t* px = 2 * st == last && fq >= 2 ? zero : q + G::tile_off(j);
        acc[j][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, *reinterpret_cast<const bf16x8*>(px), acc[j][0], 0, 0, 0);
      }
    }
  } else if constexpr (C == 32) {   // the four input rows of a filter column serve both output rows
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      thirds(s);
      bf16x8 px[4];
#pragma unroll
      for (int ir = 0; ir < 4; ++ir) px[ir] = *reinterpret_cast<const bf16x8*>(src + (ir * CW + s) * MS);
#pragma unroll
      for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int nt = 0; nt < G::NTW; ++nt) {
          const bf16x8 wf = G::W::get(w, FLIP ? (2 - r) * 3 + 2 - s : r * 3 + s, nt);
#pragma unroll
          for (int j = 0; j < G::PTW; ++j) acc[j][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, px[j + r], acc[j][nt], 0, 0, 0);
        }
    }
  } else {
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      thirds(r);
#pragma unroll
      for (int s = 0; s < 3; ++s)
#pragma unroll
        for (int ks = 0; ks < C / 32; ++ks) {
          const bf16x8 px = *reinterpret_cast<const bf16x8*>(src + (r * CW + s) * MS + ks * 32);
#pragma unroll
          for (int nt = 0; nt < G::NTW; ++nt)
            acc[0][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(G::W::get(w, (FLIP ? (2 - r) * 3 + 2 - s : r * 3 + s) * (C / 32) + ks, nt), px, acc[0][nt], 0, 0, 0);
        }
      keep_order();
    }
  }
}

// ---- The block that leads a run in: it halves the image and doubles the channels (CI -> C), its first convolution and the projection have stride 2.
template <int C>
struct Lead {
  static constexpr int CI = C / 2;
  using I = Geo<CI>;                                             // of the block's input
  using W1 = WStage<C, (9 * CI + 31) / 32 * 32>;          // forward: conv1 and projection (packed: zero beyond CI)
  using WP = WStage<C, 32>;
  using D1 = WStage<CI, 9 * C>;                           // their data gradients
  using DP = WStage<CI, C>;
  static constexpr int FWD_LDS = I::CANVAS + W1::BYTES + WP::BYTES + CI * 8, BWD_LDS = D1::BYTES + DP::BYTES;
  // Input pixels by the parity (pr, pc) of their row and column: a class has the shape of the output image, so its tiles of 16 pixels are the
  // output's.  A tile of class (pr, pc) takes (1 + pr)*(1 + pc) filter taps.  A wave's tiles j: C = 32: both its output rows, all four classes;
  // C = 64: one tile, waves 0 ... 3 the classes (0, 0) and (1, 1), the others (0, 1) and (1, 0): five and four taps.
  static constexpr int TI = C == 32 ? 8 : 2, NTI = CI / 16;
};
// stride 2 forward from the canvas of the input (CI channels).  src: tap (0, 0) of the lane's pixel (+ channels as for conv3x3)
template <int C>
__device__ __forceinline__ void conv3x3_s2(const bf16_t* src, const bf16_t* zero, const bf16_t* w, int fq, floatx4 (&acc)[Geo<C>::PTW][Geo<C>::NTW]) {
  using G = Geo<C>;
  using I = typename Lead<C>::I;
  using W1 = typename Lead<C>::W1;
  constexpr int MS = I::MS, CW = I::CW;
#pragma unroll
  for (int st = 0; st < (C == 32 ? 5 : 9); ++st) {
    const int ta = C == 32 ? 2 * st : st, tb = C == 32 ? (2 * st + 1 > 8 ? 8 : 2 * st + 1) : st;   // 16 channels: two taps per step, as in conv3x3
    const int oa = ta / 3 * CW + ta % 3, ob = tb / 3 * CW + tb % 3;
    const bf16_t* q = src + (C == 32 && fq >= 2 ? ob : oa) * MS;
#pragma unroll
    for (int j = 0; j < G::PTW; ++j) {
      const bf16_t* px = C == 32 && st == 4 && fq >= 2 ? zero : q + j * 2 * CW * MS;
      const bf16x8 x = *reinterpret_cast<const bf16x8*>(px);
#pragma unroll
      for (int nt = 0; nt < G::NTW; ++nt) acc[j][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W1::get(w, st, nt), x, acc[j][nt], 0, 0, 0);
    }
  }
}
// projection, stride 2, from the same canvas
template <int C>
__device__ __forceinline__ void proj_s2(const bf16_t* src, const bf16_t* zero, const bf16_t* w, int fq, floatx4 (&acc)[Geo<C>::PTW][Geo<C>::NTW]) {
  using G = Geo<C>;
  using I = typename Lead<C>::I;
#pragma unroll
  for (int j = 0; j < G::PTW; ++j) {
    const bf16_t* px = C == 32 && fq >= 2 ? zero : src + (I::CW + 1 + j * 2 * I::CW) * I::MS;
    const bf16x8 x = *reinterpret_cast<const bf16x8*>(px);
#pragma unroll
    for (int nt = 0; nt < G::NTW; ++nt) acc[j][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Lead<C>::WP::get(w, 0, nt), x, acc[j][nt], 0, 0, 0);
  }
}
// data gradient of conv1 for a tile of class (PR, PC), from the canvas of its output's gradient.  src: the canvas at the lane's output pixel, + fq*8
template <int C, int PR, int PC>
__device__ __forceinline__ void dgrad_s2(const bf16_t* src, const bf16_t* w, floatx4 (&acc)[Lead<C>::NTI]) {
  using G = Geo<C>;
  // input row 2*i + PR comes from output row i by tap 1 (PR = 0), from rows i + 1 and i by taps 0 and 2 (PR = 1)
#pragma unroll
  for (int r = 0; r <= PR; ++r)
#pragma unroll
    for (int s = 0; s <= PC; ++s) {
      const int tr = PR == 0 ? 1 : 2 * r, ts = PC == 0 ? 1 : 2 * s, dr = PR == 0 ? 0 : 1 - r, ds = PC == 0 ? 0 : 1 - s;
#pragma unroll
      for (int ks = 0; ks < C / 32; ++ks) {
        const bf16x8 x = *reinterpret_cast<const bf16x8*>(src + (dr * G::CW + ds) * G::MS + ks * 32);
#pragma unroll
        for (int nt = 0; nt < Lead<C>::NTI; ++nt)
          acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Lead<C>::D1::get(w, (tr * 3 + ts) * (C / 32) + ks, nt), x, acc[nt], 0, 0, 0);
      }
    }
}

// what every kernel of a lane's place needs
template <int C>
struct Lane {
  int tid, lane, wave, fr, fq, pw, cg;
  unsigned off;                 // of its channels in an image
  int cw, cr;                   // canvas: where it writes (its pixel, its channels) and tap (0, 0) of its reads
  __device__ __forceinline__ Lane() {
    using G = Geo<C>;
    tid = threadIdx.x; lane = tid & 63; wave = wave_index(); fr = lane & 15; fq = lane >> 4;
    pw = G::CG == 1 ? wave : wave % G::NPW; cg = G::CG == 1 ? 0 : wave / G::NPW;
    const int p = pw * G::NPX + fr, row = p / G::IMG, col = p % G::IMG, c0 = cg * G::NTW * 16;
    off = C == 16 ? (unsigned)(p * C + fq * 4) : px_offset(p, C, fq) + (unsigned)c0;
    cw = ((row + 1) * G::CW + col + 1) * G::MS + c0 + fq * 4;
    cr = (row * G::CW + col) * G::MS + (C == 16 ? (fq & 1) * 8 : fq * 8);
  }
};

}  // namespace
}  // namespace hpf
