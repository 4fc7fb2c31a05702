// Image-resident kernels for runs of basic blocks (two 3x3 convolutions of C channels, identity shortcut), residual stream in
// registers; bf16 mode.  Pre-activation (ResNet-20 / ResNet-110):  a1 = relu(bn1(x)); c1 = conv1(a1); a2 = relu(bn2(c1)); y = x + conv2(a2).
// Post-activation (ResNet-v1):  c1 = conv1(x); a1 = relu(bn1(c1)); c2 = conv2(a1); y = relu(bn2(c2) + x).
// Ownership, exchange and register layout: kernels_resident_reg.hip.  Both convolutions read their operand from one canvas
// in LDS (zero border); everything else of a block stays in registers.
//
// Shapes and how the 8 waves share an image (of the tiles of 16 pixels):
//   C = 16, 32 x 32: 64 tiles, eight per wave; two filter taps per MFMA step
//   C = 32, 16 x 16: 16 tiles, two image rows per wave, whose input rows overlap
//   C = 64,  8 x  8: 4 tiles (two image rows each); two waves share a tile's channels
// What bounds them is latency: two exchanges per block and direction (1.5 us each) and the chain canvas - barrier -
// contraction - statistics.  The form with LDS tiles measured 17.4 / 10.7 / 12 us per block forward.  A run of 9 blocks of 32 channels and one
// of 3 blocks of 64 on 128 images: 139 -> 104 us forward, 154 -> 120 us backward; the three runs of ResNet-110 v1 (52 blocks):
// 683 -> 477 and 820 -> 568 us.
// Few images (4 or 8 of a batch) leave no other work-group to hide a wave that waits for the memory pipeline to take its loads:
// at 64 channels 2.2 us of an inference block were spent asking for the next matrix in one go.  With the loads dealt out over the
// contraction the same runs take 97 and 111 us (128 images), 440 and 541 us (v1), and inference of ResNet-110 on 4 images 317 -> 278 us.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "hpf_resident_reg.h"

namespace hpf {
namespace {

template <int C>
struct Geo {
  static constexpr int IMG = C == 16 ? 32 : C == 32 ? 16 : 8, P = IMG * IMG;
  static constexpr int CG = C == 64 ? 2 : 1, NPW = RG_NW / CG;          // waves per tile, waves along the pixels
  static constexpr int PTW = P / 16 / NPW, NTW = C / 16 / CG;           // pixel tiles and channel tiles per wave
  static constexpr int CW = IMG + 2, MS = C + 8;                        // canvas row and pixel pitch (elements)
  static constexpr int NPX = PTW * 16;
  // tile j of a wave in the canvas, from its first one
  static constexpr int tile_off(int j) { return C == 16 ? ((j >> 1) * CW + (j & 1) * 16) * MS : j * CW * MS; }
  using W = WStage<C, (9 * C + 31) / 32 * 32, false>;
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

template <int C, bool INFER>
constexpr int basic_fwd_lds() {
  using G = Geo<C>;
  return G::CANVAS + G::W::BYTES + 2 * C * 8 + (INFER ? 0 : G::NPW * 2 * C * 4) + 16;
}

template <int C, bool POST, bool INFER>
__global__ void __launch_bounds__(RG_NT) k_basic_forward(const ResArgs a) {
  static_assert(!(POST && INFER), "post-activation runs: training only");
  using G = Geo<C>;
  constexpr int PTW = G::PTW, NTW = G::NTW;
  const Lane<C> L;
  const int tid = L.tid, lane = L.lane, wave = L.wave, fr = L.fr, fq = L.fq;
  const int z = blockIdx.x % a.ngroup, me = blockIdx.x / a.ngroup;   // with g == 8 micro-batch z lives on XCD z
  ResCtx cx{(char*)pick(a.base, z), pick(a.act_in, z), pick(a.act_out, z), nullptr, nullptr};
  u64* xchg = reinterpret_cast<u64*>(cx.base + a.xchg_off);
  unsigned* tagp = reinterpret_cast<unsigned*>(cx.base + a.tag_off);
  const unsigned tag0 = INFER ? 0u : *tagp;
  unsigned phase = 0;
  auto slot = [&]() { return xchg + (size_t)(phase & 1u) * resident_slot_members(a.nmem) * (2 * C); };
  auto image = [&](unsigned long long off) { return cx.tensor(off) + (size_t)me * (G::P * C); };

  extern __shared__ __align__(16) unsigned char smem[];
  bf16_t* canvas = reinterpret_cast<bf16_t*>(smem);
  bf16_t* sW = reinterpret_cast<bf16_t*>(smem + G::CANVAS);
  float2* coef1 = reinterpret_cast<float2*>(smem + G::CANVAS + G::W::BYTES);   // of the first / second BatchNorm
  float2* coef2 = coef1 + C;
  int* fail = reinterpret_cast<int*>(coef2 + C);
  float* red = reinterpret_cast<float*>(fail + 4);     // training: NPW x 2*C
  float* const red_w = red + L.pw * 2 * C + L.cg * NTW * 16;
  const bf16_t* const wr = sW + L.cg * NTW * 512 + lane * 8;
  const int c_at = L.cg * NTW * 16 + fq * 4;           // the lane's first channel
  const float inv_n = 1.f / (float)a.nmem;

  typename G::W w;
  floatx4 X[PTW][NTW];
  uint2 pk[PTW][NTW];
  auto to_canvas = [&] {
#pragma unroll
    for (int j = 0; j < PTW; ++j)
#pragma unroll
      for (int nt = 0; nt < NTW; ++nt) *reinterpret_cast<uint2*>(canvas + L.cw + G::tile_off(j) + nt * 16) = pk[j][nt];
  };
  auto bn_pack = [&](const floatx4 (&v)[PTW][NTW], const float2* cf) {
#pragma unroll
    for (int nt = 0; nt < NTW; ++nt)
#pragma unroll
      for (int j = 0; j < PTW; ++j) pk[j][nt] = bn_relu_pack(v[j][nt], cf + c_at + nt * 16);
  };
  auto round_to = [&](floatx4 (&v)[PTW][NTW], uint2 (&p)[PTW][NTW]) {   // v rounded to bf16, p its packed form
#pragma unroll
    for (int j = 0; j < PTW; ++j)
#pragma unroll
      for (int nt = 0; nt < NTW; ++nt) { p[j][nt] = pack4(v[j][nt]); v[j][nt] = unpack4(p[j][nt]); }
  };
  // inference: the coefficients of a block, one channel per lane: wave 0 takes those of the first BatchNorm, wave 1 those of the second.  Read a
  // block ahead of their use, as the loads of a wave that waits for them hold up the work-group
  const bool t_on = wave < 2 && lane < C;
  float rc_mean, rc_var, rc_gamma, rc_beta;
  auto load_coef = [&](int b) {
    const ResBlock* t = a.blocks + b;
    if (t_on) {
      const float* run = a.running + t->run_off[wave];
      rc_mean = run[lane];
      rc_var = run[C + lane];
      rc_gamma = (a.params + t->gamma_off[wave])[lane];
      rc_beta = (a.params + t->beta_off[wave])[lane];
    }
  };
  auto store_coef = [&](int q, float2* dst) {
    if (t_on && wave == q) dst[lane] = bn_scale_shift(rc_mean, 1.0f / sqrtf(rc_var + a.eps), rc_gamma, rc_beta);
  };
  // statistics of v -> coef of BatchNorm q of block B; `late` runs behind the polls
  auto exchange = [&](const floatx4 (&v)[PTW][NTW], const ResBlock& B, int q, float2* coef, auto&& late) -> bool {
    const int gc = gather_channel<C>(wave, lane);
    const float gamma = (a.params + B.gamma_off[q])[gc], beta = (a.params + B.beta_off[q])[gc];
    stats_wave(v, red_w, C, fr, fq);
    __syncthreads();
    const unsigned tag = tag0 + 1u + phase;
    stats_publish_waves<C, G::NPX, G::NPW>(red, slot(), me, tag);
    const StatsOut o{coef, me == 0 ? reinterpret_cast<float*>(cx.base + B.stats_off[q]) : nullptr};
    collect_stats<C>(slot(), a.nmem, tag, inv_n, (float)G::P, a.eps, gamma, beta, o, wave, lane, fail);
    ++phase;
    late();
    __syncthreads();
    if (*fail) {
      if (tid == 0) atomicExch(a.abort_flag, 1);
      return false;
    }
    return true;
  };
  {
    const ResBlock B0 = a.blocks[0];
    w.issue(a.packed + B0.wf_off[0], wave, fr, fq);
    if constexpr (INFER) load_coef(0);
    px_load(pk, image(B0.x_off), L.off);
    for (int i = tid; i < G::CANVAS / 16; i += RG_NT) reinterpret_cast<u32x4*>(canvas)[i] = u32x4{0u, 0u, 0u, 0u};
    if (tid == 0) *fail = 0;
    px_arrange(pk);
#pragma unroll
    for (int j = 0; j < PTW; ++j)
#pragma unroll
      for (int nt = 0; nt < NTW; ++nt) X[j][nt] = unpack4(pk[j][nt]);
    w.commit(sW, wave, lane);
    if constexpr (INFER) { store_coef(0, coef1); store_coef(1, coef2); }
    __syncthreads();
    if constexpr (!POST && !INFER)
      if (!exchange(X, B0, 0, coef1, [] {})) return;
  }
  ResBlock B = a.blocks[0], Bn = B;
  for (int bi = 0; bi < a.nblk; ++bi, B = Bn) {
    const bool more = bi + 1 < a.nblk;
    Bn = a.blocks[more ? bi + 1 : bi];   // a block ahead of its use
    // ---- conv1 on relu(bn1(x)) | x
    if constexpr (!POST) bn_pack(X, coef1);
    else {
#pragma unroll
      for (int j = 0; j < PTW; ++j)
#pragma unroll
        for (int nt = 0; nt < NTW; ++nt) pk[j][nt] = pack4(X[j][nt]);
    }
    to_canvas();
    __syncthreads();
    if constexpr (INFER) load_coef(more ? bi + 1 : bi);
    floatx4 acc[PTW][NTW];
#pragma unroll
    for (int j = 0; j < PTW; ++j)
#pragma unroll
      for (int nt = 0; nt < NTW; ++nt) acc[j][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
    conv3x3<C, false>(canvas + L.cr, canvas, wr, fq, acc, [&](auto i) { w.template issue_third<i.value>(a.packed + B.wf_off[1], wave, fr, fq); });
    uint2 cp[PTW][NTW];
    round_to(acc, cp);
    if constexpr (INFER) {
      store_coef(0, coef1);   // every wave has used this block's
      __syncthreads();   // the canvas and conv1's matrix have been read
      w.commit(sW, wave, lane);
    } else {
      if (!exchange(acc, B, POST ? 0 : 1, coef2, [&] {
            w.commit(sW, wave, lane);
            if constexpr (POST) { if (bi > 0) px_store(image(a.blocks[bi - 1].y_off), L.off, pk); }   // the block before's output
            px_store(image(B.c1_off), L.off, cp);
          }))
        return;
    }
    // ---- conv2 on relu(bn2(c1)), onto x | on its own
    bn_pack(acc, coef2);
    to_canvas();
    __syncthreads();
    auto next_matrix = [&](auto i) { if (more) w.template issue_third<i.value>(a.packed + Bn.wf_off[0], wave, fr, fq); };
    if constexpr (!POST) {
      conv3x3<C, false>(canvas + L.cr, canvas, wr, fq, X, next_matrix);
      round_to(X, cp);
      if constexpr (INFER) {
        if (!more) { px_store(image(B.y_off), L.off, cp); break; }
        store_coef(1, coef2);   // every wave has used this block's
        __syncthreads();
        w.commit(sW, wave, lane);
      } else if (more) {
        if (!exchange(X, Bn, 0, coef1, [&] {
              w.commit(sW, wave, lane);
              px_store(image(B.y_off), L.off, cp);
            }))
          return;
      } else {
        px_store(image(B.y_off), L.off, cp);
      }
    } else {
#pragma unroll
      for (int j = 0; j < PTW; ++j)
#pragma unroll
        for (int nt = 0; nt < NTW; ++nt) acc[j][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
      conv3x3<C, false>(canvas + L.cr, canvas, wr, fq, acc, next_matrix);
      round_to(acc, cp);
      if (!exchange(acc, B, 1, coef1, [&] {
            if (more) w.commit(sW, wave, lane);
            px_store(image(B.c2_off), L.off, cp);
          }))
        return;
#pragma unroll
      for (int nt = 0; nt < NTW; ++nt) {
        const float4 p = reinterpret_cast<const float4*>(coef1 + c_at + nt * 16)[0], q = reinterpret_cast<const float4*>(coef1 + c_at + nt * 16)[1];
        const float sc[4] = {p.x, p.z, q.x, q.z}, sh[4] = {p.y, p.w, q.y, q.w};
#pragma unroll
        for (int j = 0; j < PTW; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) X[j][nt][e] = fmaxf(fmaf(acc[j][nt][e], sc[e], sh[e]) + X[j][nt][e], 0.f);
      }
      round_to(X, cp);
      if (!more) px_store(image(B.y_off), L.off, cp);
    }
  }
  // every member has read the counter before it took part in the first exchange, which member 0 has left
  if (!INFER && me == 0 && tid == 0) *tagp = tag0 + phase;
}

template <int C>
constexpr int basic_bwd_lds() {
  using G = Geo<C>;
  return G::CANVAS + G::W::BYTES + (2 * 4 * C + 3 * C + G::NPW * 2 * C) * 4 + 16;
}

template <int C, bool POST>
__global__ void __launch_bounds__(RG_NT) k_basic_backward(const ResArgs a) {
  using G = Geo<C>;
  constexpr int PTW = G::PTW, NTW = G::NTW;
  // BatchNorm parameter gradients: stored for the run's weight-gradient launch, or added here where there is none that knows of them
  constexpr bool DIRECT = POST || C == 16;
  const Lane<C> L;
  const int tid = L.tid, lane = L.lane, wave = L.wave, fr = L.fr, fq = L.fq;
  const int z = blockIdx.x % a.ngroup, me = blockIdx.x / a.ngroup;
  ResCtx cx{(char*)pick(a.base, z), pick(a.act_in, z), pick(a.act_out, z), pick(a.err_in, z), pick(a.err_out, z)};
  u64* xchg = reinterpret_cast<u64*>(cx.base + a.xchg_off);
  unsigned* tagp = reinterpret_cast<unsigned*>(cx.base + a.tag_off);
  const unsigned tag0 = *tagp;
  unsigned phase = 0;
  auto slot = [&]() { return xchg + (size_t)(phase & 1u) * resident_slot_members(a.nmem) * (2 * C); };
  auto image = [&](unsigned long long off) { return cx.tensor(off) + (size_t)me * (G::P * C); };

  extern __shared__ __align__(16) unsigned char smem[];
  bf16_t* canvas = reinterpret_cast<bf16_t*>(smem);
  bf16_t* sW = reinterpret_cast<bf16_t*>(smem + G::CANVAS);
  float* cf1 = reinterpret_cast<float*>(smem + G::CANVAS + G::W::BYTES);
  float* cf2 = cf1 + 4 * C;
  float* tab = cf2 + 4 * C;
  int* fail = reinterpret_cast<int*>(tab + 3 * C);
  float* red = reinterpret_cast<float*>(fail + 4);     // NPW x 2*C
  const int c0 = L.cg * NTW * 16;
  float* const red_w = red + L.pw * 2 * C + c0;
  const bf16_t* const wr = sW + L.cg * NTW * 512 + lane * 8;
  const float inv_M = 1.f / ((float)a.nmem * (float)G::P);

  typename G::W w;
  uint2 DY[PTW][NTW], xa[PTW][NTW], xb[PTW][NTW], yv[PTW][NTW], dcp[PTW][NTW];
  // tables: wave 0 the channels of the first BatchNorm, wave 1 those of the second
  CfRegs tb;
  float* const t_dst = wave == 0 ? cf1 : cf2;
  const bool t_on = wave < 2 && lane < C;
  auto load_tables = [&](int bi) {
    if (t_on) {
      const ResBlock* t = a.blocks + bi;
      tb.load(reinterpret_cast<const float*>(cx.base + t->stats_off[wave]), a.params + t->gamma_off[wave], a.params + t->beta_off[wave], lane, C);
    }
  };
  auto store_tables = [&] { if (t_on) tb.store(t_dst, lane, C); };
  auto to_canvas = [&](const uint2 (&v)[PTW][NTW]) {
#pragma unroll
    for (int j = 0; j < PTW; ++j)
#pragma unroll
      for (int nt = 0; nt < NTW; ++nt) *reinterpret_cast<uint2*>(canvas + L.cw + G::tile_off(j) + nt * 16) = v[j][nt];
  };
  // sums of a BatchNorm backward -> tab; `late` runs behind the polls
  auto exchange = [&](auto relu, floatx4 (&dz)[PTW][NTW], const uint2 (&x)[PTW][NTW], const float* cf, const ResBlock& B, int q, auto&& late) -> bool {
    const CfChannel ck(cf, gather_channel<C>(wave, lane), C);
    bwd_sums_wave<decltype(relu)::value>(dz, x, cf + c0, red_w, C, fr, fq);
    __syncthreads();
    const unsigned tag = tag0 + 1u + phase;
    sums_publish_waves<C, G::NPW>(red, slot(), me, tag);
    collect_bwd<C, 32>(slot(), a.nmem, tag, inv_M, ck, tab, !DIRECT && me == 0 ? reinterpret_cast<float*>(cx.base + B.dgb_off[q]) : nullptr, wave, lane, fail,
                       DIRECT && me == 0 ? a.grads + B.beta_off[q] : nullptr, a.grads + B.gamma_off[q]);
    ++phase;
    late();
    __syncthreads();
    if (*fail) {
      if (tid == 0) atomicExch(a.abort_flag, 1);
      return false;
    }
    return true;
  };
  auto apply = [&](const floatx4 (&dz)[PTW][NTW], const uint2 (&x)[PTW][NTW]) {   // -> dcp
#pragma unroll
    for (int nt = 0; nt < NTW; ++nt)
#pragma unroll
      for (int j = 0; j < PTW; ++j) dcp[j][nt] = pack4(bwd_apply<C>(dz[j][nt], x[j][nt], tab + c0 + nt * 16 + fq * 4));
  };
  auto zero = [&](floatx4 (&v)[PTW][NTW]) {
#pragma unroll
    for (int j = 0; j < PTW; ++j)
#pragma unroll
      for (int nt = 0; nt < NTW; ++nt) v[j][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
  };
  using Relu = std::true_type;
  using NoRelu = std::false_type;
  {
    const ResBlock BL = a.blocks[a.nblk - 1];
    w.issue(a.packed + BL.wd_off[1], wave, fr, fq);
    load_tables(a.nblk - 1);
    px_load(DY, image(BL.gy_off), L.off);
    if constexpr (POST) { px_load(yv, image(BL.y_off), L.off); px_load(xa, image(BL.c2_off), L.off); }
    else px_load(xa, image(BL.c1_off), L.off);
    for (int i = tid; i < G::CANVAS / 16; i += RG_NT) reinterpret_cast<u32x4*>(canvas)[i] = u32x4{0u, 0u, 0u, 0u};
    if (tid == 0) *fail = 0;
    px_arrange(DY);
    w.commit(sW, wave, lane);
    store_tables();
  }
  __syncthreads();
  ResBlock B = a.blocks[a.nblk - 1], Bn = B;
  for (int bi = a.nblk - 1; bi >= 0; --bi, B = Bn) {
    const bool more = bi > 0;
    Bn = a.blocks[more ? bi - 1 : 0];   // a block ahead of its use
    floatx4 acc[PTW][NTW];
    auto store_gx = [&] { if (bi + 1 < a.nblk) px_store(image(a.blocks[bi + 1].gx_off), L.off, DY); };   // the gradient of the input of the block above
    if constexpr (!POST) {
      // ---- conv2 data gradient, BN2 + ReLU backward -> dc1
      to_canvas(DY);
      __syncthreads();
      zero(acc);
      conv3x3<C, true>(canvas + L.cr, canvas, wr, fq, acc, [&](auto i) { w.template issue_third<i.value>(a.packed + B.wd_off[0], wave, fr, fq); });
      px_arrange(xa);
      if (!exchange(Relu{}, acc, xa, cf2, B, 1, [&] {
            w.commit(sW, wave, lane);
            store_gx();
            px_load(xb, image(B.x_off), L.off);
          }))
        return;
      apply(acc, xa);
      to_canvas(dcp);
      __syncthreads();
      // ---- conv1 data gradient, BN1 + ReLU backward, plus the shortcut
      zero(acc);
      conv3x3<C, true>(canvas + L.cr, canvas, wr, fq, acc, [&](auto i) { if (more) w.template issue_third<i.value>(a.packed + Bn.wd_off[1], wave, fr, fq); });
      if (more) load_tables(bi - 1);
      px_arrange(xb);
      if (!exchange(Relu{}, acc, xb, cf1, B, 0, [&] {
            if (more) { w.commit(sW, wave, lane); store_tables(); px_load(xa, image(Bn.c1_off), L.off); }
            px_store(image(B.dc1_off), L.off, dcp);
          }))
        return;
#pragma unroll
      for (int nt = 0; nt < NTW; ++nt)
#pragma unroll
        for (int j = 0; j < PTW; ++j)
          DY[j][nt] = pack4(bwd_apply<C>(acc[j][nt], xb[j][nt], tab + c0 + nt * 16 + fq * 4) + unpack4(DY[j][nt]));
    } else {
      // ---- through the join and BN2: dz = dy*[y > 0] -> dc2
      floatx4 dz[PTW][NTW];
      px_arrange(yv);
      px_arrange(xa);
#pragma unroll
      for (int j = 0; j < PTW; ++j)
#pragma unroll
        for (int nt = 0; nt < NTW; ++nt)
#pragma unroll
          for (int e = 0; e < 4; ++e) dz[j][nt][e] = elem4(yv[j][nt], e) > 0.f ? elem4(DY[j][nt], e) : 0.f;
      if (bi + 1 < a.nblk) w.issue(a.packed + B.wd_off[1], wave, fr, fq);
      if (!exchange(NoRelu{}, dz, xa, cf2, B, 1, [&] {
            if (bi + 1 < a.nblk) w.commit(sW, wave, lane);   // conv1's data gradient of the block above is behind the barrier
            store_gx();
            px_load(xb, image(B.c1_off), L.off);
          }))
        return;
      apply(dz, xa);
      to_canvas(dcp);
      __syncthreads();
      // ---- conv2 data gradient, BN1 + ReLU backward -> dc1
      zero(acc);
      conv3x3<C, true>(canvas + L.cr, canvas, wr, fq, acc, [&](auto i) { w.template issue_third<i.value>(a.packed + B.wd_off[0], wave, fr, fq); });
      if (more) load_tables(bi - 1);
      px_arrange(xb);
      if (!exchange(Relu{}, acc, xb, cf1, B, 0, [&] {
            w.commit(sW, wave, lane);
            px_store(image(B.dc2_off), L.off, dcp);
            if (more) { px_load(yv, image(Bn.y_off), L.off); px_load(xa, image(Bn.c2_off), L.off); }
          }))
        return;
      apply(acc, xb);
      to_canvas(dcp);
      if (more) store_tables();   // both tables of this block have been used
      __syncthreads();
      px_store(image(B.dc1_off), L.off, dcp);
      // ---- conv1 data gradient plus the shortcut
      conv3x3<C, true>(canvas + L.cr, canvas, wr, fq, dz, [](auto) {});
#pragma unroll
      for (int j = 0; j < PTW; ++j)
#pragma unroll
        for (int nt = 0; nt < NTW; ++nt) DY[j][nt] = pack4(dz[j][nt]);
    }
  }
  px_store(image(a.blocks[0].gx_off), L.off, DY);
  if (me == 0 && tid == 0) *tagp = tag0 + phase;
}

template <class K>
hipError_t launch_basic(K kernel, int lds, int g, const ResArgs& a, hipStream_t stream) {
  ResArgs b = a;
  b.ngroup = g;
  kernel<<<dim3((unsigned)(a.nmem * g)), RG_NT, (size_t)lds, stream>>>(b);
  return hipGetLastError();
}

}  // namespace

bool resident_basic_shape(int kind, int C, int H, int W) {
  return (kind == 0 || kind == 2) && ((C == 16 && H == 32 && W == 32) || (C == 32 && H == 16 && W == 16) || (C == 64 && H == 8 && W == 8));
}
hipError_t resident_basic_prepare() {
  const void* const kernels[] = {
      reinterpret_cast<const void*>(k_basic_forward<16, false, false>), reinterpret_cast<const void*>(k_basic_forward<32, false, false>),
      reinterpret_cast<const void*>(k_basic_forward<64, false, false>), reinterpret_cast<const void*>(k_basic_forward<16, false, true>),
      reinterpret_cast<const void*>(k_basic_forward<32, false, true>),  reinterpret_cast<const void*>(k_basic_forward<64, false, true>),
      reinterpret_cast<const void*>(k_basic_forward<16, true, false>),  reinterpret_cast<const void*>(k_basic_forward<32, true, false>),
      reinterpret_cast<const void*>(k_basic_forward<64, true, false>),  reinterpret_cast<const void*>(k_basic_backward<16, false>),
      reinterpret_cast<const void*>(k_basic_backward<32, false>),       reinterpret_cast<const void*>(k_basic_backward<64, false>),
      reinterpret_cast<const void*>(k_basic_backward<16, true>),        reinterpret_cast<const void*>(k_basic_backward<32, true>),
      reinterpret_cast<const void*>(k_basic_backward<64, true>)};
  for (const void* f : kernels) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}
template <int C>
static hipError_t fwd_c(int kind, int g, const ResArgs& a, bool infer, hipStream_t stream) {
  if (infer) return launch_basic(k_basic_forward<C, false, true>, basic_fwd_lds<C, true>(), g, a, stream);
  return kind == 2 ? launch_basic(k_basic_forward<C, true, false>, basic_fwd_lds<C, false>(), g, a, stream)
                   : launch_basic(k_basic_forward<C, false, false>, basic_fwd_lds<C, false>(), g, a, stream);
}
template <int C>
static hipError_t bwd_c(int kind, int g, const ResArgs& a, hipStream_t stream) {
  return kind == 2 ? launch_basic(k_basic_backward<C, true>, basic_bwd_lds<C>(), g, a, stream)
                   : launch_basic(k_basic_backward<C, false>, basic_bwd_lds<C>(), g, a, stream);
}
hipError_t launch_basic_forward(int kind, int g, int C, const ResArgs& a, bool infer, hipStream_t stream) {
  if (kind == 2 && infer) return hipErrorInvalidValue;
  return C == 16 ? fwd_c<16>(kind, g, a, infer, stream) : C == 32 ? fwd_c<32>(kind, g, a, infer, stream) : fwd_c<64>(kind, g, a, infer, stream);
}
hipError_t launch_basic_backward(int kind, int g, int C, const ResArgs& a, hipStream_t stream) {
  return C == 16 ? bwd_c<16>(kind, g, a, stream) : C == 32 ? bwd_c<32>(kind, g, a, stream) : bwd_c<64>(kind, g, a, stream);
}

}  // namespace hpf
