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
//
// The block in front of a run of 32 or 64 channels halves the image and doubles the channels; it leads the run in (LEAD): the same launch starts, or
// in the backward pass ends, with it.  Layer by layer it took five launches forward and five backward of 4 to 13 us each, which a few images leave
// nearly empty; as part of the run it takes two exchanges and four contractions a direction, and its output never comes back from memory.  ResNet-20
// on 4 images (two such blocks) 336 -> 260 us a batch, a quarter of ResNet-110 on 128 images (one) 359 -> 309, ResNet-110 v1 1437 -> 1333,
// inference of ResNet-110 on 4 images 271 -> 242.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "hpf_resident_basic.h"

namespace hpf {
namespace {

template <int C, bool LEAD>
constexpr int lead_lds(bool fwd) {
  if constexpr (LEAD) return fwd ? Lead<C>::FWD_LDS : Lead<C>::BWD_LDS;
  return 0;
}
template <int C, bool LEAD>
constexpr int lead_proj_bytes() {
  if constexpr (LEAD) return Lead<C>::DP::BYTES;
  return 0;
}
template <int C, bool INFER, bool LEAD>
constexpr int basic_fwd_lds() {
  using G = Geo<C>;
  return G::CANVAS + G::W::BYTES + 2 * C * 8 + (INFER ? 0 : G::NPW * 2 * C * 4) + 16 + lead_lds<C, LEAD>(true);
}

// FEW: micro-batches of up to 16 images, which take one chunk of 16 records.  17 blocks, 16 images, us forward and backward, chunks of 32 / 16: 64 channels
// 150 and 186 / 143 and 176, 32 channels 127 and 151 / 124 and 147, 16 channels 149 and 189 / 146 and 186; 4 images of 64 channels 146 and 170 / 145 and 168.
constexpr int BASIC_FEW = 16;

// LEAD: the run's first block is the one that halves the image and doubles the channels (Lead).
template <int C, bool POST, bool INFER, bool LEAD, bool FEW>
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
  auto join = [&](const floatx4 (&v)[PTW][NTW], const float2* cf) {   // X = relu(bn(v) + X)
#pragma unroll
    for (int nt = 0; nt < NTW; ++nt) {
      const float4 p = reinterpret_cast<const float4*>(cf + c_at + nt * 16)[0], q = reinterpret_cast<const float4*>(cf + c_at + nt * 16)[1];
      const float sc[4] = {p.x, p.z, q.x, q.z}, sh[4] = {p.y, p.w, q.y, q.w};
#pragma unroll
      for (int j = 0; j < PTW; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) X[j][nt][e] = fmaxf(fmaf(v[j][nt][e], sc[e], sh[e]) + X[j][nt][e], 0.f);
    }
  };
  // inference: the coefficients of a block, one channel per lane: wave 0 takes those of the first BatchNorm, wave 1 those of the second.  Read a
  // block ahead of their use, as the loads of a wave that waits for them hold up the work-group
  const bool t_on = wave < 2 && lane < C;
  float rc_mean, rc_var, rc_gamma, rc_beta;
  auto load_coef = [&](int b) {
    const ResBlock* t = a.blocks + b;
    const int n = LEAD && b == 0 && wave == 0 ? C / 2 : C;
    if (t_on && lane < n) {
      const float* run = a.running + t->run_off[wave];
      rc_mean = run[lane];
      rc_var = run[n + lane];
      rc_gamma = (a.params + t->gamma_off[wave])[lane];
      rc_beta = (a.params + t->beta_off[wave])[lane];
    }
  };
  auto store_coef = [&](int q, float2* dst) {
    if (t_on && wave == q) dst[lane] = bn_scale_shift(rc_mean, 1.0f / sqrtf(rc_var + a.eps), rc_gamma, rc_beta);
  };
  // statistics of v, a tensor of geometry GV -> coef of BatchNorm q of block B; `late` runs behind the polls
  auto exchange_of = [&](auto gv, const auto& v, float* row, const ResBlock& B, int q, float2* coef, auto&& late) -> bool {
    using GV = decltype(gv);
    constexpr int Cc = GV::NC;
    const int gc = gather_channel<Cc>(wave, lane);
    const float gamma = (a.params + B.gamma_off[q])[gc], beta = (a.params + B.beta_off[q])[gc];
    stats_wave(v, row, Cc, fr, fq);
    __syncthreads();
    const unsigned tag = tag0 + 1u + phase;
    stats_publish_waves<Cc, GV::NPX, GV::NPW>(red, slot(), me, tag);
    const StatsOut o{coef, me == 0 ? reinterpret_cast<float*>(cx.base + B.stats_off[q]) : nullptr};
    collect_stats<Cc, FEW ? BASIC_FEW : 32>(slot(), a.nmem, tag, inv_n, (float)GV::P, a.eps, gamma, beta, o, wave, lane, fail);
    ++phase;
    late();
    __syncthreads();
    if (*fail) {
      if (tid == 0) atomicExch(a.abort_flag, 1);
      return false;
    }
    return true;
  };
  auto exchange = [&](const floatx4 (&v)[PTW][NTW], const ResBlock& B, int q, float2* coef, auto&& late) -> bool {
    return exchange_of(G{}, v, red_w, B, q, coef, late);
  };
  constexpr int FIRST = LEAD ? 1 : 0;   // the run's first identity block
  if constexpr (LEAD) {
    using LD = Lead<C>;
    using I = typename LD::I;
    constexpr int CI = LD::CI;
    const Lane<CI> LI;
    unsigned char* base = smem + basic_fwd_lds<C, INFER, false>();
    bf16_t* canvas_x = reinterpret_cast<bf16_t*>(base);
    bf16_t* sW1 = reinterpret_cast<bf16_t*>(base + I::CANVAS);
    bf16_t* sWP = reinterpret_cast<bf16_t*>(base + I::CANVAS + LD::W1::BYTES);
    float2* coef_x = reinterpret_cast<float2*>(base + I::CANVAS + LD::W1::BYTES + LD::WP::BYTES);
    const ResBlock T = a.blocks[0];
    const bool more = a.nblk > 1;
    const ResBlock Tn = a.blocks[more ? 1 : 0];
    uint2 px[I::PTW][I::NTW];
    px_load(px, cx.tensor(T.x_off) + (size_t)me * (I::P * CI), LI.off);
    typename LD::W1 w1;
    typename LD::WP wp;
    w1.issue(a.packed + T.wf_off[0], wave, fr, fq);
    wp.issue(a.packed + T.pf_off, wave, fr, fq);
    w.issue(a.packed + T.wf_off[1], wave, fr, fq);
    if constexpr (INFER) load_coef(0);
    for (int i = tid; i < G::CANVAS / 16; i += RG_NT) reinterpret_cast<u32x4*>(canvas)[i] = u32x4{0u, 0u, 0u, 0u};
    for (int i = tid; i < I::CANVAS / 16; i += RG_NT) reinterpret_cast<u32x4*>(canvas_x)[i] = u32x4{0u, 0u, 0u, 0u};
    if (tid == 0) *fail = 0;
    px_arrange(px);
    w1.commit(sW1, wave, lane);
    wp.commit(sWP, wave, lane);
    w.commit(sW, wave, lane);
    if constexpr (INFER) { if (lane < CI) store_coef(0, coef_x); store_coef(1, coef2); }
    __syncthreads();
    // ---- conv1 and the projection on relu(bn1(x)) | x
    if constexpr (!POST) {
      floatx4 xf[I::PTW][I::NTW];
#pragma unroll
      for (int j = 0; j < I::PTW; ++j)
#pragma unroll
        for (int nt = 0; nt < I::NTW; ++nt) xf[j][nt] = unpack4(px[j][nt]);
      if constexpr (!INFER)
        if (!exchange_of(I{}, xf, red + wave * 2 * CI, T, 0, coef_x, [] {})) return;
#pragma unroll
      for (int nt = 0; nt < I::NTW; ++nt)
#pragma unroll
        for (int j = 0; j < I::PTW; ++j) px[j][nt] = bn_relu_pack(xf[j][nt], coef_x + nt * 16 + fq * 4);
    }
#pragma unroll
    for (int j = 0; j < I::PTW; ++j)
#pragma unroll
      for (int nt = 0; nt < I::NTW; ++nt) *reinterpret_cast<uint2*>(canvas_x + LI.cw + I::tile_off(j) + nt * 16) = px[j][nt];
    __syncthreads();
    if constexpr (INFER) { if (more) load_coef(1); }
    floatx4 acc[PTW][NTW];
#pragma unroll
    for (int j = 0; j < PTW; ++j)
#pragma unroll
      for (int nt = 0; nt < NTW; ++nt) acc[j][nt] = X[j][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
    const int p = L.pw * G::NPX + fr, row = p / G::IMG, col = p % G::IMG, at = L.cg * NTW * 512 + lane * 8;
    const bf16_t* src = canvas_x + (2 * row * I::CW + 2 * col) * I::MS + (CI == 16 ? (fq & 1) * 8 : fq * 8);
    conv3x3_s2<C>(src, canvas_x, sW1 + at, fq, acc);
    proj_s2<C>(src, canvas_x, sWP + at, fq, X);
    uint2 cp[PTW][NTW], sp[PTW][NTW];
    round_to(acc, cp);
    round_to(X, sp);   // the shortcut is a tensor of its own
    if constexpr (INFER) {
      if (more) store_coef(0, coef1);
    } else {
      if (!exchange(acc, T, POST ? 0 : 1, coef2, [&] {
            px_store(image(T.c1_off), L.off, cp);
            if constexpr (POST) px_store(image(T.sc_off), L.off, sp);
          }))
        return;
    }
    // ---- conv2 on relu(bn2(c1)), onto the shortcut | on its own
    bn_pack(acc, coef2);
    to_canvas();
    if constexpr (POST) px_store(image(T.a1_off), L.off, pk);   // no kernel reads it, but hpf_stash_read has always given it out for these blocks
    __syncthreads();
    auto next_matrix = [&](auto i) { if (more) w.template issue_third<i.value>(a.packed + Tn.wf_off[0], wave, fr, fq); };
    if constexpr (!POST) {
      conv3x3<C, false>(canvas + L.cr, canvas, wr, fq, X, next_matrix);
      round_to(X, cp);
      if (!more) {
        px_store(image(T.y_off), L.off, cp);
      } else if constexpr (INFER) {
        store_coef(1, coef2);   // every wave has used the lead's
        __syncthreads();
        w.commit(sW, wave, lane);
      } else {
        if (!exchange(X, Tn, 0, coef1, [&] {
              w.commit(sW, wave, lane);
              px_store(image(T.y_off), L.off, cp);
            }))
          return;
      }
    } else {
#pragma unroll
      for (int j = 0; j < PTW; ++j)
#pragma unroll
        for (int nt = 0; nt < NTW; ++nt) acc[j][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
      conv3x3<C, false>(canvas + L.cr, canvas, wr, fq, acc, next_matrix);
      round_to(acc, cp);
      if (!exchange(acc, T, 1, coef1, [&] {
            if (more) w.commit(sW, wave, lane);
            px_store(image(T.c2_off), L.off, cp);
          }))
        return;
      join(acc, coef1);
      round_to(X, cp);
      if (!more) px_store(image(T.y_off), L.off, cp);   // else stored by the next block
    }
  } else {
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
  ResBlock B = a.blocks[FIRST < a.nblk ? FIRST : 0], Bn = B;
  for (int bi = FIRST; bi < a.nblk; ++bi, B = Bn) {
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
            if constexpr (POST) { if (bi > 0) px_store(image(a.blocks[bi - 1].y_off), L.off, pk); }   // the output of the block before
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
      join(acc, coef1);
      round_to(X, cp);
      if (!more) px_store(image(B.y_off), L.off, cp);
    }
  }
  // every member has read the counter before it took part in the first exchange, which member 0 has left
  if (!INFER && me == 0 && tid == 0) *tagp = tag0 + phase;
}

template <int C, bool LEAD>
constexpr int basic_bwd_lds() {
  using G = Geo<C>;
  return G::CANVAS + G::W::BYTES + (2 * 4 * C + 3 * C + G::NPW * 2 * C) * 4 + 16 + lead_lds<C, LEAD>(false);
}

template <int C, bool POST, bool LEAD, bool FEW>
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

  bf16_t* const sD1 = reinterpret_cast<bf16_t*>(smem + basic_bwd_lds<C, false>());   // the lead's conv1 and projection
  bf16_t* const sDP = reinterpret_cast<bf16_t*>(smem + basic_bwd_lds<C, false>() + (LEAD ? lead_lds<C, LEAD>(false) - lead_proj_bytes<C, LEAD>() : 0));
  typename G::W w;
  uint2 DY[PTW][NTW], xa[PTW][NTW], xb[PTW][NTW], yv[PTW][NTW], dcp[PTW][NTW];
  // tables: wave 0 the channels of the first BatchNorm, wave 1 those of the second
  CfRegs tb;
  float* const t_dst = wave == 0 ? cf1 : cf2;
  int t_n = C;   // channels of this wave's BatchNorm (the lead's first one has C/2)
  auto t_on = [&] { return wave < 2 && lane < t_n; };
  auto load_tables = [&](int bi) {
    if (LEAD && !POST && bi == 0 && wave == 0) t_n = C / 2;
    if (t_on()) {
      const ResBlock* t = a.blocks + bi;
      tb.load(reinterpret_cast<const float*>(cx.base + t->stats_off[wave]), a.params + t->gamma_off[wave], a.params + t->beta_off[wave], lane, t_n);
    }
  };
  auto store_tables = [&] { if (t_on()) tb.store(t_dst, lane, t_n); };
  auto to_canvas = [&](const uint2 (&v)[PTW][NTW]) {
#pragma unroll
    for (int j = 0; j < PTW; ++j)
#pragma unroll
      for (int nt = 0; nt < NTW; ++nt) *reinterpret_cast<uint2*>(canvas + L.cw + G::tile_off(j) + nt * 16) = v[j][nt];
  };
  // sums of a BatchNorm backward over a tensor of geometry GV -> tab; `late` runs behind the polls.  at: the wave's first channel, row: its row of
  // red there; direct: DIRECT for this block
  auto exchange_of = [&](auto gv, auto relu, auto direct, auto& dz, const auto& x, const float* cf, int at, float* row, const ResBlock& B, int q, auto&& late) -> bool {
    using GV = decltype(gv);
    constexpr int Cc = GV::NC;
    constexpr bool D = decltype(direct)::value;
    const CfChannel ck(cf, gather_channel<Cc>(wave, lane), Cc);
    bwd_sums_wave<decltype(relu)::value>(dz, x, cf + at, row, Cc, fr, fq);
    __syncthreads();
    const unsigned tag = tag0 + 1u + phase;
    sums_publish_waves<Cc, GV::NPW>(red, slot(), me, tag);
    collect_bwd<Cc, FEW ? BASIC_FEW : 32>(slot(), a.nmem, tag, inv_M * (float)G::P / (float)GV::P, ck, tab, !D && me == 0 ? reinterpret_cast<float*>(cx.base + B.dgb_off[q]) : nullptr, wave,
                        lane, fail, D && me == 0 ? a.grads + B.beta_off[q] : nullptr, a.grads + B.gamma_off[q]);
    ++phase;
    late();
    __syncthreads();
    if (*fail) {
      if (tid == 0) atomicExch(a.abort_flag, 1);
      return false;
    }
    return true;
  };
  auto exchange = [&](auto relu, floatx4 (&dz)[PTW][NTW], const uint2 (&x)[PTW][NTW], const float* cf, const ResBlock& B, int q, auto&& late) -> bool {
    return exchange_of(G{}, relu, std::integral_constant<bool, DIRECT>{}, dz, x, cf, c0, red_w, B, q, late);
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
    if constexpr (LEAD) {
      const ResBlock T = a.blocks[0];
      typename Lead<C>::D1 d1;
      typename Lead<C>::DP dp;
      d1.issue(a.packed + T.wd_off[0], wave, fr, fq);
      dp.issue(a.packed + T.pd_off, wave, fr, fq);
      d1.commit(sD1, wave, lane);
      dp.commit(sDP, wave, lane);
    }
  }
  __syncthreads();
  constexpr int FIRST = LEAD ? 1 : 0;   // the run's first identity block
  ResBlock B = a.blocks[a.nblk - 1], Bn = B;
  for (int bi = a.nblk - 1; bi >= FIRST; --bi, B = Bn) {
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
  if constexpr (!LEAD) {
    px_store(image(a.blocks[0].gx_off), L.off, DY);
  } else {
    using LD = Lead<C>;
    constexpr int CI = LD::CI, TI = LD::TI, NTI = LD::NTI;
    B = a.blocks[0];
    auto store_gx = [&] { if (a.nblk > 1) px_store(image(a.blocks[1].gx_off), L.off, DY); };
    // the lane's output pixel of its first tile, in the canvas, and the input pixel of class (0, 0) below it
    const int t0 = C == 32 ? wave * 2 : wave & 3, ro = C == 32 ? t0 : 2 * t0 + (fr >> 3), co = C == 32 ? fr : fr & 7;
    const bf16_t* const src = canvas + ((ro + 1) * G::CW + co + 1) * G::MS + fq * 8;
    const bf16_t* const d1r = sD1 + lane * 8;
    const bf16_t* const dpr = sDP + lane * 8;
    const unsigned px0 = (unsigned)(2 * ro * (2 * G::IMG) + 2 * co);
    const bool hi = C == 64 && wave >= 4;
    auto px_at = [&](int j) -> unsigned {   // input pixel of tile j
      const int pr = C == 32 ? (j >> 1) & 1 : j, pc = C == 32 ? j & 1 : hi ? 1 - j : j;
      return px0 + (unsigned)((pr + (C == 32 ? 2 * (j >> 2) : 0)) * (2 * G::IMG) + pc);
    };
    bf16_t* const gx = cx.tensor(B.gx_off) + (size_t)me * (4 * G::P * CI);
    floatx4 da[TI][NTI];
#pragma unroll
    for (int j = 0; j < TI; ++j)
#pragma unroll
      for (int nt = 0; nt < NTI; ++nt) da[j][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto proj = [&] {   // its data gradient reaches the pixels of class (0, 0)
      if (C == 64 && hi) return;
#pragma unroll
      for (int j = 0; j < TI; j += 4)
#pragma unroll
        for (int ks = 0; ks < C / 32; ++ks) {
          const bf16x8 v = *reinterpret_cast<const bf16x8*>(src + (j >> 2) * G::CW * G::MS + ks * 32);
#pragma unroll
          for (int nt = 0; nt < NTI; ++nt) da[j][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(LD::DP::get(dpr, ks, nt), v, da[j][nt], 0, 0, 0);
        }
    };
    auto conv1 = [&] {
      if constexpr (C == 32) {
#pragma unroll
        for (int r = 0; r < 2; ++r) {
          const bf16_t* q = src + r * G::CW * G::MS;
          dgrad_s2<C, 0, 0>(q, d1r, da[4 * r]);
          dgrad_s2<C, 0, 1>(q, d1r, da[4 * r + 1]);
          dgrad_s2<C, 1, 0>(q, d1r, da[4 * r + 2]);
          dgrad_s2<C, 1, 1>(q, d1r, da[4 * r + 3]);
        }
      } else if (!hi) {
        dgrad_s2<C, 0, 0>(src, d1r, da[0]);
        dgrad_s2<C, 1, 1>(src, d1r, da[1]);
      } else {
        dgrad_s2<C, 0, 1>(src, d1r, da[0]);
        dgrad_s2<C, 1, 0>(src, d1r, da[1]);
      }
    };
    auto store = [&](const uint2 (&v)[TI][NTI]) {
#pragma unroll
      for (int j = 0; j < TI; ++j) {
        if constexpr (CI == 16) {
          *reinterpret_cast<uint2*>(gx + px_at(j) * CI + fq * 4) = v[j][0];
        } else {
          uint2 e = v[j][0], o = v[j][1];
          pair_swap(e, o);
          *reinterpret_cast<uint4*>(gx + px_offset((int)px_at(j), CI, fq)) = make_uint4(e.x, e.y, o.x, o.y);
        }
      }
    };
    uint2 out[TI][NTI];
    floatx4 acc[PTW][NTW];
    if constexpr (!POST) {
      // ---- conv2 data gradient, BN2 + ReLU backward -> dc1; the projection's data gradient from the same canvas
      to_canvas(DY);
      __syncthreads();
      zero(acc);
      conv3x3<C, true>(canvas + L.cr, canvas, wr, fq, acc, [](auto) {});
      proj();
      px_arrange(xa);
      uint2 xi[TI][NTI];
      if (!exchange_of(G{}, Relu{}, std::true_type{}, acc, xa, cf2, c0, red_w, B, 1, [&] {
            store_gx();
            const bf16_t* x = cx.tensor(B.x_off) + (size_t)me * (4 * G::P * CI);
#pragma unroll
            for (int j = 0; j < TI; ++j) {
              if constexpr (CI == 16) {
                xi[j][0] = *reinterpret_cast<const uint2*>(x + px_at(j) * CI + fq * 4);
              } else {
                const uint4 q = *reinterpret_cast<const uint4*>(x + px_offset((int)px_at(j), CI, fq));
                xi[j][0] = make_uint2(q.x, q.y);
                xi[j][1] = make_uint2(q.z, q.w);
              }
            }
          }))
        return;
      apply(acc, xa);
      to_canvas(dcp);
      __syncthreads();
      // ---- conv1 data gradient, BN1 + ReLU backward
      conv1();
      px_arrange(xi);
      if (!exchange_of(typename LD::I{}, Relu{}, std::true_type{}, da, xi, cf1, 0, red + wave * 2 * CI, B, 0, [&] { px_store(image(B.dc1_off), L.off, dcp); })) return;
#pragma unroll
      for (int nt = 0; nt < NTI; ++nt)
#pragma unroll
        for (int j = 0; j < TI; ++j) out[j][nt] = pack4(bwd_apply<CI>(da[j][nt], xi[j][nt], tab + nt * 16 + fq * 4));
    } else {
      // ---- through the join and BN2: dz = dy*[y > 0] -> dc2; the projection's data gradient of dz
      floatx4 dz[PTW][NTW];
      px_arrange(yv);
      px_arrange(xa);
      uint2 dzp[PTW][NTW];
#pragma unroll
      for (int j = 0; j < PTW; ++j)
#pragma unroll
        for (int nt = 0; nt < NTW; ++nt) {
#pragma unroll
          for (int e = 0; e < 4; ++e) dz[j][nt][e] = elem4(yv[j][nt], e) > 0.f ? elem4(DY[j][nt], e) : 0.f;
          dzp[j][nt] = pack4(dz[j][nt]);
        }
      if (a.nblk > 1) w.issue(a.packed + B.wd_off[1], wave, fr, fq);
      if (a.nblk > 1) __syncthreads();   // conv1's data gradient of the block above reads the canvas
      to_canvas(dzp);
      if (!exchange_of(G{}, NoRelu{}, std::true_type{}, dz, xa, cf2, c0, red_w, B, 1, [&] {
            if (a.nblk > 1) w.commit(sW, wave, lane);
            store_gx();
            px_store(image(B.dsc_off), L.off, dzp);
            px_load(xb, image(B.c1_off), L.off);
          }))
        return;
      proj();
      apply(dz, xa);
      __syncthreads();
      to_canvas(dcp);
      __syncthreads();
      // ---- conv2 data gradient, BN1 + ReLU backward -> dc1
      zero(acc);
      conv3x3<C, true>(canvas + L.cr, canvas, wr, fq, acc, [](auto) {});
      px_arrange(xb);
      if (!exchange_of(G{}, Relu{}, std::true_type{}, acc, xb, cf1, c0, red_w, B, 0, [&] { px_store(image(B.dc2_off), L.off, dcp); })) return;
      apply(acc, xb);
      to_canvas(dcp);
      __syncthreads();
      px_store(image(B.dc1_off), L.off, dcp);
      // ---- conv1 data gradient
      conv1();
#pragma unroll
      for (int nt = 0; nt < NTI; ++nt)
#pragma unroll
        for (int j = 0; j < TI; ++j) out[j][nt] = pack4(da[j][nt]);
    }
    store(out);
  }
  if (me == 0 && tid == 0) *tagp = tag0 + phase;
}

template <class K>
hipError_t launch_basic(K kernel, int lds, int g, const ResArgs& a, hipStream_t stream) {
  ResArgs b = a;
  b.ngroup = g;
  kernel<<<dim3((unsigned)(a.nmem * g)), RG_NT, (size_t)lds, stream>>>(b);
  return hipGetLastError();
}
template <int C, bool POST, bool LEAD>
hipError_t fwd_p(int g, const ResArgs& a, hipStream_t stream) {
  if (a.nmem <= BASIC_FEW) return launch_basic(k_basic_forward<C, POST, false, LEAD, true>, basic_fwd_lds<C, false, LEAD>(), g, a, stream);
  return launch_basic(k_basic_forward<C, POST, false, LEAD, false>, basic_fwd_lds<C, false, LEAD>(), g, a, stream);
}
template <int C, bool LEAD>
hipError_t fwd_c(int kind, int g, const ResArgs& a, bool infer, hipStream_t stream) {
  if (infer) return launch_basic(k_basic_forward<C, false, true, LEAD, false>, basic_fwd_lds<C, true, LEAD>(), g, a, stream);
  return kind == 2 ? fwd_p<C, true, LEAD>(g, a, stream) : fwd_p<C, false, LEAD>(g, a, stream);
}
template <int C, bool POST, bool LEAD>
hipError_t bwd_p(int g, const ResArgs& a, hipStream_t stream) {
  if (a.nmem <= BASIC_FEW) return launch_basic(k_basic_backward<C, POST, LEAD, true>, basic_bwd_lds<C, LEAD>(), g, a, stream);
  return launch_basic(k_basic_backward<C, POST, LEAD, false>, basic_bwd_lds<C, LEAD>(), g, a, stream);
}
template <int C, bool LEAD>
hipError_t bwd_c(int kind, int g, const ResArgs& a, hipStream_t stream) {
  return kind == 2 ? bwd_p<C, true, LEAD>(g, a, stream) : bwd_p<C, false, LEAD>(g, a, stream);
}
template <class K>
hipError_t raise_limit(K kernel) { return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024); }
template <int C, bool LEAD, bool FEW>
hipError_t prepare_f() {
  hipError_t e = raise_limit(k_basic_forward<C, false, false, LEAD, FEW>);
  if (e == hipSuccess) e = raise_limit(k_basic_forward<C, true, false, LEAD, FEW>);
  if (e == hipSuccess) e = raise_limit(k_basic_backward<C, false, LEAD, FEW>);
  if (e == hipSuccess) e = raise_limit(k_basic_backward<C, true, LEAD, FEW>);
  return e;
}
template <int C, bool LEAD>
hipError_t prepare_c() {
  hipError_t e = raise_limit(k_basic_forward<C, false, true, LEAD, false>);
  if (e == hipSuccess) e = prepare_f<C, LEAD, false>();
  if (e == hipSuccess) e = prepare_f<C, LEAD, true>();
  return e;
}
static_assert(basic_fwd_lds<64, false, true>() <= 160 * 1024 && basic_fwd_lds<32, false, true>() <= 160 * 1024 && basic_bwd_lds<64, true>() <= 160 * 1024, "LDS of a CU");

}  // namespace

bool resident_basic_shape(int kind, int C, int H, int W) {
  return (kind == 0 || kind == 2) && ((C == 16 && H == 32 && W == 32) || (C == 32 && H == 16 && W == 16) || (C == 64 && H == 8 && W == 8));
}
bool resident_lead_shape(int kind, int c_in, int c_mid, int c_out, int h_out, int w_out) {
  if (c_in * 2 != c_out) return false;
  return kind == 1 ? c_out == 128 && resident_reg_shape(kind, c_out, c_mid, h_out, w_out) : c_out >= 32 && c_mid == c_out && resident_basic_shape(kind, c_out, h_out, w_out);
}
hipError_t resident_basic_prepare() {
  hipError_t e = prepare_c<16, false>();
  if (e == hipSuccess) e = prepare_c<32, false>();
  if (e == hipSuccess) e = prepare_c<64, false>();
  if (e == hipSuccess) e = prepare_c<32, true>();
  if (e == hipSuccess) e = prepare_c<64, true>();
  return e;
}
hipError_t launch_basic_forward(int kind, int g, int C, const ResArgs& a, bool infer, hipStream_t stream) {
  if ((kind == 2 && infer) || (a.lead && C == 16)) return hipErrorInvalidValue;
  if (a.lead) return C == 32 ? fwd_c<32, true>(kind, g, a, infer, stream) : fwd_c<64, true>(kind, g, a, infer, stream);
  return C == 16 ? fwd_c<16, false>(kind, g, a, infer, stream) : C == 32 ? fwd_c<32, false>(kind, g, a, infer, stream) : fwd_c<64, false>(kind, g, a, infer, stream);
}
hipError_t launch_basic_backward(int kind, int g, int C, const ResArgs& a, hipStream_t stream) {
  if (a.lead && C == 16) return hipErrorInvalidValue;
  if (a.lead) return C == 32 ? bwd_c<32, true>(kind, g, a, stream) : bwd_c<64, true>(kind, g, a, stream);
  return C == 16 ? bwd_c<16, false>(kind, g, a, stream) : C == 32 ? bwd_c<32, false>(kind, g, a, stream) : bwd_c<64, false>(kind, g, a, stream);
}

}  // namespace hpf
