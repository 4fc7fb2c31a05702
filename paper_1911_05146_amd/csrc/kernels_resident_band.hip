// Image-resident kernels of runs whose image is cut into row bands, in registers (bf16 mode): 64-16 bottlenecks on 32 x 32 images, the first stage of
// ResNet-1001.
//
// An image is cut into four bands of eight rows, one work-group each; in NHWC a band is a contiguous range of 256 pixels, so every tensor of
// a band lies at member * 256 * channels like an image of kernels_resident_reg.hip, whose layout and exchange these kernels have: a wave owns one image
// row (two 16-pixel tiles) for the whole run, the 1x1 convolutions read registers, the 3x3 one a canvas in LDS with a border.  The members of
// an exchange are the bands of all images of the micro-batch.
// The 3x3 convolution needs the image rows above and below the band.  They travel with the exchange that lies ahead of it anyway: the waves
// of the first and the last row publish them as tagged words (forward c1 in bf16, two values a word; backward the masked gradient in fp32, to which
// the neighbour applies the BatchNorm map itself), and those of the facing rows collect them, in the same register layout.
// Sixteen channels fill half a reduction step: the 3x3 convolution takes two taps a step (conv3x3<16>), the convolution out of 16 channels runs
// against columns of zeros.
//
// Bound by the exchanges: the products of a block are under 0.2 us.  111 blocks of ResNet-1001, 8 micro-batches of 8 images, us per block, before (bands
// in LDS tiles, records gathered there) and now: forward 15.0 / 10.1, backward 18.2 / 12.8.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "hpf_resident_reg.h"

namespace hpf {
namespace {

constexpr int RB_C = 64, RB_MID = 16, RB_W = 32, RB_ROWS = 8, RB_BANDS = 4, RB_P = RB_W * RB_ROWS;
constexpr int RB_PT = 2, RB_NC = RB_C / 16, RB_NPX = RB_PT * 16;           // pixel tiles, channel tiles and pixels of a wave
constexpr int RB_CW = RB_W + 2, RB_MS = RB_MID + 8;                         // canvas row, pixel pitch
constexpr int RB_HALO = RB_W * RB_MID;                                      // words of a row (backward; forward half as many)
static_assert(RB_ROWS == RG_NW, "a wave per image row");
using RBDown = WStage<RB_MID, RB_C>;                // conv1 | conv3's data gradient
using RB3x3 = WStage<RB_MID, 160>;                  // nine taps of 16 channels, padded
using RBUp = WStage<RB_C, 32>;                      // conv3 | conv1's data gradient, 16 columns and 16 of zeros
constexpr int RB_CANVAS = (RB_ROWS + 2) * RB_CW * RB_MS * 2;
constexpr int RB_LDS = RB_CANVAS + RBDown::BYTES + RB3x3::BYTES + RBUp::BYTES + 16 + RG_NW * 2 * RB_C * 4;
constexpr int RB_FWD_LDS = RB_LDS + (RB_C + 2 * RB_MID) * 8, RB_BWD_LDS = RB_LDS + (4 * (RB_C + 2 * RB_MID) + 3 * RB_C) * 4;

__host__ __device__ constexpr size_t band_slot_words(int members) { return (size_t)((members + 31) / 32 * 32) * 2 * RB_C + (size_t)members * 2 * RB_HALO; }

// 3x3 convolution of the wave's row.  src: the canvas at the lane's pixel of the first tile, tap (0, 0), + (fq & 1)*8; zero: eight zeros; FLIP: taps mirrored
template <bool FLIP>
__device__ __forceinline__ void band_conv(const bf16_t* src, const bf16_t* zero, const bf16_t* w, int fq, floatx4 (&acc)[RB_PT][1]) {
#pragma unroll
  for (int j = 0; j < RB_PT; ++j) acc[j][0] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int st = 0; st < 5; ++st) {
    constexpr int last = 8;
    const int ta = 2 * st, tb = 2 * st + 1 > last ? last : 2 * st + 1;
    const int oa = FLIP ? (2 - ta / 3) * RB_CW + 2 - ta % 3 : ta / 3 * RB_CW + ta % 3, ob = FLIP ? (2 - tb / 3) * RB_CW + 2 - tb % 3 : tb / 3 * RB_CW + tb % 3;
    const bf16_t* q = src + (fq < 2 ? oa : ob) * RB_MS;
    const bf16x8 wf = RB3x3::get(w, st, 0);
#pragma unroll
    for (int j = 0; j < RB_PT; ++j) {
      const bf16_t* px = 2 * st == last && fq >= 2 ? zero : q + j * 16 * RB_MS;   // no tap there: zeros, not another tap's values times the zero weights
      acc[j][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, *reinterpret_cast<const bf16x8*>(px), acc[j][0], 0, 0, 0);
    }
  }
}
__device__ __forceinline__ bf16x8 half_frag(const uint2& v) { return frag_of(v, make_uint2(0u, 0u)); }

// N words per lane of a row, to and from a place in the slot
template <int N>
__device__ __forceinline__ void row_publish(u64* at, const unsigned (&v)[N], int lane, unsigned tag) {
#pragma unroll
  for (int i = 0; i < N; ++i) __hip_atomic_store(at + i * 64 + lane, ((u64)tag << 32) | (u64)v[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <int N>
__device__ __forceinline__ void row_collect(unsigned (&v)[N], const u64* at, int lane, unsigned tag, int* fail) {
  SpinBudget budget;
  for (;;) {
    u64 q[N];
    bool ok = true;
#pragma unroll
    for (int i = 0; i < N; ++i) q[i] = __hip_atomic_load(at + i * 64 + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int i = 0; i < N; ++i) { ok = ok && (unsigned)(q[i] >> 32) == tag; v[i] = (unsigned)q[i]; }
    if (__all(ok)) break;
    if (!budget.again()) { *fail = 1; break; }
  }
}

// what both directions need of a lane's place
struct BandLane {
  int tid, lane, wave, fr, fq, z, me, nwg;
  int facing;                  // the member whose row lies next to this wave's: waves 0 and 7, else -1
  unsigned offC, offM;
  int cw, cr, ch;              // canvas: where it writes, tap (0, 0) of its reads, where the facing row goes
  __device__ __forceinline__ explicit BandLane(const ResArgs& a) {
    tid = threadIdx.x; lane = tid & 63; wave = wave_index(); fr = lane & 15; fq = lane >> 4;
    z = blockIdx.x % a.ngroup; me = blockIdx.x / a.ngroup; nwg = a.nmem * RB_BANDS;
    const int band = me % RB_BANDS;
    facing = wave == 0 && band > 0 ? me - 1 : wave == RG_NW - 1 && band < RB_BANDS - 1 ? me + 1 : -1;
    offC = px_offset(wave * RB_W + fr, RB_C, fq);
    offM = (unsigned)((wave * RB_W + fr) * RB_MID + fq * 4);
    cw = ((wave + 1) * RB_CW + fr + 1) * RB_MS + fq * 4;
    cr = (wave * RB_CW + fr) * RB_MS + (fq & 1) * 8;
    ch = ((wave == 0 ? 0 : RB_ROWS + 1) * RB_CW + fr + 1) * RB_MS + fq * 4;
  }
  // the row that this wave publishes, and the one that it collects
  __device__ __forceinline__ u64* row_out(u64* slot) const { return row(slot, me, wave == 0 ? 0 : 1); }
  __device__ __forceinline__ u64* row_in(u64* slot) const { return row(slot, facing, wave == 0 ? 1 : 0); }
  __device__ __forceinline__ u64* row(u64* slot, int m, int last) const {
    return slot + (size_t)resident_slot_members(nwg) * 2 * RB_C + (size_t)(2 * m + last) * RB_HALO;
  }
};

// FEW: micro-batches of up to four images, whose 16 bands are one chunk of records.  Eight blocks, us a step, chunks of 32 / 16: one image 172 / 164, four
// images 185 / 180.
constexpr int BAND_FEW = 16;

template <bool FEW>
__global__ void __launch_bounds__(RG_NT) k_band_forward(const ResArgs a) {
  constexpr int C = RB_C, MID = RB_MID;
  const BandLane L(a);
  const int tid = L.tid, lane = L.lane, wave = L.wave, fr = L.fr, fq = L.fq, me = L.me;
  ResCtx cx{(char*)pick(a.base, L.z), pick(a.act_in, L.z), pick(a.act_out, L.z), nullptr, nullptr};
  u64* xchg = reinterpret_cast<u64*>(cx.base + a.xchg_off);
  unsigned* tagp = reinterpret_cast<unsigned*>(cx.base + a.tag_off);
  const unsigned tag0 = *tagp;
  unsigned phase = 0;
  auto slot = [&]() { return xchg + (phase & 1u) * band_slot_words(L.nwg); };
  auto image = [&](unsigned long long off, int CT) { return cx.tensor(off) + (size_t)me * (RB_P * CT); };

  extern __shared__ __align__(16) unsigned char smem[];
  bf16_t* canvas = reinterpret_cast<bf16_t*>(smem);
  bf16_t* sW1 = reinterpret_cast<bf16_t*>(smem + RB_CANVAS);
  bf16_t* sW2 = reinterpret_cast<bf16_t*>(smem + RB_CANVAS + RBDown::BYTES);
  bf16_t* sW3 = reinterpret_cast<bf16_t*>(smem + RB_CANVAS + RBDown::BYTES + RB3x3::BYTES);
  int* fail = reinterpret_cast<int*>(smem + RB_CANVAS + RBDown::BYTES + RB3x3::BYTES + RBUp::BYTES);
  float* red = reinterpret_cast<float*>(fail + 4);
  float2* coefC = reinterpret_cast<float2*>(smem + RB_LDS);
  float2* coefM = coefC + C;
  float2* coefM3 = coefM + MID;

  RBDown w1; RB3x3 w2; RBUp w3;
  floatx4 X[RB_PT][RB_NC];
  const float inv_n = 1.f / (float)L.nwg;
  // statistics of the wave's values v -> coef of the BatchNorm q of block B; `late` runs behind the polls.  False: a partner did not show up
  auto exchange = [&](auto cc, const auto& v, const ResBlock& B, int q, float2* coef, auto&& late) -> bool {
    constexpr int Cc = decltype(cc)::value;
    const int gc = gather_channel<Cc>(wave, lane);
    const float gamma = (a.params + B.gamma_off[q])[gc], beta = (a.params + B.beta_off[q])[gc];
    stats_wave(v, red + wave * 2 * Cc, Cc, fr, fq);
    __syncthreads();
    const unsigned tag = tag0 + 1u + phase;
    stats_publish_waves<Cc, RB_NPX>(red, slot(), me, tag);
    const StatsOut o{coef, me == 0 ? reinterpret_cast<float*>(cx.base + B.stats_off[q]) : nullptr};
    collect_stats<Cc, FEW ? BAND_FEW : 32>(slot(), L.nwg, tag, inv_n, (float)RB_P, a.eps, gamma, beta, o, wave, lane, fail);
    late(tag);
    ++phase;
    __syncthreads();
    if (*fail) {
      if (tid == 0) atomicExch(a.abort_flag, 1);
      return false;
    }
    return true;
  };
  using IC = std::integral_constant<int, C>;
  using IM = std::integral_constant<int, MID>;
  {
    const ResBlock B0 = a.blocks[0];
    uint2 q[RB_PT][RB_NC];
    px_load(q, image(B0.x_off, C), L.offC);
    w1.issue(a.packed + B0.wf_off[0], wave, fr, fq);
    w2.issue(a.packed + B0.wf_off[1], wave, fr, fq);
    w3.issue(a.packed + B0.wf_off[2], wave, fr, fq);
    for (int i = tid; i < RB_CANVAS / 16; i += RG_NT) reinterpret_cast<u32x4*>(canvas)[i] = u32x4{0u, 0u, 0u, 0u};
    if (tid == 0) *fail = 0;
    px_arrange(q);
#pragma unroll
    for (int j = 0; j < RB_PT; ++j)
#pragma unroll
      for (int nt = 0; nt < RB_NC; ++nt) X[j][nt] = unpack4(q[j][nt]);
    w1.commit(sW1, wave, lane);
    w2.commit(sW2, wave, lane);
    w3.commit(sW3, wave, lane);
    __syncthreads();
    if (!exchange(IC{}, X, B0, 0, coefC, [](unsigned) {})) return;
  }
  for (int bi = 0; bi < a.nblk; ++bi) {
    const bool more = bi + 1 < a.nblk;
    const ResBlock B = a.blocks[bi], Bn = a.blocks[more ? bi + 1 : bi];
    // ---- conv1 (1x1, C -> MID) on relu(bn1(x))
    floatx4 acc[RB_PT][1];
#pragma unroll
    for (int j = 0; j < RB_PT; ++j) acc[j][0] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < C / 32; ++ks) {
      const bf16x8 wf = RBDown::get(sW1 + lane * 8, ks, 0);
#pragma unroll
      for (int j = 0; j < RB_PT; ++j) {
        const bf16x8 x = frag_of(bn_relu_pack(X[j][2 * ks], coefC + 2 * ks * 16 + fq * 4), bn_relu_pack(X[j][2 * ks + 1], coefC + (2 * ks + 1) * 16 + fq * 4));
        acc[j][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, x, acc[j][0], 0, 0, 0);
      }
    }
    uint2 cp[RB_PT][1], hp[RB_PT];   // hp: c1 of the facing row
#pragma unroll
    for (int j = 0; j < RB_PT; ++j) { cp[j][0] = pack4(acc[j][0]); acc[j][0] = unpack4(cp[j][0]); }
    if (L.facing >= 0) {
      const unsigned v[4] = {cp[0][0].x, cp[0][0].y, cp[1][0].x, cp[1][0].y};
      row_publish(L.row_out(slot()), v, lane, tag0 + 1u + phase);
    }
    if (!exchange(IM{}, acc, B, 1, coefM, [&](unsigned tag) {
          if (L.facing >= 0) {
            unsigned v[4];
            row_collect(v, L.row_in(slot()), lane, tag, fail);
            hp[0] = make_uint2(v[0], v[1]);
            hp[1] = make_uint2(v[2], v[3]);
          }
          px_store<false>(image(B.c1_off, MID), L.offM, cp);
        }))
      return;
#pragma unroll
    for (int j = 0; j < RB_PT; ++j) {
      *reinterpret_cast<uint2*>(canvas + L.cw + j * 16 * RB_MS) = bn_relu_pack(acc[j][0], coefM + fq * 4);
      if (L.facing >= 0) *reinterpret_cast<uint2*>(canvas + L.ch + j * 16 * RB_MS) = bn_relu_pack(unpack4(hp[j]), coefM + fq * 4);
    }
    __syncthreads();
    // ---- conv2 (3x3, MID -> MID)
    band_conv<false>(canvas + L.cr, canvas, sW2 + lane * 8, fq, acc);
#pragma unroll
    for (int j = 0; j < RB_PT; ++j) { cp[j][0] = pack4(acc[j][0]); acc[j][0] = unpack4(cp[j][0]); }
    if (!exchange(IM{}, acc, B, 2, coefM3, [&](unsigned) {
          w1.issue(a.packed + Bn.wf_off[0], wave, fr, fq);
          w2.issue(a.packed + Bn.wf_off[1], wave, fr, fq);
          px_store<false>(image(B.c2_off, MID), L.offM, cp);
        }))
      return;
    // ---- conv3 (1x1, MID -> C) on relu(bn3(c2)), accumulated onto x
    bf16x8 bf[RB_PT];
#pragma unroll
    for (int j = 0; j < RB_PT; ++j) bf[j] = half_frag(bn_relu_pack(acc[j][0], coefM3 + fq * 4));
#pragma unroll
    for (int nt = 0; nt < RB_NC; ++nt) {
      const bf16x8 wf = RBUp::get(sW3 + lane * 8, 0, nt);
#pragma unroll
      for (int j = 0; j < RB_PT; ++j) X[j][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, bf[j], X[j][nt], 0, 0, 0);
    }
    uint2 yp[RB_PT][RB_NC];
#pragma unroll
    for (int j = 0; j < RB_PT; ++j)
#pragma unroll
      for (int nt = 0; nt < RB_NC; ++nt) { yp[j][nt] = pack4(X[j][nt]); X[j][nt] = unpack4(yp[j][nt]); }
    if (!more) {
      px_store<false>(image(B.y_off, C), L.offC, yp);
      break;
    }
    w3.issue(a.packed + Bn.wf_off[2], wave, fr, fq);
    if (!exchange(IC{}, X, Bn, 0, coefC, [&](unsigned) {   // every wave is past the matrices of this block
          w1.commit(sW1, wave, lane);
          w2.commit(sW2, wave, lane);
          w3.commit(sW3, wave, lane);
          px_store<false>(image(B.y_off, C), L.offC, yp);
        }))
      return;
  }
  // every member has read the counter before it took part in the first exchange, which member 0 has left
  if (me == 0 && tid == 0) *tagp = tag0 + phase;
}

// The same ownership, walking the blocks in reverse with the gradient of the residual stream in registers (packed).  BatchNorm parameter gradients are
// added here: the run has no weight-gradient launch that knows of them.
template <bool FEW>
__global__ void __launch_bounds__(RG_NT) k_band_backward(const ResArgs a) {
  constexpr int C = RB_C, MID = RB_MID;
  const BandLane L(a);
  const int tid = L.tid, lane = L.lane, wave = L.wave, fr = L.fr, fq = L.fq, me = L.me;
  ResCtx cx{(char*)pick(a.base, L.z), pick(a.act_in, L.z), pick(a.act_out, L.z), pick(a.err_in, L.z), pick(a.err_out, L.z)};
  u64* xchg = reinterpret_cast<u64*>(cx.base + a.xchg_off);
  unsigned* tagp = reinterpret_cast<unsigned*>(cx.base + a.tag_off);
  const unsigned tag0 = *tagp;
  unsigned phase = 0;
  auto slot = [&]() { return xchg + (phase & 1u) * band_slot_words(L.nwg); };
  auto image = [&](unsigned long long off, int CT) { return cx.tensor(off) + (size_t)me * (RB_P * CT); };

  extern __shared__ __align__(16) unsigned char smem[];
  bf16_t* canvas = reinterpret_cast<bf16_t*>(smem);
  bf16_t* sW3 = reinterpret_cast<bf16_t*>(smem + RB_CANVAS);
  bf16_t* sW2 = reinterpret_cast<bf16_t*>(smem + RB_CANVAS + RBDown::BYTES);
  bf16_t* sW1 = reinterpret_cast<bf16_t*>(smem + RB_CANVAS + RBDown::BYTES + RB3x3::BYTES);
  int* fail = reinterpret_cast<int*>(smem + RB_CANVAS + RBDown::BYTES + RB3x3::BYTES + RBUp::BYTES);
  float* red = reinterpret_cast<float*>(fail + 4);
  float* cf1 = reinterpret_cast<float*>(smem + RB_LDS);
  float* cf2 = cf1 + 4 * C;
  float* cf3 = cf2 + 4 * MID;
  float* tab = cf3 + 4 * MID;

  RBDown w3; RB3x3 w2; RBUp w1;   // of the data gradients
  uint2 DY[RB_PT][RB_NC], xx[RB_PT][RB_NC], xc2[RB_PT][1], xc1[RB_PT][1], hx[RB_PT];   // hx: c2 of the facing row
  const float inv_M = 1.f / ((float)L.nwg * (float)RB_P);
  // the tables of a block: wave 0 takes the channels of the first BatchNorm, waves 1 and 2 the others'
  CfRegs tb;
  float* const t_dst = wave == 0 ? cf1 : wave == 1 ? cf2 : cf3;
  const bool t_on = wave == 0 || (wave < 3 && lane < MID);
  auto load_tables = [&](int bi) {
    if (!t_on) return;
    const ResBlock* t = a.blocks + bi;
    tb.load(reinterpret_cast<const float*>(cx.base + t->stats_off[wave]), a.params + t->gamma_off[wave], a.params + t->beta_off[wave], lane, wave == 0 ? C : MID);
  };
  auto store_tables = [&] { if (t_on) tb.store(t_dst, lane, wave == 0 ? C : MID); };
  auto load_c2 = [&](const ResBlock& B) {
    const bf16_t* g = image(B.c2_off, MID);
    px_load(xc2, g, L.offM);
    if (L.facing < 0) return;
    g += wave == 0 ? -RB_W * RB_MID : RB_W * RB_MID;   // a row up or down: the neighbouring band lies right there
#pragma unroll
    for (int j = 0; j < RB_PT; ++j) hx[j] = *reinterpret_cast<const uint2*>(g + j * 256 + L.offM);
  };
  // exchange of the sums of a BatchNorm backward; mid runs when dz is masked, `late` behind the polls
  auto exchange = [&](auto cc, auto& dz, const auto& x, const float* cf, const ResBlock& B, int q, auto&& mid, auto&& late) -> bool {
    constexpr int Cc = decltype(cc)::value;
    const CfChannel ck(cf, gather_channel<Cc>(wave, lane), Cc);
    const unsigned tag = tag0 + 1u + phase;
    bwd_sums_wave(dz, x, cf, red + wave * 2 * Cc, Cc, fr, fq);
    mid(tag);
    __syncthreads();
    sums_publish_waves<Cc>(red, slot(), me, tag);
    collect_bwd<Cc, FEW ? BAND_FEW : 32>(slot(), L.nwg, tag, inv_M, ck, tab, nullptr, wave, lane, fail, me == 0 ? a.grads + B.beta_off[q] : nullptr, a.grads + B.gamma_off[q]);
    late(tag);
    ++phase;
    __syncthreads();
    if (*fail) {
      if (tid == 0) atomicExch(a.abort_flag, 1);
      return false;
    }
    return true;
  };
  using IC = std::integral_constant<int, C>;
  using IM = std::integral_constant<int, MID>;
  {
    const ResBlock BL = a.blocks[a.nblk - 1];
    px_load(DY, image(BL.gy_off, C), L.offC);
    load_tables(a.nblk - 1);
    load_c2(BL);
    w3.issue(a.packed + BL.wd_off[2], wave, fr, fq);
    w2.issue(a.packed + BL.wd_off[1], wave, fr, fq);
    w1.issue(a.packed + BL.wd_off[0], wave, fr, fq);
    for (int i = tid; i < RB_CANVAS / 16; i += RG_NT) reinterpret_cast<u32x4*>(canvas)[i] = u32x4{0u, 0u, 0u, 0u};
    if (tid == 0) *fail = 0;
    px_arrange(DY);
    w3.commit(sW3, wave, lane);
    w2.commit(sW2, wave, lane);
    w1.commit(sW1, wave, lane);
    store_tables();
  }
  __syncthreads();
  for (int bi = a.nblk - 1; bi >= 0; --bi) {
    const bool more = bi > 0;
    const ResBlock B = a.blocks[bi], Bn = a.blocks[more ? bi - 1 : 0];
    // ---- conv3 data gradient, BN3 + ReLU backward -> dc2
    floatx4 acc[RB_PT][1], hz[RB_PT];   // hz: the masked gradient of the facing row
#pragma unroll
    for (int j = 0; j < RB_PT; ++j) acc[j][0] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < C / 32; ++ks) {
      const bf16x8 wf = RBDown::get(sW3 + lane * 8, ks, 0);
#pragma unroll
      for (int j = 0; j < RB_PT; ++j) acc[j][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, frag_of(DY[j][2 * ks], DY[j][2 * ks + 1]), acc[j][0], 0, 0, 0);
    }
    if (!exchange(IM{}, acc, xc2, cf3, B, 2,
                  [&](unsigned tag) {
                    if (L.facing < 0) return;
                    unsigned v[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[i] = __float_as_uint(acc[i >> 2][0][i & 3]);
                    row_publish(L.row_out(slot()), v, lane, tag);
                  },
                  [&](unsigned tag) {
                    if (L.facing >= 0) {
                      unsigned v[8];
                      row_collect(v, L.row_in(slot()), lane, tag, fail);
#pragma unroll
                      for (int i = 0; i < 8; ++i) hz[i >> 2][i & 3] = __uint_as_float(v[i]);
                    }
                    px_load(xc1, image(B.c1_off, MID), L.offM);
                    px_load(xx, image(B.x_off, C), L.offC);
                    if (bi + 1 < a.nblk) px_store<false>(image(a.blocks[bi + 1].gx_off, C), L.offC, DY);   // the gradient of the input of the block above
                  }))
      return;
    uint2 dcp[RB_PT][1];
#pragma unroll
    for (int j = 0; j < RB_PT; ++j) {
      dcp[j][0] = pack4(bwd_apply<MID>(acc[j][0], xc2[j][0], tab + fq * 4));
      *reinterpret_cast<uint2*>(canvas + L.cw + j * 16 * RB_MS) = dcp[j][0];
      if (L.facing >= 0) *reinterpret_cast<uint2*>(canvas + L.ch + j * 16 * RB_MS) = pack4(bwd_apply<MID>(hz[j], hx[j], tab + fq * 4));
    }
    __syncthreads();
    // ---- conv2 data gradient, BN2 + ReLU backward -> dc1
    band_conv<true>(canvas + L.cr, canvas, sW2 + lane * 8, fq, acc);
    if (!exchange(IM{}, acc, xc1, cf2, B, 1, [](unsigned) {}, [&](unsigned) {
          load_c2(Bn);
          load_tables(more ? bi - 1 : 0);
          w3.issue(a.packed + Bn.wd_off[2], wave, fr, fq);
          w2.issue(a.packed + Bn.wd_off[1], wave, fr, fq);
          px_store<false>(image(B.dc2_off, MID), L.offM, dcp);
        }))
      return;
#pragma unroll
    for (int j = 0; j < RB_PT; ++j) dcp[j][0] = pack4(bwd_apply<MID>(acc[j][0], xc1[j][0], tab + fq * 4));
    // ---- conv1 data gradient, BN1 + ReLU backward, plus the shortcut
    floatx4 da[RB_PT][RB_NC];
#pragma unroll
    for (int nt = 0; nt < RB_NC; ++nt) {
      const bf16x8 wf = RBUp::get(sW1 + lane * 8, 0, nt);
#pragma unroll
      for (int j = 0; j < RB_PT; ++j) da[j][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, half_frag(dcp[j][0]), floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    }
    px_arrange(xx);
    w1.issue(a.packed + Bn.wd_off[0], wave, fr, fq);
    if (!exchange(IC{}, da, xx, cf1, B, 0, [](unsigned) {}, [&](unsigned) {   // every wave is past the matrices and the tables of this block
          w3.commit(sW3, wave, lane);
          w2.commit(sW2, wave, lane);
          w1.commit(sW1, wave, lane);
          store_tables();
          px_store<false>(image(B.dc1_off, MID), L.offM, dcp);
        }))
      return;
#pragma unroll
    for (int nt = 0; nt < RB_NC; ++nt)
#pragma unroll
      for (int j = 0; j < RB_PT; ++j) DY[j][nt] = pack4(bwd_apply<C>(da[j][nt], xx[j][nt], tab + nt * 16 + fq * 4) + unpack4(DY[j][nt]));
  }
  px_store<false>(image(a.blocks[0].gx_off, C), L.offC, DY);
  if (me == 0 && tid == 0) *tagp = tag0 + phase;
}

hipError_t launch_band(void (*kernel)(const ResArgs), int lds, int g, const ResArgs& a, hipStream_t stream) {
  ResArgs b = a;
  b.ngroup = g;
  kernel<<<dim3((unsigned)(a.nmem * RB_BANDS * g)), RG_NT, (size_t)lds, stream>>>(b);
  return hipGetLastError();
}
static_assert(RB_FWD_LDS <= 64 * 1024 && RB_BWD_LDS <= 64 * 1024, "needs no raised limit");

}  // namespace

int resident_bands(int kind, int C, int MID, int H, int W) {
  return kind == 1 && C == RB_C && MID == RB_MID && H == RB_BANDS * RB_ROWS && W == RB_W ? RB_BANDS : 1;
}
size_t band_xchg_bytes(int members) { return 2 * band_slot_words(members) * sizeof(u64); }
hipError_t launch_band_forward(int g, const ResArgs& a, hipStream_t stream) {
  return launch_band(a.nmem * RB_BANDS <= BAND_FEW ? k_band_forward<true> : k_band_forward<false>, RB_FWD_LDS, g, a, stream);
}
hipError_t launch_band_backward(int g, const ResArgs& a, hipStream_t stream) {
  return launch_band(a.nmem * RB_BANDS <= BAND_FEW ? k_band_backward<true> : k_band_backward<false>, RB_BWD_LDS, g, a, stream);
}

}  // namespace hpf
