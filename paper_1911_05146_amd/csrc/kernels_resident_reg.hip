// Image-resident kernels whose residual stream lives in registers (bf16 mode): bottleneck runs on 16 x 16 images.
//
// Ownership and exchange are those of kernels_resident.hip: one work-group keeps "its" image for a whole run of identity
// blocks, the BatchNorm records of a micro-batch are all-gathered through tagged words in device memory.  What differs is
// where the tensors of a block live.  A wave owns two image rows (two 16-pixel MFMA tiles) for the whole run and keeps
// their residual stream, all channels, in the layout of an MFMA result: lane (fr, fq) holds channels nt*16 + fq*4 + 0..3 of
// pixel fr.  Two neighbouring 16-channel tiles of that layout ARE the second operand of the next 1x1 convolution if its
// reduction runs over the channels in the order (tile, fq, element); the weight matrices are staged into LDS with their
// columns permuted to match.  So the 1x1 convolutions read no activations from LDS, the shortcut is the initial value
// of the accumulators, BatchNorm statistics are taken from registers, and only the operand of the 3x3 convolution goes
// through LDS (a canvas with a zero border: every filter tap is a constant offset).
//
// What bounds the LDS-tile form (20.8 us per 128-32 block forward on 256 images): 2 500 VALU and 200 LDS instructions per wave and
// block, 25 barriers, and exchanges whose records went through LDS twice.
// Measured on 256 images (8 micro-batches), per block, images in LDS tiles / now: forward 20.7 / 13.5 us (128-32) and 28.2 / 22.1 (128-64), backward
// 26.1 / 20.1 and 37.3 / 32.9.  What is left: three exchanges per direction (1.5 us each), the stores of the stash (24 MiB per block,
// 4 us at the memory's rate), and issue: 8 waves per CU leave the matrix cores idle while they do BatchNorm.  The backward of 128-64 blocks spills: 30 registers
// (92 bytes of scratch a lane), 34 (100) with few images, 74 (284) and 72 (280) with a lead.
//
// The block in front of a run that halves the image and doubles the channels (64 -> 128, projection) leads it in (LEAD): the same launch starts, or
// ends, with it.  Layer by layer it took about nine launches of 4 to 9 us a direction; here it adds 19 us forward (the whole input, 128 KiB an image,
// is read for BatchNorm 1) and backward.  Seven blocks of ResNet-1001 with one such block, 13 images, one call per micro-batch: 1257 -> 1055 us for
// five micro-batches.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "hpf_ahead.h"
#include "hpf_resident_reg.h"

namespace hpf {
namespace {

constexpr int RG_IMG = 16, RG_P = RG_IMG * RG_IMG, RG_CW = RG_IMG + 2;   // image edge, pixels, canvas edge
constexpr int RG_PTW = 2;                        // image rows (pixel tiles) per wave
constexpr int RG_NPX = RG_PTW * 16;              // pixels per wave

// 3x3 convolution of the wave's two image rows from the canvas: the four input rows serve both.  src: the canvas at
// (first row of the wave, fr, fk); FLIP: the data gradient (taps mirrored).
template <int MID, bool FLIP, class W2>
__device__ __forceinline__ void conv3x3_rows(const bf16_t* src, const bf16_t* w2, floatx4 (&acc)[RG_PTW][MID / 16]) {
  constexpr int MS = MID + 8, NT = MID / 16;
#pragma unroll
  for (int s = 0; s < 3; ++s) {
#pragma unroll
    for (int ks = 0; ks < MID / 32; ++ks) {
      keep_order();
      bf16x8 px[4];
#pragma unroll
      for (int ir = 0; ir < 4; ++ir) px[ir] = *reinterpret_cast<const bf16x8*>(src + (ir * RG_CW + s) * MS + ks * 32);
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        const int tap = FLIP ? (2 - r) * 3 + (2 - s) : r * 3 + s;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const bf16x8 wf = W2::get(w2, tap * (MID / 32) + ks, nt);
#pragma unroll
          for (int j = 0; j < RG_PTW; ++j) acc[j][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, px[j + r], acc[j][nt], 0, 0, 0);
        }
      }
    }
  }
}

// The block that leads a run in (LEAD): CI = C/2 channels on 32 x 32 pixels -> C on 16 x 16, its first convolution and the projection 1x1 with
// stride 2.  They read one input pixel in four, the class (0, 0) of the parities of row and column; the others count in BatchNorm 1 alone.  Tile
// 4*j + q of a wave: class q under row j of its output rows.
constexpr int RG_LT = 4 * RG_PTW;
template <int C>
struct LeadPx {
  static constexpr int CI = C / 2, NI = CI / 16;
  unsigned off;   // of the lane's place in the input image
  __device__ __forceinline__ LeadPx(int row0, int fr, int fq) : off(px_offset(2 * row0 * (2 * RG_IMG) + 2 * fr, CI, fq)) {}
  static constexpr int at(int t, int k) { return ((2 * (t >> 2) + ((t >> 1) & 1)) * (2 * RG_IMG) + (t & 1)) * CI + k * 32; }
  __device__ __forceinline__ void load(uint2 (&v)[NI], const bf16_t* g, int t) const {
#pragma unroll
    for (int k = 0; k < NI / 2; ++k) {
      const uint4 q = *reinterpret_cast<const uint4*>(g + at(t, k) + off);
      v[2 * k] = make_uint2(q.x, q.y);
      v[2 * k + 1] = make_uint2(q.z, q.w);
    }
  }
  static __device__ __forceinline__ void arrange(uint2 (&v)[NI]) {
#pragma unroll
    for (int k = 0; k < NI / 2; ++k) pair_swap(v[2 * k], v[2 * k + 1]);
  }
  __device__ __forceinline__ void store(bf16_t* g, int t, const uint2 (&v)[NI]) const {
#pragma unroll
    for (int k = 0; k < NI / 2; ++k) {
      uint2 e = v[2 * k], o = v[2 * k + 1];
      pair_swap(e, o);
      *reinterpret_cast<uint4*>(g + at(t, k) + off) = make_uint4(e.x, e.y, o.x, o.y);
    }
  }
};

template <int C, int S = 1>
struct Channels { static constexpr int value = C, pixels = S; };

template <int C, int MID, bool INFER>
constexpr int rg_fwd_lds() {
  using W1 = WStage<MID, C>;
  using W2 = WStage<MID, 9 * MID, 3>;
  using W3 = WStage<C, MID>;
  const int w13 = INFER ? W1::BYTES + W3::BYTES : (W1::BYTES > W3::BYTES ? W1::BYTES : W3::BYTES);
  return RG_CW * RG_CW * (MID + 8) * 2 + W2::BYTES + w13 + (C + 2 * MID) * 8 + (INFER ? 0 : RG_NW * 2 * C * 4) + 16;
}

// FEW: micro-batches of up to eight images, which take one chunk of eight records (111 blocks of ResNet-1001, 8 images: 3.1 -> 2.85 ms both ways).  A branch
// for them in the one kernel cost the others 1 % in registers.
constexpr int RG_FEW = 8;

// Forward of a run.  INFER: BatchNorm by running statistics; nothing is exchanged or stashed, only the output of the last
// block is written.
// Barriers per block: 7 (training), 2 (inference).  The matrices of conv1 and conv3 take turns in one LDS area in training
// (conv1's is dead when conv3's is staged, behind the barrier that ends conv1, and the other way round); conv2's of the next
// block is staged behind the barrier that ends conv2, in one piece (WHOLE) or in three, which 64 inner channels need to stay within the registers.
// Inference is bounded by latency (3.8 us per 128-32 block, of which the products take 0.9): every matrix and table is asked for as soon as the
// registers of the one before are free, a whole block ahead of its use, and the tables of the three BatchNorms are read by waves of their
// own.  Asked for within the block, the tables three dependent reads in one wave, 21 blocks took 95 us, now 80.
template <int C, int MID, bool INFER, bool LEAD, bool FEW>
__global__ void __launch_bounds__(RG_NT) k_reg_forward(const ResArgs a) {
  constexpr int MS = MID + 8, NC = C / 16, NM = MID / 16;
  using W1 = WStage<MID, C>;
  // Training of 128-32 blocks: conv2's matrix travels in one piece (12 registers), and the next block's matrices are asked for behind the polls of an exchange.
  // Ahead of them, in fragment order, they hold up its words: 21 blocks, 8 micro-batches of 32 / 16 images, 302 / 288 us, behind them 297 / 281 (with matrices in
  // row order, ahead of the polls, 294 / 283); 13 images, one micro-batch, 285 / 281; 8 micro-batches of 8 images 257 / 252.
  constexpr bool WHOLE = !INFER && MID == 32;
  using W2 = WStage<MID, 9 * MID, INFER || WHOLE ? 1 : 3>;
  using W3 = WStage<C, MID>;
  const int tid = threadIdx.x, lane = tid & 63, wave = wave_index();
  const int fr = lane & 15, fq = lane >> 4, fk = fq * 8;
  const int z = blockIdx.x % a.ngroup, me = blockIdx.x / a.ngroup;   // with g == 8 micro-batch z lives on XCD z
  ResCtx cx{(char*)pick(a.base, z), pick(a.act_in, z), pick(a.act_out, z), nullptr, nullptr};
  u64* xchg = reinterpret_cast<u64*>(cx.base + a.xchg_off);
  unsigned* tagp = reinterpret_cast<unsigned*>(cx.base + a.tag_off);
  const unsigned tag0 = INFER ? 0u : *tagp;
  unsigned phase = 0;
  auto slot = [&]() { return xchg + (size_t)(phase & 1u) * resident_slot_members(a.nmem) * (2 * C); };

  extern __shared__ __align__(16) unsigned char smem[];
  bf16_t* canvas = reinterpret_cast<bf16_t*>(smem);
  bf16_t* sW2 = canvas + RG_CW * RG_CW * MS;
  bf16_t* sW1 = reinterpret_cast<bf16_t*>(reinterpret_cast<char*>(sW2) + W2::BYTES);
  bf16_t* sW3 = INFER ? reinterpret_cast<bf16_t*>(reinterpret_cast<char*>(sW1) + W1::BYTES) : sW1;
  float2* coefC = reinterpret_cast<float2*>(reinterpret_cast<char*>(sW1) +
                                            (INFER ? W1::BYTES + W3::BYTES : (W1::BYTES > W3::BYTES ? W1::BYTES : W3::BYTES)));
  float2* coefM = coefC + C;
  float2* coefM3 = coefM + MID;
  int* fail = reinterpret_cast<int*>(coefM3 + MID);
  float* red = reinterpret_cast<float*>(fail + 4);   // training: RG_NW x 2*C

  const int row0 = wave * RG_PTW;                                    // the wave's first image row
  const unsigned offC = px_offset(row0 * 16 + fr, C, fq), offM = px_offset(row0 * 16 + fr, MID, fq);
  auto image = [&](unsigned long long off, int CT) { return cx.tensor(off) + (size_t)me * (RG_P * CT); };
  bf16_t* const cv_w = canvas + ((row0 + 1) * RG_CW + fr + 1) * MS + fq * 4;   // where the lane writes
  const bf16_t* const cv_r = canvas + (row0 * RG_CW + fr) * MS + fk;           // tap (0, 0) of its reads
  const bf16_t* const w1r = sW1 + lane * 8;
  const bf16_t* const w2r = sW2 + lane * 8;
  const bf16_t* const w3r = sW3 + lane * 8;

  W1 w1; W2 w2; W3 w3;
  floatx4 X[RG_PTW][NC];
  auto stage_w2 = [&](const bf16_t* g) {   // training: of the first block
    w2.template issue<0>(g, wave, fr, fq); w2.template commit<0>(sW2, wave, lane);
    if constexpr (!WHOLE) {
      w2.template issue<1>(g, wave, fr, fq); w2.template commit<1>(sW2, wave, lane);
      w2.template issue<2>(g, wave, fr, fq); w2.template commit<2>(sW2, wave, lane);
    }
  };
  // Inference: the coefficients of a block, one channel per thread: waves 0 .. C/64 - 1 take the first BatchNorm, the next two waves the others.
  static_assert(C / 64 + 2 <= RG_NW && MID <= 64, "a channel per lane");
  float rc_mean, rc_var, rc_gamma, rc_beta;
  const int tq = wave < C / 64 ? 0 : wave - C / 64 + 1, tc = tq == 0 ? tid : lane;
  const bool t_on = tq == 0 || (tq < 3 && lane < MID);
  float2* const t_dst = coefC + (tq == 0 ? 0 : tq == 1 ? C : C + MID);
  const int last = a.nblk - 1;
  struct { unsigned long long w1, w2, w3, run, gamma, beta; } nx;   // offsets of what is asked for next
  auto next_offsets = [&](int b01, int b2) {   // matrices and tables of the first two convolutions of block b01, of the third of block b2
    const ResBlock *t01 = a.blocks + b01, *t2 = a.blocks + (b2 < last ? b2 : last);
    nx.w1 = t01->wf_off[0];
    nx.w2 = t01->wf_off[1];
    nx.w3 = t2->wf_off[2];
    const ResBlock* t = tq < 2 ? t01 : t2;
    const int q = tq < 3 ? tq : 2;
    nx.run = t->run_off[q];
    nx.gamma = t->gamma_off[q];
    nx.beta = t->beta_off[q];
  };
  constexpr int CI = LEAD ? LeadPx<C>::CI : C;   // channels of the run's input
  int n0 = CI;                                   // channels of the first BatchNorm of the block
  auto load_coef = [&] {
    if (!t_on || (LEAD && tq == 0 && tc >= n0)) return;
    const float* run = a.running + nx.run;
    rc_mean = run[tc];
    rc_var = run[(tq == 0 ? (LEAD ? n0 : C) : MID) + tc];
    rc_gamma = (a.params + nx.gamma)[tc];
    rc_beta = (a.params + nx.beta)[tc];
  };
  auto store_coef = [&] {
    if (t_on && (!LEAD || tq > 0 || tc < n0)) t_dst[tc] = bn_scale_shift(rc_mean, 1.0f / sqrtf(rc_var + a.eps), rc_gamma, rc_beta);
  };
  const float inv_n = 1.f / (float)a.nmem;
  // training: statistics of the wave's values v -> coef of the BatchNorm q of block B; `late` runs behind the polls.  Returns false when a
  // partner did not show up.
  auto exchange = [&](auto cc, const auto& v, const ResBlock& B, int q, float2* coef, auto&& late) -> bool {
    constexpr int Cc = decltype(cc)::value, S = decltype(cc)::pixels;   // S: pixels per pixel of a block's output
    const int gc = gather_channel<Cc>(wave, lane);
    const float gamma = (a.params + B.gamma_off[q])[gc], beta = (a.params + B.beta_off[q])[gc];
    stats_wave(v, red + wave * 2 * Cc, Cc, fr, fq);
    __syncthreads();
    const unsigned tag = tag0 + 1u + phase;
    stats_publish_waves<Cc, S * RG_NPX>(red, slot(), me, tag);
    const StatsOut o{coef, me == 0 ? reinterpret_cast<float*>(cx.base + B.stats_off[q]) : nullptr};
    collect_stats<Cc, FEW ? 8 : 32>(slot(), a.nmem, tag, inv_n, (float)(S * RG_P), a.eps, gamma, beta, o, wave, lane, fail);
    ++phase;
    late();
    __syncthreads();
    if (*fail) {
      if (tid == 0) atomicExch(a.abort_flag, 1);
      return false;
    }
    return true;
  };
  using IC = Channels<C>;
  using IM = Channels<MID>;
  floatx4 acc0[RG_PTW][NM];   // conv1 of the lead
  if constexpr (LEAD) {
    using LP = LeadPx<C>;
    using WL1 = WStage<MID, CI>;
    using WLP = WStage<C, CI>;
    constexpr int NI = LP::NI;
    static_assert(WLP::BYTES <= RG_CW * RG_CW * MS * 2 && WL1::BYTES <= W1::BYTES, "the lead's matrices lie where the canvas and conv1's will");
    const LP lp(row0, fr, fq);
    const ResBlock T = a.blocks[0];
    const bf16_t* x = cx.tensor(T.x_off) + (size_t)me * (4 * RG_P * CI);
    WL1 l1;
    WLP lw;
    uint2 px[RG_LT][NI];
    l1.issue(a.packed + T.wf_off[0], wave, fr, fq);
    lw.issue(a.packed + T.pf_off, wave, fr, fq);
#pragma unroll
    for (int t = 0; t < RG_LT; t += INFER ? 4 : 1) lp.load(px[t], x, t);
    if constexpr (INFER) {
      next_offsets(0, 0);
      w2.issue(a.packed + nx.w2, wave, fr, fq);
      w3.issue(a.packed + nx.w3, wave, fr, fq);
      load_coef();
    }
    if (tid == 0) *fail = 0;
    l1.commit(sW1, wave, lane);
    lw.commit(canvas, wave, lane);
    if constexpr (INFER) {
      w2.commit(sW2, wave, lane);
      store_coef();
      n0 = C;
      if (const int b = block_ahead(true, 0, 1, a.nblk); b > 0) {
        next_offsets(b, 0);
        w1.issue(a.packed + nx.w1, wave, fr, fq);
        w2.issue(a.packed + nx.w2, wave, fr, fq);
        load_coef();
      }
    } else {
      stage_w2(a.packed + T.wf_off[1]);
    }
#pragma unroll
    for (int t = 0; t < RG_LT; t += INFER ? 4 : 1) LP::arrange(px[t]);
    __syncthreads();
    if constexpr (!INFER) {
      if (!exchange(Channels<CI, 4>{}, px, T, 0, coefC, [] {})) return;
    }
    // ---- conv1 (CI -> MID) and the projection (CI -> C), on relu(bn1(x)) of the pixels of class (0, 0)
#pragma unroll
    for (int j = 0; j < RG_PTW; ++j) {
#pragma unroll
      for (int nt = 0; nt < NM; ++nt) acc0[j][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int nt = 0; nt < NC; ++nt) X[j][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int ks = 0; ks < CI / 32; ++ks) {
      bf16x8 bf[RG_PTW];
#pragma unroll
      for (int j = 0; j < RG_PTW; ++j)
        bf[j] = frag_of(bn_relu_pack(unpack4(px[4 * j][2 * ks]), coefC + 2 * ks * 16 + fq * 4), bn_relu_pack(unpack4(px[4 * j][2 * ks + 1]), coefC + (2 * ks + 1) * 16 + fq * 4));
#pragma unroll
      for (int nt = 0; nt < NM; ++nt) {
        const bf16x8 wf = WL1::get(w1r, ks, nt);
#pragma unroll
        for (int j = 0; j < RG_PTW; ++j) acc0[j][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, bf[j], acc0[j][nt], 0, 0, 0);
      }
#pragma unroll
      for (int nt = 0; nt < NC; ++nt) {
        const bf16x8 wf = WLP::get(canvas + lane * 8, ks, nt);
#pragma unroll
        for (int j = 0; j < RG_PTW; ++j) X[j][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, bf[j], X[j][nt], 0, 0, 0);
      }
    }
#pragma unroll
    for (int j = 0; j < RG_PTW; ++j)
#pragma unroll
      for (int nt = 0; nt < NC; ++nt) X[j][nt] = unpack4(pack4(X[j][nt]));   // the shortcut is a tensor of its own
    __syncthreads();
    for (int i = tid; i < RG_CW * RG_CW * MS / 8; i += RG_NT) reinterpret_cast<u32x4*>(canvas)[i] = u32x4{0u, 0u, 0u, 0u};
    __syncthreads();
  } else {
    const ResBlock B0 = a.blocks[0];
    w1.issue(a.packed + B0.wf_off[0], wave, fr, fq);
    if constexpr (INFER) {
      next_offsets(0, 0);
      w2.issue(a.packed + nx.w2, wave, fr, fq);
      w3.issue(a.packed + nx.w3, wave, fr, fq);
      load_coef();
    }
    for (int i = tid; i < RG_CW * RG_CW * MS / 8; i += RG_NT) reinterpret_cast<u32x4*>(canvas)[i] = u32x4{0u, 0u, 0u, 0u};
    if (tid == 0) *fail = 0;
    uint2 q[RG_PTW][NC];
    px_load(q, image(B0.x_off, C), offC);
    px_arrange(q);
#pragma unroll
    for (int j = 0; j < RG_PTW; ++j)
#pragma unroll
      for (int nt = 0; nt < NC; ++nt) X[j][nt] = unpack4(q[j][nt]);
    w1.commit(sW1, wave, lane);
    if constexpr (INFER) {
      w2.commit(sW2, wave, lane);
      store_coef();
      next_offsets(block_ahead(false, 0, 1, a.nblk), 0);
      w1.issue(a.packed + nx.w1, wave, fr, fq);   // w3 and the table of the third BatchNorm are kept for the first block, where they are staged
      w2.issue(a.packed + nx.w2, wave, fr, fq);
      load_coef();
    } else {
      stage_w2(a.packed + B0.wf_off[1]);
    }
    __syncthreads();
    if constexpr (!INFER) {
      if (!exchange(IC{}, X, a.blocks[0], 0, coefC, [] {})) return;
    }
  }
  if constexpr (LEAD) {
    constexpr bool LD = true;
    const int bi = 0;
#include "resident_reg_forward_block.inl"
  }
  for (int bi = LEAD ? 1 : 0; bi < a.nblk; ++bi) {
    constexpr bool LD = false;
#include "resident_reg_forward_block.inl"
  }
  // every member has read the counter before it took part in the first exchange, which member 0 has left
  if (!INFER && me == 0 && tid == 0) *tagp = tag0 + phase;
}

// ------------------------------------------------------------------------------------------ backward
template <int C, int MID>
constexpr int rg_bwd_lds() {
  using W3 = WStage<MID, C>;
  using W2 = WStage<MID, 9 * MID, 3>;
  using W1 = WStage<C, MID>;
  return RG_CW * RG_CW * (MID + 8) * 2 + W2::BYTES + (W1::BYTES > W3::BYTES ? W1::BYTES : W3::BYTES) + (4 * (C + 2 * MID) + 3 * C) * 4 +
         RG_NW * 2 * C * 4 + 16;
}

// Backward of a run: the same ownership, walking the blocks in reverse with the gradient of the residual stream in
// registers (packed).  c1, c2 and x of a block are read straight into the register layout, each behind the polls of an exchange
// well ahead of its use; what leaves (dc2, dc1, gx) is stored behind the polls of the exchange after.
template <int C, int MID, bool LEAD, bool FEW>
__global__ void __launch_bounds__(RG_NT) k_reg_backward(const ResArgs a) {
  constexpr int MS = MID + 8, NC = C / 16, NM = MID / 16;
  using W3 = WStage<MID, C>;           // conv3 data gradient [MID][C]
  using W2 = WStage<MID, 9 * MID, 3>;    // conv2 data gradient [MID][9*MID]
  using W1 = WStage<C, MID>;           // conv1 data gradient [C][MID]
  const int tid = threadIdx.x, lane = tid & 63, wave = wave_index();
  const int fr = lane & 15, fq = lane >> 4, fk = fq * 8;
  const int z = blockIdx.x % a.ngroup, me = blockIdx.x / a.ngroup;   // with g == 8 micro-batch z lives on XCD z
  ResCtx cx{(char*)pick(a.base, z), pick(a.act_in, z), pick(a.act_out, z), pick(a.err_in, z), pick(a.err_out, z)};
  u64* xchg = reinterpret_cast<u64*>(cx.base + a.xchg_off);
  unsigned* tagp = reinterpret_cast<unsigned*>(cx.base + a.tag_off);
  const unsigned tag0 = *tagp;
  unsigned phase = 0;
  auto slot = [&]() { return xchg + (size_t)(phase & 1u) * resident_slot_members(a.nmem) * (2 * C); };

  extern __shared__ __align__(16) unsigned char smem[];
  bf16_t* canvas = reinterpret_cast<bf16_t*>(smem);
  bf16_t* sW2 = canvas + RG_CW * RG_CW * MS;
  bf16_t* sW13 = reinterpret_cast<bf16_t*>(reinterpret_cast<char*>(sW2) + W2::BYTES);
  float* cf1 = reinterpret_cast<float*>(reinterpret_cast<char*>(sW13) + (W1::BYTES > W3::BYTES ? W1::BYTES : W3::BYTES));
  float* cf2 = cf1 + 4 * C;
  float* cf3 = cf2 + 4 * MID;
  float* tab = cf3 + 4 * MID;
  int* fail = reinterpret_cast<int*>(tab + 3 * C);
  float* red = reinterpret_cast<float*>(fail + 4);

  const int row0 = wave * RG_PTW;
  const unsigned offC = px_offset(row0 * 16 + fr, C, fq), offM = px_offset(row0 * 16 + fr, MID, fq);
  auto image = [&](unsigned long long off, int CT) { return cx.tensor(off) + (size_t)me * (RG_P * CT); };
  bf16_t* const cv_w = canvas + ((row0 + 1) * RG_CW + fr + 1) * MS + fq * 4;
  const bf16_t* const cv_r = canvas + (row0 * RG_CW + fr) * MS + fk;
  const bf16_t* const w3r = sW13 + lane * 8;
  const bf16_t* const w2r = sW2 + lane * 8;
  const bf16_t* const w1r = sW13 + lane * 8;
  const float inv_M = 1.f / ((float)a.nmem * (float)RG_P);

  W3 w3; W2 w2; W1 w1;
  uint2 DY[RG_PTW][NC], xc2[RG_PTW][NM], xc1[RG_PTW][NM], xx[RG_PTW][NC];
  // the tables of a block: waves 0 .. C/64 - 1 take the channels of the first, the next two waves the others'
  static_assert(C / 64 + 2 <= RG_NW && MID <= 64, "a channel per lane");
  CfRegs tb;
  const int tq = wave < C / 64 ? 0 : wave - C / 64 + 1, tc = tq == 0 ? tid : lane;
  float* const t_dst = tq == 0 ? cf1 : tq == 1 ? cf2 : cf3;
  const bool t_on = tq == 0 || (tq < 3 && lane < MID);
  int n0 = C;   // channels of the first BatchNorm (the lead's has C/2)
  auto load_tables = [&](int bi) {   // tq is uniform: the offsets come by scalar loads from the table of blocks
    if (LEAD && bi == 0) n0 = C / 2;
    if (t_on && (!LEAD || tq > 0 || tc < n0)) {
      const ResBlock* t = a.blocks + bi;
      tb.load(reinterpret_cast<const float*>(cx.base + t->stats_off[tq]), a.params + t->gamma_off[tq], a.params + t->beta_off[tq], tc, tq == 0 ? n0 : MID);
    }
  };
  auto store_tables = [&] {
    if (t_on && (!LEAD || tq > 0 || tc < n0)) tb.store(t_dst, tc, tq == 0 ? n0 : MID);
  };
  {
    const ResBlock BL = a.blocks[a.nblk - 1];
    w3.issue(a.packed + BL.wd_off[2], wave, fr, fq);
    load_tables(a.nblk - 1);
    for (int i = tid; i < RG_CW * RG_CW * MS / 8; i += RG_NT) reinterpret_cast<u32x4*>(canvas)[i] = u32x4{0u, 0u, 0u, 0u};
    if (tid == 0) *fail = 0;
    px_load(DY, image(BL.gy_off, C), offC);
    px_arrange(DY);
    px_load(xc2, image(BL.c2_off, MID), offM);
    w3.commit(sW13, wave, lane);
    {
      const bf16_t* g = a.packed + BL.wd_off[1];
      w2.template issue<0>(g, wave, fr, fq); w2.template commit<0>(sW2, wave, lane);
      w2.template issue<1>(g, wave, fr, fq); w2.template commit<1>(sW2, wave, lane);
      w2.template issue<2>(g, wave, fr, fq); w2.template commit<2>(sW2, wave, lane);
    }
    store_tables();
  }
  __syncthreads();
  // exchange of the sums of a BatchNorm backward; `late` runs behind the polls.  lead: S = 4 input pixels per output pixel, and its BatchNorm parameter
  // gradients are added here, as the run's weight-gradient launch does not know of it
  auto exchange = [&](auto cc, auto lead, auto& dz, const auto& x, const float* cf, const ResBlock& B, int q, auto&& late) -> bool {
    constexpr int Cc = decltype(cc)::value;
    constexpr bool ld = decltype(lead)::value;
    const CfChannel ck(cf, gather_channel<Cc>(wave, lane), Cc);
    bwd_sums_wave(dz, x, cf, red + wave * 2 * Cc, Cc, fr, fq);
    __syncthreads();
    const unsigned tag = tag0 + 1u + phase;
    sums_publish_waves<Cc>(red, slot(), me, tag);
    collect_bwd<Cc, FEW ? 8 : (Cc == C ? 16 : 1024 / MID)>(slot(), a.nmem, tag, ld && q == 0 ? 0.25f * inv_M : inv_M, ck, tab,
                                                  !ld && me == 0 ? reinterpret_cast<float*>(cx.base + B.dgb_off[q]) : nullptr, wave, lane, fail,
                                                  ld && me == 0 ? a.grads + B.beta_off[q] : nullptr, a.grads + B.gamma_off[q]);
    ++phase;
    late();
    __syncthreads();
    if (*fail) {
      if (tid == 0) atomicExch(a.abort_flag, 1);
      return false;
    }
    return true;
  };
  using IC = std::integral_constant<int, C>;
  using IM = std::integral_constant<int, MID>;
  for (int bi = a.nblk - 1; bi >= (LEAD ? 1 : 0); --bi) {
    constexpr bool LD = false;
#include "resident_reg_backward_block.inl"
  }
  if constexpr (LEAD) {
    constexpr bool LD = true;
    const int bi = 0;
#include "resident_reg_backward_block.inl"
  } else {
    px_store<MID == 32>(image(a.blocks[0].gx_off, C), offC, DY);
  }
  if (me == 0 && tid == 0) *tagp = tag0 + phase;
}

template <class K>
hipError_t launch_reg(K kernel, int lds, int g, const ResArgs& a, hipStream_t stream) {
  ResArgs b = a;
  b.ngroup = g;
  kernel<<<dim3((unsigned)(a.nmem * g)), RG_NT, (size_t)lds, stream>>>(b);
  return hipGetLastError();
}

}  // namespace

bool resident_reg_shape(int kind, int C, int MID, int H, int W) {
  return kind == 1 && ((C == 128 && (MID == 32 || MID == 64) && H == RG_IMG && W == RG_IMG) || (C == 256 && MID == 64 && H == 8 && W == 8));
}
template <int MID, bool LEAD>
static hipError_t prepare_m() {
  const void* const kernels[] = {reinterpret_cast<const void*>(k_reg_forward<128, MID, false, LEAD, false>), reinterpret_cast<const void*>(k_reg_forward<128, MID, false, LEAD, true>),
                                 reinterpret_cast<const void*>(k_reg_forward<128, MID, true, LEAD, false>),
                                 reinterpret_cast<const void*>(k_reg_backward<128, MID, LEAD, false>), reinterpret_cast<const void*>(k_reg_backward<128, MID, LEAD, true>)};
  for (const void* f : kernels) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}
hipError_t resident_reg_prepare() {
  hipError_t e = prepare_m<32, false>();
  if (e == hipSuccess) e = prepare_m<64, false>();
  if (e == hipSuccess) e = prepare_m<32, true>();
  if (e == hipSuccess) e = prepare_m<64, true>();
  if (e == hipSuccess) e = resident_reg8_prepare();
  return e;
}
template <int MID, bool INFER, bool LEAD>
static hipError_t forward_l(int g, const ResArgs& a, hipStream_t stream) {
  constexpr int lds = rg_fwd_lds<128, MID, INFER>();
  if constexpr (!INFER)
    if (a.nmem <= RG_FEW) return launch_reg(k_reg_forward<128, MID, false, LEAD, true>, lds, g, a, stream);
  return launch_reg(k_reg_forward<128, MID, INFER, LEAD, false>, lds, g, a, stream);
}
template <int MID, bool INFER>
static hipError_t forward_m(int g, const ResArgs& a, hipStream_t stream) {
  return a.lead ? forward_l<MID, INFER, true>(g, a, stream) : forward_l<MID, INFER, false>(g, a, stream);
}
template <int MID, bool LEAD>
static hipError_t backward_l(int g, const ResArgs& a, hipStream_t stream) {
  return a.nmem <= RG_FEW ? launch_reg(k_reg_backward<128, MID, LEAD, true>, rg_bwd_lds<128, MID>(), g, a, stream)
                          : launch_reg(k_reg_backward<128, MID, LEAD, false>, rg_bwd_lds<128, MID>(), g, a, stream);
}
template <int MID>
static hipError_t backward_m(int g, const ResArgs& a, hipStream_t stream) {
  return a.lead ? backward_l<MID, true>(g, a, stream) : backward_l<MID, false>(g, a, stream);
}
hipError_t launch_reg_forward(int g, int C, int MID, const ResArgs& a, hipStream_t stream) {
  if (C == 256) return launch_reg8_forward(g, a, stream);
  return MID == 32 ? forward_m<32, false>(g, a, stream) : forward_m<64, false>(g, a, stream);
}
hipError_t launch_reg_backward(int g, int C, int MID, const ResArgs& a, hipStream_t stream) {
  if (C == 256) return launch_reg8_backward(g, a, stream);
  return MID == 32 ? backward_m<32>(g, a, stream) : backward_m<64>(g, a, stream);
}
hipError_t launch_reg_inference(int g, int C, int MID, const ResArgs& a, hipStream_t stream) {
  if (C == 256) return launch_reg8_inference(g, a, stream);
  return MID == 32 ? forward_m<32, true>(g, a, stream) : forward_m<64, true>(g, a, stream);
}
static_assert(rg_bwd_lds<128, 64>() <= 160 * 1024 && rg_fwd_lds<128, 64, false>() <= 160 * 1024 && rg_fwd_lds<128, 64, true>() <= 160 * 1024, "LDS of a CU");

}  // namespace hpf
