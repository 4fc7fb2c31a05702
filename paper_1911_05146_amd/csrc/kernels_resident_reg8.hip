// Image-resident kernels whose residual stream lives in registers (bf16 mode): 256-64 bottleneck runs on 8 x 8 images.
//
// Ownership of images and the exchange of BatchNorm records are those of kernels_resident.hip, the register layout that of
// kernels_resident_reg.hip.  Here the eight waves of a work-group divide the CHANNELS: a wave keeps 32 channels of the residual stream for all 64
// pixels, and 16 channels of the inner tensors for one half of the pixels (two waves share those channels; each publishes a record of its own).
// So a wave has everything that its BatchNorm channels need: it sums over its registers, publishes, collects and applies without the others, and
// an exchange takes no barrier and no pass through LDS.  What a convolution reduces over lies in LDS (a tile of 256 channels, the canvas of the 3x3
// convolution, a tile of 64 channels), with one barrier each: three per block and direction.  No two waves (conv3) or only two
// (conv1, conv2) read the same weights, so they go from memory to registers, a block ahead, and the LDS serves the pixels alone.
//
// Measured, 111 blocks of ResNet-1001, 8 micro-batches of 8 images, us per block, before (images in LDS tiles) and now: forward 15.2 / 10.7, backward
// 22.5 / 12.9.  A form after kernels_resident_reg.hip, waves dividing the pixels, with the sums and the weights of all through LDS, took 13.2 and 16.1.
// What bounds it now: 240 KiB of weights a block and work-group (1.6 us at the 16 cycles a KiB that a CU takes at best; none of them at all: 8.5 and 12.5 us),
// and every exchange about 1.1 us from its records' leaving to the last one's arrival.  On more than eight images the kernels spill: 7 registers forward
// (32 bytes of scratch a lane), 8 backward (36).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "hpf_resident_reg.h"

namespace hpf {
namespace {

constexpr int R8_C = 256, R8_MID = 64, R8_P = 64;
constexpr int R8_CS = R8_C + 8, R8_MS = R8_MID + 8;   // pixel pitch of the tiles
// canvas: rows of 10 pixels, 416 dwords apart (32 modulo the 64 banks: the two image rows of a fragment fall on banks that do not meet)
constexpr int R8_CW = 10, R8_RP = 832;
static_assert(R8_RP >= R8_CW * R8_MS && R8_RP / 2 % 64 == 32, "canvas rows");
constexpr int R8_TILE_C = R8_P * R8_CS * 2, R8_CANVAS = R8_CW * R8_RP * 2, R8_TILE_M = R8_P * R8_MS * 2;
constexpr int R8_LDS = R8_TILE_C + R8_CANVAS + R8_TILE_M + 16;
constexpr int r8_fwd_lds() { return R8_LDS + RG_NW * (32 + 2 * 16) * 8; }
constexpr int r8_bwd_lds() { return R8_LDS + RG_NW * (4 * (32 + 2 * 16) + 3 * 32) * 4; }

// Where a wave's channels are.  T = 2: residual stream, channel tiles 2*wave and 2*wave + 1 of four pixel tiles; T = 1: inner tensors, one channel
// tile of two pixel tiles.
struct Own8 {
  int tid, lane, wave, fr, fq, mt, ph;
  unsigned offC, offM;          // the lane's place in an image
  int tc_w, cv_w, op_w;         // where it writes in the tile of 256 channels, in the canvas, in the tile of 64
  int tc_r, cv_r, op_r;         // where its fragments of the first pixel tile begin
  __device__ __forceinline__ Own8() {
    tid = threadIdx.x; lane = tid & 63; wave = wave_index(); fr = lane & 15; fq = lane >> 4;
    mt = wave & 3; ph = wave >> 2;
    const int row = 4 * ph + (fr >> 3), col = fr & 7, px = ph * 32 + fr;
    offC = px_offset(fr, R8_C, fq) + (unsigned)(wave * 32);
    offM = (unsigned)(px * R8_MID + mt * 16 + fq * 4);
    tc_w = fr * R8_CS + wave * 32 + fq * 4;
    cv_w = (row + 1) * R8_RP + (col + 1) * R8_MS + mt * 16 + fq * 4;
    op_w = px * R8_MS + mt * 16 + fq * 4;
    tc_r = px * R8_CS + fq * 8;
    cv_r = row * R8_RP + col * R8_MS + fq * 8;
    op_r = fr * R8_MS + fq * 8;
  }
};
__device__ __forceinline__ void own_load(uint2 (&v)[4][2], const bf16_t* g, const Own8& L) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint4 q = *reinterpret_cast<const uint4*>(g + j * 16 * R8_C + L.offC);
    v[j][0] = make_uint2(q.x, q.y);
    v[j][1] = make_uint2(q.z, q.w);
  }
}
__device__ __forceinline__ void own_store(bf16_t* g, const Own8& L, const uint2 (&v)[4][2]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint2 e = v[j][0], o = v[j][1];
    pair_swap(e, o);
    *reinterpret_cast<uint4*>(g + j * 16 * R8_C + L.offC) = make_uint4(e.x, e.y, o.x, o.y);
  }
}
__device__ __forceinline__ void own_load(uint2 (&v)[2][1], const bf16_t* g, const Own8& L) {
#pragma unroll
  for (int j = 0; j < 2; ++j) v[j][0] = *reinterpret_cast<const uint2*>(g + j * 16 * R8_MID + L.offM);
}
__device__ __forceinline__ void own_store(bf16_t* g, const Own8& L, const uint2 (&v)[2][1]) {
#pragma unroll
  for (int j = 0; j < 2; ++j) *reinterpret_cast<uint2*>(g + j * 16 * R8_MID + L.offM) = v[j][0];
}

// A wave's rows of a packed weight matrix of NT row tiles (fragment_at): RT of them, STEPS fragments of 32 elements each
template <int NT, int STEPS, int RT = 1>
struct WRegs {
  static constexpr int N = STEPS * RT;
  bf16x8 f[N];   // [row tile][step]
  __device__ __forceinline__ void issue(const bf16_t* w, int tile, int lane, int i0 = 0, int i1 = N) {
    const bf16_t* g = w + tile * 512;
    const unsigned off = (unsigned)lane * 8;
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (i >= i0 && i < i1) f[i] = *reinterpret_cast<const bf16x8*>(g + (i % STEPS * NT + i / STEPS) * 512 + off);
  }
};
using WDown = WRegs<R8_MID / 16, R8_C / 32>;
using W3x3 = WRegs<R8_MID / 16, 9 * R8_MID / 32>;
using WUp = WRegs<R8_C / 16, R8_MID / 32, 2>;

// conv1 | conv3's data gradient: the wave's 16 inner channels on its two pixel tiles, from the tile of 256 channels
__device__ __forceinline__ void conv_down(const bf16_t* t, const WDown& w, floatx4 (&acc)[2][1]) {
#pragma unroll
  for (int j = 0; j < 2; ++j) acc[j][0] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < R8_C / 32; ++k) {
    if (k % 4 == 0) keep_order();
#pragma unroll
    for (int j = 0; j < 2; ++j)
      acc[j][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.f[k], *reinterpret_cast<const bf16x8*>(t + j * 16 * R8_CS + k * 32), acc[j][0], 0, 0, 0);
  }
}
// conv2 | its data gradient (FLIP: taps mirrored) from the canvas.  The two pixel tiles are two image rows apart: five row offsets serve the six
// pairs of tile and filter row.
template <bool FLIP>
__device__ __forceinline__ void conv_3x3(const bf16_t* cv, const W3x3& w, floatx4 (&acc)[2][1]) {
#pragma unroll
  for (int j = 0; j < 2; ++j) acc[j][0] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < 3; ++s)
#pragma unroll
    for (int ks = 0; ks < R8_MID / 32; ++ks) {
      keep_order();
      bf16x8 px[5];
#pragma unroll
      for (int o = 0; o < 5; ++o) px[o] = *reinterpret_cast<const bf16x8*>(cv + o * R8_RP + s * R8_MS + ks * 32);
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        const int tap = FLIP ? (2 - r) * 3 + 2 - s : r * 3 + s;
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[j][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.f[tap * (R8_MID / 32) + ks], px[2 * j + r], acc[j][0], 0, 0, 0);
      }
    }
}
// conv3 | conv1's data gradient, onto acc: the wave's 32 channels of the residual stream on all pixels, from the tile of 64 channels
__device__ __forceinline__ void conv_up(const bf16_t* t, const WUp& w, floatx4 (&acc)[4][2]) {
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int ks = 0; ks < R8_MID / 32; ++ks) {
      if (j == 2 && ks == 0) keep_order();
      const bf16x8 px = *reinterpret_cast<const bf16x8*>(t + j * 16 * R8_MS + ks * 32);
#pragma unroll
      for (int nt = 0; nt < 2; ++nt) acc[j][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.f[nt * (R8_MID / 32) + ks], px, acc[j][nt], 0, 0, 0);
    }
}
template <int PT, int NT>
__device__ __forceinline__ void round_acc(floatx4 (&v)[PT][NT], uint2 (&p)[PT][NT]) {   // v rounded to bf16, p its packed form
#pragma unroll
  for (int j = 0; j < PT; ++j)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) { p[j][nt] = pack4(v[j][nt]); v[j][nt] = unpack4(p[j][nt]); }
}

// ---- exchange of a wave's channels: NT channel tiles, records of 2*Cc words in the slot; {first, second} of channel c are words 2c and 2c + 1
template <int NT>
struct Rec8 {
  static constexpr int Cc = NT == 2 ? R8_C : R8_MID, W = 2 * Cc, WPW = NT * 32, MG = 64 / WPW, PER = NT == 2 ? 1 : 2;   // PER: records of an image
  int ch0, rec, nrec;    // the wave's first channel, its record, records of the micro-batch
  __device__ __forceinline__ Rec8(const Own8& L, int me, int nmem) : ch0(NT == 2 ? L.wave * 32 : L.mt * 16), rec(NT == 2 ? me : 2 * me + L.ph), nrec(nmem * PER) {}
  static __device__ __forceinline__ int channel(int lane) { return (lane & (WPW - 1)) >> 1; }   // that a lane collects, from the wave's first
  // the sums of halve_sum(), one word from every second lane
  __device__ __forceinline__ void publish(u64* slot, int nt, float v, int fr, int fq, unsigned tag) const {
    if (!(fr & 1)) publish_word(slot, rec, W, 2 * (ch0 + nt * 16 + fq * 4 + ((fr >> 1) & 3)) + (fr >> 3), v, tag);
  }
  // words of the records r0 + lane/WPW + i*MG, i < N; the first poll waits (Gather::poll)
  template <int N>
  __device__ __forceinline__ void poll(u64 (&v)[N], const u64* slot, int r0, unsigned tag, int lane, int* fail, SpinBudget& budget) const {
    const unsigned off = (unsigned)((lane / WPW) * W + 2 * ch0 + (lane & (WPW - 1)));
    const int mine = records(r0, lane);
    const u64* base = slot + (size_t)r0 * W;
    __builtin_amdgcn_s_sleep(12);   // 4: backward 12.9 -> 13.3 us a block; 24: 13.5, forward 10.7 -> 11.4
    for (;;) {
      bool ok = true;
#pragma unroll
      for (int i = 0; i < N; ++i) v[i] = __hip_atomic_load(base + i * (MG * W) + off, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
      for (int i = 0; i < N; ++i) ok = ok && ((unsigned)(v[i] >> 32) == tag || i >= mine);
      if (__all(ok)) break;
      if (!budget.again()) { *fail = 1; break; }
    }
  }
  __device__ __forceinline__ int records(int r0, int lane) const { return (nrec - r0 - lane / WPW + MG - 1) / MG; }   // of a lane, from r0 on
};
// N: records that a lane asks for at a time.  A slot has room for them beyond the last record: 32 (images) or 64 records more than a multiple
template <int NT, int N>
__device__ __forceinline__ void collect_own(const Rec8<NT>& R, const u64* slot, unsigned tag, int lane, int* fail, float& sum, float& first, float& dev1, float& dev2) {
  using G = Rec8<NT>;
  constexpr int CHUNK = N * G::MG;
  u64 v[N];
  SpinBudget budget;
  const float inv_n = 1.f / (float)R.nrec;
  float s1 = 0.f, s2 = 0.f, sw = 0.f, m0 = 0.f;
  for (int b = 0; more_chunks(b, R.nrec, budget); b += CHUNK) {
    R.poll(v, slot, b, tag, lane, fail, budget);
    const int mine = R.records(b, lane);
    float f[N], d[N];
#pragma unroll
    for (int i = 0; i < N; ++i) f[i] = i < mine ? __uint_as_float((unsigned)v[i]) : 0.f;
    sw += tree_sum(f);
    if (b == 0) m0 = lanes_sum<G::WPW>(sw) * (R.nrec < CHUNK ? inv_n : 1.f / (float)CHUNK);
#pragma unroll
    for (int i = 0; i < N; ++i) f[i] = i < mine ? f[i] - m0 : 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i) d[i] = f[i] * f[i];
    s1 += tree_sum(f);
    s2 += tree_sum(d);
  }
  sum = lanes_sum<G::WPW>(sw);
  dev1 = lanes_sum<G::WPW>(s1);
  dev2 = lanes_sum<G::WPW>(s2);
  first = m0;
}
template <int NT, int N>
__device__ __forceinline__ float collect_own_sum(const Rec8<NT>& R, const u64* slot, unsigned tag, int lane, int* fail) {
  using G = Rec8<NT>;
  u64 v[N];
  SpinBudget budget;
  float sw = 0.f;
  for (int b = 0; more_chunks(b, R.nrec, budget); b += N * G::MG) {
    R.poll(v, slot, b, tag, lane, fail, budget);
    const int mine = R.records(b, lane);
    float f[N];
#pragma unroll
    for (int i = 0; i < N; ++i) f[i] = i < mine ? __uint_as_float((unsigned)v[i]) : 0.f;
    sw += tree_sum(f);
  }
  return lanes_sum<G::WPW>(sw);
}
// the wave's {mean, M2} per channel about its first pixel (stats_wave), published
template <int PT, int NT>
__device__ __forceinline__ void stats_own(const floatx4 (&v)[PT][NT], const Rec8<NT>& R, u64* slot, unsigned tag, int fr, int fq) {
  const bool b3 = fr & 8, b2 = fr & 4, b1 = fr & 2;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    float K[4], s1[4], s2[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      K[e] = row_first(v[0][nt][e]);
#pragma unroll
      for (int j = 0; j < PT; ++j) {
        const float d = v[j][nt][e] - K[e];
        s1[e] = j == 0 ? d : s1[e] + d;
        s2[e] = j == 0 ? d * d : fmaf(d, d, s2[e]);
      }
    }
    const float r = halve_sum(s1, s2, b3, b2, b1);
    const float first = dpp_mov<0x128>(r);
    const float k = b2 ? (b1 ? K[3] : K[2]) : (b1 ? K[1] : K[0]);
    constexpr float inv = 1.f / (float)(PT * 16);
    R.publish(slot, nt, b3 ? fmaxf(fmaf(-first * inv, first, r), 0.f) : fmaf(r, inv, k), fr, fq, tag);
  }
}
// N records at a time from a lane: eight where that is all of them
constexpr int R8_FEW = 8, R8_MANY = 16;

// Forward of a run.  INFER: BatchNorm by running statistics; nothing is exchanged or stashed, only the output of the last block is written.
template <bool INFER, int N>
__global__ void __launch_bounds__(RG_NT) k_reg8_forward(const ResArgs a) {
  constexpr int C = R8_C, MID = R8_MID;
  const Own8 L;
  const int tid = L.tid, lane = L.lane, wave = L.wave, fr = L.fr, fq = L.fq;
  const int z = blockIdx.x % a.ngroup, me = blockIdx.x / a.ngroup;   // with g == 8 micro-batch z lives on XCD z
  ResCtx cx{(char*)pick(a.base, z), pick(a.act_in, z), pick(a.act_out, z), nullptr, nullptr};
  u64* xchg = reinterpret_cast<u64*>(cx.base + a.xchg_off);
  unsigned* tagp = reinterpret_cast<unsigned*>(cx.base + a.tag_off);
  const unsigned tag0 = INFER ? 0u : *tagp;
  unsigned phase = 0;
  auto slot = [&]() { return xchg + (size_t)(phase & 1u) * resident_slot_members(a.nmem) * (2 * C); };
  auto image = [&](unsigned long long off, int CT) { return cx.tensor(off) + (size_t)me * (R8_P * CT); };

  extern __shared__ __align__(16) unsigned char smem[];
  bf16_t* tileC = reinterpret_cast<bf16_t*>(smem);
  bf16_t* canvas = reinterpret_cast<bf16_t*>(smem + R8_TILE_C);
  bf16_t* tileM = reinterpret_cast<bf16_t*>(smem + R8_TILE_C + R8_CANVAS);
  int* fail = reinterpret_cast<int*>(smem + R8_LDS - 16);
  float2* coef = reinterpret_cast<float2*>(smem + R8_LDS) + wave * 64;   // the wave's own: 32 of the first BatchNorm, 16 of each of the others

  WDown w1; W3x3 w2; WUp w3;
  floatx4 X[4][2];
  // inference: a channel per lane of the wave's three BatchNorms, read a block ahead
  float rc_mean, rc_var, rc_gamma, rc_beta;
  const int tq = lane < 32 ? 0 : lane < 48 ? 1 : 2, tch = tq == 0 ? wave * 32 + lane : L.mt * 16 + (lane & 15);
  auto load_coef = [&](int b) {
    const ResBlock* t = a.blocks + b;
    auto by = [&](const unsigned long long (&o)[3]) { return tq == 0 ? o[0] : tq == 1 ? o[1] : o[2]; };
    const float* run = a.running + by(t->run_off);
    rc_mean = run[tch];
    rc_var = run[(tq == 0 ? C : MID) + tch];
    rc_gamma = (a.params + by(t->gamma_off))[tch];
    rc_beta = (a.params + by(t->beta_off))[tch];
  };
  auto store_coef = [&] { coef[lane] = bn_scale_shift(rc_mean, 1.0f / sqrtf(rc_var + a.eps), rc_gamma, rc_beta); };
  const Rec8<2> RC(L, me, a.nmem);
  const Rec8<1> RM(L, me, a.nmem);
  // training: statistics of the wave's values v -> its coefficients cf of the BatchNorm q of block B
  auto exchange = [&](const auto& R, const auto& v, const ResBlock& B, int q, float2* cf) {
    using G = std::decay_t<decltype(R)>;
    const unsigned tag = tag0 + 1u + phase;
    const int cl = G::channel(lane), c = R.ch0 + cl;
    stats_own(v, R, slot(), tag, fr, fq);
    const float gamma = (a.params + B.gamma_off[q])[c], beta = (a.params + B.beta_off[q])[c];
    float sw, m0, s1, s2;
    collect_own<G::WPW / 32, N>(R, slot(), tag, lane, fail, sw, m0, s1, s2);
    constexpr float P = (float)(R8_P / G::PER);
    const float inv_n = 1.f / (float)R.nrec;
    const float M2 = fmaf(P, fmaf(-s1 * inv_n, s1, s2), dpp_mov<0xb1>(sw));   // even lanes: the neighbour's sum of M2
    const float mean = fmaf(s1, inv_n, m0), is = inv_sqrt(fmaf(M2, inv_n / P, a.eps));
    if (lane < G::WPW && !(lane & 1)) {
      cf[cl] = bn_scale_shift(mean, is, gamma, beta);
      if (me == 0 && (G::PER == 1 || L.ph == 0)) {
        float* st = reinterpret_cast<float*>(cx.base + B.stats_off[q]);
        st[c] = mean;
        st[G::Cc + c] = is;
      }
    }
    __builtin_amdgcn_wave_barrier();
    ++phase;
  };
  // behind a barrier: has any wave given up waiting?
  auto failed = [&] {
    if (INFER || !*fail) return false;
    if (tid == 0) atomicExch(a.abort_flag, 1);
    return true;
  };
  {
    const ResBlock B0 = a.blocks[0];
    uint2 q[4][2];
    own_load(q, image(B0.x_off, C), L);
    if constexpr (INFER) load_coef(0);
    w1.issue(a.packed + B0.wf_off[0], L.mt, lane);
    w2.issue(a.packed + B0.wf_off[1], L.mt, lane, 0, INFER ? 18 : 9);
    if constexpr (INFER) w3.issue(a.packed + B0.wf_off[2], 2 * wave, lane);
    for (int i = tid; i < R8_CANVAS / 16; i += RG_NT) reinterpret_cast<u32x4*>(canvas)[i] = u32x4{0u, 0u, 0u, 0u};
    if (tid == 0) *fail = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      pair_swap(q[j][0], q[j][1]);
#pragma unroll
      for (int nt = 0; nt < 2; ++nt) X[j][nt] = unpack4(q[j][nt]);
    }
    if constexpr (INFER) store_coef();
    __syncthreads();
    if constexpr (!INFER) exchange(RC, X, B0, 0, coef);
  }
  for (int bi = 0;; ++bi) {
    const bool more = bi + 1 < a.nblk;
    const ResBlock B = a.blocks[bi], Bn = a.blocks[more ? bi + 1 : bi];
    if constexpr (!INFER) {
      w2.issue(a.packed + B.wf_off[1], L.mt, lane, 9, 18);
      w3.issue(a.packed + B.wf_off[2], 2 * wave, lane);
    }
    // ---- conv1 (1x1, C -> MID) on relu(bn1(x))
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
      for (int j = 0; j < 4; ++j) *reinterpret_cast<uint2*>(tileC + L.tc_w + j * 16 * R8_CS + nt * 16) = bn_relu_pack(X[j][nt], coef + nt * 16 + fq * 4);
    __syncthreads();
    if (failed()) return;
    floatx4 acc[2][1];
    uint2 cp[2][1];
    conv_down(tileC + L.tc_r, w1, acc);
    round_acc(acc, cp);
    // A share of the next block's weights behind every exchange: in front of the polls they would hold these up, and they are through before the next
    // records leave
    auto next_w1 = [&](int i0, int i1) { w1.issue(a.packed + Bn.wf_off[0], L.mt, lane, i0, i1); };
    auto next_w2 = [&](int i0, int i1) { w2.issue(a.packed + Bn.wf_off[1], L.mt, lane, i0, i1); };
    if constexpr (INFER) {
      next_w1(0, 8);
    } else {
      exchange(RM, acc, B, 1, coef + 32);
      next_w1(0, 8);
      own_store(image(B.c1_off, MID), L, cp);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) *reinterpret_cast<uint2*>(canvas + L.cv_w + j * 2 * R8_RP) = bn_relu_pack(acc[j][0], coef + 32 + fq * 4);
    __syncthreads();
    if (failed()) return;
    // ---- conv2 (3x3, MID -> MID)
    conv_3x3<false>(canvas + L.cv_r, w2, acc);
    round_acc(acc, cp);
    if constexpr (INFER) {
      next_w2(0, 18);
    } else {
      exchange(RM, acc, B, 2, coef + 48);
      next_w2(0, 9);
      own_store(image(B.c2_off, MID), L, cp);
    }
    // ---- conv3 (1x1, MID -> C) on relu(bn3(c2)), accumulated onto x
#pragma unroll
    for (int j = 0; j < 2; ++j) *reinterpret_cast<uint2*>(tileM + L.op_w + j * 16 * R8_MS) = bn_relu_pack(acc[j][0], coef + 48 + fq * 4);
    if constexpr (INFER) {
      __builtin_amdgcn_wave_barrier();
      load_coef(more ? bi + 1 : bi);
    }
    __syncthreads();
    if (failed()) return;
    conv_up(tileM + L.op_r, w3, X);
    uint2 yp[4][2];
    round_acc(X, yp);
    if (!more) {
      own_store(image(B.y_off, C), L, yp);
      break;
    }
    if constexpr (INFER) {
      w3.issue(a.packed + Bn.wf_off[2], 2 * wave, lane);
      store_coef();
      __builtin_amdgcn_wave_barrier();
    } else {
      exchange(RC, X, Bn, 0, coef);
      own_store(image(B.y_off, C), L, yp);
    }
  }
  // every member has read the counter before it took part in the first exchange, which member 0 has left
  if (!INFER && me == 0 && tid == 0) *tagp = tag0 + phase;
}

// Backward of a run: the same ownership, walking the blocks in reverse with the gradient of the residual stream in registers (packed).
template <int N>
__global__ void __launch_bounds__(RG_NT) k_reg8_backward(const ResArgs a) {
  constexpr int C = R8_C, MID = R8_MID;
  const Own8 L;
  const int tid = L.tid, lane = L.lane, wave = L.wave, fr = L.fr, fq = L.fq;
  const int z = blockIdx.x % a.ngroup, me = blockIdx.x / a.ngroup;   // with g == 8 micro-batch z lives on XCD z
  ResCtx cx{(char*)pick(a.base, z), pick(a.act_in, z), pick(a.act_out, z), pick(a.err_in, z), pick(a.err_out, z)};
  u64* xchg = reinterpret_cast<u64*>(cx.base + a.xchg_off);
  unsigned* tagp = reinterpret_cast<unsigned*>(cx.base + a.tag_off);
  const unsigned tag0 = *tagp;
  unsigned phase = 0;
  auto slot = [&]() { return xchg + (size_t)(phase & 1u) * resident_slot_members(a.nmem) * (2 * C); };
  auto image = [&](unsigned long long off, int CT) { return cx.tensor(off) + (size_t)me * (R8_P * CT); };

  extern __shared__ __align__(16) unsigned char smem[];
  bf16_t* tileC = reinterpret_cast<bf16_t*>(smem);
  bf16_t* canvas = reinterpret_cast<bf16_t*>(smem + R8_TILE_C);
  bf16_t* tileM = reinterpret_cast<bf16_t*>(smem + R8_TILE_C + R8_CANVAS);
  int* fail = reinterpret_cast<int*>(smem + R8_LDS - 16);
  // the wave's own tables: rows of its channels
  float* const cf1 = reinterpret_cast<float*>(smem + R8_LDS) + wave * (4 * 64 + 3 * 32);
  float* const cf2 = cf1 + 4 * 32;
  float* const cf3 = cf2 + 4 * 16;
  float* const tab = cf3 + 4 * 16;

  WDown w3; W3x3 w2; WUp w1;   // of the data gradients
  uint2 DY[4][2], xx[4][2], xc2[2][1], xc1[2][1];
  CfRegs tb;   // a channel per lane of the wave's three BatchNorms
  const int tq = lane < 32 ? 0 : lane < 48 ? 1 : 2, tl = tq == 0 ? lane : lane & 15, tch = (tq == 0 ? wave * 32 : L.mt * 16) + tl;
  float* const t_dst = cf1 + (tq == 0 ? 0 : tq == 1 ? 4 * 32 : 4 * 32 + 4 * 16);
  const int t_n = tq == 0 ? 32 : 16;
  auto load_tables = [&](int bi) {
    const ResBlock* t = a.blocks + bi;
    auto by = [&](const unsigned long long (&o)[3]) { return tq == 0 ? o[0] : tq == 1 ? o[1] : o[2]; };
    tb.load(reinterpret_cast<const float*>(cx.base + by(t->stats_off)), a.params + by(t->gamma_off), a.params + by(t->beta_off), tch, tq == 0 ? C : MID);
  };
  auto store_tables = [&] {
    __builtin_amdgcn_wave_barrier();
    tb.store(t_dst, tl, t_n);
    __builtin_amdgcn_wave_barrier();
  };
  const Rec8<2> RC(L, me, a.nmem);
  const Rec8<1> RM(L, me, a.nmem);
  const float inv_M = 1.f / ((float)a.nmem * (float)R8_P);
  // sums of a BatchNorm + ReLU backward (bwd_sums_wave, collect_bwd) -> tab
  auto exchange = [&](const auto& R, auto& dz, const auto& x, const float* cf, const ResBlock& B, int q) {
    using G = std::decay_t<decltype(R)>;
    constexpr int NT = G::WPW / 32, PT = 4 / G::PER, n = NT * 16;
    const unsigned tag = tag0 + 1u + phase;
    const int cl = G::channel(lane);
    const CfChannel k(cf, cl, n);
    const bool b3 = fr & 8, b2 = fr & 4, b1 = fr & 2;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      floatx4 t[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) t[i] = *reinterpret_cast<const floatx4*>(cf + i * n + nt * 16 + fq * 4);
      float sb[4], sg[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
#pragma unroll
        for (int j = 0; j < PT; ++j) {
          const float v = elem4(x[j][nt], e);
          const float d = fmaf(v, t[0][e], t[1][e]) > 0.f ? dz[j][nt][e] : 0.f;
          const float xh = fmaf(v, t[2][e], t[3][e]);
          dz[j][nt][e] = d;
          sb[e] = j == 0 ? d : sb[e] + d;
          sg[e] = j == 0 ? d * xh : fmaf(d, xh, sg[e]);
        }
      }
      R.publish(slot(), nt, halve_sum(sb, sg, b3, b2, b1), fr, fq, tag);
      keep_order();
    }
    const float sb = collect_own_sum<NT, N>(R, slot(), tag, lane, fail), sg = dpp_mov<0xb1>(sb);   // even lanes
    if (lane < G::WPW && !(lane & 1)) {
      tab[cl] = k.sc;                               // scale*(dz - sb/M - (x*is + nm)*sg/M)
      tab[n + cl] = -k.sc * sg * inv_M * k.is;
      tab[2 * n + cl] = -k.sc * inv_M * (sb + k.nm * sg);
      if (me == 0 && (G::PER == 1 || L.ph == 0)) {
        float* dgb = reinterpret_cast<float*>(cx.base + B.dgb_off[q]);
        dgb[R.ch0 + cl] = sb;
        dgb[G::Cc + R.ch0 + cl] = sg;
      }
    }
    __builtin_amdgcn_wave_barrier();
    ++phase;
  };
  auto failed = [&] {
    if (!*fail) return false;
    if (tid == 0) atomicExch(a.abort_flag, 1);
    return true;
  };
  {
    const ResBlock BL = a.blocks[a.nblk - 1];
    own_load(DY, image(BL.gy_off, C), L);
    load_tables(a.nblk - 1);
    w3.issue(a.packed + BL.wd_off[2], L.mt, lane);
    own_load(xc2, image(BL.c2_off, MID), L);
    w2.issue(a.packed + BL.wd_off[1], L.mt, lane, 0, 9);
    for (int i = tid; i < R8_CANVAS / 16; i += RG_NT) reinterpret_cast<u32x4*>(canvas)[i] = u32x4{0u, 0u, 0u, 0u};
    if (tid == 0) *fail = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) pair_swap(DY[j][0], DY[j][1]);
    store_tables();
  }
  __syncthreads();
  for (int bi = a.nblk - 1; bi >= 0; --bi) {
    const bool more = bi > 0;
    const ResBlock B = a.blocks[bi], Bn = a.blocks[more ? bi - 1 : 0];   // behind the last one: loads that nobody reads
    w2.issue(a.packed + B.wd_off[1], L.mt, lane, 9, 18);
    w1.issue(a.packed + B.wd_off[0], 2 * wave, lane);
    // ---- conv3 data gradient, BN3 + ReLU backward -> dc2
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
      for (int j = 0; j < 4; ++j) *reinterpret_cast<uint2*>(tileC + L.tc_w + j * 16 * R8_CS + nt * 16) = DY[j][nt];
    __syncthreads();
    if (failed()) return;
    auto next_w3 = [&](int i0, int i1) { w3.issue(a.packed + Bn.wd_off[2], L.mt, lane, i0, i1); };
    auto next_w2 = [&](int i0, int i1) { w2.issue(a.packed + Bn.wd_off[1], L.mt, lane, i0, i1); };
    floatx4 acc[2][1];
    conv_down(tileC + L.tc_r, w3, acc);
    exchange(RM, acc, xc2, cf3, B, 2);
    // what later steps read from memory: behind the polls, which would wait for it, and a convolution or more ahead of its use
    own_load(xc1, image(B.c1_off, MID), L);
    own_load(xx, image(B.x_off, C), L);
    next_w3(0, 8);
    if (bi + 1 < a.nblk) own_store(image(a.blocks[bi + 1].gx_off, C), L, DY);   // the gradient of the input of the block above
    uint2 dcp[2][1];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      dcp[j][0] = pack4(bwd_apply<16>(acc[j][0], xc2[j][0], tab + fq * 4));
      *reinterpret_cast<uint2*>(canvas + L.cv_w + j * 2 * R8_RP) = dcp[j][0];
    }
    __syncthreads();
    if (failed()) return;
    // ---- conv2 data gradient, BN2 + ReLU backward -> dc1
    conv_3x3<true>(canvas + L.cv_r, w2, acc);
    exchange(RM, acc, xc1, cf2, B, 1);
    own_load(xc2, image(Bn.c2_off, MID), L);
    load_tables(more ? bi - 1 : 0);
    next_w2(0, 9);
    own_store(image(B.dc2_off, MID), L, dcp);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      dcp[j][0] = pack4(bwd_apply<16>(acc[j][0], xc1[j][0], tab + fq * 4));
      *reinterpret_cast<uint2*>(tileM + L.op_w + j * 16 * R8_MS) = dcp[j][0];
    }
    __syncthreads();
    if (failed()) return;
    // ---- conv1 data gradient, BN1 + ReLU backward, plus the shortcut
    floatx4 da[4][2];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int nt = 0; nt < 2; ++nt) da[j][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
    conv_up(tileM + L.op_r, w1, da);
#pragma unroll
    for (int j = 0; j < 4; ++j) pair_swap(xx[j][0], xx[j][1]);
    exchange(RC, da, xx, cf1, B, 0);
    own_store(image(B.dc1_off, MID), L, dcp);
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
      for (int j = 0; j < 4; ++j) DY[j][nt] = pack4(bwd_apply<32>(da[j][nt], xx[j][nt], tab + nt * 16 + fq * 4) + unpack4(DY[j][nt]));
    store_tables();
  }
  own_store(image(a.blocks[0].gx_off, C), L, DY);
  // the last exchange has no barrier behind it
  __syncthreads();
  if (failed()) return;
  if (me == 0 && tid == 0) *tagp = tag0 + phase;
}

hipError_t launch_reg8(void (*kernel)(const ResArgs), int lds, int g, const ResArgs& a, hipStream_t stream) {
  ResArgs b = a;
  b.ngroup = g;
  kernel<<<dim3((unsigned)(a.nmem * g)), RG_NT, (size_t)lds, stream>>>(b);
  return hipGetLastError();
}

}  // namespace

hipError_t resident_reg8_prepare() {
  hipError_t e = hipSuccess;
  for (const void* f : {reinterpret_cast<const void*>(k_reg8_forward<false, R8_FEW>), reinterpret_cast<const void*>(k_reg8_forward<false, R8_MANY>),
                        reinterpret_cast<const void*>(k_reg8_forward<true, R8_FEW>), reinterpret_cast<const void*>(k_reg8_backward<R8_FEW>),
                        reinterpret_cast<const void*>(k_reg8_backward<R8_MANY>)})
    if (e == hipSuccess) e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  return e;
}
hipError_t launch_reg8_forward(int g, const ResArgs& a, hipStream_t stream) {
  return launch_reg8(a.nmem <= R8_FEW ? k_reg8_forward<false, R8_FEW> : k_reg8_forward<false, R8_MANY>, r8_fwd_lds(), g, a, stream);
}
hipError_t launch_reg8_inference(int g, const ResArgs& a, hipStream_t stream) { return launch_reg8(k_reg8_forward<true, R8_FEW>, r8_fwd_lds(), g, a, stream); }
hipError_t launch_reg8_backward(int g, const ResArgs& a, hipStream_t stream) {
  return launch_reg8(a.nmem <= R8_FEW ? k_reg8_backward<R8_FEW> : k_reg8_backward<R8_MANY>, r8_bwd_lds(), g, a, stream);
}

}  // namespace hpf
