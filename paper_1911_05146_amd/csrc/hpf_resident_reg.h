// Device-side helpers of the image-resident kernels that keep the residual stream in registers (kernels_resident_reg.hip: bottleneck
// runs, kernels_resident_basic.hip: runs of basic blocks).  The layout is that of an MFMA result: lane (fr, fq) holds
// channels nt*16 + fq*4 + 0..3 of pixel fr of a 16-pixel tile; v[j][nt]: channel tile nt of the wave's pixel tile j.
#pragma once
#include "hpf_resident.h"

namespace hpf {
namespace {

constexpr int RG_NT = 512, RG_NW = RG_NT / 64;   // 8 waves

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// Instructions stay on their side: without it the scheduler pulls the table reads of all channel tiles to the front and spills.
__device__ __forceinline__ void keep_order() { __builtin_amdgcn_sched_barrier(0); }

// value of lane 0 of the 16-lane row, in all its lanes
__device__ __forceinline__ float row_first(float v) { return dpp_mov<0x150>(v); }

// Sum over the lanes that are congruent modulo N (N = 4 ... 64 a power of two); every lane gets it.
template <int N>
__device__ __forceinline__ float lanes_sum(float v) {
  static_assert(N == 4 || N == 8 || N == 16 || N == 32 || N == 64, "lane stride");
  if constexpr (N <= 32) {
    const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(r.x) + __uint_as_float(r.y);
  }
  if constexpr (N <= 16) {
    const u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(r.x) + __uint_as_float(r.y);
  }
  if constexpr (N <= 8) v += dpp_mov<0x128>(v);
  if constexpr (N <= 4) v += dpp_mov<0x124>(v);
  return v;
}

// ---- tensors in memory <-> the register layout.  Per pair of channel tiles (32 channels) and pixel, a lane moves 16 bytes
// (8 channels) and swaps half of them with the lane 16 away.
__device__ __forceinline__ void pair_swap(uint2& even, uint2& odd) {
  const u32x2 a = __builtin_amdgcn_permlane16_swap(even.x, odd.x, false, false);
  const u32x2 b = __builtin_amdgcn_permlane16_swap(even.y, odd.y, false, false);
  even = make_uint2(a.x, b.x);
  odd = make_uint2(a.y, b.y);
}
// g: the image (uniform); off: the lane's place in it, px_offset()
__device__ __forceinline__ unsigned px_offset(int px, int CT, int fq) { return (unsigned)(px * CT + (fq & 1) * 16 + (fq >> 1) * 8); }
template <int PTW, int NTL>
__device__ __forceinline__ void px_load(uint2 (&v)[PTW][NTL], const bf16_t* g, unsigned off) {
#pragma unroll
  for (int j = 0; j < PTW; ++j)
#pragma unroll
    for (int k = 0; k < NTL / 2; ++k) {
      const uint4 q = *reinterpret_cast<const uint4*>(g + j * 16 * NTL * 16 + k * 32 + off);
      v[j][2 * k] = make_uint2(q.x, q.y);
      v[j][2 * k + 1] = make_uint2(q.z, q.w);
    }
}
// what px_load asked for, in the register layout (waits for it: to be called where the values are needed)
template <int PTW, int NTL>
__device__ __forceinline__ void px_arrange(uint2 (&v)[PTW][NTL]) {
#pragma unroll
  for (int j = 0; j < PTW; ++j)
#pragma unroll
    for (int k = 0; k < NTL / 2; ++k) pair_swap(v[j][2 * k], v[j][2 * k + 1]);
}
// NT: streaming stores.  They keep the tensors (read again only much later) out of the caches, but bursts of them reach
// the memory's rate; the forward of 128-32 blocks runs 8 % faster with stores that the L2 takes.  In the backward kernels it is the other way round: 128-32 950 us a
// step without and 930 with them, 128-64 1504 and 1522.
template <bool NT = true, int PTW, int NTL>
__device__ __forceinline__ void px_store(bf16_t* g, unsigned off, const uint2 (&v)[PTW][NTL]) {
#pragma unroll
  for (int j = 0; j < PTW; ++j)
#pragma unroll
    for (int k = 0; k < NTL / 2; ++k) {
      uint2 e = v[j][2 * k], o = v[j][2 * k + 1];
      pair_swap(e, o);
      const u32x4 q = {e.x, e.y, o.x, o.y};
      if (NT) __builtin_nontemporal_store(q, reinterpret_cast<u32x4*>(g + j * 16 * NTL * 16 + k * 32 + off));
      else *reinterpret_cast<u32x4*>(g + j * 16 * NTL * 16 + k * 32 + off) = q;
    }
}
// the same for 16-channel tensors: 8 bytes per lane, already in place
template <int PTW>
__device__ __forceinline__ void px_load(uint2 (&v)[PTW][1], const bf16_t* g, unsigned off) {
#pragma unroll
  for (int j = 0; j < PTW; ++j) v[j][0] = *reinterpret_cast<const uint2*>(g + j * 256 + off);
}
template <int PTW>
__device__ __forceinline__ void px_arrange(uint2 (&)[PTW][1]) {}
template <bool NT = true, int PTW>
__device__ __forceinline__ void px_store(bf16_t* g, unsigned off, const uint2 (&v)[PTW][1]) {
#pragma unroll
  for (int j = 0; j < PTW; ++j) {
    const u32x2 q = {v[j][0].x, v[j][0].y};
    if (NT) __builtin_nontemporal_store(q, reinterpret_cast<u32x2*>(g + j * 256 + off));
    else *reinterpret_cast<u32x2*>(g + j * 256 + off) = q;
  }
}
__device__ __forceinline__ floatx4 unpack4(const uint2& q) { return floatx4{bf_lo(q.x), bf_hi(q.x), bf_lo(q.y), bf_hi(q.y)}; }

// ---- weights: a [ROWS][LEN] bf16 matrix staged in LDS by the whole work-group, MFMA fragment by fragment (64 lanes x 16 bytes, so a
// fragment read is one conflict-free 1 KiB access at a constant offset and staging needs no per-unit addresses), as it lies in memory
// (fragment_at).  issue() asks for this wave's fragments, commit() stores them.  The operand of a convolution that reduces over the channels of a
// register tensor is packed permuted: lane (fr, fq) of step kt holds columns kt*32 + {0, 16} + fq*4 + 0..3 of its row.
// PARTS: the matrix travels in that many pieces, so that fewer registers hold what is on its way.
template <int ROWS, int LEN, int PARTS = 1>
struct WStage {
  static constexpr int KT = LEN / 32, NT = ROWS / 16, FR = KT * NT, FP = FR / PARTS, NU = (FP + RG_NW - 1) / RG_NW;
  static constexpr int BYTES = FR * 1024;
  static_assert(FR % PARTS == 0, "equal pieces");
  u32x4 st[NU];
  // third I of the loads (a wave that asks for all of a wide matrix at once stands still until the memory pipeline has taken them:
  // 0.8 us for 64 x 576)
  template <int I>
  __device__ __forceinline__ void issue_third(const bf16_t* w, int wave, int fr, int fq) { issue<0>(w, wave, fr, fq, NU * I / 3, NU * (I + 1) / 3); }
  template <int PART = 0>
  __device__ __forceinline__ void issue(const bf16_t* w, int wave, int fr, int fq, int i0 = 0, int i1 = NU) {
    const unsigned off = (unsigned)((fq * 16 + fr) * 8);
#pragma unroll
    for (int i = 0; i < NU; ++i) {
      if (i < i0 || i >= i1) continue;
      const int f = PART * FP + wave + i * RG_NW;
      if (FP % RG_NW == 0 || f < (PART + 1) * FP) {
        st[i] = *reinterpret_cast<const u32x4*>(w + f * 512 + off);
      }
    }
  }
  template <int PART = 0>
  __device__ __forceinline__ void commit(bf16_t* s, int wave, int lane) const {
#pragma unroll
    for (int i = 0; i < NU; ++i) {
      const int f = PART * FP + wave + i * RG_NW;
      if (FP % RG_NW == 0 || f < (PART + 1) * FP) *reinterpret_cast<u32x4*>(s + f * 512 + lane * 8) = st[i];
    }
  }
  // fragment: rows nt*16 .. +15 of reduction step kt; s: the staged matrix + lane*8
  static __device__ __forceinline__ bf16x8 get(const bf16_t* s, int kt, int nt) {
    return *reinterpret_cast<const bf16x8*>(s + (kt * NT + nt) * 512);
  }
};

// sum of N values by pairs (a chain would be N latencies long)
template <int N>
__device__ __forceinline__ float tree_sum(const float (&v)[N]) {
  float t[N];
#pragma unroll
  for (int i = 0; i < N; ++i) t[i] = v[i];
#pragma unroll
  for (int d = 1; d < N; d *= 2)
#pragma unroll
    for (int i = 0; i + d < N; i += 2 * d) t[i] += t[i + d];
  return t[0];
}
// Sums of eight values over the 16 lanes of a row: at every step a lane keeps one of two values, so the number of values halves
// with the distance (22 instead of 32 instructions) and one LDS write takes the result.  Lane fr gets (b3 ? s2 : s1)[(fr >> 1) & 3].
__device__ __forceinline__ float halve_sum(const float (&s1)[4], const float (&s2)[4], bool b3, bool b2, bool b1) {
  float t[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float p = b3 ? s2[e] : s1[e], q = b3 ? s1[e] : s2[e];
    t[e] = p + dpp_mov<0x128>(q);           // row_ror:8
  }
  float w[2];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const float p = b2 ? t[e + 2] : t[e], q = b2 ? t[e] : t[e + 2];
    w[e] = p + dpp_mov<0x141>(q);           // row_half_mirror
  }
  const float r = (b1 ? w[1] : w[0]) + dpp_mov<0x4e>(b1 ? w[0] : w[1]);   // quad_perm 2,3,0,1
  return r + dpp_mov<0xb1>(r);              // quad_perm 1,0,3,2
}
// ---- BatchNorm statistics from registers.  v: the wave's rounded values.  Sums run about the wave's first pixel, so a large common
// offset does not cancel; the wave's {mean, M2} over its pixels go to red: the wave's row of 2*Cc floats, at the wave's
// first channel.  Plain sums about a value that all work-groups have at hand (the mean of the block before) would be 0.3 us (128-32) / 1.3 us
// (128-64) per block faster, but the variance then loses a factor (distance / sigma)^2 of its digits: invstd of a channel that a block
// moves by 40 sigma was off by 1.6e-4 instead of 1e-7.
__device__ __forceinline__ float elem(const floatx4& v, int e) { return v[e]; }
__device__ __forceinline__ float elem(const uint2& v, int e) { return elem4(v, e); }
template <class V, int PTW, int NTL>   // V: floatx4, or uint2 (packed)
__device__ __forceinline__ void stats_wave(const V (&v)[PTW][NTL], float* red, int Cc, int fr, int fq) {
  const bool b3 = fr & 8, b2 = fr & 4, b1 = fr & 2;
  float* dst = red + (b3 ? Cc : 0) + fq * 4 + ((fr >> 1) & 3);
#pragma unroll
  for (int nt = 0; nt < NTL; ++nt) {
    float K[4], s1[4], s2[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      K[e] = row_first(elem(v[0][nt], e));
#pragma unroll
      for (int j = 0; j < PTW; ++j) {
        const float d = elem(v[j][nt], e) - K[e];
        s1[e] = j == 0 ? d : s1[e] + d;
        s2[e] = j == 0 ? d * d : fmaf(d, d, s2[e]);
      }
    }
    const float r = halve_sum(s1, s2, b3, b2, b1);
    // this lane: channel element (fr >> 1) & 3; its first sum sits 8 lanes away for the lanes of the second ones
    const float first = dpp_mov<0x128>(r);
    const float k = b2 ? (b1 ? K[3] : K[2]) : (b1 ? K[1] : K[0]);
    constexpr float inv = 1.f / (float)(PTW * 16);
    const float o = b3 ? fmaxf(fmaf(-first * inv, first, r), 0.f) : fmaf(r, inv, k);
    if (!(fr & 1)) dst[nt * 16] = o;
  }
}
// Sums {S1, S2} of the waves (rows of red) added up, published by Cc threads per sum as words 2c and 2c + 1
template <int Cc, int NPW = RG_NW>   // NPW: waves along the pixels = rows of red
__device__ __forceinline__ void sums_publish_waves(const float* red, u64* slot, int me, unsigned tag) {
  if ((int)threadIdx.x < 2 * Cc) {
    const int w = threadIdx.x;   // w < Cc: first sums
    float r[NPW];
#pragma unroll
    for (int i = 0; i < NPW; ++i) r[i] = red[i * 2 * Cc + w];
    const float s = tree_sum(r);
    publish_word(slot, me, 2 * Cc, w < Cc ? 2 * w : 2 * (w - Cc) + 1, s, tag);
  }
}
// The image's {mean, M2} from the waves' records (equal pixel counts), published as words 2c and 2c + 1.
template <int Cc, int NPX, int NPW = RG_NW>   // NPX: pixels per wave
__device__ __forceinline__ void stats_publish_waves(const float* red, u64* slot, int me, unsigned tag) {
  if ((int)threadIdx.x < Cc) {
    const int c = threadIdx.x;
    float m[NPW], s = 0.f, q = 0.f;
#pragma unroll
    for (int i = 0; i < NPW; ++i) { m[i] = red[i * 2 * Cc + c]; s += m[i]; }
    const float mean = s * (1.f / NPW);
#pragma unroll
    for (int i = 0; i < NPW; ++i) { const float d = m[i] - mean; q += fmaf((float)NPX * d, d, red[i * 2 * Cc + Cc + c]); }
    publish_word(slot, me, 2 * Cc, 2 * c, mean, tag);
    publish_word(slot, me, 2 * Cc, 2 * c + 1, q, tag);
  }
}

// ---- exchange.  Every wave collects the words of its own Cc/8 channels from all members and merges them in registers
// (lanes = words x member groups), so nothing is gathered in LDS and no barrier lies between the words' arrival and the
// coefficients.  The same order of additions in every work-group.  A wave whose partners do not show up sets *fail, which all waves
// test behind the next barrier.
// CH: members polled at a time (a slot has room for a multiple of 32)
template <int Cc, int CH = 32>
struct Gather {
  static constexpr int W = 2 * Cc, WPW = W / RG_NW, MG = 64 / WPW, CHUNK = CH, INFL = CHUNK / MG;
  static_assert(INFL >= 1, "a member for every group of lanes");
  // words of members m0 + mg + i*MG, i < INFL.  The first poll waits: loads that reach the
  // words before the partners' stores do delay those stores, by more than a microsecond (the record exchange of a 32-channel
  // tensor among 32 work-groups: 2.6 us from publish to coefficients when polled at once, 1.4-1.6 us with the pause; 128-32 blocks
  // forward 357 -> 286 us per launch of 21 blocks; pauses of 8 to 40 measured 303 ... 286 ... 305; with the
  // present weight loads 12 instead of 16: ResNet-110 v1 1262 -> 1251, quarter of ResNet-110 294 -> 290; 8: 1260, 291).  By the second chunk the words are there: with a
  // pause ahead of it too, the sixteenth of the wide ResNet-1001 took 1538 us, now 1512.
  // The slot has room for a multiple of CHUNK members, so all addresses are one lane offset from uniform bases, and words of members that there are
  // not are asked for as well.  A branch around them ends a group of loads, whose words are waited for before the next group is asked for: with
  // one for every eight members, eight blocks of 64 channels on 20 images took 182 us a step and on 32 images 200, without 168 and 174.  Kernels for
  // few members poll a smaller chunk instead.
  static __device__ __forceinline__ void poll(u64 (&v)[INFL], const u64* slot, int m0, int nmem, unsigned tag, int wave, int lane, int* fail, SpinBudget& budget) {
    const unsigned off = (unsigned)((lane / WPW) * W + wave * WPW + (lane & (WPW - 1)));
    const int mine = lane_members(m0, nmem, lane);
    const u64* base = slot + (size_t)m0 * W;
    if (m0 == 0) __builtin_amdgcn_s_sleep(Cc < 128 ? 12 : 8);
    for (;;) {
      bool ok = true;
#pragma unroll
      for (int i = 0; i < INFL; ++i) v[i] = __hip_atomic_load(base + i * (MG * W) + off, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
      for (int i = 0; i < INFL; ++i) ok = ok && ((unsigned)(v[i] >> 32) == tag || i >= mine);
      if (__all(ok)) break;
      if (!budget.again()) { *fail = 1; break; }
    }
  }
  // how many of v[] are members of the micro-batch
  static __device__ __forceinline__ int lane_members(int m0, int nmem, int lane) { return (nmem - m0 - lane / WPW + MG - 1) / MG; }
};
// 1 / sqrt(x): the hardware's estimate (1 ulp) and one Newton step, which has no meaning for x = 0 and x = infinity (0 * infinity): there the
// estimate is the value
__device__ __forceinline__ float inv_sqrt(float x) {
  const float r = __builtin_amdgcn_rsqf(x);
  return r > 0.f && r < INFINITY ? fmaf(0.5f * r, fmaf(-x * r, r, 1.f), r) : r;
}
struct StatsOut { float2* coef; float* stats; };   // stats: member 0 only, else null
template <int Cc>
__device__ __forceinline__ void stats_out(const StatsOut& o, float mean, float var_eps, float gamma, float beta, int wave, int lane) {
  using G = Gather<Cc>;
  const float is = inv_sqrt(var_eps);
  const int mg = lane / G::WPW, wl = lane & (G::WPW - 1);
  if (mg == 0 && !(wl & 1)) {
    const int c = (wave * G::WPW + wl) >> 1;
    o.coef[c] = bn_scale_shift(mean, is, gamma, beta);
    if (o.stats) { o.stats[c] = mean; o.stats[Cc + c] = is; }
  }
}
// {mean, M2} records of equal pixel counts -> coef[c] = {scale, shift}, the mean, and (member 0) stats = {mean(Cc), invstd(Cc)}
template <int Cc, int CH>
__device__ __forceinline__ void collect_stats(const u64* slot, int nmem, unsigned tag, float inv_n, float P, float eps, float gamma, float beta,
                                              const StatsOut& o, int wave, int lane, int* fail) {
  using G = Gather<Cc, CH>;
  u64 v[G::INFL];
  SpinBudget budget;
  float m0 = 0.f, s1 = 0.f, s2 = 0.f, sw = 0.f;   // sw: plain sum of the words (the M2 of the odd lanes)
  for (int b = 0; more_chunks(b, nmem, budget); b += G::CHUNK) {
    G::poll(v, slot, b, nmem, tag, wave, lane, fail, budget);
    const int mine = G::lane_members(b, nmem, lane);
    float f[G::INFL], d[G::INFL];
#pragma unroll
    for (int i = 0; i < G::INFL; ++i) f[i] = i < mine ? __uint_as_float((unsigned)v[i]) : 0.f;
    sw += tree_sum(f);
    if (b == 0) m0 = lanes_sum<G::WPW>(sw) * (nmem < G::CHUNK ? inv_n : 1.f / (float)G::CHUNK);
#pragma unroll
    for (int i = 0; i < G::INFL; ++i) f[i] = i < mine ? f[i] - m0 : 0.f;
#pragma unroll
    for (int i = 0; i < G::INFL; ++i) d[i] = f[i] * f[i];
    s1 += tree_sum(f);
    s2 += tree_sum(d);
  }
  s1 = lanes_sum<G::WPW>(s1);
  s2 = lanes_sum<G::WPW>(s2);
  sw = lanes_sum<G::WPW>(sw);
  const float q = fmaf(-s1 * inv_n, s1, s2);
  const float M2 = fmaf(P, q, dpp_mov<0xb1>(sw));   // even lanes: the neighbour's sum of M2
  stats_out<Cc>(o, fmaf(s1, inv_n, m0), fmaf(M2, inv_n / P, eps), gamma, beta, wave, lane);
}
// the channel whose words this lane collects
template <int Cc>
__device__ __forceinline__ int gather_channel(int wave, int lane) {
  return (wave * Gather<Cc>::WPW + (lane & (Gather<Cc>::WPW - 1))) >> 1;
}

// relu(v*scale + shift) of a channel tile, packed; cf: the coefficients at this lane's fq*4
__device__ __forceinline__ uint2 bn_relu_pack(const floatx4& v, const float2* cf) {
  const float4 a = reinterpret_cast<const float4*>(cf)[0], b = reinterpret_cast<const float4*>(cf)[1];
  return make_uint2(pack_bf16x2(fmaxf(fmaf(v[0], a.x, a.y), 0.f), fmaxf(fmaf(v[1], a.z, a.w), 0.f)),
                    pack_bf16x2(fmaxf(fmaf(v[2], b.x, b.y), 0.f), fmaxf(fmaf(v[3], b.z, b.w), 0.f)));
}
__device__ __forceinline__ bf16x8 frag_of(const uint2& lo, const uint2& hi) {
  return __builtin_bit_cast(bf16x8, make_uint4(lo.x, lo.y, hi.x, hi.y));
}

// ---- BatchNorm + ReLU backward on a gradient in the register layout:
//   dz = da * [z > 0];  sums over the micro-batch {sum dz, sum dz*xhat} (exchange);  out = a1*dz + a2*x + a3 per channel.
// Tables in LDS, one row of Cc floats each: cf = {scale, shift, invstd, -mean*invstd}, tab = {a1, a2, a3}.
// RELU = false: dz arrives masked (the ReLU sits behind a join), the BatchNorm has none of its own.
template <bool RELU = true, int PTW, int NTL>
__device__ __forceinline__ void bwd_sums_wave(floatx4 (&dz)[PTW][NTL], const uint2 (&x)[PTW][NTL], const float* cf, float* red, int Cc,
                                              int fr, int fq) {
  const bool b3 = fr & 8, b2 = fr & 4, b1 = fr & 2;
  float* dst = red + (b3 ? Cc : 0) + fq * 4 + ((fr >> 1) & 3);
#pragma unroll
  for (int nt = 0; nt < NTL; ++nt) {
    floatx4 k[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) k[i] = *reinterpret_cast<const floatx4*>(cf + i * Cc + nt * 16 + fq * 4);
    float sb[4], sg[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
#pragma unroll
      for (int j = 0; j < PTW; ++j) {
        const float v = elem4(x[j][nt], e);
        const float d = !RELU || fmaf(v, k[0][e], k[1][e]) > 0.f ? dz[j][nt][e] : 0.f;
        const float xh = fmaf(v, k[2][e], k[3][e]);
        dz[j][nt][e] = d;
        sb[e] = j == 0 ? d : sb[e] + d;
        sg[e] = j == 0 ? d * xh : fmaf(d, xh, sg[e]);
      }
    }
    const float r = halve_sum(sb, sg, b3, b2, b1);
    if (!(fr & 1)) dst[nt * 16] = r;
    keep_order();
  }
}
// the table entries of the channel whose words a lane collects; read ahead of the exchange, behind whose first barrier the tables may
// be replaced by the next block's
struct CfChannel {
  float sc, is, nm;
  __device__ __forceinline__ CfChannel(const float* cf, int c, int Cc) : sc(cf[c]), is(cf[2 * Cc + c]), nm(cf[3 * Cc + c]) {}
};
// {sum dz, sum dz*xhat} of all members -> tab; dgb (member 0 only, else null): the two sums
// CH: fewer words in flight than the forward collects, or they spill next to the gradients of a wide tensor
template <int Cc, int CH>
__device__ __forceinline__ void collect_bwd(const u64* slot, int nmem, unsigned tag, float inv_M, const CfChannel& k, float* tab, float* dgb, int wave,
                                            int lane, int* fail, float* g_beta = nullptr, float* g_gamma = nullptr) {
  using G = Gather<Cc, CH>;
  const int mg = lane / G::WPW, wl = lane & (G::WPW - 1), c = (wave * G::WPW + wl) >> 1;
  u64 v[G::INFL];
  SpinBudget budget;
  float sw = 0.f;
  for (int b = 0; more_chunks(b, nmem, budget); b += G::CHUNK) {
    G::poll(v, slot, b, nmem, tag, wave, lane, fail, budget);
    const int mine = G::lane_members(b, nmem, lane);
    float f[G::INFL];
#pragma unroll
    for (int i = 0; i < G::INFL; ++i) f[i] = i < mine ? __uint_as_float((unsigned)v[i]) : 0.f;
    sw += tree_sum(f);
  }
  sw = lanes_sum<G::WPW>(sw);
  const float sb = sw, sg = dpp_mov<0xb1>(sw);   // even lanes
  if (mg == 0 && !(wl & 1)) {
    tab[c] = k.sc;                               // scale*(dz - sb/M - (x*is + nm)*sg/M)
    tab[Cc + c] = -k.sc * sg * inv_M * k.is;
    tab[2 * Cc + c] = -k.sc * inv_M * (sb + k.nm * sg);
    if (dgb) { dgb[c] = sb; dgb[Cc + c] = sg; }
    if (g_beta) { atomicAdd(g_beta + c, sb); atomicAdd(g_gamma + c, sg); }   // runs whose weight-gradient launch does not add the stored sums
  }
}
// tab at the lane's channels.  x is hidden from the compiler, which would otherwise keep the values that the sums unpacked in
// registers over the whole exchange.
template <int Cc>
__device__ __forceinline__ floatx4 bwd_apply(const floatx4& dz, uint2 x, const float* tab) {
  asm volatile("" : "+v"(x.x), "+v"(x.y));
  const floatx4 a1 = *reinterpret_cast<const floatx4*>(tab), a2 = *reinterpret_cast<const floatx4*>(tab + Cc),
                a3 = *reinterpret_cast<const floatx4*>(tab + 2 * Cc);
  floatx4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = fmaf(a1[e], dz[e], fmaf(a2[e], elem4(x, e), a3[e]));
  return o;
}
// one channel of a cf table: loaded ahead, stored later
struct CfRegs {
  float mean, is, g, b;
  __device__ __forceinline__ void load(const float* stats, const float* gamma, const float* beta, int c, int Cc) {
    mean = stats[c]; is = stats[Cc + c]; g = gamma[c]; b = beta[c];
  }
  __device__ __forceinline__ void store(float* cf, int c, int Cc) const {
    const float2 ss = bn_scale_shift(mean, is, g, b);
    cf[c] = ss.x; cf[Cc + c] = ss.y; cf[2 * Cc + c] = is; cf[3 * Cc + c] = -mean * is;
  }
};

}  // namespace
}  // namespace hpf
