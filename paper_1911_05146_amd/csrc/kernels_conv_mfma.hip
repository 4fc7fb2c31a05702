// Implicit-GEMM convolution forward and data-gradient on bf16 MFMA (v_mfma_f32_16x16x32_bf16),
// fp32 accumulation, NHWC tiles staged through LDS.
//
// Both passes are the same gather-GEMM
//     out[m, n] = sum_k W[n, k] * src[row(m, tap(k)), c(k)],      k = tap*Cs + c,
// with the reduction index k running over (filter tap, source channel).  The packed weights are
// [N][Kpad] (k contiguous), the source tensor is NHWC, so for a fixed pixel row 8 consecutive k are
// 16 contiguous bytes of one source pixel (Cs is a multiple of 8): the im2col matrix is never
// materialised, each LDS-staging thread decodes (tap, c) for its 16-byte unit and either loads the
// source pixel or writes zeros (padding, stride holes of the data-gradient, K padding).
//
// MFMA orientation: the weight tile is the first operand (rows = output channels) and the pixel
// tile the second (columns = pixels), so each lane ends up with 4 consecutive output channels of
// one pixel: the epilogue stores (and reads the optional residual) 8 bytes per lane, and the 4
// lane groups of a wave cover 16 consecutive channels = 32 contiguous bytes per pixel.
//
// Work-group: 256 threads = 4 waves arranged WR x WC over a BM (pixels) x BN (channels) tile;
// K advances 64 per step (32 in the 128-row tile and where K is short), double-buffered in LDS with one barrier per step and the
// next steps' global loads in flight during the MFMAs.
#include <mutex>

#include "hpf_device.h"

namespace hpf {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int KC = 32;          // reduction elements of one MFMA; packed weights are padded to it
constexpr size_t BIG_MAX_LDS = 128 * 1024;   // dynamic LDS limit set for the 128 x 128 x 64 kernels (stages + coefficients)

// relu(bn(x)) of the 8 bf16 values in q, channels c..c+7 (c a multiple of 8); coef holds per channel
// {scale = gamma*invstd, shift = beta - mean*scale}, so the operand is max(x*scale + shift, 0).
__device__ __forceinline__ uint4 bn_relu_unit(const uint4& q, const float2* coef, int c) {
  const uint32_t w[4] = {q.x, q.y, q.z, q.w};
  const float4* cf = reinterpret_cast<const float4*>(coef + c);   // two channels per 16-byte read
  uint32_t r[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float4 k = cf[i];
    const float x0 = __uint_as_float(w[i] << 16), x1 = __uint_as_float(w[i] & 0xffff0000u);
    r[i] = pack_bf16x2(fmaxf(fmaf(x0, k.x, k.y), 0.f), fmaxf(fmaf(x1, k.z, k.w), 0.f));
  }
  return make_uint4(r[0], r[1], r[2], r[3]);
}

// {scale, shift} of all source channels from finished or running statistics
template <int NT>
__device__ __forceinline__ void bn_coefficients(const ConvPro& pro, int Cs, float2* coef) {
  const float* stt = pro.running ? pro.running : (const float*)pick(pro.stats, blockIdx.z);
  for (int c = threadIdx.x; c < Cs; c += NT) {
    const float is = pro.running ? 1.0f / sqrtf(stt[Cs + c] + pro.eps) : stt[Cs + c];
    const float sc = pro.gamma[c] * is;
    coef[c] = make_float2(sc, pro.beta[c] - stt[c] * sc);
  }
}

// EPI_BIAS: a rounded output value as the layer behind the convolution takes it.  In a pass of its own the bias cost a launch and a second trip of
// the tensor through memory: 4.4 to 7.4 us for each of VGG-16's 15 layers, of a training step of 1563 us that now takes 1526.
__device__ __forceinline__ float bias_act(float v, float bias, int relu) {
  const float z = v + bias;
  return relu && !(z > 0.f) ? 0.f : z;
}
// Epilogue of a BM x BN tile whose accumulators are spread over WR x WC waves (wave (wr, wc) holds pixel rows
// wr*PT*16.. and channels wc*CT*16..): residual add, bf16 store, and the optional per-channel sums (statistics of
// the stored values, or BatchNorm-backward sums) written as one partial record per tile row and channel.
// `scratch` is LDS that no wave reads as operand storage any more: BN + WR*BN*2 floats; tile_row is the index of
// the tile's partial record.
template <int BM, int BN, int WR, int WC, int PT, int CT, int EPI>
__device__ __forceinline__ void conv_epilogue(floatx4 (&acc)[CT][PT], int wr, int wc, int tile_row, int row0, int ch0, float* scratch,
                                              const ConvGeom& g, const ConvEpi& epi, const bf16_t* add, bf16_t* out) {
  constexpr int WPX = PT * 16, WCH = CT * 16;
  static_assert(WR * WPX == BM && WC * WCH == BN, "wave grid covers the tile");
  const int tid = threadIdx.x, lane = tid & 63;
  // acc[i][j][v]: channel = ch0 + wc*WCH + i*16 + (lane>>4)*4 + v, pixel row = row0 + wr*WPX + j*16 + (lane&15)
  // Epilogue scratch in the (now idle) staging LDS: shift per channel and per-wave-row sums.
  float* sK = scratch;                                     // [BN]
  float* sS = sK + BN;                                     // [WR][BN][2]
  float s1[CT][4], s2[CT][4];
#pragma unroll
  for (int i = 0; i < CT; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) { s1[i][v] = 0.f; s2[i][v] = 0.f; }

  // per-channel BN constants of this lane's channels (EPI_BNBWD), loaded once
  float mu_[CT][4], is_[CT][4], ga_[CT][4], be_[CT][4];
  if (EPI == EPI_BNBWD) {
    const float* stt = (const float*)pick(epi.stats, blockIdx.z);
#pragma unroll
    for (int i = 0; i < CT; ++i) {
      const int ch = ch0 + wc * WCH + i * 16 + (lane >> 4) * 4;
      const float4 mu = *reinterpret_cast<const float4*>(stt + ch);
      const float4 is = *reinterpret_cast<const float4*>(stt + g.N + ch);
      const float4 ga = *reinterpret_cast<const float4*>(epi.gamma + ch);
      const float4 be = *reinterpret_cast<const float4*>(epi.beta + ch);
      mu_[i][0] = mu.x; mu_[i][1] = mu.y; mu_[i][2] = mu.z; mu_[i][3] = mu.w;
      is_[i][0] = is.x; is_[i][1] = is.y; is_[i][2] = is.z; is_[i][3] = is.w;
      ga_[i][0] = ga.x; ga_[i][1] = ga.y; ga_[i][2] = ga.z; ga_[i][3] = ga.w;
      be_[i][0] = be.x; be_[i][1] = be.y; be_[i][2] = be.z; be_[i][3] = be.w;
    }
  }

#pragma unroll
  for (int j = 0; j < PT; ++j) {
    const int m = row0 + wr * WPX + j * 16 + (lane & 15);
    const bool mv = m < g.M;
#pragma unroll
    for (int i = 0; i < CT; ++i) {
      const int chl = wc * WCH + i * 16 + (lane >> 4) * 4;
      const int ch = ch0 + chl;
      const size_t o = (size_t)(mv ? m : 0) * g.N + ch;
      float vv[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
      if (add && mv) {
        const uint2 t = *reinterpret_cast<const uint2*>(add + o);
        vv[0] += __uint_as_float(t.x << 16); vv[1] += __uint_as_float(t.x & 0xffff0000u);
        vv[2] += __uint_as_float(t.y << 16); vv[3] += __uint_as_float(t.y & 0xffff0000u);
      }
      uint2 st;
      st.x = pack_bf16x2(vv[0], vv[1]);
      st.y = pack_bf16x2(vv[2], vv[3]);
      if (EPI != EPI_NONE) {   // continue with the values as stored
        vv[0] = __uint_as_float(st.x << 16); vv[1] = __uint_as_float(st.x & 0xffff0000u);
        vv[2] = __uint_as_float(st.y << 16); vv[3] = __uint_as_float(st.y & 0xffff0000u);
      }
      if (EPI == EPI_BNBWD) {
        if (mv) {
          const bf16_t* xt = (const bf16_t*)pick(epi.x, blockIdx.z);
          const uint2 xr = *reinterpret_cast<const uint2*>(xt + o);
          const float xv[4] = {__uint_as_float(xr.x << 16), __uint_as_float(xr.x & 0xffff0000u),
                               __uint_as_float(xr.y << 16), __uint_as_float(xr.y & 0xffff0000u)};
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const float xh = (xv[v] - mu_[i][v]) * is_[i][v];
            const float z = ga_[i][v] * xh + be_[i][v];
            const float dz = z > 0.f ? vv[v] : 0.f;
            vv[v] = dz;
            s1[i][v] += dz;
            s2[i][v] += dz * xh;
          }
          st.x = pack_bf16x2(vv[0], vv[1]);   // exact: dz is a stored value or 0
          st.y = pack_bf16x2(vv[2], vv[3]);
        }
      }
      if (EPI == EPI_BIAS) {
        const float4 b = *reinterpret_cast<const float4*>(epi.bias + ch);
        st.x = pack_bf16x2(bias_act(vv[0], b.x, epi.relu), bias_act(vv[1], b.y, epi.relu));
        st.y = pack_bf16x2(bias_act(vv[2], b.z, epi.relu), bias_act(vv[3], b.w, epi.relu));
      }
      if (EPI == EPI_STATS) {
        if (j == 0 && wr == 0 && (lane & 15) == 0) {   // the tile's first row gives the shift
#pragma unroll
          for (int v = 0; v < 4; ++v) sK[chl + v] = vv[v];
        }
        // keep the stored values for the second pass over the registers
        acc[i][j][0] = vv[0]; acc[i][j][1] = vv[1]; acc[i][j][2] = vv[2]; acc[i][j][3] = vv[3];
      }
      if (mv) *reinterpret_cast<uint2*>(out + o) = st;
    }
  }
  if (EPI == EPI_NONE || EPI == EPI_BIAS) return;

  if (EPI == EPI_STATS) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < CT; ++i) {
      const int chl = wc * WCH + i * 16 + (lane >> 4) * 4;
      const float4 k4 = *reinterpret_cast<const float4*>(sK + chl);
      const float k_[4] = {k4.x, k4.y, k4.z, k4.w};
#pragma unroll
      for (int j = 0; j < PT; ++j) {
        const int m = row0 + wr * WPX + j * 16 + (lane & 15);
        if (m < g.M) {
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const float d = acc[i][j][v] - k_[v];
            s1[i][v] += d;
            s2[i][v] += d * d;
          }
        }
      }
    }
  }
  // sum over the 16 pixel lanes of each lane group, then over the wave rows through LDS (fixed order)
#pragma unroll
  for (int i = 0; i < CT; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) { s1[i][v] = sum16(s1[i][v]); s2[i][v] = sum16(s2[i][v]); }
  if ((lane & 15) == 0) {
#pragma unroll
    for (int i = 0; i < CT; ++i) {
      const int chl = wc * WCH + i * 16 + (lane >> 4) * 4;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        sS[(wr * BN + chl + v) * 2] = s1[i][v];
        sS[(wr * BN + chl + v) * 2 + 1] = s2[i][v];
      }
    }
  }
  __syncthreads();
  if (tid < BN) {
    float a1 = 0.f, a2 = 0.f;
#pragma unroll
    for (int w = 0; w < WR; ++w) { a1 += sS[(w * BN + tid) * 2]; a2 += sS[(w * BN + tid) * 2 + 1]; }
    float* part = (float*)pick(epi.partials, blockIdx.z);
    if (EPI == EPI_STATS) {
      const int nrows = min(BM, g.M - row0);
      *reinterpret_cast<float4*>(part + ((size_t)tile_row * g.N + ch0 + tid) * 4) = make_float4(sK[tid], a1, a2, (float)nrows);
    } else {
      *reinterpret_cast<float2*>(part + ((size_t)tile_row * g.N + ch0 + tid) * 2) = make_float2(a1, a2);
    }
  }
}

// What bounds the launches this kernel takes (few work-groups, each with one wave per SIMD and nothing to hide behind) is the chain of
// a step: addresses, LDS reads, MFMA, LDS stores, barrier.  Steps of 64 reduction elements in the 64-row tiles: half as
// many chains as with 32, and no integer loops in the addresses.  3x3 convolutions of ResNet-20's transitions, 8 images: 64 -> 64
// channels at 8x8 13.4 -> 10.0 us (two forms of it 13.2 -> 11.5 and 11.1 -> 7.9), 64 -> 32 gradient at 16x16 12.0 -> 10.7; 1x1
// 256 -> 1024 on 12 544 rows 34.5 -> 30.9.  Four chunks in flight instead of two: no faster (ResNet-20 439 against 433 us per
// batch), and a work-group less per CU (35.8).
// SHORT: reductions of up to SHORT_K elements are five steps of 32 at most, all of them in flight from the start, in 20 instead of 36 KiB of LDS (eight
// instead of four work-groups per CU, and no half-empty last step).  1x1 on 50 176 rows, steps of 64 / SHORT, us: 32 -> 128 channels 9.7 / 8.1,
// 128 -> 512 31.9 / 25.7, behind a BatchNorm 53 / 42, 160 -> 512 36.0 / 30.1; 3x3 16 -> 16 5.8 / 5.1; on 784 rows 64 -> 256 4.2 / 3.7, 16 -> 16 4.2 / 3.7.
template <int BM, int BN, int WR, int WC, int KS, int MODE, int EPI, int PRO>
__global__ __launch_bounds__(256) void k_conv_mfma(PtrTab srcs, const bf16_t* __restrict__ wpk, PtrTab outs, PtrTab adds,
                                                   ConvGeom g, ConvEpi epi, ConvPro pro) {
  extern __shared__ float2 coef[];   // PRO: per source channel {scale, shift}
  const bf16_t* __restrict__ src = (const bf16_t*)pick(srcs, blockIdx.z);
  bf16_t* out = (bf16_t*)pick(outs, blockIdx.z);
  const bf16_t* add = (const bf16_t*)pick(adds, blockIdx.z);
  static_assert(WR * WC == 4, "4 waves");
  constexpr int WPX = BM / WR, WCH = BN / WC, PT = WPX / 16, CT = WCH / 16;
  static_assert(PT >= 1 && CT >= 1, "tile too small");
  constexpr int UPR = KS / 8, RPP = 256 / UPR;   // KS: reduction elements per step; 16-byte units per row, rows per pass of the threads
  constexpr bool SHORT = BM == 64 && KS == 32;   // the whole reduction, up to SHORT_K elements, is in flight at once
  constexpr int LSTR = KS + 8;       // LDS row stride in bf16 (144 or 80 bytes: conflict-free 16-byte reads)
  constexpr int A_UNITS = BM / RPP;
  static_assert(A_UNITS >= 1, "BM >= 64");
  constexpr int W_UNITS = (BN + RPP - 1) / RPP;

  __shared__ __attribute__((aligned(16))) bf16_t sA[2][BM * LSTR];
  __shared__ __attribute__((aligned(16))) bf16_t sW[2][BN * LSTR];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = wave / WC, wc = wave % WC;
  const int row0 = blockIdx.x * BM, ch0 = blockIdx.y * BN;
  const int grp = tid % UPR, trow = tid / UPR;
  const int HoWo = g.Ho * g.Wo;
  const int sshift = g.stride - 1;  // stride is 1 or 2

  int a_img[A_UNITS], a_h[A_UNITS], a_w[A_UNITS];
#pragma unroll
  for (int u = 0; u < A_UNITS; ++u) {
    const int m = row0 + trow + u * RPP;
    const int mm = m < g.M ? m : 0;
    const int img = mm / HoWo;
    const int rem = mm - img * HoWo;
    const int p = rem / g.Wo, q = rem - p * g.Wo;
    a_img[u] = img * g.Hs * g.Ws;
    if (MODE == CONV_FWD) { a_h[u] = p * g.stride - g.pad; a_w[u] = q * g.stride - g.pad; }
    else { a_h[u] = p + g.pad; a_w[u] = q + g.pad; }
    if (m >= g.M) a_h[u] = -(1 << 20);   // a row outside every image
  }

  // NPRE chunks are kept in flight in registers (SHORT: all there are).  Every load of a chunk is issued unconditionally (outside the image, the tensor or the reduction
  // it reads a clamped address and is zeroed when it is stored to LDS; past the last chunk the last one is loaded again), so
  // the number of outstanding loads is known at every wait.
  constexpr int NPRE = 2;
  struct Slot { uint4 a[A_UNITS]; uint4 w[W_UNITS]; int c; bool av[A_UNITS], wv; };
  Slot sl0, sl1, sl2, sl3, sl4;   // named, not an array: they must stay in registers (SHORT: all five)
  if (PRO) {
    if (pro.rows) {
      float* stt = (float*)pick(pro.stats, blockIdx.z);
      const bool first = blockIdx.x == 0 && blockIdx.y == 0;
      const int nch = g.Cs < 64 ? g.Cs : 64;
      for (int c0 = 0; c0 < g.Cs; c0 += nch)
        bn_finalize_records((const float4*)pick(pro.records, blockIdx.z), pro.rows, g.Cs, c0, nch, pro.M, pro.eps, reinterpret_cast<float*>(&sA[0][0]),
                            [&](int c, float mean, float is) {
                              const float sc = pro.gamma[c] * is;
                              coef[c] = make_float2(sc, pro.beta[c] - mean * sc);
                              if (first) { stt[c] = mean; stt[g.Cs + c] = is; }
                            });
    } else {
      bn_coefficients<256>(pro, g.Cs, coef);
    }
    __syncthreads();
  }

  // filter tap and channel of this thread's unit: k / Cs by a multiplication (exact for the k here: k*Cs < 2^32), tap / 3 likewise (taps 0..8)
  const uint32_t cs_inv = 0xffffffffu / (uint32_t)g.Cs + 1u;
  const int nk = (g.Kpad + KS - 1) / KS;
  int kc_ld = 0;
  const bf16_t* wrow = wpk + (size_t)(ch0 + trow % BN) * g.Kpad;   // tiles of fewer rows than a pass: the other threads load copies
  auto load_chunk = [&](Slot& q) {
    const int k = kc_ld * KS + grp * 8;
    kc_ld += kc_ld + 1 < nk;
    const bool kvalid = k < g.Ktot;
    const int tap = kvalid && g.R != 1 ? (int)__umulhi((uint32_t)k, cs_inv) : 0;
    const int c = kvalid ? k - tap * g.Cs : 0;
    const int r = g.R == 1 ? 0 : (tap * 11) >> 5, s = g.R == 1 ? 0 : tap - 3 * r;
    q.c = c;
#pragma unroll
    for (int u = 0; u < A_UNITS; ++u) {
      int hs, ws;
      bool v = kvalid;
      if (MODE == CONV_FWD) {
        hs = a_h[u] + r; ws = a_w[u] + s;
      } else {
        const int th = a_h[u] - r, tw = a_w[u] - s;
        v = v && th >= 0 && tw >= 0 && (((th | tw) & sshift) == 0);
        hs = th >> sshift; ws = tw >> sshift;
      }
      v = v && (unsigned)hs < (unsigned)g.Hs && (unsigned)ws < (unsigned)g.Ws;
      q.av[u] = v;
      q.a[u] = *reinterpret_cast<const uint4*>(src + (v ? (size_t)(a_img[u] + hs * g.Ws + ws) * g.Cs + c : (size_t)c));
    }
    q.wv = KS == KC || k < g.Kpad;     // a last chunk of 32
#pragma unroll
    for (int u = 0; u < W_UNITS; ++u) q.w[u] = *reinterpret_cast<const uint4*>(wrow + (size_t)u * RPP * g.Kpad + (q.wv ? k : 0));
  };
  auto store_chunk = [&](int buf, const Slot& q) {
#pragma unroll
    for (int u = 0; u < A_UNITS; ++u) {
      uint4 val = q.a[u];
      if (PRO) val = bn_relu_unit(val, coef, q.c);
      if (!q.av[u]) val = make_uint4(0u, 0u, 0u, 0u);
      *reinterpret_cast<uint4*>(&sA[buf][(trow + u * RPP) * LSTR + grp * 8]) = val;
    }
#pragma unroll
    for (int u = 0; u < W_UNITS; ++u) {
      uint4 val = q.w[u];
      if (!q.wv) val = make_uint4(0u, 0u, 0u, 0u);
      if (BN % RPP == 0 || trow < BN) *reinterpret_cast<uint4*>(&sW[buf][(trow + u * RPP) * LSTR + grp * 8]) = val;
    }
  };

  floatx4 acc[CT][PT];
#pragma unroll
  for (int i = 0; i < CT; ++i)
#pragma unroll
    for (int j = 0; j < PT; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  load_chunk(sl0);
  if (!SHORT || nk > 1) load_chunk(sl1);
  if (SHORT && nk > 2) load_chunk(sl2);
  if (SHORT && nk > 3) load_chunk(sl3);
  if (SHORT && nk > 4) load_chunk(sl4);
  store_chunk(0, sl0);
  __syncthreads();
  const int frag_row = lane & 15, frag_k = (lane >> 4) * 8;
  // one step: its chunk is in LDS buffer `buf` and its register slot `cur` is free again; `nxt` holds the chunk behind it (more: there is one)
  auto step = [&](int buf, Slot& cur, const Slot& nxt, bool more) {
    if (!SHORT) load_chunk(cur);
    bf16x8 fa[KS / KC][PT], fw[KS / KC][CT];
#pragma unroll
    for (int h = 0; h < KS / KC; ++h) {
#pragma unroll
      for (int j = 0; j < PT; ++j)
        fa[h][j] = *reinterpret_cast<const bf16x8*>(&sA[buf][(wr * WPX + j * 16 + frag_row) * LSTR + h * KC + frag_k]);
#pragma unroll
      for (int i = 0; i < CT; ++i)
        fw[h][i] = *reinterpret_cast<const bf16x8*>(&sW[buf][(wc * WCH + i * 16 + frag_row) * LSTR + h * KC + frag_k]);
    }
    if (!SHORT || more) store_chunk(buf ^ 1, nxt);
#pragma unroll
    for (int h = 0; h < KS / KC; ++h)
#pragma unroll
      for (int i = 0; i < CT; ++i)
#pragma unroll
        for (int j = 0; j < PT; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[h][i], fa[h][j], acc[i][j], 0, 0, 0);
    __syncthreads();
  };
  if (SHORT) {
    step(0, sl0, sl1, nk > 1);
    if (nk > 1) step(1, sl1, sl2, nk > 2);
    if (nk > 2) step(0, sl2, sl3, nk > 3);
    if (nk > 3) step(1, sl3, sl4, nk > 4);
    if (nk > 4) step(0, sl4, sl4, false);
  } else {
    int kc0 = 0;
    for (; kc0 + NPRE <= nk; kc0 += NPRE) {
      step(0, sl0, sl1, true);
      step(1, sl1, sl0, true);
    }
    if (kc0 < nk) step(0, sl0, sl1, true);
  }

  static_assert((BN + WR * BN * 2) * 4 <= (int)sizeof(sA), "epilogue scratch fits the staging buffer");
  conv_epilogue<BM, BN, WR, WC, PT, CT, EPI>(acc, wr, wc, blockIdx.x, row0, ch0, reinterpret_cast<float*>(&sA[0][0]), g, epi, add, out);
}

// ---- long reductions on wide tensors ---------------------------------------------------------------------
// 128 x 128 tile, 8 waves, 64 reduction elements per step, three LDS stages.  The waves form two groups of 2 x 2: both groups take
// the same 64 x 64 quadrants, group 0 over the first and group 1 over the second 32 reduction elements of every
// step, so each SIMD holds two waves (one hides the other's LDS and barrier waits) while every operand fragment
// is still read from LDS once.  At the end the groups exchange half of their sums through LDS: group 0 ends
// up with pixel rows 0..31 of each quadrant, group 1 with rows 32..63, and the epilogue sees a 4 x 2 wave grid.
// Needs Cs % 64 == 0 (a step stays within one filter tap, so tap and padding are decided per pixel row, not per
// 16-byte unit) and Kpad % 64 == 0.
constexpr int BIG_T = 128, BIG_K = 64, BIG_LS = BIG_K + 8;   // LDS rows of 144 bytes: 16-byte reads of 16 rows hit 16 bank groups
constexpr int BIG_STAGE = 2 * BIG_T * BIG_LS;                // bf16 elements per stage (pixel tile, then weight tile)
constexpr int BIG_OPERAND_BYTES = 3 * BIG_STAGE * 2;         // three stages

// SPLIT: grid y = number of work-groups that share a reduction; each takes a contiguous range of the steps and
// stores its fp32 partial tile into its slab of the member's buffer epi.splitk_ws (k_splitk_finish adds the slabs up): for long reductions
// into few output tiles (VGG-16's 512 -> 512 convolutions on 4x4 and 2x2 pixels: 32-64 tiles, 72 steps).
template <int MODE, int EPI, int PRO, bool SPLIT = false>
__global__ __launch_bounds__(512) void k_conv_big(PtrTab srcs, const bf16_t* __restrict__ wpk, PtrTab outs, PtrTab adds, ConvGeom g,
                                                  ConvEpi epi, ConvPro pro) {
  static_assert(!SPLIT || (EPI == EPI_NONE && PRO == 0), "partial sums leave the kernel as they are");
  extern __shared__ __attribute__((aligned(16))) unsigned char big_smem[];
  bf16_t* stage = reinterpret_cast<bf16_t*>(big_smem);
  float2* coef = reinterpret_cast<float2*>(big_smem + BIG_OPERAND_BYTES);   // PRO: per source channel {scale, shift}
  const bf16_t* __restrict__ src = (const bf16_t*)pick(srcs, blockIdx.z);
  bf16_t* out = (bf16_t*)pick(outs, blockIdx.z);
  const bf16_t* add = (const bf16_t*)pick(adds, blockIdx.z);

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int kh = wave >> 2, wr = (wave >> 1) & 1, wc = wave & 1;
  // Work-groups go to the 8 XCDs (each with its own L2) round-robin by index.  Tiles are numbered with the channel
  // tile fastest and every XCD takes a contiguous range of them: the work-groups that share a pixel tile run on one
  // XCD at the same time, and each XCD reads only its share of the source tensor.
  const int n_nt = g.N / BIG_T, tiles = ((g.M + BIG_T - 1) / BIG_T) * n_nt, per_xcd = (tiles + 7) >> 3;
  const int q = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (q >= tiles) return;              // the whole work-group, before any barrier
  const int mt = q / n_nt;
  const int row0 = mt * BIG_T, ch0 = (q - mt * n_nt) * BIG_T;
  const int grp = tid & 7;             // 16-byte unit within the 128-byte row of a step
  const int HoWo = g.Ho * g.Wo;
  const int sshift = g.stride - 1;     // stride is 1 or 2

  // staging: rows (tid >> 3) and (tid >> 3) + 64 of both tiles
  int a_img[2], a_h[2], a_w[2];
  bool a_ok[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int m = row0 + (tid >> 3) + u * 64;
    a_ok[u] = m < g.M;
    const int mm = a_ok[u] ? m : 0;
    const int img = mm / HoWo;
    const int rem = mm - img * HoWo;
    const int p = rem / g.Wo, q = rem - p * g.Wo;
    a_img[u] = img * g.Hs * g.Ws;
    if (MODE == CONV_FWD) { a_h[u] = p * g.stride - g.pad; a_w[u] = q * g.stride - g.pad; }
    else { a_h[u] = p + g.pad; a_w[u] = q + g.pad; }
  }
  if (PRO) {
    bn_coefficients<512>(pro, g.Cs, coef);
    __syncthreads();
  }

  // Two or three steps of global loads stay in flight, in registers.  Every step issues the same four loads
  // unconditionally (rows outside the image or the tensor read a clamped address and are zeroed when they are
  // stored to LDS; past the last step the last one is loaded again), so the counter of outstanding loads is known
  // at every wait and a wait for the oldest step never drains the younger ones.
  struct Slot { uint4 a[2]; uint4 w[2]; int c; bool av[2]; };
  Slot sl0, sl1, sl2;
  const int nk_all = g.Kpad / BIG_K;
  const int k_begin = SPLIT ? (int)((long)blockIdx.y * nk_all / gridDim.y) : 0;
  const int nk = SPLIT ? (int)((long)(blockIdx.y + 1) * nk_all / gridDim.y) - k_begin : nk_all;   // this work-group's steps
  int lk = 0, lc = 0, lr = 0, ls = 0;  // index, channel base and filter tap of the step that is loaded next (uniform)
  if (SPLIT) {
    const int tap = (k_begin * BIG_K) / g.Cs;
    lc = k_begin * BIG_K - tap * g.Cs; lr = tap / g.R; ls = tap - lr * g.R;
  }
  const bf16_t* wrow = wpk + (size_t)(ch0 + (tid >> 3)) * g.Kpad + grp * 8 + (size_t)k_begin * BIG_K;   // second unit: 64 rows further (uniform offset)
  auto load_chunk = [&](Slot& q) {
    const int cb = lc, c = cb + grp * 8, r = lr, s = ls, kc = lk;
    if (lk + 1 < nk) {                 // state only: no loads under this branch
      ++lk; lc += BIG_K;
      if (lc >= g.Cs) { lc = 0; if (++ls == g.R) { ls = 0; ++lr; } }
    }
    q.c = cb;                          // uniform: the lane's channels are q.c + grp*8
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      int hs, ws;
      bool v = a_ok[u];
      if (MODE == CONV_FWD) {
        hs = a_h[u] + r; ws = a_w[u] + s;
      } else {
        const int th = a_h[u] - r, tw = a_w[u] - s;
        v = v && th >= 0 && tw >= 0 && (((th | tw) & sshift) == 0);
        hs = th >> sshift; ws = tw >> sshift;
      }
      v = v && (unsigned)hs < (unsigned)g.Hs && (unsigned)ws < (unsigned)g.Ws;
      q.av[u] = v;
      const size_t off = v ? (size_t)(a_img[u] + hs * g.Ws + ws) * g.Cs + c : (size_t)c;
      q.a[u] = *reinterpret_cast<const uint4*>(src + off);
      q.w[u] = *reinterpret_cast<const uint4*>(wrow + (size_t)u * 64 * g.Kpad + kc * BIG_K);
    }
  };
  auto store_chunk = [&](int st, const Slot& q) {
    bf16_t* sA = stage + st * BIG_STAGE;
    bf16_t* sW = sA + BIG_T * BIG_LS;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      uint4 val = q.a[u];
      if (PRO) val = bn_relu_unit(val, coef, q.c + grp * 8);
      if (!q.av[u]) val = make_uint4(0u, 0u, 0u, 0u);
      *reinterpret_cast<uint4*>(&sA[((tid >> 3) + u * 64) * BIG_LS + grp * 8]) = val;
      *reinterpret_cast<uint4*>(&sW[((tid >> 3) + u * 64) * BIG_LS + grp * 8]) = q.w[u];
    }
  };

  floatx4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  // Three LDS stages.  During step kc the waves multiply the fragments of chunk kc (in registers since the step
  // before), read the fragments of chunk kc+1 (complete in LDS since the last barrier) into the second register
  // set, and write chunk kc+2 from its register slot to the third stage; the slot then takes the loads of a later
  // chunk.  LDS reads, LDS writes, global loads and MFMAs of a step are independent of each other, so they overlap
  // within a wave, and one barrier per step orders the stages.
  struct Frags { bf16x8 a[4], w[4]; };
  const int frag_off_a = (wr * 64 + (lane & 15)) * BIG_LS + kh * 32 + (lane >> 4) * 8;
  const int frag_off_w = BIG_T * BIG_LS + (wc * 64 + (lane & 15)) * BIG_LS + kh * 32 + (lane >> 4) * 8;
  auto read_frags = [&](int st, Frags& f) {
    const bf16_t* base = stage + st * BIG_STAGE;
#pragma unroll
    for (int j = 0; j < 4; ++j) f.a[j] = *reinterpret_cast<const bf16x8*>(&base[frag_off_a + j * 16 * BIG_LS]);
#pragma unroll
    for (int i = 0; i < 4; ++i) f.w[i] = *reinterpret_cast<const bf16x8*>(&base[frag_off_w + i * 16 * BIG_LS]);
  };
  constexpr int NS = PRO ? 2 : 3;      // register slots: with the BatchNorm prologue registers are short
  load_chunk(sl0);
  load_chunk(sl1);
  if (NS == 3) load_chunk(sl2);
  store_chunk(0, sl0);
  load_chunk(sl0);                     // chunk 3 (chunk 2 with two slots)
  store_chunk(1, sl1);
  load_chunk(sl1);                     // chunk 4 (chunk 3)
  __syncthreads();
  Frags f0, f1;
  read_frags(0, f0);
  // st = kc % 3 (stage of chunk kc); `slot` holds chunk kc+2 and then takes the loads of chunk kc+2+NS
  auto step = [&](int st, Slot& slot, const Frags& cur, Frags& nxt) {
    const int st1 = st == 2 ? 0 : st + 1, st2 = st == 0 ? 2 : st - 1;
    read_frags(st1, nxt);
    store_chunk(st2, slot);            // past the last chunk: a copy of the last one, in a stage that nobody reads
    load_chunk(slot);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cur.w[i], cur.a[j], acc[i][j], 0, 0, 0);
    __syncthreads();
  };
  int kc0 = 0;
  if (NS == 3) {
    for (; kc0 + 6 <= nk; kc0 += 6) {
      step(0, sl2, f0, f1);
      step(1, sl0, f1, f0);
      step(2, sl1, f0, f1);
      step(0, sl2, f1, f0);
      step(1, sl0, f0, f1);
      step(2, sl1, f1, f0);
    }
    if (kc0 + 0 < nk) step(0, sl2, f0, f1);
    if (kc0 + 1 < nk) step(1, sl0, f1, f0);
    if (kc0 + 2 < nk) step(2, sl1, f0, f1);
    if (kc0 + 3 < nk) step(0, sl2, f1, f0);
    if (kc0 + 4 < nk) step(1, sl0, f0, f1);
  } else {
    for (; kc0 + 6 <= nk; kc0 += 6) {
      step(0, sl0, f0, f1);
      step(1, sl1, f1, f0);
      step(2, sl0, f0, f1);
      step(0, sl1, f1, f0);
      step(1, sl0, f0, f1);
      step(2, sl1, f1, f0);
    }
    if (kc0 + 0 < nk) step(0, sl0, f0, f1);
    if (kc0 + 1 < nk) step(1, sl1, f1, f0);
    if (kc0 + 2 < nk) step(2, sl0, f0, f1);
    if (kc0 + 3 < nk) step(0, sl1, f1, f0);
    if (kc0 + 4 < nk) step(1, sl0, f0, f1);
  }

  // Epilogue through LDS (all operand reads are behind the last barrier, so the stages are free): group 1 writes
  // its sums into an fp32 tile [128 pixels][128 channels], group 0 adds its own, and then every thread takes
  // (pixel row, 8 consecutive channels) units, so that 16 lanes cover the 256 contiguous bytes of a row in the
  // residual read, the BatchNorm-input read and the store.
  constexpr int TS = BIG_T + 4;        // fp32 row stride: rows shift by 4 banks
  float* tile = reinterpret_cast<float*>(big_smem);
  float* sK = tile + BIG_T * TS;       // [128] shift per channel (EPI_STATS)
  float* sS = sK + BIG_T;              // [32 row groups][128 channels][2]
  static_assert((BIG_T * TS + BIG_T + 32 * BIG_T * 2) * 4 <= BIG_OPERAND_BYTES, "epilogue tile and sums fit the stages");
  {
    float* t0 = tile + (wr * 64 + (lane & 15)) * TS + wc * 64 + (lane >> 4) * 4;
    if (kh == 1) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) *reinterpret_cast<floatx4*>(t0 + j * 16 * TS + i * 16) = acc[i][j];
    }
    __syncthreads();
    if (kh == 0) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          floatx4* t = reinterpret_cast<floatx4*>(t0 + j * 16 * TS + i * 16);
          *t = *t + acc[i][j];
        }
    }
    __syncthreads();
  }
  const int cg = tid & 15, rg = tid >> 4;      // channels ch0 + cg*8 .. +8, rows rg + 32*u
  const int ch = ch0 + cg * 8;
  float vals[4][8];
  float s1[8], s2[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) { s1[e] = 0.f; s2[e] = 0.f; }
  float mu_[8], is_[8], ga_[8], be_[8];
  if (EPI == EPI_BNBWD) {
    const float* stt = (const float*)pick(epi.stats, blockIdx.z);
    load8(stt + ch, mu_); load8(stt + g.N + ch, is_); load8(epi.gamma + ch, ga_); load8(epi.beta + ch, be_);
  }
  if (EPI == EPI_BIAS) load8(epi.bias + ch, be_);
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int rl = rg + 32 * u, m = row0 + rl;
    const bool mv = m < g.M;
    const size_t o = (size_t)(mv ? m : 0) * g.N + ch;
    float (&vv)[8] = vals[u];
    load8(tile + rl * TS + cg * 8, vv);
    if (SPLIT) {
      if (mv) {
        float* o4 = (float*)pick(epi.splitk_ws, blockIdx.z) + ((size_t)blockIdx.y * g.M + m) * g.N + ch;
        *reinterpret_cast<float4*>(o4) = make_float4(vv[0], vv[1], vv[2], vv[3]);
        *reinterpret_cast<float4*>(o4 + 4) = make_float4(vv[4], vv[5], vv[6], vv[7]);
      }
      continue;
    }
    if (add) {
      float rv[8];
      load8(add + o, rv);
#pragma unroll
      for (int e = 0; e < 8; ++e) vv[e] += rv[e];
    }
    uint4 st;
    st.x = pack_bf16x2(vv[0], vv[1]); st.y = pack_bf16x2(vv[2], vv[3]);
    st.z = pack_bf16x2(vv[4], vv[5]); st.w = pack_bf16x2(vv[6], vv[7]);
    if (EPI != EPI_NONE) {             // continue with the values as stored
      const uint32_t w[4] = {st.x, st.y, st.z, st.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) { vv[2 * e] = __uint_as_float(w[e] << 16); vv[2 * e + 1] = __uint_as_float(w[e] & 0xffff0000u); }
    }
    if (EPI == EPI_BNBWD) {
      float xv[8];
      load8((const bf16_t*)pick(epi.x, blockIdx.z) + o, xv);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float xh = (xv[e] - mu_[e]) * is_[e];
        const float z = ga_[e] * xh + be_[e];
        const float dz = (mv && z > 0.f) ? vv[e] : 0.f;
        vv[e] = dz;
        s1[e] += dz;
        s2[e] += dz * xh;
      }
      st.x = pack_bf16x2(vv[0], vv[1]); st.y = pack_bf16x2(vv[2], vv[3]);   // exact: dz is a stored value or 0
      st.z = pack_bf16x2(vv[4], vv[5]); st.w = pack_bf16x2(vv[6], vv[7]);
    }
    if (EPI == EPI_BIAS) {
#pragma unroll
      for (int e = 0; e < 8; ++e) vv[e] = bias_act(vv[e], be_[e], epi.relu);
      st.x = pack_bf16x2(vv[0], vv[1]); st.y = pack_bf16x2(vv[2], vv[3]);
      st.z = pack_bf16x2(vv[4], vv[5]); st.w = pack_bf16x2(vv[6], vv[7]);
    }
    if (EPI == EPI_STATS && rl == 0) {   // the tile's first row gives the shift
#pragma unroll
      for (int e = 0; e < 8; ++e) sK[cg * 8 + e] = vv[e];
    }
    if (mv) *reinterpret_cast<uint4*>(out + o) = st;
  }
  if (EPI == EPI_NONE || EPI == EPI_BIAS) return;
  if (EPI == EPI_STATS) {
    __syncthreads();
    float k_[8];
    load8(sK + cg * 8, k_);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (row0 + rg + 32 * u < g.M) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float d = vals[u][e] - k_[e];
          s1[e] += d;
          s2[e] += d * d;
        }
      }
  }
  // sums over the 32 row groups through LDS, in a fixed order
#pragma unroll
  for (int e = 0; e < 8; ++e) *reinterpret_cast<float2*>(&sS[(rg * BIG_T + cg * 8 + e) * 2]) = make_float2(s1[e], s2[e]);
  __syncthreads();
  if (tid < BIG_T) {
    float a1 = 0.f, a2 = 0.f;
#pragma unroll 8
    for (int r = 0; r < 32; ++r) {
      const float2 t = *reinterpret_cast<const float2*>(&sS[(r * BIG_T + tid) * 2]);
      a1 += t.x; a2 += t.y;
    }
    float* part = (float*)pick(epi.partials, blockIdx.z);
    if (EPI == EPI_STATS) {
      const int nrows = min(BIG_T, g.M - row0);
      *reinterpret_cast<float4*>(part + ((size_t)mt * g.N + ch0 + tid) * 4) = make_float4(sK[tid], a1, a2, (float)nrows);
    } else {
      *reinterpret_cast<float2*>(part + ((size_t)mt * g.N + ch0 + tid) * 2) = make_float2(a1, a2);
    }
  }
}

// out[z][m][n] = bf16(sum over the slabs of the fp32 partial sums), bias != nullptr: with bias and ReLU as EPI_BIAS; 8 elements per thread
__global__ __launch_bounds__(256) void k_splitk_finish(PtrTab wss, PtrTab outs, int splits, size_t mn, int N, const float* __restrict__ bias,
                                                       int relu) {
  const size_t u = (size_t)blockIdx.x * 256 + threadIdx.x;   // unit of 8 elements within a member
  const int z = blockIdx.y;
  if (u * 8 >= mn) return;
  const float* __restrict__ ws = (const float*)pick(wss, z);
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < splits; ++s) {
    const float4* q = reinterpret_cast<const float4*>(ws + (size_t)s * mn + u * 8);
    const float4 a = q[0], b = q[1];
    acc[0] += a.x; acc[1] += a.y; acc[2] += a.z; acc[3] += a.w;
    acc[4] += b.x; acc[5] += b.y; acc[6] += b.z; acc[7] += b.w;
  }
  uint4 st;
  st.x = pack_bf16x2(acc[0], acc[1]); st.y = pack_bf16x2(acc[2], acc[3]);
  st.z = pack_bf16x2(acc[4], acc[5]); st.w = pack_bf16x2(acc[6], acc[7]);
  if (bias) {
    float v[8], b[8];
    load8(reinterpret_cast<const bf16_t*>(&st), v);
    load8(bias + (u * 8) % (size_t)N, b);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = bias_act(v[e], b[e], relu);
    st.x = pack_bf16x2(v[0], v[1]); st.y = pack_bf16x2(v[2], v[3]);
    st.z = pack_bf16x2(v[4], v[5]); st.w = pack_bf16x2(v[6], v[7]);
  }
  *reinterpret_cast<uint4*>((bf16_t*)pick(outs, z) + u * 8) = st;
}

bool big_tile_fits(const ConvGeom& g) { return g.N % BIG_T == 0 && g.Cs % BIG_K == 0 && g.Kpad % BIG_K == 0 && g.Kpad == g.Ktot; }

// Reductions of at least 16 steps into so few tiles that half of the CUs would idle are split over up to four
// work-groups (each keeps at least 8 steps).
int big_splits(int ng, const ConvGeom& g) {
  const long wgs = (long)((g.M + BIG_T - 1) / BIG_T) * (g.N / BIG_T) * ng;
  const int nk = g.Kpad / BIG_K;
  if (nk < 16 || wgs > 128) return 1;
  int s = (int)(256 / wgs);
  if (s > 4) s = 4;
  if (s > nk / 8) s = nk / 8;
  return s < 2 ? 1 : s;
}

hipError_t launch_big(int mode, int ng, const PtrTab& src, const bf16_t* wpk, const PtrTab& out, const PtrTab& add, const ConvGeom& g,
                      hipStream_t stream, const ConvEpi& epi, const ConvPro& pro) {
  const int tiles = ((g.M + BIG_T - 1) / BIG_T) * (g.N / BIG_T);
  const size_t dyn = BIG_OPERAND_BYTES + (pro.on ? (size_t)g.Cs * sizeof(float2) : 0);
  if (dyn > BIG_MAX_LDS) return hipErrorInvalidValue;
  const int splits = ((epi.kind == EPI_NONE || epi.kind == EPI_BIAS) && !pro.on && add.p[0] == nullptr && epi.splitk_floats) ? big_splits(ng, g) : 1;
  if (splits > 1 && (size_t)splits * g.M * g.N <= epi.splitk_floats) {
    const dim3 sgrid((unsigned)(8 * ((tiles + 7) / 8)), (unsigned)splits, (unsigned)ng);
    if (mode == CONV_FWD) k_conv_big<CONV_FWD, EPI_NONE, 0, true><<<sgrid, 512, dyn, stream>>>(src, wpk, out, add, g, epi, pro);
    else k_conv_big<CONV_DGRAD, EPI_NONE, 0, true><<<sgrid, 512, dyn, stream>>>(src, wpk, out, add, g, epi, pro);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const size_t mn = (size_t)g.M * g.N;   // a multiple of 128
    k_splitk_finish<<<dim3((unsigned)((mn / 8 + 255) / 256), (unsigned)ng), 256, 0, stream>>>(epi.splitk_ws, out, splits, mn, g.N,
                                                                                              epi.kind == EPI_BIAS ? epi.bias : nullptr, epi.relu);
    return hipGetLastError();
  }
  const dim3 grid((unsigned)(8 * ((tiles + 7) / 8)), 1u, (unsigned)ng);
#define HPF_CONV(MODE_, EPI_, PRO_) k_conv_big<MODE_, EPI_, PRO_><<<grid, 512, dyn, stream>>>(src, wpk, out, add, g, epi, pro)
  if (mode == CONV_FWD) {
    if (epi.kind == EPI_STATS) { if (pro.on) HPF_CONV(CONV_FWD, EPI_STATS, 1); else HPF_CONV(CONV_FWD, EPI_STATS, 0); }
    else if (epi.kind == EPI_NONE) { if (pro.on) HPF_CONV(CONV_FWD, EPI_NONE, 1); else HPF_CONV(CONV_FWD, EPI_NONE, 0); }
    else if (epi.kind == EPI_BIAS && !pro.on) HPF_CONV(CONV_FWD, EPI_BIAS, 0);
    else return hipErrorInvalidValue;
  } else {
    if (pro.on) return hipErrorInvalidValue;
    if (epi.kind == EPI_BNBWD) HPF_CONV(CONV_DGRAD, EPI_BNBWD, 0);
    else if (epi.kind == EPI_NONE) HPF_CONV(CONV_DGRAD, EPI_NONE, 0);
    else return hipErrorInvalidValue;
  }
#undef HPF_CONV
  return hipGetLastError();
}

template <int BM, int BN, int WR, int WC, int KS>
hipError_t launch_tile(int mode, int ng, const PtrTab& src, const bf16_t* wpk, const PtrTab& out, const PtrTab& add,
                       const ConvGeom& g, hipStream_t stream, const ConvEpi& epi, const ConvPro& pro) {
  const dim3 grid((unsigned)((g.M + BM - 1) / BM), (unsigned)(g.N / BN), (unsigned)ng);
  const size_t dyn = pro.on ? (size_t)g.Cs * sizeof(float2) : 0;
#define HPF_CONV(MODE_, EPI_, PRO_) \
  k_conv_mfma<BM, BN, WR, WC, KS, MODE_, EPI_, PRO_><<<grid, 256, dyn, stream>>>(src, wpk, out, add, g, epi, pro)
  if (mode == CONV_FWD) {
    if (epi.kind == EPI_STATS) { if (pro.on) HPF_CONV(CONV_FWD, EPI_STATS, 1); else HPF_CONV(CONV_FWD, EPI_STATS, 0); }
    else if (epi.kind == EPI_NONE) { if (pro.on) HPF_CONV(CONV_FWD, EPI_NONE, 1); else HPF_CONV(CONV_FWD, EPI_NONE, 0); }
    else if (epi.kind == EPI_BIAS && !pro.on) HPF_CONV(CONV_FWD, EPI_BIAS, 0);
    else return hipErrorInvalidValue;
  } else {
    if (pro.on) return hipErrorInvalidValue;
    if (epi.kind == EPI_BNBWD) HPF_CONV(CONV_DGRAD, EPI_BNBWD, 0);
    else if (epi.kind == EPI_NONE) HPF_CONV(CONV_DGRAD, EPI_NONE, 0);
    else return hipErrorInvalidValue;
  }
#undef HPF_CONV
  return hipGetLastError();
}

// 0: 128x128, 1: 64x64, 2: 64x32, 3: 64x16, 4: 128x128 with 64-element steps on 8 waves
constexpr int BIG_MIN_K = 256;        // reductions from here on count as wide for the choice of what is written to memory
// The 8-wave tile pays a fixed 8 us per work-group (pipeline fill, epilogue through LDS) and runs one work-group per CU; of the
// 64x64 tile four share a CU (36 KiB of LDS each) and hide each other's.  1x1 convolutions, 64x64 / 8-wave tile, us: K = 256, 12 544 rows
// into 1024 channels 24.0 / 29.3, into 128 7.0 / 8.4, 1568 rows into 1024 7.0 / 8.6; K = 512, 12 544 rows into 256 14.5 / 12.6, 3136 into
// 1024 13.9 / 12.0.  This rule does not look at the number of tiles: with 100 of them and fewer the 64x64 tile is the faster one
// at K = 512 too (12 544 rows into 128 9.6 / 11.1, 3136 into 256 7.9 / 10.6).
constexpr int BIG_MIN_K_TILE = 512;
constexpr int SHORT_K = 160;
int pick_tile(int ng, const ConvGeom& g) {
  if (big_tile_fits(g) && g.Kpad >= BIG_MIN_K_TILE) return 4;
  // the 128x128 tile pays off through operand reuse over a long reduction; short reductions are
  // latency bound and want many small work-groups
  if (g.N % 128 == 0 && g.Kpad >= 512) {
    const long wgs = (long)((g.M + 127) / 128) * (g.N / 128) * ng;
    if (wgs >= 512) return 0;   // at least two work-groups per CU, else the smaller tile hides latency better
  }
  if (g.N % 64 == 0) return 1;
  if (g.N % 32 == 0) return 2;
  return 3;
}

}  // namespace

int conv_mfma_tile_rows(int ng, const ConvGeom& g) {
  const int t = pick_tile(ng, g);
  return t == 0 || t == 4 ? 128 : 64;
}

// A launch of its own for the finalize step costs 4.7 us, nearly all of it latency.  Done by every work-group it costs the convolution a round trip
// per 64 channels, one after the other, and rows * Cs records to read.  3x3, 16 / 32 / 64 channels: 1024 records + 1.2 / 1.0 / 1.0 us,
// 4096 + 4.0 / 3.0 / 3.1, 8192 + 8.8 / 6.7 / 6.4 (64 to 512 work-groups); 1x1 out of 128 channels, 1024 + 2.8, 4096 + 3.6; out of 192 + 4.5
// whatever the records, out of 256 + 5.6, 512 + 11, 1024 + 21.  More work-groups than a chip holds at four per CU pay for it one after the
// other: 1x1 out of 32 / 64 / 128 channels, 1024 of them + 0.9 / 1.5 / 3.4, 2048 + 3.5 / 4.5 / 8.3; 1568 of them out of 128 + 7.9.
bool conv_takes_records(int ng, const ConvGeom& g, unsigned rows) {
  const int t = pick_tile(ng, g), bm = t == 0 ? 128 : 64, bn = t == 0 ? 128 : t == 1 ? 64 : t == 2 ? 32 : 16;
  return t != 4 && g.Cs <= 128 && rows * (size_t)g.Cs <= 4096 && (size_t)((g.M + bm - 1) / bm) * (g.N / bn) * ng <= 1024;
}

int conv_splitk(int ng, const ConvGeom& g) {
  if (g.N % 16 != 0 || g.Cs % 8 != 0 || g.Kpad % KC != 0) return 1;
  return pick_tile(ng, g) == 4 ? big_splits(ng, g) : 1;
}

int conv_operand_reuse(int cin, int cout, int R) {
  if (cout % BIG_T != 0 || cin % BIG_K != 0 || R * R * cin < BIG_MIN_K) return 0;
  return R * R * (cout / BIG_T);
}

// The 8-wave kernels take their LDS as dynamic shared memory above the default limit: state it once per device
// before the first launch (not a stream operation, so it stays out of captured graphs).
hipError_t conv_prepare() {
  static std::mutex mu;
  static bool done[64] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lock(mu);
  if (dev >= 0 && dev < 64 && done[dev]) return hipSuccess;
  auto set = [&](const void* f) {
    if (e == hipSuccess) e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)BIG_MAX_LDS);
  };
  set(reinterpret_cast<const void*>(k_conv_big<CONV_FWD, EPI_STATS, 1>));
  set(reinterpret_cast<const void*>(k_conv_big<CONV_FWD, EPI_STATS, 0>));
  set(reinterpret_cast<const void*>(k_conv_big<CONV_FWD, EPI_NONE, 1>));
  set(reinterpret_cast<const void*>(k_conv_big<CONV_FWD, EPI_NONE, 0>));
  set(reinterpret_cast<const void*>(k_conv_big<CONV_FWD, EPI_BIAS, 0>));
  set(reinterpret_cast<const void*>(k_conv_big<CONV_DGRAD, EPI_BNBWD, 0>));
  set(reinterpret_cast<const void*>(k_conv_big<CONV_DGRAD, EPI_NONE, 0>));
  set(reinterpret_cast<const void*>(k_conv_big<CONV_FWD, EPI_NONE, 0, true>));
  set(reinterpret_cast<const void*>(k_conv_big<CONV_DGRAD, EPI_NONE, 0, true>));
  if (e == hipSuccess && dev >= 0 && dev < 64) done[dev] = true;
  return e;
}

// Tile choice: the widest channel tile that divides N, then the pixel tile that still gives the
// chip (256 CUs) enough work-groups.
hipError_t launch_conv_mfma(int mode, int ng, const PtrTab& src, const bf16_t* wpk, const PtrTab& out, const PtrTab& add,
                            const ConvGeom& g, hipStream_t stream, const ConvEpi& epi, const ConvPro& pro) {
  if (ng < 1 || ng > MAX_GROUP) return hipErrorInvalidValue;
  if (g.N % 16 != 0 || g.Cs % 8 != 0 || g.Kpad % KC != 0 || (g.stride != 1 && g.stride != 2)) return hipErrorInvalidValue;
  switch (pick_tile(ng, g)) {
    case 4: return launch_big(mode, ng, src, wpk, out, add, g, stream, epi, pro);
    case 0: return launch_tile<128, 128, 2, 2, 32>(mode, ng, src, wpk, out, add, g, stream, epi, pro);
    case 1:
      return g.Kpad <= SHORT_K ? launch_tile<64, 64, 2, 2, 32>(mode, ng, src, wpk, out, add, g, stream, epi, pro)
                               : launch_tile<64, 64, 2, 2, 64>(mode, ng, src, wpk, out, add, g, stream, epi, pro);
    case 2:
      return g.Kpad <= SHORT_K ? launch_tile<64, 32, 4, 1, 32>(mode, ng, src, wpk, out, add, g, stream, epi, pro)
                               : launch_tile<64, 32, 4, 1, 64>(mode, ng, src, wpk, out, add, g, stream, epi, pro);
    default:
      return g.Kpad <= SHORT_K ? launch_tile<64, 16, 4, 1, 32>(mode, ng, src, wpk, out, add, g, stream, epi, pro)
                               : launch_tile<64, 16, 4, 1, 64>(mode, ng, src, wpk, out, add, g, stream, epi, pro);
  }
}

}  // namespace hpf
