// Small kernels around the convolutions: stem im2col, classification head (global average pool,
// FC, softmax cross-entropy -- the loss of the last partition, paper Eq. 1-2), SGD with momentum
// (apply_gradients) with the weight packing for the MFMA operands, fills and copies.
#include "hpf_device.h"

namespace hpf {
namespace {

// col[m, k] for k = (r*3+s)*Cin + c, zero for taps outside the image and for k >= 9*Cin; Kc % 8 == 0.  A thread makes 16 bytes of a row: with a
// thread per element, its position a chain of 64-bit divisions, 128 images of 32x32x3 took 21 us for the 8 MiB that it writes, now 7.9.
__global__ __launch_bounds__(256) void k_im2col3x3(PtrTab imgs, PtrTab cols, int b, int H, int W, int Cin, int Kc) {
  const float* __restrict__ img = (const float*)pick(imgs, blockIdx.z);
  bf16_t* __restrict__ col = (bf16_t*)pick(cols, blockIdx.z);
  const unsigned units = (unsigned)Kc / 8;
  const size_t total = (size_t)b * H * W * units;
  const uint32_t cin_inv = 0xffffffffu / (uint32_t)Cin + 1u;   // k / Cin, exact while k * Cin < 2^32 (Cin == 1: k itself)
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
    const unsigned m = total < (1ull << 32) ? (unsigned)i / units : (unsigned)(i / units), k0 = (unsigned)(i - (size_t)m * units) * 8;
    const unsigned row = m / (unsigned)W, n = row / (unsigned)H;
    const int q = (int)(m - row * (unsigned)W), p = (int)(row - n * (unsigned)H);
    const float* src = img + ((size_t)n * H * W + (size_t)p * W + q) * Cin;
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const unsigned k = k0 + e, tap = Cin == 1 ? k : __umulhi(k, cin_inv);
      const int c = (int)(k - tap * (unsigned)Cin), dr = (int)(tap * 11 >> 5) - 1, ds = (int)tap - 3 * dr - 4;   // tap / 3 for taps 0..8
      const bool in = tap < 9 && (unsigned)(p + dr) < (unsigned)H && (unsigned)(q + ds) < (unsigned)W;
      const float x = src[in ? (dr * W + ds) * Cin + c : 0];
      v[e] = in ? x : 0.f;
    }
    store8(col + i * 8, v);
  }
}

__device__ __forceinline__ float block_reduce_max(float v, float* sh) {
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  float r = sh[0];
  for (int w = 1; w < (int)(blockDim.x >> 6); ++w) r = fmaxf(r, sh[w]);
  __syncthreads();
  return r;
}

__device__ __forceinline__ float block_reduce_sum(float v, float* sh) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  float r = sh[0];
  for (int w = 1; w < (int)(blockDim.x >> 6); ++w) r += sh[w];
  __syncthreads();
  return r;
}

// Global average pool of one sample into gs[0 .. C) (LDS), C a multiple of 8.  A thread takes 8 channels (16 bytes in
// bf16) of every S-th pixel and the S pixel slices are added in a fixed order: at 8x8 pixels x 64 channels two loads per
// thread where one thread per channel walked 64.  part: HEAD_PART floats of LDS.  Ends with a barrier.
constexpr int HEAD_PART = 16 * 260;   // >= 256 * 8, and 16 rows of 256 with a pad (fc_logits)
template <class T>
__device__ __forceinline__ void head_pool(const T* __restrict__ an, float* gs, float* part, int hw, int C) {
  const float inv_hw = 1.0f / (float)hw;
  const int groups = C >> 3;
  for (int g0 = 0; g0 < groups; g0 += 256) {
    const int ng = min(256, groups - g0), S = 256 / ng, sl = threadIdx.x / ng, gi = threadIdx.x - sl * ng;
    if (sl < S) {
      float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
      for (int i = sl; i < hw; i += S) {
        float v[8];
        load8(an + (size_t)i * C + (g0 + gi) * 8, v);
#pragma unroll
        for (int e = 0; e < 8; ++e) s[e] += v[e];
      }
      store8(part + (sl * ng + gi) * 8, s);
    }
    __syncthreads();
    for (int c = threadIdx.x; c < ng * 8; c += 256) {
      float t = 0.f;
#pragma unroll 8
      for (int k = 0; k < S; ++k) t += part[k * ng * 8 + c];
      gs[g0 * 8 + c] = t * inv_hw;
    }
    __syncthreads();
  }
}

// logits[j] = bias[j] + sum_c gs[c] * W[c][j] for one sample, all 256 threads at work whatever the class count.
// part: HEAD_PART floats of LDS.  Ends with a barrier; lg[0 .. classes) is then complete.
__device__ __forceinline__ void fc_logits(const float* gs, const float* __restrict__ wfc, const float* __restrict__ bfc, float* lg, float* part,
                                          int C, int classes) {
  if (classes <= 16) {
    // few classes (the benchmark heads have 10): every thread takes channels tid, tid + 256, ... for all classes -- its
    // loads are independent of each other (consecutive threads read consecutive weight rows) and in flight together,
    // where a thread per (class, channel slice) walked C/16 dependent steps.  The 256 partial sums of a class are a row
    // of LDS: 16 threads per class add 16 of them each, then their own by row rotations (16 wave-wide shuffle trees took 5 us).
    float acc[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[j] = 0.f;
    for (int c = threadIdx.x; c < C; c += 256) {
      const float gv = gs[c];
      const float* wr = wfc + (size_t)c * classes;
#pragma unroll
      for (int j = 0; j < 16; ++j)
        if (j < classes) acc[j] = fmaf(gv, wr[j], acc[j]);
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) part[j * 260 + threadIdx.x] = acc[j];
    __syncthreads();
    const int j = threadIdx.x >> 4, sl = threadIdx.x & 15;
    float v = 0.f;
#pragma unroll
    for (int k = 0; k < 16; ++k) v += part[j * 260 + k * 16 + sl];
    for (int o = 8; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if (sl == 0 && j < classes) lg[j] = bfc[j] + v;
    __syncthreads();
    return;
  }
  // the threads form CS slices over the channels x JT class lanes (JT = the power of two that covers min(classes, 256));
  // every thread sums its channel slice for its classes and the slices are added in a fixed order through LDS
  int jt = 1;
  while (jt < classes && jt < 256) jt <<= 1;
  const int cs_n = 256 / jt, jl = threadIdx.x % jt, cs = threadIdx.x / jt;
  for (int j0 = 0; j0 < classes; j0 += jt) {
    const int j = j0 + jl;
    float s = 0.f;
    if (j < classes)
      for (int c = cs; c < C; c += cs_n) s = fmaf(gs[c], wfc[(size_t)c * classes + j], s);
    part[cs * jt + jl] = s;
    __syncthreads();
    if (cs == 0 && j < classes) {
      float t = bfc[j];
      for (int k = 0; k < cs_n; ++k) t += part[k * jt + jl];
      lg[j] = t;
    }
    __syncthreads();
  }
}

// One block per sample.  Dynamic LDS: C + classes floats.  Bound by latency (4 to 32 blocks a micro-batch): 25 us at 8x8x64
// with a thread per channel in the pool and shuffle trees over the classes, now 6.0.
template <class T>
__global__ __launch_bounds__(256) void k_head_fwd(PtrTab as, const float* __restrict__ wfc, const float* __restrict__ bfc,
                                                  PtrTab labelss, PtrTab gs_, PtrTab dls, float* loss_accum, int hw, int C,
                                                  int classes, float inv_div) {
  const T* __restrict__ a = (const T*)pick(as, blockIdx.z);
  const int32_t* __restrict__ labels = (const int32_t*)pick(labelss, blockIdx.z);
  float* __restrict__ g = (float*)pick(gs_, blockIdx.z);
  float* __restrict__ dlogits = (float*)pick(dls, blockIdx.z);
  extern __shared__ __attribute__((aligned(16))) float dyn[];
  __shared__ float red[8];
  __shared__ __attribute__((aligned(16))) float part[HEAD_PART];
  float* gs = dyn;
  float* lg = dyn + C;
  const int n = blockIdx.x;
  const int y = labels[n];
  head_pool(a + (size_t)n * hw * C, gs, part, hw, C);
  for (int c = threadIdx.x; c < C; c += 256) g[(size_t)n * C + c] = gs[c];
  fc_logits(gs, wfc, bfc, lg, part, C, classes);
  float mx = -3.0e38f;
  for (int j = threadIdx.x; j < classes; j += blockDim.x) mx = fmaxf(mx, lg[j]);
  mx = block_reduce_max(mx, red);
  float den = 0.f;
  for (int j = threadIdx.x; j < classes; j += blockDim.x) den += expf(lg[j] - mx);
  den = block_reduce_sum(den, red);
  for (int j = threadIdx.x; j < classes; j += blockDim.x)
    dlogits[(size_t)n * classes + j] = (expf(lg[j] - mx) / den - (j == y ? 1.f : 0.f)) * inv_div;
  if (threadIdx.x == 0) atomicAdd(loss_accum, -(lg[y] - mx - logf(den)) * inv_div);
}

// Inference head, one block per sample: logits = mean_{h,w}(a) * Wfc + bfc.  Dynamic LDS: C + classes floats.
template <class T>
__global__ __launch_bounds__(256) void k_head_logits(PtrTab as, const float* __restrict__ wfc, const float* __restrict__ bfc,
                                                     PtrTab outs, int hw, int C, int classes) {
  const T* __restrict__ a = (const T*)pick(as, blockIdx.z);
  float* __restrict__ out = (float*)pick(outs, blockIdx.z);
  extern __shared__ __attribute__((aligned(16))) float dyn[];
  __shared__ __attribute__((aligned(16))) float part[HEAD_PART];
  float* gs = dyn;
  float* lg = dyn + C;
  const int n = blockIdx.x;
  head_pool(a + (size_t)n * hw * C, gs, part, hw, C);
  fc_logits(gs, wfc, bfc, lg, part, C, classes);
  for (int j = threadIdx.x; j < classes; j += blockDim.x) out[(size_t)n * classes + j] = lg[j];
}

// Blocks [0, b) of every member, one per sample: dbfc += dlogits, da[n,i,c] = (dlogits[n] . Wfc[c]) / hw.
// The blocks behind them (member 0 only): dWfc[c][j] += sum over the samples of all members of g[n][c] * dlogits[n][j], a
// thread per output element walking the samples (one atomic per element and launch; a block per sample adding its outer
// product cost b*g atomics per element).  One launch: the two parts do not depend on each other.
// Dynamic LDS: max(C + classes, ng * b * classes) floats.
template <class T>
__global__ __launch_bounds__(256) void k_head_bwd(PtrTab gs_, PtrTab dls, const float* __restrict__ wfc, float* g_wfc,
                                                  float* g_bfc, PtrTab das, int ng, int b, int hw, int C, int classes) {
  extern __shared__ float dyn[];
  if ((int)blockIdx.x >= b) {
    if (blockIdx.z != 0) return;
    for (int z = 0; z < ng; ++z) {
      const float* __restrict__ dl = (const float*)pick(dls, z);
      for (int i = threadIdx.x; i < b * classes; i += 256) dyn[z * b * classes + i] = dl[i];
    }
    __syncthreads();
    const int i = (blockIdx.x - b) * 256 + threadIdx.x;
    if (i >= C * classes) return;
    const int c = i / classes, j = i - c * classes;
    float s = 0.f;
    for (int z = 0; z < ng; ++z) {
      const float* __restrict__ g = (const float*)pick(gs_, z);
#pragma unroll 8
      for (int n = 0; n < b; ++n) s = fmaf(g[(size_t)n * C + c], dyn[(z * b + n) * classes + j], s);
    }
    atomicAdd(&g_wfc[i], s);
    return;
  }
  const float* __restrict__ dlogits = (const float*)pick(dls, blockIdx.z);
  T* __restrict__ da = (T*)pick(das, blockIdx.z);
  float* dl = dyn;          // classes
  float* dg = dyn + classes;  // C
  const int n = blockIdx.x;
  for (int j = threadIdx.x; j < classes; j += blockDim.x) {
    const float d = dlogits[(size_t)n * classes + j];
    dl[j] = d;
    atomicAdd(&g_bfc[j], d);
  }
  __syncthreads();
  const float inv_hw = 1.0f / (float)hw;
  for (int c = threadIdx.x; c < C; c += blockDim.x) {
    float s = 0.f;
    for (int j = 0; j < classes; ++j) s = fmaf(dl[j], wfc[(size_t)c * classes + j], s);
    dg[c] = s * inv_hw;
  }
  __syncthreads();
  T* dan = da + (size_t)n * hw * C;
  for (int i = threadIdx.x; i < hw * C; i += blockDim.x) from_f32(&dan[i], dg[i % C]);
}

// invalid (may be null): set when the batch's gradients are not to be trusted (an image-resident launch gave up
// waiting for its partners); the step then leaves parameters, momentum and gradients alone.
__global__ __launch_bounds__(256) void k_sgd(float* __restrict__ w, float* __restrict__ v, float* __restrict__ g,
                                             size_t n, float lr, float mu, const int* __restrict__ invalid) {
  if (invalid && *invalid) return;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const float vel = fmaf(mu, v[i], g[i]);
    v[i] = vel;
    w[i] = fmaf(-lr, vel, w[i]);
    g[i] = 0.f;
  }
}

__global__ __launch_bounds__(256) void k_zero_f32(float* __restrict__ p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0.f;
}

// Every work-group copies contiguous 16 KiB chunks (four 16-byte units per lane in flight) with streaming
// loads and stores: measured 5.6-5.9 TB/s on 1 GiB, against 4.2-4.6 TB/s for a grid-stride loop over the
// whole buffer and 4.8 TB/s for the runtime's device-to-device copy.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr size_t COPY_CHUNK = 1024;   // 16-byte units per work-group and step
__global__ __launch_bounds__(256) void k_copy16(u32x4* __restrict__ dst, const u32x4* __restrict__ src, size_t n16,
                                                unsigned char* dtail, const unsigned char* stail, int ntail) {
  for (size_t c0 = (size_t)blockIdx.x * COPY_CHUNK; c0 < n16; c0 += (size_t)gridDim.x * COPY_CHUNK) {
    const size_t i = c0 + threadIdx.x;
    if (c0 + COPY_CHUNK <= n16) {
      u32x4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = __builtin_nontemporal_load(src + i + u * 256);
#pragma unroll
      for (int u = 0; u < 4; ++u) __builtin_nontemporal_store(v[u], dst + i + u * 256);
    } else {
      for (size_t j = i; j < n16; j += 256) dst[j] = src[j];
    }
  }
  if (blockIdx.x == 0 && (int)threadIdx.x < ntail) dtail[threadIdx.x] = stail[threadIdx.x];
}

// eight consecutive columns of a row, in the fragment order
__device__ __forceinline__ void store_fragment(bf16_t* m, int row, int col, int rows, bool permuted, const uint4& v) {
  if (permuted) {
    *reinterpret_cast<uint2*>(m + fragment_at(row, col, rows, true)) = make_uint2(v.x, v.y);
    *reinterpret_cast<uint2*>(m + fragment_at(row, col + 4, rows, true)) = make_uint2(v.z, v.w);
  } else {
    *reinterpret_cast<uint4*>(m + fragment_at(row, col, rows, false)) = v;
  }
}

// bf16 operand copies of the convolution weights; STEP: behind the SGD step, which then needs no pass of its own (28 bytes per weight
// instead of 24 + 12, and one launch; 32 where register-resident kernels read the weights, whose fragment order is written beside the rows).  grid (Y, n_convs): the Y blocks of a convolution share its 64 x 64 tiles of the fp32 master
// [k = tap*Cin + c][n] round-robin.  A tile is updated as it is loaded, and the copies are written from LDS with 16-byte stores: the
// forward one is its transpose, the data-gradient one takes its rows.  Channel counts and offsets are multiples of 16 (the stem's Cin
// excepted).  Parameters that are no convolution weights follow the convolution in front of them (rest_*; the first also the ones before it).
// The blocks of a convolution are consecutive, so they go to all dies: with the convolutions in x a matrix stayed on the dies that x mod 8 gave it
// (the last quarter of VGG-16, 16.8 of 23.6 M weights in one of four matrices: 197 us, now 95).
// ResNet-20 (0.27 M parameters): 4.5 + 25 us as two launches with a serial data-gradient copy, now 6.2; VGG-16 (33.6 M): 129 + 77, now 143.
template <bool STEP>
__global__ __launch_bounds__(256) void k_sgd_pack(float* __restrict__ params, float* __restrict__ mom, float* __restrict__ grads,
                                                  bf16_t* __restrict__ packed, const PackDesc* __restrict__ table, float lr, float mu,
                                                  const int* __restrict__ invalid) {
  if (STEP && invalid && *invalid) return;
  __shared__ float tile[64][65];
  const PackDesc d = table[blockIdx.y];
  const int tid = threadIdx.x;
  if (STEP) {
    for (int part = 0; part < 2; ++part) {
      const size_t off = part ? d.rest_off : 0;
      const int len = part ? d.rest_len : d.first_len;
      for (int i = blockIdx.x * 256 + tid; i < len; i += gridDim.x * 256) {
        const float vel = fmaf(mu, mom[off + i], grads[off + i]);
        mom[off + i] = vel;
        params[off + i] = fmaf(-lr, vel, params[off + i]);
        grads[off + i] = 0.f;
      }
    }
  }
  const int ktot = d.T * d.Cin, tk = (d.Kf + 63) / 64, tn = (d.Cout + 63) / 64;
  bf16_t* wf = packed + d.wf_off;  // [Cout][Kf], k = tap*Cin + c
  for (int t = blockIdx.x; t < tk * tn; t += gridDim.x) {
    const int k0 = (t / tn) * 64, n0 = (t % tn) * 64;
    __syncthreads();
    {
      // load: a thread takes 4 consecutive n of one k row (16 lanes per row, 16 rows per pass)
      const int c4 = (tid & 15) * 4, r0 = tid >> 4;
      float4 w[4], v[4], g[4];
      bool on[4];
      size_t at[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int k = k0 + r0 + 16 * i, n = n0 + c4;
        on[i] = k < ktot && n < d.Cout;
        at[i] = d.w_off + (on[i] ? (size_t)k * d.Cout + n : (size_t)0);
        w[i] = *reinterpret_cast<const float4*>(params + at[i]);
        if (STEP) { v[i] = *reinterpret_cast<const float4*>(mom + at[i]); g[i] = *reinterpret_cast<const float4*>(grads + at[i]); }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (STEP) {
          v[i].x = fmaf(mu, v[i].x, g[i].x); v[i].y = fmaf(mu, v[i].y, g[i].y); v[i].z = fmaf(mu, v[i].z, g[i].z); v[i].w = fmaf(mu, v[i].w, g[i].w);
          w[i].x = fmaf(-lr, v[i].x, w[i].x); w[i].y = fmaf(-lr, v[i].y, w[i].y); w[i].z = fmaf(-lr, v[i].z, w[i].z); w[i].w = fmaf(-lr, v[i].w, w[i].w);
          if (on[i]) {
            *reinterpret_cast<float4*>(params + at[i]) = w[i];
            *reinterpret_cast<float4*>(mom + at[i]) = v[i];
            *reinterpret_cast<float4*>(grads + at[i]) = make_float4(0.f, 0.f, 0.f, 0.f);
          }
        }
        if (!on[i]) w[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        float* q = &tile[r0 + 16 * i][c4];
        q[0] = w[i].x; q[1] = w[i].y; q[2] = w[i].z; q[3] = w[i].w;
      }
    }
    __syncthreads();
    // store: a thread takes 8 consecutive elements of a row of either copy (8 lanes per row, 32 rows per pass)
    const int e8 = (tid & 7) * 8;
#pragma unroll
    for (int r = tid >> 3; r < 64; r += 32) {
      const int n = n0 + r, k = k0 + e8;
      if (n < d.Cout && k < d.Kf) {
        uint4 st;
        st.x = pack_bf16x2(tile[e8][r], tile[e8 + 1][r]); st.y = pack_bf16x2(tile[e8 + 2][r], tile[e8 + 3][r]);
        st.z = pack_bf16x2(tile[e8 + 4][r], tile[e8 + 5][r]); st.w = pack_bf16x2(tile[e8 + 6][r], tile[e8 + 7][r]);
        *reinterpret_cast<uint4*>(wf + (size_t)n * d.Kf + k) = st;
        if (d.ff_off != ~0ull) store_fragment(packed + d.ff_off, n, k, d.Cout, d.f_perm, st);
      }
    }
    if (d.wd_off == ~0ull) continue;
#pragma unroll
    for (int r = tid >> 3; r < 64; r += 32) {
      const int k = k0 + r, n = n0 + e8;
      if (k >= ktot) continue;
      const int tap = k / d.Cin, c = k - tap * d.Cin;
      bf16_t* row = packed + d.wd_off + (size_t)c * d.Kd;   // [Cin][Kd], k = tap*Cout + n
      if (n < d.Cout) {
        const float* q = &tile[r][e8];
        uint4 st;
        st.x = pack_bf16x2(q[0], q[1]); st.y = pack_bf16x2(q[2], q[3]); st.z = pack_bf16x2(q[4], q[5]); st.w = pack_bf16x2(q[6], q[7]);
        *reinterpret_cast<uint4*>(row + tap * d.Cout + n) = st;
        if (d.fd_off != ~0ull) store_fragment(packed + d.fd_off, c, tap * d.Cout + n, d.Cin, d.d_perm, st);
      }
      if (tap == d.T - 1 && n0 + 64 >= d.Cout)              // padding
        for (int p = d.T * d.Cout + e8; p < d.Kd; p += 64) {
          *reinterpret_cast<uint4*>(row + p) = make_uint4(0u, 0u, 0u, 0u);
          if (d.fd_off != ~0ull) store_fragment(packed + d.fd_off, c, p, d.Cin, d.d_perm, make_uint4(0u, 0u, 0u, 0u));
        }
    }
  }
}

// LDS of the pooling heads: C + classes floats beside head_pool's and fc_logits' own.  Up to 64 KiB together needs nothing; above it
// the limit of the kernel is stated first (not a stream operation, so a capture does not see it).
constexpr size_t HEAD_MAX_DYN = 63 * 1024;
hipError_t head_lds(const void* kernel, size_t dyn) {
  if (dyn > HEAD_MAX_DYN) return hipErrorInvalidValue;
  if (dyn + (HEAD_PART + 8) * sizeof(float) <= 64 * 1024) return hipSuccess;
  return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)HEAD_MAX_DYN);
}

unsigned grid_for(size_t n, unsigned cap = 2048) {
  size_t g = (n + 255) / 256;
  if (g < 1) g = 1;
  return (unsigned)(g > cap ? cap : g);
}

}  // namespace

hipError_t launch_im2col3x3(int ng, const PtrTab& img, const PtrTab& col, int b, int H, int W, int Cin, int Kc,
                            hipStream_t stream) {
  if (Kc % 8 != 0) return hipErrorInvalidValue;
  k_im2col3x3<<<dim3(grid_for((size_t)b * H * W * (Kc / 8)), 1, (unsigned)ng), 256, 0, stream>>>(img, col, b, H, W, Cin, Kc);
  return hipGetLastError();
}

hipError_t launch_head_fwd(int dt, int ng, const PtrTab& a, const float* wfc, const float* bfc, const PtrTab& labels,
                           const PtrTab& gp, const PtrTab& dlogits, float* loss_accum, int b, int hw, int C,
                           int classes, float divisor, hipStream_t stream) {
  const size_t lds = (size_t)(C + classes) * sizeof(float);
  const dim3 grid((unsigned)b, 1, (unsigned)ng);
  const hipError_t e = head_lds(dt == DT_BF16 ? reinterpret_cast<const void*>(k_head_fwd<bf16_t>) : reinterpret_cast<const void*>(k_head_fwd<float>), lds);
  if (e != hipSuccess) return e;
  if (dt == DT_BF16)
    k_head_fwd<bf16_t><<<grid, 256, lds, stream>>>(a, wfc, bfc, labels, gp, dlogits, loss_accum, hw, C, classes, 1.0f / divisor);
  else
    k_head_fwd<float><<<grid, 256, lds, stream>>>(a, wfc, bfc, labels, gp, dlogits, loss_accum, hw, C, classes, 1.0f / divisor);
  return hipGetLastError();
}

hipError_t launch_head_logits(int dt, int ng, const PtrTab& a, const float* wfc, const float* bfc, const PtrTab& logits, int b,
                              int hw, int C, int classes, hipStream_t stream) {
  const size_t lds = (size_t)(C + classes) * sizeof(float);
  const dim3 grid((unsigned)b, 1, (unsigned)ng);
  const hipError_t e = head_lds(dt == DT_BF16 ? reinterpret_cast<const void*>(k_head_logits<bf16_t>) : reinterpret_cast<const void*>(k_head_logits<float>), lds);
  if (e != hipSuccess) return e;
  if (dt == DT_BF16) k_head_logits<bf16_t><<<grid, 256, lds, stream>>>(a, wfc, bfc, logits, hw, C, classes);
  else k_head_logits<float><<<grid, 256, lds, stream>>>(a, wfc, bfc, logits, hw, C, classes);
  return hipGetLastError();
}

hipError_t launch_head_bwd(int dt, int ng, const PtrTab& gp, const PtrTab& dlogits, const float* wfc, float* g_wfc,
                           float* g_bfc, const PtrTab& da, int b, int hw, int C, int classes, hipStream_t stream) {
  const size_t wl = (size_t)ng * b * classes * sizeof(float), bl = (size_t)(C + classes) * sizeof(float);
  if (wl > 48 * 1024) return hipErrorInvalidValue;
  const dim3 grid((unsigned)(b + (C * classes + 255) / 256), 1, (unsigned)ng);
  const size_t lds = wl > bl ? wl : bl;
  if (dt == DT_BF16)
    k_head_bwd<bf16_t><<<grid, 256, lds, stream>>>(gp, dlogits, wfc, g_wfc, g_bfc, da, ng, b, hw, C, classes);
  else
    k_head_bwd<float><<<grid, 256, lds, stream>>>(gp, dlogits, wfc, g_wfc, g_bfc, da, ng, b, hw, C, classes);
  return hipGetLastError();
}

hipError_t launch_sgd(float* w, float* v, float* g, size_t n, float lr, float mu, const int* invalid, hipStream_t stream) {
  k_sgd<<<grid_for(n, 4096), 256, 0, stream>>>(w, v, g, n, lr, mu, invalid);
  return hipGetLastError();
}

hipError_t launch_zero_f32(float* p, size_t n, hipStream_t stream) {
  k_zero_f32<<<grid_for(n, 4096), 256, 0, stream>>>(p, n);
  return hipGetLastError();
}

namespace {
constexpr int MAX_GRID_Y = 65535;
// blocks per convolution: one per tile of the largest one (blocks with nothing to do leave at once)
dim3 pack_grid(int n_convs, size_t max_elems) {
  const size_t y = (max_elems + 4095) / 4096;
  return dim3((unsigned)(y < 8 ? 8 : (y > 1024 ? 1024 : y)), (unsigned)(n_convs < MAX_GRID_Y ? n_convs : MAX_GRID_Y));
}
}  // namespace

hipError_t launch_pack_weights(const float* params, bf16_t* packed, const PackDesc* table_dev, int n_convs, size_t max_elems,
                               hipStream_t stream) {
  if (n_convs <= 0) return hipSuccess;
  for (int c = 0; c < n_convs; c += MAX_GRID_Y)
    k_sgd_pack<false><<<pack_grid(n_convs - c, max_elems), 256, 0, stream>>>(const_cast<float*>(params), nullptr, nullptr, packed, table_dev + c, 0.f, 0.f, nullptr);
  return hipGetLastError();
}

hipError_t launch_sgd_pack(float* params, float* mom, float* grads, bf16_t* packed, const PackDesc* table_dev, int n_convs, size_t max_elems,
                           float lr, float mu, const int* invalid, hipStream_t stream) {
  for (int c = 0; c < n_convs; c += MAX_GRID_Y)
    k_sgd_pack<true><<<pack_grid(n_convs - c, max_elems), 256, 0, stream>>>(params, mom, grads, packed, table_dev + c, lr, mu, invalid);
  return hipGetLastError();
}

// Register-only MFMA loops: independent accumulator tiles per wave, `iters` rounds of one MFMA on each.  No
// memory traffic inside the loop; the sums are written once so that the loop cannot be dropped.  The MFMA is
// written as an in-place accumulate (the builtin in this loop shape made the compiler rotate the accumulators
// through ~70 register moves per round, which measured the moves, not the matrix unit).
// WIDE = false: 8 tiles of v_mfma_f32_16x16x32_bf16; WIDE = true: 4 tiles of v_mfma_f32_32x32x16_bf16 (twice the
// flop per instruction): 131 072 flop per round and wave either way.
template <bool WIDE>
__global__ __launch_bounds__(256) void k_probe_mfma_bf16(float* __restrict__ sink, int iters) {
  typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
  typedef float floatx4 __attribute__((ext_vector_type(4)));
  typedef float floatx16 __attribute__((ext_vector_type(16)));
  const uint32_t seed = 0x3f803f80u + ((threadIdx.x & 7u) << 16);   // bf16 pairs near 1.0
  const bf16x8 a = __builtin_bit_cast(bf16x8, make_uint4(seed, seed ^ 0x00010000u, seed, seed ^ 0x00000001u));
  const bf16x8 b = __builtin_bit_cast(bf16x8, make_uint4(seed ^ 0x80000000u, seed, seed ^ 0x00008000u, seed));
  float t = 0.f;
  if (WIDE) {
    floatx16 acc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
    for (int it = 0; it < iters; ++it) {
#pragma unroll
      for (int i = 0; i < 4; ++i) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc[i]) : "v"(a), "v"(b));
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) t += acc[i][e];
  } else {
    floatx4 acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int it = 0; it < iters; ++it) {
#pragma unroll
      for (int i = 0; i < 8; ++i) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc[i]) : "v"(a), "v"(b));
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) t += acc[i][0] + acc[i][1] + acc[i][2] + acc[i][3];
  }
  sink[(size_t)blockIdx.x * 256 + threadIdx.x] = t;
}

hipError_t launch_probe_mfma_bf16(float* sink, int workgroups, int iters, bool wide, hipStream_t stream) {
  if (wide) k_probe_mfma_bf16<true><<<workgroups, 256, 0, stream>>>(sink, iters);
  else k_probe_mfma_bf16<false><<<workgroups, 256, 0, stream>>>(sink, iters);
  return hipGetLastError();
}

hipError_t launch_copy_bytes(void* dst, const void* src, size_t bytes, hipStream_t stream) {
  const size_t n16 = bytes / 16;
  const int ntail = (int)(bytes - n16 * 16);
  const size_t chunks = (n16 + COPY_CHUNK - 1) / COPY_CHUNK;
  const unsigned grid = (unsigned)(chunks < 1 ? 1 : chunks > (1u << 20) ? (1u << 20) : chunks);
  k_copy16<<<grid, 256, 0, stream>>>((u32x4*)dst, (const u32x4*)src, n16, (unsigned char*)dst + n16 * 16,
                                                    (const unsigned char*)src + n16 * 16, ntail);
  return hipGetLastError();
}

}  // namespace hpf
