// Device-side helpers shared by the HIP kernels: bf16 conversion and 8-element vector access.
#pragma once
#include "hpf_kernels.h"

namespace hpf {

// Member z of a pointer table passed by value in the kernel arguments.  A chain of scalar selects:
// indexing the argument struct with a run-time index would make the compiler copy it to scratch memory.
__device__ __forceinline__ void* pick(const PtrTab& t, unsigned z) {
  void* r = t.p[0];
#pragma unroll
  for (int i = 1; i < MAX_GROUP; ++i) r = (z == (unsigned)i) ? t.p[i] : r;
  return r;
}

__device__ __forceinline__ float bf16_to_f32(bf16_t h) { return __uint_as_float((uint32_t)h << 16); }

// float -> bfloat16, round-to-nearest-even, two at a time: one v_cvt_pk_bf16_f32 on gfx950
typedef __bf16 hpf_bf16x2 __attribute__((ext_vector_type(2)));
typedef float hpf_floatx2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  const hpf_floatx2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, hpf_bf16x2));
}
__device__ __forceinline__ bf16_t f32_to_bf16(float f) { return (bf16_t)(pack_bf16x2(f, 0.f) & 0xffffu); }

// 8 consecutive elements <-> 8 floats
__device__ __forceinline__ void load8(const float* p, float (&v)[8]) {
  const float4 a = *reinterpret_cast<const float4*>(p);
  const float4 b = *reinterpret_cast<const float4*>(p + 4);
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
__device__ __forceinline__ void load8(const bf16_t* p, float (&v)[8]) {
  const uint4 a = *reinterpret_cast<const uint4*>(p);
  v[0] = __uint_as_float(a.x << 16); v[1] = __uint_as_float(a.x & 0xffff0000u);
  v[2] = __uint_as_float(a.y << 16); v[3] = __uint_as_float(a.y & 0xffff0000u);
  v[4] = __uint_as_float(a.z << 16); v[5] = __uint_as_float(a.z & 0xffff0000u);
  v[6] = __uint_as_float(a.w << 16); v[7] = __uint_as_float(a.w & 0xffff0000u);
}
__device__ __forceinline__ void store8(float* p, const float (&v)[8]) {
  *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
  *reinterpret_cast<float4*>(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
}
__device__ __forceinline__ void store8(bf16_t* p, const float (&v)[8]) {
  uint4 a;
  a.x = pack_bf16x2(v[0], v[1]); a.y = pack_bf16x2(v[2], v[3]);
  a.z = pack_bf16x2(v[4], v[5]); a.w = pack_bf16x2(v[6], v[7]);
  *reinterpret_cast<uint4*>(p) = a;
}

__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(bf16_t v) { return bf16_to_f32(v); }
__device__ __forceinline__ void from_f32(float* p, float v) { *p = v; }
__device__ __forceinline__ void from_f32(bf16_t* p, float v) { *p = f32_to_bf16(v); }

// Sums within a row of 16 lanes by DPP row rotations (one VALU instruction per step, no LDS round trip).
// row_sum<N>(v): every lane gets the sum over the lanes of its row that are congruent to it modulo N.
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
template <int N>
__device__ __forceinline__ float row_sum(float v) {
  static_assert(N == 1 || N == 2 || N == 4 || N == 8 || N == 16, "N divides 16");
  if (N <= 8) v += dpp_mov<0x128>(v);   // row_ror:8
  if (N <= 4) v += dpp_mov<0x124>(v);   // row_ror:4
  if (N <= 2) v += dpp_mov<0x122>(v);   // row_ror:2
  if (N <= 1) v += dpp_mov<0x121>(v);   // row_ror:1
  return v;
}
__device__ __forceinline__ float sum16(float v) { return row_sum<1>(v); }   // over the 16 pixels of a tile

// Where the consumer of a BatchNorm takes its {mean, invstd} from (bf16 mode).
enum : int { BN_FROM_STATS = 0, BN_FROM_RECORDS = 1, BN_FROM_RUNNING = 2 };
// Records of row blocks ([row][C]) are added up in one order wherever it is done, so a result does not depend on who does it: row b belongs
// to group b % FIN_GROUPS, a group is added in ascending rows and the groups in ascending order.  A work-group of 256 threads takes nch <= 64
// channels; FinMap: thread j * nch + cl has the rows j, j + rg, ... of channel cl, which are `vg` groups.  FIN_RECS records of a thread are in
// flight together, so up to FIN_RECS * rg rows cost one round trip.
constexpr int FIN_RECS = 8, FIN_GROUPS = 16, FIN_SH = FIN_GROUPS * 64;   // FIN_SH: floats of LDS, a row of 64 channels per group
struct FinMap {
  int nch, rg, vg, j, cl;
  bool on;
  __device__ __forceinline__ explicit FinMap(int nch_) : nch(nch_), rg(nch_ > 32 ? 4 : nch_ > 16 ? 8 : 16), vg(FIN_GROUPS / rg) {
    j = (int)threadIdx.x / nch;
    cl = (int)threadIdx.x - j * nch;
    on = j < rg;
  }
};
// Sums of a thread's groups
struct FinAcc {
  float a[4] = {0.f, 0.f, 0.f, 0.f};
  template <class V>
  __device__ __forceinline__ void add(const FinMap& m, V v) {   // v(i): value of the thread's record i in a round of FIN_RECS * rg rows
    if (m.vg == 4) {
#pragma unroll
      for (int i = 0; i < FIN_RECS; ++i) a[i & 3] += v(i);
    } else if (m.vg == 2) {
#pragma unroll
      for (int i = 0; i < FIN_RECS; ++i) a[i & 1] += v(i);
    } else {
#pragma unroll
      for (int i = 0; i < FIN_RECS; ++i) a[0] += v(i);
    }
  }
  __device__ __forceinline__ void store(const FinMap& m, float* sh) const {
    if (!m.on) return;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (k < m.vg) sh[(m.j + k * m.rg) * 64 + m.cl] = a[k];
  }
  static __device__ __forceinline__ float sum(const FinMap& m, const float* sh) {
    float t = sh[m.cl];
#pragma unroll
    for (int g = 1; g < FIN_GROUPS; ++g) t += sh[g * 64 + m.cl];
    return t;
  }
};
// {mean, invstd} of channels [c_base, c_base + nch), nch <= 64, from the statistics records {K, S1, S2, n} of nrows row blocks
// ([row][C], S1 / S2 sums about K), by a work-group of 256 threads; out(c, mean, invstd) is called by one thread per channel.
// Two passes: the mean from the block sums, then the squared deviations about it, M2 = sum [S2 - S1^2/n + n (mean_b - mean)^2].
// sh: FIN_SH floats of LDS.
template <class OUT>
__device__ __forceinline__ void bn_finalize_records(const float4* __restrict__ rec, unsigned nrows, int C, int c_base, int nch, int M, float eps,
                                                    float* sh, OUT out) {
  const FinMap m(nch);
  const int c = c_base + m.cl;
  const bool on = m.on && c < C;
  const char* p = (const char*)rec;
  const unsigned row_bytes = (unsigned)C * 16, col = (unsigned)c * 16;
  float4 q[FIN_RECS];
  auto load = [&](unsigned b0) {   // all loads in flight together
#pragma unroll
    for (int i = 0; i < FIN_RECS; ++i) {
      const unsigned b = b0 + (unsigned)(m.j + i * m.rg);
      q[i] = on && b < nrows ? *(const float4*)(p + (b * row_bytes + col)) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  };
  const unsigned step = (unsigned)(FIN_RECS * m.rg);
  FinAcc acc;
  for (unsigned b0 = 0; b0 < nrows; b0 += step) {
    load(b0);
    acc.add(m, [&](int i) { return q[i].w * q[i].x + q[i].y; });   // n*K + S1 = sum of the block's values
  }
  if (nrows > step) load(0);   // on its way during the sum over the groups
  auto publish = [&](const FinAcc& a) {
    __syncthreads();
    a.store(m, sh);
    __syncthreads();
  };
  publish(acc);
  const float mean = FinAcc::sum(m, sh) / (float)M;
  FinAcc dev;
  for (unsigned b0 = 0;;) {
    dev.add(m, [&](int i) {                   // squared deviations of the block about the overall mean
      if (!(q[i].w > 0.f)) return 0.f;
      const float s1n = q[i].y / q[i].w, d = q[i].x + s1n - mean;
      return q[i].z - q[i].y * s1n + q[i].w * d * d;
    });
    b0 += step;
    if (b0 >= nrows) break;
    load(b0);
  }
  publish(dev);
  if (on && m.j == 0) {
    float var = FinAcc::sum(m, sh) / (float)M;
    var = var > 0.f ? var : 0.f;
    out(c, mean, 1.0f / sqrtf(var + eps));
  }
}

}  // namespace hpf
