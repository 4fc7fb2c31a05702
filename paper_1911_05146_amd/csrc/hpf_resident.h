// Device-side helpers shared by the image-resident kernels (kernels_resident.hip, kernels_resident_reg.hip).
#pragma once
#include "hpf_device.h"
#include "hpf_wait.h"

namespace hpf {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef unsigned long long u64;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int RES_NT = 512;            // threads per work-group (8 waves)
constexpr int RES_NWV = RES_NT / 64;

// The wave's index within the work-group as a scalar: conditions on it become scalar branches instead of
// compare / exec-mask sequences.
__device__ __forceinline__ int wave_index() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }

__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// {scale, shift} of a BatchNorm channel: bn(x) = x*scale + shift
__device__ __forceinline__ float2 bn_scale_shift(float mean, float invstd, float gamma, float beta) {
  const float sc = gamma * invstd;
  return make_float2(sc, fmaf(-mean, sc, beta));
}

__device__ __forceinline__ void publish_word(u64* slot, int me, int nw, int w, float v, unsigned tag) {
  __hip_atomic_store(slot + (size_t)me * nw + w, ((u64)tag << 32) | (u64)__float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bf16x8 frag_bn_relu(const uint4& q, const float2 (&cf)[8]) {
  const uint32_t w[4] = {q.x, q.y, q.z, q.w};
  uint32_t r[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    r[i] = pack_bf16x2(fmaxf(fmaf(bf_lo(w[i]), cf[2 * i].x, cf[2 * i].y), 0.f),
                       fmaxf(fmaf(bf_hi(w[i]), cf[2 * i + 1].x, cf[2 * i + 1].y), 0.f));
  return __builtin_bit_cast(bf16x8, make_uint4(r[0], r[1], r[2], r[3]));
}
__device__ __forceinline__ bf16x8 frag_zero() { return __builtin_bit_cast(bf16x8, make_uint4(0u, 0u, 0u, 0u)); }
__device__ __forceinline__ uint2 pack4(const floatx4& v) { return make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])); }
__device__ __forceinline__ float elem4(const uint2& q, int e) {
  return e == 0 ? bf_lo(q.x) : e == 1 ? bf_hi(q.x) : e == 2 ? bf_lo(q.y) : bf_hi(q.y);
}
struct ResCtx {
  char* base; void* act_in; void* act_out; void* err_in; void* err_out;
  __device__ __forceinline__ bf16_t* tensor(unsigned long long off) const {
    void* p = base + off;
    p = off == RES_ACT_IN ? act_in : p;
    p = off == RES_ACT_OUT ? act_out : p;
    p = off == RES_ERR_IN ? err_in : p;
    p = off == RES_ERR_OUT ? err_out : p;
    return (bf16_t*)p;
  }
};

}  // namespace
}  // namespace hpf
