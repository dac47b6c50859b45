// What the bf16 attention kernels (hpd_attn_stream.hip, hpd_attn_dense.hip) share: their arguments, loads to LDS,
// conversions, the rotation of a row.
#pragma once

#include "hpd_internal.h"
#include "hpd_device.h"

// What the lookup of a workgroup's descriptor takes stands in front of these in a kernel's arguments, which the build has
// loaded into registers before the kernel starts: the descriptor is requested at once instead of behind a trip for the
// arguments (us a step, before -> now: fp32, 8 prompts x 12 branches 11.4 -> 11.1; 32 prompts x 16 branches 24.4 -> 24.0;
// launches of several rounds as before: there the arguments are in the scalar cache).  The launch functions take them from here, so that both are the same.
struct StreamArgs {
  hpd_dev_tables tb;
  int32_t step, Hq, Hkv, Tcap, RG, n_groups, out_f32, fused, live_base;
  int32_t Gr;  // query heads per kv head; the kernel's G is the next power of two (padding rows are neither loaded nor stored)
  int32_t at_once;  // attn_dense_kernel: all workgroups run at a time, if three per CU do
  int64_t NP;
  float scale_log2;
};

// decode attention of launches with many rows per unit (hpd_attn_dense.hip); G: the kernel's rows per branch
hipError_t hpd_launch_attention_dense(const hpd_layout* L, StreamArgs a, int32_t G, bool paper, const void* q,
                                      const void* k_prefix, const void* v_prefix, void* k_tail, void* v_tail,
                                      const void* k_new, const void* v_new, void* out, hipStream_t s);

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int D = 128;
constexpr int SLOT_U4 = 16 * 64;  // one 32-key block: 8 K + 8 V fragments of 64 x 16 bytes
constexpr float NEG_BIG = -1.0e30f;
// read-only for the whole launch: a wave-uniform address is read through the scalar cache
typedef __attribute__((address_space(4))) int32_t const_i32;

enum { MODE_BLOCK = 0, MODE_PAPER = 1, MODE_PREFILL = 2, MODE_PAGED = 3, MODE_PREFILL_LIST = 4 };

#define HPD_GLL(gptr, lptr)                                                                   \
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(gptr),   \
                                   (__attribute__((address_space(3))) void*)(lptr), 16, 0, 0)
// the same with the streaming (non-temporal) cache hint
#define HPD_GLL_NT(gptr, lptr)                                                                \
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(gptr),   \
                                   (__attribute__((address_space(3))) void*)(lptr), 16, 0, 2)

__device__ __forceinline__ uint32_t cvt_pk_bf16(float lo, float hi) {
  floatx2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ bf16x8 pack8(const float* v) {
  uint4 u;
  u.x = cvt_pk_bf16(v[0], v[1]); u.y = cvt_pk_bf16(v[2], v[3]);
  u.z = cvt_pk_bf16(v[4], v[5]); u.w = cvt_pk_bf16(v[6], v[7]);
  return __builtin_bit_cast(bf16x8, u);
}
__device__ __forceinline__ void unpack8(uint4 a, float out[8]) {
  out[0] = __uint_as_float(a.x << 16); out[1] = __uint_as_float(a.x & 0xffff0000u);
  out[2] = __uint_as_float(a.y << 16); out[3] = __uint_as_float(a.y & 0xffff0000u);
  out[4] = __uint_as_float(a.z << 16); out[5] = __uint_as_float(a.z & 0xffff0000u);
  out[6] = __uint_as_float(a.w << 16); out[7] = __uint_as_float(a.w & 0xffff0000u);
}
// 8 keys of the cache: rounded to bf16, written as halves
__device__ __forceinline__ uint4 pack8_key(const float* v) {
  float r[8];
  unpack8(__builtin_bit_cast(uint4, pack8(v)), r);
  return make_uint4(hpd::cache_bits_pair(r[0], r[1]), hpd::cache_bits_pair(r[2], r[3]),
                    hpd::cache_bits_pair(r[4], r[5]), hpd::cache_bits_pair(r[6], r[7]));
}
// 8 bf16 values as cache elements
__device__ __forceinline__ uint4 cache8(uint4 w) {
  return make_uint4(hpd::cache_bits_from_bf16_pair(w.x), hpd::cache_bits_from_bf16_pair(w.y),
                    hpd::cache_bits_from_bf16_pair(w.z), hpd::cache_bits_from_bf16_pair(w.w));
}
// 8 values (of the query, of the softmax weights) as halves, rounded to nearest
__device__ __forceinline__ f16x8 pack8_half(const float* v) {
  f16x8 h;
#pragma unroll
  for (int e = 0; e < 8; ++e) h[e] = (_Float16)v[e];
  return h;
}
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
constexpr float MAX_SLACK = 8.f;  // log2 units: how far a score may exceed the reference point of its row

// c + the two halves of w (v_dot2_f32_f16 with a pair of ones)
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float sum_half_pair(uint32_t w, float c) {
  return __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, w), __builtin_bit_cast(f16x2, 0x3c003c00u), c, false);
}

// A 32-bit word at a wave-uniform address through the scalar data cache (read only).  The
// loaders use it for table lookups: a vector load would have to wait for every DMA instruction
// in front of it, because vector memory operations of a wave complete in order.
__device__ __forceinline__ int32_t scalar_load(const int32_t* p) {
  // (the address is wave-uniform by the caller's construction; where the compiler keeps it in
  // vector registers all the same, it is moved to scalar ones here)
  const uint64_t u = reinterpret_cast<uint64_t>(p);
  // (readfirstlane returns a signed int: without the casts a low half with its top bit set
  // would be sign-extended over the high half)
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(u >> 32));
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)u);
  p = reinterpret_cast<const int32_t*>(((uint64_t)hi << 32) | (uint64_t)lo);
  int32_t v;
  asm volatile("s_load_dword %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)" : "=s"(v) : "s"(p) : "memory");
  return v;
}

// the same address in scalar registers: wave-uniform by the caller's construction
__device__ __forceinline__ const char* uniform(const char* p) {
  const uint64_t u = reinterpret_cast<uint64_t>(p);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(u >> 32));
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)u);
  return reinterpret_cast<const char*>(((uint64_t)hi << 32) | (uint64_t)lo);
}

// 8 channel pairs (c .. c+7, 64+c .. 64+c+7) of one row, rotated at the (cos, sin) row cs_row
__device__ __forceinline__ void rotate16(uint4 raw_lo, uint4 raw_hi, const float2* cs_row, int c,
                                         float rl[8], float rh[8]) {
  float lo[8], hi[8];
  unpack8(raw_lo, lo);
  unpack8(raw_hi, hi);
  const float4* csp = reinterpret_cast<const float4*>(cs_row + c);
#pragma unroll
  for (int e2 = 0; e2 < 4; ++e2) {
    const float4 cs = csp[e2];
    hpd::rope_pair(lo[2 * e2], hi[2 * e2], cs.x, cs.y, rl[2 * e2], rh[2 * e2]);
    hpd::rope_pair(lo[2 * e2 + 1], hi[2 * e2 + 1], cs.z, cs.w, rl[2 * e2 + 1], rh[2 * e2 + 1]);
  }
}

}  // namespace
