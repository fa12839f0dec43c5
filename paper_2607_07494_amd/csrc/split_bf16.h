// Device helpers of the split-bf16 products (k_lowrank.hip, k_strip.hip): hi /
// lo splits, the three-product accumulation, LDS fragment slots, stores and
// waits that leave loads in flight.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gift {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ float4 ld4(const float *p) { return *reinterpret_cast<const float4 *>(p); }
__device__ __forceinline__ float4 zero4() { return make_float4(0.f, 0.f, 0.f, 0.f); }
// 16 bytes at p when ok, else zeros.  p must be a valid address either way:
// the load itself is unconditional and the zeros come from a select, because
// a load under a branch makes every later wait for loads a full one.
__device__ __forceinline__ float4 ld4_if(bool ok, const float *p) {
  const float4 v = ld4(p);
  return ok ? v : zero4();
}

// Stores the compiler does not track.  On this target a store and a load in
// flight share one counter, and the compiler, seeing both kinds pending,
// turns every wait for a load into a wait for everything; with these stores
// its waits cover its own loads only.  The hardware counter still counts the
// stores, so those waits can only last longer, never too short.  The s_nop
// gives a wide store the wait state it needs before its data registers may
// be rewritten.
__device__ __forceinline__ void st_u32_untracked(void *p, uint32_t v) {
  asm volatile("global_store_dword %0, %1, off\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");
}
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void st_u128_untracked(void *p, uint4 v) {
  const u32x4_t w = {v.x, v.y, v.z, v.w};
  asm volatile("global_store_dwordx4 %0, %1, off\n\ts_nop 1" ::"v"(p), "v"(w) : "memory");
}

// 4 x 4 transpose across the four 16-lane rows: word t of lane row u <-> word
// u of lane row t
__device__ __forceinline__ uint4 transpose_rows(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3) {
  const auto a = __builtin_amdgcn_permlane32_swap(w0, w2, false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(w1, w3, false, false);
  const auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
  const auto d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
  return make_uint4(c[0], c[1], d[0], d[1]);
}

// hi / lo bf16 pairs of two float32 values (round to nearest even)
__device__ __forceinline__ void split2(float x, float y, uint32_t &hi, uint32_t &lo) {
  const bf16x2 h = __builtin_convertvector((floatx2){x, y}, bf16x2);
  hi = __builtin_bit_cast(uint32_t, h);
  const float hx = __uint_as_float(hi << 16), hy = __uint_as_float(hi & 0xffff0000u);
  const bf16x2 l = __builtin_convertvector((floatx2){x - hx, y - hy}, bf16x2);
  lo = __builtin_bit_cast(uint32_t, l);
}

// eight float32 values (a: steps 0-3, b: steps 4-7) -> hi and lo fragments
__device__ __forceinline__ void split8(const float4 &a, const float4 &b, uint4 &hi, uint4 &lo) {
  split2(a.x, a.y, hi.x, lo.x);
  split2(a.z, a.w, hi.y, lo.y);
  split2(b.x, b.y, hi.z, lo.z);
  split2(b.z, b.w, hi.w, lo.w);
}

__device__ __forceinline__ bf16x8 frag(const uint4 &v) { return __builtin_bit_cast(bf16x8, v); }

__device__ __forceinline__ floatx4 mfma3(const uint4 &ahi, const uint4 &alo, const uint4 &bhi,
                                         const uint4 &blo, floatx4 acc) {
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag(ahi), frag(bhi), acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag(ahi), frag(blo), acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag(alo), frag(bhi), acc, 0, 0, 0);
  return acc;
}

__device__ __forceinline__ int lds_slot(int c, int g) { return 4 * c + (g ^ ((c >> 2) & 3)); }

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const uint32_t u = (uint32_t)__shfl_xor((int)v, o);
    v = u > v ? u : v;
  }
  return v;
}

#define GIFT_LDS __attribute__((address_space(3)))

// s_waitcnt vmcnt(N) alone (expcnt and lgkmcnt at their maxima): at most N
// vector memory operations of this wave still outstanding
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt is six bits");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// A workgroup barrier for LDS written by copies that other copies still in
// flight do not touch: this wave's vector-memory operations down to N
// outstanding (its copies that must have landed) and all its LDS accesses
// done, then the barrier.  No memory fence: a workgroup-scope release would
// also wait for the copies meant to stay in flight across the barrier.  The
// empty asm statements keep the compiler from moving memory accesses across.
template <int N>
__device__ __forceinline__ void copies_barrier() {
  static_assert(N >= 0 && N < 64, "vmcnt is six bits");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (0 << 8));
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

}  // namespace
}  // namespace gift
