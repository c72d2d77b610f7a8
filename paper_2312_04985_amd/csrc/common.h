// Device-side helpers shared by the libsparq kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sparq {

constexpr int kWave = 64;
constexpr float kLog2e = 1.4426950408889634f;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// ---- 16-bit storage formats: exact widening to fp32, round-to-nearest-even narrowing ----
struct F16 {
  static __device__ __forceinline__ float lo(uint32_t w) {
    return (float)__builtin_bit_cast(_Float16, (uint16_t)(w & 0xffffu));
  }
  static __device__ __forceinline__ float hi(uint32_t w) {
    return (float)__builtin_bit_cast(_Float16, (uint16_t)(w >> 16));
  }
  static __device__ __forceinline__ float widen(uint16_t c) { return (float)__builtin_bit_cast(_Float16, c); }
  static __device__ __forceinline__ uint16_t narrow(float x) { return __builtin_bit_cast(uint16_t, (_Float16)x); }
  // c[m][n] += sum_k a[m][k] b[n][k] over 32 k: lane l holds a[l % 16], b[l % 16] at k = 8 (l / 16) .. + 7 and
  // c[4 (l / 16) + i][l % 16]
  static __device__ __forceinline__ f32x4 mfma_16x16x32(const uint4& a, const uint4& b, f32x4 c) {
    typedef _Float16 v8 __attribute__((ext_vector_type(8)));
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8, a), __builtin_bit_cast(v8, b), c, 0, 0, 0);
  }
};

struct BF16 {
  static __device__ __forceinline__ float lo(uint32_t w) { return __uint_as_float(w << 16); }
  static __device__ __forceinline__ float hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
  static __device__ __forceinline__ float widen(uint16_t c) { return __uint_as_float((uint32_t)c << 16); }
  static __device__ __forceinline__ uint16_t narrow(float x) {
    uint32_t u = __float_as_uint(x);
    u += 0x7fffu + ((u >> 16) & 1u);   // finite inputs only
    return (uint16_t)(u >> 16);
  }
  static __device__ __forceinline__ f32x4 mfma_16x16x32(const uint4& a, const uint4& b, f32x4 c) {   // as F16's
    typedef __bf16 v8 __attribute__((ext_vector_type(8)));
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8, a), __builtin_bit_cast(v8, b), c, 0, 0, 0);
  }
};

template <class T>
__device__ __forceinline__ void unpack8(const uint4& v, float (&f)[8]) {
  f[0] = T::lo(v.x); f[1] = T::hi(v.x); f[2] = T::lo(v.y); f[3] = T::hi(v.y);
  f[4] = T::lo(v.z); f[5] = T::hi(v.z); f[6] = T::lo(v.w); f[7] = T::hi(v.w);
}

// 16 bytes of cache data: every such load in this library reads what the launch uses once (rows of Kt, K and V,
// sorted keys), so it is marked non-temporal: the line is not kept in L2 or in the memory-side cache on account of
// this read.  Measured against plain loads: the decode step 6-10 % faster on every many-head workload (512 heads
// of 4096 positions 52.8 -> 47.6 us, 2048 of 8192 157.3 -> 147.4, 512 ragged ones of 256 channels 243.6 -> 222.1), 1-3 % slower only where the query heads of
// a KV group select for themselves in the one-launch kernel and find each other's rows in L2.
// KEEP: an ordinary load, for lines that other workgroups of the launch use too.
template <class V, bool KEEP = false>
__device__ __forceinline__ V load16_as(const void* p) {
  if (KEEP) return __builtin_bit_cast(V, *reinterpret_cast<const u32x4*>(p));
  return __builtin_bit_cast(V, __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p)));
}
__device__ __forceinline__ uint4 load16(const void* p) { return load16_as<uint4>(p); }

// ---- order-preserving map fp32 -> uint32 (larger float <=> larger key; -0 == +0) ----
// Every finite float maps to a key >= 0x00800000, so key 0 is below all of them.
__device__ __forceinline__ uint32_t float_to_key(float x) {
  const uint32_t u = __float_as_uint(x + 0.0f);          // (-0 becomes +0)
  return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}
__device__ __forceinline__ float key_to_float(uint32_t k) {
  return __uint_as_float(k ^ (~(uint32_t)((int32_t)k >> 31) | 0x80000000u));
}

// 2^x as the hardware's one instruction.  exp2f() wraps it in range scaling so that results below 2^-126 come
// out as denormals; a softmax weight that small adds nothing to a sum whose largest term is 1.
__device__ __forceinline__ float exp2_weight(float x) { return __builtin_amdgcn_exp2f(x); }

// log2 of a number that is no denormal, as the hardware's one instruction (log2f() scales denormals first).
__device__ __forceinline__ float log2_normal(float x) { return __builtin_amdgcn_logf(x); }

// ---- wave64 primitives (DPP: no LDS traffic, a few cycles each) ----
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float lane_f(float v, int lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}
// Butterfly all-reduce over aligned groups of N lanes (N = 8 or 16): xor 1 and xor 2 by quad
// permutes, then half-row mirror and row mirror, which act as xor 4 / xor 8 once the quads (halves)
// are uniform.  Every step adds a pair commutatively, so all lanes of a group end with the same bits.
template <int N>
__device__ __forceinline__ float group_sum(float v) {
  v += dpp_f<0xB1>(v);                  // quad_perm [1,0,3,2]
  v += dpp_f<0x4E>(v);                  // quad_perm [2,3,0,1]
  v += dpp_f<0x141>(v);                 // row_half_mirror
  if (N >= 16) v += dpp_f<0x140>(v);    // row_mirror
  return v;
}
template <int N>
__device__ __forceinline__ float group_max(float v) {
  v = fmaxf(v, dpp_f<0xB1>(v));
  v = fmaxf(v, dpp_f<0x4E>(v));
  v = fmaxf(v, dpp_f<0x141>(v));
  if (N >= 16) v = fmaxf(v, dpp_f<0x140>(v));
  return v;
}
// reductions over the whole wave: the result is wave-uniform
__device__ __forceinline__ float wave_sum(float v) {
  v = group_sum<16>(v);
  return (lane_f(v, 0) + lane_f(v, 16)) + (lane_f(v, 32) + lane_f(v, 48));
}
__device__ __forceinline__ float wave_max(float v) {
  v = group_max<16>(v);
  return fmaxf(fmaxf(lane_f(v, 0), lane_f(v, 16)), fmaxf(lane_f(v, 32), lane_f(v, 48)));
}
// Lanes l and l ^ O (O = 8, 16, 32) as a pair: both get (a, b) = (value of the lower, value of the upper), so that what they
// make of it is the same.  Rows and halves of a wave change places in one vector instruction, 8 lanes by DPP.
template <int O>
__device__ __forceinline__ void lane_pair(float v, float& a, float& b) {
  const uint32_t u = __float_as_uint(v);
  if (O == 8) {                          // row_ror:8
    const uint32_t w = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)u, 0x128, 0xf, 0xf, false);
    const bool upper = (threadIdx.x & 8u) != 0;
    a = __uint_as_float(upper ? w : u); b = __uint_as_float(upper ? u : w);
  } else if (O == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    a = __uint_as_float(r[0]); b = __uint_as_float(r[1]);
  } else {
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    a = __uint_as_float(r[0]); b = __uint_as_float(r[1]);
  }
}
// sum over aligned groups of LPR lanes (8, 16 or 32), same value in every lane of a group
template <int LPR>
__device__ __forceinline__ float lanes_sum(float v) {
  if (LPR == 8) return group_sum<8>(v);
  v = group_sum<16>(v);
  if (LPR == 32) {
    float a, b;
    lane_pair<16>(v, a, b);
    v = a + b;
  }
  return v;
}
// inclusive prefix sum across the 64 lanes with DPP row shifts and row broadcasts
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_or_zero(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xf, false);
}
__device__ __forceinline__ uint32_t wave_scan_incl(uint32_t v) {
  v += dpp_or_zero<0x111, 0xf>(v);   // row_shr:1
  v += dpp_or_zero<0x112, 0xf>(v);   // row_shr:2
  v += dpp_or_zero<0x114, 0xf>(v);   // row_shr:4
  v += dpp_or_zero<0x118, 0xf>(v);   // row_shr:8   -> scan inside each row of 16
  v += dpp_or_zero<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
  v += dpp_or_zero<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
  return v;
}

// LDS words that other lanes of the same wave wrote (a wave's LDS accesses are served in order: this only keeps the
// compiler from moving them past each other)
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// ---- results handed to the workgroup of a group that finishes last, inside one launch ----
// The workgroups of a launch run on 8 XCDs whose L2 caches do not see each other's lines.  What one of them leaves for
// another is therefore stored and loaded with agent scope (past the L2), word by word: a release fence would write
// the whole L2 back, which was measured as four times the time of a launch.
__device__ __forceinline__ void store_agent(float* p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ float load_agent(const float* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void store_agent(double* p, double v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ double load_agent(const double* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// 16 bytes at byte offset `off` of `base` (wave-uniform), the same way (bit 4 of the cache policy is the agent scope's sc1)
__device__ __forceinline__ void store_agent4(const float* base, uint32_t off, const float4& v) {
  const u32x4 w = {__float_as_uint(v.x), __float_as_uint(v.y), __float_as_uint(v.z), __float_as_uint(v.w)};
  __builtin_amdgcn_raw_buffer_store_b128(w, __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, 0xffffffffu, 0x00027000), off, 0, 16);
}
__device__ __forceinline__ float4 load_agent4(const float* base, uint32_t off) {
  const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(__builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, 0xffffffffu, 0x00027000), off, 0, 16);
  return make_float4(__uint_as_float(w.x), __uint_as_float(w.y), __uint_as_float(w.z), __uint_as_float(w.w));
}

// Called by all threads of each of the `n` workgroups of a group after their store_agent calls; true in all threads of
// the one that arrives last, whose load_agent calls then see every store of the others: each wave waits until its own
// stores have been acknowledged, the workgroup's waves meet, and only then one thread counts the workgroup in.
// The counter is 0 before the launch and is left 0.  No workgroup waits for another.  `flag`: one word of LDS.
__device__ __forceinline__ bool last_to_arrive(int* counter, int n, int* flag) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    const int before = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (before == n - 1) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *flag = before == n - 1;
  }
  __syncthreads();
  asm volatile("" ::: "memory");
  return *flag != 0;
}

// exp2 that maps (-inf) - (-inf) situations to weight 0 instead of NaN
__device__ __forceinline__ float weight_exp2(float m, float m_ref) {
  return (m == -INFINITY) ? 0.0f : exp2_weight(m - m_ref);
}

}  // namespace sparq
