// Device-side helpers shared by the gfx950 kernels: bf16 storage conversions and
// 16-byte vector access.  bf16 values are stored as raw uint16 bit patterns.
#pragma once
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "kernels.h"

// Launch helper: plain hipLaunchKernelGGL, or hipExtLaunchKernelGGL with the profiler's
// pending events (then cleared) when a profiled launch is in progress.
#define FF_LAUNCH(kernel, grid, block, shmem, stream, ...)                                          \
  do {                                                                                              \
    ::ff::LaunchEvents& ff_ev_ = ::ff::g_launch_events;                                             \
    if (ff_ev_.start) {                                                                             \
      hipExtLaunchKernelGGL(kernel, grid, block, shmem, stream, ff_ev_.start, ff_ev_.stop, 0, __VA_ARGS__); \
      ff_ev_.start = ff_ev_.stop = nullptr;                                                         \
    } else {                                                                                        \
      hipLaunchKernelGGL(kernel, grid, block, shmem, stream, __VA_ARGS__);                          \
    }                                                                                               \
  } while (0)

namespace ff {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));  // 16-byte moves (native vector, not a struct)
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

// fp32 -> bf16, round to nearest even (NaN stays NaN): gfx950's v_cvt_pk_bf16_f32, one
// instruction per pair instead of the integer rounding sequence per value.
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  const f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

// Storage traits: 8 elements per 16-byte chunk for bf16, 4 for fp32.
template <int DT> struct St;
template <> struct St<DT_BF16> {
  static constexpr int V = 8;
  __device__ __forceinline__ static void load(const void* p, size_t i, float* v) {
    uint4 w = *reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(p) + i);
    uint32_t a[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[2 * j] = __uint_as_float(a[j] << 16);
      v[2 * j + 1] = __uint_as_float(a[j] & 0xffff0000u);
    }
  }
  __device__ __forceinline__ static void store(void* p, size_t i, const float* v) {
    uint32_t a[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) a[j] = pack_bf16x2(v[2 * j], v[2 * j + 1]);
    *reinterpret_cast<uint4*>(reinterpret_cast<uint16_t*>(p) + i) = make_uint4(a[0], a[1], a[2], a[3]);
  }
  // the same 16-byte load with the non-temporal hint, for data read once (history slots)
  __device__ __forceinline__ static void load_nt(const void* p, size_t i, float* v) {
    const u32x4_t w = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(reinterpret_cast<const uint16_t*>(p) + i));
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[2 * j] = __uint_as_float(w[j] << 16);
      v[2 * j + 1] = __uint_as_float(w[j] & 0xffff0000u);
    }
  }
  __device__ __forceinline__ static float rnd(float x) { return bf2f(f2bf(x)); }
  __device__ __forceinline__ static float ld1(const void* p, size_t i) {
    return bf2f(reinterpret_cast<const uint16_t*>(p)[i]);
  }
  __device__ __forceinline__ static void st1(void* p, size_t i, float x) {
    reinterpret_cast<uint16_t*>(p)[i] = f2bf(x);
  }
};
template <> struct St<DT_F32> {
  static constexpr int V = 4;
  __device__ __forceinline__ static void load(const void* p, size_t i, float* v) {
    float4 w = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(p) + i);
    v[0] = w.x; v[1] = w.y; v[2] = w.z; v[3] = w.w;
  }
  __device__ __forceinline__ static void store(void* p, size_t i, const float* v) {
    *reinterpret_cast<float4*>(reinterpret_cast<float*>(p) + i) = make_float4(v[0], v[1], v[2], v[3]);
  }
  __device__ __forceinline__ static void load_nt(const void* p, size_t i, float* v) {
    const f32x4_t w = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(reinterpret_cast<const float*>(p) + i));
    v[0] = w[0]; v[1] = w[1]; v[2] = w[2]; v[3] = w[3];
  }
  __device__ __forceinline__ static float rnd(float x) { return x; }
  __device__ __forceinline__ static float ld1(const void* p, size_t i) {
    return reinterpret_cast<const float*>(p)[i];
  }
  __device__ __forceinline__ static void st1(void* p, size_t i, float x) {
    reinterpret_cast<float*>(p)[i] = x;
  }
};

__device__ __forceinline__ float silu_f(float x) { return x / (1.0f + expf(-x)); }

// GELU, tanh form: 0.5 z (1 + tanh(u)) with u = sqrt(2/pi) (z + 0.044715 z^3).  Since
// 1 + tanh(u) = 2 / (1 + exp(-2u)), this is z / (1 + exp(-2u)) = z / (1 + 2^(z (c1 + c3 z^2)))
// with c1 = -2 log2(e) sqrt(2/pi) and c3 = 0.044715 c1 folded into the polynomial: five
// VALU operations, one hardware exp2 (v_exp_f32) and one reciprocal (v_rcp_f32), a few
// ulp of fp32 and no branches (the epilogue of the MLP's first GEMM is bound by this
// arithmetic).  For u -> -inf the exp overflows to +inf and the result is -0; for
// u -> +inf it is z.
__device__ __forceinline__ float gelu_tanh_f(float z) {
  const float c1 = -2.302208198144325f;    // -2 log2(e) sqrt(2/pi)
  const float c3 = -0.1029432395800235f;   // 0.044715 * c1
  const float e = __builtin_amdgcn_exp2f(z * fmaf(c3, z * z, c1));   // exp(-2u)
  return z * __builtin_amdgcn_rcpf(1.0f + e);
}

// Sum over the 64 lanes of a wavefront (fixed butterfly order: deterministic).
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

inline int cdiv(long a, long b) { return (int)((a + b - 1) / b); }

// ---------------------------------------------------------------- LDS reads and DMA by hand
// Kernels that keep global -> LDS DMA in flight across their LDS reads issue both by hand:
// the compiler would wait for all DMA before a read that may alias it.  A fragment read
// here is complete after an s_waitcnt lgkmcnt that covers it and must then pass FF_TIE
// before its first use, in the same straight-line code, so that no use or copy moves above
// the wait.
#define FF_AS1(p) ((const __attribute__((address_space(1))) void*)(p))
#define FF_AS3(p) ((__attribute__((address_space(3))) void*)(p))
#define FF_TIE(x) asm volatile("" : "+v"(x))

template <int OFF>
__device__ __forceinline__ bf16x8_t lds_rd128_at(uint32_t addr) {
  static_assert(OFF >= 0 && OFF < 65536, "LDS immediate offset");
  u32x4_t v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF) : "memory");
  return __builtin_bit_cast(bf16x8_t, v);
}
// the same with an offset that is a constant once the caller's loop is unrolled
__device__ __forceinline__ bf16x8_t lds_rd128_off(uint32_t addr, int off) {
  u32x4_t v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "i"(off) : "memory");
  return __builtin_bit_cast(bf16x8_t, v);
}
// 4 rows x 16 columns of 16-bit elements per 16 lanes, transposed: lane i of the 16 addresses
// row i / 4, columns 4 (i % 4) .. + 3 and gets column i, rows 0-3
__device__ __forceinline__ u32x2_t lds_rd64_tr(uint32_t addr, int off) {
  u32x2_t v;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "i"(off) : "memory");
  return v;
}
template <int N>
__device__ __forceinline__ void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
template <int V> struct Int { static constexpr int value = V; };
// f(Int<I>) for I = A .. B - 1
template <int A, int B, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (A < B) {
    f(Int<A>{});
    static_for<A + 1, B>(f);
  }
}

}  // namespace ff
