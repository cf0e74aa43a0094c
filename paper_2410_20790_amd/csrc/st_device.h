// Device helpers shared by the gfx950 kernels: storage types and their
// conversions, activations, 8-channel vectors and the pre-activation state's
// storage.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

namespace st {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));

struct bf16_t {
  uint16_t v;
};

// ------------------------------------------------------------ conversions
__device__ __forceinline__ float to_f(float x) { return x; }
__device__ __forceinline__ float to_f(_Float16 x) { return (float)x; }
__device__ __forceinline__ float to_f(bf16_t x) {
  return __uint_as_float((uint32_t)x.v << 16);
}
template <typename T> __device__ __forceinline__ T from_f(float x);
template <> __device__ __forceinline__ float from_f<float>(float x) {
  return x;
}
template <> __device__ __forceinline__ _Float16 from_f<_Float16>(float x) {
  return (_Float16)x;  // hardware conversion, round to nearest even
}
template <> __device__ __forceinline__ bf16_t from_f<bf16_t>(float x) {
  // hardware conversion (gfx950), round to nearest even
  return bf16_t{__builtin_bit_cast(uint16_t, (__bf16)x)};
}
template <typename T> __device__ __forceinline__ T zero_v() {
  return from_f<T>(0.f);
}

// Activation f: 0 identity, 1 ReLU, 2 SiLU (x / (1 + e^-x)).
template <int ACT>
__device__ __forceinline__ float act_c(float x) {
  if constexpr (ACT == 1)
    return __builtin_amdgcn_fmed3f(x, 0.f, __builtin_inff());  // max(x, 0)
  else if constexpr (ACT == 2)
    return x / (1.f + expf(-x));
  else
    return x;
}
__device__ __forceinline__ float act_f(float x, int a) {
  if (a == 1) return act_c<1>(x);
  if (a == 2) return act_c<2>(x);
  return x;
}
// Calls f(std::integral_constant<int, ACT>{}) for the activation act, so
// that f's body is built once per activation.
template <class F>
__device__ __forceinline__ void with_act(int act, F&& f) {
  if (act == 1)
    f(std::integral_constant<int, 1>{});
  else if (act == 2)
    f(std::integral_constant<int, 2>{});
  else
    f(std::integral_constant<int, 0>{});
}

// 8 consecutive storage elements <-> 8 floats (16- or 32-byte aligned).
template <typename T> struct Vec8;
template <> struct Vec8<float> {
  __device__ __forceinline__ static void load(const float* p, float* f) {
    const float4 a = *(const float4*)p, b = *(const float4*)(p + 4);
    f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w;
    f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
  }
  // stores the rounded values, returns their largest magnitude
  __device__ __forceinline__ static float store(float* p, const float* f) {
    *(float4*)p = make_float4(f[0], f[1], f[2], f[3]);
    *(float4*)(p + 4) = make_float4(f[4], f[5], f[6], f[7]);
    float m = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) m = fmaxf(m, fabsf(f[e]));
    return m;
  }
};
template <typename T> struct Vec8Half {
  __device__ __forceinline__ static void load(const T* p, float* f) {
    const uint4 v = *(const uint4*)p;
    const T* h = (const T*)&v;
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = to_f(h[e]);
  }
  // stores the rounded values, returns their largest magnitude: rounding
  // to nearest is monotone and odd, so that is the rounded largest
  // magnitude of the unrounded values (one conversion instead of eight)
  __device__ __forceinline__ static float store(T* p, const float* f) {
    uint4 v;
    T* h = (T*)&v;
    float m = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      h[e] = from_f<T>(f[e]);
      m = fmaxf(m, fabsf(f[e]));
    }
    *(uint4*)p = v;
    return to_f(from_f<T>(m));
  }
};
template <> struct Vec8<_Float16> : Vec8Half<_Float16> {};
template <> struct Vec8<bf16_t> : Vec8Half<bf16_t> {};

// Stores a[e] * b[e] - c[e], f16 rounded once from the exact product and
// difference (the mixed-precision multiply-add; left to the compiler it is
// that or an f32 result rounded again, by how it vectorised the code around);
// returns what Vec8::store of the f32 results would.
template <typename T>
__device__ __forceinline__ float store8_fma(T* p, const float* a,
                                            const float* b, const float* c) {
  float f[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) f[e] = __builtin_fmaf(a[e], b[e], -c[e]);
  if constexpr (__is_same(T, _Float16)) {
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    uint32_t* h = (uint32_t*)&v;
    float m = 0.f;
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      asm("v_fma_mixlo_f16 %0, %1, %2, -%3"
          : "+v"(h[e / 2])
          : "v"(a[e]), "v"(b[e]), "v"(c[e]));
      asm("v_fma_mixhi_f16 %0, %1, %2, -%3"
          : "+v"(h[e / 2])
          : "v"(a[e + 1]), "v"(b[e + 1]), "v"(c[e + 1]));
      m = fmaxf(m, fmaxf(fabsf(f[e]), fabsf(f[e + 1])));
    }
    *(uint4*)p = v;
    return to_f(from_f<_Float16>(m));
  } else {
    return Vec8<T>::store(p, f);
  }
}

__device__ __forceinline__ void load8f(const float* p, float* f) {
  Vec8<float>::load(p, f);
}
__device__ __forceinline__ void store8f(float* p, const float* f) {
  *(float4*)p = make_float4(f[0], f[1], f[2], f[3]);
  *(float4*)(p + 4) = make_float4(f[4], f[5], f[6], f[7]);
}

// The values a row of type T holds after rounding, as f32, added to zero (the
// view that a residual-carry reference frame starts from its emitted rows: no
// -0, as in a view that rows were added to).
template <typename T>
__device__ __forceinline__ void store8f_rounded(float* p, const float* f) {
  float r[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] = to_f(from_f<T>(f[e])) + 0.f;
  store8f(p, r);
}

// 8-channel vectors of a site that adjacent threads of a 256-thread block
// take in the dense pass's per-site kernels: all of them, or the largest
// divisor between 16 and 64 (no thread idle), or 64.
inline int octets_per_block(int v) {
  if (v <= 64) return v;
  for (int t = 64; t >= 16; --t)
    if (v % t == 0) return t;
  return 64;
}

// Pre-activation state storage: f32, or bf16 (nets created with a bf16
// state), which holds every value rounded to nearest even.  `half` is the
// net's choice (uniform); indices count values, not bytes.
__device__ __forceinline__ float state_round(bool half, float x) {
  return half ? to_f(from_f<bf16_t>(x)) : x;
}
__device__ __forceinline__ void state_load8(const float* P, bool half,
                                            int64_t i, float* f) {
  if (half)
    Vec8<bf16_t>::load((const bf16_t*)P + i, f);
  else
    load8f(P + i, f);
}
__device__ __forceinline__ void state_store8(float* P, bool half, int64_t i,
                                             const float* f) {
  if (half)
    (void)Vec8<bf16_t>::store((bf16_t*)P + i, f);
  else
    store8f(P + i, f);
}
__device__ __forceinline__ float4 state_load4(const float* P, bool half,
                                              int64_t i) {
  if (!half) return *(const float4*)(P + i);
  const uint2 v = *(const uint2*)((const bf16_t*)P + i);
  const bf16_t* h = (const bf16_t*)&v;
  return make_float4(to_f(h[0]), to_f(h[1]), to_f(h[2]), to_f(h[3]));
}
__device__ __forceinline__ void state_store4(float* P, bool half, int64_t i,
                                             float4 f) {
  if (!half) {
    *(float4*)(P + i) = f;
    return;
  }
  uint2 v;
  bf16_t* h = (bf16_t*)&v;
  h[0] = from_f<bf16_t>(f.x);
  h[1] = from_f<bf16_t>(f.y);
  h[2] = from_f<bf16_t>(f.z);
  h[3] = from_f<bf16_t>(f.w);
  *(uint2*)((bf16_t*)P + i) = v;
}
// The gate slot in use: base + (*par ^ flip) * sz (two slots of one
// squeeze-excitation layer's per-image gates, chosen by a parity word in
// device memory so that a captured frame replays with either).
__device__ __forceinline__ const float* gate_slot(const float* base,
                                                  const int* par, int64_t sz,
                                                  int flip) {
  return base + (int64_t)((*par) ^ flip) * sz;
}
__device__ __forceinline__ float state_load1(const float* P, bool half,
                                             int64_t i) {
  return half ? to_f(((const bf16_t*)P)[i]) : P[i];
}

}  // namespace st
