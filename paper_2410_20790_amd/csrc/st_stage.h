// Staged operands of the matrix products that go from global memory straight
// into LDS (gfx950): 128-byte rows of eight 16-byte slots, slot s of row r
// holding the row's vector s ^ (r & 7), set by the address each lane loads
// from.  S stages live in S separate LDS arrays.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "st_device.h"
#include "st_kernels.h"

namespace st {

// ------------------------------------------- shared by the gather kernels
__device__ __forceinline__ unsigned lane_prefix(u64 ballot) {
  return __builtin_amdgcn_mbcnt_hi((unsigned)(ballot >> 32),
                                   __builtin_amdgcn_mbcnt_lo((unsigned)ballot,
                                                             0u));
}

// Four channels of a delta row stored in the storage type; returns the
// largest magnitude of the rounded values (the rounded largest magnitude,
// as rounding to nearest is monotone and odd).
template <typename T>
__device__ __forceinline__ float store4(T* p, const float* f) {
  float m = 0.f;
#pragma unroll
  for (int e = 0; e < 4; ++e) m = fmaxf(m, fabsf(f[e]));
  if constexpr (sizeof(T) == 4) {
    *(float4*)p = make_float4(f[0], f[1], f[2], f[3]);
    return m;
  } else {
    uint2 v;
    T* h = (T*)&v;
#pragma unroll
    for (int e = 0; e < 4; ++e) h[e] = from_f<T>(f[e]);
    *(uint2*)p = v;
    return to_f(from_f<T>(m));
  }
}

// Splits of the reduction per output tile for this frame: enough work units
// (tiles x splits) to give every CU several, at most split_max (which leaves
// every split at least kSplitStages of the planner's stages).  The kernels
// that write the partial tiles and the split epilogue that adds them derive
// it from the same two numbers, whatever the stages of either; the dense pass
// sums in as many parts (st_dense.hip).
constexpr int kSplitTarget = 1024;
__host__ __device__ __forceinline__ int split_count(int64_t ntiles,
                                                    int split_max) {
  if (split_max <= 1 || ntiles <= 0) return 1;
  const int64_t sp = (kSplitTarget + ntiles - 1) / ntiles;
  return sp < split_max ? (int)sp : split_max;
}

// Reduction stages of a layer that hold real (not padding) columns, for
// stages of KC columns.
template <int KC>
__device__ __forceinline__ int gemm_stages_kc(const ConvArgs& a) {
  return min((int)a.ktot_p, (a.K * a.cin_p + KC - 1) / KC * KC) / KC;
}

// --------------------------------------------------------- staged rows
constexpr int kRowBytes = 128;  // a staged row: 64 half or 32 f32 columns
__device__ __forceinline__ void load_to_lds(const void* g, char* lds) {
  __builtin_amdgcn_global_load_lds(
      (__attribute__((address_space(1))) const uint32_t*)(uintptr_t)g,
      (__attribute__((address_space(3))) uint32_t*)lds, 16, 0, 0);
}

// Wait until at most N of this wave's vector-memory operations are
// outstanding (and its LDS reads are done), then meet the block's waves.
template <int N>
__device__ __forceinline__ void stage_ready() {
  static_assert(N < 64, "vmcnt");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | ((N >> 4) << 14));
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// One stage's products from the stage buffer: WM pixels (in blocks of 16,
// from row pr) by WN channels (weight rows from wr).
template <typename T, int IM, int JN>
__device__ __forceinline__ void stage_products(const char* buf, int pr,
                                               int wr, int l16, int lg,
                                               v4f (&acc)[IM][JN]) {
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) {
    const int slot = ((kk * 4 + lg) ^ (l16 & 7)) * 16;
    uint4 pv[IM], wv[JN];
#pragma unroll
    for (int i = 0; i < IM; ++i)
      pv[i] = *(const uint4*)(buf + (pr + i * 16 + l16) * kRowBytes + slot);
#pragma unroll
    for (int j = 0; j < JN; ++j)
      wv[j] = *(const uint4*)(buf + (wr + (j >> 1) * 32 + (l16 >> 2) * 8 +
                                     (j & 1) * 4 + (l16 & 3)) *
                                        kRowBytes +
                              slot);
#pragma unroll
    for (int i = 0; i < IM; ++i) {
#pragma unroll
      for (int j = 0; j < JN; ++j) {
        if constexpr (sizeof(T) == 4) {
          const float4 w = __builtin_bit_cast(float4, wv[j]);
          const float4 p = __builtin_bit_cast(float4, pv[i]);
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.x, p.x,
                                                           acc[i][j], 0, 0, 0);
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.y, p.y,
                                                           acc[i][j], 0, 0, 0);
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.z, p.z,
                                                           acc[i][j], 0, 0, 0);
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.w, p.w,
                                                           acc[i][j], 0, 0, 0);
        } else if constexpr (__is_same(T, _Float16)) {
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
              __builtin_bit_cast(v8h, wv[j]), __builtin_bit_cast(v8h, pv[i]),
              acc[i][j], 0, 0, 0);
        } else {
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              __builtin_bit_cast(v8bf, wv[j]), __builtin_bit_cast(v8bf, pv[i]),
              acc[i][j], 0, 0, 0);
        }
      }
    }
  }
}

// One turn of the stage ring: stage `rd` has arrived once at most AHEAD
// later loads of this wave are outstanding; the loads of the stage S - 1
// ahead go to `wr`, which every wave finished reading before the barrier.
template <typename T, int BM, int AHEAD, int IM, int JN, class Loader>
__device__ __forceinline__ void stage_turn(const ConvArgs& a, Loader& ld,
                                           const char* __restrict__ rd,
                                           char* __restrict__ wr, int pr,
                                           int wrow, int l16, int lg,
                                           v4f (&acc)[IM][JN]) {
  stage_ready<AHEAD>();
  ld.template issue<BM>(a, wr);
  stage_products<T, IM, JN>(rd, pr, wrow, l16, lg, acc);
}

}  // namespace st
