// Arguments and small helpers shared by the GEMM kernels.
#pragma once

#include "device.h"
#include "kernels.h"

namespace jetk {

template <typename T>
struct GemmArgs {
  const T *A;
  const T *B;
  int64_t lda, ldb;
  int M, N;
  int K, KA, KB;  // K steps over K columns; A column k mod KA, B column k mod KB
  void *out;
  int64_t ldo;
  int pair_out;   // SwiGLU / QKV-RoPE: write (hi, lo) pairs
  float oscale;   // every product is multiplied by oscale before the epilogue
  QkvRope rope;   // EPI_QKV_ROPE only
  // grouped GEMM: row tile t uses B + tile_group[t] * group_stride; tiles
  // with tile_group -1 do nothing (null: one B for all tiles)
  const int *tile_group = nullptr;
  int64_t group_stride = 0;
  // int8 B (LOAD 9 configurations): fp16 scales [K / 32][ceil(N / 128)][32][4]
  const uint16_t *Bs = nullptr;
};

// silu(gate) * up, silu(g) = g / (1 + e^-g) with the hardware reciprocal (~1
// ulp). PAIR (the result is split into a (hi, lo) pair): the product is rounded
// before the remainder v - hi is taken from it. Left to the compiler, a fused
// multiply-subtract may take it from the unrounded product in one kernel and
// not in another, and a row's last bits would depend on its tile.
template <bool PAIR>
__device__ __forceinline__ float swiglu(float gate, float up) {
  float v = gate * __builtin_amdgcn_rcpf(1.0f + __expf(-gate)) * up;
  if constexpr (PAIR) asm("" : "+v"(v));
  return v;
}

// (hi, lo) split of v stored at p[0] and p[ps] (lo only with pair).
template <typename T>
__device__ __forceinline__ void put_split(T *p, int64_t ps, float v, int pair) {
  const T hi = from_f<T>(v);
  p[0] = hi;
  if (pair) p[ps] = from_f<T>(v - to_f<T>(hi));
}

// Kernels whose LDS exceeds the default 64 KB limit must opt in once.
template <class C>
static hipError_t allow_lds(const void *fn) {
  if (C::LDS_BYTES <= 65536) return hipSuccess;
  return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::LDS_BYTES);
}

}  // namespace jetk
