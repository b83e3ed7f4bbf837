// Shared by the attention kernels.
#pragma once

#include "device.h"
#include "kernels.h"

namespace jetk {

// Eight floats as one MFMA operand.
template <typename T> __device__ __forceinline__ Frag<T> pack8(const float (&x)[8]) {
  static_assert(sizeof(T) == 2, "16-bit types");
  Frag<T> f;
  const uint4 u = make_uint4(pack2<T>(x[0], x[1]), pack2<T>(x[2], x[3]), pack2<T>(x[4], x[5]), pack2<T>(x[6], x[7]));
  f.v = __builtin_bit_cast(typename Vec8<T>::type, u);
  return f;
}
template <> __device__ __forceinline__ Frag<float> pack8<float>(const float (&x)[8]) {
  Frag<float> f;
#pragma unroll
  for (int j = 0; j < 8; ++j) f.v[j] = x[j];
  return f;
}

}  // namespace jetk
