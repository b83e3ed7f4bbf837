// The tile configurations of gemm_small.h that are built, and what one
// workgroup of each costs.
#pragma once

#include "gemm_small.h"

namespace jetk {

// Operand kinds: fp16, (hi, lo) fp16 pairs, (hi, lo) bf16 pairs, fp16 with an
// int8 / int4 block-quantized B.
enum { SMALL_F16 = 0, SMALL_F16P = 1, SMALL_BF16P = 2, SMALL_Q8 = 3, SMALL_Q4 = 4 };

// One round of workgroups (one per CU) takes about a + b K / 1000
// microseconds. Fitted to launches of one to three rounds on one MI355X,
// weights coming from memory (decoder shapes N = 1536 .. 19456, K = 1536 ..
// 9728, 8 to 6000 rows). In a kernel trace, launches of up to 256 workgroups take
// the estimated time within 15% on the plain tiles, and 1.15 to 1.5 times it on
// the SwiGLU and RoPE ones (K = 1536: SwiGLU 16 x 128 13.7 us for 9.3, 64 x 128
// 16.7 for 12.0, 256 x 128 28.0 for 24; RoPE 32 x 32 7.2 for 5.4, 64 x 32 8.5 for
// 6.7): too little alike in all of them, which the choice between the tiles of
// one epilogue needs, but not the line to the 256x256 ones.
struct TileCost {
  int bm, bn, bk, ahead;
  double a, b;
};

template <class C>
constexpr TileCost tile_cost(double a, double b) {
  return TileCost{C::BM, C::BN, C::BK, C::AHEAD, a, b};
}

// Cfg<i>::type for the epilogue classes: plain (fp32 store, residual add,
// store T), SwiGLU, RoPE. Few rows take the shortest tiles, so that the K loop
// (one serial chain per output) is spread over the most CUs; the LDS holds as
// many stages as fit, since a tile's loads in flight are all that hides the
// memory latency.
template <typename T, int NPL, int QB>
struct SmallPlain;
template <typename T, int NPL, int QB>
struct SmallSwiglu;
template <typename T, int NPL, int QB>
struct SmallRope;

template <class... Cs>
struct TileTypes {
  template <class F>
  static hipError_t call(int i, F f) {
    hipError_t e = hipErrorInvalidValue;
    int k = 0;
    ((k++ == i ? (void)(e = f(std::integral_constant<Cs *, nullptr>{})) : (void)0), ...);
    return e;
  }
};

// (the grouped GEMMs of launch_gemm_grouped name c1 and c3 of SmallPlain and c0
// and c1 of SmallSwiglu)
template <typename T>
struct SmallPlain<T, 1, 0> {
  using c0 = SCfg<T, 1, 0, 1, 1, 2, 1, 6>;      // 32 x 16
  using c1 = SCfg<T, 1, 0, 1, 2, 1, 4, 4>;      // 16 x 128
  using c2 = SCfg<T, 1, 0, 1, 1, 4, 2, 6>;      // 64 x 32
  using c3 = SCfg<T, 1, 0, 1, 2, 4, 2, 5>;      // 64 x 64
  using c4 = SCfg<T, 1, 0, 2, 2, 4, 2, 3>;      // 128 x 64
  using c5 = SCfg<T, 1, 0, 2, 4, 4, 2, 5, 64>;  // 128 x 128
  using c6 = SCfg<T, 1, 0, 4, 4, 4, 2, 3, 64>;  // 256 x 128
  using types = TileTypes<c0, c1, c2, c3, c4, c5, c6>;
  static constexpr TileCost cost[] = {tile_cost<c0>(2.4, 1.55), tile_cost<c1>(2.5, 4.4), tile_cost<c2>(2.0, 2.8),
                                      tile_cost<c3>(3.0, 3.8),  tile_cost<c4>(4.0, 5.4), tile_cost<c5>(9.0, 7.8),
                                      tile_cost<c6>(14.0, 11.5)};
};
template <typename T>
struct SmallSwiglu<T, 1, 0> {
  using c0 = SCfg<T, 1, 0, 1, 2, 1, 4, 4>;      // 16 x 128
  using c1 = SCfg<T, 1, 0, 2, 2, 2, 4, 3>;      // 64 x 128
  using c2 = SCfg<T, 1, 0, 2, 4, 4, 2, 5, 64>;  // 128 x 128
  using c3 = SCfg<T, 1, 0, 4, 4, 4, 2, 3, 64>;  // 256 x 128
  using types = TileTypes<c0, c1, c2, c3>;
  static constexpr TileCost cost[] = {tile_cost<c0>(2.5, 4.4), tile_cost<c1>(4.0, 5.2), tile_cost<c2>(4.0, 7.0),
                                      tile_cost<c3>(6.0, 11.7)};
};
template <typename T>
struct SmallRope<T, 1, 0> {
  using c0 = SCfg<T, 1, 0, 1, 2, 1, 4, 4>;      // 16 x 128
  using c1 = SCfg<T, 1, 0, 2, 2, 2, 4, 3>;      // 64 x 128
  using c2 = SCfg<T, 1, 0, 4, 2, 2, 4, 5, 64>;  // 128 x 128
  using c3 = SCfg<T, 1, 0, 1, 2, 2, 1, 8>;      // 32 x 32
  using c4 = SCfg<T, 1, 0, 1, 2, 4, 1, 6>;      // 64 x 32
  using types = TileTypes<c0, c1, c2, c3, c4>;
  static constexpr TileCost cost[] = {tile_cost<c0>(2.5, 4.4), tile_cost<c1>(4.0, 5.4), tile_cost<c2>(8.0, 7.8),
                                      tile_cost<c3>(2.2, 2.1), tile_cost<c4>(2.2, 2.9)};
};

template <typename T>
struct SmallPlain<T, 2, 0> {
  using c0 = SCfg<T, 2, 0, 1, 1, 1, 2, 8>;      // 16 x 32
  using c1 = SCfg<T, 2, 0, 1, 1, 2, 2, 6>;      // 32 x 32
  using c2 = SCfg<T, 2, 0, 1, 2, 4, 2, 3>;      // 64 x 64
  using c3 = SCfg<T, 2, 0, 2, 2, 4, 2, 4, 64>;  // 128 x 64
  using c4 = SCfg<T, 2, 0, 2, 4, 4, 2, 3, 64>;  // 128 x 128
  using types = TileTypes<c0, c1, c2, c3, c4>;
  static constexpr TileCost cost[] = {tile_cost<c0>(2.2, 2.0), tile_cost<c1>(1.6, 3.1), tile_cost<c2>(1.0, 6.2),
                                      tile_cost<c3>(4.1, 9.1), tile_cost<c4>(10.0, 13.3)};
};
template <typename T>
struct SmallSwiglu<T, 2, 0> {
  using c0 = SCfg<T, 2, 0, 1, 2, 1, 4, 3>;      // 16 x 128
  using c1 = SCfg<T, 2, 0, 2, 2, 2, 4, 5, 64>;  // 64 x 128
  using c2 = SCfg<T, 2, 0, 2, 4, 4, 2, 3, 64>;  // 128 x 128
  using types = TileTypes<c0, c1, c2>;
  static constexpr TileCost cost[] = {tile_cost<c0>(2.0, 5.8), tile_cost<c1>(3.0, 8.0), tile_cost<c2>(4.0, 13.2)};
};
template <typename T>
struct SmallRope<T, 2, 0> {
  using c0 = SCfg<T, 2, 0, 1, 2, 1, 4, 3>;      // 16 x 128
  using c1 = SCfg<T, 2, 0, 2, 2, 2, 4, 5, 64>;  // 64 x 128
  using c2 = SCfg<T, 2, 0, 4, 2, 2, 4, 3, 64>;  // 128 x 128
  using c3 = SCfg<T, 2, 0, 1, 2, 2, 1, 6>;      // 32 x 32
  using types = TileTypes<c0, c1, c2, c3>;
  static constexpr TileCost cost[] = {tile_cost<c0>(2.0, 5.8), tile_cost<c1>(3.0, 8.0), tile_cost<c2>(9.0, 13.3),
                                      tile_cost<c3>(1.8, 3.6)};
};

// Block-quantized B: a tile holds one row group of scales, 64 or 128 columns.
template <typename T, int QB>
struct SmallPlain<T, 1, QB> {
  using c0 = SCfg<T, 1, QB, 1, 1, 1, 4, 6>;  // 16 x 64
  using c1 = SCfg<T, 1, QB, 2, 1, 1, 4, 6>;  // 32 x 64
  using c2 = SCfg<T, 1, QB, 2, 2, 2, 2, 5>;  // 64 x 64
  using c3 = SCfg<T, 1, QB, 4, 2, 2, 4, 3>;  // 128 x 128
  using types = TileTypes<c0, c1, c2, c3>;
  static constexpr TileCost cost[] = {tile_cost<c0>(2.5, 2.5), tile_cost<c1>(2.5, 3.2), tile_cost<c2>(3.0, 4.4),
                                      tile_cost<c3>(8.0, 9.0)};
};
template <typename T, int QB>
struct SmallSwiglu<T, 1, QB> {
  using c0 = SCfg<T, 1, QB, 1, 2, 1, 4, 5>;  // 16 x 128
  using c1 = SCfg<T, 1, QB, 2, 2, 2, 4, 4>;  // 64 x 128
  using c2 = SCfg<T, 1, QB, 4, 2, 2, 4, 3>;  // 128 x 128
  using types = TileTypes<c0, c1, c2>;
  static constexpr TileCost cost[] = {tile_cost<c0>(2.5, 4.4), tile_cost<c1>(4.0, 5.6), tile_cost<c2>(5.0, 9.0)};
};
template <typename T, int QB>
struct SmallRope<T, 1, QB> {
  using c0 = SCfg<T, 1, QB, 1, 2, 1, 4, 5>;  // 16 x 128
  using c1 = SCfg<T, 1, QB, 2, 2, 2, 4, 4>;  // 64 x 128
  using c2 = SCfg<T, 1, QB, 4, 2, 2, 4, 3>;  // 128 x 128
  using c3 = SCfg<T, 1, QB, 1, 2, 2, 1, 8>;  // 32 x 32
  using types = TileTypes<c0, c1, c2, c3>;
  static constexpr TileCost cost[] = {tile_cost<c0>(2.5, 4.4), tile_cost<c1>(4.0, 5.6), tile_cost<c2>(5.0, 9.0),
                                      tile_cost<c3>(2.2, 2.3)};
};

template <typename T, int NPL, int QB>
hipError_t run_small_tiles(int epi, int cfg, const GemmArgs<T> &g, hipStream_t st) {
  auto with = [&](auto epi_c, auto types) {
    return decltype(types)::call(cfg, [&](auto c) {
      using C = std::remove_pointer_t<typename decltype(c)::value_type>;
      return run_small<C, decltype(epi_c)::value>(g, st);
    });
  };
  using P = typename SmallPlain<T, NPL, QB>::types;
  switch (epi) {
    case EPI_STORE_F32: return with(std::integral_constant<int, 0>{}, P{});
    case EPI_RESID_ADD: return with(std::integral_constant<int, 1>{}, P{});
    case EPI_SWIGLU: return with(std::integral_constant<int, 2>{}, typename SmallSwiglu<T, NPL, QB>::types{});
    case EPI_QKV_ROPE: return with(std::integral_constant<int, 4>{}, typename SmallRope<T, NPL, QB>::types{});
    case EPI_STORE_T:
      if constexpr (NPL == 1 && QB == 0) return with(std::integral_constant<int, 3>{}, P{});
      return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
  }
}

hipError_t small_gemm_f16(int epi, int cfg, const GemmArgs<f16> &g, hipStream_t st);
hipError_t small_gemm_f16p(int epi, int cfg, const GemmArgs<f16> &g, hipStream_t st);
hipError_t small_gemm_bf16p(int epi, int cfg, const GemmArgs<bf16> &g, hipStream_t st);
hipError_t small_gemm_q8(int epi, int cfg, const GemmArgs<f16> &g, hipStream_t st);
hipError_t small_gemm_q4(int epi, int cfg, const GemmArgs<f16> &g, hipStream_t st);

}  // namespace jetk
