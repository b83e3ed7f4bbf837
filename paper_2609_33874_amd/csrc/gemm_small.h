// Matrix-core GEMM for problems of few output tiles (decode steps, one
// question's candidates or prefix): C[M x N] (epilogue) A[M x K] * B[N x K]^T,
// both K-contiguous, fp32 accumulation.
//
// What bounds it: the weights are read once and every workgroup runs the whole
// K loop, one or two workgroups per CU, so nothing but the workgroup's own
// loads in flight hides the memory latency and nothing but short dependent
// chains hides the MFMA latency. Hence
//   * K steps of 128 columns (64 in the largest tiles) in a ring of NS LDS
//     stages, NS - 1 steps of direct global->LDS loads in flight, one barrier
//     per step;
//   * 16x16x32 MFMAs: a quarter of the 32x32x16 product's output per wave, so
//     four times the waves share a tile and a K step's dependent chain is 4
//     short MFMAs instead of 8 long ones.
// The sums are those of the large tiles bit for bit: a 16x16x32 MFMA adds its
// 32 products to the accumulator exactly as two 32x32x16 MFMAs do (checked on
// gfx950 over fp16 and bf16 operands), and K runs in ascending order (pair
// operands: hi then lo within every 16 columns). A row's result therefore does
// not depend on which kernel its batch size selects.
#pragma once

#include "gemm_args.h"
#include "gemm_core.h"

namespace jetk {

// f(L), f(L - 1), .., f(0) with compile-time arguments.
template <int L, class F>
__device__ __forceinline__ void count_down(F &f) {
  f(std::integral_constant<int, L>{});
  if constexpr (L > 0) count_down<L - 1>(f);
}

// Waits until at most N of the wave's direct loads are in flight and its LDS
// reads are done, then for the workgroup. (The builtin, not inline asm: the
// compiler then knows that the reads are done and adds no wait of its own.)
template <int N>
__device__ __forceinline__ void wait_barrier() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | 7 << 4 | 0 << 8 | (N >> 4) << 14);  // vmcnt(N) expcnt(7) lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// v is in its register from here on.
template <typename V>
__device__ __forceinline__ void tie_reg(V &v) {
  asm volatile("" : "+v"(v));
}

// T: operand type. NPL: planes of A (2: (hi, lo) pairs, lo K columns after
// hi). QB: bits of a block-quantized B (0: B is T). A wave takes MI x NI
// blocks of 16x16; WGM x WGN waves.
template <typename T, int NPL_, int QB_, int MI_, int NI_, int WGM_, int WGN_, int NS_, int BK_ = 128>
struct SCfg {
  using type = T;
  static constexpr int NPL = NPL_, QB = QB_, MI = MI_, NI = NI_, WGM = WGM_, WGN = WGN_, NS = NS_;
  static constexpr int BM = 16 * MI * WGM, BN = 16 * NI * WGN, NW = WGM * WGN, NT = 64 * NW;
  static constexpr int BK = BK_, AHEAD = NS - 1;
  static constexpr int AROW = 2 * BK, BROW = QB ? BK * QB / 8 : AROW;  // bytes of a row's K step
  static constexpr int A_BYTES = BM * AROW, B_BYTES = BN * BROW, S_BYTES = QB ? 1024 : 0;
  static constexpr int STAGE = NPL * A_BYTES + B_BYTES + S_BYTES;
  static constexpr size_t LDS_BYTES = (size_t)NS * STAGE;
  static constexpr int A_LD = A_BYTES / 1024 / NW, B_LD = B_BYTES / 1024 / NW;  // direct loads per wave
  static constexpr int PT = NPL * A_LD + B_LD + (QB ? 1 : 0);
  static_assert(sizeof(T) == 2, "16-bit operands");
  static_assert((A_BYTES / 1024) % NW == 0 && (B_BYTES / 1024) % NW == 0 && A_LD >= 1 && B_LD >= 1,
                "whole direct loads per wave");
  static_assert(PT * AHEAD < 64, "vmcnt range");
  static_assert(LDS_BYTES <= 160 * 1024, "LDS of a CU");
  static_assert(BK == 128 || (BK == 64 && !QB), "K step");
  static_assert(!QB || (BN <= 128 && 128 % BN == 0), "one scale group per tile");
};

// First column (within the tile) of block j of wave column wn. The blocks are
// adjacent, except where an epilogue needs two columns of one lane: SwiGLU
// (gate and up column, 32 apart) and RoPE (dims d and d + 64 of a head).
template <class C, int EPI>
__device__ __forceinline__ int small_col(int wn, int j) {
  if constexpr (EPI == 2 && C::NI % 4 == 0) return wn * 16 * C::NI + (j >> 2) * 64 + (j & 1) * 32 + ((j >> 1) & 1) * 16;
  else if constexpr (EPI == 2) return (wn >> 1) * 64 + (wn & 1) * 16 + j * 32;
  else if constexpr (EPI == 4 && !(C::BN == 32)) return (wn >> 2) * 128 + (wn & 3) * 16 + j * 64;
  else return (wn * C::NI + j) * 16;
}

// RoPE tiles of 32 columns: 16 dims d and the 16 dims d + 64 of one head (four
// tiles per head), so that few rows still spread over many CUs.
template <class C, int EPI>
constexpr bool small_split = EPI == 4 && C::BN == 32;

// First column of tile tn of B, and the column of the tile's LDS row r past it.
template <class C, int EPI>
__device__ __forceinline__ int small_n0(int tn) {
  return small_split<C, EPI> ? (tn >> 2) * 128 + (tn & 3) * 16 : tn * C::BN;
}
template <class C, int EPI>
__device__ __forceinline__ int small_row(int r) {
  return small_split<C, EPI> ? (r & 15) + (r >> 4) * 64 : r;
}

// Swizzle of the 16-byte chunks of a row of CH chunks: the 16 rows that a
// fragment read touches at one logical chunk spread over all banks.
template <int CH>
__device__ __forceinline__ int small_swz(int r) {
  return CH == 16 ? (r & 15) : CH == 8 ? ((r >> 1) & 7) : ((r >> 2) & 3);
}

// acc = A[m0 ..][K] * B[n0 ..][K]^T over a workgroup's tile. ldb_bytes and the
// byte layout of a quantized B as in launch_gemm_q8 / _q4. Needs K a multiple
// of BK and K / BK >= NS - 1. Rows past M / N load the last valid row.
template <class C, int EPI>
__device__ __forceinline__ void small_tile(const typename C::type *__restrict__ A, int64_t lda, const char *B,
                                           int64_t ldb_bytes, const uint16_t *__restrict__ Bs, int M, int N, int K,
                                           int m0, int n0, char *lds, f32x4 (&acc)[C::MI][C::NI]) {
  using T = typename C::type;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / C::WGN, wn = wave % C::WGN;
#pragma unroll
  for (int i = 0; i < C::MI; ++i)
#pragma unroll
    for (int j = 0; j < C::NI; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  // Direct loads: an instruction fills 1 KB (64 lanes of 16 bytes in lane
  // order), i.e. 1024 / row bytes rows, chunk c of row r stored at c ^ swz(r).
  constexpr int CA = C::AROW / 16, CB = C::BROW / 16;  // chunks per row
  const char *pa[C::A_LD], *pb[C::B_LD];
#pragma unroll
  for (int i = 0; i < C::A_LD; ++i) {
    const int u = (i * C::NW + wave) * 64 + lane, r = u / CA, c = (u % CA) ^ small_swz<CA>(r);
    pa[i] = (const char *)(A + (int64_t)min(m0 + r, M - 1) * lda) + c * 16;
  }
#pragma unroll
  for (int i = 0; i < C::B_LD; ++i) {
    const int u = (i * C::NW + wave) * 64 + lane, r = u / CB, c = (u % CB) ^ small_swz<CB>(r);
    pb[i] = B + (int64_t)min(n0 + small_row<C, EPI>(r), N - 1) * ldb_bytes + c * 16;
  }
  const char *ps = nullptr;  // scales: 256 bytes per (K block of 32, row group of 128); 4 blocks per K step
  int64_t s_step = 0;
  if constexpr (C::QB > 0) {
    const int ng = (N + 127) / 128;
    ps = (const char *)Bs + ((int64_t)(lane >> 4) * ng + (n0 >> 7)) * 256 + (lane & 15) * 16;
    s_step = (int64_t)ng * 1024;
  }
  auto issue = [&](int kt, int stage) {
    char *a = lds + stage * C::STAGE, *b = a + C::NPL * C::A_BYTES;
#pragma unroll
    for (int pl = 0; pl < C::NPL; ++pl)
#pragma unroll
      for (int i = 0; i < C::A_LD; ++i)
        __builtin_amdgcn_global_load_lds((const void *)(pa[i] + (int64_t)pl * K * 2 + (int64_t)kt * C::AROW),
                                         (lds_void *)(a + pl * C::A_BYTES + (i * C::NW + wave) * 1024), 16, 0, 0);
#pragma unroll
    for (int i = 0; i < C::B_LD; ++i)
      __builtin_amdgcn_global_load_lds((const void *)(pb[i] + (int64_t)kt * C::BROW),
                                       (lds_void *)(b + (i * C::NW + wave) * 1024), 16, 0, 0);
    // every wave writes the same kilobyte of scales, so that each wave has
    // the same number of loads in flight
    if constexpr (C::QB > 0)
      __builtin_amdgcn_global_load_lds((const void *)(ps + kt * s_step), (lds_void *)(b + C::B_BYTES), 16, 0, 0);
  };

  const int nk = K / C::BK, r16 = lane & 15, g = lane >> 4;
  // MFMA kk of a K step takes columns 32 kk + 8 g .. + 7 from lane group g;
  // with pairs, columns 16 kk + 8 (g % 2) .. + 7 of plane g / 2 against the
  // same columns of B twice, which adds hi * b and then lo * b over 16 columns.
  // The fragments are read in two halves of KH MFMAs, each half while the
  // other one's MFMAs run.
  constexpr int KH = C::BK / 64 * C::NPL;
  Frag<T> fa[2][KH][C::MI], fb[2][KH][C::NI];
  uint2 rb[2][KH][C::NI];
  uint32_t sb[2][KH][C::NI];
  auto read = [&](int stage, auto half) {
    constexpr int h = decltype(half)::value;
    const char *a = lds + stage * C::STAGE + (C::NPL == 2 ? (g >> 1) * C::A_BYTES : 0);
    const char *b = lds + stage * C::STAGE + C::NPL * C::A_BYTES;
#pragma unroll
    for (int k = 0; k < KH; ++k) {
      const int kk = h * KH + k;
      const int c = C::NPL == 2 ? kk * 2 + (g & 1) : kk * 4 + g;  // logical 16-byte chunk of a row
#pragma unroll
      for (int i = 0; i < C::MI; ++i)
        frag_load(fa[h][k][i],
                  (const T *)(a + ((wm * C::MI + i) * 16 + r16) * C::AROW + ((c ^ small_swz<CA>(r16)) << 4)));
#pragma unroll
      for (int j = 0; j < C::NI; ++j) {
        const int r = small_col<C, EPI>(wn, j) + r16;
        if constexpr (C::QB == 0) {
          frag_load(fb[h][k][j], (const T *)(b + r * C::BROW + ((c ^ small_swz<CB>(r16)) << 4)));
        } else {
          if constexpr (C::QB == 8)
            rb[h][k][j] = *(const uint2 *)(b + r * 128 + (((kk * 2 + (g >> 1)) ^ small_swz<CB>(r16)) << 4) + (g & 1) * 8);
          else rb[h][k][j].x = *(const uint32_t *)(b + r * 64 + ((kk ^ small_swz<CB>(r16)) << 4) + g * 4);
          const int n = (n0 & 127) + small_row<C, EPI>(r);
          sb[h][k][j] = *(const uint16_t *)(b + C::B_BYTES + kk * 256 + (n & 31) * 8 + (n >> 5) * 2);
        }
      }
    }
  };
  auto mma = [&](auto half) {
    constexpr int h = decltype(half)::value;
#pragma unroll
    for (int k = 0; k < KH; ++k) {
#pragma unroll
      for (int j = 0; j < C::NI; ++j) {
        if constexpr (C::QB == 8) fb[h][k][j] = q8_frag(rb[h][k][j], sb[h][k][j]);
        if constexpr (C::QB == 4) fb[h][k][j] = q4_frag(rb[h][k][j].x, sb[h][k][j]);
      }
#pragma unroll
      for (int i = 0; i < C::MI; ++i)
#pragma unroll
        for (int j = 0; j < C::NI; ++j) mma16(acc[i][j], fa[h][k][i], fb[h][k][j]);
    }
  };
  // The compiler waits for a half's reads here, where they are the only LDS
  // reads in flight. At their use the other half's would be too, and with
  // direct loads in flight it waits for all of them.
  auto arrived = [&](auto half) {
    constexpr int h = decltype(half)::value;
#pragma unroll
    for (int k = 0; k < KH; ++k) {
#pragma unroll
      for (int i = 0; i < C::MI; ++i) tie_reg(fa[h][k][i].v);
#pragma unroll
      for (int j = 0; j < C::NI; ++j) {
        if constexpr (C::QB == 0) {
          tie_reg(fb[h][k][j].v);
        } else {
          tie_reg(rb[h][k][j].x);
          if constexpr (C::QB == 8) tie_reg(rb[h][k][j].y);
          tie_reg(sb[h][k][j]);
        }
      }
    }
  };
  // The barrier at the end of step kt certifies that every wave's loads of
  // tile kt + 1 have landed and that every wave has tile kt's fragments in
  // registers, so the loads of step kt + 1 may fill that stage. `left`: tiles
  // that may still be in flight then (-1: tile kt is the last).
  constexpr std::integral_constant<int, 0> h0{};
  constexpr std::integral_constant<int, 1> h1{};
  int st = 0, sl = C::AHEAD;
  auto step = [&](int next, auto left) {
    // (the scheduling barriers keep each half's reads ahead of the other
    // half's MFMAs; the compiler would otherwise read next to the use)
    arrived(h0);
    read(st, h1);
    __builtin_amdgcn_sched_barrier(0);
    if (next >= 0) issue(next, sl);
    mma(h0);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (decltype(left)::value >= 0) {
      wait_barrier<decltype(left)::value * C::PT>();
      st = st + 1 == C::NS ? 0 : st + 1;
      sl = sl + 1 == C::NS ? 0 : sl + 1;
      read(st, h0);
      __builtin_amdgcn_sched_barrier(0);
    }
    mma(h1);
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int s = 0; s < C::AHEAD; ++s) issue(s, s);
  wait_barrier<(C::AHEAD - 1) * C::PT>();
  read(0, h0);
  for (int kt = 0; kt < nk - C::AHEAD; ++kt) step(kt + C::AHEAD, std::integral_constant<int, C::AHEAD - 1>{});
  auto last = [&](auto left) { step(-1, std::integral_constant<int, decltype(left)::value - 1>{}); };
  count_down<C::AHEAD - 1>(last);
}

// The epilogues of gemm_kernel on the small tiles of gemm_small.h (the same
// operations per element).
template <class C, int EPI>
__global__ __launch_bounds__(C::NT) void gemm_small_kernel(GemmArgs<typename C::type> g) {
  using T = typename C::type;
  extern __shared__ uint4 lds[];
  const int nt_m = (g.M + C::BM - 1) / C::BM, nt_n = (g.N + C::BN - 1) / C::BN;
  int tm, tn;
  tile_coords(nt_m, nt_n, &tm, &tn);
  const int m0 = tm * C::BM, n0 = small_n0<C, EPI>(tn);
  const T *B = g.B;
  if (g.tile_group) {
    const int grp = g.tile_group[tm];
    if (grp < 0) return;
    B += (int64_t)grp * g.group_stride;
  }
  f32x4 acc[C::MI][C::NI];
  small_tile<C, EPI>(g.A, g.lda, (const char *)B, C::QB ? g.ldb : g.ldb * (int64_t)sizeof(T), g.Bs, g.M, g.N, g.KB, m0,
                     n0, (char *)lds, acc);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wm = wave / C::WGN, wn = wave % C::WGN;
#pragma unroll
  for (int i = 0; i < C::MI; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = m0 + (wm * C::MI + i) * 16 + 4 * (lane >> 4) + e;
      if (row >= g.M) continue;
      if constexpr (EPI == 2) {
        static_assert(C::NI % 4 == 0 || (C::NI == 2 && C::WGN % 2 == 0), "pairs of a gate and an up block per wave");
#pragma unroll
        for (int j = 0; j < C::NI; j += 2) {
          const int col = small_col<C, 2>(wn, j), gcol = n0 + (col & ~63);  // first column of the gate block
          if (gcol >= g.N) continue;
          const int f = (gcol >> 6) * 32 + (col & 31) + (lane & 15);
          const float v = swiglu<C::NPL == 2>(acc[i][j][e] * g.oscale, acc[i][j + 1][e] * g.oscale);
          put_split<T>((T *)g.out + (int64_t)row * g.ldo + f, g.N >> 1, v, g.pair_out);
        }
      } else if constexpr (EPI == 4) {
        static_assert(C::NI == 2 && (small_split<C, 4> || C::WGN % 4 == 0), "dims d and d + 64 of a head per wave");
        const QkvRope &q = g.rope;
        const int head = (n0 >> 7) + (wn >> 2);  // query heads, then key heads, then value heads
        if (head >= q.Hq + 2 * q.Hkv) continue;
        const int64_t ps = head < q.Hq ? q.q_ps : q.kv_ps;
        T *dst;
        if (head < q.Hq) dst = (T *)q.q_out + ((int64_t)row * q.Hq + head) * 128;
        else if (head < q.Hq + q.Hkv) dst = (T *)q.k_cache + ((int64_t)(head - q.Hq) * q.S + q.slot0 + row) * 128;
        else dst = (T *)q.v_cache + ((int64_t)(head - q.Hq - q.Hkv) * q.S + q.slot0 + row) * 128;
        const int d = (small_split<C, 4> ? n0 & 63 : (wn & 3) * 16) + (lane & 15);
        const float x1 = acc[i][0][e] * g.oscale, x2 = acc[i][1][e] * g.oscale;
        if (head < q.Hq + q.Hkv) {
          const int64_t p = q.pos[row];
          const float c = q.cos_t[p * 64 + d], s = q.sin_t[p * 64 + d];
          put_split<T>(dst + d, ps, fmaf(x1, c, -(x2 * s)), g.pair_out);
          put_split<T>(dst + d + 64, ps, fmaf(x2, c, x1 * s), g.pair_out);
        } else {
          put_split<T>(dst + d, ps, x1, g.pair_out);
          put_split<T>(dst + d + 64, ps, x2, g.pair_out);
        }
      } else {
#pragma unroll
        for (int j = 0; j < C::NI; ++j) {
          const int col = n0 + small_col<C, EPI>(wn, j) + (lane & 15);
          if (col >= g.N) continue;
          const int64_t o = (int64_t)row * g.ldo + col;
          const float v = acc[i][j][e] * g.oscale;
          if constexpr (EPI == 0) ((float *)g.out)[o] = v;
          else if constexpr (EPI == 1) ((float *)g.out)[o] += v;
          else ((T *)g.out)[o] = from_f<T>(v);
        }
      }
    }
}

template <class C, int EPI>
static hipError_t run_small(const GemmArgs<typename C::type> &g, hipStream_t st) {
  static const hipError_t once = allow_lds<C>((const void *)gemm_small_kernel<C, EPI>);
  if (once != hipSuccess) return once;
  if (g.KB % C::BK || g.KB / C::BK < C::AHEAD || (g.tile_group && g.M % C::BM)) return hipErrorInvalidValue;
  const int tiles = ((g.M + C::BM - 1) / C::BM) * ((g.N + C::BN - 1) / C::BN);
  hipLaunchKernelGGL((gemm_small_kernel<C, EPI>), dim3(tiles), dim3(C::NT), C::LDS_BYTES, st, g);
  return hipGetLastError();
}

}  // namespace jetk
