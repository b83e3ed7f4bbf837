// Matrix-core GEMMs for gfx950: C[M x N] = A[M x K] * B[N x K]^T, both
// operands K-contiguous, fp32 accumulation, with the epilogues the decoder
// needs fused in (fp32 store, residual add, SwiGLU), and the LM head with a
// full-vocabulary online log-sum-exp epilogue that never writes logits.
//
// Large problems use 256x256 tiles (MFMA fragments read one step ahead; in the
// pair mode the hi and lo planes of A share each B tile) fed by direct
// global->LDS loads, one barrier per K step. Problems of few tiles
// take the smaller tiles of gemm_small.h; which one is chosen by the estimated
// time of its rounds of workgroups (tile_for). Tiles are ordered so that
// each XCD works on a contiguous band (see tile_coords).
#include <algorithm>
#include <cmath>

#include "gemm_core.h"
#include "gemm_small_tiles.h"
#include "kernels.h"

namespace jetk {

// Orders a wave's LDS writes before its following LDS reads of other lanes'
// data (a wave's LDS operations complete in order).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// fp32 store, residual add and SwiGLU epilogues through the LDS (free once
// the K loop has ended): each wave writes a slab of its accumulators (16 rows
// of fp32, or 32 rows of T for SwiGLU) into its own LDS region and reads it back as 16-byte
// row chunks, so every global access moves 16 bytes instead of 2 or 4. The
// arithmetic is that of the per-element epilogues in gemm_kernel. Returns
// false (nothing done) for tiles of fewer than 256 rows, where the output rows
// are not 16-byte aligned, or where the LDS is too small.
template <class C, int EPI>
__device__ __forceinline__ bool staged_epilogue(const GemmArgs<typename C::type> &g, int m0, int n0,
                                                f32x16 (&acc)[C::MI][C::NI], uint4 *lds) {
  using T = typename C::type;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave / C::WAVES_N, wn = wave % C::WAVES_N;
  if constexpr (C::BM < 256) {
    // smaller tiles run several workgroups per CU; the staging registers
    // would cost one of them
    return false;
  } else if constexpr (EPI == 0 || EPI == 1) {
    constexpr int SC = C::WN < 64 ? C::WN : 64, LDF = SC + 4;  // slab columns, padded row (floats)
    constexpr int CH = 16 * SC / 4 / 64;                        // float4 chunks per lane per slab
    static_assert(CH >= 1 && (16 * SC / 4) % 64 == 0, "slab of whole chunk rounds");
    if constexpr ((size_t)C::NWAVES * 16 * LDF * 4 > C::LDS_BYTES) {
      return false;
    } else {
      if ((g.ldo & 3) || (g.N & 3)) return false;
      float *wl = reinterpret_cast<float *>(lds) + wave * 16 * LDF;
      constexpr int JH = C::WN / SC, NSLAB = 2 * C::MI * JH;
      // residual rows are loaded DEEP slabs ahead where one wave per SIMD has
      // the registers (and no other wave to hide the latency)
      constexpr int DEEP = EPI == 1 && C::WIDE ? 4 : 1;
      float4 x[DEEP][CH];
      // row (hr: rows 16 hr .. 16 hr + 15 of the 32-row block) and column of chunk t of slab n
      auto at = [&](int n, int t, int *row, int *col) {
        const int q = t * 64 + lane, i = n / (2 * JH), hr = n / JH % 2, jh = n % JH;
        *row = m0 + wm * C::WM + i * 32 + 16 * hr + q / (SC / 4);
        *col = n0 + wn * C::WN + jh * SC + 4 * (q % (SC / 4));
        return *row < g.M && *col < g.N;
      };
      auto fetch = [&](int n, float4 (&v)[CH]) {
#pragma unroll
        for (int t = 0; t < CH; ++t) {
          int row, col;
          if (at(n, t, &row, &col)) v[t] = *reinterpret_cast<const float4 *>((const float *)g.out + (int64_t)row * g.ldo + col);
        }
      };
      if constexpr (DEEP > 1) {
#pragma unroll
        for (int n = 0; n < DEEP; ++n) fetch(n, x[n]);
      }
      static_for<NSLAB>([&](auto n_) {
        constexpr int n = decltype(n_)::value, i = n / (2 * JH), hr = n / JH % 2, jh = n % JH;
#pragma unroll
        for (int jj = 0; jj < SC / 32; ++jj)
#pragma unroll
          for (int e = 8 * hr; e < 8 * hr + 8; ++e) {
            const int r = 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3) - 16 * hr;
            wl[r * LDF + jj * 32 + (lane & 31)] = acc[i][jh * (SC / 32) + jj][e] * g.oscale;
          }
        wave_lds_sync();
#pragma unroll
        for (int t = 0; t < CH; ++t) {
          int row, col;
          if (at(n, t, &row, &col)) {
            const int q = t * 64 + lane;
            const float4 v = *reinterpret_cast<const float4 *>(wl + q / (SC / 4) * LDF + 4 * (q % (SC / 4)));
            float4 *o = reinterpret_cast<float4 *>((float *)g.out + (int64_t)row * g.ldo + col);
            if constexpr (EPI == 0) {
              *o = v;
            } else {
              float4 y;
              if constexpr (DEEP > 1) y = x[n % DEEP][t];
              else y = *o;
              y.x += v.x; y.y += v.y; y.z += v.z; y.w += v.w;
              *o = y;
            }
          }
        }
        if constexpr (DEEP > 1 && n + DEEP < NSLAB) fetch(n + DEEP, x[n % DEEP]);
        wave_lds_sync();
      });
      return true;
    }
  } else if constexpr (EPI == 2 && sizeof(T) == 2) {
    constexpr int OC = C::WN / 2, LDH = OC + 8;  // output columns of a wave, padded row (elements)
    constexpr int CH = 32 * OC / 8 / 64;         // 16-byte chunks per lane per 32-row slab
    static_assert(CH >= 1 && (32 * OC / 8) % 64 == 0, "slab of whole chunk rounds");
    if constexpr ((size_t)(C::PAIRA ? 2 : 1) * C::NWAVES * 32 * LDH * sizeof(T) > C::LDS_BYTES) {
      return false;
    } else {
      if ((g.ldo & 7) || (g.pair_out && ((g.N & 15) || !C::PAIRA))) return false;
      T *wl = reinterpret_cast<T *>(lds) + wave * 32 * LDH, *wl_lo = wl + C::NWAVES * 32 * LDH;
      const int f0 = (n0 + wn * C::WN) >> 1;  // first output column of the wave
#pragma unroll
      for (int i = 0; i < C::MI; ++i) {
#pragma unroll
        for (int jp = 0; jp < C::NI / 2; ++jp)
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const float v = swiglu<C::PAIRA>(acc[i][2 * jp][e] * g.oscale, acc[i][2 * jp + 1][e] * g.oscale);
            const int r = 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
            const T hi = from_f<T>(v);
            wl[r * LDH + jp * 32 + (lane & 31)] = hi;
            if constexpr (C::PAIRA) wl_lo[r * LDH + jp * 32 + (lane & 31)] = from_f<T>(v - to_f<T>(hi));
          }
        wave_lds_sync();
#pragma unroll
        for (int t = 0; t < CH; ++t) {
          const int q = t * 64 + lane, r = q / (OC / 8), c8 = q % (OC / 8);
          const int row = m0 + wm * C::WM + i * 32 + r;
          const int gcol = n0 + wn * C::WN + 64 * (c8 / 4);  // first gate column of the chunk's block
          if (row < g.M && gcol < g.N) {
            T *o = (T *)g.out + (int64_t)row * g.ldo + f0 + 8 * c8;
            *reinterpret_cast<uint4 *>(o) = *reinterpret_cast<const uint4 *>(wl + r * LDH + 8 * c8);
            if constexpr (C::PAIRA)
              if (g.pair_out)
                *reinterpret_cast<uint4 *>(o + (g.N >> 1)) = *reinterpret_cast<const uint4 *>(wl_lo + r * LDH + 8 * c8);
          }
        }
        wave_lds_sync();
      }
      return true;
    }
  } else {
    return false;
  }
}

// EPI: 0 = store fp32, 1 = fp32 residual add, 2 = SwiGLU into T (B rows
// interleaved in blocks of 32 gate rows / 32 up rows), 3 = store T, 4 = RoPE
// and scatter of q, K, V (waves of 128 columns = one head).
template <class C, int EPI>
__global__ __launch_bounds__(C::NT) void gemm_kernel(GemmArgs<typename C::type> g) {
  using T = typename C::type;
  extern __shared__ uint4 lds[];
  const int nt_m = (g.M + C::BM - 1) / C::BM, nt_n = (g.N + C::BN - 1) / C::BN;
  int tm, tn;
  tile_coords(nt_m, nt_n, &tm, &tn);
  const int m0 = tm * C::BM, n0 = tn * C::BN;
  const T *B = g.B;
  if (g.tile_group) {
    const int grp = g.tile_group[tm];
    if (grp < 0) return;
    B += (int64_t)grp * g.group_stride;
  }
  f32x16 acc[C::MI][C::NI];
  gemm_tile<C>(g.A, g.lda, B, g.ldb, g.M, g.N, g.K, g.KA, g.KB, m0, n0, lds, acc, g.Bs);
  if (staged_epilogue<C, EPI>(g, m0, n0, acc, lds)) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave / C::WAVES_N, wn = wave % C::WAVES_N;
  if constexpr (EPI == 4) {
    static_assert(C::WN == 128 && C::NI == 4, "a wave's columns must be one head of 128");
    const QkvRope &q = g.rope;
    const int head = (n0 + wn * C::WN) >> 7;  // query heads, then key heads, then value heads
    const int64_t ps = head < q.Hq ? q.q_ps : q.kv_ps;
#pragma unroll
    for (int i = 0; i < C::MI; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int row = m0 + wm * C::WM + i * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
        if (row >= g.M || head >= q.Hq + 2 * q.Hkv) continue;
        T *dst;
        if (head < q.Hq) dst = (T *)q.q_out + ((int64_t)row * q.Hq + head) * 128;
        else if (head < q.Hq + q.Hkv) dst = (T *)q.k_cache + ((int64_t)(head - q.Hq) * q.S + q.slot0 + row) * 128;
        else dst = (T *)q.v_cache + ((int64_t)(head - q.Hq - q.Hkv) * q.S + q.slot0 + row) * 128;
        if (head < q.Hq + q.Hkv) {
          const int64_t p = q.pos[row];
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const int d = j * 32 + (lane & 31);
            const float x1 = acc[i][j][e] * g.oscale, x2 = acc[i][j + 2][e] * g.oscale;
            const float c = q.cos_t[p * 64 + d], s = q.sin_t[p * 64 + d];
            // the same operations as rope_scatter_kernel, so both paths round alike
            put_split<T>(dst + d, ps, fmaf(x1, c, -(x2 * s)), g.pair_out);
            put_split<T>(dst + d + 64, ps, fmaf(x2, c, x1 * s), g.pair_out);
          }
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) put_split<T>(dst + j * 32 + (lane & 31), ps, acc[i][j][e] * g.oscale, g.pair_out);
        }
      }
  } else if constexpr (EPI == 2) {
    T *out = (T *)g.out;
#pragma unroll
    for (int i = 0; i < C::MI; ++i)
#pragma unroll
      for (int jp = 0; jp < C::NI / 2; ++jp) {
        const int gcol = n0 + wn * C::WN + jp * 64;  // first column of the gate block
        const int f = (gcol >> 6) * 32 + (lane & 31);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int row = m0 + wm * C::WM + i * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
          if (row < g.M && gcol < g.N) {
            const float v = swiglu<C::PAIRA>(acc[i][2 * jp][e] * g.oscale, acc[i][2 * jp + 1][e] * g.oscale);
            put_split<T>(out + (int64_t)row * g.ldo + f, g.N >> 1, v, g.pair_out);
          }
        }
      }
  } else {
#pragma unroll
    for (int i = 0; i < C::MI; ++i)
#pragma unroll
      for (int j = 0; j < C::NI; ++j) {
        const int col = n0 + wn * C::WN + j * 32 + (lane & 31);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int row = m0 + wm * C::WM + i * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
          if (row >= g.M || col >= g.N) continue;
          const int64_t o = (int64_t)row * g.ldo + col;
          const float v = acc[i][j][e] * g.oscale;
          if constexpr (EPI == 0) ((float *)g.out)[o] = v;
          else if constexpr (EPI == 1) ((float *)g.out)[o] += v;
          else ((T *)g.out)[o] = from_f<T>(v);
        }
      }
  }
}

// LM head with online log-sum-exp (Section 3.1 Eq. 2 evaluated over vocabulary
// tiles): logits = F[R x K] * W[V x K]^T tile by tile, transposed in the
// accumulators (C::SWAP), so each lane owns rows of F: it keeps a running
// (max, sum of exp) in base 2 for them, and one partial per (row, vocabulary
// split) is written. The logits stay in registers. With pair operands F holds
// (hi, lo) rows [hi (K) | lo (K)] and each W fragment serves both.
// The tile of F rows (C::BM) follows the number of rows; a row's partials are
// the same in every one of them (same vocabulary tiles, same order).
// With target (one vocabulary index per row of F), the product of a row with
// its target's W row is kept as well, zt[row] (unscaled): the very
// accumulator the log-sum-exp takes in, written by the one lane that holds it.
template <class C>
__global__ __launch_bounds__(C::NT) void lmhead_lse_kernel(const typename C::type *__restrict__ W,
                                                          const typename C::type *__restrict__ F, int V, int R,
                                                          int K, int tiles_per_split, int nsplit, int strided,
                                                          float zscale,
                                                          float *__restrict__ part_m, float *__restrict__ part_s,
                                                          const int32_t *__restrict__ target,
                                                          float *__restrict__ zt) {
  extern __shared__ uint4 lds[];
  // Workgroups go round-robin to the 8 XCDs. strided: XCD x takes the splits
  // x, x + 8, .., each with all its row tiles in a row, so a vocabulary tile is
  // read into one L2 only and the XCDs walk the row tiles in step. Else each
  // XCD takes a band of the (split, row tile) pairs, even to one workgroup.
  const int nrt = (R + C::BM - 1) / C::BM, id = blockIdx.x, per = nsplit * nrt / 8;
  int split, rt;
  if (strided) {
    split = (id >> 3) / nrt * 8 + (id & 7), rt = (id >> 3) % nrt;
    if (split >= nsplit) return;
  } else {
    const int seq = id < per * 8 ? (id & 7) * per + (id >> 3) : id;
    split = seq / nrt, rt = seq % nrt;
  }
  const int m0 = rt * C::BM;
  const int ntiles = (V + C::BN - 1) / C::BN;
  const int vt0 = split * tiles_per_split, vt1 = min(vt0 + tiles_per_split, ntiles);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave / C::WAVES_N, wn = wave % C::WAVES_N;
  float rm[C::MI], rs[C::MI];
  int tj[C::MI];  // this lane's rows' targets (-1: none)
#pragma unroll
  for (int i = 0; i < C::MI; ++i) {
    rm[i] = -INFINITY;
    rs[i] = 0.0f;
    const int row = m0 + wm * C::WM + i * 32 + (lane & 31);
    tj[i] = target && row < R ? target[row] : -1;
  }
  f32x16 acc[C::MI][C::NI];
  for (int vt = vt0; vt < vt1; ++vt) {
    const int n0 = vt * C::BN;
    gemm_tile<C>(F, C::PAIRA ? 2 * K : K, W, K, R, V, K, K, K, m0, n0, lds, acc);
    // element e of acc[i][j] is vocabulary index vb + 32 j + 8 (e / 4) + e % 4
    const int vb = n0 + wn * C::WN + 4 * (lane >> 5);
#pragma unroll
    for (int i = 0; i < C::MI; ++i) {
      const int dv = tj[i] - vb;
      if (dv >= 0 && dv < 32 * C::NI && (dv & 4) == 0) {
        const int row = m0 + wm * C::WM + i * 32 + (lane & 31);
        float z = 0.0f;
#pragma unroll
        for (int j = 0; j < C::NI; ++j)
#pragma unroll
          for (int e = 0; e < 16; ++e) z = dv == 32 * j + 8 * (e >> 2) + (e & 3) ? acc[i][j][e] : z;
        zt[row] = z;
      }
    }
#pragma unroll
    for (int i = 0; i < C::MI; ++i) {
      float mx = -INFINITY;
#pragma unroll
      for (int j = 0; j < C::NI; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int v = vb + 32 * j + 8 * (e >> 2) + (e & 3);
          const float z = v < V ? acc[i][j][e] * zscale : -INFINITY;
          acc[i][j][e] = z;
          mx = fmaxf(mx, z);
        }
      if (mx == -INFINITY) continue;
      const float nm = fmaxf(rm[i], mx);
      float s = rs[i] * exp2f(rm[i] - nm);
#pragma unroll
      for (int j = 0; j < C::NI; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) s += exp2f(acc[i][j][e] - nm);
      rm[i] = nm;
      rs[i] = s;
    }
  }
  // merge the two lane halves that hold the same row, then the waves along
  // the vocabulary dimension through LDS
  float *sm = reinterpret_cast<float *>(lds);  // [WAVES_N][BM] maxima, then sums
#pragma unroll
  for (int i = 0; i < C::MI; ++i) {
    const float om = __shfl_xor(rm[i], 32), os = __shfl_xor(rs[i], 32);
    const float nm = fmaxf(rm[i], om);
    float s = 0.0f;
    if (nm != -INFINITY) s = rs[i] * exp2f(rm[i] - nm) + os * exp2f(om - nm);
    if (lane < 32) {
      const int rl = wm * C::WM + i * 32 + lane;
      sm[wn * C::BM + rl] = nm;
      sm[C::WAVES_N * C::BM + wn * C::BM + rl] = s;
    }
  }
  __syncthreads();
  for (int rl = threadIdx.x; rl < C::BM; rl += C::NT) {
    const int row = m0 + rl;
    if (row >= R) continue;
    float M = -INFINITY;
    for (int w = 0; w < C::WAVES_N; ++w) M = fmaxf(M, sm[w * C::BM + rl]);
    float S = 0.0f;
    if (M != -INFINITY)
      for (int w = 0; w < C::WAVES_N; ++w)
        S += sm[C::WAVES_N * C::BM + w * C::BM + rl] * exp2f(sm[w * C::BM + rl] - M);
    part_m[(int64_t)split * R + row] = M;
    part_s[(int64_t)split * R + row] = S;
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

// Direct-load pipelines with bank-conflict-free swizzles and 128-byte tile
// rows: the 256x256 tiles with fragments read one MFMA step ahead (two stages
// of 64 KB), the 256x128 tiles with three stages.
using BigB = GCfg<bf16, 256, 256, 128, 64, 4, 1, 2, 8>;
// Pair mode: 256x256 tiles of four waves, the (hi, lo) planes of A against one
// B tile (wide_pair_tile). Against eight waves of 64 x 128 over 64-byte rows
// of B (LOAD 7), ms: 27700 rows, gate/up 19456 x 2560 4.29 -> 4.15, down
// 2560 x 9728 2.43 -> 2.28, output projection 2560 x 2048 0.60 -> 0.57;
// 16868 rows, gate/up 34816 x 5120 9.60 -> 9.12, down 5120 x 17408 5.15 -> 4.79.
using PairB = GCfg<bf16, 256, 256, 128, 128, 12, 2, 3, 4>;
// ... and 128x128 tiles (8 waves of 32x64, three 24 KB stages, two workgroups
// per CU) for problems of few tiles whose K is too short for gemm_small.h.
using PairS = GCfg<bf16, 128, 128, 32, 64, 7, 2, 3, 4>;
using SmallB = GCfg<bf16, 256, 128, 64, 64, 2, 1, 3, 8>;
using CfgF = GCfg<float, 128, 128, 64, 64, 0, 1>;
// fp16 operands: 256x256 tiles of four waves (wide_tile). Against eight waves
// of 64 x 128 over 64-byte rows (LOAD 8), 67007 rows, ms: gate/up 17920 x 1536
// 3.50 -> 3.39, down 1536 x 8960 2.01 -> 1.73; output projection 1536 x 1536
// 0.49 (256x128 tiles, two workgroups per CU) -> 0.46. Without the direct loads the down projection takes 1.57, without
// the fragment reads too 1.43 (a power-limited MFMA rate).
using HalfB = GCfg<f16, 256, 256, 128, 128, 11, 1, 2, 8>;
// ... and 128x128 tiles on the LOAD 8 schedule (the last round of a large
// launch, grouped GEMMs, and problems whose K is too short for the others).
using HalfS = GCfg<f16, 128, 128, 32, 64, 8, 2, 3, 4>;
// (hi, lo) fp16 pair A operands: the bf16 pair schedules with fp16 operands
using HalfPairB = GCfg<f16, 256, 256, 128, 128, 12, 2, 3, 4>;
using HalfPairS = GCfg<f16, 128, 128, 32, 64, 7, 2, 3, 4>;
// 256x256 tiles of eight waves of 64 x 128, two per SIMD, for work that one wave
// per SIMD cannot hide behind another's: the first loads and the epilogue of a
// short K (below), and the RoPE epilogue, whose loads of positions and angles
// and 2-byte stores it waits for. QKV of 2048 x 1536, us with eight waves and
// with four: 57600 rows fp16 530 and 657, pairs 805 and 943; 67000 rows 590 and
// 750, 905 and 1072.
using HalfE = GCfg<f16, 256, 256, 64, 128, 8, 2, 3, 4>;
using PairE = GCfg<bf16, 256, 256, 64, 128, 7, 2, 3, 4>;
using HalfPairE = GCfg<f16, 256, 256, 64, 128, 7, 2, 3, 4>;
// Residual add with a short K: 256x128 tiles, two workgroups per CU, so that one
// tile's fp32 read-modify-write epilogue overlaps another's K loop (17204 x 1920
// x 128: 47.5 us, 62.5 with HalfE; 17920 x 5120 x 192: 201 and 219).
using HalfM = GCfg<f16, 256, 128, 64, 64, 8, 2, 3, 4>;
// K loops that the tiles of four waves run, and faster than those of eight.
// Launches of 128 tiles and more, time with four waves over time with eight:
// fp16 1.09-1.19 at K = 128, 1.06-1.18 at 256, 0.97-1.10 at 512, 0.99-1.07 at
// 640, 0.90-1.02 at 768, 0.95-1.02 at 1536; pairs 1.02-1.23, 1.05-1.21,
// 0.99-1.11, 1.03-1.21, 0.96-1.15 and 0.98-1.01.
constexpr int kShortK = 768;
static bool wide_k(int K) { return K % 64 == 0 && K >= kShortK; }
// LM head: the 256x256 schedules transposed (F rows x 256 vocabulary rows), and
// 64- and 128-row tiles for few rows.
template <typename T, bool PAIR>
using Lm = std::conditional_t<PAIR, GCfg<T, 256, 256, 128, 128, 12, 2, 3, 4, 1>,
                              GCfg<T, 256, 256, 128, 128, 11, 1, 2, 8, 1>>;
template <typename T, bool PAIR>
using LmMid = GCfg<T, 128, 256, 64, 128, PAIR ? 7 : 8, 2, 3, 4, 1>;
template <typename T, bool PAIR>
using LmSmall = GCfg<T, 64, 256, 64, 128, PAIR ? 7 : 8, 2, 4, 4, 1>;
// ... and single planes on 256x256 tiles of eight waves (run_lmhead_rows).
template <typename T>
using LmE = GCfg<T, 256, 256, 64, 128, 8, 2, 3, 4, 1>;
using LmF = GCfg<float, 128, 128, 64, 64, 0, 1, 2, 8, 1>;
// int8 B operand (block-quantized weights): the LOAD 8 schedule with int8 B
// tiles and per-block scales (three 24.5 KB stages), 256x256 tiles of 8
// waves, or 128x128 tiles of 4 waves for problems with fewer tiles.
using Q8B = GCfg<f16, 256, 256, 64, 128, 9, 2, 3, 4>;
using Q8S = GCfg<f16, 128, 128, 64, 64, 9, 2, 3, 4>;
// int4 B (packed two per byte), the same schedule
using Q4B = GCfg<f16, 256, 256, 64, 128, 10, 2, 3, 4>;
using Q4S = GCfg<f16, 128, 128, 64, 64, 10, 2, 3, 4>;

template <class C, int EPI>
static hipError_t run_gemm(const void *A, int64_t lda, const void *B, int64_t ldb, int M, int N, int K, int pair,
                           void *out, int64_t ldo, float oscale, hipStream_t st) {
  using T = typename C::type;
  static const hipError_t once = allow_lds<C>((const void *)gemm_kernel<C, EPI>);
  if (once != hipSuccess) return once;
  GemmArgs<T> g{(const T *)A, (const T *)B, lda, ldb, M, N, pair ? 2 * K : K, pair ? 2 * K : K, K, out, ldo, pair,
                oscale, QkvRope{}};
  const int tiles = ((M + C::BM - 1) / C::BM) * ((N + C::BN - 1) / C::BN);
  hipLaunchKernelGGL((gemm_kernel<C, EPI>), dim3(tiles), dim3(C::NT), C::LDS_BYTES, st, g);
  return hipGetLastError();
}

template <class C>
static hipError_t run_epi(int epi, const void *A, int64_t lda, const void *B, int64_t ldb, int M, int N, int K,
                          int pair, void *out, int64_t ldo, float oscale, hipStream_t st) {
  switch (epi) {
    case EPI_STORE_F32: return run_gemm<C, 0>(A, lda, B, ldb, M, N, K, pair, out, ldo, oscale, st);
    case EPI_RESID_ADD: return run_gemm<C, 1>(A, lda, B, ldb, M, N, K, pair, out, ldo, oscale, st);
    case EPI_SWIGLU: return run_gemm<C, 2>(A, lda, B, ldb, M, N, K, pair, out, ldo, oscale, st);
    default: return run_gemm<C, 3>(A, lda, B, ldb, M, N, K, pair, out, ldo, oscale, st);
  }
}

int gemm_k_step(int dtype) { return dtype == 1 ? CfgF::BK : BigB::BK; }

// Workgroups of gemm_kernel<C, EPI> the device holds at once (0 if unknown).
template <class C, int EPI>
static int resident_groups() {
  static const int n = [] {
    int dev = 0, cus = 0, per_cu = 0;
    if (allow_lds<C>((const void *)gemm_kernel<C, EPI>) != hipSuccess || hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)gemm_kernel<C, EPI>, C::NT,
                                                     C::LDS_BYTES) != hipSuccess)
      return 0;
    return cus * per_cu;
  }();
  return n;
}

// fp16 GEMM on the tile configuration C whose last round of tiles would
// leave over half of the device idle: the row tiles holding that round run
// as a second launch of 128x128 tiles (several per CU), which fills the
// device better; every output element is computed alike in both.
template <class C, int EPI>
static hipError_t run_gemm_tail(const void *A, int64_t lda, const void *B, int64_t ldb, int M, int N, int K, void *out,
                                int64_t ldo, float oscale, hipStream_t st) {
  const int nt_m = (M + C::BM - 1) / C::BM, nt_n = (N + C::BN - 1) / C::BN;
  const int64_t tiles = (int64_t)nt_m * nt_n;
  const int slots = resident_groups<C, EPI>();
  const int64_t rem = slots > 0 ? tiles % slots : 0;
  const int tail_mt = rem > 0 ? (int)((rem + nt_n - 1) / nt_n) : 0;
  if (rem == 0 || rem > slots / 2 || tail_mt >= nt_m) return run_gemm<C, EPI>(A, lda, B, ldb, M, N, K, 0, out, ldo, oscale, st);
  const int M1 = (nt_m - tail_mt) * C::BM;
  const size_t osz = EPI == 0 || EPI == 1 ? sizeof(float) : sizeof(f16);
  hipError_t e = run_gemm<C, EPI>(A, lda, B, ldb, M1, N, K, 0, out, ldo, oscale, st);
  if (e != hipSuccess) return e;
  return run_gemm<HalfS, EPI>((const f16 *)A + (int64_t)M1 * lda, lda, B, ldb, M - M1, N, K, 0,
                              (char *)out + (size_t)M1 * (size_t)ldo * osz, ldo, oscale, st);
}

// Estimated time of a launch: rounds of workgroups, one per CU of 256. Infinite (never
// the cheapest) for a tile that cannot run this K.
static double tile_us(const TileCost &c, int M, int N, int K) {
  if (K % c.bk || K / c.bk < c.ahead) return INFINITY;
  const int64_t tiles = (int64_t)((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
  return (double)((tiles + 255) / 256) * (c.a + c.b * K / 1000.0);
}

template <int N>
static int cheapest(const TileCost (&c)[N], int M, int Nn, int K, double *us) {
  int best = -1;
  for (int i = 0; i < N; ++i) {
    const double t = tile_us(c[i], M, Nn, K);
    if (t < *us) *us = t, best = i;
  }
  return best;
}

template <typename T, int NPL, int QB>
static int cheapest_of(int epi, int M, int N, int K, double *us) {
  if (epi == EPI_SWIGLU) return cheapest(SmallSwiglu<T, NPL, QB>::cost, M, N, K, us);
  if (epi == EPI_QKV_ROPE) return cheapest(SmallRope<T, NPL, QB>::cost, M, N, K, us);
  return cheapest(SmallPlain<T, NPL, QB>::cost, M, N, K, us);
}

// The tile to use for a problem: a small one (its index), kMid (128x128 tiles
// of eight waves, two workgroups per CU), or kBig (256x256 tiles).
enum { kBig = -1, kMid = -2 };

// big and mid: costs of the 256x256 tiles (per round of 256) and of the 128x128
// ones (per round of 512), null where they are not considered. The 256x256
// tiles keep every launch of 1024 or more of them (where mid is considered, of
// 512): over so many rounds the last one does not matter, and per
// element they are the fastest. kBig too where nothing else runs this K.
template <typename T, int NPL, int QB>
static int tile_for(int epi, int M, int N, int K, const TileCost *big, const TileCost *mid) {
  const int64_t big_tiles = (int64_t)((M + 255) / 256) * ((N + 255) / 256);
  if (epi == EPI_STORE_T && (NPL == 2 || QB)) return big_tiles >= 512 ? kBig : kMid;  // (no small tiles)
  if (big_tiles >= (mid ? 512 : 1024)) return kBig;
  double us = big ? tile_us(*big, M, N, K) : INFINITY;
  int best = kBig;
  if (mid) {
    const int64_t tiles = (int64_t)((M + mid->bm - 1) / mid->bm) * ((N + mid->bn - 1) / mid->bn);
    const double t = (double)((tiles + 511) / 512) * (mid->a + mid->b * K / 1000.0);
    if (t < us) us = t, best = kMid;
  }
  const int c = cheapest_of<T, NPL, QB>(epi, M, N, K, &us);
  return c >= 0 ? c : best;
}

// Costs of the 256x256 tiles: fp16, (hi, lo) pairs, block-quantized B. (The
// first two were fitted to tiles of eight waves; those of four take 3 to 14%
// less at K >= 1536, so they are chosen a little late.)
static constexpr TileCost kBigF16{256, 256, 32, 1, 14.0, 23.0}, kBigPair{256, 256, 32, 1, 12.0, 43.0},
    kBigQ{256, 256, 32, 1, 14.0, 27.0};
// K too short for the tiles of four waves: the 256x256 tiles of eight. And the
// 128x128 ones, considered up to K = 1536: from there on the small tiles are
// faster (block-quantized B: below 768, or where no small tile runs K). Fitted
// to 370 launches of each kind of 64 <= K < 1536, 1 to 32768 rows, 384 to 40000
// columns, three epilogues. Time against 128x128 tiles below 512 256x256 ones
// and those from there on, in the mean and at worst: fp16 0.82 and 1.13 below K
// = 768, 0.65 and 1.04 above, pairs 0.79 and 1.11, 0.69 and 1.06 (with the
// small tiles and those of four waves alone 0.89 and 1.80, 0.65 and 1.18; pairs
// 0.82 and 1.66, 0.67 and 1.32).
static constexpr TileCost kShortF16{256, 256, 32, 1, 10.0, 25.0}, kShortPair{256, 256, 32, 1, 6.0, 25.0},
    kMidF16{128, 128, 32, 1, 4.0, 20.0}, kMidPair{128, 128, 32, 1, 4.0, 14.0}, kMidQ{128, 128, 32, 1, 5.0, 17.0};

template <typename T, int NPL>
static int float_tile_for(int epi, int M, int N, int K) {
  const bool wide = wide_k(K), mid = K < 1536;
  if constexpr (NPL == 2)
    return tile_for<T, 2, 0>(epi, M, N, K, wide ? &kBigPair : &kShortPair, mid ? &kMidPair : nullptr);
  else return tile_for<T, 1, 0>(epi, M, N, K, wide ? &kBigF16 : &kShortF16, mid ? &kMidF16 : nullptr);
}

// Arguments of one GEMM launch.
template <typename T>
static GemmArgs<T> gemm_args(const void *A, int64_t lda, const void *B, int64_t ldb, int M, int N, int K, int pair,
                             void *out, int64_t ldo, float oscale, const uint16_t *Bs = nullptr) {
  GemmArgs<T> g{(const T *)A, (const T *)B, lda, ldb, M, N, pair ? 2 * K : K, pair ? 2 * K : K, K, out, ldo, pair,
                oscale, QkvRope{}};
  g.Bs = Bs;
  return g;
}

// Pair operands: small tiles, 128x128 (S), 256x256 of four (B) or eight (E) waves.
template <class B, class E, class S>
static hipError_t run_pair(int epi, const void *A, int64_t lda, const void *Bm, int64_t ldb, int M, int N, int K,
                           void *out, int64_t ldo, float oscale, hipStream_t st) {
  using T = typename B::type;
  const int c = float_tile_for<T, 2>(epi, M, N, K);
  if (c >= 0) {
    const GemmArgs<T> g = gemm_args<T>(A, lda, Bm, ldb, M, N, K, 1, out, ldo, oscale);
    if constexpr (std::is_same_v<T, f16>) return small_gemm_f16p(epi, c, g, st);
    else return small_gemm_bf16p(epi, c, g, st);
  }
  if (c == kMid) return run_epi<S>(epi, A, lda, Bm, ldb, M, N, K, 1, out, ldo, oscale, st);
  return wide_k(K) ? run_epi<B>(epi, A, lda, Bm, ldb, M, N, K, 1, out, ldo, oscale, st)
                   : run_epi<E>(epi, A, lda, Bm, ldb, M, N, K, 1, out, ldo, oscale, st);
}

template <class C>
static hipError_t run_epi_tail(int epi, const void *A, int64_t lda, const void *B, int64_t ldb, int M, int N, int K,
                               void *out, int64_t ldo, float oscale, hipStream_t st) {
  switch (epi) {
    case EPI_STORE_F32: return run_gemm_tail<C, 0>(A, lda, B, ldb, M, N, K, out, ldo, oscale, st);
    case EPI_RESID_ADD: return run_gemm_tail<C, 1>(A, lda, B, ldb, M, N, K, out, ldo, oscale, st);
    case EPI_SWIGLU: return run_gemm_tail<C, 2>(A, lda, B, ldb, M, N, K, out, ldo, oscale, st);
    default: return run_gemm_tail<C, 3>(A, lda, B, ldb, M, N, K, out, ldo, oscale, st);
  }
}

hipError_t launch_gemm(int dtype, int epi, const void *A, int64_t lda, const void *B, int64_t ldb, int M, int N,
                       int K, int pair, void *out, int64_t ldo, float oscale, hipStream_t st) {
  if (M <= 0 || N <= 0) return hipSuccess;
  if (dtype == 0) {
    if (pair) return run_pair<PairB, PairE, PairS>(epi, A, lda, B, ldb, M, N, K, out, ldo, oscale, st);
    const int64_t big_tiles = (int64_t)((M + 255) / 256) * ((N + 255) / 256);
    if (big_tiles >= 512) return run_epi<BigB>(epi, A, lda, B, ldb, M, N, K, pair, out, ldo, oscale, st);
    return run_epi<SmallB>(epi, A, lda, B, ldb, M, N, K, pair, out, ldo, oscale, st);
  }
  if (dtype == 2) {
    if (pair) return run_pair<HalfPairB, HalfPairE, HalfPairS>(epi, A, lda, B, ldb, M, N, K, out, ldo, oscale, st);
    const int c = float_tile_for<f16, 1>(epi, M, N, K);
    if (c >= 0) return small_gemm_f16(epi, c, gemm_args<f16>(A, lda, B, ldb, M, N, K, 0, out, ldo, oscale), st);
    if (c == kMid) return run_epi<HalfS>(epi, A, lda, B, ldb, M, N, K, 0, out, ldo, oscale, st);
    if (wide_k(K)) return run_epi_tail<HalfB>(epi, A, lda, B, ldb, M, N, K, out, ldo, oscale, st);
    if (epi == EPI_RESID_ADD) return run_gemm_tail<HalfM, 1>(A, lda, B, ldb, M, N, K, out, ldo, oscale, st);
    return run_epi_tail<HalfE>(epi, A, lda, B, ldb, M, N, K, out, ldo, oscale, st);
  }
  return run_epi<CfgF>(epi, A, lda, B, ldb, M, N, K, 0, out, ldo, oscale, st);
}

template <class C, int EPI>
static hipError_t run_gemm_q8(const void *A, int64_t lda, const void *Bq, const uint16_t *Bs, int M, int N, int K,
                              void *out, int64_t ldo, float oscale, hipStream_t st) {
  static const hipError_t once = allow_lds<C>((const void *)gemm_kernel<C, EPI>);
  if (once != hipSuccess) return once;
  GemmArgs<f16> g{(const f16 *)A, (const f16 *)Bq, lda, (int64_t)K * C::QBITS / 8, M, N, K, K, K, out, ldo, 0,
                  oscale, QkvRope{}};
  g.Bs = Bs;
  const int tiles = ((M + C::BM - 1) / C::BM) * ((N + C::BN - 1) / C::BN);
  hipLaunchKernelGGL((gemm_kernel<C, EPI>), dim3(tiles), dim3(C::NT), C::LDS_BYTES, st, g);
  return hipGetLastError();
}

template <class C>
static hipError_t run_q8_epi(int epi, const void *A, int64_t lda, const void *Bq, const uint16_t *Bs, int M, int N,
                             int K, void *out, int64_t ldo, float oscale, hipStream_t st) {
  switch (epi) {
    case EPI_STORE_F32: return run_gemm_q8<C, 0>(A, lda, Bq, Bs, M, N, K, out, ldo, oscale, st);
    case EPI_RESID_ADD: return run_gemm_q8<C, 1>(A, lda, Bq, Bs, M, N, K, out, ldo, oscale, st);
    case EPI_SWIGLU: return run_gemm_q8<C, 2>(A, lda, Bq, Bs, M, N, K, out, ldo, oscale, st);
    default: return run_gemm_q8<C, 3>(A, lda, Bq, Bs, M, N, K, out, ldo, oscale, st);
  }
}

// Block-quantized B of QB bits: small tiles, 128x128 (S), 256x256 (B).
template <int QB, class B, class S>
static hipError_t run_quant(int epi, const void *A, int64_t lda, const void *Bq, const uint16_t *Bs, int M, int N, int K,
                            void *out, int64_t ldo, float oscale, hipStream_t st) {
  if (M <= 0 || N <= 0) return hipSuccess;
  if (K % 32 != 0) return hipErrorInvalidValue;
  const int c = tile_for<f16, 1, QB>(epi, M, N, K, &kBigQ, K < kShortK || K % 128 ? &kMidQ : nullptr);
  if (c >= 0) {
    const GemmArgs<f16> g = gemm_args<f16>(A, lda, Bq, (int64_t)K * QB / 8, M, N, K, 0, out, ldo, oscale, Bs);
    return QB == 8 ? small_gemm_q8(epi, c, g, st) : small_gemm_q4(epi, c, g, st);
  }
  return c == kMid ? run_q8_epi<S>(epi, A, lda, Bq, Bs, M, N, K, out, ldo, oscale, st)
                   : run_q8_epi<B>(epi, A, lda, Bq, Bs, M, N, K, out, ldo, oscale, st);
}

hipError_t launch_gemm_q8(int epi, const void *A, int64_t lda, const void *Bq, const uint16_t *Bs, int M, int N,
                          int K, void *out, int64_t ldo, float oscale, hipStream_t st) {
  return run_quant<8, Q8B, Q8S>(epi, A, lda, Bq, Bs, M, N, K, out, ldo, oscale, st);
}

hipError_t launch_gemm_q4(int epi, const void *A, int64_t lda, const void *Bq, const uint16_t *Bs, int M, int N,
                          int K, void *out, int64_t ldo, float oscale, hipStream_t st) {
  return run_quant<4, Q4B, Q4S>(epi, A, lda, Bq, Bs, M, N, K, out, ldo, oscale, st);
}

template <class C, int EPI>
static hipError_t run_gemm_grouped(const void *A, int64_t lda, const void *B, int64_t ldb, int64_t group_stride,
                                   const int *tile_group, int M, int N, int K, void *out, int64_t ldo, float oscale,
                                   hipStream_t st) {
  using T = typename C::type;
  static const hipError_t once = allow_lds<C>((const void *)gemm_kernel<C, EPI>);
  if (once != hipSuccess) return once;
  GemmArgs<T> g{(const T *)A, (const T *)B, lda, ldb, M, N, K, K, K, out, ldo, 0, oscale, QkvRope{},
                tile_group, group_stride};
  const int tiles = (M / C::BM) * ((N + C::BN - 1) / C::BN);
  hipLaunchKernelGGL((gemm_kernel<C, EPI>), dim3(tiles), dim3(C::NT), C::LDS_BYTES, st, g);
  return hipGetLastError();
}

template <class C>
static hipError_t run_grouped_epi(int epi, const void *A, int64_t lda, const void *B, int64_t ldb,
                                  int64_t group_stride, const int *tile_group, int M, int N, int K, void *out,
                                  int64_t ldo, float oscale, hipStream_t st) {
  switch (epi) {
    case EPI_STORE_F32:
      return run_gemm_grouped<C, 0>(A, lda, B, ldb, group_stride, tile_group, M, N, K, out, ldo, oscale, st);
    case EPI_RESID_ADD:
      return run_gemm_grouped<C, 1>(A, lda, B, ldb, group_stride, tile_group, M, N, K, out, ldo, oscale, st);
    case EPI_SWIGLU:
      return run_gemm_grouped<C, 2>(A, lda, B, ldb, group_stride, tile_group, M, N, K, out, ldo, oscale, st);
    case EPI_STORE_T:
      return run_gemm_grouped<C, 3>(A, lda, B, ldb, group_stride, tile_group, M, N, K, out, ldo, oscale, st);
    default: return hipErrorInvalidValue;
  }
}

// Rows per tile of the grouped GEMMs of a mixture of experts (K columns d for
// gate/up, F for down), for segments of `avg` rows on average. A tile belongs
// to one expert, so the padding is half a tile per expert. 256-row tiles
// (fp16) from 512 rows a segment: at 656 rows (256 experts, d 2048, F 512)
// gate/up took 1190 us with 128-row tiles and 1010 with 256-row ones of eight
// waves, down 755 and 691 (gate/up on those of four waves, at 656 rows: 839).
// 128-row tiles from 64; below, small tiles, where the stream of the experts'
// weights bounds the launch, as far as K fills their ring of stages (46 rows:
// gate/up 346 -> 279 us with 64-row tiles, down 197 -> 208; 16-row tiles up to
// 12 rows a segment).
int gemm_group_rows(int dtype, double avg, int d, int F) {
  if (dtype == 1) return CfgF::BM;
  if (dtype != 2) return SmallB::BM;
  if (avg >= 512.0) return HalfB::BM;
  if (avg >= 64.0) return HalfS::BM;
  using S = SmallSwiglu<f16, 1, 0>;
  using P = SmallPlain<f16, 1, 0>;
  auto fits = [](const TileCost &c, int K) { return K % c.bk == 0 && K / c.bk >= c.ahead; };
  if (avg <= 12.0 && fits(S::cost[0], d) && fits(P::cost[1], F)) return S::cost[0].bm;
  if (fits(S::cost[1], d) && fits(P::cost[3], F)) return S::cost[1].bm;
  return HalfS::BM;
}
int gemm_group_rows_max(int dtype) { return dtype == 2 ? HalfB::BM : dtype == 1 ? CfgF::BM : SmallB::BM; }

hipError_t launch_gemm_grouped(int dtype, int bm, int epi, const void *A, int64_t lda, const void *B, int64_t ldb,
                               int64_t group_stride, const int *tile_group, int M, int N, int K, void *out,
                               int64_t ldo, float oscale, hipStream_t st) {
  if (M <= 0 || N <= 0) return hipSuccess;
  if (!tile_group || bm <= 0 || M % bm) return hipErrorInvalidValue;
  if (dtype == 2 && bm == HalfB::BM && !wide_k(K))
    return run_grouped_epi<HalfE>(epi, A, lda, B, ldb, group_stride, tile_group, M, N, K, out, ldo, oscale, st);
  if (dtype == 2 && bm == HalfB::BM)
    return run_grouped_epi<HalfB>(epi, A, lda, B, ldb, group_stride, tile_group, M, N, K, out, ldo, oscale, st);
  if (dtype == 2 && bm == HalfS::BM)
    return run_grouped_epi<HalfS>(epi, A, lda, B, ldb, group_stride, tile_group, M, N, K, out, ldo, oscale, st);
  if (dtype == 2) {
    GemmArgs<f16> g = gemm_args<f16>(A, lda, B, ldb, M, N, K, 0, out, ldo, oscale);
    g.tile_group = tile_group;
    g.group_stride = group_stride;
    // the tiles of 16 and 64 rows: SwiGLU c0, c1; plain c1, c3
    if (bm == 16) return small_gemm_f16(epi, epi == EPI_SWIGLU ? 0 : 1, g, st);
    if (bm == 64) return small_gemm_f16(epi, epi == EPI_SWIGLU ? 1 : 3, g, st);
    return hipErrorInvalidValue;
  }
  if (bm != gemm_group_rows_max(dtype)) return hipErrorInvalidValue;
  if (dtype == 1)
    return run_grouped_epi<CfgF>(epi, A, lda, B, ldb, group_stride, tile_group, M, N, K, out, ldo, oscale, st);
  return run_grouped_epi<SmallB>(epi, A, lda, B, ldb, group_stride, tile_group, M, N, K, out, ldo, oscale, st);
}

template <class C>
static hipError_t run_qkv_rope(const void *A, int64_t lda, const void *B, int64_t ldb, int M, int N, int K,
                               int pair, float oscale, const QkvRope &r, hipStream_t st) {
  using T = typename C::type;
  static const hipError_t once = allow_lds<C>((const void *)gemm_kernel<C, 4>);
  if (once != hipSuccess) return once;
  GemmArgs<T> g{(const T *)A, (const T *)B, lda, ldb, M, N, pair ? 2 * K : K, pair ? 2 * K : K, K, nullptr, 0,
                pair, oscale, r};
  const int tiles = ((M + C::BM - 1) / C::BM) * ((N + C::BN - 1) / C::BN);
  hipLaunchKernelGGL((gemm_kernel<C, 4>), dim3(tiles), dim3(C::NT), C::LDS_BYTES, st, g);
  return hipGetLastError();
}

// Small RoPE tile for a problem (-1: none), and whether the 256x256 tiles,
// whose waves of 128 columns hold a head each, can run it. Neither: the
// projection and the rotation run as two kernels (block-quantized B of K = 128,
// shorter than the ring of any small tile, or of 1024 256x256 tiles and more).
static int rope_tile_for(int dtype, int qbits, int pair, int M, int N, int K) {
  if (qbits == 8) return tile_for<f16, 1, 8>(EPI_QKV_ROPE, M, N, K, nullptr, nullptr);
  if (qbits == 4) return tile_for<f16, 1, 4>(EPI_QKV_ROPE, M, N, K, nullptr, nullptr);
  if (dtype == 0) return pair ? tile_for<bf16, 2, 0>(EPI_QKV_ROPE, M, N, K, &kBigPair, nullptr) : -1;
  if (pair) return tile_for<f16, 2, 0>(EPI_QKV_ROPE, M, N, K, &kBigPair, nullptr);
  return tile_for<f16, 1, 0>(EPI_QKV_ROPE, M, N, K, &kBigF16, nullptr);
}
static bool rope_big_ok(int dtype, int qbits, int pair, int M, int N) {
  return !qbits && (dtype == 2 || (dtype == 0 && pair)) &&
         (int64_t)((M + 255) / 256) * ((N + 255) / 256) >= 128;
}

bool gemm_qkv_rope_ok(int dtype, int qbits, int pair, int M, int N, int K, int head_dim) {
  if (head_dim != 128 || N % 128 || M <= 0 || dtype == 1) return false;
  return rope_tile_for(dtype, qbits, pair, M, N, K) >= 0 || rope_big_ok(dtype, qbits, pair, M, N);
}

hipError_t launch_gemm_qkv_rope(int dtype, int qbits, const void *A, int64_t lda, const void *B, const uint16_t *Bs,
                                int64_t ldb, int M, int N, int K, int pair, float oscale, const QkvRope &r,
                                hipStream_t st) {
  if (!gemm_qkv_rope_ok(dtype, qbits, pair, M, N, K, 128)) return hipErrorInvalidValue;
  const int c = rope_tile_for(dtype, qbits, pair, M, N, K);
  if (c >= 0) {
    if (dtype == 0) {
      GemmArgs<bf16> g = gemm_args<bf16>(A, lda, B, ldb, M, N, K, pair, nullptr, 0, oscale);
      g.rope = r;
      return small_gemm_bf16p(EPI_QKV_ROPE, c, g, st);
    }
    GemmArgs<f16> g = gemm_args<f16>(A, lda, B, qbits ? (int64_t)K * qbits / 8 : ldb, M, N, K, pair, nullptr, 0,
                                     oscale, Bs);
    g.rope = r;
    if (qbits == 8) return small_gemm_q8(EPI_QKV_ROPE, c, g, st);
    if (qbits == 4) return small_gemm_q4(EPI_QKV_ROPE, c, g, st);
    return pair ? small_gemm_f16p(EPI_QKV_ROPE, c, g, st) : small_gemm_f16(EPI_QKV_ROPE, c, g, st);
  }
  if (dtype == 0) return run_qkv_rope<PairE>(A, lda, B, ldb, M, N, K, pair, oscale, r, st);
  if (pair) return run_qkv_rope<HalfPairE>(A, lda, B, ldb, M, N, K, pair, oscale, r, st);
  return run_qkv_rope<HalfE>(A, lda, B, ldb, M, N, K, 0, oscale, r, st);
}

void lmhead_plan(int dtype, int V, int R, int *tiles_per_split, int *nsplit) {
  (void)R;
  // The split of the vocabulary depends on V only, so that a row's
  // log-sum-exp is merged in the same order whatever batch it is in; about
  // 256 splits keep even a one-row-tile launch spread over the CUs.
  const int bn = dtype == 1 ? LmF::BN : Lm<f16, false>::BN;
  const int vt = (V + bn - 1) / bn;
  const int tps = std::max(1, vt / 256);
  *tiles_per_split = tps;
  *nsplit = (vt + tps - 1) / tps;
}

template <class C>
static hipError_t run_lmhead(const void *W, const void *F, int V, int R, int K, int tiles_per_split, float wscale,
                             float *part_m, float *part_s, const int32_t *target, float *zt, hipStream_t st) {
  using T = typename C::type;
  static const hipError_t once = allow_lds<C>((const void *)lmhead_lse_kernel<C>);
  if (once != hipSuccess) return once;
  const int nsplit = ((V + C::BN - 1) / C::BN + tiles_per_split - 1) / tiles_per_split;
  const int nrt = (R + C::BM - 1) / C::BM;
  // Splits dealt to the XCDs whole leave some with one more than others: only
  // where that costs no further round of 32 workgroups an XCD. (fp16, us, whole
  // splits and even bands: 2560 x 151936, 6400 rows, 30 rounds both 3856 and
  // 4115; 1500 rows, 8 rounds and 7 984 and 914; 2560 x 40000, 3328 rows, 9 and
  // 8 573 and 539.)
  const int per_xcd = (nsplit + 7) / 8 * nrt, strided = (per_xcd + 31) / 32 <= (nsplit * nrt + 255) / 256;
  hipLaunchKernelGGL((lmhead_lse_kernel<C>), dim3(strided ? per_xcd * 8 : nsplit * nrt), dim3(C::NT), C::LDS_BYTES, st,
                     (const T *)W, (const T *)F, V, R, K, tiles_per_split, nsplit, strided, wscale * kLog2e, part_m,
                     part_s, target, zt);
  return hipGetLastError();
}

// The row tile: 64 rows up to 64 and 128 up to 128, where the launch is bound by
// the stream of W and not by the matrix cores; above, 256. Single planes take
// the tiles of four waves there for a long K and more than one workgroup per CU
// (151936 x 2560: 1000 rows 636 us, 714 with eight waves, 6400 rows 3856 and
// 4429; 40000 x 2560, 512 rows 125 and 125), else those of eight, two per SIMD,
// whose exponentials do not wait for each other (four and eight waves: 40000 x
// 896, 1000 rows 102 and 80; 151936 x 128, 6400 rows 826 and 531; 40000 x 2560,
// 129 rows 65 and 59; 151936 x 1536, 1500 rows 684 and 624, 6400 rows 2713 and
// 2577). Pairs always (151936 x 128, 6400 rows 1119 against 1110).
template <typename T, bool PAIR>
static hipError_t run_lmhead_rows(const void *W, const void *F, int V, int R, int K, int tiles_per_split,
                                  float wscale, float *part_m, float *part_s, const int32_t *target, float *zt,
                                  hipStream_t st) {
  if (R <= 64)
    return run_lmhead<LmSmall<T, PAIR>>(W, F, V, R, K, tiles_per_split, wscale, part_m, part_s, target, zt, st);
  if (R <= 128)
    return run_lmhead<LmMid<T, PAIR>>(W, F, V, R, K, tiles_per_split, wscale, part_m, part_s, target, zt, st);
  if constexpr (!PAIR) {
    const int groups = ((V + 255) / 256 + tiles_per_split - 1) / tiles_per_split * ((R + 255) / 256);
    if (K < 2048 || groups <= 256)
      return run_lmhead<LmE<T>>(W, F, V, R, K, tiles_per_split, wscale, part_m, part_s, target, zt, st);
  } else if (K % 64 || K < 128) {
    return run_lmhead<LmMid<T, PAIR>>(W, F, V, R, K, tiles_per_split, wscale, part_m, part_s, target, zt, st);
  }
  return run_lmhead<Lm<T, PAIR>>(W, F, V, R, K, tiles_per_split, wscale, part_m, part_s, target, zt, st);
}

hipError_t launch_lmhead_lse(int dtype, const void *W, const void *F, int V, int R, int K, int pair,
                             int tiles_per_split, float wscale, float *part_m, float *part_s, const int32_t *target,
                             float *zt, hipStream_t st) {
  if (R <= 0) return hipSuccess;
  if ((target == nullptr) != (zt == nullptr)) return hipErrorInvalidValue;
  if (dtype == 1) return run_lmhead<LmF>(W, F, V, R, K, tiles_per_split, wscale, part_m, part_s, target, zt, st);
  if (dtype == 2)
    return run_lmhead_rows<f16, false>(W, F, V, R, K, tiles_per_split, wscale, part_m, part_s, target, zt, st);
  return pair ? run_lmhead_rows<bf16, true>(W, F, V, R, K, tiles_per_split, wscale, part_m, part_s, target, zt, st)
              : run_lmhead_rows<bf16, false>(W, F, V, R, K, tiles_per_split, wscale, part_m, part_s, target, zt, st);
}

}  // namespace jetk
