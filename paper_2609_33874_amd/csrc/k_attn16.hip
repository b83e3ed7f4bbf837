// Grouped-query attention for single 16-bit planes and head_dim 128 (the
// decoders' shapes): the arithmetic of attn_kernel (k_attn.hip) per query, key tile by
// key tile of 64, with the staging done by direct global->LDS loads.
//
// What bounds it: at few items per CU the serial chain of a key tile (scores,
// maximum, exponentials, values: about 0.7 us) and the latency of its loads;
// at many items the matrix cores and the LDS reads of K and V. Passing tiles
// through registers (one tile ahead, V transposed element by element on the way
// to the LDS, two barriers per tile) took 2.3-3 us per tile. Here
//   * K and V rows go straight into one of two stages while the other is
//     computed, one barrier per tile; own-candidate tiles are part of the same
//     stream;
//   * V stays row-major and is read transposed (ds_read_b64_tr_b16).
// Two stages of 32 KB let two workgroups share a CU, one's chain under the
// other's. A ring of four (one workgroup per CU, three tiles in flight) is no
// faster even where every workgroup has a CU of its own: 12 query heads, 2 KV
// heads, candidates' launch with K and V evicted between calls, us: one question
// of 731 keys (12 items) 24.9 with four stages, 23.9 with two; 16 questions
// of 700 (192 items) 24.8 and 23.7; past 256 items it runs a second round: 132
// questions of 700 (264 items) 53.1 and 33.0.
// A workgroup of NW waves takes 16 QB NW query slots of one (question, KV
// head); every query runs the same operations in the same order whatever QB
// and NW are, so a candidate rounds alike in any batch.
#include "attn_common.h"
#include "gemm_core.h"

namespace jetk {

template <int N>
__device__ __forceinline__ void wait_lgkmcnt() {
  static_assert(N >= 0 && N < 16, "lgkmcnt range");
  asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N) : "memory");
}

// Four 16-bit elements per lane, transposed within groups of 16 lanes: lane l
// supplies elements 4 (l % 4) .. + 3 of row (l % 16) / 4 of a 4 x 16 block and
// receives column l % 16.
template <int OFF>
__device__ __forceinline__ void ds_read8_tr(uint2 &v, uint32_t addr) {
  static_assert(OFF >= 0 && OFF < 65536, "ds offset range");
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF) : "memory");
}

// max / sum over the four lane groups that hold one query (lanes l, l ^ 16,
// l ^ 32, l ^ 48)
__device__ __forceinline__ float group_max(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

template <typename T, int MODE, int QB, int NW>
__global__ __launch_bounds__(64 * NW, 2) void attn16_kernel(AttnArgs a) {
  constexpr int HD = 128, KT = 64, BLOCK = 16 * QB * NW;
  constexpr int PLANE = KT * HD * 2, STAGE = 2 * PLANE;  // bytes: K, then V
  constexpr int LD = KT / 4 / NW;                          // direct loads per wave of a tile of K or V
  static_assert(KT / 4 % NW == 0, "whole loads per wave");
  extern __shared__ __align__(16) char smem[];

  const AttnItem it = a.items[blockIdx.x];
  const int G = a.Hq / a.Hkv, qrow0 = a.qs.qrow0[it.q];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, l16 = lane & 15;
  const int r_first = qrow0 + it.slot0 / G, r_last = qrow0 + (it.slot0 + it.nslots - 1) / G;
  const bool own = MODE == 1 && a.s_suf > 0;
  const int npre = MODE == 0 ? it.nkeys_pre : a.qs.pre_len[it.q];
  const int64_t pbase = ((int64_t)it.kvh * a.s_pre + a.qs.pre_slot0[it.q]) * HD;
  const T *Kp = (const T *)a.Kp + pbase, *Vp = (const T *)a.Vp + pbase;
  const T *Ko = own ? (const T *)a.Ks + (int64_t)it.kvh * a.s_suf * HD : nullptr;
  const T *Vo = own ? (const T *)a.Vs + (int64_t)it.kvh * a.s_suf * HD : nullptr;

  // The stream of key tiles: the prefix (cs < 0), then for every candidate with
  // rows in the item (first body row cs) its rows up to the item's last one,
  // in tiles that start at cs. t0: first key (prefix) or body row, nk keys;
  // nk = 0 past the end.
  struct Tile {
    int cs, t0, nk;
  };
  // row_n of the item's rows (at most BLOCK), one or two per lane
  int cs_first = 0, n_a = 1, n_b = 1;
  if (own) {
    cs_first = r_first - a.row_t[r_first] + 1;
    n_a = a.row_n[min(r_first + lane, r_last)];
    if constexpr (BLOCK > 64) n_b = a.row_n[min(r_first + 64 + lane, r_last)];
  }
  auto own_n = [&](int cs) {  // body rows of the candidate that starts at row cs
    const int i = max(cs, r_first) - r_first;
    if (BLOCK > 64 && i >= 64) return __builtin_amdgcn_readlane(n_b, i - 64);
    return __builtin_amdgcn_readlane(n_a, i);
  };
  auto own_tile = [&](int cs, int ts) {  // the first tile at or after row ts of candidate cs
    if (cs > r_last) return Tile{0, 0, 0};
    const int cend = min(cs + own_n(cs) - 1, r_last);
    return Tile{cs, ts, min(KT, cend - ts + 1)};
  };
  auto next_tile = [&](const Tile &t) {
    if (t.nk == 0) return t;
    if (t.cs < 0) {
      const int kb = t.t0 + KT;
      if (kb < npre) return Tile{-1, kb, min(KT, npre - kb)};
      return own ? own_tile(cs_first, cs_first) : Tile{0, 0, 0};
    }
    const int n = own_n(t.cs);
    if (t.t0 + KT <= min(t.cs + n - 1, r_last)) return own_tile(t.cs, t.t0 + KT);
    return own_tile(t.cs + n, t.cs + n);
  };
  // Rows past nk load the last one (they are masked). 16-byte chunk c of row r
  // is stored at c ^ (r mod 16) (K: the 16 rows of a fragment read) or at
  // c ^ 2 (r mod 8) (V: the rows of a transposed read).
  auto issue = [&](const Tile &t, int stage) {
    const T *K = t.cs < 0 ? Kp : Ko, *V = t.cs < 0 ? Vp : Vo;
    char *dst = smem + stage * STAGE;
#pragma unroll
    for (int i = 0; i < LD; ++i) {
      const int blk = i * NW + wave, r = blk * 4 + g;
      const int64_t off = (int64_t)(t.t0 + min(r, t.nk - 1)) * HD;
      const int ck = l16 ^ (r & 15), cv = l16 ^ ((r & 7) << 1);
      __builtin_amdgcn_global_load_lds((const void *)(K + off + ck * 8), (lds_void *)(dst + blk * 1024), 16, 0, 0);
      __builtin_amdgcn_global_load_lds((const void *)(V + off + cv * 8), (lds_void *)(dst + PLANE + blk * 1024), 16, 0,
                                       0);
    }
  };
  Tile cur{-1, 0, min(KT, npre)};  // (every prefix has a key)
  if (cur.nk > 0) issue(cur, 0);
  Tile ahead = next_tile(cur);

  bool valid[QB];
  int row[QB], head[QB], qi[QB], first[QB];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const int sl = (wave * QB + qb) * 16 + l16;
    valid[qb] = sl < it.nslots;
    const int slot = it.slot0 + (valid[qb] ? sl : 0);
    head[qb] = it.kvh * G + slot % G;
    qi[qb] = slot / G;
    row[qb] = qrow0 + qi[qb];
    first[qb] = own && valid[qb] ? row[qb] - a.row_t[row[qb]] + 1 : -1;
  }
  const bool idle = (wave * QB) * 16 >= it.nslots;  // no query: loads and barriers only
  const T *Q = (const T *)a.Q;
  Frag<T> qf[QB][4];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb)
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
      frag_load(qf[qb][ks], Q + ((int64_t)row[qb] * a.Hq + head[qb]) * HD + ks * 32 + g * 8);

  const float scale2 = a.scale * kLog2e;
  float m_run[QB], l_run[QB];
  f32x4 acc[QB][HD / 16];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    m_run[qb] = -INFINITY;
    l_run[qb] = 0.0f;
#pragma unroll
    for (int d = 0; d < HD / 16; ++d) acc[qb][d] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  }
  // Fragment reads as inline asm, so that they are waited for here and not by
  // the compiler (which would wait for the direct loads in flight as well).
  // K rows at stage + kb * 4096; the transposed V read: lane l supplies 4
  // elements of key 4 g + (l % 16) / 4 and receives keys 4 g .. + 3 of dim
  // l % 16 of the block.
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void *)smem;
  uint32_t koff[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) koff[ks] = lds0 + l16 * 256 + (((ks * 4 + g) ^ l16) << 4);
  const int vrow = 4 * g + (l16 >> 2), vsw = (vrow & 7) << 5;
  const uint32_t voff = lds0 + PLANE + vrow * 256 + ((l16 >> 1) & 1) * 16 + (l16 & 1) * 8;

  // Q has arrived (with it the first tile, which was issued before it): the
  // compiler would otherwise wait for every load in flight at each use of Q in
  // the loop
  __builtin_amdgcn_s_waitcnt(0 | 7 << 4 | 15 << 8);
  int stage = 0;
  while (cur.nk > 0) {
    // this tile has landed (own loads; with the barrier every wave's), and
    // every wave is done with the other stage, which is filled next
    wait_vmcnt<0>();
    wait_lgkmcnt0();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (ahead.nk > 0) {
      issue(ahead, stage ^ 1);
      ahead = next_tile(ahead);
    }
    const int nk = cur.nk;
    if (!idle) {
      const uint32_t so = (uint32_t)(stage * STAGE);
      f32x4 s[QB][4];
      Frag<T> fk[2][4];
      auto read_k = [&](int ks, int kb, Frag<T> &f) { ds_read16<0>(f.v, koff[ks] + so + kb * 4096); };
      auto score = [&](int ks, int kb, Frag<T> &f) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) mma16(s[qb][kb], f, qf[qb][ks]);
      };
      auto arrived = [&](Frag<T> (&f)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(f[i].v));
      };
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) s[qb][kb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      if (nk > 48) {
        // 32 dims at a time over all four key blocks (four independent chains
        // of MFMAs), the next ones' reads ahead. No read is in flight across a
        // branch: the compiler must not get to copy its registers.
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) read_k(0, kb, fk[0][kb]);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          if (ks < 3) {
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) read_k(ks + 1, kb, fk[(ks + 1) & 1][kb]);
            wait_lgkmcnt<4>();
          } else {
            wait_lgkmcnt<0>();
          }
          arrived(fk[ks & 1]);
#pragma unroll
          for (int kb = 0; kb < 4; ++kb) score(ks, kb, fk[ks & 1][kb]);
          __builtin_amdgcn_sched_barrier(0);
        }
      } else {
#pragma unroll
        for (int kb = 0; kb < 3; ++kb)
          if (kb * 16 < nk) {
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) read_k(ks, kb, fk[0][ks]);
            wait_lgkmcnt<0>();
            arrived(fk[0]);
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) score(ks, kb, fk[0][ks]);
            __builtin_amdgcn_sched_barrier(0);
          }
      }
      Frag<T> pf[QB][2];
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        float mx = -INFINITY;
        // prefix tiles every key of which every query of the block sees skip the mask
        if (cur.cs < 0 && __all(nk == KT && (MODE != 0 || cur.t0 + KT - 1 <= qi[qb]))) {
#pragma unroll
          for (int kb = 0; kb < 4; ++kb)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              s[qb][kb][e] *= scale2;
              mx = fmaxf(mx, s[qb][kb][e]);
            }
        } else {
          // last visible key of the tile: the prefix tile's (causal: the
          // query's own position), or the query's own row of its candidate's tile
          const int last = cur.cs < 0 ? (MODE == 0 ? min(nk - 1, qi[qb] - cur.t0) : nk - 1)
                                      : (first[qb] == cur.cs ? min(nk - 1, row[qb] - cur.t0) : -1);
#pragma unroll
          for (int kb = 0; kb < 4; ++kb)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float z = kb * 16 + 4 * g + e <= last ? s[qb][kb][e] * scale2 : -INFINITY;
              s[qb][kb][e] = z;
              mx = fmaxf(mx, z);
            }
        }
        mx = group_max(mx);
        // Every query sees key 0 of the first tile, so m_new is finite: exp2 of
        // the (<= 0) differences directly, with exp2(-inf) = 0 for masked
        // keys and for the initial m_run. A tile with no key visible to a
        // query leaves its m_run, l_run and acc unchanged (alpha = 1, p = 0).
        const float m_new = fmaxf(m_run[qb], mx);
        const float alpha = __builtin_amdgcn_exp2f(m_run[qb] - m_new);
        float p[4][4], psum = 0.0f;
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            p[kb][e] = __builtin_amdgcn_exp2f(s[qb][kb][e] - m_new);
            psum += p[kb][e];
          }
        l_run[qb] = l_run[qb] * alpha + psum;
        if (__any(alpha != 1.0f)) {
#pragma unroll
          for (int d = 0; d < HD / 16; ++d) acc[qb][d] *= alpha;
        }
        m_run[qb] = m_new;
#pragma unroll
        for (int mm = 0; mm < 2; ++mm) {
          const float x8[8] = {p[2 * mm][0], p[2 * mm][1], p[2 * mm][2], p[2 * mm][3],
                               p[2 * mm + 1][0], p[2 * mm + 1][1], p[2 * mm + 1][2], p[2 * mm + 1][3]};
          pf[qb][mm] = pack8<T>(x8);
        }
      }
#pragma unroll
      for (int mm = 0; mm < 2; ++mm) {
        if (mm * 32 >= nk) continue;
        // DB blocks of 16 dims at a time, the next ones' reads ahead
        constexpr int DB = 4, NC = HD / 16 / DB;
        uint2 fv[2][DB][2];  // [set][block][keys 0..15, 16..31 of the half]
        auto read_v = [&](int c, uint2 (&f)[DB][2]) {
#pragma unroll
          for (int d = 0; d < DB; ++d) {
            const uint32_t at = voff + so + mm * 8192 + (((c * DB + d) << 5) ^ vsw);
            ds_read8_tr<0>(f[d][0], at);
            ds_read8_tr<4096>(f[d][1], at);
          }
        };
        read_v(0, fv[0]);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          if (c + 1 < NC) {
            read_v(c + 1, fv[(c + 1) & 1]);
            wait_lgkmcnt<2 * DB>();
          } else {
            wait_lgkmcnt<0>();
          }
          uint2(&f)[DB][2] = fv[c & 1];
#pragma unroll
          for (int d = 0; d < DB; ++d) asm volatile("" : "+v"(f[d][0]), "+v"(f[d][1]));
#pragma unroll
          for (int d = 0; d < DB; ++d) {
            Frag<T> v;
            v.v = __builtin_bit_cast(typename Vec8<T>::type, make_uint4(f[d][0].x, f[d][0].y, f[d][1].x, f[d][1].y));
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) mma16(acc[qb][c * DB + d], v, pf[qb][mm]);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    cur = next_tile(cur);
    stage ^= 1;
  }

#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    float l_tot = l_run[qb] + __shfl_xor(l_run[qb], 16);
    l_tot += __shfl_xor(l_tot, 32);
    if (!valid[qb]) continue;
    const float inv = 1.0f / l_tot;
    T *O = (T *)a.O;
#pragma unroll
    for (int db = 0; db < HD / 16; ++db) {
      // dims 16 db + 4 g .. + 3 of this lane's query, one 8-byte store per plane
      float o[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = acc[qb][db][e] * inv;
      T *dst = O + (int64_t)row[qb] * a.o_ld + (int64_t)head[qb] * HD + db * 16 + 4 * g;
      *reinterpret_cast<uint2 *>(dst) = make_uint2(pack2<T>(o[0], o[1]), pack2<T>(o[2], o[3]));
    }
  }
}

template <typename T, int MODE, int QB>
static hipError_t run16(const AttnArgs &a, hipStream_t st) {
  constexpr int NW = 4, lds = 2 * 2 * 64 * 256;
  static_assert(lds <= 65536, "within the default limit, two workgroups per CU");
  hipLaunchKernelGGL((attn16_kernel<T, MODE, QB, NW>), dim3(a.n_items), dim3(64 * NW), lds, st, a);
  return hipGetLastError();
}

template <typename T, int MODE>
static hipError_t run16_block(const AttnArgs &a, hipStream_t st) {
  if (a.block == 64) return run16<T, MODE, 1>(a, st);
  if (a.block == 128) return run16<T, MODE, 2>(a, st);
  return hipErrorInvalidValue;
}

hipError_t launch_attn16(int dtype, const AttnArgs &a, hipStream_t st) {
  if (a.n_items <= 0) return hipSuccess;
  if (!attn16_ok(dtype, a.pair, a.hd)) return hipErrorInvalidValue;
  if (dtype == 0) return a.mode == 0 ? run16_block<bf16, 0>(a, st) : run16_block<bf16, 1>(a, st);
  return a.mode == 0 ? run16_block<f16, 0>(a, st) : run16_block<f16, 1>(a, st);
}

}  // namespace jetk
