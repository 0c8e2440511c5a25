// Dense FP16 decode attention, softmax(q K^T / sqrt d) V with FP32 accumulation:
// the O_dense the paper's Rung 3 / Rung 4 return (its "Fallback Ladder" section).
// One launch serves every KV group of a call (or the one group of a fallback) over FP16 K, V of
// [n_tokens][128], split over the sequence; a second kernel merges the splits and also rewrites
// the served heads' certificates.  With one split per group the first kernel finishes the rows
// itself and there is no second one.
#include <algorithm>

#include "cqa_internal.h"
#include "reduce_inl.h"

namespace cqa {

constexpr int DP_FLOATS = 4 + D;  // m (base 2), l, pad, pad, o[128]
constexpr int DENSE_WAVES = 8;    // waves per workgroup of the dense pass
constexpr int DENSE_WG_TARGET = 256;  // one workgroup of eight waves on each of the compute units
constexpr int PAGED_WG = 16;      // a paged KV group with fewer workgroups is attended by single waves
constexpr int DENSE_TILE = 32;    // tokens a wave takes per iteration
// ... when the ladder reads the pinned originals, where the host link is the bound and more requests in
// flight only make the workgroups' shares of it uneven.  One group of 131072 tokens: 8 tokens 1213 us,
// 32 tokens 1221, no prefetch 1270; two of 20000: 401, 447, 452; four or five of 32768: 1240 / 1565,
// 1249 / 1575, 1249 / 1548.
constexpr int LADDER_TILE = 8;
constexpr float M_EMPTY = -1.0e30f;   // running maximum of a state that has seen no token: finite, below every score

// Splits per KV group that the caller's workspace holds for a sequence of this length when one
// group of four heads is served at a time: what cqa_dense_workspace_bytes is sized by.
static int64_t dense_ws_units(int64_t n_tokens) {
  const int64_t tiles = (n_tokens + BLK - 1) / BLK;
  int64_t s = std::min<int64_t>((tiles + 7) / 8, 1024);
  const int64_t tps = (tiles + s - 1) / s;
  return (tiles + tps - 1) / tps;
}

int64_t dense_ws_floats(int group, int64_t n_tokens) {
  return (int64_t)group * dense_ws_units(n_tokens) * DP_FLOATS;
}

// Splits per KV group of a call that serves `groups` KV groups (a fallback, which may serve fewer
// of them, uses the geometry of its whole layer, so that its rows are bit-equal to the dense
// call's): one workgroup per compute unit over all groups, but at least a tile per wave, and no
// more than the workspace (sized for the groups one after the other) holds for all groups at
// once.  At most 256, which is what a cache's own workspace holds for one group at any length
// that allows so many.
static int dense_splits(int group, int64_t groups, int64_t n_tokens) {
  const int64_t tiles = (n_tokens + DENSE_TILE - 1) / DENSE_TILE;
  int64_t s = std::min<int64_t>(DENSE_WG_TARGET / std::min<int64_t>(groups, DENSE_WG_TARGET),
                                (tiles + DENSE_WAVES - 1) / DENSE_WAVES);
  s = std::min<int64_t>(s, 4 * dense_ws_units(n_tokens) / ((int64_t)group * groups));
  if (s < 1) s = 1;
  const int64_t tps = (tiles + s - 1) / s;
  return (int)((tiles + tps - 1) / tps);
}

template <bool NT>
__device__ __forceinline__ uint4 ld_dense(const char* p) {
  const u32x4_any* x = reinterpret_cast<const u32x4_any*>(p);
  const u32x4_any v = NT ? __builtin_nontemporal_load(x) : *x;
  return make_uint4(v.x, v.y, v.z, v.w);
}

template <int G, int W>
struct DenseSmem {
  float mo[W][G][D];
  float ms[W][G][2];
};

// Wave w of W attends its tiles of [t0, t1), dealt round-robin, of k, v ([n_tokens][128], device or
// mapped host memory) for G heads of one KV group, and leaves its state at mo [G][mo_stride] (the channels)
// and ms [G][ms_stride] (maximum in base 2, sum).  AHEAD: tiles whose loads are in flight.
// Bound by the memory stream.  Every load covers 1 KB of consecutive memory: a row of 16 lanes
// holds one token, a lane 8 channels of it, so a wave's four rows take tokens r, 4 + r, 8 + r, ...
// of a tile.  A score is 8 products per head and a row sum on DPP; after it every lane of the row
// holds the score, so the softmax state is kept per row and nothing goes through LDS before the
// end.  Registers are re-requested for the wave's next tile right after their last use: with tiles
// of 32 tokens 16 KB in flight per wave, 128 KB per compute unit.  Measured on 16 groups of 32775
// tokens, 268 MB, four heads per group: 46.4 us = 5.8 TB/s (plain loads, tiles of 32: 85 us with the
// reduction; the non-temporal hint: 49; one launch pair per group before: 2074).
template <int G, int W, int TILE, bool NT, int AHEAD = 1>
__device__ __forceinline__ void dense_wave_work(const __half* __restrict__ q, const __half* __restrict__ k,
                                                const __half* __restrict__ v, int64_t n_tokens, int64_t t0,
                                                int64_t t1, int w, float* mo, int mo_stride, float* ms, int ms_stride) {
  constexpr int T = TILE / 4;   // tokens per row and tile
  const int l = threadIdx.x & 63;
  const int c8 = l & 15, row = l >> 4;
  const float scale = 0.08838834764831845f * 1.4426950408889634f;   // 1 / sqrt(128), in base-2 units

  uint4 qr[G];
#pragma unroll
  for (int h = 0; h < G; ++h) qr[h] = ld16_any(q + h * D + c8 * 8);

  float m_run[G], l_run[G], acc[8][G];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    m_run[h] = M_EMPTY;
    l_run[h] = 0.0f;
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j][h] = 0.0f;
  }

  uint4 kr[AHEAD][T], vr[AHEAD][T];
  // address = the tile's wave-uniform base + a 32-bit lane offset; tokens past the end read the last
  // token's row, their scores are masked.  The request of a wave's last iteration is not used:
  // it is aimed at the first query row, in cache, and costs no memory traffic.
#define CQA_DENSE_LOAD(DST, SRC, TI, ON)                                                        \
  {                                                                                             \
    const char* base__ = reinterpret_cast<const char*>((ON) ? (SRC) + (TI) * (TILE * D) : q); \
    const int last__ = (ON) ? (int)min((int64_t)(TILE - 1), n_tokens - 1 - (TI) * TILE) : 0; \
    _Pragma("unroll") for (int i = 0; i < T; ++i)                                               \
      DST[i] = ld_dense<NT>(base__ + (uint32_t)(min(i * 4 + row, last__) * (D * 2) + c8 * 16)); \
  }
  int64_t tile = t0 + __builtin_amdgcn_readfirstlane(w);
#pragma unroll
  for (int u = 0; u < AHEAD; ++u)
    if (tile + u * W < t1) {
      CQA_DENSE_LOAD(kr[u], k, tile + u * W, true)
      CQA_DENSE_LOAD(vr[u], v, tile + u * W, true)
    }
  while (tile < t1) {
#pragma unroll
    for (int u = 0; u < AHEAD; ++u, tile += W) {
      if (u > 0 && tile >= t1) break;
      const int64_t nxt = tile + AHEAD * W;
      const int live = (int)min((int64_t)TILE, n_tokens - tile * TILE);
      float s[T][G];
#pragma unroll
      for (int i = 0; i < T; ++i) {
        const __half2* kh = reinterpret_cast<const __half2*>(&kr[u][i]);
#pragma unroll
        for (int h = 0; h < G; ++h) {
          const __half2* qh = reinterpret_cast<const __half2*>(&qr[h]);
          float d = 0.0f;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            d = fmaf(__low2float(qh[j]), __low2float(kh[j]), d);
            d = fmaf(__high2float(qh[j]), __high2float(kh[j]), d);
          }
          s[i][h] = d;
        }
      }
      CQA_DENSE_LOAD(kr[u], k, nxt, nxt < t1)
#pragma unroll
      for (int h = 0; h < G; ++h) {
        float m_new = m_run[h];
#pragma unroll
        for (int i = 0; i < T; ++i) {
          const float sum16 = row_sum(s[i][h]);
          s[i][h] = i * 4 + row < live ? sum16 * scale : -INFINITY;
          m_new = fmaxf(m_new, s[i][h]);
        }
        const float alpha = __builtin_amdgcn_exp2f(m_run[h] - m_new);
        float sum = 0.0f;
#pragma unroll
        for (int i = 0; i < T; ++i) {
          s[i][h] = __builtin_amdgcn_exp2f(s[i][h] - m_new);
          sum += s[i][h];
        }
        l_run[h] = fmaf(l_run[h], alpha, sum);
        m_run[h] = m_new;
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j][h] *= alpha;
      }
      // 16 tokens at a time: where none of them exists nothing is added, not zero weights times the last token's
      // value, which may be infinite
#pragma unroll
      for (int i0 = 0; i0 < T; i0 += 4) {
        if (i0 > 0 && i0 * 4 >= live) break;
#pragma unroll
        for (int i = i0; i < i0 + 4 && i < T; ++i) {
          const __half2* vh = reinterpret_cast<const __half2*>(&vr[u][i]);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float v0 = __low2float(vh[j]), v1 = __high2float(vh[j]);
#pragma unroll
            for (int h = 0; h < G; ++h) {
              acc[2 * j][h] = fmaf(s[i][h], v0, acc[2 * j][h]);
              acc[2 * j + 1][h] = fmaf(s[i][h], v1, acc[2 * j + 1][h]);
            }
          }
        }
      }
      CQA_DENSE_LOAD(vr[u], v, nxt, nxt < t1)
    }
  }
#undef CQA_DENSE_LOAD

  // merge the wave's four rows
#pragma unroll
  for (int h = 0; h < G; ++h) {
    const float M = max_x32(max_x16(m_run[h]));
    const float f = __builtin_amdgcn_exp2f(m_run[h] - M);
    const float L = sum_x32(sum_x16(l_run[h] * f));
    float x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = sum_x32(sum_x16(acc[j][h] * f));
    if (row == 0) {
      *reinterpret_cast<float4*>(&mo[h * mo_stride + c8 * 8]) = make_float4(x[0], x[1], x[2], x[3]);
      *reinterpret_cast<float4*>(&mo[h * mo_stride + c8 * 8 + 4]) = make_float4(x[4], x[5], x[6], x[7]);
      ms[h * ms_stride] = M;
      ms[h * ms_stride + 1] = L;
    }
  }
}

// The W waves of a workgroup attend tiles [t0, t1) for the G heads of one KV group; on return (after a
// workgroup barrier) each wave's state is in LDS.
template <int G, int W, int TILE, bool NT>
__device__ __forceinline__ void dense_split_work(const __half* __restrict__ q, const __half* __restrict__ k,
                                                 const __half* __restrict__ v, int64_t n_tokens, int64_t t0,
                                                 int64_t t1, DenseSmem<G, W>& sm) {
  const int w = threadIdx.x >> 6;
  dense_wave_work<G, W, TILE, NT>(q, k, v, n_tokens, t0, t1, w, sm.mo[w][0], D, sm.ms[w][0], 2);
  __syncthreads();
}

// (m, l, o) of one channel over the waves of a split
template <int W>
__device__ __forceinline__ void dense_wave_merge(const float (&m)[W], const float (&l)[W], const float (&x)[W], float& M,
                                                 float& L, float& o) {
  M = m[0];
#pragma unroll
  for (int w = 1; w < W; ++w) M = fmaxf(M, m[w]);
  L = 0.0f;
  o = 0.0f;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    const float f = __builtin_amdgcn_exp2f(m[w] - M);
    L = fmaf(f, l[w], L);
    o = fmaf(f, x[w], o);
  }
}
// ... of head h, channel c over the workgroup's waves, from LDS
template <int G, int W>
__device__ __forceinline__ void dense_wg_merge(const DenseSmem<G, W>& sm, int h, int c, float& M, float& L, float& o) {
  float m[W], l[W], x[W];
#pragma unroll
  for (int w = 0; w < W; ++w) {
    m[w] = sm.ms[w][h][0];
    l[w] = sm.ms[w][h][1];
    x[w] = sm.mo[w][h][c];
  }
  dense_wave_merge<W>(m, l, x, M, L, o);
}

// this workgroup's partial sets: ws[h][split]
template <int G, int W>
__device__ __forceinline__ void dense_store_partials(const DenseSmem<G, W>& sm, float* ws, int nsplit, int split) {
  for (int idx = threadIdx.x; idx < G * D; idx += 64 * W) {
    const int h = idx / D, c = idx % D;
    float M, L, o;
    dense_wg_merge<G, W>(sm, h, c, M, L, o);
    float* p = ws + ((int64_t)h * nsplit + split) * DP_FLOATS;
    p[4 + c] = o;
    if (c == 0) {
      p[0] = M;
      p[1] = L;
    }
  }
}

// Output channel c of one row over its `nsplit` partial sets.  All threads of a wave work on the
// same row; the loads of eight sets are in flight at a time.
__device__ __forceinline__ float dense_merge_row(const float* part, int nsplit, int c) {
  float M = M_EMPTY;
  for (int s = 0; s < nsplit; s += 64) M = fmaxf(M, part[(int64_t)min(s + (int)(threadIdx.x & 63), nsplit - 1) * DP_FLOATS]);
  M = wave_max(M);
  float L = 0.0f, o = 0.0f;
  for (int s0 = 0; s0 < nsplit; s0 += 8) {
    float m[8], l[8], x[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float* p = part + (int64_t)min(s0 + i, nsplit - 1) * DP_FLOATS;
      m[i] = p[0];
      l[i] = p[1];
      x[i] = p[4 + c];
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const bool in = s0 + i < nsplit;
      const float f = in ? __builtin_amdgcn_exp2f(m[i] - M) : 0.0f;
      L = fmaf(f, l[i], L);
      o = fmaf(f, in ? x[i] : 0.0f, o);   // (the last set's sum may be infinite)
    }
  }
  return o / L;
}

// ... where the waves of a split have left their states one by one (dense_paged_kernel): nsplit * DENSE_WAVES sets
__device__ __forceinline__ float dense_merge_row_of_waves(const float* part, int nsplit, int c) {
  float M = M_EMPTY;
  const int sets = nsplit * DENSE_WAVES;
  for (int s = 0; s < sets; s += 64) M = fmaxf(M, part[(int64_t)min(s + (int)(threadIdx.x & 63), sets - 1) * DP_FLOATS]);
  M = wave_max(M);
  float L = 0.0f, o = 0.0f;
  for (int s = 0; s < nsplit; ++s, part += DENSE_WAVES * DP_FLOATS) {
    float m[DENSE_WAVES], l[DENSE_WAVES], x[DENSE_WAVES], Ms, Ls, os;
#pragma unroll
    for (int w = 0; w < DENSE_WAVES; ++w) {
      m[w] = part[w * DP_FLOATS];
      l[w] = part[w * DP_FLOATS + 1];
      x[w] = part[w * DP_FLOATS + 4 + c];
    }
    dense_wave_merge<DENSE_WAVES>(m, l, x, Ms, Ls, os);
    const float f = __builtin_amdgcn_exp2f(Ms - M);
    L = fmaf(f, Ls, L);
    o = fmaf(f, os, o);
  }
  return o / L;
}

__device__ __forceinline__ void dense_mark_served(cqa_head_cert* cert, uint32_t* flags, int64_t row, int rung) {
  if (cert != nullptr) {
    cert[row].E_key = 0.0f;
    cert[row].E_val = 0.0f;
    cert[row].served_rung = rung;
  }
  if (flags != nullptr) flags[row] = (flags[row] & ~(7u << CQA_RUNG_SHIFT)) | ((uint32_t)rung << CQA_RUNG_SHIFT);
}

struct DenseArgs {
  const __half* q;          // [groups][G][128]
  const __half* k;          // [groups][n_tokens][128]
  const __half* v;
  int64_t n_tokens;
  int nsplit, tiles_per_split;
  int by_wave;              // 1: the partial sets are those of the single waves, nsplit * DENSE_WAVES of them
  int units;                // KV groups, or parts of them (below)
  int per_group;            // parts, of G heads each, that a KV group's heads are served in
  float* ws;                // [groups][G][partial sets][DP_FLOATS], unused with one
  float* O;                 // [groups][G][128]
  const uint32_t* select;   // [groups][G] or null = all: rows that are written
  cqa_head_cert* cert;      // or null
  uint32_t* flags;          // or null
  int rung;
};

// SPREAD: the heads of a KV group are served in parts, each by workgroups of its own, where a workgroup per group and split would
// leave half of the chip or more idle: the caller's workspace allows few splits then (it is sized for one group at a time), and
// the vector ALU of the few compute units is the bound.  The parts of one (group, split) lie eight workgroups apart, so on one die
// as a rule, and read the same keys and values from its cache, without the non-temporal hint.  A head's arithmetic
// does not depend on the part it is in.  8 KV heads x 4: 200 tokens 7.8 -> 5.1 us, 1000 18.2 -> 7.9, 4000 21.7 -> 11.2; 16 x 4 of 4000
// 35.6 -> 16.2, of 16000 (in halves) 40.3 -> 32.0; 32 x 2 of 4000 26.6 -> 17.6.
template <int G, bool SPREAD>
__global__ __launch_bounds__(64 * DENSE_WAVES, 2) void dense_split_kernel(DenseArgs a) {
  __shared__ __align__(16) DenseSmem<G, DENSE_WAVES> sm;
  int64_t grp = blockIdx.x / a.nsplit, kv = grp;   // grp: the unit
  int split = (int)(blockIdx.x - grp * a.nsplit);
  if (SPREAD) {
    const int eight = (int)blockIdx.x >> 3, part = eight % a.per_group;
    const int item = (eight / a.per_group) * 8 + ((int)blockIdx.x & 7);
    kv = item / a.nsplit;
    split = item - (int)kv * a.nsplit;
    grp = kv * a.per_group + part;
    if (grp >= a.units) return;
  }
  const int64_t tiles = (a.n_tokens + DENSE_TILE - 1) / DENSE_TILE;
  const int64_t t0 = (int64_t)split * a.tiles_per_split;
  const int64_t t1 = min(t0 + (int64_t)a.tiles_per_split, tiles);
  dense_split_work<G, DENSE_WAVES, DENSE_TILE, !SPREAD>(a.q + grp * G * D, a.k + kv * a.n_tokens * D, a.v + kv * a.n_tokens * D,
                                   a.n_tokens, t0, t1, sm);
  if (a.nsplit > 1) {
    dense_store_partials<G, DENSE_WAVES>(sm, a.ws + grp * G * a.nsplit * DP_FLOATS, a.nsplit, split);
    return;
  }
  for (int idx = threadIdx.x; idx < G * D; idx += 64 * DENSE_WAVES) {
    const int h = idx / D, c = idx % D;
    const int64_t row = grp * G + h;
    if (a.select != nullptr && a.select[row] == 0) continue;
    float M, L, o;
    dense_wg_merge<G, DENSE_WAVES>(sm, h, c, M, L, o);
    a.O[row * D + c] = o / L;
    if (c == 0) dense_mark_served(a.cert, a.flags, row, a.rung);
  }
}

// One paged KV group of a layer that has many: the dense call gives such a group fewer than PAGED_WG workgroups, often
// one, but here it is alone on the chip.  Every (split, wave, head) is a workgroup of one wave, so the group spreads
// over 8 x heads as many compute units; the arithmetic of a head is that of dense_split_kernel, and
// dense_merge_row_of_waves merges in the same order, so the rows are bit-equal to the dense call's.
// Bound by the chain of a wave's tiles: 0.8 us each with two requested ahead, 1.05 with one.
// One group of 32768 tokens in a layer of 136 or more groups: this kernel and the merge 116 us against 452 for one
// workgroup; the fallback call with its copies (295) 812 -> 470 us.
__global__ __launch_bounds__(64) void dense_paged_kernel(DenseArgs a) {
  const int h = blockIdx.y, unit = blockIdx.x;   // unit = split * DENSE_WAVES + wave
  if (a.select != nullptr && a.select[h] == 0) return;
  const int split = unit / DENSE_WAVES;
  const int64_t tiles = (a.n_tokens + DENSE_TILE - 1) / DENSE_TILE;
  const int64_t t0 = (int64_t)split * a.tiles_per_split;
  const int64_t t1 = min(t0 + (int64_t)a.tiles_per_split, tiles);
  float* p = a.ws + ((int64_t)h * a.nsplit * DENSE_WAVES + unit) * DP_FLOATS;
  dense_wave_work<1, DENSE_WAVES, DENSE_TILE, false, 2>(a.q + h * D, a.k, a.v, a.n_tokens, t0, t1, unit % DENSE_WAVES, p + 4, 0, p, 0);
}

// One workgroup of 128 threads per row.  (Before: one thread per channel walked all splits twice,
// one load in flight: 112 us for 256 splits of one group, which made it 16 times 125 us for the
// 268 MB call.)
__global__ __launch_bounds__(128) void dense_reduce_kernel(DenseArgs a) {
  const int64_t row = blockIdx.x;
  if (a.select != nullptr && a.select[row] == 0) return;
  const int c = threadIdx.x;
  a.O[row * D + c] = a.by_wave ? dense_merge_row_of_waves(a.ws + row * a.nsplit * DENSE_WAVES * DP_FLOATS, a.nsplit, c)
                               : dense_merge_row(a.ws + row * a.nsplit * DP_FLOATS, a.nsplit, c);
  if (c == 0) dense_mark_served(a.cert, a.flags, row, a.rung);
}

// The (KV group, split) items of the groups that a rung serves, walked by the first `walkers` of the launch's workgroups
// of W waves.
// flagged(row): whether a row asked for the fallback (uniform in the wave).  mark: also rewrite the
// served rows' certificates and rung bits.
template <int G, int W, typename F>
__device__ __forceinline__ void ladder_serve(const LadderArgs& a, int rung, int walkers, F flagged, bool mark,
                                             DenseSmem<G, W>& sm) {
  __shared__ int s_last;
  const int64_t items = (int64_t)a.groups * a.nsplit;
  if ((int)blockIdx.x >= walkers) return;
  for (int64_t item = blockIdx.x; item < items; item += walkers) {
    const int64_t grp = item / a.nsplit;
    const int split = (int)(item - grp * a.nsplit);
    const int64_t row0 = grp * G;
    bool mine = rung == 4;
    for (int h = 0; h < G && !mine; ++h) mine = flagged(row0 + h);
    if (!mine) continue;   // uniform over the workgroup
    float* ws = a.ws + row0 * a.nsplit * DP_FLOATS;
    const int64_t t0 = (int64_t)split * a.tiles_per_split;
    const int64_t t1 = min(t0 + (int64_t)a.tiles_per_split, (a.n_tokens + LADDER_TILE - 1) / LADDER_TILE);
    __syncthreads();       // the previous item's LDS has been read
    dense_split_work<G, W, LADDER_TILE, false>(a.q + row0 * D, a.t2_k + grp * a.max_tokens * D,
                                               a.t2_v + grp * a.max_tokens * D, a.n_tokens, t0, t1, sm);
    dense_store_partials<G, W>(sm, ws, a.nsplit, split);
    // every thread publishes its partial stores device-wide before the workgroup draws its ticket
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t* tk = a.tickets + grp;
      const uint32_t t = __hip_atomic_fetch_add(tk, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const bool last = t == (uint32_t)a.nsplit - 1u;
      if (last) __hip_atomic_store(tk, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // next launch
      s_last = last ? 1 : 0;
    }
    __syncthreads();
    if (s_last == 0) continue;
    __threadfence();
    for (int idx = threadIdx.x; idx < G * D; idx += 64 * W) {
      const int h = idx / D, c = idx % D;
      const int64_t row = row0 + h;
      if (rung != 4 && !flagged(row)) continue;   // Rung 3 serves flagged heads only
      // (a wave's 64 channels belong to one row, so the branch above is uniform in the wave)
      a.O[row * D + c] = dense_merge_row(ws + (int64_t)h * a.nsplit * DP_FLOATS, a.nsplit, c);
      if (mark && c == 0) dense_mark_served(a.cert, a.flags, row, rung);
    }
  }
}

static_assert(sizeof(LadderArgs) % 8 == 0 && alignof(ReduceArgs) == 8, "the second argument follows the first");

// The fallback ladder resolved on the device (the paper's "Fallback Ladder": Rung 3 returns the
// dense FP16 result for the flagged heads, Rung 4 for every head of the layer-step).  Launched
// behind the reduction on every step.  The reduction leaves the step's number in `raised` when it
// flags a head; without it every workgroup leaves at once (one word instead of all flag words:
// 2.5 -> 1.6 us at 8K, 7.3 -> 5.7 us with 64 x 8 KV groups).  Otherwise every workgroup reads the step's flag words and takes the ladder decision itself -- no head flagged: nothing to do;
// a PRECOND flag anywhere, or at least rung4_min_groups (> 0) flagged KV groups: all groups
// are served (Rung 4); else the flagged groups (Rung 3) -- and walks the (KV group, split) items of the
// served groups.  An item attends a run of the group's FP16 originals
// straight from the pinned host arrays (the device reads host memory over the link: no copy
// call, no staging buffer, no host decision), and the last of a group's items to arrive merges the
// splits and rewrites O, the certificate and the rung bits of the heads that are served.
// Behind a split pass that reduces the rows itself every wave also looks at the numbers that it left.  Where one is not
// this step's, every workgroup reduces all rows, to know every flag without waiting for another one, and the
// first one writes them, leaving out the outputs that a rung replaces.  That is for once: a step of 32 rows takes 47 us instead of 10 so, of 256
// 266 instead of 15, of 512 516 instead of 15, so the first workgroup also tells the host, whose later steps reduce in a launch
// of their own (a recorded step goes on as it was recorded).
// Leaving is what nearly every launch does, so no more than the first line of the arguments is read up to there (with all of
// them first, 0.6 us more for a step of 64 x 4 heads, 2000 tokens).
template <int G, typename... RA>
__global__ __launch_bounds__(256) void dense_ladder_kernel(LadderArgs first, RA...) {
  constexpr bool CHECK = sizeof...(RA) > 0;
  bool strayed = false;
  asm volatile("" ::"s"(first.raised), "s"(first.raised_tag), "s"(first.groups), "s"(first.split_tickets));   // one wait
  int zero = 0;   // (a vector load, under way together with the others: a scalar one would be waited for ahead of them)
  if constexpr (CHECK) asm volatile("" : "+v"(zero));
  const uint32_t raised = first.raised[zero];
  if constexpr (CHECK) {
    const uint32_t* const reduced = first.split_tickets + (int64_t)first.groups * TICKET_STRIDE;
    for (int g = threadIdx.x & 63; g < first.groups; g += 64) strayed = strayed | (reduced[g] != first.raised_tag);
    strayed = __any(strayed);
  }
  if (!__any(raised == first.raised_tag) && !strayed) return;
  const LadderArgs a = arg_read_here<LadderArgs>(0);
  __shared__ int s_rung, s_walkers;
  __shared__ int s_cnt[4], s_pre[4];
  __shared__ uint32_t s_flags[CHECK ? REDUCED_ROWS : 1];   // of rows reduced here
  if constexpr (CHECK) {
    if (strayed) {
      const ReduceArgs ra = arg_read_here<ReduceArgs>(sizeof(LadderArgs));
      for (int r = threadIdx.x >> 6; r < a.n_rows; r += 4) {
        const HeadRow row = reduce_row_wave(ra, r);
        if ((threadIdx.x & 63) == 0) s_flags[r] = row.fl;
      }
      if (blockIdx.x == 0) {
        for (int i = threadIdx.x; i < a.groups * DIES; i += 256)
          a.split_tickets[(int64_t)(i / DIES) * TICKET_STRIDE + i % DIES] = 0u;
        if (threadIdx.x == 0) __hip_atomic_store(a.strayed, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      }
      __syncthreads();
    }
  }
  const auto flag_of = [&](int64_t r) { return CHECK && strayed ? s_flags[r] : a.flags[r]; };
  {
    // each wave takes every fourth chunk of 64 flag words (a group's heads never straddle a
    // chunk: G divides 64), four chunks per trip with all loads issued first
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    int flagged_groups = 0;
    bool precond = false;
    for (int base = 0; base < a.n_rows; base += 1024) {
      uint32_t f[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i = base + (j * 4 + w) * 64 + l;
        f[j] = i < a.n_rows ? flag_of(i) : 0u;
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint64_t m = __ballot((f[j] & CQA_FLAG_ANY) != 0u);
        precond = precond || __ballot((f[j] & CQA_FLAG_PRECOND) != 0u) != 0ull;
        uint64_t gm = m;
#pragma unroll
        for (int jj = 1; jj < G; ++jj) gm |= m >> jj;
        gm &= G == 1 ? ~0ull : (G == 2 ? 0x5555555555555555ull : 0x1111111111111111ull);
        flagged_groups += __popcll(gm);
      }
    }
    if (l == 0) {
      s_cnt[w] = flagged_groups;
      s_pre[w] = precond ? 1 : 0;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      const int cnt = s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3];
      const bool pre = (s_pre[0] | s_pre[1] | s_pre[2] | s_pre[3]) != 0;
      int rung = cnt > 0 ? 3 : 0;
      if (rung != 0 && (pre || (a.rung4_min_groups > 0 && cnt >= a.rung4_min_groups))) rung = 4;
      s_rung = rung;
      // Few items: a workgroup each, wherever they lie in the layer.  Many: the link is kept busy by fewer workgroups,
      // each with its own run of tokens to read, and runs better on fewer runs at a time.  Layers of 264 groups of 500
      // tokens, 320 of 300 and 512 of 1000, all served, on 512 workgroups and on 128: 1447 -> 1321, 1301 -> 987 and
      // 5451 -> 4853 us (a workgroup per item: 1427, 1133, 5191).  128 items on 128 as well: 333 -> 362.
      s_walkers = (int64_t)(rung == 4 ? a.groups : cnt) * a.nsplit > a.many_items ? min((int)gridDim.x, a.many_walkers)
                                                                                 : (int)gridDim.x;
      if (rung != 0 && blockIdx.x == 0) atomicAdd(a.counts + (rung - 3), 1u);
    }
  }
  __syncthreads();
  const int rung = s_rung;
  if constexpr (CHECK) {
    for (int r = threadIdx.x >> 6; r < (strayed && blockIdx.x == 0 ? a.n_rows : 0); r += 4) {
      HeadRow row = reduce_row_wave(arg_read_here<ReduceArgs>(sizeof(LadderArgs)), r);
      if (rung == 4 || (rung == 3 && (row.fl & CQA_FLAG_ANY) != 0u)) {
        row.ct.E_key = 0.0f;
        row.ct.E_val = 0.0f;
        row.ct.served_rung = rung;
        row.fl = (row.fl & ~(7u << CQA_RUNG_SHIFT)) | ((uint32_t)rung << CQA_RUNG_SHIFT);
      } else {
        reinterpret_cast<float2*>(a.O + (int64_t)r * D)[threadIdx.x & 63] = row.out;
      }
      if ((threadIdx.x & 63) == 0) {
        a.cert[r] = row.ct;
        a.flags[r] = row.fl;
      }
    }
  }
  if (rung == 0) return;

  __shared__ __align__(16) DenseSmem<G, 4> sm;
  // (the rung bits that a finished group's rows get do not touch the bits looked at here)
  ladder_serve<G, 4>(a, rung, s_walkers, [&](int64_t row) { return (flag_of(row) & CQA_FLAG_ANY) != 0u; }, !strayed, sm);
}

// Reduction and ladder of a short step of few rows (ladder_reduces) in one launch: every workgroup merges all rows, one per
// wave, and so knows every flag without waiting for another one; the first one writes the rows, leaving out the outputs that a
// rung replaces, and the others leave unless a head asks for a fallback.  A step in two launches and in one:
// 4 rows 12.4, 10.5 us at 3 sets and 11.8, 10.9 at 8; 8 rows of 8 KV heads 13.3, 12.3 at 3 and 13.0, 12.4 at 8, of
// 2 KV heads level (11.9, 12.0; 12.1, 12.1).  (32 rows, two per wave of 16, with an earlier merge: 13 -> 23 us, the workgroups'
// copies of the work get in each other's way.)
template <int G>
__global__ __launch_bounds__(64 * FINISH_ROWS) void finish_ladder_kernel(ReduceArgs ra, LadderArgs a) {
  const int r = threadIdx.x >> 6, l = threadIdx.x & 63;   // this wave's row
  __shared__ uint32_t s_fl[FINISH_ROWS];
  HeadRow row;
  row.fl = 0u;
  if (r < a.n_rows) row = reduce_row_wave(ra, r);
  if (l == 0) s_fl[r] = row.fl;
  __syncthreads();
  const uint32_t f = l < FINISH_ROWS ? s_fl[l] : 0u;
  const uint32_t any = (uint32_t)__ballot((f & CQA_FLAG_ANY) != 0u);       // bit i: row i
  const bool pre = __ballot((f & CQA_FLAG_PRECOND) != 0u) != 0ull;
  uint32_t gm = any;
#pragma unroll
  for (int jj = 1; jj < G; ++jj) gm |= any >> jj;
  gm &= G == 1 ? ~0u : (G == 2 ? 0x55555555u : 0x11111111u);
  const int cnt = __popc(gm);
  int rung = cnt > 0 ? 3 : 0;
  if (rung != 0 && (pre || (a.rung4_min_groups > 0 && cnt >= a.rung4_min_groups))) rung = 4;
  if (blockIdx.x == 0 && r < a.n_rows) {
    if (rung == 4 || (rung == 3 && ((any >> r) & 1u) != 0u)) {
      row.ct.E_key = 0.0f;
      row.ct.E_val = 0.0f;
      row.ct.served_rung = rung;
      row.fl = (row.fl & ~(7u << CQA_RUNG_SHIFT)) | ((uint32_t)rung << CQA_RUNG_SHIFT);
    } else {
      reinterpret_cast<float2*>(a.O + (int64_t)r * D)[l] = row.out;
    }
    if (l == 0) {
      a.cert[r] = row.ct;
      a.flags[r] = row.fl;
    }
    if (rung != 0 && threadIdx.x == 0) atomicAdd(a.counts + (rung - 3), 1u);
  }
  if (rung == 0) return;
  __shared__ __align__(16) DenseSmem<G, FINISH_ROWS> sm;
  ladder_serve<G, FINISH_ROWS>(a, rung, (int)gridDim.x, [&](int64_t i) { return ((any >> (int)i) & 1u) != 0u; }, false, sm);
}

int ladder_splits(const Cache* c, int64_t n_tokens) {
  const int64_t groups = (int64_t)c->desc.batch * c->desc.n_kv_heads;
  int64_t want = (2 * (int64_t)c->n_cu) / groups;   // the launch's cost does not depend on it
  if (want < 4) want = 4;
  if (want > LADDER_MAX_SPLITS) want = LADDER_MAX_SPLITS;
  const int64_t tiles = (n_tokens + LADDER_TILE - 1) / LADDER_TILE;
  if (want > tiles) want = tiles;
  const int64_t tps = (tiles + want - 1) / want;
  return (int)((tiles + tps - 1) / tps);
}

int64_t ladder_ws_floats(int64_t rows) { return rows * LADDER_MAX_SPLITS * DP_FLOATS; }

int32_t launch_dense_ladder(Cache* c, int layer, const __half* q, int rung4_min_groups, float* O,
                            cqa_head_cert* cert, uint32_t* flags, uint32_t raised_tag, hipStream_t st,
                            RowsBy by, const ReduceArgs* reduce) {
  if (c->desc.tier2_mode != CQA_TIER2_PINNED) return CQA_ERR_NO_TIER2;
  const int64_t len = c->length[layer];
  if (len <= 0 || q == nullptr || O == nullptr || cert == nullptr || flags == nullptr)
    return CQA_ERR_INVALID_ARG;
  const int bt = c->desc.batch, hq = c->desc.n_q_heads, hkv = c->desc.n_kv_heads;
  const int g = hq / hkv;
  const int64_t layer_head0 = (int64_t)layer * bt * hkv;
  LadderArgs a{};
  a.q = q;
  a.t2_k = c->t2_k + layer_head0 * c->desc.max_tokens * D;
  a.t2_v = c->t2_v + layer_head0 * c->desc.max_tokens * D;
  a.max_tokens = c->desc.max_tokens;
  a.n_tokens = len;
  a.n_rows = bt * hq;
  a.nsplit = ladder_splits(c, len);
  const int64_t tiles = (len + LADDER_TILE - 1) / LADDER_TILE;
  a.tiles_per_split = (int)((tiles + a.nsplit - 1) / a.nsplit);
  a.rung4_min_groups = rung4_min_groups;
  a.ws = c->ladder_ws;
  a.tickets = c->ladder_tickets;
  a.counts = c->ladder_counts;
  a.raised = ladder_raised(c);
  a.raised_tag = raised_tag;
  a.groups = bt * hkv;
  a.many_items = c->n_cu;
  a.many_walkers = std::max(c->n_cu / 2, 1);
  a.O = O;
  a.cert = cert;
  a.flags = flags;
  const dim3 grid((unsigned)std::min<int64_t>((int64_t)a.nsplit * a.groups, 2 * (int64_t)c->n_cu));
  if (by == RowsBy::ladder) {
    // Each of the workgroups merges the rows: no more of them than keep the host link busy when a rung serves.  Eight
    // groups of one head, all served, on 64, 128, 256 and 512 workgroups: 600 tokens 121, 111, 116, 119 us, 1100
    // tokens 165, 146, 162, 188, 2000 tokens 242, 250, 277, 278 (without a flag all four take 13.1 - 14.2; 512 16).
    const dim3 fgrid((unsigned)std::min<int64_t>((int64_t)a.nsplit * a.groups, std::max(c->n_cu / 2, 1)));
    switch (g) {
      case 1: hipLaunchKernelGGL(finish_ladder_kernel<1>, fgrid, dim3(64 * FINISH_ROWS), 0, st, *reduce, a); break;
      case 2: hipLaunchKernelGGL(finish_ladder_kernel<2>, fgrid, dim3(64 * FINISH_ROWS), 0, st, *reduce, a); break;
      case 4: hipLaunchKernelGGL(finish_ladder_kernel<4>, fgrid, dim3(64 * FINISH_ROWS), 0, st, *reduce, a); break;
      default: return CQA_ERR_UNSUPPORTED;
    }
  } else if (by == RowsBy::split) {
    a.split_tickets = c->split_tickets;
    a.strayed = c->strayed;
    switch (g) {
      case 1: hipLaunchKernelGGL((dense_ladder_kernel<1, ReduceArgs>), grid, dim3(256), 0, st, a, *reduce); break;
      case 2: hipLaunchKernelGGL((dense_ladder_kernel<2, ReduceArgs>), grid, dim3(256), 0, st, a, *reduce); break;
      case 4: hipLaunchKernelGGL((dense_ladder_kernel<4, ReduceArgs>), grid, dim3(256), 0, st, a, *reduce); break;
      default: return CQA_ERR_UNSUPPORTED;
    }
  } else {
    switch (g) {
      case 1: hipLaunchKernelGGL(dense_ladder_kernel<1>, grid, dim3(256), 0, st, a); break;
      case 2: hipLaunchKernelGGL(dense_ladder_kernel<2>, grid, dim3(256), 0, st, a); break;
      case 4: hipLaunchKernelGGL(dense_ladder_kernel<4>, grid, dim3(256), 0, st, a); break;
      default: return CQA_ERR_UNSUPPORTED;
    }
  }
  CQA_HIP(hipGetLastError());
  return CQA_OK;
}

int32_t launch_dense(const __half* q, const __half* k, const __half* v, int group, int64_t groups,
                     int64_t layer_groups, int64_t n_tokens, float* O, const uint32_t* select, cqa_head_cert* cert,
                     uint32_t* flags, int rung, float* ws, hipStream_t st) {
  if (n_tokens <= 0 || groups <= 0) return CQA_ERR_INVALID_ARG;
  if (group != 1 && group != 2 && group != 4) return CQA_ERR_UNSUPPORTED;   // the kernels and the parts below are for these
  const int64_t tiles = (n_tokens + DENSE_TILE - 1) / DENSE_TILE;
  DenseArgs a{};
  a.q = q;
  a.k = k;
  a.v = v;
  a.n_tokens = n_tokens;
  a.nsplit = dense_splits(group, layer_groups, n_tokens);
  a.tiles_per_split = (int)((tiles + a.nsplit - 1) / a.nsplit);
  a.ws = ws;
  a.O = O;
  a.select = select;
  a.cert = cert;
  a.flags = flags;
  a.rung = rung;
  // by single waves: where a workgroup per split would leave most of the chip idle, it has more than a tile per wave to
  // do, and the workspace of one group (dense_ws_units sets per head) holds the waves' states.  One group of 32768
  // tokens with its copies, a workgroup per split and by waves: 4 splits 470, 383 us; 2 582, 410; 1 812, 470 (16
  // splits, a workgroup each: 385).  4107 tokens, every group of 32: 77 -> 70 us a group.
  a.by_wave = groups == 1 && a.nsplit < PAGED_WG && a.tiles_per_split > DENSE_WAVES &&
              a.nsplit * DENSE_WAVES <= dense_ws_units(n_tokens);
  if (a.by_wave) {
    hipLaunchKernelGGL(dense_paged_kernel, dim3((unsigned)(a.nsplit * DENSE_WAVES), (unsigned)group), dim3(64), 0, st, a);
  } else {
    // a grid dimension holds fewer than 2^32 threads: 8388607 workgroups a launch (as many KV groups: with so many of
    // them a group is one workgroup, which finishes its rows)
    int part = group;            // heads per workgroup: halved while twice the workgroups are still one to a compute unit
    while (part > 1 && groups * a.nsplit * (group / part) * 2 <= DENSE_WG_TARGET) part /= 2;
    if (part < group) {
      a.per_group = group / part;
      a.units = (int)groups * a.per_group;
      const dim3 grid((unsigned)((groups * a.nsplit + 7) / 8 * 8 * a.per_group));
      if (part == 1)
        hipLaunchKernelGGL((dense_split_kernel<1, true>), grid, dim3(64 * DENSE_WAVES), 0, st, a);
      else
        hipLaunchKernelGGL((dense_split_kernel<2, true>), grid, dim3(64 * DENSE_WAVES), 0, st, a);
    }
    const int64_t most = 0xFFFFFFFFll / (64 * DENSE_WAVES * a.nsplit);
    for (int64_t g0 = part < group ? groups : 0; g0 < groups; g0 += most) {
      DenseArgs chunk = a;
      chunk.q += g0 * group * D;
      chunk.k += g0 * n_tokens * D;
      chunk.v += g0 * n_tokens * D;
      chunk.O += g0 * group * D;
      if (chunk.select != nullptr) chunk.select += g0 * group;
      if (chunk.cert != nullptr) chunk.cert += g0 * group;
      if (chunk.flags != nullptr) chunk.flags += g0 * group;
      if (a.nsplit > 1) chunk.ws += g0 * group * a.nsplit * DP_FLOATS;
      const dim3 grid((unsigned)(std::min(most, groups - g0) * a.nsplit));
      switch (group) {
        case 1: hipLaunchKernelGGL((dense_split_kernel<1, false>), grid, dim3(64 * DENSE_WAVES), 0, st, chunk); break;
        case 2: hipLaunchKernelGGL((dense_split_kernel<2, false>), grid, dim3(64 * DENSE_WAVES), 0, st, chunk); break;
        default: hipLaunchKernelGGL((dense_split_kernel<4, false>), grid, dim3(64 * DENSE_WAVES), 0, st, chunk); break;
      }
    }
  }
  CQA_HIP(hipGetLastError());
  if (a.nsplit > 1 || a.by_wave) {
    hipLaunchKernelGGL(dense_reduce_kernel, dim3((unsigned)(groups * group)), dim3(128), 0, st, a);
    CQA_HIP(hipGetLastError());
  }
  return CQA_OK;
}

}  // namespace cqa
