// Cross-split reduction of one (batch, query head).  Two forms: reduce_row, by a workgroup of three to ten waves with a
// barrier (every wave calls it, the first gets the row), and reduce_row_wave, by one wave, its parts in turn; both are
// built of merge_sets, trail_state, key_terms and finish_row, each by one wave of 64 lanes, and give the same bits for up
// to eight sets.
//
// Merges the per-split partial states (m, l, o[128], value-term sums, maxima, two largest block
// log-masses) with the usual log-sum-exp factors, attends the trailing FP16 tokens exactly
// (their keys and values are not quantized: eta = 0, no contribution to Delta_h), and
// evaluates the certificate of the paper's total error bound:
//   E_val = sum_b rho_b eta_b,   E_key = 2 V_max min(tanh Delta_h, min{1, e^{c Delta_h} alpha_hat}(e^{2 Delta_h} - 1))
// (key_bound_mode 1 / 2 select the second / first factor alone), the interval form of the
// ranking test  l_(1) - l_(2) <= 2 Delta_h + eps_guard,  and the flag word.
// Used by the split pass (rows of one workgroup, and short steps of several), the reduction kernels of the one-pass and of the adaptive
// decode, the selector, and the ladder's launch where rows are few or the workgroups of a short step were not on one die.
#pragma once

#include "cqa_internal.h"

namespace cqa {

struct ReduceArgs {
  const float* partials;  // [Bt][Hq][nsplit][PART_FLOATS]
  const __half* q;        // [Bt][Hq][128]
  const __half* trail_k;  // layer base [Bt*Hkv][16][128]
  const __half* trail_v;
  float* O;
  cqa_head_cert* cert;
  uint32_t* flags;
  uint32_t* flags_mirror;  // optional second copy of the flag words (mapped pinned host memory)
  uint32_t mirror_tag;     // OR-ed into each mirrored word (bits 16-31): the host polls for it
  uint32_t* raised;        // optional: set to raised_tag when a head requests a fallback (the ladder kernel
  uint32_t raised_tag;     // looks at the flag words only then)
  cqa_tolerances tol;
  int nsplit, nb, r, n_q, n_kv;
  int pstride;           // partial sets per (batch, q-head) row of `partials`; 0 = nsplit
};

// LDS operations of one wave execute in order; this only stops the compiler from moving LDS
// accesses across a point where the lanes of a wave exchange data through LDS.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// merges top-2 state (t1, i1, t2) with (u1, j1, u2); ties go to the lower block index
__device__ __forceinline__ void top2_merge(float& t1, int& i1, float& t2, float u1, int j1,
                                           float u2) {
  const bool keep = (t1 > u1) || (t1 == u1 && (unsigned)i1 <= (unsigned)j1);
  if (keep) {
    t2 = fmaxf(t2, u1);
  } else {
    t2 = fmaxf(u2, t1);
    t1 = u1;
    i1 = j1;
  }
}
// DPP move inside a row of 16 lanes (no LDS round trip)
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float x) {
  return __uint_as_float(
      (uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ int dpp_movi(int x) {
  return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xf, 0xf, true);
}
// all-reduce over the 16 lanes of a row: quad xor 1, quad xor 2, half-row mirror, row mirror
__device__ __forceinline__ float row_max(float x) {
  x = fmaxf(x, dpp_mov<0xB1>(x));
  x = fmaxf(x, dpp_mov<0x4E>(x));
  x = fmaxf(x, dpp_mov<0x141>(x));
  x = fmaxf(x, dpp_mov<0x140>(x));
  return x;
}
__device__ __forceinline__ float row_sum(float x) {
  x += dpp_mov<0xB1>(x);
  x += dpp_mov<0x4E>(x);
  x += dpp_mov<0x141>(x);
  x += dpp_mov<0x140>(x);
  return x;
}
// Exchanges across the rows of a wave on the vector ALU (gfx950 lane swaps; a __shfl_xor is an LDS round
// trip of ~100 cycles, and these sit on the serial chains that bound the short kernels: reduction
// 5.4 -> 4.7 us at 8K, selector 20.5 -> 18.9 and adaptive reduction 14.9 -> 13.6 us at 128K).  After swap16 every lane of rows 2i and 2i + 1 holds the pair
// (row 2i's value, row 2i + 1's value) of its column; after swap32 the pair (lane l, lane l + 32).
__device__ __forceinline__ void swap16(uint32_t x, uint32_t& even, uint32_t& odd) {
  const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  even = r[0];
  odd = r[1];
}
__device__ __forceinline__ void swap32(uint32_t x, uint32_t& lo, uint32_t& hi) {
  const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  lo = r[0];
  hi = r[1];
}
// x (+, max) the value of the lane 16 / 32 away, in every lane
__device__ __forceinline__ float sum_x16(float x) {
  uint32_t a, b;
  swap16(__float_as_uint(x), a, b);
  return __uint_as_float(a) + __uint_as_float(b);
}
__device__ __forceinline__ float sum_x32(float x) {
  uint32_t a, b;
  swap32(__float_as_uint(x), a, b);
  return __uint_as_float(a) + __uint_as_float(b);
}
__device__ __forceinline__ float max_x16(float x) {
  uint32_t a, b;
  swap16(__float_as_uint(x), a, b);
  return fmaxf(__uint_as_float(a), __uint_as_float(b));
}
__device__ __forceinline__ float max_x32(float x) {
  uint32_t a, b;
  swap32(__float_as_uint(x), a, b);
  return fmaxf(__uint_as_float(a), __uint_as_float(b));
}
// all-reduce over the 64 lanes of the wave: the row step on DPP, two cross-row exchanges
__device__ __forceinline__ float wave_sum(float v) { return sum_x32(sum_x16(row_sum(v))); }
__device__ __forceinline__ float wave_max(float v) { return max_x32(max_x16(row_max(v))); }
// ... of values that the four lanes of a quad have in common, each counted once
__device__ __forceinline__ float quads_sum(float x) {
  x += dpp_mov<0x141>(x);
  x += dpp_mov<0x140>(x);
  return sum_x32(sum_x16(x));
}
__device__ __forceinline__ float quads_max(float x) {
  x = fmaxf(x, dpp_mov<0x141>(x));
  x = fmaxf(x, dpp_mov<0x140>(x));
  return max_x32(max_x16(x));
}
__device__ __forceinline__ double pack_d(uint32_t lo, uint32_t hi) {
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
template <int CTRL>
__device__ __forceinline__ double dpp_mov_d(double x) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(x);
  return pack_d((uint32_t)dpp_movi<CTRL>((int)(uint32_t)u), (uint32_t)dpp_movi<CTRL>((int)(uint32_t)(u >> 32)));
}
__device__ __forceinline__ double wave_sum_d(double x) {
  x += dpp_mov_d<0xB1>(x);
  x += dpp_mov_d<0x4E>(x);
  x += dpp_mov_d<0x141>(x);
  x += dpp_mov_d<0x140>(x);
  unsigned long long u = (unsigned long long)__double_as_longlong(x);
  uint32_t al, bl, ah, bh;
  swap16((uint32_t)u, al, bl);
  swap16((uint32_t)(u >> 32), ah, bh);
  x = pack_d(al, ah) + pack_d(bl, bh);
  u = (unsigned long long)__double_as_longlong(x);
  swap32((uint32_t)u, al, bl);
  swap32((uint32_t)(u >> 32), ah, bh);
  return pack_d(al, ah) + pack_d(bl, bh);
}
// v plus the lane that DPP control CTRL points at (0 where there is none, or where ROWS masks the row out)
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_or_zero(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, true);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t scan_step(uint32_t v) { return v + dpp_or_zero<CTRL, ROWS>(v); }
template <int CTRL, int ROWS>
__device__ __forceinline__ int scan_step(int v) { return v + (int)dpp_or_zero<CTRL, ROWS>((uint32_t)v); }
template <int CTRL, int ROWS>
__device__ __forceinline__ double scan_step(double v) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  return v + pack_d(dpp_or_zero<CTRL, ROWS>((uint32_t)u), dpp_or_zero<CTRL, ROWS>((uint32_t)(u >> 32)));
}
__device__ __forceinline__ uint32_t row_total(uint32_t v) {
  v += (uint32_t)dpp_movi<0xB1>((int)v);
  v += (uint32_t)dpp_movi<0x4E>((int)v);
  v += (uint32_t)dpp_movi<0x141>((int)v);
  return v + (uint32_t)dpp_movi<0x140>((int)v);
}
__device__ __forceinline__ int row_total(int v) { return (int)row_total((uint32_t)v); }
__device__ __forceinline__ double row_total(double v) {
  v += dpp_mov_d<0xB1>(v);
  v += dpp_mov_d<0x4E>(v);
  v += dpp_mov_d<0x141>(v);
  return v + dpp_mov_d<0x140>(v);
}
// Inclusive scan over the lanes of a wave.
template <typename T>
__device__ __forceinline__ T wave_scan_incl(T v) {
  v = scan_step<0x111, 0xf>(v);   // row_shr 1, 2, 4, 8
  v = scan_step<0x112, 0xf>(v);
  v = scan_step<0x114, 0xf>(v);
  v = scan_step<0x118, 0xf>(v);
  v = scan_step<0x142, 0xa>(v);   // row_bcast 15 into rows 1 and 3
  return scan_step<0x143, 0xc>(v);   // row_bcast 31 into rows 2 and 3
}
// Inclusive scan over the threads of a workgroup with two barriers: DPP shifts inside each row of
// 16 lanes, the totals of the preceding rows by DPP broadcasts, then the preceding waves' totals.
// `tot` = one word of LDS scratch per wave.
template <typename T>
__device__ __forceinline__ T block_scan_incl(T v, T* tot, int tid) {
  const int l = tid & 63, w = tid >> 6;
  v = wave_scan_incl(v);
  __syncthreads();            // protects `tot` against the previous use
  if (l == 63) tot[w] = v;
  __syncthreads();
  // at most 16 waves: every row of lanes adds up the totals of the waves before this one
  return v + row_total((l & 15) < w ? tot[l & 15] : T(0));
}

// larger value wins; equal values: the lower index (-1 = nothing seen loses)
__device__ __forceinline__ void best_merge(float& v, int& i, float ov, int oi) {
  if (oi >= 0 && (i < 0 || ov > v || (ov == v && oi < i))) {
    v = ov;
    i = oi;
  }
}
__device__ __forceinline__ void wave_best(float& v, int& i) {
  best_merge(v, i, dpp_mov<0xB1>(v), dpp_movi<0xB1>(i));
  best_merge(v, i, dpp_mov<0x4E>(v), dpp_movi<0x4E>(i));
  best_merge(v, i, dpp_mov<0x141>(v), dpp_movi<0x141>(i));
  best_merge(v, i, dpp_mov<0x140>(v), dpp_movi<0x140>(i));
  uint32_t a, b, ai, bi;
  swap16(__float_as_uint(v), a, b);
  swap16((uint32_t)i, ai, bi);
  v = __uint_as_float(a);
  i = (int)ai;
  best_merge(v, i, __uint_as_float(b), (int)bi);
  swap32(__float_as_uint(v), a, b);
  swap32((uint32_t)i, ai, bi);
  v = __uint_as_float(a);
  i = (int)ai;
  best_merge(v, i, __uint_as_float(b), (int)bi);
}

// What the adaptive decode (gated key precision) substitutes in the certificate (the paper's total
// error bound with the achieved tail mass, and its ranking-consistency check): the estimated mass
// of the blocks left in INT8 and Delta_h come from the first (all-INT8) pass, the ranking verdict from a scan
// over the block log-masses of both passes.
struct AdaptiveIn {
  float alpha;       // sum over unpromoted blocks of the first pass's normalised masses
  float delta;       // Delta_h of the first pass
  float top_fp16;    // largest FP16 log-mass among promoted blocks (-inf if none)
  float kth_fp16;    // the r-th largest (r = ranking depth; = top_fp16 at depth 1)
  float tail_ub;     // largest unpromoted INT8 log-mass + Delta_h (-inf if none)
  int top_block;     // the promoted block with the largest FP16 log-mass (-1 if none)
  int rank_fail;     // the two rankings disagree on the top block, or the boundary test failed
  int precond;       // the score-consistency check found a score outside its declared bound
  // The mass, the value term and the largest rho_b eta_b of the blocks that are NOT listed, from the scan over the
  // block log-masses, relative to the first pass's lse8:  L8u = sum exp(l_b - lse8),
  // EV8u = sum exp(l_b - lse8) eta_b,  maxc8 = max exp(l_b - lse8) eta_b.
  float L8u, EV8u, maxc8, lse8;
};

// Merged softmax state of one (batch, query head): scalars in every lane, o2 = channels 2l, 2l + 1 of lane l.
struct HeadState {
  float M, L, EV, EVM, DM, VM, T1, T2;
  int I1;
  float2 o2;
};

__device__ __forceinline__ float lane_of(float x, int lane) {
  return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(x), lane));
}

// ---- merging states.  A state is nine scalars (in the order of the partial set's) and 128 channels.
// max, sum, smallest unsigned over the eight lanes of a half row, in each of them
__device__ __forceinline__ float oct_max(float x) {
  x = fmaxf(x, dpp_mov<0xB1>(x));
  x = fmaxf(x, dpp_mov<0x4E>(x));
  return fmaxf(x, dpp_mov<0x141>(x));
}
__device__ __forceinline__ float oct_sum(float x) {
  x += dpp_mov<0xB1>(x);
  x += dpp_mov<0x4E>(x);
  return x + dpp_mov<0x141>(x);
}
__device__ __forceinline__ uint32_t oct_minu(uint32_t x) {
  x = min(x, (uint32_t)dpp_movi<0xB1>((int)x));
  x = min(x, (uint32_t)dpp_movi<0x4E>((int)x));
  return min(x, (uint32_t)dpp_movi<0x141>((int)x));
}

// The scalars of up to eight merged states: lane 8 j + i holds scalar j (P_M .. P_T2) of the result.
struct OctState {
  float x;
  float M, T1;   // scalars P_M and P_T1, in every lane
  int i1;        // P_I1, in every lane
};
// Merges up to eight states.  Lane 8 j + i brings scalar j of state i (v) and the state's m, t1, t2, i1; on: there is a
// state i; sums: its mass and value term count.  f: the factor of state i's channels.
// One wave-wide reduction per scalar, six steps each and a long chain for the two largest log-masses, made this
// 2700 cycles of a lone wave; with a lane per scalar and state all scalars share three steps.
// Products and sums are kept apart: fused, the lanes of a pair would round differently, and every lane holds the bits
// that a partial set carries, whichever launch finishes the row.
__device__ __forceinline__ OctState merge_oct(float v, float m, float t1, float t2, int i1, bool on, bool sums, float& f) {
#pragma clang fp contract(off)
  const int j = (threadIdx.x & 63) >> 3;
  OctState r;
  r.M = oct_max(on ? m : -INFINITY);
  f = on ? __expf(m - (r.M == -INFINITY ? 0.0f : r.M)) : 0.0f;
  r.T1 = oct_max(on ? t1 : -INFINITY);
  const bool top = on && t1 == r.T1;
  const uint32_t best = oct_minu(top ? (uint32_t)i1 : 0xFFFFFFFFu);   // equal log-masses: the lower index (-1, none, is the largest)
  r.i1 = (int)best;
  const float second = top && (uint32_t)i1 == best ? t2 : t1;
  const float scaled = (sums ? f : 0.0f) * v;
  float x = j >= P_L && j <= P_EVMAX ? scaled : (j == P_T2 ? second : v);
  if (!on) x = j >= P_L && j <= P_VMAX ? 0.0f : -INFINITY;
  const float sum = oct_sum(x), mx = oct_max(x);
  r.x = j == P_M ? r.M : (j <= P_EV ? sum : mx);
  return r;
}
// ... of two results of it; fa, fb: the factors of their channels
__device__ __forceinline__ OctState merge_two(const OctState& a, const OctState& b, float& fa, float& fb) {
#pragma clang fp contract(off)
  const int j = (threadIdx.x & 63) >> 3;
  OctState r;
  r.M = fmaxf(a.M, b.M);
  const float base = r.M == -INFINITY ? 0.0f : r.M;
  fa = __expf(a.M - base);
  fb = __expf(b.M - base);
  r.T1 = fmaxf(a.T1, b.T1);
  r.i1 = a.T1 > b.T1 || (a.T1 == b.T1 && (uint32_t)a.i1 <= (uint32_t)b.i1) ? a.i1 : b.i1;
  const bool scaled = j >= P_L && j <= P_EVMAX;
  const float xa = scaled ? fa * a.x : a.x, xb = scaled ? fb * b.x : b.x;
  const float mx = fmaxf(xa, xb);
  r.x = j == P_M ? r.M : (j <= P_EV ? xa + xb : (j == P_T2 ? fmaxf(mx, fminf(a.T1, b.T1)) : mx));
  return r;
}
__device__ __forceinline__ HeadState head_state(const OctState& m, float2 o2) {
  HeadState r;
  r.M = m.M;
  r.L = lane_of(m.x, 8 * P_L);
  r.EV = lane_of(m.x, 8 * P_EV);
  r.EVM = lane_of(m.x, 8 * P_EVMAX);
  r.DM = lane_of(m.x, 8 * P_DMAX);
  r.VM = lane_of(m.x, 8 * P_VMAX);
  r.T1 = m.T1;
  r.T2 = lane_of(m.x, 8 * P_T2);
  r.I1 = m.i1;
  r.o2 = o2;
  return r;
}

// Eight partial sets' scalars, as merge_oct takes them, and channels 2l, 2l + 1 of each.  LIVE: other workgroups of the same launch and
// die have stored them: past the compute unit's own cache.
struct SetRegs {
  float v, m, t1, t2, i1;
  float2 x[8];
};
template <bool LIVE>
__device__ __forceinline__ float ld_set(const float* part, uint32_t at) {
  const float* p = part + at;
  return LIVE ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *p;
}
// sets s0, s0 + 1, ... of one head's n_sets (set s at part + s * PART_FLOATS; 32 bits hold the offsets of MAX_SPLITS sets)
template <bool LIVE>
__device__ __forceinline__ SetRegs load_sets(const float* part, int s0, int n_sets) {
  const uint32_t l = threadIdx.x & 63;
  SetRegs r;
  const uint32_t at = (uint32_t)min(s0 + (int)(l & 7), n_sets - 1) * PART_FLOATS;
  r.v = ld_set<LIVE>(part, at + (l >> 3));
  r.m = ld_set<LIVE>(part, at + P_M);
  r.t1 = ld_set<LIVE>(part, at + P_T1);
  r.t2 = ld_set<LIVE>(part, at + P_T2);
  r.i1 = ld_set<LIVE>(part, at + P_I1);
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float* po = part + (uint32_t)min(s0 + i, n_sets - 1) * PART_FLOATS + P_O;   // (uniform)
    if (LIVE) {
      const unsigned long long u =
          __hip_atomic_load(reinterpret_cast<const unsigned long long*>(po) + l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      r.x[i] = make_float2(__uint_as_float((uint32_t)u), __uint_as_float((uint32_t)(u >> 32)));
    } else {
      r.x[i] = reinterpret_cast<const float2*>(po)[l];
    }
  }
  return r;
}
// ... merged; of sets outside [pos0, pos1) only the channels (and maxima) count
__device__ __forceinline__ OctState merge_loaded(const SetRegs& g, int s0, int n_sets, int pos0, int pos1, float2& o) {
  const int s = s0 + (threadIdx.x & 7);
  float f;
  const OctState t = merge_oct(g.v, g.m, g.t1, g.t2, __float_as_int(g.i1), s < n_sets, s >= pos0 && s < pos1, f);
  o = make_float2(0.0f, 0.0f);
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float fi = lane_of(f, i);            // zero for sets past the end
    o.x = fmaf(fi, g.x[i].x, o.x);
    o.y = fmaf(fi, g.x[i].y, o.y);
  }
  return t;
}

// Merges partial sets first, first + 1, ..., first + 7, first + jump, ... of one head's n_sets; of sets outside
// [pos0, pos1) only the channels (and maxima) count.  o2: channels 2l, 2l + 1.
// All loads of a trip are issued before anything is consumed.
__device__ __forceinline__ OctState merge_sets(const float* part, int first, int jump, int n_sets, int pos0, int pos1, float2& o2) {
  const int l = threadIdx.x & 63;
  OctState r;
  r.M = r.T1 = -INFINITY;
  r.i1 = -1;
  r.x = (l >> 3) >= P_L && (l >> 3) <= P_VMAX ? 0.0f : -INFINITY;
  o2 = make_float2(0.0f, 0.0f);
  for (int s0 = first; s0 < n_sets; s0 += jump) {
    float2 o;
    const OctState t = merge_loaded(load_sets<false>(part, s0, n_sets), s0, n_sets, pos0, pos1, o);
    if (s0 == first) {
      r = t;
      o2 = o;
    } else {
      float fa, fb;
      r = merge_two(r, t, fa, fb);
      o2.x = fmaf(fa, o2.x, fb * o.x);
      o2.y = fmaf(fa, o2.y, fb * o.y);
    }
  }
  return r;
}

// Merges the states of n <= 8 waves kept in LDS: scalars at ms + i * ms_stride, channels at mo + i * mo_stride.
// Waves that saw no block hold zeros and a maximum of -infinity; the result of only such waves is one more of the kind.
// N: the number when it is known, and all reads are on their way at once (else four at a time).
template <int N = 0>
__device__ __forceinline__ OctState merge_lds(const float* ms, int ms_stride, const float* mo, int mo_stride, int n, float2& o2) {
  const int l = threadIdx.x & 63, i = l & 7;
  if (N > 0) n = N;
  const float* m = ms + (i < n ? i : 0) * ms_stride;
  float f;
  const OctState r = merge_oct(m[l >> 3], m[P_M], m[P_T1], m[P_T2], __float_as_int(m[P_I1]), i < n, true, f);
  o2 = make_float2(0.0f, 0.0f);
  if (N > 0) {
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const float fk = lane_of(f, k);
      const float2 x = *reinterpret_cast<const float2*>(mo + k * mo_stride + 2 * l);
      o2.x = fmaf(fk, x.x, o2.x);
      o2.y = fmaf(fk, x.y, o2.y);
    }
    return r;
  }
  for (int k0 = 0; k0 < n; k0 += 4) {
    float2 x[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = *reinterpret_cast<const float2*>(mo + min(k0 + k, n - 1) * mo_stride + 2 * l);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (k0 + k >= n) break;
      const float fk = lane_of(f, k0 + k);
      o2.x = fmaf(fk, x[k].x, o2.x);
      o2.y = fmaf(fk, x[k].y, o2.y);
    }
  }
  return r;
}

// state a, channels o2, joined by one that store_state has left: what merge_lds gives for the two, bit for bit
__device__ __forceinline__ OctState join_lds(const OctState& a, const float* ms, const float* mo, float2& o2) {
#pragma clang fp contract(off)
  const int l = threadIdx.x & 63;
  OctState b;
  b.x = ms[l >> 3];
  b.M = ms[P_M];
  b.T1 = ms[P_T1];
  b.i1 = __float_as_int(ms[P_I1]);
  const float2 x = *reinterpret_cast<const float2*>(mo + 2 * l);
  float fa, fb;
  const OctState r = merge_two(a, b, fa, fb);
  o2.x = fmaf(fb, x.x, fa * o2.x);
  o2.y = fmaf(fb, x.y, fa * o2.y);
  return r;
}
// a state as merge_lds reads it / as a partial set
__device__ __forceinline__ void store_state(const OctState& m, float2 o2, float* ms, float* mo) {
  const int l = threadIdx.x & 63;
  if ((l & 7) == 0) ms[l >> 3] = m.x;
  if (l == 1) ms[P_I1] = __int_as_float(m.i1);
  *reinterpret_cast<float2*>(mo + 2 * l) = o2;
}

// Trailing FP16 tokens of one head (at most 15), requested before the partial sets and used after them.
//   scores / norms: lane (t = l >> 2, cpart = l & 3) covers channels 32 cpart .. 32 cpart + 31 of
//   token t; values for the output: lane l covers channels 2l, 2l + 1 of every token.
__device__ __forceinline__ int64_t row_of(const ReduceArgs& a, int b, int hq) { return (int64_t)b * a.n_q + hq; }
__device__ __forceinline__ int64_t group_of(const ReduceArgs& a, int b, int hq) {
  return (int64_t)b * a.n_kv + (hq >> group_shift(a.n_q, a.n_kv));
}
struct TrailRegs {
  uint4 kq[4], vq[4], qq[4];
  __half2 vt[BLK - 1];
};

// new_k, new_v (null = none): the last trailing token, when the launch that calls this also appends it
__device__ __forceinline__ void load_trail(const ReduceArgs& a, int64_t grp, int64_t row, const __half* new_k,
                                           const __half* new_v, TrailRegs& t) {
  const int l = threadIdx.x & 63;
  const __half* tk = a.trail_k + grp * BLK * D;
  const __half* tv = a.trail_v + grp * BLK * D;
  const int last = max(a.r - 1, 0);
  const int tt = min(l >> 2, last), cpart = l & 3;
  const bool fresh = new_k != nullptr && tt == last;
  const __half* kp = (fresh ? new_k + grp * D : tk + tt * D) + cpart * 32;
  const __half* vp = (fresh ? new_v + grp * D : tv + tt * D) + cpart * 32;
  const __half* qp = a.q + row * D + cpart * 32;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    t.kq[i] = ld16_any(kp + 8 * i);
    t.vq[i] = ld16_any(vp + 8 * i);
    t.qq[i] = ld16_any(qp + 8 * i);
  }
#pragma unroll
  for (int i = 0; i < BLK - 1; ++i) {
    const int j = min(i, last);
    const __half* row = new_v != nullptr && j == last ? new_v + grp * D : tv + j * D;
    t.vt[i] = ld_half2_any(row + 2 * l);
  }
}

// The result of one (batch, query head): certificate and flag word in every lane, out = channels 2l, 2l + 1 of lane l.
struct HeadRow {
  cqa_head_cert ct;
  float top;      // largest block log-mass
  uint32_t fl;
  float2 out;
};

// The trailing tokens as a state of their own: exact keys and values, eta = 0, no contribution to Delta_h.
struct TrailState {
  float M, L, V;   // maximum, mass, largest value norm; in every lane
  float2 o;
};
__device__ __forceinline__ TrailState trail_state(const ReduceArgs& a, const TrailRegs& tr) {
#pragma clang fp contract(off)
  const int l = threadIdx.x & 63;
  const float inv_sqrt_d = 0.08838834764831845f;
  float dot = 0.0f, n2 = 0.0f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const __half2* kh = reinterpret_cast<const __half2*>(&tr.kq[i]);
    const __half2* vh = reinterpret_cast<const __half2*>(&tr.vq[i]);
    const __half2* qh = reinterpret_cast<const __half2*>(&tr.qq[i]);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      dot = fmaf(__low2float(qh[e]), __low2float(kh[e]), dot);
      dot = fmaf(__high2float(qh[e]), __high2float(kh[e]), dot);
      n2 = fmaf(__low2float(vh[e]), __low2float(vh[e]), n2);
      n2 = fmaf(__high2float(vh[e]), __high2float(vh[e]), n2);
    }
  }
  dot += dpp_mov<0xB1>(dot);      // the four parts of a token are one quad of lanes
  dot += dpp_mov<0x4E>(dot);
  n2 += dpp_mov<0xB1>(n2);
  n2 += dpp_mov<0x4E>(n2);
  const bool live = (l >> 2) < a.r;
  const float st = live ? dot * inv_sqrt_d : -INFINITY;
  TrailState t;
  t.M = quads_max(st);
  t.V = quads_max(live ? sqrtf(n2) : 0.0f);
  const float pt = live ? __expf(st - (t.M == -INFINITY ? 0.0f : t.M)) : 0.0f;
  t.L = quads_sum(pt);
  t.o = make_float2(0.0f, 0.0f);
#pragma unroll
  for (int i = 0; i < BLK - 1; ++i) {
    const float p = lane_of(pt, 4 * i);       // zero for tokens past the last
    t.o.x = fmaf(p, __low2float(tr.vt[i]), t.o.x);
    t.o.y = fmaf(p, __high2float(tr.vt[i]), t.o.y);
  }
  return t;
}

// What the key term takes from Delta_h alone.  No cap on the exponents: beyond the binary32 range the factors are +inf, the
// tail form of the key term with them, and a non-finite key term raises PRECOND (in the default
// mode the tanh form, at most 1, still wins the min).
struct KeyTerms {
  float full, grow, widen;   // tanh Delta_h, e^{c Delta_h}, e^{2 Delta_h} - 1
};
__device__ __forceinline__ KeyTerms key_terms(const ReduceArgs& a, float delta) {
  return KeyTerms{tanhf(delta), expf((float)a.tol.mass_exp * delta), expm1f(2.0f * delta)};
}

// Joins the sealed blocks' state and the trailing tokens' and evaluates the certificate.
__device__ __forceinline__ HeadRow finish_row(const ReduceArgs& a, const HeadState& hs, const TrailState& ts,
                                              const KeyTerms& kt, const AdaptiveIn* ad) {
#pragma clang fp contract(off)
  float M = hs.M, L = hs.L, EV = hs.EV, EVM = hs.EVM, VM = hs.VM;
  const float DM = hs.DM, T1 = hs.T1, T2 = hs.T2;
  int I1 = hs.I1;
  float2 o2 = hs.o2;
  if (ad != nullptr) {
    // the blocks no second pass touched: their mass and value term from the scan
    const float g8 = __expf(ad->lse8 - M);
    L += g8 * ad->L8u;
    EV += g8 * ad->EV8u;
    EVM = fmaxf(EVM, g8 * ad->maxc8);
  }
  float L_sealed = L;
  if (a.r > 0) {
    const float M2 = fmaxf(M, ts.M);
    const float fs = __expf(M - M2), ft = __expf(ts.M - M2);
    VM = fmaxf(VM, ts.V);
    EV *= fs;
    EVM *= fs;
    L_sealed = L * fs;
    L = fmaf(ft, ts.L, L_sealed);
    o2.x = fmaf(ft, ts.o.x, o2.x * fs);
    o2.y = fmaf(ft, ts.o.y, o2.y * fs);
    M = M2;
  }

  HeadRow row;
  row.out = make_float2(o2.x / L, o2.y / L);
  const bool bad = __any(!isfinite(row.out.x) || !isfinite(row.out.y));

  // certificate scalars in FP32 (a handful of operations; their rounding is ~1e-7 relative); three quotients by one division, a lane each
  const int lane = threadIdx.x & 63;
  const float share = (lane == 0 ? EV : (lane == 1 ? EVM : L_sealed)) / L;
  const float e_val = lane_of(share, 0);
  const float lse = M + logf(L);
  const float maxc = lane_of(share, 1);
  const float alpha_hat = ad != nullptr ? ad->alpha : lane_of(share, 2);
  const float delta = ad != nullptr ? ad->delta : DM;
  const float vmax = VM;
  float t_tail = 0.0f;
  if (alpha_hat > 0.0f && delta != 0.0f) t_tail = fminf(1.0f, kt.grow * alpha_hat) * kt.widen;
  const float t_full = kt.full;
  const float tv = a.tol.key_bound_mode == 0 ? fminf(t_full, t_tail) : (a.tol.key_bound_mode == 1 ? t_tail : t_full);
  const float e_key = 2.0f * vmax * tv;
  float margin = a.nb >= 2 ? T1 - T2 : INFINITY;
  float rho_top = a.nb >= 1 ? expf(T1 - lse) : 0.0f;
  bool rank_flag = a.tol.rank_depth >= 1 && a.nb >= 2 && rho_top >= a.tol.rank_min_mass &&
                   margin <= 2.0f * delta + a.tol.eps_guard;
  if (ad != nullptr) {
    const bool any = ad->top_block >= 0;
    margin = any ? ad->kth_fp16 - ad->tail_ub : INFINITY;
    rho_top = any ? expf(ad->top_fp16 - lse) : 0.0f;
    rank_flag = a.tol.rank_depth >= 1 && any && rho_top >= a.tol.rank_min_mass && ad->rank_fail != 0;
    I1 = ad->top_block;
  }

  uint32_t fl = 0;
  if (e_key > a.tol.eps_key) fl |= CQA_FLAG_KEY;
  if (e_val > a.tol.eps_val || maxc > a.tol.v_tol) fl |= CQA_FLAG_VAL;
  if (rank_flag) fl |= CQA_FLAG_RANK;
  if (ad != nullptr && ad->precond != 0) fl |= CQA_FLAG_PRECOND;
  if (bad || !isfinite(e_key) || !isfinite(e_val) || !isfinite(delta) || !isfinite(vmax) || !isfinite(lse))
    fl |= CQA_FLAG_PRECOND;
  if (e_key + e_val > a.tol.eps_total) fl |= CQA_FLAG_TOTAL;
  fl |= a.tol.force_flags;

  row.ct.E_key = e_key;
  row.ct.E_val = e_val;
  row.ct.delta_h = delta;
  row.ct.v_max = VM;
  row.ct.alpha_tail_hat = alpha_hat;
  row.ct.lse = lse;
  row.ct.max_block_contrib = maxc;
  row.ct.rank_margin = margin;
  row.ct.top_block = I1;
  row.ct.served_rung = 0;
  row.fl = fl;
  row.top = T1;
  return row;
}

// mirror: the row's own store of its mirrored flag word (the caller makes it otherwise, behind these stores)
__device__ __forceinline__ void store_row(const ReduceArgs& a, int64_t r, const HeadRow& row, bool mirror = true) {
  const int l = threadIdx.x & 63;
  reinterpret_cast<float2*>(a.O + r * D)[l] = row.out;
  if (l == 0) {
    a.cert[r] = row.ct;
    a.flags[r] = row.fl;
    if (a.raised != nullptr && (row.fl & CQA_FLAG_ANY) != 0u) *a.raised = a.raised_tag;
    // last store of this head: a host thread polling the mirror may take the tagged word as
    // "this head's row, certificate and flags have been issued" (device consumers rely on
    // stream order, not on this word)
    if (mirror && a.flags_mirror != nullptr)
      __hip_atomic_store(a.flags_mirror + r, row.fl | a.mirror_tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

__device__ __forceinline__ void finish_head(const ReduceArgs& a, int b, int hq, const HeadState& hs, const TrailState& ts,
                                            const KeyTerms& kt, const AdaptiveIn* ad) {
  store_row(a, row_of(a, b, hq), finish_row(a, hs, ts, kt, ad));
}

// One (batch, query head) by a workgroup of `waves` waves, at least three.  It runs on the critical tail of a step, alone on the
// chip, and is bound by the length of its instruction chain, so the chain is cut into parts that run side by side: up to RED_WAVES
// waves merge eight partial sets a trip each, one attends the trailing tokens, one takes Delta_h through the
// key term's functions; the first then joins their results and returns true.  Where one wave per head did all this in turn
// (8500 cycles), a step of 8 KV heads, four layers: 8229 tokens 64.4 -> 57.7 us, 3000 tokens 59.6 -> 50.6.
constexpr int RED_WAVES = 8;
// waves of such a workgroup: one per eight sets, while there are, and two
__host__ __device__ inline int reduce_waves(int nsplit) {
  const int nw = (nsplit + 7) / 8;
  return (nw < 1 ? 1 : (nw > RED_WAVES ? RED_WAVES : nw)) + 2;
}
struct ReduceSmem {
  float sc[RED_WAVES][12];
  float o[RED_WAVES][D];
  float trail_o[D];
  float trail[4], key[4];
};
// the parts of the waves beside the merging ones, and what they leave, in every lane
__device__ __forceinline__ void trail_part(const ReduceArgs& a, int b, int hq, ReduceSmem& sm) {
  if (a.r <= 0) return;
  const int l = threadIdx.x & 63;
  TrailRegs tr;
  load_trail(a, group_of(a, b, hq), row_of(a, b, hq), nullptr, nullptr, tr);
  const TrailState ts = trail_state(a, tr);
  *reinterpret_cast<float2*>(&sm.trail_o[2 * l]) = ts.o;
  if (l == 0) {
    sm.trail[0] = ts.M;
    sm.trail[1] = ts.L;
    sm.trail[2] = ts.V;
  }
}
__device__ __forceinline__ void key_part(const ReduceArgs& a, float delta, ReduceSmem& sm) {
  const KeyTerms kt = key_terms(a, delta);
  if ((threadIdx.x & 63) == 0) {
    sm.key[0] = kt.full;
    sm.key[1] = kt.grow;
    sm.key[2] = kt.widen;
  }
}
__device__ __forceinline__ TrailState trail_of(const ReduceSmem& sm) {
  return TrailState{sm.trail[0], sm.trail[1], sm.trail[2], *reinterpret_cast<const float2*>(&sm.trail_o[2 * (threadIdx.x & 63)])};
}
__device__ __forceinline__ KeyTerms key_of(const ReduceSmem& sm) { return KeyTerms{sm.key[0], sm.key[1], sm.key[2]}; }

__device__ __forceinline__ bool reduce_row(const ReduceArgs& a, int b, int hq, int waves, ReduceSmem& sm, HeadRow& row) {
  const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nw = min(waves - 2, RED_WAVES);
  const float* part = a.partials + ((int64_t)b * a.n_q + hq) * (a.pstride > 0 ? a.pstride : a.nsplit) * PART_FLOATS;
  OctState st{};
  float2 o2 = make_float2(0.0f, 0.0f);
  if (w < nw) {
    st = merge_sets(part, 8 * w, 8 * nw, a.nsplit, 0, a.nsplit, o2);
    if (nw > 1) store_state(st, o2, sm.sc[w], sm.o[w]);
  } else if (w == nw) {
    trail_part(a, b, hq, sm);
  } else if (w == nw + 1) {
    float delta = 0.0f;
    for (int s = l; s < a.nsplit; s += 64) delta = fmaxf(delta, part[(int64_t)s * PART_FLOATS + P_DMAX]);
    key_part(a, wave_max(delta), sm);
  }
  __syncthreads();
  if (w != 0) return false;
  if (nw > 1) st = merge_lds(sm.sc[0], 12, sm.o[0], D, nw, o2);
  row = finish_row(a, head_state(st, o2), trail_of(sm), key_of(sm), nullptr);
  return true;
}

// ... by one wave, its parts one after the other.
__device__ __forceinline__ HeadRow reduce_row_wave(const ReduceArgs& a, int64_t row) {
  TrailRegs tr;
  TrailState ts{};
  if (a.r > 0) load_trail(a, row >> group_shift(a.n_q, a.n_kv), row, nullptr, nullptr, tr);
  float2 o2;
  const OctState st = merge_sets(a.partials + row * (a.pstride > 0 ? a.pstride : a.nsplit) * PART_FLOATS, 0, 8, a.nsplit, 0, a.nsplit, o2);
  if (a.r > 0) ts = trail_state(a, tr);
  const HeadState hs = head_state(st, o2);
  return finish_row(a, hs, ts, key_terms(a, hs.DM), nullptr);
}

// The exploration draw: 32-bit multiply-xorshift mixer over (block, KV group, seed).
__device__ __forceinline__ uint32_t explore_mix(uint32_t blk, uint32_t grp, uint32_t seed) {
  uint32_t x = blk * 0x9E3779B1u ^ grp * 0x85EBCA77u ^ seed * 0xC2B2AE3Du;
  x ^= x >> 16;
  x *= 0x7FEB352Du;
  x ^= x >> 15;
  x *= 0x846CA68Bu;
  x ^= x >> 16;
  return x;
}

// Promotion bits of one word (32 blocks) of a KV group, from its heads' masks: key bits kh and value bits vh per head;
// explored blocks are key-promoted for every head, and with per-group promotion every head has the unions.
struct PromBits {
  uint32_t kh[4], vh[4], k, v;
};
__device__ __forceinline__ PromBits prom_bits(const PromMasks& p, int64_t grp, int group, int word, uint32_t only) {
  PromBits r;
  r.k = r.v = 0u;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t at = (grp * group + i) * p.mask_words + word;
    r.kh[i] = i < group ? p.umask[at] & only : 0u;
    r.vh[i] = i < group && p.vmask != nullptr ? p.vmask[at] & only : 0u;
    r.k |= r.kh[i];
    r.v |= r.vh[i];
  }
  if (p.explore_threshold != 0u) {
    uint32_t x = 0u;
    for (uint32_t m = only; m != 0u; m &= m - 1u) {
      const int j = __ffs((int)m) - 1;
      if (explore_mix((uint32_t)(word * 32 + j), (uint32_t)grp, p.explore_seed) < p.explore_threshold) x |= 1u << j;
    }
    r.k |= x;
#pragma unroll
    for (int i = 0; i < 4; ++i) r.kh[i] |= x;
  }
  const uint32_t in = word * 32 + 32 <= p.nb ? ~0u : (1u << (p.nb & 31)) - 1u;   // nothing past nb
  r.k &= in;
  r.v &= in;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    r.kh[i] = i < group ? (p.per_head ? r.kh[i] & in : r.k) : 0u;
    r.vh[i] = i < group ? (p.per_head ? r.vh[i] & in : r.v) : 0u;
  }
  return r;
}
// flag word of the word's block j: bit 0 some head scores it with FP16 keys, bit 1 some head attends its FP16 values, then
// which heads
__device__ __forceinline__ int prom_flags(const PromBits& m, int j) {
  uint32_t f = ((m.k >> j) & 1u) | (((m.v >> j) & 1u) << 1);
#pragma unroll
  for (int i = 0; i < 4; ++i)
    f |= (((m.kh[i] >> j) & 1u) << (SLOT_HK_SHIFT + i)) | (((m.vh[i] >> j) & 1u) << (SLOT_HV_SHIFT + i));
  return (int)f;
}

}  // namespace cqa
