// Adaptive key precision: selector, promoted-set bookkeeping, and the reduction of the attend
// pass with its ranking check.
//
// Follows the paper's "Adaptive Precision Selection" (rank blocks by INT8-estimated mass, K* =
// smallest prefix that covers tau_cov, clamp to [K_min, K_max]), the first rung of its "Fallback
// Ladder" (grow K while the key term is over its threshold), its total error bound with the
// achieved INT8-estimated tail mass, and its "Ranking-Consistency Check" with the boundary
// verification, at depth r <= MAX_RANK_DEPTH.  Key and value precision are chosen per KV group
// (the union of the group's query heads' selections: the paper's per-KV-group selection variant)
// or, with cqa_selector.per_head, per query head over the head's own promoted set (its default).
//
// Sequence on one stream (launch_adaptive): the certified pass over all sealed blocks in INT8 /
// INT4 (it emits the block log-masses, eta_b and the usual partial sets) -> select_kernel (per head and ranking: keys, values; it
// reduces the head's partial sets for the total log-mass, Delta_h and V_max) -> promoted-block
// pass over the listed blocks only (each workgroup makes its share of the list from the selection masks):
// positive partial sets computed with the originals the flags ask
// for (read straight from the pinned Tier-2 arrays over the host link) and negated sets computed as
// the first pass did, so that the merge replaces those blocks' contribution; beside it, a workgroup per head sums up what
// is left in INT8 -> adaptive_reduce_kernel.
// Tier-1 is read once per step; the paper's two passes (score, then attend) become one pass plus a
// correction for a few dozen blocks.
#include <algorithm>

#include "cqa_internal.h"
#include "reduce_inl.h"

namespace cqa {

// defined in decode.hip
int32_t launch_promoted_pass(const DecodeArgs& a, const PromArgs& p, int group, dim3 grid, hipStream_t st);

namespace {

// order-preserving map float -> uint32 (larger float <=> larger integer)
__device__ __forceinline__ uint32_t ord32(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float from_ord32(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k ^ 0x80000000u) : ~k);
}

// What one ranking of a head's blocks reads and writes: by log-mass (keys) or by contribution (values).
struct SelectSide {
  int32_t* sel;                // [Bt][Hq][MAX_K_LIMIT]
  int32_t* kstar;              // [Bt][Hq]
  uint32_t* umask;             // [Bt][Hq][mask_words]: the head's own selection
  int k_min, k_max, k_limit;
};
struct SelectArgs {
  SelectSide side[2];          // [0] keys, [1] values
  const float* lm8;            // [Bt][Hq][nb]: log-masses of the pass over all blocks
  const float* eta_blk;        // [Bt][Hkv][nb] (values)
  float* contrib;              // [Bt][Hq][nb]: estimated contributions p_b eta_b, written here (values)
  ReduceArgs ra;               // reduction of the pass over all blocks
  float* first;                // [Bt][Hq][4]: lse, delta_h, v_max of that pass, written here
  int32_t* slot;               // [Bt][Hkv][slot_stride]: the flag words of the previous call's list are taken back here
  int64_t slot_stride;
  const int32_t* ulist;        // [Bt][Hkv][MAX_UNION]
  const int32_t* ucount;       // [Bt][Hkv]
  float v_tol, eps_val;        // value selection: local threshold and budget
  float* score_dev;            // [Bt][Hq] canary output, cleared here (null = no canary)
  int v_greedy;
  int64_t mask_words;
  int nb, n_q, n_kv;
  float tau_cov;
  float eps_key;
  int mass_exp, key_bound_mode;
};

constexpr int ST = 1024;          // threads of the selector workgroup
constexpr int SBATCH = 8;         // loads in flight per thread

// The selector walks its row of log-masses several times.  Rows of up to LDS_KEYS blocks are read
// from memory once, as order-preserving integer keys and their histogram bins kept in LDS; longer rows are re-read.
constexpr int LDS_KEYS = 10240;   // 40 KB of keys, 20 KB of bins: contexts up to 160K tokens
#define CQA_KEY_PASS(ROW, N, TID, CACHED, KEYS, BODY)                             \
  for (int base__ = 0; base__ < (N); base__ += ST * SBATCH) {                      \
    uint32_t key__[SBATCH];                                                         \
    _Pragma("unroll") for (int j__ = 0; j__ < SBATCH; ++j__) {                      \
      const int i__ = base__ + j__ * ST + (TID);                                  \
      key__[j__] = i__ < (N) ? ((CACHED) ? (KEYS)[i__] : ord32((ROW)[i__])) : 0u;  \
    }                                                                              \
    _Pragma("unroll") for (int j__ = 0; j__ < SBATCH; ++j__) {                      \
      const int i = base__ + j__ * ST + (TID);                                    \
      const uint32_t k = key__[j__];                                               \
      const bool in = i < (N);                                                     \
      BODY                                                                         \
    }                                                                              \
  }

// E_key / (1) from Delta_h, the estimated tail mass and V_max, in double (decision only)
__device__ double key_term_d(double delta, double alpha, double vmax, int mass_exp, int mode) {
  double t_tail = 0.0;
  if (alpha > 0.0 && delta != 0.0) {
    const double grow = exp(fmin((double)mass_exp * delta, 700.0));
    const double widen = expm1(fmin(2.0 * delta, 700.0));
    t_tail = fmin(1.0, grow * alpha) * widen;
  }
  const double t_full = tanh(delta);
  const double tv = mode == 0 ? fmin(t_full, t_tail) : (mode == 1 ? t_tail : t_full);
  return 2.0 * vmax * tv;
}

// Histogram increment for a whole wave.  Log-masses of one head share their leading bits, so in
// the first passes most lanes hit the same bin and plain LDS atomics would serialise 64 ways: up
// to two bins are first counted by ballot (one atomic each), the rest go one by one.
__device__ __forceinline__ void hist_add(uint32_t* hist, uint32_t bin, bool pred) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const unsigned long long active = __ballot(pred);
    if (active == 0ull) return;
    const int leader = __ffsll((long long)active) - 1;
    const uint32_t lb = (uint32_t)__shfl((int)bin, leader);
    const bool same = pred && bin == lb;
    const unsigned long long votes = __ballot(same);
    if (lane == leader) atomicAdd(&hist[lb], (uint32_t)__popcll(votes));
    if (same) pred = false;
  }
  if (pred) atomicAdd(&hist[bin], 1u);
}

// Histogram bin of a value in the selector's first pass: not decreasing with the value in the order the
// selection keeps (that of ord32: what is not a number, with the sign set, is last), 1024 bins where the KL-th best can lie -- log-masses by their distance below the largest
// one, 1/32 apart up to 16 (diffuse heads), 1/8 up to 64, 1 beyond (heads with a few dominant blocks; a distance below the
// total log-mass would put all blocks into the last bin where the trailing tokens hold nearly all of it: 128K, such a head
// 23 us against 10);
// contributions by octave eighths of the binary representation.
template <bool VALUES>
__device__ __forceinline__ int select_bin(float x, float top) {
  if (VALUES) {
    const int i = (int)(__float_as_uint(x) >> 20) - 18;
    return __float_as_uint(x) >> 31 ? 0 : min(max(i, 0), ST - 1);
  }
  if (__float_as_uint(x) > 0xFF800000u) return 0;
  const float d = top - x;
  const float t = d < 16.0f ? d * 32.0f : (d < 64.0f ? fmaf(d - 16.0f, 8.0f, 512.0f) : 832.0f + d);
  return ST - 1 - (int)fminf(fmaxf(t, 0.0f), (float)(ST - 1));
}

// One workgroup per (batch, query head) and ranking (blockIdx.z: 0 keys, 1 values).  Finds the
// KL = min(k_limit, nb) best blocks
// under the total order (larger value first, equal values: lower index first), ranks them, and takes a prefix.
//   VALUES = false: the row holds INT8 block log-masses; the prefix is the smallest one whose
//                   estimated masses cover tau_cov, clamped, then grown by Rung 1.
//   VALUES = true : the row holds estimated contributions c_b = p_b eta_b (the paper's rho_hat_b eta_b of its
//                   value-promotion rule, formed here; second rung of the ladder); the prefix is every
//                   block with c_b > v_tol and, in the hard-budget
//                   variant, as many more as bring the estimate left under eps_val; cap k_limit.
// Bound by its chain of barriers, scans and passes over the row, so there are few of them: one pass
// over memory with a 1024-bin histogram; the blocks from the bin of the KL-th best up, usually a few dozen
// more than KL, are rank-sorted as they are.  Only when that bin is crowded (equal
// or nearly equal values) a radix selection narrows them down to KL.
// 128K, 32 heads: 18.9 -> 14.6 us (four radix passes before).  4 x 32K, keys and values in one launch: 9.9 us
// (16.1 + 15.1 in two launches and 4.8 for one that formed the contributions, before).  The reduction at its head, under
// which the row's first loads come in, adds 2.5 us and saves a launch of 4.8 us.  Places handed out per wave instead of per lane,
// the first covering place by ballot, bins below the largest log-mass: 128K step 102.7 -> 99.6 us.
constexpr int CAND_SLACK = 256;   // blocks beyond KL that the rank sort takes rather than another pass

struct SelectSmem {
  unsigned long long cand[MAX_K_LIMIT + CAND_SLACK + 32];   // candidates, unordered
  unsigned long long sorted[MAX_K_LIMIT];   // the winners, best first: (key, ~index)
  double pm[MAX_K_LIMIT];                   // prefix sums of their masses
  uint32_t hist[ST];
  uint16_t bins[LDS_KEYS];                  // histogram bins of the keys
  union {
    uint32_t keys[LDS_KEYS];
    ReduceSmem red;                         // (before there are keys)
  };
};

template <bool VALUES>
__device__ __forceinline__ void select_rows(const SelectArgs& a, SelectSmem& sm) {
  const int tid = threadIdx.x;
  const int hq = blockIdx.x, b = blockIdx.y;
  const int64_t row = (int64_t)b * a.n_q + hq;
  const SelectSide& side = a.side[VALUES ? 1 : 0];
  const int nb = a.nb;
  float* contrib = VALUES ? a.contrib + row * nb : nullptr;
  const float* lm = a.lm8 + row * nb;
  const float* eta = VALUES ? a.eta_blk + ((int64_t)b * a.n_kv + (hq >> group_shift(a.n_q, a.n_kv))) * nb : nullptr;
  const float* ranked = VALUES ? contrib : lm;         // the row as later passes re-read it
  const int KL = min(max(side.k_limit, side.k_max), min(nb, MAX_K_LIMIT));

  uint32_t* const hist = sm.hist;
  uint32_t* const keys = sm.keys;
  unsigned long long* const cand = sm.cand;
  unsigned long long* const sorted = sm.sorted;
  double* const pm = sm.pm;
  const bool cached = nb <= LDS_KEYS;
  __shared__ double dtot[ST / 64], dsum[ST / 64];
  __shared__ uint32_t utot[ST / 64];
  __shared__ uint32_t s_prefix, s_want, s_cnt;
  __shared__ uint32_t s_idx_prefix, s_idx_want;
  __shared__ int s_k, s_first, s_bin, s_found, s_done;

  // ---- the first blocks of the row are requested, the head's partial sets are reduced meanwhile, and what the previous
  //      call left behind is taken back: the head's mask, and by one head the flag words of the group's list
  //      (The waves that reduce ask for their sets first.)
  float v[SBATCH], e[SBATCH];
  const auto load_row = [&](int base) {
#pragma unroll
    for (int j = 0; j < SBATCH; ++j) {
      const int i = base + j * ST + tid;
      v[j] = i < nb ? lm[i] : 0.0f;
      e[j] = VALUES && i < nb ? eta[i] : 0.0f;
    }
  };
  const int reducing = reduce_waves(a.ra.nsplit);   // waves
  uint32_t* const um = side.umask + row * a.mask_words;
  if ((tid >> 6) >= reducing) {
    load_row(0);
    const int t = tid - 64 * reducing, step = ST - 64 * reducing;
    for (int i = t; i < ((nb + 31) >> 5); i += step) um[i] = 0u;
    const int shift = group_shift(a.n_q, a.n_kv);
    if (!VALUES && (hq & ((1 << shift) - 1)) == 0) {
      const int64_t grp = (int64_t)b * a.n_kv + (hq >> shift);
      const int n_prev = min(a.ucount[grp], MAX_UNION);
      for (int i = t; i < n_prev; i += step) {
        const int blk = a.ulist[grp * MAX_UNION + i];
        if (blk >= 0 && blk < a.slot_stride) a.slot[grp * a.slot_stride + blk] = 0;
      }
    }
  }
  hist[tid] = 0u;
  __shared__ float s_lse, s_delta, s_vmax, s_top;
  {
    HeadRow hr;
    if (reduce_row(a.ra, b, hq, reducing, sm.red, hr) && tid == 0) {
      s_lse = hr.ct.lse;
      s_delta = hr.ct.delta_h;
      s_vmax = hr.ct.v_max;
      s_top = hr.top;
      if (!VALUES) *reinterpret_cast<float4*>(a.first + row * 4) = make_float4(hr.ct.lse, hr.ct.delta_h, hr.ct.v_max, 0.0f);
    }
  }
  if (tid == 0) {
    s_cnt = 0u;
    s_first = MAX_K_LIMIT + 1;
    s_bin = 0;
    s_found = nb;
  }
  if ((tid >> 6) < reducing) load_row(0);
  if (!VALUES && tid == 0 && a.score_dev != nullptr) a.score_dev[row] = 0.0f;
  if (KL == 0) {
    if (tid == 0) side.kstar[row] = 0;
    return;
  }
  __syncthreads();
  const float lse_f = s_lse, top = s_top;
  const double lse = (double)lse_f;

  // ---- the one pass over memory: keys to LDS, the estimated mass of the sealed blocks (single-
  //      precision exponentials, accumulated in double; the rest of 1 is the exact trailing tokens), histogram
  double part = 0.0;
  for (int base = 0; base < nb; base += ST * SBATCH) {
    if (base > 0) load_row(base);
#pragma unroll
    for (int j = 0; j < SBATCH; ++j) {
      const int i = base + j * ST + tid;
      if (i < nb) {
        float x = __expf(v[j] - lse_f);
        if (VALUES) {
          x *= e[j];
          contrib[i] = x;
        }
        part += (double)x;
        const float ranks = VALUES ? x : v[j];
        const int bin = select_bin<VALUES>(ranks, top);
        if (cached) {
          keys[i] = ord32(ranks);
          sm.bins[i] = (uint16_t)bin;
        }
        atomicAdd(&hist[bin], 1u);
      }
    }
  }
  part = wave_sum_d(part);
  if ((tid & 63) == 0) dsum[tid >> 6] = part;
  __syncthreads();
  // thread t looks at bin ST - 1 - t, so an inclusive scan over threads counts from the top bin down;
  // the bin to stop at is the one where that count first reaches KL
  {
    const uint32_t mine = hist[ST - 1 - tid];
    const uint32_t upto = block_scan_incl<uint32_t>(mine, utot, tid);
    if (upto >= (uint32_t)KL && upto - mine < (uint32_t)KL) {
      s_bin = ST - 1 - tid;
      s_found = (int)upto;
    }
  }
  __syncthreads();
  double total = 0.0;
  for (int w = 0; w < ST / 64; ++w) total += dsum[w];

  // s_first = the smallest thread (= place) for which `hit` holds; a wave's lanes are settled by ballot (an LDS minimum over
  // lanes of different values is walked lane by lane: 2.5 us where a head's first blocks cover everything)
  const auto first_of = [&](bool hit) {
    const unsigned long long m = __ballot(hit);
    if (m != 0ull && (tid & 63) == __ffsll((long long)m) - 1) atomicMin(&s_first, tid);
  };
  // Candidates into LDS in any order.  (Short code on purpose: it runs once per launch and has to be fetched first.)
  const auto collect = [&](int most, auto wanted) {
#pragma unroll 1
    for (int i = tid; (i & ~63) < nb; i += ST) {
      const unsigned long long m = __ballot(i < nb && wanted(i));
      if (m == 0ull) continue;
      int at = 0;
      if ((tid & 63) == 0) at = (int)atomicAdd(&s_cnt, (uint32_t)__popcll(m));
      at = __builtin_amdgcn_readfirstlane(at);
      const int pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, (uint32_t)at));
      if (((m >> (tid & 63)) & 1ull) && pos < most) {
        const uint32_t k = cached ? keys[i] : ord32(ranked[i]);
        cand[pos] = ((unsigned long long)k << 32) | (unsigned long long)(0xFFFFFFFFu - (uint32_t)i);
      }
    }
  };
  // ... those of bin `bin` and up: a place per wave and eight passes, not one per wave and pass
  const auto collect_bins = [&](int bin) {
    for (int base = 0; base < nb; base += ST * SBATCH) {
      uint32_t mine = 0u;
#pragma unroll
      for (int j = 0; j < SBATCH; ++j) {
        const int i = base + j * ST + tid;
        mine |= i < nb && (int)sm.bins[min(i, LDS_KEYS - 1)] >= bin ? 1u << j : 0u;
      }
      if (__ballot(mine != 0u) == 0ull) continue;
      const uint32_t n = (uint32_t)__popc(mine), upto = wave_scan_incl(n);
      uint32_t at = 0u;
      if ((tid & 63) == 63) at = atomicAdd(&s_cnt, upto);
      at = (uint32_t)__builtin_amdgcn_readlane((int)at, 63) + upto - n;
      for (; mine != 0u; mine &= mine - 1u, ++at) {
        const int i = base + (__ffs((int)mine) - 1) * ST + tid;
        if (at < (uint32_t)(MAX_K_LIMIT + CAND_SLACK))
          cand[at] = ((unsigned long long)keys[i] << 32) | (unsigned long long)(0xFFFFFFFFu - (uint32_t)i);
      }
    }
  };
  if (s_found <= KL + CAND_SLACK) {
    // ---- every block from that bin up is a candidate
    const int bin = s_bin;
    if (cached)
      collect_bins(bin);
    else
      collect(MAX_K_LIMIT + CAND_SLACK, [&](int i) { return select_bin<VALUES>(ranked[i], top) >= bin; });
  } else {
    // ---- radix selection of the KL-th largest key, 8 bits at a time from the top
    if (tid == 0) {
      s_prefix = 0u;
      s_want = (uint32_t)KL;
      s_done = 0;
    }
    for (int pass = 0; pass < 4; ++pass) {
      const int shift = 24 - 8 * pass;
      const uint32_t himask = pass == 0 ? 0u : (0xFFFFFFFFu << (shift + 8));
      if (tid < 256) hist[tid] = 0u;
      __syncthreads();
      const uint32_t prefix = s_prefix;
      const uint32_t want = s_want;
      CQA_KEY_PASS(ranked, nb, tid, cached, keys, {
        hist_add(hist, (k >> shift) & 255u, in && (k & himask) == prefix);
      })
      __syncthreads();
      const uint32_t mine = tid < 256 ? hist[255 - tid] : 0u;
      const uint32_t upto = block_scan_incl<uint32_t>(mine, utot, tid);
      if (upto >= want && upto - mine < want) {
        s_want = want - (upto - mine);               // still to take inside the chosen bin
        s_prefix = prefix | ((uint32_t)(255 - tid) << shift);
        // every block of the chosen bin is taken: its lower edge already is the threshold (with
        // distinct log-masses this happens once a bin holds a single block, usually a pass early)
        if (want - (upto - mine) == mine) s_done = 1;
      }
      __syncthreads();
      if (s_done != 0) break;
    }
    const uint32_t T = s_prefix;                   // key of the KL-th best block
    // blocks with key == T: s_want of them are needed, the ones with the lowest indices.  The last
    // histogram still holds how many there are: when all of them are wanted, which is the rule
    // unless log-masses tie exactly, no index needs to be selected.
    const bool all_ties = s_done != 0 || hist[T & 255u] == s_want;
    __syncthreads();
    if (tid == 0) {
      s_idx_prefix = all_ties ? 0xFFFFFFFFu : 0u;
      s_idx_want = s_want;
    }
    for (int pass = 0; pass < (all_ties ? 0 : 4); ++pass) {
      const int shift = 24 - 8 * pass;
      const uint32_t himask = pass == 0 ? 0u : (0xFFFFFFFFu << (shift + 8));
      if (tid < 256) hist[tid] = 0u;
      __syncthreads();
      const uint32_t prefix = s_idx_prefix;
      const uint32_t want = s_idx_want;
      CQA_KEY_PASS(ranked, nb, tid, cached, keys, {
        hist_add(hist, (((uint32_t)i) >> shift) & 255u, in && k == T && (((uint32_t)i) & himask) == prefix);
      })
      __syncthreads();
      const uint32_t mine = tid < 256 ? hist[tid] : 0u;   // ascending: the lowest indices are taken first
      const uint32_t upto = block_scan_incl<uint32_t>(mine, utot, tid);
      if (upto >= want && upto - mine < want) {
        s_idx_want = want - (upto - mine);
        s_idx_prefix = prefix | ((uint32_t)tid << shift);
      }
      __syncthreads();
    }
    __syncthreads();
    const uint32_t Tidx = s_idx_prefix;            // largest index taken among the ties
    // ---- collect the KL winners as composite keys (log-mass order, then lower index first)
    collect(MAX_K_LIMIT, [&](int i) {
      const uint32_t k = cached ? keys[i] : ord32(ranked[i]);
      return k > T || (k == T && (uint32_t)i <= Tidx);
    });
  }
  __syncthreads();
  const int nc = (int)min(s_cnt, (uint32_t)(MAX_K_LIMIT + CAND_SLACK));
  const int n = min(nc, KL);
  // ---- rank sort: a candidate's place is the number of candidates that precede it (keys are distinct)
  //      Four threads share a candidate, each against a quarter of the others.
  if (tid < 32) cand[nc + tid] = 0ull;             // precede nothing: 32 candidates per round of the four
  __syncthreads();
  for (int i = tid >> 2; i < nc; i += ST / 4) {
    const unsigned long long mine = cand[i];
    int rank = 0;
    for (int j = 0; j < nc; j += 32) {
      ulonglong2 c[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) c[u] = reinterpret_cast<const ulonglong2*>(&cand[j + 8 * (tid & 3)])[u];
#pragma unroll
      for (int u = 0; u < 4; ++u) rank += (c[u].x > mine ? 1 : 0) + (c[u].y > mine ? 1 : 0);
    }
    rank += dpp_movi<0xB1>(rank);
    rank += dpp_movi<0x4E>(rank);
    if ((tid & 3) == 0 && rank < n) sorted[rank] = mine;
  }
  __syncthreads();
  // ---- masses of the winners, best first, and their inclusive prefix sums: thread t owns place t
  const float val0 = tid < n ? from_ord32((uint32_t)(sorted[tid] >> 32)) : 0.0f;
  const double m0 = tid < n ? (VALUES ? (double)val0 : exp((double)val0 - lse)) : 0.0;
  const double upto1 = block_scan_incl<double>(m0, dtot, tid);
  if (tid < MAX_K_LIMIT) pm[tid] = upto1;
  __syncthreads();
  if (!VALUES) {
    // ---- covering prefix: C_k = rho_trail + (mass of the k best); K* never exceeds k_max, so
    //      the search stops there; then clamps and Rung-1 growth
    const double rho_trail = 1.0 - total;
    const int look = min(n, side.k_max);
    first_of(tid <= look && rho_trail + (tid > 0 ? pm[min(tid, n) - 1] : 0.0) >= (double)a.tau_cov);
    __syncthreads();
    if (tid == 0) {
      int k = s_first <= look ? s_first : nb;             // no prefix up to k_max covers tau_cov
      k = max(side.k_min, min(k, side.k_max));
      k = min(k, nb);
      k = min(k, n);
      // Rung 1 (an infinite threshold is never exceeded: its test, a chain of double-precision functions, is skipped)
      const double delta = (double)s_delta, vmax = (double)s_vmax;
      const int cap = a.eps_key == INFINITY ? 0 : min(max(side.k_limit, side.k_max), n);
      while (k < cap) {
        const double tail = total - (k > 0 ? pm[k - 1] : 0.0);
        if (!(key_term_d(delta, tail, vmax, a.mass_exp, a.key_bound_mode) > (double)a.eps_key)) break;
        k = min(max(2 * k, 1), cap);
      }
      s_k = k;
      side.kstar[row] = k;
    }
  } else {
    // ---- value selection: the blocks over the local threshold form a prefix of the ranking
    //      (count them), the hard-budget rule asks for the smallest prefix that leaves at most
    //      eps_val of the estimate; the longer of the two, capped
    __shared__ int s_over;
    if (tid == 0) s_over = 0;
    __syncthreads();
    const int over = __popcll(__ballot(tid < n && val0 > a.v_tol));
    if ((tid & 63) == 0 && over > 0) atomicAdd(&s_over, over);
    if (a.v_greedy) first_of(tid <= n && total - (tid > 0 ? pm[min(tid, n) - 1] : 0.0) <= (double)a.eps_val);
    __syncthreads();
    if (tid == 0) {
      int k = s_over;
      if (a.v_greedy) k = max(k, s_first <= n ? s_first : nb);
      k = min(k, min(n, nb));
      s_k = k;
      side.kstar[row] = k;
    }
  }
  __syncthreads();
  const int k = s_k;
  for (int i = tid; i < k; i += ST) {
    const int idx = (int)(0xFFFFFFFFu - (uint32_t)(sorted[i] & 0xFFFFFFFFull));
    side.sel[row * MAX_K_LIMIT + i] = idx;
    if (idx >= 0 && idx < nb) atomicOr(&um[idx >> 5], 1u << (idx & 31));
  }
}

__global__ __launch_bounds__(ST) void select_kernel(SelectArgs a) {
  fetch_args<sizeof(SelectArgs)>();
  __shared__ __align__(16) SelectSmem sm;
  if (blockIdx.z == 0)
    select_rows<false>(a, sm);
  else
    select_rows<true>(a, sm);
}

struct CompactArgs {
  PromMasks masks;
  int group;           // query heads per KV group
  int32_t* slot;       // [Bt][Hkv][slot_stride]
  int64_t slot_stride;
  int32_t* ulist;      // [Bt][Hkv][MAX_UNION]
  int32_t* ucount;     // [Bt][Hkv]
  int nb;
  // FP16 scratch of the layer
  int32_t* sc_map;     // [Bt][Hkv][sc_map_stride]
  int64_t sc_map_stride;
  int32_t* sc_tag;     // [Bt][Hkv][sc_cap]
  uint32_t* sc_age;    // [Bt][Hkv][sc_cap]
  int32_t* sc_have;    // [Bt][Hkv][sc_cap]
  uint32_t* sc_stats;  // [2]
  int sc_cap, sc_slots;
  uint32_t sc_step;    // stamp of this step (larger than every stamp before it, never 0)
};

// With the FP16 scratch in use (otherwise the promoted-block pass reads the masks itself: a launch less).
// One workgroup per KV group: the heads' bit masks (FP16 keys, FP16 values) -> per-block flags
// (bit 0: some head scores the block with FP16 keys, bit 1: some head attends its FP16 values,
// bits 24-27 / 28-31: which heads; 0 = neither) and the ascending list of blocks with any flag.
// Per-group promotion gives every head the union's bits.
__global__ __launch_bounds__(256) void compact_kernel(CompactArgs a) {
  fetch_args<sizeof(CompactArgs)>();
  const int tid = threadIdx.x;
  const int64_t grp = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
  int32_t* slot = a.slot + grp * a.slot_stride;
  int32_t* ulist = a.ulist + grp * MAX_UNION;
  const int words = (a.nb + 31) >> 5;
  __shared__ int itot_c[4];
  __shared__ int s_base;
  // (every flag word is zero: only listed blocks' words are ever set, and the selector has taken those of the
  // previous call's list back)
  // thread t owns the contiguous run of mask words [t wpt, (t + 1) wpt): the list comes out ascending
  constexpr int WPT_MAX = 8;             // up to 256 x 8 x 32 blocks (1M tokens) in one sweep
  const int wpt = (words + 255) >> 8;
  int base_total = 0;
  for (int w00 = 0; w00 < words; w00 += 256 * WPT_MAX) {
    const int wpt_here = min(wpt, WPT_MAX);
    PromBits m[WPT_MAX];
    int cnt = 0;
#pragma unroll
    for (int u = 0; u < WPT_MAX; ++u) {
      const int w = w00 + tid * wpt_here + u;
      m[u].k = m[u].v = 0u;
      if (u < wpt_here && w < words) m[u] = prom_bits(a.masks, grp, a.group, w, ~0u);
      cnt += __popc(m[u].k | m[u].v);
    }
    int pos = base_total + block_scan_incl<int>(cnt, itot_c, tid) - cnt;   // slot of my run's first promoted block
    if (tid == 255) s_base = pos + cnt;
#pragma unroll
    for (int u = 0; u < WPT_MAX; ++u) {
      const int w = w00 + tid * wpt_here + u;
      uint32_t bits = m[u].k | m[u].v;
      while (bits != 0u) {
        const int j = __ffs((int)bits) - 1;
        bits &= bits - 1u;
        const int blk = w * 32 + j;
        // the list cannot overflow (4 heads x MAX_K_LIMIT for keys and as many for values) but by explored blocks;
        // one that does not fit stays unpromoted
        if (pos < MAX_UNION) {
          slot[blk] = prom_flags(m[u], j);
          ulist[pos] = blk;
        }
        ++pos;
      }
    }
    __syncthreads();
    base_total = s_base;
  }
  const int s_base_final = base_total;
  if (tid == 0) a.ucount[grp] = min(s_base_final, MAX_UNION);

  // ---- FP16 scratch: which listed blocks are held on the device, and where the others go.
  // A promoted block found in the map keeps its slot (stamped with this step); a half of it (keys,
  // values) that this step needs and the slot does not hold yet is filled on the way.  The others
  // take over the least recently used slots -- found by a radix selection over the slots' stamps,
  // only in steps that miss -- never one used in this step; the pass that reads their originals
  // from the host stores them into the slot (SLOT_FILL for the keys, SLOT_VFILL for the values).
  // Misses beyond the free slots are read from the host without being kept.
  const int n = min(s_base_final, MAX_UNION);
  int32_t* map = a.sc_map + grp * a.sc_map_stride;
  int32_t* tag = a.sc_tag + grp * (int64_t)a.sc_cap;
  uint32_t* age = a.sc_age + grp * (int64_t)a.sc_cap;
  int32_t* have = a.sc_have + grp * (int64_t)a.sc_cap;
  __shared__ int s_hits, s_part, s_nmiss, s_elig;
  __shared__ int misslist[SC_MAX_SLOTS];
  if (tid == 0) {
    s_hits = 0;
    s_part = 0;
    s_nmiss = 0;
    s_elig = 0;
  }
  __syncthreads();
  for (int i = tid; i < n; i += 256) {
    const int blk = ulist[i];
    const int f = slot[blk];
    const int need = f & (SLOT_KEYS | SLOT_VALUES);
    if (need) {
      const int m = map[blk];
      if (m > 0 && m <= a.sc_slots && tag[m - 1] == blk) {
        const int missing = need & ~have[m - 1];
        age[m - 1] = a.sc_step;
        have[m - 1] |= need;
        slot[blk] = f | (m << SLOT_SC_SHIFT) | ((missing & SLOT_KEYS) ? SLOT_FILL : 0) |
                    ((missing & SLOT_VALUES) ? SLOT_VFILL : 0);
        atomicAdd(missing ? &s_part : &s_hits, 1);
      } else {
        const int k = atomicAdd(&s_nmiss, 1);
        if (k < SC_MAX_SLOTS) misslist[k] = blk;
      }
    }
  }
  __syncthreads();
  const int nmiss = min(s_nmiss, SC_MAX_SLOTS);
  if (tid == 0) {
    atomicAdd(a.sc_stats + 0, (uint32_t)s_hits);
    atomicAdd(a.sc_stats + 1, (uint32_t)(s_nmiss + s_part));
  }
  if (nmiss == 0) return;
  // The `usable` least recently used slots, ties to the lower slot index: radix selection over
  // the 32-bit stamps of the slots that this step does not use (four 8-bit passes: histogram,
  // scan, descend), then two scans in slot order rank the chosen slots.  Thread t owns slots
  // 4t .. 4t+3.
  __shared__ uint32_t hist[256];
  __shared__ uint32_t s_prefix, s_need;
  __shared__ int itot[4];
  __shared__ uint32_t utot[4];
  uint32_t st4[4];
  bool el4[4];
  int elig = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int i = tid * 4 + j;
    st4[j] = i < a.sc_slots ? age[i] : 0xFFFFFFFFu;
    el4[j] = i < a.sc_slots && st4[j] != a.sc_step;
    elig += el4[j] ? 1 : 0;
  }
  atomicAdd(&s_elig, elig);
  __syncthreads();
  const int usable = min(nmiss, s_elig);
  if (usable == 0) return;
  if (tid == 0) {
    s_prefix = 0u;
    s_need = (uint32_t)usable;
  }
  for (int shift = 24; shift >= 0; shift -= 8) {
    hist[tid] = 0u;
    __syncthreads();
    const uint32_t prefix = s_prefix, need = s_need;
    const uint32_t himask = shift == 24 ? 0u : (0xFFFFFFFFu << (shift + 8));
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (el4[j] && (st4[j] & himask) == prefix) atomicAdd(&hist[(st4[j] >> shift) & 255u], 1u);
    __syncthreads();
    const uint32_t mine = hist[tid];
    const uint32_t upto = block_scan_incl<uint32_t>(mine, utot, tid);
    if (upto >= need && upto - mine < need) {      // the bin where the count first reaches `need`
      s_need = need - (upto - mine);
      s_prefix = prefix | ((uint32_t)tid << shift);
    }
    __syncthreads();
  }
  const uint32_t T = s_prefix;          // stamp of the last slot taken
  const int need_eq = (int)s_need;      // how many slots with exactly that stamp are taken
  int eq = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) eq += (el4[j] && st4[j] == T) ? 1 : 0;
  int eq_before = block_scan_incl<int>(eq, itot, tid) - eq;
  bool take[4];
  int nt = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const bool is_eq = el4[j] && st4[j] == T;
    take[j] = el4[j] && (st4[j] < T || (is_eq && eq_before < need_eq));
    eq_before += is_eq ? 1 : 0;
    nt += take[j] ? 1 : 0;
  }
  int rank = block_scan_incl<int>(nt, itot, tid) - nt;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (!take[j]) continue;
    if (rank < usable) {
      const int v = tid * 4 + j;
      const int blk = misslist[rank];
      const int old = tag[v];
      if (old >= 0 && old < a.nb && map[old] == v + 1) map[old] = 0;
      tag[v] = blk;
      map[blk] = v + 1;
      age[v] = a.sc_step;
      const int need = slot[blk] & (SLOT_KEYS | SLOT_VALUES);
      have[v] = need;
      slot[blk] |= ((v + 1) << SLOT_SC_SHIFT) | ((need & SLOT_KEYS) ? SLOT_FILL : 0) |
                   ((need & SLOT_VALUES) ? SLOT_VFILL : 0);
    }
    ++rank;
  }
}

struct AdaptiveReduceArgs {
  ReduceArgs ra{};
  const float* lm8;      // [Bt][Hq][nb]
  const float* lmx;      // [Bt][Hq][nb]
  const int32_t* slot;   // [Bt][Hkv][slot_stride]
  int64_t slot_stride;
  const float* first;    // [Bt][Hq][4]
  const ScanPart* scan;  // [Bt][Hq][parts]
  int parts;
  float* alpha_out;      // [Bt][Hq]
  const float* score_dev;  // [Bt][Hq] canary deviations, or null
  // The promoted-block pass's positive partial sets.  Those outside [pos_set0, pos_set1) -- the one pass over all sealed
  // blocks and the negated sets that take the listed blocks back out of it -- contribute their output
  // accumulators only.  A difference of two nearly equal sums would leave the certificate's
  // scalars with the rounding of the large terms, so these come from the scan over the block log-masses.
  int pos_set0, pos_set1;
  const int32_t* ulist;  // [Bt][Hkv][MAX_UNION] listed blocks of the group
  const int32_t* ucount; // [Bt][Hkv]
};

// One workgroup per (batch, query head): eight waves merge the partial sets of the pass over all blocks and of the
// promoted-block pass, one attends the trailing tokens, one prepares the key term and adds up the sums' parts, all of them look through the list of promoted blocks for
// the best under either ranking, and the first joins the results.  (What the other blocks add up to has been summed
// beside the promoted-block pass.)
// Bound by latency: 128K, 32 heads 9.3 -> 6.4 us, 4K 8.2 -> 6.7 (with the scan over all log-masses in this launch, before).
constexpr int AR_WAVES = RED_WAVES + 2;
constexpr int ART = 64 * AR_WAVES;
struct RankBest {
  float x[AR_WAVES], e[AR_WAVES];   // by FP16 / by INT8 log-mass
  int ix[AR_WAVES], ie[AR_WAVES];
};
// the best of the waves' results, in every lane of a wave
__device__ __forceinline__ void rank_join(const RankBest& r, float& x, int& ix, float& e, int& ie) {
  const int l = threadIdx.x & 63;
  const bool on = l < AR_WAVES;
  x = on ? r.x[l] : -INFINITY;
  e = on ? r.e[l] : -INFINITY;
  ix = on ? r.ix[l] : -1;
  ie = on ? r.ie[l] : -1;
  wave_best(x, ix);
  wave_best(e, ie);
}
__global__ __launch_bounds__(ART) void adaptive_reduce_kernel(AdaptiveReduceArgs a) {
  fetch_args<sizeof(AdaptiveReduceArgs)>();
  const int tid = threadIdx.x, l = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hq = blockIdx.x, b = blockIdx.y;
  const ReduceArgs& ra = a.ra;
  const int64_t row = (int64_t)b * ra.n_q + hq;
  const int shift = group_shift(ra.n_q, ra.n_kv);
  const int64_t grp = (int64_t)b * ra.n_kv + (hq >> shift);
  const float* l8 = a.lm8 + row * ra.nb;
  const float* lx = a.lmx + row * ra.nb;
  const int32_t* slot = a.slot + grp * a.slot_stride;
  const int32_t* ulist = a.ulist + grp * MAX_UNION;
  const int kbit = 1 << (SLOT_HK_SHIFT + (hq & ((1 << shift) - 1)));   // this head scores the block with FP16 keys
  const float lse8 = a.first[row * 4], delta = a.first[row * 4 + 1];
  const int n_list = min(a.ucount[grp], MAX_UNION);
  int blk = ulist[tid];                    // valid for tid < n_list

  __shared__ __align__(16) ReduceSmem sm;
  __shared__ RankBest rb;
  __shared__ ScanPart sums;
  if (w < RED_WAVES) {
    float2 o2;
    const OctState st = merge_sets(ra.partials + row * ra.pstride * PART_FLOATS, 8 * w, 8 * RED_WAVES, ra.nsplit, a.pos_set0,
                                   a.pos_set1, o2);
    store_state(st, o2, sm.sc[w], sm.o[w]);
  } else if (w == RED_WAVES) {
    trail_part(ra, b, hq, sm);
  } else {
    key_part(ra, delta, sm);
    ScanPart t{0.0, 0.0, 0.0, -INFINITY, 0.0f};
    for (int i = l; i < a.parts; i += 64) {
      const ScanPart x = a.scan[row * a.parts + i];
      t.alpha += x.alpha;
      t.l8u += x.l8u;
      t.ev8u += x.ev8u;
      t.top = fmaxf(t.top, x.top);
      t.maxc8 = fmaxf(t.maxc8, x.maxc8);
    }
    if (a.parts > 1) {
      t.alpha = wave_sum_d(t.alpha);
      t.l8u = wave_sum_d(t.l8u);
      t.ev8u = wave_sum_d(t.ev8u);
      t.top = wave_max(t.top);
      t.maxc8 = wave_max(t.maxc8);
    }
    if (l == 0) sums = t;
  }
  float best_x = -INFINITY, best_8 = -INFINITY;
  int ix = -1, i8 = -1;
  for (int i = tid; i < n_list; i += ART) {
    if (i != tid) blk = ulist[i];
    if (blk < 0 || blk >= ra.nb || !(slot[blk] & kbit)) continue;
    const float vx = lx[blk], v8 = l8[blk];
    if (vx > -INFINITY) best_merge(best_x, ix, vx, blk);   // a block without a log-mass (not a number, for a
    if (v8 > -INFINITY) best_merge(best_8, i8, v8, blk);   // query that is none) tops no ranking
  }
  wave_best(best_x, ix);
  wave_best(best_8, i8);
  if (l == 0) {
    rb.x[w] = best_x;
    rb.ix[w] = ix;
    rb.e[w] = best_8;
    rb.ie[w] = i8;
  }
  __syncthreads();
  // ---- ranking check (the paper's "Ranking-Consistency Check" with its boundary verification)
  //      at depth r: the r best promoted blocks under the FP16 and under the INT8 log-masses must
  //      be the same blocks in the same order, and no unpromoted block may reach the r-th FP16
  //      log-mass with its upper-bounded one.  Depth 1 is what the look through the list has found; each further
  //      place is one more arg-max over the group's listed blocks (a few dozen, held in registers),
  //      restricted to what comes after the previous place in the order (larger log-mass first,
  //      equal log-masses by lower index).  Fewer promoted blocks than r: the depth is their number.
  float top_x, top_8;
  int top_ix, top_i8;
  rank_join(rb, top_x, top_ix, top_8, top_i8);
  bool disagree = top_ix >= 0 && top_ix != top_i8;
  float kth_x = top_x;
  const int depth = min(ra.tol.rank_depth, MAX_RANK_DEPTH);
  if (depth > 1 && top_ix >= 0) {          // uniform over the workgroup
    constexpr int CAND = (MAX_UNION + ART - 1) / ART;
    float cx[CAND], c8[CAND];
    int cb[CAND];
#pragma unroll
    for (int j = 0; j < CAND; ++j) {
      const int i = j * ART + tid;
      const int c = i < n_list ? ulist[i] : -1;
      const bool keyp = c >= 0 && c < ra.nb && (slot[c] & kbit);
      cb[j] = keyp ? c : -1;
      cx[j] = keyp ? lx[c] : 0.0f;
      c8[j] = keyp ? l8[c] : 0.0f;
    }
    float px = top_x, p8 = top_8;
    int pix = top_ix, pi8 = top_i8;
    for (int k = 1; k < depth; ++k) {
      float bx = -INFINITY, b8 = -INFINITY;
      int jx = -1, j8 = -1;
#pragma unroll
      for (int j = 0; j < CAND; ++j) {
        if (cb[j] < 0) continue;
        if ((cx[j] < px || (cx[j] == px && cb[j] > pix)) &&
            (jx < 0 || cx[j] > bx || (cx[j] == bx && cb[j] < jx))) {
          bx = cx[j];
          jx = cb[j];
        }
        if ((c8[j] < p8 || (c8[j] == p8 && cb[j] > pi8)) &&
            (j8 < 0 || c8[j] > b8 || (c8[j] == b8 && cb[j] < j8))) {
          b8 = c8[j];
          j8 = cb[j];
        }
      }
      wave_best(bx, jx);
      wave_best(b8, j8);
      __syncthreads();                      // the previous place has been read
      if (l == 0) {
        rb.x[w] = bx;
        rb.ix[w] = jx;
        rb.e[w] = b8;
        rb.ie[w] = j8;
      }
      __syncthreads();
      float nx, n8;
      int nix, ni8;
      rank_join(rb, nx, nix, n8, ni8);
      if (nix < 0) break;                   // fewer promoted blocks than the depth (uniform)
      disagree = disagree || nix != ni8;
      kth_x = nx;
      px = nx;
      pix = nix;
      p8 = n8;
      pi8 = ni8;
    }
  }
  if (w != 0) return;
  const float tmax = sums.top;
  const bool has_tail = tmax > -INFINITY;
  AdaptiveIn ad;
  ad.alpha = (float)sums.alpha;
  ad.delta = delta;
  ad.top_block = top_ix;
  ad.top_fp16 = top_ix >= 0 ? top_x : -INFINITY;
  ad.kth_fp16 = top_ix >= 0 ? kth_x : -INFINITY;
  ad.tail_ub = has_tail ? tmax + delta : -INFINITY;
  const bool boundary = top_ix >= 0 && has_tail && tmax + delta + ra.tol.eps_guard > kth_x;
  ad.rank_fail = (disagree || boundary) ? 1 : 0;
  ad.precond = (a.score_dev != nullptr && a.score_dev[row] > delta + ra.tol.eps_guard) ? 1 : 0;
  ad.L8u = (float)sums.l8u;
  ad.EV8u = (float)sums.ev8u;
  ad.maxc8 = sums.maxc8;
  ad.lse8 = lse8;
  if (l == 0) a.alpha_out[row] = ad.alpha;
  float2 o2;
  const OctState st = merge_lds<RED_WAVES>(sm.sc[0], 12, sm.o[0], D, RED_WAVES, o2);
  finish_head(ra, b, hq, head_state(st, o2), trail_of(sm), key_of(sm), &ad);
}

}  // namespace

int32_t launch_adaptive(Cache* c, int layer, const __half* q, const cqa_tolerances& tol,
                        const cqa_selector& sel, float* O, cqa_head_cert* cert, uint32_t* flags,
                        uint32_t* flags_mirror, uint32_t mirror_tag, hipStream_t st, uint32_t* raised,
                        uint32_t raised_tag) {
  // quantised-query scoring: the pass over all blocks scores on the INT8 matrix cores, the
  // promoted-block pass reproduces those scores for the blocks (and heads) that stay in INT8
  if (tol.int8_query != 0 && c->variant != 0) return CQA_ERR_UNSUPPORTED;
  const int bt = c->desc.batch, hq = c->desc.n_q_heads, hkv = c->desc.n_kv_heads;
  const int g = hq / hkv;
  const int64_t len = c->length[layer];
  const int64_t nb = len / BLK;
  const int r = (int)(len % BLK);
  AdaptiveWs& w = c->ad;

  // ---- 1. one pass over all sealed blocks in INT8 / INT4 (the ordinary certified pass): block
  //         log-masses, eta_b and the partial sets the promoted-block pass will correct.  Every
  //         threshold is off: its certificate only feeds the selector (lse, Delta_h, V_max) and
  //         is overwritten below.
  int nsplit = 0, wpb = 0;
  split_geometry(c, nb, &nsplit, &wpb);
  const int total = nsplit + 2 * PROM_SPLITS;
  cqa_tolerances loose = tol;
  loose.eps_total = loose.eps_key = loose.eps_val = loose.v_tol = INFINITY;
  loose.rank_depth = 0;
  loose.force_flags = 0;
  if (nb == 0) {
    // nothing sealed: the exact trailing tokens are the answer, with the caller's thresholds
    return launch_certified(c, layer, q, tol, O, cert, flags, flags_mirror, mirror_tag, nullptr, st, nullptr, nullptr, 0,
                            nullptr, nullptr, raised, raised_tag);
  }
  ReduceArgs first{};   // its reduction is left to the selector
  int32_t rc = launch_certified(c, layer, q, loose, O, cert, flags, nullptr, 0u, w.lm8, st, nullptr, nullptr,
                                total, w.eta_blk, nullptr, nullptr, 0u, &first);
  if (rc != CQA_OK) return rc;

  // ---- 2. selection per head (+ Rung 1), union bit mask per group
  const bool values = sel.v_limit > 0;   // value promotion ranks the estimated contributions p_b eta_b
  SelectArgs sa{};
  sa.side[0] = {w.sel, w.kstar, w.umask, sel.k_min, sel.k_max, sel.k_limit};
  sa.side[1] = {w.vsel, w.vcount, w.vmask, 0, sel.v_limit, sel.v_limit};
  sa.lm8 = w.lm8;
  sa.eta_blk = w.eta_blk;
  sa.contrib = w.contrib;
  sa.ra = first;
  sa.first = w.first;
  sa.slot = w.slot;
  sa.slot_stride = c->nq_cap * 4;
  sa.ulist = w.ulist;
  sa.ucount = w.ucount;
  sa.mask_words = w.mask_words;
  sa.nb = (int)nb;
  sa.n_q = hq;
  sa.n_kv = hkv;
  sa.tau_cov = sel.tau_cov;
  sa.eps_key = tol.eps_key;
  sa.mass_exp = tol.mass_exp;
  sa.key_bound_mode = tol.key_bound_mode;
  sa.v_tol = tol.v_tol;
  sa.eps_val = tol.eps_val;
  sa.v_greedy = sel.v_greedy;
  sa.score_dev = sel.canary ? w.score_dev : nullptr;
  hipLaunchKernelGGL(select_kernel, dim3(hq, bt, values ? 2 : 1), dim3(ST), 0, st, sa);
  CQA_HIP(hipGetLastError());

  // ---- 3. with the FP16 scratch, flag words and ordered list per group
  const double thr = (double)sel.explore_frac * 4294967296.0;
  const uint32_t explore_threshold = sel.explore_frac > 0.0f ? (uint32_t)std::min(thr, 4294967295.0) : 0u;
  const PromMasks masks{w.umask, values ? w.vmask : nullptr, w.mask_words, (int)nb, sel.per_head, explore_threshold, sel.explore_seed};
  CompactArgs ca{};
  ca.masks = masks;
  ca.group = g;
  ca.slot = w.slot;
  ca.slot_stride = c->nq_cap * 4;
  ca.ulist = w.ulist;
  ca.ucount = w.ucount;
  ca.nb = (int)nb;
  const int64_t layer_head0 = head_index(c, layer, 0, 0);
  ca.sc_slots = w.sc_slots;
  if (w.sc_slots > 0) {
    w.sc_step += 1u;
    ca.sc_map = w.sc_map + layer_head0 * c->nb_cap;
    ca.sc_map_stride = c->nb_cap;
    ca.sc_tag = w.sc_tag + layer_head0 * w.sc_cap;
    ca.sc_age = w.sc_age + layer_head0 * w.sc_cap;
    ca.sc_have = w.sc_have + layer_head0 * w.sc_cap;
    ca.sc_stats = w.sc_stats;
    ca.sc_cap = w.sc_cap;
    ca.sc_step = w.sc_step;
    hipLaunchKernelGGL(compact_kernel, dim3(hkv, bt), dim3(256), 0, st, ca);
    CQA_HIP(hipGetLastError());
  }

  // ---- 4. promoted-block pass: the listed blocks once more with the originals their flags ask
  //         for (positive sets) and once as the first pass saw them (negated sets)
  ReduceArgs ra{};
  ra.partials = c->partials;
  ra.q = q;
  ra.trail_k = c->trail_k + layer_head0 * BLK * D;
  ra.trail_v = c->trail_v + layer_head0 * BLK * D;
  ra.O = O;
  ra.cert = cert;
  ra.flags = flags;
  ra.flags_mirror = flags_mirror;
  ra.mirror_tag = mirror_tag;
  ra.raised = raised;
  ra.raised_tag = raised_tag;
  ra.tol = tol;
  ra.nsplit = total;
  ra.pstride = total;
  ra.nb = (int)nb;
  ra.r = r;
  ra.n_q = hq;
  ra.n_kv = hkv;
  DecodeArgs a{};   // every field starts null / zero
  a.t1 = c->t1 + layer_head0 * c->nq_cap * QUAD_BYTES;
  a.sigmax = c->sigmax + layer_head0;
  a.q = q;
  a.partials = c->partials;
  a.blk_logmass = w.lmx;
  a.nq_cap = c->nq_cap;
  a.nb = (int)nb;
  a.nsplit = nsplit;
  a.pstride = total;
  a.n_q = hq;
  a.n_kv = hkv;
  a.sc_k = w.sc_slots > 0 ? w.sc_k + layer_head0 * w.sc_cap * BLK * D : nullptr;
  a.sc_v = w.sc_slots > 0 ? w.sc_v + layer_head0 * w.sc_cap * BLK * D : nullptr;
  a.sc_cap = w.sc_cap;
  a.t2_k = c->t2_k + layer_head0 * c->desc.max_tokens * D;
  a.t2_v = c->t2_v + layer_head0 * c->desc.max_tokens * D;
  a.eta_out = nullptr;
  a.score_dev = sel.canary ? w.score_dev : nullptr;
  a.int8_query = tol.int8_query;
  a.max_tokens = c->desc.max_tokens;
  a.split0 = nsplit;
  PromArgs pa{};
  pa.masks = masks;
  if (w.sc_slots > 0) pa.masks.umask = nullptr;
  pa.slot = w.slot;
  pa.ulist = w.ulist;
  pa.ucount = w.ucount;
  pa.lm8 = w.lm8;
  pa.eta = w.eta_blk;
  pa.first = w.first;
  pa.scan = w.scan;
  pa.groups = bt * hkv;
  pa.parts = (int)scan_parts(nb);
  // Order of the workgroups.  Where not all are resident at once (taking two to a compute unit), the summing ones would keep the
  // link idle while they hold a place that a workgroup with originals to fetch could have, so they come last: 128 groups of
  // 4000 tokens 2291 -> 2263 us a step.  With somewhat more than one to a compute unit, a few compute units get two.  Group by
  // group that is, on some, two that fetch originals, which take the longer the more they fetch; so the order wraps
  // round: the surplus are negated sets, sharing with negated sets.  Up to one in eight more, that is; beyond, so many share
  // that it evens out.  Steps of 20000 tokens, group by group, wrapped, sums last, 4 heads per group: 8 groups, 512 blocks a head
  // 714.6, 692.1, 692.7, few blocks 176.2, 178.8, 177.5; 9 groups 789.1, 773.4, 796.7 and 182.5, 187.3, 187.3; 11 groups 941.1,
  // 939.1, 942.5 and 224.8, 222.8, 227.1; 14 groups 1172.9, 1186.2, 1174.6 and 265.6, 267.6, 269.6; 8 groups of 128K, 128 blocks a
  // head 386.5, 377.0, 376.2, few blocks 92.6, 92.5, 94.6.
  int64_t wgs = (int64_t)(2 * PROM_SPLITS + g * pa.parts) * pa.groups;
  // With the FP16 scratch, originals mostly lie on the device and the sums are the longer part: last there (512
  // slots, 8 groups of 4000 tokens: group by group 51.1, wrapped 54.0, last 50.2).
  const bool many = wgs > 2 * c->n_cu;
  pa.order = many ? PROM_SUMS_LAST
                  : (8 * wgs > 9 * (int64_t)c->n_cu || wgs <= c->n_cu ? PROM_BY_GROUP : (w.sc_slots > 0 ? PROM_SUMS_LAST : PROM_WRAPPED));
  // Sums that come last run while nothing is fetched any more, so for many groups of short contexts a workgroup takes a group's
  // heads, a wave each: 64 x 8 groups, 4 heads, of 500 tokens 1301.5 -> 1272.8 us, of 550 1421.5 -> 1389.7, of 700 1738.7 -> 1718.6,
  // of 1300 3187.0 -> 3175.5; level from 10000 tokens on, which is where a wave takes more than a trip.
  if (many && nb <= SUM_WAVE_BLOCKS) {
    pa.sum_waves = 1;
    wgs = (int64_t)(2 * PROM_SPLITS + 1) * pa.groups;
  }
  // Lists that reach fewer than eight of a group's workgroups leave dies of the chip without any (a group has a multiple of
  // eight, so the same splits of all groups lie on the same die), so each group's list starts as many workgroups
  // away as it can reach.  64 x 8 groups, 4 heads, of 50 tokens 381.6 -> 218.7 us a step, of 120 442.3 -> 401.6, of 250 704.1 -> 681.4,
  // of 400 1149.9 -> 1058.3, of 460 1221.3 -> 1189.0 (but 32 x 16 of 200 559.8 -> 565.2); 128 groups of 120 126.9 -> 114.2.  Where
  // eight or more are reached it gains nothing: 700 tokens 1734, 1754; 850 2128, 2140.  16 groups of 400 72.1, 74.7.
  pa.turn = nb <= 4 * 7 && pa.groups >= 32 ? (int)((nb + 3) / 4) : 0;
  pa.ahead = (int)std::min<int64_t>(std::max<int64_t>(wgs - c->n_cu, 0), (int64_t)PROM_SPLITS * pa.groups);
  const unsigned gx = (unsigned)std::min<int64_t>(wgs, 1 << 22);   // (a grid dimension holds fewer than 2^32 threads)
  rc = launch_promoted_pass(a, pa, g, dim3(gx, (unsigned)((wgs + gx - 1) / gx)), st);
  if (rc != CQA_OK) return rc;

  // ---- 5. merge, certificate with the achieved tail, ranking check
  AdaptiveReduceArgs ar{};
  ar.ra = ra;
  ar.lm8 = w.lm8;
  ar.lmx = w.lmx;
  ar.slot = w.slot;
  ar.slot_stride = c->nq_cap * 4;
  ar.alpha_out = w.alpha;
  ar.score_dev = sel.canary ? w.score_dev : nullptr;
  ar.first = w.first;
  ar.scan = w.scan;
  ar.parts = pa.parts;
  ar.pos_set0 = nsplit;
  ar.pos_set1 = nsplit + PROM_SPLITS;
  ar.ulist = w.ulist;
  ar.ucount = w.ucount;
  hipLaunchKernelGGL(adaptive_reduce_kernel, dim3(hq, bt), dim3(ART), 0, st, ar);
  CQA_HIP(hipGetLastError());
  return CQA_OK;
}

}  // namespace cqa
