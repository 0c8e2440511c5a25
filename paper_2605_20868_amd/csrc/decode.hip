// Certified decode: split-K pass over Tier-1 and the cross-split reduction.
//
// What is computed (the paper's Algorithm 1 with no promoted blocks, its
// scaled-query scoring identity, and its two-term bound):
//   per sealed block b:  q~ = q (.) sigma^(b),  c_b = q . z^(b),
//                        s_t = (q~ . code_t + c_b) / sqrt(d),
//                        m_b = max_t s_t,  S_b = sum_t exp(s_t - m_b),  l_b = m_b + log S_b,
//                        Delta_b = (1 / (2 sqrt d)) sum_c |q_c| sigma_c^(b);
//   FP32 online softmax (m, l, o) with v_hat = code * scale + offset;
//   alongside it  sum_b rho_b eta_b  (value term),  max_b rho_b eta_b,
//   Delta_h = max_b Delta_b,  V_max = max_b nu_b,  and the two largest l_b;
//   the reduction merges the splits, attends the trailing FP16 tokens exactly and
//   evaluates  E_key = 2 V_max min(tanh Delta_h, min{1, e^{c Delta_h} alpha_hat}(e^{2 Delta_h} - 1)),
//   E_val = sum_b rho_b eta_b  and the flag word.
#include <algorithm>
#include <mutex>

#include "cqa_internal.h"
#include "reduce_inl.h"

namespace cqa {

// The share of workgroup psplit in its KV group's list of promoted blocks, which is dealt in fours: positions 4 psplit .. + 3, and
// every 4 * PROM_SPLITS further, to s_blk (block) and s_pf (flag word); returns the list's length.  The list comes from the
// selection masks (every workgroup walks them, one, `write`, also stores list and flag words for the reduction),
// or, when the FP16 scratch is in use, is there already.  As a launch of its own this took 5 - 10 us.
constexpr int PROM_SHARE = MAX_UNION / PROM_SPLITS;
__device__ __forceinline__ int prom_list(const DecodeArgs& a, const PromArgs& p, int64_t grp, int group, int psplit, bool write,
                                         int* s_blk, int* s_pf) {
  const int tid = threadIdx.x;
  int32_t* const slot = p.slot + grp * (a.nq_cap * 4);
  int32_t* const ulist = p.ulist + grp * MAX_UNION;
  if (p.masks.umask == nullptr) {
    const int n = min(p.ucount[grp], MAX_UNION);
    const int pos = (tid >> 2) * (4 * PROM_SPLITS) + psplit * 4 + (tid & 3);
    if (pos < n) {
      const int blk = ulist[pos];
      s_blk[tid] = blk;
      s_pf[tid] = blk >= 0 && blk < a.nb ? slot[blk] : 0;
    }
    __syncthreads();
    return n;
  }
  __shared__ int s_tot[4], s_base;
  const int words = (a.nb + 31) >> 5;
  // a thread takes a word, or a half, a quarter, an eighth of one while there are threads: set bits are walked one by one
  int per = 0;                          // log2 of the pieces per word
  while (per < 3 && (words << (per + 1)) <= 256) ++per;
  const int bits = 32 >> per, pieces = words << per;
  int total = 0;
  for (int p0 = 0; p0 < pieces; p0 += 256) {
    const int piece = p0 + tid, word = piece >> per, off = (piece & ((1 << per) - 1)) * bits;
    PromBits m;
    m.k = m.v = 0u;
    if (piece < pieces) m = prom_bits(p.masks, grp, group, word, (bits == 32 ? ~0u : (1u << bits) - 1u) << off);
    uint32_t any = m.k | m.v;
    const int cnt = __popc(any);
    const int upto = total + block_scan_incl<int>(cnt, s_tot, tid);
    if (tid == 255) s_base = upto;
    // the list cannot overflow (4 heads x MAX_K_LIMIT for keys and as many for values) but by explored
    // blocks; one that does not fit stays unpromoted
    for (int pos = upto - cnt; any != 0u; any &= any - 1u, ++pos) {
      const bool mine = ((pos >> 2) & (PROM_SPLITS - 1)) == psplit;
      if (pos >= MAX_UNION || !(mine || write)) continue;
      const int j = __ffs((int)any) - 1, blk = word * 32 + j;
      const int f = prom_flags(m, j);
      if (mine) {
        const int at = (pos / (4 * PROM_SPLITS)) * 4 + (pos & 3);
        s_blk[at] = blk;
        s_pf[at] = f;
      }
      if (write) {
        slot[blk] = f;
        ulist[pos] = blk;
      }
    }
    __syncthreads();
    total = s_base;
  }
  total = min(total, MAX_UNION);
  if (write && tid == 0) p.ucount[grp] = total;
  return total;
}

// What blocks SCAN_PART part .. + SCAN_PART - 1 left in INT8 add up to for one head, by one workgroup beside the promoted-block
// pass: 128K tokens are one part, which runs under the pass's own time.  (One workgroup per head at any length was the
// longest thing in the launch beyond that: 1 KV head of 1M tokens 67 us where the pass takes 5, the step 162.7 -> 107.2 us
// with the sums in parts; 4 x 4 heads of 512K 173.1 -> 149.5.)
// WAVES: by one wave, and one workgroup takes all heads of the group (at most SUM_WAVE_BLOCKS blocks, fewer than a list holds).
template <bool WAVES>
__device__ __forceinline__ void prom_scan(const DecodeArgs& a, const PromArgs& p, int64_t grp, int group, int h, int part, int64_t row) {
  constexpr int T = WAVES ? 64 : 256;
  static_assert(SUM_WAVE_BLOCKS <= 64 * 32 && SUM_WAVE_BLOCKS <= MAX_UNION, "a word per lane, and no list that overflows");
  const int tid = threadIdx.x & (T - 1);
  const int32_t* const slot = p.slot + grp * (a.nq_cap * 4);
  const float* l8 = p.lm8 + row * a.nb;
  const float* eta = p.eta + grp * a.nb;
  const float lse8 = p.first[row * 4];
  const int kbit = 1 << (SLOT_HK_SHIFT + h);
  __shared__ uint32_t s_key_all[SCAN_PART / 32], s_any_all[SCAN_PART / 32];   // key-promoted for the head, listed
  uint32_t* const s_key = s_key_all + (WAVES ? 64 * h : 0);
  uint32_t* const s_any = s_any_all + (WAVES ? 64 * h : 0);
  __shared__ double s_sum[4][3];
  __shared__ float s_max[4][2];
  __shared__ int s_scan[4], s_total;
  const int b0 = part * SCAN_PART, b1 = min(b0 + SCAN_PART, a.nb);
  if (p.masks.umask != nullptr) {
    // blocks listed before this part: they matter only where the list can overflow, which takes explored blocks
    int listed = 0;
    if (!WAVES && p.masks.explore_threshold != 0u && part > 0) {
      int mine = 0;
      for (int w0 = tid; w0 < b0 >> 5; w0 += 256) {
        const PromBits m = prom_bits(p.masks, grp, group, w0, ~0u);
        mine += __popc(m.k | m.v);
      }
      const int upto = block_scan_incl<int>(mine, s_scan, tid);
      if (tid == 255) s_total = upto;
      __syncthreads();
      listed = s_total;
    }
    PromBits m;
    m.k = m.v = m.kh[0] = m.kh[1] = m.kh[2] = m.kh[3] = 0u;
    if (b0 + tid * 32 < b1) m = prom_bits(p.masks, grp, group, (b0 >> 5) + tid, ~0u);
    uint32_t any = m.k | m.v;
    if (!WAVES) {
      const int upto = listed + block_scan_incl<int>(__popc(any), s_scan, tid);
      // what does not fit the list stays unpromoted: the highest blocks
      for (int over = upto - MAX_UNION; over > 0 && any != 0u; --over) any &= ~(0x80000000u >> __clz((int)any));
    }
    const uint32_t keys = h == 0 ? m.kh[0] : (h == 1 ? m.kh[1] : (h == 2 ? m.kh[2] : m.kh[3]));
    s_key[tid] = keys & any;
    s_any[tid] = any;
    if (WAVES) wave_sync(); else __syncthreads();
  }
  float tail_max = -INFINITY, maxc8 = 0.0f;
  double tail_mass = 0.0, l8u = 0.0, ev8u = 0.0;
  for (int base = b0; base < b1; base += T * 8) {
    float b8[8], be[8];
    int bs[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int i = base + j * T + tid;
      const bool in = i < b1;
      b8[j] = in ? l8[i] : 0.0f;
      be[j] = in ? eta[i] : 0.0f;
      if (p.masks.umask != nullptr) {
        const int wd = in ? (i - b0) >> 5 : 0;
        bs[j] = !in || ((s_key[wd] >> (i & 31)) & 1u) ? kbit : (int)((s_any[wd] >> (i & 31)) & 1u);
      } else {
        bs[j] = in ? slot[i] : kbit;
      }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (bs[j] & kbit) continue;            // key-promoted for this head (or past the end)
      const float mass = expf(b8[j] - lse8);
      tail_max = fmaxf(tail_max, b8[j]);
      tail_mass += (double)mass;
      if (bs[j] == 0) {
        // not listed: the promoted-block pass does not revisit it, it keeps its INT8 mass and its eta_b
        l8u += (double)mass;
        ev8u += (double)(mass * be[j]);
        maxc8 = fmaxf(maxc8, mass * be[j]);
      }
    }
  }
  const int w = WAVES ? 0 : tid >> 6;
  tail_mass = wave_sum_d(tail_mass);
  l8u = wave_sum_d(l8u);
  ev8u = wave_sum_d(ev8u);
  tail_max = wave_max(tail_max);
  maxc8 = wave_max(maxc8);
  if (WAVES) {
    if (tid == 0) p.scan[row] = ScanPart{tail_mass, l8u, ev8u, tail_max, maxc8};
    return;
  }
  if ((tid & 63) == 0) {
    s_sum[w][0] = tail_mass;
    s_sum[w][1] = l8u;
    s_sum[w][2] = ev8u;
    s_max[w][0] = tail_max;
    s_max[w][1] = maxc8;
  }
  __syncthreads();
  if (tid == 0) {
    ScanPart t;
    t.alpha = s_sum[0][0] + s_sum[1][0] + s_sum[2][0] + s_sum[3][0];
    t.l8u = s_sum[0][1] + s_sum[1][1] + s_sum[2][1] + s_sum[3][1];
    t.ev8u = s_sum[0][2] + s_sum[1][2] + s_sum[2][2] + s_sum[3][2];
    t.top = fmaxf(fmaxf(s_max[0][0], s_max[1][0]), fmaxf(s_max[2][0], s_max[3][0]));
    t.maxc8 = fmaxf(fmaxf(s_max[0][1], s_max[1][1]), fmaxf(s_max[2][1], s_max[3][1]));
    p.scan[row * p.parts + part] = t;
  }
}

// PROM = false: the vector-ALU split pass over a contiguous range of sealed blocks (INT8 keys).
// PROM = true : the promoted-block pass of the adaptive decode (gated precision): the workgroups
//               of a KV group walk the group's list of promoted blocks.  A key-promoted block is
//               scored from its FP16 keys (sigma = 1, z = 0, no score error), a value-promoted
//               block is attended from its FP16 values and counts with eta_b = 0; both kinds of
//               originals are read by the device straight from the pinned Tier-2 arrays over the
//               host link.  Writes partial sets split0 + split, the split decoded from the
//               workgroup's linear index.  Further workgroups sum up the blocks left in INT8.
template <int G, bool PROM>
__global__ __launch_bounds__(256) void certified_split_kernel(DecodeArgs a, PromArgs p) {
  fetch_args<sizeof(DecodeArgs) + (PROM ? sizeof(PromArgs) : 0)>();
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int tok = l & 15, kg = l >> 4;              // roles in the score phase
  const int vn = l & 15, vgh = (l >> 4) & 1, vo = l >> 5;  // roles in the value phase
  int split = blockIdx.x, kvh = blockIdx.y, b = blockIdx.z;
  if (PROM) {   // one index: (KV group, split), splits 0 .. 15 the positive sets, .. 31 the negated ones, then the sums
    int L = (int)(blockIdx.y * gridDim.x + blockIdx.x);
    const int sums = p.sum_waves ? 1 : G * p.parts, all = (2 * PROM_SPLITS + sums) * p.groups;
    int g, passes;
    if (L >= all) return;
    if (p.order == PROM_BY_GROUP) {
      g = L / (2 * PROM_SPLITS + sums);
      split = L % (2 * PROM_SPLITS + sums);
    } else if (p.order == PROM_SUMS_LAST) {
      passes = 2 * PROM_SPLITS * p.groups;
      g = L < passes ? L / (2 * PROM_SPLITS) : (L - passes) / sums;
      split = L < passes ? L % (2 * PROM_SPLITS) : 2 * PROM_SPLITS + (L - passes) % sums;
    } else {
      L = L < p.ahead ? L + all - p.ahead : L - p.ahead;
      passes = (PROM_SPLITS + sums) * p.groups;
      g = L < passes ? L / (PROM_SPLITS + sums) : (L - passes) / PROM_SPLITS;
      split = L < passes ? L % (PROM_SPLITS + sums) : PROM_SPLITS + (L - passes) % PROM_SPLITS;
      if (L < passes && split >= PROM_SPLITS) split += PROM_SPLITS;
    }
    if (split < 2 * PROM_SPLITS) split = (split & PROM_SPLITS) | ((split + p.turn * g) & (PROM_SPLITS - 1));
    b = g / a.n_kv;
    kvh = g - b * a.n_kv;
  }
  const int64_t head_rec = ((int64_t)b * a.n_kv + kvh) * a.nq_cap;
  // blocks are dealt evenly over the splits (every split gets at least one: nsplit <= nb)
  const int64_t grp = (int64_t)b * a.n_kv + kvh;
  // PROM: positions psplit * 4 + w, + 4 * PROM_SPLITS, ... of the group's list; else a block range
  // PROM: the second half of the workgroups (neg) walks the same list with INT8 keys and INT4
  // values whatever the flags say and writes its partial set negated: it takes back what the one
  // pass over all sealed blocks added for the listed blocks, the first half adds them again with
  // the originals the flags ask for.  Further ones, per head and part, sum up the blocks left in INT8.
  if (PROM && split >= 2 * PROM_SPLITS) {
    if (p.sum_waves) {
      if (w < G) prom_scan<true>(a, p, grp, G, w, 0, (int64_t)b * a.n_q + kvh * G + w);
      return;
    }
    const int part = (split - 2 * PROM_SPLITS) / G, h = (split - 2 * PROM_SPLITS) % G;
    prom_scan<false>(a, p, grp, G, h, part, (int64_t)b * a.n_q + kvh * G + h);
    return;
  }
  const bool neg = PROM && split >= PROM_SPLITS;
  const int psplit = PROM ? split & (PROM_SPLITS - 1) : split;
  __shared__ int s_blk[PROM ? PROM_SHARE : 1], s_pf[PROM ? PROM_SHARE : 1];
  const int n_list = PROM ? prom_list(a, p, grp, G, psplit, split == PROM_SPLITS, s_blk, s_pf) : 0;
  const int b0 = PROM ? psplit * 4 : (int)(((int64_t)split * a.nb) / a.nsplit);
  const int b1 = PROM ? n_list : (int)(((int64_t)(split + 1) * a.nb) / a.nsplit);
  const int bstep = PROM ? 4 * PROM_SPLITS : 4;
  const int out_split = PROM ? a.split0 + split : split;
  const float inv_sqrt_d = 0.08838834764831845f;  // 1 / sqrt(128)

  __shared__ __align__(16) float qs[4][G][D];     // scaled query of the block in flight, per wave
  __shared__ __align__(16) float ps[4][BLK][G];   // its probabilities
  __shared__ float ms[4][G][12];                  // per-wave scalars for the merge
  // FP16 values of a value-promoted block, one buffer per wave (rows padded against bank conflicts)
  __shared__ __align__(16) __half vst[PROM ? 4 : 1][PROM ? BLK : 1][PROM ? D + 8 : 8];

  float qv[G][2];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    const __half2 t = ld_half2_any(a.q + ((int64_t)b * a.n_q + kvh * G + h) * D + 2 * l);
    qv[h][0] = __low2float(t);
    qv[h][1] = __high2float(t);
  }

  float m_run[G], l_run[G], ev[G], evmax[G], dmax[G], t1[G], t2[G];
  int i1[G];
  float acc[4][G];
  float vmax = 0.0f;
  float dev[G];               // canary: largest |s_fp16 - s_int8| seen on key-promoted tokens
#pragma unroll
  for (int h = 0; h < G; ++h) dev[h] = 0.0f;
#pragma unroll
  for (int h = 0; h < G; ++h) {
    m_run[h] = -INFINITY;
    l_run[h] = 0.0f;
    ev[h] = 0.0f;
    evmax[h] = 0.0f;
    dmax[h] = 0.0f;
    t1[h] = -INFINITY;
    t2[h] = -INFINITY;
    i1[h] = -1;
#pragma unroll
    for (int gq = 0; gq < 4; ++gq) acc[gq][h] = 0.0f;
  }

  int at = w;   // PROM: this wave's entry of the share
  for (int pos = b0 + w; pos < b1; pos += bstep, at += 4) {
    // every index is bounded on the way in: a list entry outside [0, nb) is skipped
    const int blk = PROM ? __builtin_amdgcn_readfirstlane(s_blk[at]) : pos;
    if (PROM && (blk < 0 || blk >= a.nb)) continue;
    // Every load of the block is requested here, before anything is consumed: the block sits at
    // an address nothing else in this launch touches, so each dependent load costs a full
    // memory (and page-walk) latency.  First everything whose address follows from blk alone
    // (flags, INT8 codes, key and value metadata, INT4 codes), then the originals the flags ask
    // for.
    const int pf = PROM ? __builtin_amdgcn_readfirstlane(s_pf[at]) : 0;   // bit 0: FP16 keys, bit 1: FP16 values
    const float* kmb = reinterpret_cast<const float*>(a.t1 + t1_offset(head_rec, blk, Q_KM, KM_BYTES));
    const float2 sg8 = reinterpret_cast<const float2*>(kmb)[l];
    const float2 zz8 = reinterpret_cast<const float2*>(kmb + D)[l];
    float2 an = *reinterpret_cast<const float2*>(a.t1 + t1_offset(head_rec, blk, Q_AN, AN_BYTES));
    const uint8_t* kcb = a.t1 + t1_offset(head_rec, blk, Q_KC, KC_BYTES);
    uint4 kc8[2];
#pragma unroll
    for (int cq = 0; cq < 2; ++cq) kc8[cq] = reinterpret_cast<const uint4*>(kcb + cq * 1024)[l];
    const uint4 vx = reinterpret_cast<const uint4*>(a.t1 + t1_offset(head_rec, blk, Q_VC, VC_BYTES))[l];
    const __half* vmb = reinterpret_cast<const __half*>(a.t1 + t1_offset(head_rec, blk, Q_VM, VM_BYTES));
    uint4 sraw4[4], oraw4[4];
#pragma unroll
    for (int gq = 0; gq < 4; ++gq) {
      const int g = vgh * 4 + gq;
      sraw4[gq] = *reinterpret_cast<const uint4*>(vmb + vo * 64 + g * 8);
      oraw4[gq] = *reinterpret_cast<const uint4*>(vmb + BLK * NG + vo * 64 + g * 8);
    }
    // which heads of the group score this block with FP16 keys / attend its FP16 values (the
    // per-head bits of the flag word; with per-group promotion they are all alike)
    const int hkb = (PROM && !neg) ? (pf >> SLOT_HK_SHIFT) & ((1 << G) - 1) : 0;
    const int hvb = (PROM && !neg) ? (pf >> SLOT_HV_SHIFT) & ((1 << G) - 1) : 0;
    const bool kfp = hkb != 0, vfp = hvb != 0;
    const bool kall = hkb == (1 << G) - 1;
    // FP16 keys of the block, [token][128 channels]: from its slot of the device-resident
    // scratch if it is held there, else from the host-resident originals -- and then, if the
    // block has just been given a slot, stored into it on the way
    uint4 k16[2][2];
    const int sc0 = (pf >> SLOT_SC_SHIFT) & 0xFFFF;   // bits 8-23: scratch slot + 1
    const int sc = (PROM && a.sc_k != nullptr && sc0 <= a.sc_cap) ? sc0 : 0;   // bounded whatever the word holds
    if (kfp) {
      const bool fill = sc > 0 && (pf & SLOT_FILL);
      __half* sck = sc > 0 ? a.sc_k + (((grp * a.sc_cap + (sc - 1)) * BLK) + tok) * D : nullptr;
      const __half* kf16 = (sc > 0 && !fill) ? sck
                                             : a.t2_k + ((grp * a.max_tokens + (int64_t)blk * BLK) + tok) * D;
#pragma unroll
      for (int cq = 0; cq < 2; ++cq) {
        const int c0 = cq * 64 + kg * 16;
        k16[cq][0] = *reinterpret_cast<const uint4*>(kf16 + c0);
        k16[cq][1] = *reinterpret_cast<const uint4*>(kf16 + c0 + 8);
      }
      if (fill) {
#pragma unroll
        for (int cq = 0; cq < 2; ++cq) {
          const int c0 = cq * 64 + kg * 16;
          *reinterpret_cast<uint4*>(sck + c0) = k16[cq][0];
          *reinterpret_cast<uint4*>(sck + c0 + 8) = k16[cq][1];
        }
      }
    }
    if (vfp) {
      // its FP16 values, row-major [token][128], coalesced into this wave's LDS buffer: from the
      // value half of the block's scratch slot, or from the host-resident originals (and then
      // into the slot, if the block has just been given one)
      const bool vfill = sc > 0 && (pf & SLOT_VFILL);
      const int64_t in_blk = (int64_t)(l >> 2) * D + (l & 3) * 32;
      __half* scv = sc > 0 ? a.sc_v + (grp * a.sc_cap + (sc - 1)) * (int64_t)(BLK * D) + in_blk : nullptr;
      const __half* v16 = (sc > 0 && !vfill) ? scv
                                             : a.t2_v + (grp * a.max_tokens + (int64_t)blk * BLK) * D + in_blk;
      uint4 v16r[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) v16r[j] = *reinterpret_cast<const uint4*>(v16 + j * 8);
      if (vfill) {
#pragma unroll
        for (int j = 0; j < 4; ++j) *reinterpret_cast<uint4*>(scv + j * 8) = v16r[j];
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)
        *reinterpret_cast<uint4*>(&vst[w][l >> 2][(l & 3) * 32 + j * 8]) = v16r[j];
    }
    // ---- scores.  Lane (tok, kg) covers channels cq*64 + kg*16 + 0..15, cq = 0, 1.  First from
    //      the FP16 keys (sigma = 1, z = 0: the query itself in the LDS buffer) when some head asks
    //      for them, then from the INT8 codes (scaled query q~ = q sigma, block constant
    //      c_b = q.z, bound Delta_b) when some head keeps them -- or when the score-consistency
    //      check compares the two.
    float s16[G], s8[G], dsum[G];
#pragma unroll
    for (int h = 0; h < G; ++h) {
      s16[h] = 0.0f;
      s8[h] = 0.0f;
      dsum[h] = 0.0f;
    }
    if (kfp) {
#pragma unroll
      for (int h = 0; h < G; ++h)
        reinterpret_cast<float2*>(&qs[w][h][0])[l] = make_float2(qv[h][0], qv[h][1]);
      wave_sync();
      float dot[G];
#pragma unroll
      for (int h = 0; h < G; ++h) dot[h] = 0.0f;
#pragma unroll
      for (int cq = 0; cq < 2; ++cq) {
        const int c0 = cq * 64 + kg * 16;
        const __half2* h0 = reinterpret_cast<const __half2*>(&k16[cq][0]);
        const __half2* h1 = reinterpret_cast<const __half2*>(&k16[cq][1]);
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const __half2 pr = (j < 8) ? h0[j >> 1] : h1[(j - 8) >> 1];
          const float kf = (j & 1) ? __high2float(pr) : __low2float(pr);
#pragma unroll
          for (int h = 0; h < G; ++h) dot[h] = fmaf(qs[w][h][c0 + j], kf, dot[h]);
        }
      }
#pragma unroll
      for (int h = 0; h < G; ++h) {
        dot[h] = sum_x32(sum_x16(dot[h]));
        s16[h] = dot[h] * inv_sqrt_d;
      }
      wave_sync();   // the LDS buffer is rewritten below
    }
    const bool canary = PROM && kfp && a.score_dev != nullptr;
    if (!kfp || !kall || canary) {
      // a.int8_query: the scaled query is quantised to 8 bits per (head, block) exactly as the pass
      // over all blocks does it (binary32 decisions: s_q = max|q~| / 127, T = round-half-even of
      // q~ * fl(127 / max)), the codes T take the scaled query's place in the dot product, which is
      // then exact integer arithmetic, and the residual sum |q~ - s_q T| widens the block's bound
      float csum[G], tsum[G], rsum[G], sqv[G];
#pragma unroll
      for (int h = 0; h < G; ++h) {
        float q0 = qv[h][0] * sg8.x, q1 = qv[h][1] * sg8.y;
        dsum[h] = fabsf(qv[h][0]) * sg8.x + fabsf(qv[h][1]) * sg8.y;
        tsum[h] = 0.0f;
        rsum[h] = 0.0f;
        sqv[h] = 1.0f;
        if (a.int8_query) {
          const float amax = wave_max(fmaxf(fabsf(q0), fabsf(q1)));
          const float inv = amax > 0.0f ? 127.0f / amax : 0.0f;
          const float sq = amax / 127.0f;
          const float MAGIC = 12582912.0f;   // 1.5 * 2^23: fl(x + MAGIC) - MAGIC = round-half-even(x)
          const float t0 = fmaf(q0, inv, MAGIC) - MAGIC, t1 = fmaf(q1, inv, MAGIC) - MAGIC;
          rsum[h] = fabsf(fmaf(-sq, t0, q0)) + fabsf(fmaf(-sq, t1, q1));
          q0 = t0;
          q1 = t1;
          tsum[h] = t0 + t1;                 // small integers: every partial sum below is exact
          sqv[h] = sq;
          csum[h] = qv[h][0] * zz8.x + qv[h][1] * zz8.y;
        } else {
          // stored bytes are code + 128: fold the -128 * sum(q~) into the block constant
          csum[h] = qv[h][0] * zz8.x + qv[h][1] * zz8.y - 128.0f * (q0 + q1);
        }
        reinterpret_cast<float2*>(&qs[w][h][0])[l] = make_float2(q0, q1);
      }
#pragma unroll
      for (int h = 0; h < G; ++h) {
        csum[h] = wave_sum(csum[h]);
        dsum[h] = wave_sum(dsum[h]);
        if (a.int8_query) {
          tsum[h] = wave_sum(tsum[h]);
          rsum[h] = wave_sum(rsum[h]);
        }
      }
      if (a.int8_query) {
#pragma unroll
        for (int h = 0; h < G; ++h) dsum[h] = fmaf(256.0f, rsum[h], dsum[h]);   // (Delta_b + Delta^q_b) * 2 sqrt d
      }
      wave_sync();
      float dot[G];
#pragma unroll
      for (int h = 0; h < G; ++h) dot[h] = 0.0f;
#pragma unroll
      for (int cq = 0; cq < 2; ++cq) {
        const uint32_t wd[4] = {kc8[cq].x, kc8[cq].y, kc8[cq].z, kc8[cq].w};
        const int c0 = cq * 64 + kg * 16;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const float kf = (float)((wd[j >> 2] >> (8 * (j & 3))) & 0xffu);
#pragma unroll
          for (int h = 0; h < G; ++h) dot[h] = fmaf(qs[w][h][c0 + j], kf, dot[h]);
        }
      }
#pragma unroll
      for (int h = 0; h < G; ++h) {
        dot[h] = sum_x32(sum_x16(dot[h]));
        // quantised query: s_q * (sum T byte - 128 sum T) + q.z, the bracket in exact integers
        s8[h] = fmaf(sqv[h], dot[h] - 128.0f * tsum[h], csum[h]) * inv_sqrt_d;
      }
    }
    if (canary) {
      // score-consistency check: FP16 against INT8 scores, token by token, for the heads that
      // score this block from its FP16 keys
#pragma unroll
      for (int h = 0; h < G; ++h)
        if ((hkb >> h) & 1) dev[h] = fmaxf(dev[h], fabsf(s16[h] - s8[h]));
    }
    float p[G], alpha[G];
#pragma unroll
    for (int h = 0; h < G; ++h) {
      const bool use16 = ((hkb >> h) & 1) != 0;
      const float s = use16 ? s16[h] : s8[h];
      const float mb = row_max(s);
      const float pt = __expf(s - mb);
      const float sb = row_sum(pt);
      const float lb = mb + __logf(sb);
      const float m_new = fmaxf(m_run[h], mb);
      alpha[h] = __expf(m_run[h] - m_new);
      const float f = __expf(mb - m_new);
      p[h] = pt * f;
      const float sf = sb * f;
      const float ce = ((hvb >> h) & 1) ? 0.0f : sf * an.x;   // exact values add nothing to the value term
      l_run[h] = l_run[h] * alpha[h] + sf;
      ev[h] = ev[h] * alpha[h] + ce;
      evmax[h] = fmaxf(evmax[h] * alpha[h], ce);
      dmax[h] = fmaxf(dmax[h], use16 ? 0.0f : dsum[h] * (0.5f * inv_sqrt_d));
      m_run[h] = m_new;
      if (lb > t1[h]) {
        t2[h] = t1[h];
        t1[h] = lb;
        i1[h] = blk;
      } else if (lb > t2[h]) {
        t2[h] = lb;
      }
      if (a.blk_logmass != nullptr && l == 0 && !neg)
        a.blk_logmass[((int64_t)b * a.n_q + kvh * G + h) * a.nb + blk] = lb;
      if (kg == 0) ps[w][tok][h] = p[h];
    }
    vmax = fmaxf(vmax, an.y);
    wave_sync();

    // ---- values: lane (vo, vgh, vn) covers tokens vo*8..+7 of channels (vgh*4+gq)*16 + vn
    const uint32_t vw[4] = {vx.x, vx.y, vx.z, vx.w};
    float pi[8][G];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int h = 0; h < G; ++h) pi[i][h] = ps[w][vo * 8 + i][h];
#pragma unroll
    for (int gq = 0; gq < 4; ++gq) {
      const int g = vgh * 4 + gq;
      const __half2* sh = reinterpret_cast<const __half2*>(&sraw4[gq]);
      const __half2* oh = reinterpret_cast<const __half2*>(&oraw4[gq]);
#pragma unroll
      for (int h = 0; h < G; ++h) acc[gq][h] *= alpha[h];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float sc = (i & 1) ? __high2float(sh[i >> 1]) : __low2float(sh[i >> 1]);
        const float of = (i & 1) ? __high2float(oh[i >> 1]) : __low2float(oh[i >> 1]);
        const float v4 = fmaf((float)((vw[gq] >> (4 * i)) & 15u), sc, of);
        const float v16 = vfp ? __half2float(vst[w][vo * 8 + i][g * 16 + vn]) : v4;
#pragma unroll
        for (int h = 0; h < G; ++h) acc[gq][h] = fmaf(pi[i][h], ((hvb >> h) & 1) ? v16 : v4, acc[gq][h]);
      }
    }
    wave_sync();
  }

  if (PROM && a.score_dev != nullptr) {
    // deviations are non-negative floats: their bit patterns order like integers
#pragma unroll
    for (int h = 0; h < G; ++h) {
      const float d = wave_max(dev[h]);
      if (l == 0 && d > 0.0f)
        atomicMax(reinterpret_cast<int*>(a.score_dev + (int64_t)b * a.n_q + kvh * G + h), __float_as_int(d));
    }
  }
  // ---- merge the four waves of the workgroup, then write one partial per q-head
  float* mo = &qs[0][0][0];  // reuse: [4][G][D]
  __syncthreads();
#pragma unroll
  for (int gq = 0; gq < 4; ++gq)
#pragma unroll
    for (int h = 0; h < G; ++h) {
      const float v = sum_x32(acc[gq][h]);
      if (vo == 0) mo[(w * G + h) * D + (vgh * 4 + gq) * 16 + vn] = v;
    }
  if (l == 0) {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      ms[w][h][0] = m_run[h];
      ms[w][h][1] = l_run[h];
      ms[w][h][2] = ev[h];
      ms[w][h][3] = evmax[h];
      ms[w][h][4] = dmax[h];
      ms[w][h][5] = vmax;
      ms[w][h][6] = t1[h];
      ms[w][h][7] = t2[h];
      ms[w][h][8] = __int_as_float(i1[h]);
    }
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < G * D; idx += 256) {
    const int h = idx / D, c = idx % D;
    float M = -INFINITY;
#pragma unroll
    for (int ww = 0; ww < 4; ++ww) M = fmaxf(M, ms[ww][h][0]);
    const float Mr = (M == -INFINITY) ? 0.0f : M;   // a workgroup without blocks writes zeros
    float o = 0.0f;
#pragma unroll
    for (int ww = 0; ww < 4; ++ww) o += __expf(ms[ww][h][0] - Mr) * mo[(ww * G + h) * D + c];
    a.partials[(((int64_t)b * a.n_q + kvh * G + h) * a.pstride + out_split) * PART_FLOATS + P_O + c] =
        neg ? -o : o;
  }
  if (threadIdx.x < G) {
    const int h = threadIdx.x;
    float M = -INFINITY;
    for (int ww = 0; ww < 4; ++ww) M = fmaxf(M, ms[ww][h][0]);
    const float Mr = (M == -INFINITY) ? 0.0f : M;
    float L = 0.0f, EV = 0.0f, EVM = 0.0f, DM = 0.0f, VM = 0.0f, T1 = -INFINITY, T2 = -INFINITY;
    int I1 = -1;
    for (int ww = 0; ww < 4; ++ww) {
      const float f = __expf(ms[ww][h][0] - Mr);
      L += f * ms[ww][h][1];
      EV += f * ms[ww][h][2];
      EVM = fmaxf(EVM, f * ms[ww][h][3]);
      DM = fmaxf(DM, ms[ww][h][4]);
      VM = fmaxf(VM, ms[ww][h][5]);
      top2_merge(T1, I1, T2, ms[ww][h][6], __float_as_int(ms[ww][h][8]), ms[ww][h][7]);
    }
    float* pp = a.partials + (((int64_t)b * a.n_q + kvh * G + h) * a.pstride + out_split) * PART_FLOATS;
    pp[P_M] = M;
    pp[P_L] = neg ? -L : L;
    pp[P_EV] = neg ? -EV : EV;
    pp[P_EVMAX] = neg ? 0.0f : EVM;
    pp[P_DMAX] = DM;
    pp[P_VMAX] = VM;
    pp[P_T1] = T1;
    pp[P_T2] = T2;
    pp[P_I1] = __int_as_float(I1);
  }
}

// Stand-alone cross-split reduction.
__global__ __launch_bounds__(64 * (RED_WAVES + 2)) void certified_reduce_kernel(ReduceArgs a) {
  fetch_args<sizeof(ReduceArgs)>();
  __shared__ __align__(16) ReduceSmem sm;
  HeadRow row;
  if (reduce_row(a, blockIdx.y, blockIdx.x, reduce_waves(a.nsplit), sm, row)) store_row(a, row_of(a, blockIdx.y, blockIdx.x), row);
}

__global__ __launch_bounds__(64) void certified_reduce_wave_kernel(ReduceArgs a) {
  fetch_args<sizeof(ReduceArgs)>();
  const int64_t row = row_of(a, blockIdx.y, blockIdx.x);
  store_row(a, row, reduce_row_wave(a, row));
}

// Workgroups ("splits") per (batch, kv-head) and waves per workgroup of the matrix-core split pass.
// A compute unit holds eight of its waves: one workgroup of eight, or two of four.  The quads of a
// head are dealt evenly over its waves, so a workgroup takes ceil(quads / (waves * splits)) rounds of
// one quad per wave, and the launch costs about  generations * (rounds + 1):  every generation of
// resident workgroups walks its rounds and pays about one more for start-up and merge.
//   Up to one sequence per compute unit: as many splits as fit ONE generation (rounding up instead
//     left a second, nearly empty one: 48 sequences of 20011 tokens, 6 splits 82.5 us, 5 splits
//     63.2 us for pass and reduction; 72 of 14000: 86.6 -> 64.9; 25 x 4 of 10000: 83.3 -> 64.9).
//     Eight-wave workgroups when both forms take the same rounds (half as many partial sets,
//     all waves dispatched in one sweep: 200 of 5000: 66.9 against 72.1 us), four-wave ones where they
//     divide better (130 of 8000: 74.3 against 81.3 us; 152 of 7000: 73.3 against 75.8 us), and where a quad
//     per wave needs no more of them than there are compute units: a wave that has its SIMD to itself is
//     through its only quad 0.9 us earlier (1 sequence of 1029: 13.9 -> 13.3 us, 8 of 1000: 14.4 -> 13.8; 1 of 10000, 20
//     and 40 sets: 10.75, 9.1; 4 of 16384, 32 and 64: 12.3, 11.8; 1 of 30000, 59 and 118: 12.9, 11.6), up to 128 sets,
//     which the reduction takes in two trips (1 of 60000, 118 and 235: 14.1, 14.2).  Up to eight quads are one workgroup,
//     which finishes the rows itself: 1 KV head of 300 tokens 9.0 -> 7.9 us, of 520 9.2 -> 8.2 (with 16 quads the
//     second round costs more than the reduction's launch: 8.3 against 12.2).
//   More sequences than compute units: four-wave workgroups, up to four splits where a last
//     generation would be nearly empty (288 of 3600: 1 split 91.2, 2 90.9, 3 78.8 us; 384 of 2700: 1
//     78.5, 2 82.5; 560 of 1900: 1 93.4, 2 84.5, 3 85.1; 704 of 1500: 1 90.3, 2 84.4; 1104 of 950: 1 92.7, 2 95.1).
//     Several splits only within three generations: that bounds the partial sets (no-allocation scratch).
// Short sequences get no more workgroups than have a quad for every wave but the last workgroup's.
void split_geometry(const Cache* c, int64_t n_blocks, int* nsplit, int* wpb) {
  const int64_t heads = (int64_t)c->desc.batch * c->desc.n_kv_heads;
  const int64_t limit = std::min<int64_t>(c->max_splits, MAX_SPLITS);
  const int64_t quads = (n_blocks + 3) / 4;
  *nsplit = 0;
  *wpb = heads > c->n_cu ? 4 : 8;
  if (n_blocks <= 0) return;
  int64_t best_cost = -1;
  const auto consider = [&](int64_t w, int64_t s) {
    s = std::max<int64_t>(std::min(std::min(s, limit), (quads + w - 1) / w), 1);
    const int64_t slots = (8 / w) * (int64_t)c->n_cu;
    const int64_t cost = ((heads * s + slots - 1) / slots) * ((quads + w * s - 1) / (w * s) + 1);
    if (best_cost < 0 || cost < best_cost) {
      best_cost = cost;
      *nsplit = (int)s;
      *wpb = (int)w;
    }
  };
  if (c->forced_splits > 0) {
    consider(*wpb, c->forced_splits);
  } else if (heads <= c->n_cu) {
    if (quads <= 8) consider(8, 1);
    if (heads * ((quads + 3) / 4) <= c->n_cu && quads <= 4 * 128) consider(4, (quads + 3) / 4);
    consider(8, c->n_cu / heads);
    consider(4, 2 * c->n_cu / heads);
  } else {
    for (int64_t s = 1; s <= 4; ++s)
      if (s == 1 || heads * s <= 6 * (int64_t)c->n_cu) consider(4, s);
  }
}

// Whether the matrix-core pass reads Tier-1 with the non-temporal hint.  One decode step of a
// model walks every layer, so the bytes read between two visits of the same record are one
// pass's bytes times the layer count.  Up to the size of the memory-side cache (256 MB) plain
// loads gain from what is left there from the previous step (four layers of 8229 tokens, 76 MB:
// 70 us a pass against 75); beyond it the hinted loads stream faster: 278 MB 81 -> 76 us, 303 MB
// 64 -> 58.5 us a step when three caches take turns (INT8 x INT8 scoring 63.6 -> 58.4), 606 MB 109 -> 98 us.
// The price is paid where one layer of that size is read over and over, which a stack of layers never is: 303 MB 51.2
// -> 51.7 us a pass, up to 1.5 us more on other boxes, the step the same 57.4 (INT8 x INT8 51.0 -> 51.4; with a token
// appended each step 53.3 -> 55.7).
int stream_nt(const Cache* c, int64_t n_blocks) {
  if (c->stream_hint == 1) return 0;
  if (c->stream_hint == 2) return 1;
  const int64_t pass = (int64_t)c->desc.batch * c->desc.n_kv_heads * ((n_blocks + 3) / 4) * QUAD_BYTES;
  return pass * c->desc.n_layers > ((int64_t)256 << 20) ? 1 : 0;
}

// Whether what is launched on the stream is recorded into a graph.  (The null stream cannot be, and asking about it while another
// stream is recorded would be an error.)
static bool recorded(hipStream_t st) {
  hipStreamCaptureStatus s = hipStreamCaptureStatusNone;
  if (st == nullptr) return false;
  if (hipStreamIsCapturing(st, &s) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return s == hipStreamCaptureStatusActive;
}

// Whether the split pass of a step with the ladder behind it reduces its partial sets itself, and with how many waves per workgroup
// (0 = the reduction stays a launch of its own).  The sets that its last workgroup joins: reduced_sets.  Recorded steps (device time
// alone), us, with the launch and without: 8 KV heads x 4 of 1000 tokens 9.9, 9.8; of 3000 10.4, 10.3; x 1 of 605 11.1, 9.1; of 8000 10.7, 10.2; x 2 of 1500 10.4,
// 9.5; 2 x 4 of 2005 10.8, 9.5; 32 x 4 of 4000 14.4, 14.1; 128 x 4 of 1000 16.0, 15.1; 72 x 1 of 3145 21.0, 20.2; 136 x 2 of 3145 31.3, 30.8; 16 x 2 of 9005 19.6, 19.4.  A
// host that takes longer for a launch gains more (8 x 4 of 1000 called in a loop 12.3, 10.7).  With a second trip per wave the launch is
// better: 8 x 4 of 8229 12.6, 13.2; 16000 14.3, 16.1; 128K 57.2, 58.7; 2 x 4 of 8000 10.3, 11.8.
// A KV group's workgroups share a die, so the dies have to be evenly loaded: as many groups on each, or no more
// workgroups on the fullest than it has compute units.
// Four waves for four heads have no second row to share the tail: the launch is better (17 x 8 x 4 of 2005 tokens 25.1, 26.0; 9 x 8 x 4 of 3145 22.1,
// 23.0; 20 x 8 x 4 of 1350 21.8, 22.7).  So it is with more groups than compute units (33 x 8 x 2 of 1350 31.8, 33.4; 40 x 8 x 1 of 2005 42.7, 43.1), and
// for four heads by eight waves with two quads each at most, of which the first row's attend the trailing tokens and are not yet far ahead of
// the others (9 x 8 x 4 of 2005 18.2, 18.8; 11 x 8 x 4 of 1365 17.1, 17.8; 4 x 8 x 4 of 8005 21.6, 21.9; but with one quad, 8 x 8 x 4 of 2005, 15.2, 14.7, and with
// more, 10 x 8 x 4 of 5005, 30.0, 29.3).
static int split_reduces(const Cache* c, int64_t n_blocks, int nsplit, int wpb, int r, hipStream_t st) {
  const int64_t heads = (int64_t)c->desc.batch * c->desc.n_kv_heads;
  const int g = c->desc.n_q_heads / c->desc.n_kv_heads;
  if (c->split_tickets == nullptr || c->variant != 0 || nsplit < 2 || heads > c->n_cu) return 0;
  if (__atomic_load_n(c->strayed, __ATOMIC_RELAXED) != 0u && c->scatter != 1) return 0;   // this device deals workgroups otherwise
  if (heads % DIES != 0 && (heads + DIES - 1) / DIES * nsplit > c->n_cu / DIES) return 0;
  // Four waves with a quad each and a compute unit to themselves are joined by four or eight without: the trailing tokens are attended
  // and the key term taken beside the rest (8 x 4 of 1000 tokens 10.5 -> 9.6 us a recorded step, of 3000 11.3 -> 10.4).
  const bool alone = wpb == 4 && 4 * (int64_t)nsplit >= (n_blocks + 3) / 4 && heads * nsplit <= c->n_cu;
  const int waves = alone ? (g == 4 && nsplit > reduced_sets(4, 4, 8) ? 12 : 8) : wpb;
  // Twelve waves and nothing for the four that are to attend the trailing tokens: it is the host that gains by two launches (called
  // in a loop 12.1 -> 10.3 us), the device alone is quicker with three (recorded, three and two: 8 x 4 of 4000 tokens 10.0, 10.2; 4 x 4 9.8,
  // 10.2; 1 x 4 9.5, 10.2; 10 x 4 10.0, 10.2; 16 x 4 10.1, 10.3): a step that is being recorded takes three.
  if (waves == 12 && r == 0 && recorded(st)) return 0;
  const int64_t quads = (n_blocks + 3) / 4, quad_waves = (int64_t)wpb * nsplit;
  if (g == 4 && wpb == 8 && quads > quad_waves && quads <= 2 * quad_waves) return 0;
  return nsplit <= reduced_sets(g, wpb, waves) ? waves : 0;
}

// Whether the ladder's launch can reduce a step's rows as well (finish_ladder_kernel), and whether it does where the split pass could.
// Both ways are two launches: in the ladder's one wave per row does in turn what a group's last workgroup shares among its waves, which has to be
// waited for, through the die's cache.  Without trailing tokens, or with one KV group, the ladder's launch is no slower.  Recorded steps,
// reduced by it and by the split pass, us: no trailing tokens, 1 KV head x 4 of 1024 tokens 8.2, 9.2; x 1 8.0, 8.7; 2 x 2 8.4, 8.9; 2 x 4 8.7, 9.4; 3 x 2
// 8.7, 8.9; 4 x 1 8.3, 8.9; 5 x 1 8.6, 8.9; 8 x 1 8.9, 9.0.  With them: 1 x 4 9.1, 9.2; 1 x 1 8.7, 8.6; 1 x 2 of 2049 8.9, 9.0; but 2 x 4 10.6,
// 9.4; 2 x 2 9.4, 9.2; 8 x 1 10.8, 8.9.
static bool ladder_reduces(const Cache* c, int nsplit) {
  return nsplit > 1 && nsplit <= FINISH_SETS && (int64_t)c->desc.batch * c->desc.n_q_heads <= FINISH_ROWS;
}
static bool ladder_reduces_first(const Cache* c, int nsplit, int r) {
  return ladder_reduces(c, nsplit) && (r == 0 || (int64_t)c->desc.batch * c->desc.n_kv_heads == 1);
}

int pick_splits(const Cache* c, int64_t n_blocks) {
  int nsplit = 0, wpb = 0;
  split_geometry(c, n_blocks, &nsplit, &wpb);
  return nsplit;
}

// Promoted-block pass of the adaptive decode (see certified_split_kernel).
int32_t launch_promoted_pass(const DecodeArgs& a, const PromArgs& p, int group, dim3 grid, hipStream_t st) {
  if (p.ulist == nullptr || p.ucount == nullptr || p.slot == nullptr || a.t2_k == nullptr || a.t2_v == nullptr)
    return CQA_ERR_INVALID_ARG;
  switch (group) {
    case 1: hipLaunchKernelGGL((certified_split_kernel<1, true>), grid, dim3(256), 0, st, a, p); break;
    case 2: hipLaunchKernelGGL((certified_split_kernel<2, true>), grid, dim3(256), 0, st, a, p); break;
    case 4: hipLaunchKernelGGL((certified_split_kernel<4, true>), grid, dim3(256), 0, st, a, p); break;
    default: return CQA_ERR_UNSUPPORTED;
  }
  CQA_HIP(hipGetLastError());
  return CQA_OK;
}

// Split partials of callers that must not allocate: one array per GPU, placed by the loader when
// the code object is loaded on that GPU and held until the process ends.  In host code the name
// `scratch` is only a handle for hipGetSymbolAddress; kernels receive the resolved address.
constexpr int64_t STATIC_SCRATCH_BYTES = CQA_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

constexpr int MAX_DEVICES = 64;
static void* g_scratch_ptr[MAX_DEVICES];   // per device: address of its copy of `scratch` (null = not resolved yet)
static std::mutex g_scratch_mutex;

// Address of the current device's copy of the static scratch; resolved once per device, with that
// device current (cqa_cache_create does it for the device it creates the cache on).
int32_t static_scratch(int device, void** out) {
  if (device < 0 || device >= MAX_DEVICES) return CQA_ERR_UNSUPPORTED;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[device] == nullptr) {
    int cur = -1;
    CQA_HIP(hipGetDevice(&cur));
    if (cur != device) return CQA_ERR_INVALID_ARG;
    void* p = nullptr;
    CQA_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (p == nullptr) return CQA_ERR_HIP;
    g_scratch_ptr[device] = p;
  }
  *out = g_scratch_ptr[device];
  return CQA_OK;
}

int32_t launch_certified(Cache* c, int layer, const __half* q, const cqa_tolerances& tol, float* O,
                         cqa_head_cert* cert, uint32_t* flags, uint32_t* flags_mirror,
                         uint32_t mirror_tag, float* blk_logmass, hipStream_t st,
                         const __half* k_new, const __half* v_new, int pstride, float* eta_out,
                         float* partials, uint32_t* raised, uint32_t raised_tag, ReduceArgs* defer, RowsBy* by) {
  const bool always = defer != nullptr && by == nullptr;   // the reduction is left to the caller in any case
  const int bt = c->desc.batch, hq = c->desc.n_q_heads, hkv = c->desc.n_kv_heads;
  if (partials == nullptr) partials = c->partials;
  const int64_t len = c->length[layer];
  const int64_t nb = len / BLK;
  const int r = (int)(len % BLK);
  int nsplit = 0, wpb = 0;
  split_geometry(c, nb, &nsplit, &wpb);
  const int64_t layer_head0 = head_index(c, layer, 0, 0);
  ReduceArgs ra{};
  ra.partials = partials;
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
  ra.nsplit = nsplit;
  ra.pstride = pstride;
  ra.nb = (int)nb;
  ra.r = r;
  ra.n_q = hq;
  ra.n_kv = hkv;
  bool reduced = false;   // the matrix-core pass finishes the rows of a single split itself
  if (nb > 0) {
    DecodeArgs a{};   // every field starts null / zero
    a.t1 = c->t1 + layer_head0 * c->nq_cap * QUAD_BYTES;
    a.sigmax = c->sigmax + layer_head0;
    a.q = q;
    a.partials = partials;
    a.blk_logmass = blk_logmass;
    a.nq_cap = c->nq_cap;
    a.nb = (int)nb;
    a.nsplit = nsplit;
    a.pstride = pstride > 0 ? pstride : nsplit;
    a.t2_k = nullptr;
    a.t2_v = nullptr;
    a.eta_out = nullptr;
    a.score_dev = nullptr;
    a.max_tokens = 0;
    a.split0 = 0;
    a.eta_out = blk_logmass != nullptr ? eta_out : nullptr;
    if (k_new != nullptr) {
      // the caller has already counted the new token in length[layer]: it is token len - 1
      if (c->variant != 0 || r == 0) return CQA_ERR_INVALID_ARG;   // needs this kernel and an open block
      a.ap_k_new = k_new;
      a.ap_v_new = v_new;
      a.ap_trail_k = c->trail_k + layer_head0 * BLK * D;
      a.ap_trail_v = c->trail_v + layer_head0 * BLK * D;
      const bool t2 = c->desc.tier2_mode == CQA_TIER2_PINNED;
      a.ap_t2_k = t2 ? c->t2_k + layer_head0 * c->desc.max_tokens * D : nullptr;
      a.ap_t2_v = t2 ? c->t2_v + layer_head0 * c->desc.max_tokens * D : nullptr;
      a.ap_slot = r - 1;
      a.ap_pos = len - 1;
      a.ap_max_tokens = c->desc.max_tokens;
    }
    a.n_q = hq;
    a.n_kv = hkv;
    a.stream_nt = stream_nt(c, nb);
    a.int8_query = tol.int8_query;
    a.wpb = wpb;
    // The rows of one workgroup's sequences are finished by this launch, whether their flags are mirrored to the host or not.
    // A host-resolved step, the reduction's launch and this one finishing the rows: 4 heads per group, 32 rows 19.2, 15.9 us; 128
    // 20.9, 16.2; 256 22.2, 16.5; 1024 27.9, 17.9; 2048 40.6, 25.3; two, 1440 rows 48.6, 35.5; one, 720 42.6, 36.0.
    a.finish = nsplit == 1 && !always ? 1 : 0;
    a.heads = bt * hkv;
    const int64_t last = (int64_t)a.heads * nsplit % (2 * c->n_cu);   // workgroups of the last generation
    a.settle = wpb == 4 && last >= c->n_cu && 2 * last <= 3 * c->n_cu ? 1 : 0;
    a.waves = by != nullptr && !ladder_reduces_first(c, nsplit, r) ? split_reduces(c, nb, nsplit, wpb, r, st) : 0;
    if (a.waves != 0) {
      a.tickets = c->split_tickets;
      a.scatter = c->scatter;
    }
    // the quantised-query scoring exists in the matrix-core pass (and in the promoted-block pass of
    // the adaptive calls), not in the vector-ALU cross-check kernel
    if (tol.int8_query != 0 && c->variant != 0) return CQA_ERR_UNSUPPORTED;
    const dim3 grid(nsplit, hkv, bt);
    const bool prof = c->prof_ev != nullptr && c->prof_n < c->prof_cap;
    hipEvent_t ev0 = prof ? c->prof_ev[2 * c->prof_n] : nullptr;
    hipEvent_t ev1 = prof ? c->prof_ev[2 * c->prof_n + 1] : nullptr;
    if (prof && c->variant != 0) CQA_HIP(hipEventRecord(ev0, st));
    if (c->variant == 0 || a.eta_out != nullptr) {   // eta_b comes from this kernel only
      const dim3 by_die(DIES, nsplit, (a.heads + DIES - 1) / DIES);
      const int32_t rc = launch_split_mfma(a, ra, hq / hkv, a.tickets != nullptr ? by_die : grid, ev0, ev1, st);
      if (rc != CQA_OK) return rc;
      reduced = a.finish != 0;
      if (a.tickets != nullptr) {
        reduced = true;
        *defer = ra;
        *by = RowsBy::split;
      }
    } else {
      switch (hq / hkv) {
        case 1: hipLaunchKernelGGL((certified_split_kernel<1, false>), grid, dim3(256), 0, st, a, PromArgs{}); break;
        case 2: hipLaunchKernelGGL((certified_split_kernel<2, false>), grid, dim3(256), 0, st, a, PromArgs{}); break;
        case 4: hipLaunchKernelGGL((certified_split_kernel<4, false>), grid, dim3(256), 0, st, a, PromArgs{}); break;
        default: return CQA_ERR_UNSUPPORTED;
      }
    }
    CQA_HIP(hipGetLastError());
    if (prof) {
      if (c->variant != 0) CQA_HIP(hipEventRecord(ev1, st));
      ++c->prof_n;
    }
  }
  if (reduced) return CQA_OK;
  const bool by_ladder = by != nullptr && ladder_reduces(c, nsplit);
  if (always || by_ladder) {
    *defer = ra;
    if (by_ladder) *by = RowsBy::ladder;
    return CQA_OK;
  }
  // With a mirror and more than four rows per compute unit, one wave per row: a row's waves side by side bring the stores
  // to the mirror closer together, where they wait for one another.  A host-resolved step of 4 heads per group, three waves a row and
  // one: 1152 rows of three sets 79.5, 78.9 us; 2240 of two 97.7, 91.7; 2816 102.1, 97.0.  (Two heads per group, level: 1152
  // rows 70.4, 69.8; 1280 56.8, 57.0.)  Up to 1024 rows, and without a mirror at any number, three waves: 256 rows 10.4, 10.9 us a
  // decode; 512 13.4, 13.9; 1152 63.1, 63.6; 2240 70.3, 71.1.
  if (flags_mirror != nullptr && (int64_t)bt * hq > 4 * (int64_t)c->n_cu && nsplit <= 8)
    hipLaunchKernelGGL(certified_reduce_wave_kernel, dim3(hq, bt), dim3(64), 0, st, ra);
  else
    hipLaunchKernelGGL(certified_reduce_kernel, dim3(hq, bt), dim3(64 * reduce_waves(nsplit)), 0, st, ra);
  CQA_HIP(hipGetLastError());
  return CQA_OK;
}

int32_t launch_step(Cache* c, int layer, const __half* q, const cqa_tolerances& tol, float* O, cqa_head_cert* cert,
                    uint32_t* flags, hipStream_t st, const __half* k_new, const __half* v_new, bool* launched) {
  const uint32_t tag = next_ladder_tag(c);
  ReduceArgs ra{};
  RowsBy by = RowsBy::launch;
  const int32_t rc = launch_certified(c, layer, q, tol, O, cert, flags, nullptr, 0u, nullptr, st, k_new, v_new, 0, nullptr,
                                      nullptr, ladder_raised(c), tag, &ra, &by);
  if (launched != nullptr) *launched = rc == CQA_OK;
  if (rc != CQA_OK) return rc;
  c->rows_by = by;
  c->rows_tag = tag;
  return launch_dense_ladder(c, layer, q, tol.rung4_min_groups, O, cert, flags, tag, st, by, &ra);
}

}  // namespace cqa
