// Cache-write kernels: seal a block of 16 tokens into Tier-1.
//
// Follows the paper's "Quantization Schemes" section: per-block per-channel INT8
// keys with sigma_c = (u_c - l_c)/255, z_c = l_c + 128 sigma_c, code =
// clamp(round((k - z_c)/sigma_c), -128, 127); per-token per-16-channel-group INT4
// values with an FP16 scale and offset; and the block annotations eta_b =
// max_t ||v_hat_t - v_t||_2, nu_b = max_t ||v_t||_2.
//
// All quantizer arithmetic is IEEE binary32 with one rounding per operation in
// the order written (subtract, divide; multiply, add; subtract, divide,
// round-half-even, clamp): contraction into fused multiply-adds is switched off
// for this file so codes and scales have exactly one correct value.
// Inputs are assumed finite.
#pragma clang fp contract(off)

#include <algorithm>

#include "cqa_internal.h"

namespace cqa {

struct SealArgs {
  const __half* k_in;   // [Bt][Hkv][n_new][128]
  const __half* v_in;
  __half* trail_k;      // [heads][16][128]
  __half* trail_v;
  uint8_t* t1;          // Tier-1 quad records
  float* sigmax;        // [Bt][Hkv] running max of sigma of the layer's sequences
  int64_t nq_cap;
  int64_t nb_old;       // sealed blocks before this append
  int64_t n_new;
  int r;                // tokens in the trailing block before this append
  int r_new;            // ... and after it: the last r_new of the new tokens
  int layer, batch, n_kv;
  int n_seal, runs;     // blocks to seal, workgroups per head: blocks w first, + step, + 2 step, ... of workgroup w, `most` of them
  int first, step, most;
  // the kernel also stores the FP16 originals of the new tokens into the pinned Tier-2 arrays, unless they go
  // through the copy engines (null)
  __half* t2_k;         // [heads][t2_cap][128]
  __half* t2_v;
  int64_t t2_cap;
  int64_t len_before;
};

// Quotient x / d for the quantizers, where only  round-half-even(fl(x / d))  is needed (fl = the
// correctly rounded binary32 quotient the definition asks for) and |x / d| < 2^8.  One IEEE division
// costs ten instructions and a block needs 4096 of them, so the quotient is first approximated as
// x * r with r = 1/d refined by one Newton step: the hardware reciprocal is within one unit in the
// last place, so after the step r is the rounded value of a number within 2^-44 of 1/d (relative
// error <= 2^-24), x * r carries one more rounding (2^-24), and |x r - x/d| <= 2^8 * 2^-23 = 2^-15;
// the exact quotient's own rounding moves it by at most 2^-17.  Unless the approximation lies
// within 2^-14 of a half-integer, both therefore round to the same integer; elements that
// are closer take the exact division.  Bit-identical to rintf(x / d) by construction.  (d = 0: r = 0,
// every code is 0.  A quotient that is not a number rounds to one, and its code saturates as the
// exact division's would.)
__device__ __forceinline__ float refined_rcp(float d) {
  const float r0 = __builtin_amdgcn_rcpf(d);
  return d != 0.0f ? fmaf(fmaf(-d, r0, 1.0f), r0, r0) : 0.0f;
}
constexpr float HALF_SAFE = 0.5f - 0.00006103515625f;

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
union H2 {
  uint32_t u;
  f16x2 h;
};
__device__ __forceinline__ uint32_t pk_min(uint32_t a, uint32_t b) {
  H2 x{a}, y{b}, r;
  r.h = __builtin_elementwise_min(x.h, y.h);
  return r.u;
}
__device__ __forceinline__ uint32_t pk_max(uint32_t a, uint32_t b) {
  H2 x{a}, y{b}, r;
  r.h = __builtin_elementwise_max(x.h, y.h);
  return r.u;
}
__device__ __forceinline__ float lo_f(uint32_t u) { return (float)H2{u}.h[0]; }
__device__ __forceinline__ float hi_f(uint32_t u) { return (float)H2{u}.h[1]; }

// FP64 lane exchanges for the block annotations
template <int CTRL>
__device__ __forceinline__ double dpp_d(double x) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(x);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// sum over the 4 lanes of an aligned quad, then the largest of the wave's 16 quads
__device__ __forceinline__ double quad_sum_wave_max_d(double x) {
  x += dpp_d<0xB1>(x);
  x += dpp_d<0x4E>(x);
  x = fmax(x, dpp_d<0x141>(x));
  x = fmax(x, dpp_d<0x140>(x));
  x = fmax(x, __shfl_xor(x, 16));
  return fmax(x, __shfl_xor(x, 32));
}
__device__ __forceinline__ void lds_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A wave stores the originals of 16 new tokens, first, first + 1, ... (those that are not negative), in runs of
// 1 KB: the link takes whole lines.  (The rows are in cache: the wave has just read them.)
__device__ __forceinline__ void store_originals(const __half* in, __half* t2, int64_t first) {
  const int l = threadIdx.x & 63;
  uint4 x[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t i = first + r * 4 + (l >> 4);
    if (i >= 0) x[r] = ld16_any(in + i * D + 8 * (l & 15));
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t i = first + r * 4 + (l >> 4);
    if (i >= 0) reinterpret_cast<uint4*>(t2 + i * D)[l & 15] = x[r];
  }
}

// One workgroup of two waves seals blocks of 16 tokens of a head, every `runs`-th or consecutive ones (seal_dealt), each wave requesting its
// share of the next block while it works on one; the waves do not wait for each other.  Where they are dealt the workgroups
// advance together, so a launch writes a window of consecutive records that moves through each head.
//   wave 0, keys   : lane = channels 2 l, 2 l + 1; its 2 x 16 values give l_c, u_c, sigma_c, z_c and the
//                    32 codes;
//   wave 1, values : lane = (token t, quarter p) = (l >> 2, l & 3), groups p and 4 + p; its 2 x 16 values
//                    give lo, hi, the FP16 scales and offsets, the 32 codes and the groups' share of
//                    the token's squared reconstruction error and squared norm (FP64).
// Codes pass through LDS, inside a wave, to reach the physical layout of the Tier-1 record.
// Bound by memory (8 KB in, 4.6 KB out per block) once the vector ALU keeps up: minima and maxima
// are taken on packed FP16, a code is one subtraction, product, rounding and saturating byte
// conversion, and elements near a half-integer are looked at again only in lanes that have one.
// 65549 tokens x 8 heads (268 MB in, 151 MB out): 168 us with both roles in every wave, one after the
// other; 105 us like this one block at a time, 95 us in runs of eight consecutive ones, 93 us = 4.5 TB/s dealt like this.  (Four
// waves per SIMD instead of three spill: 112 us; runs of 21 consecutive blocks: 108 us.  FP32 annotation sums: no faster.)
// The first workgroup of a head also moves the tokens that stay unsealed into the trailing block
// (it is the one that reads the old ones), the last clears the metadata of the blocks that
// its quad record does not hold yet (the decode pass reads whole records).
// (Measured and not adopted: fetching the keys as whole rows with 128-bit loads and handing the
// columns to the channel lanes through LDS.)
__global__ __launch_bounds__(128, 3) void seal_kernel(SealArgs a) {
  fetch_args<sizeof(SealArgs)>();
  const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int j = (int)blockIdx.x * a.first;    // new block index
  const int j1 = min(j + a.most * a.step, a.n_seal);
  const int kvh = blockIdx.y, b = blockIdx.z;
  const int64_t grp = (int64_t)b * a.n_kv + kvh;
  const int64_t head = (int64_t)a.layer * a.batch * a.n_kv + grp;
  const int64_t in_head = grp * a.n_new;
  const int64_t rec = head * a.nq_cap;

  __shared__ __align__(16) uint8_t kbuf[KC_BYTES];
  constexpr int VROW = D + 16;          // bytes per token in vnib (+16: rows t and t + 8 in different banks)
  __shared__ __align__(16) uint8_t vnib[BLK * VROW];
  __shared__ __align__(16) uint32_t vout[VC_BYTES / 4];
  __shared__ __align__(16) __half vmeta[2 * BLK * NG];

  if (w == 0) {
    // ---- keys
    // channels (2 l, 2 l + 1) of each token of the block in work and of the next one.  Token i of this
    // append is one of the r waiting ones, or new token i - r.
    uint32_t kx[BLK], kn[BLK];
    const u32_any* const kin = reinterpret_cast<const u32_any*>(a.k_in + (in_head - a.r) * D);
    if (j == 0 && a.r > 0) {            // the first block of an append that finds tokens waiting
      const u32_any* ktr = reinterpret_cast<const u32_any*>(a.trail_k + head * BLK * D);
#pragma unroll
      for (int t = 0; t < BLK; ++t) kn[t] = (t < a.r ? ktr : kin)[t * (D / 2) + l];
    } else {
#pragma unroll
      for (int t = 0; t < BLK; ++t) kn[t] = (kin + (int64_t)j * (BLK * D / 2))[t * (D / 2) + l];
    }
    float smax = 0.0f;
    for (; j < j1; j += a.step) {
      const int64_t blk = a.nb_old + j;
#pragma unroll
      for (int t = 0; t < BLK; ++t) kx[t] = kn[t];
      if (j + a.step < j1) {
#pragma unroll
        for (int t = 0; t < BLK; ++t) kn[t] = (kin + (int64_t)(j + a.step) * (BLK * D / 2))[t * (D / 2) + l];
      }
      uint32_t mn = kx[0], mx = kx[0];
#pragma unroll
      for (int t = 1; t < BLK; ++t) {
        mn = pk_min(mn, kx[t]);
        mx = pk_max(mx, kx[t]);
      }
      const float lo[2] = {lo_f(mn), hi_f(mn)}, hi[2] = {lo_f(mx), hi_f(mx)};
      float sg[2], z[2], r[2], near = 0.0f;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        sg[e] = (hi[e] - lo[e]) / 255.0f;
        z[e] = lo[e] + 128.0f * sg[e];
        r[e] = refined_rcp(sg[e]);
      }
      uint32_t code[BLK];                 // two biased codes per token
#pragma unroll
      for (int t = 0; t < BLK; ++t) {
        code[t] = 0u;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const float x = fmaf(e == 0 ? lo_f(kx[t]) : hi_f(kx[t]), 1.0f, -z[e]);   // k - z, one rounding
          const float qa = x * r[e];
          const float q = rintf(qa);
          near = fmaxf(near, fabsf(qa - q));
          code[t] = __builtin_amdgcn_cvt_pk_u8_f32(q + 128.0f, e, code[t]);        // saturates at 0 and 255
        }
      }
      if (near > HALF_SAFE) {
        // (hides from the compiler that the quotients are the same: kept from above they cost 50 registers)
        asm volatile("" : "+v"(r[0]), "+v"(r[1]));
#pragma unroll
        for (int t = 0; t < BLK; ++t)
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const float x = fmaf(e == 0 ? lo_f(kx[t]) : hi_f(kx[t]), 1.0f, -z[e]);
            const float qa = x * r[e];
            if (fabsf(qa - rintf(qa)) > HALF_SAFE)
              code[t] = __builtin_amdgcn_cvt_pk_u8_f32(rintf(x / sg[e]) + 128.0f, e, code[t]);
          }
      }
      const int koff = kc_offset(0, 2 * l);
#pragma unroll
      for (int t = 0; t < BLK; ++t) *reinterpret_cast<uint16_t*>(&kbuf[koff + t * 16]) = (uint16_t)code[t];
      float* km = reinterpret_cast<float*>(a.t1 + t1_offset(rec, blk, Q_KM, KM_BYTES));
      reinterpret_cast<float2*>(km)[l] = make_float2(sg[0], sg[1]);
      reinterpret_cast<float2*>(km + D)[l] = make_float2(z[0], z[1]);
      lds_wave_sync();
      uint8_t* kc = a.t1 + t1_offset(rec, blk, Q_KC, KC_BYTES);
      reinterpret_cast<uint4*>(kc)[l] = reinterpret_cast<const uint4*>(kbuf)[l];
      reinterpret_cast<uint4*>(kc)[64 + l] = reinterpret_cast<const uint4*>(kbuf)[64 + l];
      smax = fmaxf(smax, fmaxf(sg[0], sg[1]));
      if (a.t2_k != nullptr) store_originals(a.k_in + in_head * D, a.t2_k + (head * a.t2_cap + a.len_before) * D, (int64_t)j * BLK - a.r);
      lds_wave_sync();
    }
    // running maximum of sigma over the head's blocks (used by the decode pass to pick an
    // overflow-free power-of-two scaling); sigma >= 0, so its bit pattern orders like an int
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) smax = fmaxf(smax, __shfl_xor(smax, m));
    // thousands of blocks of one head would queue up on the same word: the running maximum is
    // read first (within a launch it only grows, so a stale value merely costs a redundant atomic) and the
    // atomic is issued only by a workgroup that raises it
    if (l == 0) {
      int* const word = reinterpret_cast<int*>(a.sigmax + grp);
      if (a.nb_old == 0 && a.runs == 1)
        *word = __float_as_int(smax);   // the sequence's first blocks, and no other workgroup has any: starts afresh
      else if (__float_as_int(smax) > __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMax(word, __float_as_int(smax));
    }
  } else {
    // ---- values
    const int t = l >> 2, p = l & 3;
    uint4 raw[2][2], nxt[2][2];
    const __half* const vin = a.v_in + (in_head - a.r + t) * D;
    {
      const __half* row = (int64_t)j * BLK + t < a.r ? a.trail_v + (head * BLK + t) * D : vin + (int64_t)j * (BLK * D);
#pragma unroll
      for (int k = 0; k < 4; ++k) nxt[k >> 1][k & 1] = ld16_any(row + 8 * (8 * (k >> 1) + 2 * p + (k & 1)));
    }
    for (; j < j1; j += a.step) {
      const int64_t blk = a.nb_old + j;
#pragma unroll
      for (int k = 0; k < 4; ++k) raw[k >> 1][k & 1] = nxt[k >> 1][k & 1];
      if (j + a.step < j1) {
        const __half* row = vin + (int64_t)(j + a.step) * (BLK * D);
#pragma unroll
        for (int k = 0; k < 4; ++k) nxt[k >> 1][k & 1] = ld16_any(row + 8 * (8 * (k >> 1) + 2 * p + (k & 1)));
      }
      double e2 = 0.0, n2 = 0.0;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int g = 4 * k + p;
        const uint32_t vx[8] = {raw[k][0].x, raw[k][0].y, raw[k][0].z, raw[k][0].w,
                                raw[k][1].x, raw[k][1].y, raw[k][1].z, raw[k][1].w};
        uint32_t mn = vx[0], mx = vx[0];
#pragma unroll
        for (int e = 1; e < 8; ++e) {
          mn = pk_min(mn, vx[e]);
          mx = pk_max(mx, vx[e]);
        }
        const float vlo = fminf(lo_f(mn), hi_f(mn)), vhi = fmaxf(lo_f(mx), hi_f(mx));
        const __half sh = __float2half_rn((vhi - vlo) / 15.0f);
        const float sc = __half2float(sh);
        float rs = refined_rcp(sc);
        float q[VG], near = 0.0f;
#pragma unroll
        for (int e = 0; e < VG; ++e) {
          const float x = fmaf((e & 1) ? hi_f(vx[e >> 1]) : lo_f(vx[e >> 1]), 1.0f, -vlo);   // v - lo, one rounding
          const float qa = x * rs;
          const float qr = rintf(qa);
          near = fmaxf(near, fabsf(qa - qr));
          q[e] = fminf(fmaxf(qr, 0.0f), 15.0f);
        }
        if (near > HALF_SAFE) {
          asm volatile("" : "+v"(rs));
#pragma unroll
          for (int e = 0; e < VG; ++e) {
            const float x = fmaf((e & 1) ? hi_f(vx[e >> 1]) : lo_f(vx[e >> 1]), 1.0f, -vlo);
            const float qa = x * rs;
            if (fabsf(qa - rintf(qa)) > HALF_SAFE) q[e] = fminf(fmaxf(rintf(x / sc), 0.0f), 15.0f);
          }
        }
        uint32_t packed[4] = {0u, 0u, 0u, 0u};   // the group's 16 codes, one per byte, channel order
        const double dlo = (double)vlo, dsc = (double)sc;
#pragma unroll
        for (int e = 0; e < VG; ++e) {
          packed[e >> 2] = __builtin_amdgcn_cvt_pk_u8_f32(q[e], e & 3, packed[e >> 2]);
          // v_hat - v = code * scale + (lo - v): the product is exact (4 x 11 bits), the difference and the
          // sum are taken in double
          const double dv = (double)((e & 1) ? hi_f(vx[e >> 1]) : lo_f(vx[e >> 1]));
          const double err = fma((double)q[e], dsc, dlo - dv);
          e2 = fma(err, err, e2);
          n2 = fma(dv, dv, n2);
        }
        *reinterpret_cast<uint4*>(&vnib[t * VROW + g * VG]) = make_uint4(packed[0], packed[1], packed[2], packed[3]);
        vmeta[vm_index(t, g)] = sh;
        vmeta[BLK * NG + vm_index(t, g)] = __float2half_rn(vlo);  // exact: vlo is an FP16 input
        __builtin_amdgcn_sched_barrier(0);   // the groups one after the other (registers)
      }
      lds_wave_sync();
      // eight tokens (octet o) x four channels: token pairs share a byte, then a 4 x 4 byte transpose
      {
        const int o = l >> 5, cc = l & 31;
        uint32_t wd[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) wd[k] = *reinterpret_cast<const uint32_t*>(&vnib[(o * 8 + k) * VROW + 4 * cc]);
        uint32_t pr[4];                   // byte c = channel c of tokens 2 k (low nibble), 2 k + 1
#pragma unroll
        for (int k = 0; k < 4; ++k) pr[k] = wd[2 * k] | (wd[2 * k + 1] << 4);
        const uint32_t a01 = __builtin_amdgcn_perm(pr[1], pr[0], 0x05010400u), a23 = __builtin_amdgcn_perm(pr[3], pr[2], 0x05010400u);
        const uint32_t b01 = __builtin_amdgcn_perm(pr[1], pr[0], 0x07030602u), b23 = __builtin_amdgcn_perm(pr[3], pr[2], 0x07030602u);
        const uint32_t out[4] = {__builtin_amdgcn_perm(a23, a01, 0x05040100u), __builtin_amdgcn_perm(a23, a01, 0x07060302u),
                                 __builtin_amdgcn_perm(b23, b01, 0x05040100u), __builtin_amdgcn_perm(b23, b01, 0x07060302u)};
#pragma unroll
        for (int k = 0; k < 4; ++k) vout[vc_dword_offset(o, 4 * cc + k) / 4] = out[k];
      }
      lds_wave_sync();
      reinterpret_cast<uint4*>(a.t1 + t1_offset(rec, blk, Q_VC, VC_BYTES))[l] = reinterpret_cast<const uint4*>(vout)[l];
      reinterpret_cast<uint2*>(a.t1 + t1_offset(rec, blk, Q_VM, VM_BYTES))[l] = reinterpret_cast<const uint2*>(vmeta)[l];
      e2 = quad_sum_wave_max_d(e2);
      n2 = quad_sum_wave_max_d(n2);
      if (l == 0)
        *reinterpret_cast<float2*>(a.t1 + t1_offset(rec, blk, Q_AN, AN_BYTES)) = make_float2((float)sqrt(e2), (float)sqrt(n2));
      if (a.t2_v != nullptr) store_originals(a.v_in + in_head * D, a.t2_v + (head * a.t2_cap + a.len_before) * D, (int64_t)j * BLK - a.r);
      lds_wave_sync();
    }
  }

  if (blockIdx.x == 0) {
    // the last r_new new tokens: to the trailing block, whose old tokens this wave has consumed, and, for
    // short appends, to Tier 2 (16 lanes per token row)
    const __half* in = w == 0 ? a.k_in : a.v_in;
    __half* tr = w == 0 ? a.trail_k : a.trail_v;
    __half* t2 = w == 0 ? a.t2_k : a.t2_v;
    for (int t = l >> 4; t < a.r_new; t += 4) {
      const int64_t src = a.n_new - a.r_new + t;
      const uint4 x = ld16_any(in + (in_head + src) * D + 8 * (l & 15));
      reinterpret_cast<uint4*>(tr + (head * BLK + t) * D)[l & 15] = x;
      if (t2 != nullptr) reinterpret_cast<uint4*>(t2 + (head * a.t2_cap + a.len_before + src) * D)[l & 15] = x;
    }
  }
  if (j1 == a.n_seal && (a.step == 1 || (a.n_seal - 1) % a.step == (int)blockIdx.x)) {
    const uint4 zero = make_uint4(0u, 0u, 0u, 0u);
    for (int64_t nb = a.nb_old + a.n_seal; (nb & 3) != 0; ++nb) {
      if (w == 0) {
        reinterpret_cast<uint4*>(a.t1 + t1_offset(rec, nb, Q_KM, KM_BYTES))[l] = zero;
      } else {
        reinterpret_cast<uint2*>(a.t1 + t1_offset(rec, nb, Q_VM, VM_BYTES))[l] = make_uint2(0u, 0u);
        if (l == 0) *reinterpret_cast<float2*>(a.t1 + t1_offset(rec, nb, Q_AN, AN_BYTES)) = make_float2(0.0f, 0.0f);
      }
    }
  }
}

// The running maxima of sigma start afresh with the first blocks of a sequence.  The device does it, in stream
// order, at the one address that they always have: a decode, or an append, that was recorded into a graph and is
// replayed after a reset then reads what an eager call would.  One small launch, 2 - 3 us, ahead of a first seal of
// several workgroups (a single workgroup per head simply stores its maximum).  (Instead of it, an epoch in pinned
// memory that a reset raises and every workgroup puts above its maximum: a prompt of 65549 tokens 140 -> 435 us,
// reads of one host word are served one after the other.  A word per workgroup, all set by the first seal and
// reduced by every decode: nothing for the prompt, but 0.1 us for each short step and 101.0 -> 102.2 for 64 x 4107 tokens.)
__global__ __launch_bounds__(256) void clear_sigmax_kernel(float* sigmax, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) sigmax[i] = 0.0f;
}

// An append that completes no block: its tokens join the trailing block and, with
// Tier 2, the FP16 originals go straight into the pinned arrays (device stores to mapped host
// memory: a decode-time append of one token per head is one small launch).  16 lanes per token row.
// dst_first: slot of the first new token; n_new < 16.  t2_k / t2_v: null = Tier-2 handled elsewhere.
__global__ __launch_bounds__(256) void trail_kernel(const __half* k_in, const __half* v_in,
                                                    __half* trail_k, __half* trail_v, int n_new,
                                                    int dst_first, int layer, int batch, int n_kv,
                                                    __half* t2_k, __half* t2_v, int64_t t2_cap,
                                                    int64_t len_before) {
  const int t = threadIdx.x >> 4, c = threadIdx.x & 15;
  const int kvh = blockIdx.x, b = blockIdx.y;
  const int64_t head = ((int64_t)layer * batch + b) * n_kv + kvh;
  const int64_t in_head = ((int64_t)b * n_kv + kvh) * n_new;
  if (t >= n_new) return;
  const uint4 k = ld16_any(k_in + (in_head + t) * D + 8 * c);
  const uint4 v = ld16_any(v_in + (in_head + t) * D + 8 * c);
  reinterpret_cast<uint4*>(trail_k + (head * BLK + dst_first + t) * D)[c] = k;
  reinterpret_cast<uint4*>(trail_v + (head * BLK + dst_first + t) * D)[c] = v;
  if (t2_k != nullptr) {
    reinterpret_cast<uint4*>(t2_k + (head * t2_cap + len_before + t) * D)[c] = k;
    reinterpret_cast<uint4*>(t2_v + (head * t2_cap + len_before + t) * D)[c] = v;
  }
}

// Whether a launch that seals deals the blocks round `runs` workgroups per head, all of them resident at once (four to a compute
// unit, six, as many as there is room for, from 8192 blocks on), or cuts each head into short runs of consecutive ones, which the hardware
// hands out as workgroups end.  Dealt, the launch has no last generation that leaves part of the chip idle: us, dealt over four, over six and
// in runs of up to eight: 2 x 8 heads of 4000 tokens 37.3, 42.8, 56.8; 8 of 5000 30.7, 32.9, 39.9; 8 of 32000 63.3, 58.6, 63.6; 64 of
// 8200 115.5, 115.9, 142.7; 512 of 2000 200.3, 202.3, 222.8; 8 of 65549 112.1, 107.9, 109.8.
// That holds while the one generation fills the chip.  From about 500 heads on a head has one or two workgroups, and what is left over of a
// compute unit's six places, or a second generation of whole heads, costs more (2000 tokens, dealt and consecutive: 520 heads 244, 221; 800 348, 321;
// 1100 471, 428; 1600 738, 601; 3200 1255, 1158; but 480 196, 208; 1000 366, 390; 1500 555, 567; 290 tokens: 1100 79, 75; 1600 115, 101;
// but 700 52, 56; 1500 88, 95).  Both times in blocks of the busiest compute unit: consecutive, an equal share and a tail; dealt, blocks a workgroup
// times what w of them to a compute unit cost (two waves each: beyond four, a SIMD has a third wave), from the times at 11, 18, 40 and 125 blocks and
// 520 to 1500 heads, whose ratios it gives within 5 % (furthest off: 1300 heads of 290 tokens, dealt 87, consecutive 90, are not dealt).
// Heads of a thousand blocks and more are the better read and written one after the other when there are many (100 of 1000 blocks
// level, 130 402, 382, 330 1041, 911), and several of 32000 tokens and more because the first decode, which walks all heads side by side, finds more of them in
// the memory-side cache (8 of 65549, prompt and decode: dealt 141.5, consecutive 139.5).
// Heads of up to ten blocks lose nothing by it at any number (2000 of 4 blocks 37.6, 48.6), nor do those of up to thirteen beyond a generation (2500 of 13 113, 119).
static bool seal_dealt(int64_t n_seal, int64_t heads, int64_t runs, int n_cu) {
  const int64_t blocks = n_seal * heads;
  if (n_seal >= 2048 && blocks >= 16384) return false;
  if (n_seal >= 1000 && blocks > 100000) return false;
  if (n_seal <= 10) return true;
  if (heads * runs > 6 * (int64_t)n_cu) return n_seal <= 13;
  const double w = (double)(heads * runs) / n_cu, n = (double)n_seal;
  const double tail = std::min(std::max(0.3 * n, 7.0), std::max(55.0 - n / 20, 7.0));
  return n / runs * (w <= 4 ? 1.95 + 0.51 * w : 3.0 + 0.5 * w) <= (double)blocks / n_cu + tail;
}

int32_t launch_seal(Cache* c, int layer, const __half* k_in, const __half* v_in, int64_t n_new,
                    int64_t len_before, bool tier2_by_kernel, hipStream_t st) {
  const int r = (int)(len_before % BLK);
  const int64_t n_seal = (r + n_new) / BLK;
  const int bt = c->desc.batch, hkv = c->desc.n_kv_heads;
  if (n_seal > 0) {
    SealArgs a;
    a.k_in = k_in;
    a.v_in = v_in;
    a.trail_k = c->trail_k;
    a.trail_v = c->trail_v;
    a.t1 = c->t1;
    a.sigmax = c->sigmax + head_index(c, layer, 0, 0);
    a.nq_cap = c->nq_cap;
    a.nb_old = len_before / BLK;
    a.n_new = n_new;
    a.r = r;
    a.r_new = (int)((r + n_new) % BLK);
    a.layer = layer;
    a.batch = bt;
    a.n_kv = hkv;
    a.t2_k = tier2_by_kernel ? c->t2_k : nullptr;
    a.t2_v = tier2_by_kernel ? c->t2_v : nullptr;
    a.t2_cap = c->desc.max_tokens;
    a.len_before = len_before;
    a.n_seal = (int)n_seal;
    const int64_t heads = (int64_t)bt * hkv, most_wgs = (n_seal * heads < 8192 ? 4 : 6) * (int64_t)c->n_cu;
    const int64_t one_gen = std::min<int64_t>(n_seal, std::max<int64_t>(most_wgs / heads, 1));
    if (seal_dealt(n_seal, heads, one_gen, c->n_cu)) {
      a.runs = (int)one_gen;
      a.first = 1;
      a.step = a.runs;
      a.most = (int)((n_seal + one_gen - 1) / one_gen);
    } else {   // consecutive blocks: one per workgroup until there are two thousand of them, then up to eight
      a.most = (int)std::min<int64_t>(std::max<int64_t>(n_seal * heads / 2048, 1), 8);
      a.runs = (int)((n_seal + a.most - 1) / a.most);
      a.first = a.most;
      a.step = 1;
    }
    const unsigned runs = (unsigned)a.runs;
    if (a.nb_old == 0 && runs > 1) {
      const int n = bt * hkv;
      hipLaunchKernelGGL(clear_sigmax_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, a.sigmax, n);
      CQA_HIP(hipGetLastError());
    }
    hipLaunchKernelGGL(seal_kernel, dim3(runs, hkv, bt), dim3(128), 0, st, a);
    CQA_HIP(hipGetLastError());
    return CQA_OK;
  }
  hipLaunchKernelGGL(trail_kernel, dim3(hkv, bt), dim3(256), 0, st, k_in, v_in, c->trail_k, c->trail_v, (int)n_new, r,
                     layer, bt, hkv, tier2_by_kernel ? c->t2_k : nullptr, tier2_by_kernel ? c->t2_v : nullptr,
                     (int64_t)c->desc.max_tokens, len_before);
  CQA_HIP(hipGetLastError());
  return CQA_OK;
}

}  // namespace cqa
