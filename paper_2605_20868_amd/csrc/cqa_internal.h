// Internal declarations shared by the library's translation units (not installed).
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include "../../include/cqa.h"
#include "../../include/cqa_test.h"

namespace cqa {

// ---- fixed geometry (the paper's defaults: d = 128, B = 16, g = 16) ------------
constexpr int D = 128;          // head dimension
constexpr int BLK = 16;         // tokens per block
constexpr int VG = 16;          // value channels per group
constexpr int NG = D / VG;      // 8 value groups per token

// ---- physical Tier-1 layout, per sealed block ---------------------------------
// Five block-major streams per (layer, batch, kv-head); block b of a head lives at
// offset b * <bytes per block> in each stream, so one split of the decode pass
// reads five contiguous byte ranges.
//
// K codes (2048 B): biased bytes u = code + 128, ordered [cq][kg][token][j] with
//   channel = cq*64 + kg*16 + j  (cq in 0..1, kg in 0..3, j in 0..15), so a wave's
//   lane l = kg*16 + token reads one aligned 16-byte piece and the whole wave reads
//   1 KB contiguously per cq.
// K meta (1024 B): sigma[128] then z[128], FP32, natural channel order.
// V codes (1024 B): dwords ordered [o][gh][n][gq]; the dword of (o, g = gh*4+gq, n)
//   holds channel g*16+n of the eight tokens o*8 .. o*8+7, token i in bits 4i..4i+3.
// V meta (512 B): FP16 scale[o][g][i] (256 B) then FP16 offset[o][g][i] (256 B),
//   token = o*8 + i.
// Annotations (8 B): float eta_b, float nu_b.
constexpr int KC_BYTES = BLK * D;            // 2048
constexpr int KM_BYTES = 2 * D * 4;          // 1024
constexpr int VC_BYTES = BLK * D / 2;        // 1024
constexpr int VM_BYTES = 2 * BLK * NG * 2;   // 512
constexpr int AN_BYTES = 8;

// The five per-block pieces of four consecutive blocks (a "quad") are stored together as one
// contiguous record, piece-major inside the record:
//   [K codes 4 x 2048][K meta 4 x 1024][V codes 4 x 1024][V meta 4 x 512][annotations 4 x 8]
// so that a wave, which works on one quad at a time, streams a single 18464-byte run instead of
// five separate arrays (measured: 7.1 TB/s against 6.5 TB/s for the same bytes in five arrays).
// The sigma, z, scale, offset, eta and nu of blocks that are not sealed (yet) read as zeros in every record
// that holds a sealed block: the memory is cleared at creation, and the seal that ends inside a
// record clears the rest of it.
constexpr int Q_KC = 0;
constexpr int Q_KM = Q_KC + 4 * KC_BYTES;   //  8192
constexpr int Q_VC = Q_KM + 4 * KM_BYTES;   // 12288
constexpr int Q_VM = Q_VC + 4 * VC_BYTES;   // 16384
constexpr int Q_AN = Q_VM + 4 * VM_BYTES;   // 18432
constexpr int QUAD_DATA_BYTES = Q_AN + 4 * AN_BYTES;            // 18464 = 64 tokens x 288.5 B
// records start on 128-byte lines (96 bytes of padding, 0.5 %): every 1 KB wave load then covers
// exactly 8 lines and no line is shared between two records
constexpr int QUAD_BYTES = (QUAD_DATA_BYTES + 127) / 128 * 128;    // 18560

// address of one piece of block `blk` of head-local numbering; `head_rec` = first record of the head
__host__ __device__ inline int64_t t1_offset(int64_t head_rec, int64_t blk, int piece_off,
                                             int piece_bytes) {
  return (head_rec + (blk >> 2)) * QUAD_BYTES + piece_off + (blk & 3) * piece_bytes;
}

__host__ __device__ inline int kc_offset(int token, int channel) {
  const int cq = channel >> 6, kg = (channel >> 4) & 3, j = channel & 15;
  return cq * 1024 + kg * 256 + token * 16 + j;
}
// byte offset of the dword holding (token octet o, channel c); nibble index = token & 7
__host__ __device__ inline int vc_dword_offset(int o, int channel) {
  const int g = channel >> 4, n = channel & 15;
  return o * 512 + (g >> 2) * 256 + n * 16 + (g & 3) * 4;
}
// index (in halves) of the scale of (token, group) inside the V-meta block; offsets follow at +128
__host__ __device__ inline int vm_index(int token, int g) {
  return (token >> 3) * 64 + g * 8 + (token & 7);
}

// ---- split partial written by the decode pass, merged by the reduction ---------
// Per (batch, q-head, split): PART_FLOATS floats.
constexpr int P_M = 0;      // running max of the split
constexpr int P_L = 1;      // sum of exp(s - m)
constexpr int P_EV = 2;     // sum_b S_b e^{m_b - m} eta_b
constexpr int P_EVMAX = 3;  // max_b S_b e^{m_b - m} eta_b
constexpr int P_DMAX = 4;   // max_b Delta_b
constexpr int P_VMAX = 5;   // max_b nu_b
constexpr int P_T1 = 6;     // largest block log-mass
constexpr int P_T2 = 7;     // second largest
constexpr int P_I1 = 8;     // block index of the largest (int bits)
constexpr int P_O = 16;     // o[128]
constexpr int PART_FLOATS = 16 + D;  // 144
constexpr int MAX_SPLITS = 1024;     // upper bound on splits per (batch, kv-head)

// ---- split pass that reduces its partial sets itself (certified_split_mfma_kernel) ----
constexpr int DIES = 8;              // workgroups whose indices leave the same remainder by 8 run on one die
constexpr int TICKET_STRIDE = 32;    // words: a KV group's counters, one per die, have a line of their own
constexpr int REDUCED_ROWS = 4 * 32 * DIES;   // most (batch, query head) rows of such a step, with a KV group per compute unit: the ladder's
                                              // launch keeps as many flag words in LDS
// Most sets that its last workgroup joins, of `waves` waves, `quad_waves` of them with quads, for `group` heads: eight by each row of
// waves (one wave per head) but the one that takes the side work, so none where there is no other; the rows' results take
// the places of the quad waves' states.
__host__ __device__ constexpr int reduced_sets(int group, int quad_waves, int waves) {
  const int rows = waves / group - 1;
  return 8 * (rows < quad_waves ? rows : quad_waves);
}

// ---- adaptive key precision ------------------------------------------------------
constexpr int MAX_K_LIMIT = 512;            // blocks one head may promote (Rung-1 growth included)
constexpr int MAX_UNION = 8 * MAX_K_LIMIT;  // blocks one KV group may promote (keys and values, <= 4 heads each)
constexpr int PROM_SPLITS = 16;             // workgroups (= partial sets) per KV group of each half of the promoted-block
                                            // pass: 64 waves, about two blocks per wave for a group that promotes K_max = 128.
                                            // An adaptive step with 8, 16 and 32 per half: one group of 8000 tokens 85, 70, 71 us
                                            // (too few waves for large unions); 32K 152, 151, 154; 128K 122, 124, 126; 4 x 20000
                                            // 640, 635, 651; 16 x 4000 2105, 2103, 2155 (more sets to merge than the waves gain)

// Workspace of the adaptive path, shared by all layers (one decode step at a time).
// What a run of up to SCAN_PART blocks left in INT8 adds up to for one head: over the blocks that are not key-promoted for
// the head, the estimated mass and the largest log-mass; over those that are not listed at all, relative to lse, the mass,
// the value term and the largest share of it.
struct ScanPart {
  double alpha, l8u, ev8u;
  float top, maxc8;
};
constexpr int SCAN_PART = 8192, SUM_WAVE_BLOCKS = 2048;
inline int64_t scan_parts(int64_t n_blocks) { return (n_blocks + SCAN_PART - 1) / SCAN_PART; }

struct AdaptiveWs {
  float* lm8;        // [Bt][Hq][nb_cap]      INT8 block log-masses of the pass over all blocks
  float* lmx;        // [Bt][Hq][nb_cap]      log-masses of the listed blocks as the promoted-block pass computed them (FP16 keys where promoted)
  int32_t* sel;      // [Bt][Hq][MAX_K_LIMIT] the head's own selection, best first
  int32_t* kstar;    // [Bt][Hq]              its size after Rung-1 growth
  float* alpha;      // [Bt][Hq]              estimated mass of the blocks its group left in INT8
  uint32_t* umask;   // [Bt][Hq][mask_words]  the head's key selection, one bit per block
  uint32_t* vmask;   // [Bt][Hq][mask_words]  its value selection
  int32_t* slot;     // [Bt][Hkv][4 nq_cap]   per block: bit 0 = FP16 keys, bit 1 = FP16 values (0 = neither), per-head bits above
  float* eta_blk;    // [Bt][Hkv][nb_cap]     eta_b as read by the pass over all blocks
  float* contrib;    // [Bt][Hq][nb_cap]      estimated contributions p_b eta_b
  int32_t* vsel;     // [Bt][Hq][MAX_K_LIMIT] the head's value selection
  int32_t* vcount;   // [Bt][Hq]
  float* score_dev;  // [Bt][Hq]              canary: largest |s_fp16 - s_int8| on key-promoted tokens
  int32_t* ucount;   // [Bt][Hkv]             promoted blocks of the group
  int32_t* ulist;    // [Bt][Hkv][MAX_UNION]  their indices, ascending
  float* first;      // [Bt][Hq][4]           lse, Delta_h, V_max of the pass over all blocks
  ScanPart* scan;    // [Bt][Hq][parts]       what the blocks its group left in INT8 add up to
  int64_t mask_words;
  // FP16 scratch (the paper's VRAM scratch cache of promoted originals, LRU): per (layer, batch,
  // kv-head) `sc_cap` slots of one block each, a key half and a value half.  sc_map: block ->
  // slot + 1 (0 = not held); sc_tag: slot -> block (-1 = empty); sc_age: slot -> step stamp of its
  // last use; sc_have: slot -> which halves hold the block's data (SLOT_KEYS | SLOT_VALUES).
  __half* sc_k;      // [heads_total][sc_cap][16][128]
  __half* sc_v;      // [heads_total][sc_cap][16][128]
  int32_t* sc_map;   // [heads_total][nb_cap]
  int32_t* sc_tag;   // [heads_total][sc_cap]
  uint32_t* sc_age;  // [heads_total][sc_cap]
  int32_t* sc_have;  // [heads_total][sc_cap]
  uint32_t* sc_stats;  // [2] promoted blocks whose originals were all in the scratch / were not, over all steps
  int sc_cap;        // allocated slots per head (a power of two <= SC_MAX_SLOTS)
  int sc_slots;      // slots in use (test hook may lower it; 0 = scratch off)
  uint32_t sc_step;  // stamp of the last adaptive step
};

constexpr int MAX_RANK_DEPTH = 8;   // largest depth r of the ranking check (adaptive path)
constexpr int SC_MAX_SLOTS = 1024;
// per-block word of AdaptiveWs::slot: bit 0 FP16 keys, bit 1 FP16 values, bit 2 / bit 3 the keys /
// the values are to be stored into the scratch slot by the pass that reads them from the host,
// bits 8-23 scratch slot + 1 (0 = none)
constexpr int SLOT_KEYS = 1, SLOT_VALUES = 2, SLOT_FILL = 4, SLOT_VFILL = 8, SLOT_SC_SHIFT = 8;
// bits 24-27: query head i of the group (i = 0..3) scores this block with FP16 keys; bits 28-31: it
// attends the block's FP16 values.  With per-group promotion every head's bit follows bits 0 / 1.
constexpr int SLOT_HK_SHIFT = 24, SLOT_HV_SHIFT = 28;

// Who reduces the rows of an enqueue-only step: a launch of its own (or the split pass of a one-workgroup sequence); the split
// pass, and the ladder's launch looks after it; the ladder's launch.
enum class RowsBy { launch, split, ladder };

struct Cache {
  cqa_cache_desc desc;
  int device;
  int n_cu;
  int64_t nb_cap;            // blocks of capacity per head
  int64_t heads_total;       // n_layers * batch * n_kv_heads
  int64_t* length;           // host, per layer
  int forced_splits;
  int max_splits;
  // Tier-1: quad records, [heads_total][nq_cap][QUAD_BYTES]
  uint8_t* t1;
  int64_t nq_cap;            // quad records of capacity per head
  float* ladder_ws;          // device-resolved ladder: split partials, arrival counters, rung counters
  uint32_t* ladder_tickets;
  uint32_t* ladder_counts;   // [2] steps served by Rung 3 / 4, [1] word of the last step that raised a flag
  uint32_t ladder_seq;       // host: number of the last enqueue-only step, never 0
  uint32_t* tickets;         // the allocation of split_tickets and ladder_tickets
  uint32_t* split_tickets;   // of the split pass that reduces its partial sets itself (split_reduces): [batch * n_kv_heads][TICKET_STRIDE]
                             // arrivals on each die, zero between launches, then [batch * n_kv_heads] the number of the last
                             // step whose rows are reduced; null = it leaves the reduction to a launch of its own
  uint32_t* strayed;         // pinned, behind flags_host: not 0 once the workgroups of a KV group were not on one die in such a step, after
                             // which steps leave the reduction to a launch of its own
  int scatter;               // test hook: every other workgroup of a KV group counts as one of the next die
  RowsBy rows_by;            // of the last enqueue-only step, whose number is ...
  uint32_t rows_tag;
  float* sigmax;             // [heads_total] running max of sigma (non-negative: ordered as ints) over the sealed
                             // blocks; a sequence's first seal sets it, so it holds nothing while there are none
  // trailing FP16 partial blocks [heads_total][16][128]
  __half* trail_k;
  __half* trail_v;
  // Tier-2 (pinned host) [heads_total][max_tokens][128]
  __half* t2_k;
  __half* t2_v;
  bool t2_borrowed;           // the originals' arrays belong to the caller (not freed here)
  // workspaces
  float* partials;           // [batch][Hq][max_splits][PART_FLOATS]
  float* dense_ws;           // dense partials for one (batch, kv-head) group x 2 buffers
  __half* stage[2][2];       // [buffer][K|V] : max_tokens * 128 halves each
  uint32_t* select_dev;      // [batch][Hq]
  uint32_t* flags_host;      // pinned [batch][Hq], and a word more: strayed
  uint32_t step_seq;         // 16-bit tag of the decode step whose flags the mirror must carry
  uint32_t* need;            // host [batch][Hq]: ladder scratch, heads to recompute
  hipStream_t side;
  hipEvent_t ev_ready[2];    // staging buffer filled (recorded on side)
  hipEvent_t ev_free[2];     // staging buffer consumed (recorded on main)
  hipEvent_t ev_main;        // main-stream marker the side stream waits on
  hipEvent_t ev_copy;         // bulk append: the copies of the originals on the side stream are done
  hipEvent_t ev_t0, ev_t1;   // timing
  bool free_valid[2];
  // optional per-launch timing of the split kernel (pairs of events on the launch stream)
  hipEvent_t* prof_ev;
  int prof_cap, prof_n;
  float* prof_ms;            // host: durations of the launches timed by the last begin / end pair
  int prof_ms_n;
  int variant;               // 0 = matrix-core split kernel (default), 1 = vector-ALU split kernel
  int stream_hint;           // Tier-1 loads: 0 = chosen from the footprint, 1 = plain, 2 = non-temporal
  AdaptiveWs ad;             // allocated with the cache when Tier-2 is retained
};

struct DecodeArgs {
  // what the first loads' addresses are made of, one 64-byte line of kernel arguments (args_in_one_wait)
  const uint8_t* t1;   // layer base of the Tier-1 quad records
  const float* sigmax; // [Bt * Hkv] of the layer: running max of sigma over sealed blocks and channels
  const __half* q;     // [Bt][Hq][128]
  const __half* ap_k_new;   // [Bt][Hkv][1][128]: see below
  int64_t nq_cap;      // quad records per head
  int nb;              // sealed blocks
  int nsplit;
  int n_q, n_kv;
  int pstride;         // partial sets per (batch, q-head) row of `partials` (>= nsplit)
  int finish;          // matrix-core pass: 1 = it finishes the rows of a single split itself
  // matrix-core pass that reduces several splits itself (split_reduces)
  uint32_t* tickets;   // split_tickets, or null: it does not
  int heads;           // Bt * Hkv
  int scatter;         // test hook
  float* partials;     // [Bt][Hq][nsplit][PART_FLOATS]
  float* blk_logmass;  // [Bt][Hq][nb] or null
  int int8_query;      // matrix-core pass: 1 = INT8 x INT8 scoring of the quantised scaled query
  int wpb;             // matrix-core pass: waves per workgroup that take quads, 8 or 4 (split_geometry)
  int waves;           // ... and in all, where it reduces several splits itself (split_reduces)
  int settle;          // ... four of several quads each wait for all of their first one (certified_split_mfma_kernel)
  // promoted-block pass of the adaptive decode
  __half* sc_k;             // layer base of the FP16 scratch's key halves [Bt * Hkv][sc_cap][16][128], or null
  __half* sc_v;             // ... and of its value halves (null exactly when sc_k is)
  int sc_cap;
  const __half* t2_k;       // pinned FP16 key originals of the layer: [Bt * Hkv][max_tokens][128]
  const __half* t2_v;       // value originals, same layout
  int64_t max_tokens;
  int split0;               // promoted-block pass: index of its first partial set
  int stream_nt;            // 1 = Tier-1 loads carry the non-temporal hint (see stream_hint)
  float* eta_out;           // eta_b per (batch, kv-head, block) written alongside the log-masses, or null
  float* score_dev;         // promoted-block pass: canary output per (batch, q-head), or null
  // one-token append carried by the decode launch (null ap_k_new = none): the new (k, v) of every
  // (batch, kv-head) goes to slot `ap_slot` of the trailing FP16 block and, unless ap_t2_k is
  // null, to position ap_pos of the pinned originals
  const __half* ap_v_new;
  __half* ap_trail_k;       // layer base: [Bt * Hkv][16][128]
  __half* ap_trail_v;
  __half* ap_t2_k;          // layer base: [Bt * Hkv][max_tokens][128]
  __half* ap_t2_v;
  int ap_slot;
  int64_t ap_pos, ap_max_tokens;
};


// What the selector leaves behind, and which promoted sets follow from it.
struct PromMasks {
  const uint32_t* umask;    // [Bt][Hq][mask_words] key selections per head
  const uint32_t* vmask;    // value selections, or null
  int64_t mask_words;
  int nb;
  int per_head;             // 1: a head's promoted sets are its own selections; 0: the group's unions
  uint32_t explore_threshold;   // a block is explored (key-promoted) when its draw is below this; 0 = off
  uint32_t explore_seed;
};

// The promoted-block pass's part of the adaptive step besides DecodeArgs.  Orders of its workgroups: per KV group those of the
// positive sets, of the negated sets and of the sums; all passes and then all sums; the positive sets and the sums per
// KV group, then the negated sets, the last `ahead` of them moved to the front.
constexpr int PROM_BY_GROUP = 0, PROM_SUMS_LAST = 1, PROM_WRAPPED = 2;
struct PromArgs {
  PromMasks masks;          // umask null: the list and the flag words are there already (compact_kernel, which looks after
                            // the FP16 scratch)
  int32_t* slot;            // written from the masks: the flag words of the listed blocks, ...
  int32_t* ulist;           // ... the list, ascending, ...
  int32_t* ucount;          // ... its length
  const float* lm8;         // [Bt][Hq][nb]
  const float* eta;         // [Bt][Hkv][nb]
  const float* first;       // [Bt][Hq][4]
  ScanPart* scan;           // [Bt][Hq][parts], written
  int parts;                // workgroups that sum up the blocks left in INT8, per head, ...
  int sum_waves;            // ... or 1: one per KV group, a wave per head
  int groups;               // Bt * Hkv
  int order;                // of the workgroups, PROM_* below
  int ahead;                // PROM_WRAPPED: so many of the negated sets' workgroups come first
  int turn;                 // a KV group's list starts so many of its workgroups away from where the previous group's does
};

inline int64_t head_index(const Cache* c, int layer, int b, int kvh) {
  return ((int64_t)layer * c->desc.batch + b) * c->desc.n_kv_heads + kvh;
}

// Kernel arguments lie in memory, and the compiler loads one where it is first used: behind a branch or the wait for another,
// each 64-byte line of them is a miss of some 550 cycles of its own (in the split pass 2400 of a short step's 9400
// cycles went by before the first data was requested).  This asks for one word of each of a kernel's first 2 to 8 lines, at once, so
// that one miss is all: from here on arguments come from the scalar cache.
template <int BYTES>
__device__ __forceinline__ void fetch_args() {
  constexpr int N = (BYTES + 63) / 64 < 8 ? (BYTES + 63) / 64 : 8;
  const uint32_t* const w = (const uint32_t*)__builtin_amdgcn_kernarg_segment_ptr();
#define CQA_LINE(I) w[(I) < N ? 16 * (I) : 0]
  asm volatile("" ::"s"(CQA_LINE(0)), "s"(CQA_LINE(1)), "s"(CQA_LINE(2)), "s"(CQA_LINE(3)), "s"(CQA_LINE(4)), "s"(CQA_LINE(5)),
               "s"(CQA_LINE(6)), "s"(CQA_LINE(7)));
#undef CQA_LINE
}

// A kernel's argument at `offset`, read where this stands and not before: what only a rare branch needs would otherwise be loaded,
// and waited for, ahead of the branch.  It is read as a T, from constant memory: then the compiler takes its pointers for global ones.  As
// words they were not, and each access through them was a flat one, waited for together with everything before it (a step whose ladder
// serves all of 8 x 4 heads, 1000 tokens, 165.6, 160.1 us so; a few heads of 4 KV groups, 2000 tokens, 49.6, 48.2).
template <typename T>
__device__ __forceinline__ T arg_read_here(int offset) {
  uint64_t base = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(base));
  return *(const T*)(const __attribute__((address_space(4))) T*)(base + (uint64_t)offset);
}

// heads per KV group: 1, 2 or 4; its logarithm, without a division
__device__ __forceinline__ int group_shift(int n_q, int n_kv) { return n_q >= 4 * n_kv ? 2 : (n_q >= 2 * n_kv ? 1 : 0); }

// Reads of the caller's q, k and v, which need no more than the alignment of an FP16 number: the device reads a
// lane's 4 or 16 bytes at any address with the same instruction, the compiler only has to be told.
typedef uint32_t u32_any __attribute__((aligned(2)));
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));
__device__ __forceinline__ uint32_t ld4_any(const __half* p) { return *reinterpret_cast<const u32_any*>(p); }
__device__ __forceinline__ uint4 ld16_any(const __half* p) {
  const u32x4_any v = *reinterpret_cast<const u32x4_any*>(p);
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ __half2 ld_half2_any(const __half* p) {
  const uint32_t x = ld4_any(p);
  return __builtin_bit_cast(__half2, x);
}

extern thread_local int g_last_hip_error;
#define CQA_HIP(expr)                                   \
  do {                                                  \
    hipError_t e__ = (expr);                            \
    if (e__ != hipSuccess) {                            \
      cqa::g_last_hip_error = (int)e__;                 \
      return CQA_ERR_HIP;                               \
    }                                                   \
  } while (0)

struct ReduceArgs;
// ---- launchers implemented in the kernel translation units ---------------------
int32_t launch_seal(Cache* c, int layer, const __half* k_in, const __half* v_in, int64_t n_new,
                    int64_t len_before, bool tier2_by_kernel, hipStream_t st);
int32_t launch_certified(Cache* c, int layer, const __half* q, const cqa_tolerances& tol, float* O,
                         cqa_head_cert* cert, uint32_t* flags, uint32_t* flags_mirror,
                         uint32_t mirror_tag, float* blk_logmass, hipStream_t st,
                         const __half* k_new = nullptr,
                         const __half* v_new = nullptr, int pstride = 0, float* eta_out = nullptr,
                         float* partials = nullptr,   // null = the cache's own split workspace
                         uint32_t* raised = nullptr, uint32_t raised_tag = 0u,
                         ReduceArgs* defer = nullptr,    // the reduction's arguments, where it is not a launch of its own: it is left
                         RowsBy* by = nullptr);          // to the caller (by null) or to what *by says
int32_t static_scratch(int device, void** out);
int pick_splits(const Cache* c, int64_t n_blocks);
int stream_nt(const Cache* c, int64_t n_blocks);
void split_geometry(const Cache* c, int64_t n_blocks, int* nsplit, int* wpb);
int32_t launch_adaptive(Cache* c, int layer, const __half* q, const cqa_tolerances& tol,
                        const cqa_selector& sel, float* O, cqa_head_cert* cert, uint32_t* flags,
                        uint32_t* flags_mirror, uint32_t mirror_tag, hipStream_t st,
                        uint32_t* raised = nullptr, uint32_t raised_tag = 0u);
int32_t launch_split_mfma(const DecodeArgs& a, const ReduceArgs& ra, int group, dim3 grid, hipEvent_t ev0,
                          hipEvent_t ev1, hipStream_t st);

int32_t launch_stream_read(const uint8_t* t1, int64_t nq_cap, int nb, dim3 grid, bool nt, int wpb,
                           uint32_t* sink, hipStream_t st);

// Dense FP16 attention of `groups` consecutive KV groups: q [groups][group][128], k, v
// [groups][n_tokens][128] (device or mapped host memory).  O rows are written only where select
// (device, [groups][group]; null = all) is nonzero; cert / flags rows (null = none) are marked with
// `rung`.  layer_groups: KV groups the sequence split is chosen for (>= groups).  ws: at least
// dense_ws_floats(4, n_tokens) floats, or dense_ws_floats(group, n) for groups = 1, n >= n_tokens.
int32_t launch_dense(const __half* q, const __half* k, const __half* v, int group, int64_t groups,
                     int64_t layer_groups, int64_t n_tokens, float* O, const uint32_t* select, cqa_head_cert* cert,
                     uint32_t* flags, int rung, float* ws, hipStream_t st);
int64_t dense_ws_floats(int group, int64_t n_tokens);

// Device-resolved fallback ladder (dense_ladder_kernel).
constexpr int LADDER_MAX_SPLITS = 64;
// Steps that finish_ladder_kernel reduces as well: up to this many (batch, query head) rows and partial sets per row.
constexpr int FINISH_ROWS = 8, FINISH_SETS = 8;
struct LadderArgs {
  const uint32_t* raised;   // equals raised_tag when some head of this step requests a fallback (it may
  uint32_t raised_tag;      // do so without one: a recorded step that is replayed keeps its number)
  int groups;               // Bt * Hkv
  // the split pass was to reduce the rows: where the number that it left for a KV group is not raised_tag, its workgroups
  // were not on one die, and the rows are reduced here; null = the rows are there
  uint32_t* split_tickets;
  const __half* q;          // [Bt][Hq][128]
  const __half* t2_k;       // layer base of the pinned originals: [Bt * Hkv][max_tokens][128]
  const __half* t2_v;
  int64_t max_tokens, n_tokens;
  int n_rows;               // Bt * Hq
  int nsplit, tiles_per_split;
  int rung4_min_groups;
  float* ws;                // [Bt * Hq][nsplit][4 + 128]
  uint32_t* tickets;        // [Bt * Hkv], zero between launches
  uint32_t* counts;         // [2]: steps served by Rung 3, by Rung 4
  uint32_t* strayed;        // ... and the host learns of it here
  int many_items;           // more served (KV group, split) items than this are walked by many_walkers workgroups
  int many_walkers;
  float* O;
  cqa_head_cert* cert;
  uint32_t* flags;
};
int ladder_splits(const Cache* c, int64_t n_tokens);
int64_t ladder_ws_floats(int64_t rows);
int32_t launch_dense_ladder(Cache* c, int layer, const __half* q, int rung4_min_groups, float* O,
                            cqa_head_cert* cert, uint32_t* flags, uint32_t raised_tag, hipStream_t st,
                            RowsBy by = RowsBy::launch, const ReduceArgs* reduce = nullptr);   // reduce: null = the rows are there
// certified decode and ladder, enqueue-only (k_new, v_new: a token that rides on the split launch, or null);
// *launched (may be null) tells whether the split launch, which stores that token, was reached
int32_t launch_step(Cache* c, int layer, const __half* q, const cqa_tolerances& tol, float* O, cqa_head_cert* cert,
                    uint32_t* flags, hipStream_t st, const __half* k_new, const __half* v_new, bool* launched);
inline uint32_t* ladder_raised(Cache* c) { return c->ladder_counts + 2; }
inline uint32_t next_ladder_tag(Cache* c) {
  c->ladder_seq = c->ladder_seq == 0xFFFFFFFFu ? 1u : c->ladder_seq + 1u;
  return c->ladder_seq;
}

}  // namespace cqa
