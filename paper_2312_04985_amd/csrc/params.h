// Kernel argument blocks and launcher prototypes (internal to libsparq).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace sparq {

constexpr int kDecodeThreads = 512;     // threads per workgroup of the decode kernels (256 in the builds of four waves)
constexpr int kRadixBins = 2048;        // 11-bit digits: passes of 11, 11 and 10 bits
constexpr int kWorkspaceHeader = 256;   // bytes; word 0 is the error word
constexpr int kControlBytes = 65536;    // control block at the start of the workspace, zeroed by sparq_workspace_init
// Counters of workgroups that have finished (last_to_arrive), inside the control block behind the header: left at 0 by
// every launch (the digit-bucket plans clear theirs as well).  The rest of the control block is scratch of the bulk append.
constexpr int kTicketOffset = kWorkspaceHeader;
constexpr int kTickets = (16384 - kWorkspaceHeader) / 4;
constexpr int kAppendScratchOffset = 16384;
constexpr int kMaxSplit = 16;           // most workgroups one (sequence, head) is split over
constexpr int kSplitMaxUnits = 128;     // the digit-bucket plan (few units, long caches) serves at most this many (sequence, head) units
constexpr int kProbeBlocks = 256 * 8;   // workgroups (of 256 threads) of the bandwidth probes

// n / d for 0 <= n < 2^31, 1 <= d < 2^31, by multiplication: with l = ceil(log2 d) and mul = ceil(2^(31 + l) / d), the error
// mul d - 2^(31 + l) is below d <= 2^l, so that floor(n mul / 2^(31 + l)) is exact.  (There is no integer division in
// hardware; the compiler's sequence for it is a chain of some thirty vector instructions in front of a kernel's first loads.)
struct Divider {
  uint32_t mul = 0x80000000u, shift = 31;
};
inline Divider make_divider(int64_t d) {
  int l = 0;
  while (((int64_t)1 << l) < d) ++l;
  return Divider{(uint32_t)((((uint64_t)1 << (31 + l)) + (uint64_t)d - 1) / (uint64_t)d), (uint32_t)(31 + l)};
}
__host__ __device__ inline int divided(int n, Divider v) { return (int)(((uint64_t)(uint32_t)n * v.mul) >> v.shift); }

struct DecodeArgs {
  void* K; void* Kt; void* V;                  // written only by the fused-append variant
  const float* v_mean; const int32_t* seq_lens;
  const void* q; const int32_t* k_per_seq;
  const void* k_new; const void* v_new;          // non-null: fused append (one-launch decode step)
  float* v_mean_next; int32_t* seq_lens_next;
  void* out; float* alpha_out; int32_t* idx_out; int32_t* chan_out; int32_t* err;
  int32_t B, H, H_kv, S_max, d_h, r, k, idx_stride;   // S_max: the bound on the lengths that LDS and workspace are sized for
  int32_t S_stride;   // positions per head in K and V and per channel row in Kt (the buffers' own S_max, >= S_max)
  uint32_t flags;
  int32_t local_window;
  int32_t group = 1;                      // query heads per KV head
  int32_t helpers = 0, per_xcd = 0;       // few units: workgroups that fetch for each unit's own, units per XCD
  Divider by_xcd;                         // by per_xcd
  Divider by_H, by_H_kv, by_group;        // set by enqueue_decode, as `group`
  unsigned long long* clocks = nullptr;   // [workgroups][kStageStamps] time stamps; set only by a SPARQ_STAGE_CLOCKS build
};

// Time stamps per workgroup of the one-workgroup-per-head kernel in a SPARQ_STAGE_CLOCKS build (10 ns ticks of the
// constant 100 MHz counter): start, channels selected, own part of Step 1 done, all keys in LDS, threshold
// found, list compacted, own rows attended, all partials in LDS, end.
constexpr int kStageStamps = 9;

struct AppendArgs {
  void* K; void* Kt; void* V; float* v_mean; int32_t* seq_lens;
  float* v_mean_out; int32_t* seq_lens_out;   // where the new means / lengths go (== v_mean / seq_lens: in place)
  const void* k_new; const void* v_new; const int32_t* n_new_per_seq; int32_t* err;
  int32_t B, H_kv, S_max, d_h, n_new;   // S_max: no length may pass it
  int32_t S_stride;   // positions per head in K and V and per channel row in Kt
  int32_t tiled;   // the tiled single-copy key layout: K holds tiles of 8 positions, Kt the rows of the newest < 8
  void* scratch = nullptr; size_t scratch_bytes = 0;   // room for the partial sums of a bulk append (16-byte aligned)
  int32_t* tickets = nullptr;   // [B], then [B * H_kv]: counters of a bulk append in one launch, 0 between launches
  // set by the launcher of a bulk append: workgroups per KV head and tiles of each, their partial sums of the value
  // columns [B * H_kv][n_split][d_h], old length and row count of each KV head
  int32_t n_split = 1, tiles_per_split = 1;
  double* part_ws = nullptr; int2* span_ws = nullptr;
};

struct DenseArgs {
  const void* K; const void* V; const int32_t* seq_lens; const void* q; void* out;
  float* partials;   // [unit][n_split][heads of the bundle][d_h] numerators, then [unit][n_split][heads of the bundle][2]
                     // (max, denominator); a unit is a (sequence, KV head, bundle of query heads)
  int32_t* tickets;  // one counter per (sequence, KV head, bundle), 0 between launches; used where n_split > 1
  int32_t* err;
  int32_t B, H, H_kv, S_max, d_h, n_split, rows_per_split;
  int32_t S_stride;   // positions per head in K and V
};

// two-level plan: spans of span_len positions (a multiple of 64, at most kLongSpan), at most kMaxSpans per sequence
constexpr int kLongSpan = 8192;
constexpr int kMaxSpans = 64;

struct LongArgs {
  DecodeArgs d;
  Divider by_span;         // by n_span
  int32_t n_span;          // workgroups per (sequence, head) in the scoring launch
  int32_t span_len;        // positions per span
  int32_t cand_cap;        // candidates one span may hand on = min(k, span_len)
  float* tmax_ws;          // [B * H][n_span] largest logit numerator of each span
  float* zsum_ws;          // [B * H][n_span] sum over the span of exp((d - span max) / tau)
  int32_t* cnt_ws;         // [B * H][n_span] candidates of each span
  float* tau_ws;           // [B * H]
  uint32_t* cand_key_ws;   // [B * H][n_span][cand_cap] keys of the candidates, position-ascending
  int32_t* cand_pos_ws;    // [B * H][n_span][cand_cap] their positions
};

// grouped-query rule over several workgroups per (sequence, KV head)
struct GsArgs {
  DecodeArgs d;
  Divider by_n1, by_n2, by_split;   // by n1, n2 and n_split
  int32_t n1, span1;       // logit spans per KV unit and their length (positions)
  int32_t n2, span2;       // selection spans per KV unit and their length
  int32_t cand_cap;        // candidates one selection span may hand on = min(k, span2)
  int32_t n_split;         // gather workgroups per KV unit
  int32_t list_stride;     // entries of one KV unit's position list
  float* z_ws;             // [B * H][S_max] logit numerators
  float* stat_ws;          // [B * H_kv][n1][G][2] span maximum and sum-exp per head
  float* esc_ws;           // [B * H] log2(e) / tau
  float* alpha_ws;         // [B * H]
  int32_t* cnt_ws;         // [B * H_kv][n2]
  uint32_t* cand_key_ws;   // [B * H_kv][n2][cand_cap]
  int32_t* cand_pos_ws;    // [B * H_kv][n2][cand_cap]
  int32_t* list_ws;        // [B * H_kv][list_stride] selected positions, ascending
  float* part_ws;          // [B * H][n_split][d_h + 2] attention partials
};

// the last launch of the grouped-query plan over several workgroups
struct SplitArgs {
  DecodeArgs d;
  int32_t n_split;       // gather workgroups per (sequence, head)
  float* alpha_ws;       // [B * H]
  float* part_ws;        // [B * H][n_split][d_h + 2] attention partials
};

// digit-bucket plan (few units, long caches): spans of span_len positions, n_span of them per unit
struct BucketArgs {
  DecodeArgs d;
  Divider by_span, by_len;   // by n_span and span_len
  int32_t n_span, span_len;
  int32_t cand_cap;        // candidates (keys sharing the threshold digit) that bk_select_gather ranks out of LDS
  float* tmax_ws;          // [B * H][n_span] largest logit numerator of each span
  float* zsum_ws;          // [B * H][n_span] sum over the span of exp((d - span max) / tau)
  float* anum_ws;          // [B * H][n_span] the span's share of alpha's numerator (relative to the sequence maximum)
  float* tau_ws;           // [B * H]
  float* zden_ws;          // [B * H] softmax denominator of the approximate scores, for bk_combine
  int32_t rows = 0;        // the key cache is stored once, as rows
  int32_t merge;           // the unit's last workgroup of the gather merges (else bk_combine, in a launch of its own)
  int32_t* tickets;        // [B * H] counters of finished spans, cleared by the plan's own first launches
  uint16_t* coarse_ws;     // [B * H][n_span][64] A[32 l]
  uint16_t* fine_ws;       // [B * H][n_span][2080] A[d] = keys of the span with first digit >= d
  uint32_t* skey_ws;       // [B * H][n_span][span_len] the span's keys sorted by first digit, descending
  uint32_t* spos_ws;       // [B * H][n_span][span_len] their positions
  float* part_ws;          // [B * H][n_span][d_h + 2] attention partials of the spans
  // the grouped-query rule on this plan (group > 0): one selection per KV head from the group score; the tables
  // and sorted arrays are indexed by KV unit, the logits and per-head statistics come from gs_logits
  int32_t group = 0;       // query heads per KV head, 0 = every head selects for itself
  int32_t n1 = 0;          // logit spans per KV unit of gs_logits
  const float* z_ws = nullptr;      // [B * H][S_max] logit numerators
  const float* stat_ws = nullptr;   // [B * H_kv][n1][group][2] span maximum and sum-exp per head
  const float* esc_ws = nullptr;    // [B * H] log2(e) / tau
};

// Where bk_select_gather's arrays lie in its LDS, in 4-byte words.  The bitmap has a word per 32 positions, and a span is a
// multiple of 64: it is rounded up to whole 16-byte pieces, since the histogram behind it is read in such pieces.
struct BkSelectLds {
  int keyval;   // [span_len] keys of this span's selected positions, by position
  int list;     // [span_len] this span's selected positions, ascending
  int bitmap;   // [span_len / 32] selected positions of this span
  int ckey;     // [cand_cap] candidates: keys with the threshold digit (more than cand_cap are read again by every pass)
  int cpos;     // [cand_cap] their positions
  int hist;     // [kRadixBins]
  int tab;      // [n_span][33] A_s[32 lc + t] (at least kDecodeThreads words)
  int above;    // [n_span] entries of span s above the threshold digit
  int with;     // [n_span] entries of span s with the threshold digit
  int before;   // [n_span + 1] candidates before span s
  int taken;    // [n_span] selected candidates of span s
  int offs;     // [n_span + 1] list entries before span s
  int part;     // [waves][d_h + 2] attention partials of the waves
  int red;      // [32]
  int wcnt;     // [16]
  int ctl;      // [16]
  int words;
};
__host__ __device__ constexpr BkSelectLds bk_select_lds(int d_h, int span_len, int n_span, int cand_cap) {
  BkSelectLds l{};
  int w = 0;
  l.keyval = w; w += span_len;
  l.list = w; w += span_len;
  l.bitmap = w; w += (span_len / 32 + 3) & ~3;
  l.ckey = w; w += cand_cap;
  l.cpos = w; w += cand_cap;
  l.hist = w; w += kRadixBins;
  l.tab = w; w += n_span * 33 > kDecodeThreads ? n_span * 33 : kDecodeThreads;
  l.above = w; w += kMaxSpans + 8;
  l.with = w; w += kMaxSpans + 8;
  l.before = w; w += kMaxSpans + 8;
  l.taken = w; w += kMaxSpans + 8;
  l.offs = w; w += kMaxSpans + 8;
  l.part = w; w += kDecodeThreads / 64 * (d_h + 2);
  l.red = w; w += 32;
  l.wcnt = w; w += 16;
  l.ctl = w; w += 16;
  l.words = w;
  return l;
}

// LDS bytes the fused decode kernel needs for a cache of S_max rows and head dimension d_h
size_t decode_lds_bytes(int S_max, int d_h);
size_t decode_shared_lds_bytes(int S_max, int d_h, int g);   // LDS that admits S_max; 0: no grouped-query kernel for this shape

hipError_t launch_decode(const DecodeArgs& a, int dtype, hipStream_t s);
bool decode_helped(const DecodeArgs& a);                // few units: launch_decode goes on with launch_decode_helped
hipError_t launch_decode_helped(const DecodeArgs& a, int dtype, hipStream_t s);
bool decode_runs(const DecodeArgs& a);                  // row strides near 32 KiB: ... with launch_decode_runs
hipError_t launch_decode_runs(const DecodeArgs& a, int dtype, hipStream_t s);
bool decode_apart(const DecodeArgs& a);                 // a step of many units: ... with launch_step_apart
hipError_t launch_step_apart(const DecodeArgs& a, int dtype, hipStream_t s);
bool decode_short(const DecodeArgs& a);                 // many units with short caches: ... with launch_decode_short
hipError_t launch_decode_short(const DecodeArgs& a, int dtype, hipStream_t s);
size_t decode_single_k_lds_bytes(int S_max, int d_h);   // LDS that admits S_max
hipError_t launch_decode_single_k(const DecodeArgs& a, int dtype, hipStream_t s);
bool decode_single_k_short(const DecodeArgs& a);        // many units with short caches: ... with launch_decode_single_k_short
hipError_t launch_decode_single_k_short(const DecodeArgs& a, int dtype, hipStream_t s);
size_t long_scores_lds_bytes(int span_len, int d_h);
size_t long_merge_lds_bytes(int n_span, int cand_cap);
hipError_t launch_decode_long(const LongArgs& a, int dtype, hipStream_t s);
size_t bk_scores_lds_bytes(int span_len, int d_h);
size_t bk_select_lds_bytes(int span_len, int d_h, int n_span, int cand_cap);
int bk_fine_len();
hipError_t launch_decode_bucket(const BucketArgs& a, int dtype, hipStream_t s);
size_t bk_group_scores_lds_bytes(int span_len);
// the grouped-query rule on the digit-bucket plan: after gs_logits (launch_group_logits), uses a.group, n1, z_ws, stat_ws, esc_ws
hipError_t launch_decode_bucket_group(const BucketArgs& a, int dtype, hipStream_t s);
// the first launch of the grouped-query plans alone: logit numerators and per-head span statistics (uses d, n1, span1,
// z_ws, stat_ws, esc_ws of `a`)
hipError_t launch_group_logits(const GsArgs& a, int dtype, hipStream_t s);
hipError_t launch_split_combine(const SplitArgs& a, int dtype, hipStream_t s);
size_t gs_select_lds_bytes(int span2);
size_t gs_merge_lds_bytes(int n2, int cand_cap);
hipError_t launch_decode_shared_split(const GsArgs& a, int dtype, hipStream_t s);
// z_ws: [B * H][S_max] fp32 scratch for the logit numerators
hipError_t launch_decode_shared(const DecodeArgs& a, float* z_ws, int dtype, hipStream_t s);
// what a bulk append on a cache of S_max positions can use of AppendArgs::scratch (with less it runs on fewer workgroups)
size_t append_scratch_bytes(int64_t heads, int S_max, int d_h);
hipError_t launch_append(const AppendArgs& a, int dtype, hipStream_t s);
constexpr int kDenseSplits = 128;   // most workgroups one unit of dense_decode is split over (two per lane in the merge)
// Query heads that share a pass over their KV head's rows, for g query heads per KV head: the kernel's width (up to 8; 4 at
// d_h 256, by registers), and the bundles of at most that many.  A group that is no multiple of 4 is not cut into bundles of
// 2 or 1, which would each read all rows again: the width's last heads repeat the bundle's last one (64 KV heads of 5000
// rows, d_h 128: 3 heads 65 us as three bundles, 32 as one of width 4; 6 heads 66 and 34).
constexpr int dense_width(int g, int d_h) {
  return g <= 2 ? g : (g % 8 == 0 && d_h <= 128 ? 8 : (g % 4 == 0 || g == 3 || d_h > 128 ? 4 : 8));
}
constexpr int dense_bundles(int g, int d_h) { return (g + dense_width(g, d_h) - 1) / dense_width(g, d_h); }
hipError_t launch_dense(const DenseArgs& a, int dtype, hipStream_t s);
hipError_t launch_copy_probe(void* dst, const void* src, size_t n_bytes, hipStream_t s);
hipError_t launch_read_probe(const void* src, size_t n_bytes, void* sink, hipStream_t s);
hipError_t launch_clear(void* workspace, int n_bytes, hipStream_t s);

// A kernel that takes more than 64 KiB of dynamic LDS has to be allowed to, once per kernel and device
// (not per launch: the call costs host time).  `lds` = the bytes the coming launch asks for; `limit` = what the
// kernel is allowed from then on (a kernel with static LDS arrays as well must stay below 160 KiB minus those).
template <auto Kern>
hipError_t allow_lds(size_t lds, int limit = 160 * 1024) {
  if (lds <= 64 * 1024) return hipSuccess;
  static unsigned long long allowed = 0;   // bit d: done on device d (benign race: the call is idempotent)
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64 || !((allowed >> dev) & 1ull)) {
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(Kern), hipFuncAttributeMaxDynamicSharedMemorySize, limit);
    if (e != hipSuccess) return e;
    if (dev >= 0 && dev < 64) allowed |= 1ull << dev;
  }
  return hipSuccess;
}

}  // namespace sparq
