// C ABI of libsparq (see include/sparq.h): argument validation, launch planning, enqueue.
// No allocation, no synchronisation (sparq_async_error excepted), no host-side arithmetic of
// the method.
#include "../../include/sparq.h"

#include <hip/hip_runtime.h>

#include "params.h"

namespace {

using namespace sparq;

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int check_shape(const sparq_shape* s) {
  if (!s) return SPARQ_EINVAL;
  if (s->B < 1 || s->H < 1 || s->H_kv < 1 || s->S_max < 1 || s->d_h < 1) return SPARQ_EINVAL;
  if (s->H % s->H_kv != 0) return SPARQ_EINVAL;
  if (s->r < 1 || s->r > s->d_h || s->k < 1) return SPARQ_EINVAL;
  if (s->dtype != SPARQ_F16 && s->dtype != SPARQ_BF16) return SPARQ_EINVAL;
  if (s->S_max % 64 != 0) return SPARQ_EINVAL;
  if (s->flags & ~(uint32_t)(SPARQ_FLAG_NO_REALLOC | SPARQ_FLAG_GQA_SHARED | SPARQ_FLAG_RAGGED_BATCH |
                             SPARQ_FLAG_TAU_SQRT_DH | SPARQ_FLAG_TAU_SQRT_R | SPARQ_FLAG_SINGLE_K | SPARQ_FLAG_TILED_K)) return SPARQ_EINVAL;
  if ((s->flags & SPARQ_FLAG_SINGLE_K) && (s->flags & SPARQ_FLAG_TILED_K)) return SPARQ_EINVAL;
  if ((s->flags & SPARQ_FLAG_TAU_SQRT_DH) && (s->flags & SPARQ_FLAG_TAU_SQRT_R)) return SPARQ_EINVAL;
  if (s->local_window < 0) return SPARQ_EINVAL;
  if (s->S_bound < 0 || s->S_bound > s->S_max || s->S_bound % 64 != 0) return SPARQ_EINVAL;
  if (s->d_h != 64 && s->d_h != 128 && s->d_h != 256) return SPARQ_EUNSUPPORTED;
  // element offsets inside one tensor are formed in size_t; the counts themselves stay in int32
  if ((int64_t)s->B * s->H > (int64_t)1 << 30) return SPARQ_EUNSUPPORTED;
  return SPARQ_OK;
}

int check_cache(const sparq_cache* c, const sparq_shape* s) {
  if (!c || !c->K || !c->V || !c->v_mean || !c->seq_lens) return SPARQ_EINVAL;
  if (!aligned16(c->K) || !aligned16(c->V) || !aligned16(c->v_mean)) return SPARQ_EINVAL;
  if (!(s->flags & SPARQ_FLAG_SINGLE_K) && (!c->Kt || !aligned16(c->Kt))) return SPARQ_EINVAL;
  return SPARQ_OK;
}

// runs of at least 256 rows, about `target` workgroups over `units`, at most `most` runs (0: any number)
void dense_split(const sparq_shape* s, int64_t units, int64_t target, int64_t most, int* n_split, int* rows_per_split) {
  int64_t want = (target + units - 1) / units;
  const int64_t cap = s->S_max / 256 > 0 ? s->S_max / 256 : 1;
  if (want > cap) want = cap;
  if (most && want > most) want = most;
  if (want < 1) want = 1;
  int rows = (int)((s->S_max + want - 1) / want);
  rows = (rows + 63) / 64 * 64;
  *rows_per_split = rows;
  *n_split = (s->S_max + rows - 1) / rows;
}

// Split-sequence plan of dense_decode.  Two workgroups fit on a CU.  Lengths that differ are evened out by 2048 of them, where
// the caller says that they do (128 and 264 units of up to 8192 rows with lengths over 16x at 256 / 512 / 1024 / 2048 workgroups:
// 252 / 256 / 199 / 190 and 143 / 140 / 110 / 100 us).  Otherwise 1024 are two rounds of the chip, but a workgroup has a start
// and a merge to pay, so runs keep to 64 Ki elements of K at least, if need be with 512 or 256 workgroups (256 / 512 / 1024,
// one query head: 64 units of 5000 rows of 64 16.9 / 16.9 / 19.8, 128 of 2500 16.5 / 16.8 / 19.0, 64 of 2500 of 128 16.9 /
// 17.0 / 19.2, 128 of 2500 28.5 / 29.0 / 30.3; long runs the other way: 512 of 4096 of 128 155 / 155 / 159, lengths that
// differ without the flag, 128 of up to 16 000, 142 / 133 / 121).  Few units would be merged from very many partial results:
// 8 units of 32 768 rows 28.5 us from 31 each, 31.6 from 57; fewer units need that many to fill the chip (one unit of
// 40 000 rows, 8 heads: 43 us from 64 each, 36 from 126).
void dense_plan(const sparq_shape* s, int* n_split, int* rows_per_split) {
  const int64_t units = (int64_t)s->B * s->H_kv * dense_bundles(s->H / s->H_kv, s->d_h);
  const int64_t most = units >= 8 ? 32 : (units >= 3 ? 64 : kDenseSplits);
  const bool ragged = (s->flags & SPARQ_FLAG_RAGGED_BATCH) != 0;
  for (int target = ragged ? 2048 : 1024; target >= 256; target >>= 1) {
    dense_split(s, units, target, most, n_split, rows_per_split);
    if ((int64_t)*rows_per_split * s->d_h >= (ragged ? 32768 : 65536)) break;
  }
}

// Partial results that the workspace has room for, per (sequence, KV head): what 2048 workgroups would leave.
int dense_room(const sparq_shape* s) {
  int n_split, rows;
  dense_split(s, (int64_t)s->B * s->H_kv, 2048, 0, &n_split, &rows);
  return n_split;
}

// The shape that plans, LDS and workspace are sized for: the caller's bound on the lengths (S_bound), where one is
// given, stands in for S_max; the buffers keep the strides of the shape's own S_max.
sparq_shape bounded(const sparq_shape* s) {
  sparq_shape e = *s;
  if (s->S_bound > 0) e.S_max = s->S_bound;
  e.S_bound = 0;
  return e;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// LDS a workgroup may use: the device's, or gfx950's 160 KiB where no device can be asked (sizing
// queries on a machine without a GPU)
int max_lds_bytes() {
  static int cached = -1;   // same for every device of one machine; benign race
  if (cached < 0) {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 160 * 1024;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) return 160 * 1024;
    cached = v;
  }
  return cached;
}

// the paper's grouped-query rule is a kernel of its own; with one query head per KV head it is
// the ordinary rule
bool wants_shared(const sparq_shape* shape) {
  return (shape->flags & SPARQ_FLAG_GQA_SHARED) && shape->H != shape->H_kv;
}

bool single_k(const sparq_shape* shape) { return (shape->flags & SPARQ_FLAG_SINGLE_K) != 0; }
bool tiled_k(const sparq_shape* shape) { return (shape->flags & SPARQ_FLAG_TILED_K) != 0; }

// Which kernels serve a shape.  Every plan keeps one 4-byte key per position (or per candidate) of its
// unit of work in LDS; that decides what fits.
enum Plan { kPlanNone, kPlanFused, kPlanLong, kPlanShared, kPlanSharedSplit, kPlanSingleK, kPlanSingleBucket, kPlanBucket, kPlanSharedBucket };
struct PlanInfo { Plan plan; int n_split, n_span, span_len, cand_cap, n1, span1; };

// The two-level plan: spans of `span` positions select their own top-k, one workgroup per unit merges at
// most n_span * min(k, span) candidates.  It serves what no single workgroup can hold (S_max beyond the LDS)
// for batches with more units than the digit-bucket plan takes.
bool two_level_plan(const sparq_shape* s, int span, size_t lds_max, PlanInfo* p) {
  const int64_t n_span = ((int64_t)s->S_max + span - 1) / span;
  if (n_span > kMaxSpans) return false;
  const int cap = s->k < span ? s->k : span;
  if (long_scores_lds_bytes(span, s->d_h) > lds_max || long_merge_lds_bytes((int)n_span, cap) > lds_max) return false;
  p->n_span = (int)n_span; p->span_len = span; p->cand_cap = cap;
  return true;
}

// The digit-bucket plan for few units with long caches: about 512 workgroups in all, spans of 1024 to 8192
// positions (a multiple of 64), at most kMaxSpans of them.
bool bucket_plan(const sparq_shape* s, size_t lds_max, PlanInfo* p) {
  const int64_t units = (int64_t)s->B * s->H;
  int64_t n_span = 512 / units;
  if (n_span < 2) n_span = 2;
  // (units x n_span <= 512: both kernels hold two workgroups per CU, and a second round of workgroups costs
  // more than longer spans do)
  if (n_span > kMaxSpans) n_span = kMaxSpans;
  int64_t span = (s->S_max + n_span - 1) / n_span;
  if (span < 1024) span = 1024;
  span = (span + 63) / 64 * 64;
  if (span > kLongSpan) span = kLongSpan;
  n_span = (s->S_max + span - 1) / span;
  if (n_span > kMaxSpans) return false;
  // the keys that share the threshold digit are a few percent of the sequence unless many keys are identical
  const int cap = s->S_max <= 40000 ? 2048 : (s->S_max <= 100000 ? 4096 : 8192);
  if (bk_scores_lds_bytes((int)span, s->d_h) > lds_max ||
      bk_select_lds_bytes((int)span, s->d_h, (int)n_span, cap) > lds_max) return false;
  p->n_span = (int)n_span; p->span_len = (int)span; p->cand_cap = cap;
  return true;
}

// The grouped-query rule over several workgroups per KV unit: n1 spans for the logits (at most 256 workgroups,
// at least 1024 positions each), spans of 4096 / 8192 positions for the two-level selection.
bool shared_split_plan(const sparq_shape* s, size_t lds_max, PlanInfo* p) {
  const int64_t ukv = (int64_t)s->B * s->H_kv;
  // (gs_logits with 4 heads' accumulators runs one workgroup per CU: more than 256 workgroups would come in two
  // rounds, which was measured as 58 instead of 47 us per decode just above S = 32768 with 8 KV units)
  int64_t n1 = 256 / ukv;
  if (n1 > kMaxSpans) n1 = kMaxSpans;
  if (n1 < 1) n1 = 1;
  int64_t span1 = (s->S_max + n1 - 1) / n1;
  if (span1 < 1024) span1 = 1024;
  span1 = (span1 + 63) / 64 * 64;
  n1 = (s->S_max + span1 - 1) / span1;
  const int span2 = s->S_max >= 32768 ? kLongSpan : kLongSpan / 2;
  const int64_t n2 = ((int64_t)s->S_max + span2 - 1) / span2;
  if (n1 > kMaxSpans || n2 > kMaxSpans) return false;
  const int cap = s->k < span2 ? s->k : span2;
  if (gs_select_lds_bytes(span2) > lds_max || gs_merge_lds_bytes((int)n2, cap) > lds_max) return false;
  int64_t n = 512 / ukv;
  if (n > kMaxSplit) n = kMaxSplit;
  if (n > s->k / 64) n = s->k / 64;
  if (n < 1) n = 1;
  p->n1 = (int)n1; p->span1 = (int)span1; p->n_span = (int)n2; p->span_len = span2; p->cand_cap = cap; p->n_split = (int)n;
  return true;
}

// The grouped-query rule on the digit-bucket plan: gs_logits over n1 spans per KV unit (at most 256 workgroups, at
// least 1024 positions each), then the bucket plan's spans for the selection.
bool shared_bucket_plan(const sparq_shape* s, size_t lds_max, PlanInfo* p) {
  const int64_t ukv = (int64_t)s->B * s->H_kv;
  int64_t n1 = 256 / ukv;                   // one round of gs_logits workgroups, as above
  if (n1 > kMaxSpans) n1 = kMaxSpans;
  if (n1 < 1) n1 = 1;
  int64_t span1 = (s->S_max + n1 - 1) / n1;
  if (span1 < 1024) span1 = 1024;
  span1 = (span1 + 63) / 64 * 64;
  n1 = (s->S_max + span1 - 1) / span1;
  if (n1 > kMaxSpans) return false;
  if (!bucket_plan(s, lds_max, p)) return false;
  if (bk_group_scores_lds_bytes(p->span_len) > lds_max) return false;
  p->n1 = (int)n1; p->span1 = (int)span1;
  return true;
}

// Few units whose idle CUs fetch for them (decode_helped): what one workgroup per unit takes grows with the positions, the channel rows
// and the selected rows (0.2 us per 1000 positions, 0.025 for each of their channels, 4.3-13 for 1000 selected rows of 64-256 channels);
// the digit-bucket plan takes 22 to 31 us wherever between 12 288 and 35 000 positions, least with 32 units, most with 64.  us per decode,
// helped / bucket, caches in HBM, 32 units of 128 channels, positions, r, k: 12 300 32, 256 22.4 / 24.6; 32, 1024 28.0 / 26.1; 64, 512 33.9 / 29.3; 16 300 8, 256
// 16.5 / 22.6; 16, 700 22.6 / 25.1; 20 000 16, 500 22.8 / 24.6; 24 000 8, 256 19.7 / 23.1; 16, 300 23.3 / 24.8; 8, 900 24.7 / 24.2; 28 000 8, 256 20.4 / 23.8; 16, 150
// 23.4 / 25.3; 8, 900 25.2 / 24.8; 32 000 8, 256 23.4 / 23.9; 12, 300 27.3 / 25.3; 8, 900 28.5 / 25.1 (a lane's 64 keys lie a whole round of LDS banks apart); of 64
// channels 12 350 32, 512 22.8 / 24.7; 24 000 16, 800 26.5 / 25.6; 28 000 8, 1500 26.1 / 25.2; of 256 12 350 32, 128 21.0 / 24.1; 28 000 8, 400 24.2 / 24.7; 32 000 8, 300
// 26.3 / 24.5.  48 and 64 units: 24 000 16, 300 23.3 / 26.8 and 24.2 / 29.4; 32 000 8, 900 28.9 / 27.2 and 28.9 / 28.8; 12, 300 27.5 / 28.2 and 27.8 / 30.6; 34 000 8, 800
// 27.6 / 27.3 and 27.8 / 29.8; 12, 128 26.2 / 28.3 and 26.1 / 30.3; of 64 channels 32 000 8, 1500 30.0 / 27.1 and 29.8 / 28.5.  Next to the lines, 17 / 32 / 64
// units: 12 280 32, 480 21.2 / 22.1, 22.7 / 25.0, 24.8 / 28.7; 28 600 14, 30 21.1 / 25.7, 21.2 / 24.5, 22.0 / 29.2; 33, 48 and 64 units 28 000 8, 900 25.2 / 26.2,
// 25.1 / 26.4, 26.0 / 28.9.  (17 to 30 units stand between: 24 000 8, 900 24.1 / 25.5 with 24; the line is that of 32.)  16 units 12 300 32, 256 21.5 / 21.3.
bool helped_faster(const sparq_shape* s) {
  const int64_t units = (int64_t)s->B * s->H, S = s->S_max, k = s->k < s->S_max ? s->k : s->S_max;
  if (units <= 16 || units > 64) return false;
  const int64_t rows = k * (s->d_h + 64);
  const bool few_reads = S * s->r * 2 + k * s->d_h * 4 <= 1000000;
  if (S > 28672) return units > 32 && few_reads && rows <= 153600;
  return S * (2 * s->r + 16) + k * (3 * s->d_h + 200) <= 1280000 || (few_reads && rows <= (units > 32 ? 172800 : 96000));
}

// A key cache stored once, few units: Step 1 reads whole rows, which one workgroup gets at 60 GB/s.  us per decode, one workgroup per
// unit / digit buckets, 128 channels, k 256 unless said: 1 unit at 2000 positions 16.8 / 22.3, 4096 28.8 / 22.9; 20 on 5 KV heads at 15 202,
// k 1901, 102.7 / 39.4; 32 at 3000 26.0 / 25.9, 4096 30.8 / 26.0, 16 384 with k 1024 96.7 / 45.5; of 64 channels at 4096 20.7 / 22.4; of 256 at
// 2000 33.1 / 34.6, 4096 52.8 / 33.9; 64 units at 4918 37.8 / 35.9, 12 000 72.3 / 52.7; 96 at 4096 34.1 / 37.5, 12 000 76.1 / 72.1; 128 at
// 4096 36.5 / 43.7, 20 000 130.6 / 130.6.
bool single_bucket_faster(const sparq_shape* s) {
  return (int64_t)s->B * s->H <= 64 && s->S_max >= 2048 + 2048 * 128 / s->d_h;
}

// by_size: as if helped_faster were not; workspaces are sized by that, so that a call with another r or k is not refused.
PlanInfo choose_plan(const sparq_shape* s, bool by_size = false) {
  PlanInfo p{kPlanNone, 0, 0, 0, 0, 0, 0};
  const size_t lds_max = (size_t)max_lds_bytes();
  if (single_k(s)) {
    const size_t need = wants_shared(s) ? 0 : decode_single_k_lds_bytes(s->S_max, s->d_h);
    if (need != 0 && need <= lds_max) p.plan = single_bucket_faster(s) && bucket_plan(s, lds_max, &p) ? kPlanSingleBucket : kPlanSingleK;
    return p;
  }
  if (tiled_k(s)) {            // one kernel reads the tiled layout: one workgroup per head
    if (!wants_shared(s) && decode_lds_bytes(s->S_max, s->d_h) <= lds_max) p.plan = kPlanFused;
    return p;
  }
  if (wants_shared(s)) {
    const size_t need = decode_shared_lds_bytes(s->S_max, s->d_h, s->H / s->H_kv);
    if (need == 0) return p;                                    // no kernel for this group size
    const bool one_wg = need <= lds_max;
    // measured: the one-workgroup kernel is faster from about 64 KV units on (116 vs 123 us at 128 units,
    // S = 8192) and far slower below (230 vs 70 us at 8 units, S = 32768)
    const int64_t ukv = (int64_t)s->B * s->H_kv;
    const bool few = (ukv <= 32 && s->S_max >= 8192) || (ukv <= 64 && s->S_max >= 16384);
    // few heads with long caches: the digit-bucket selection, one for the group (measured against the two-level
    // selection per KV head: 59 vs 87 us at 8 KV units, S = 32768; 107 vs 166 us at S = 131072)
    if ((few || !one_wg) && (int64_t)s->B * s->H <= kSplitMaxUnits && s->S_max >= 8192 && shared_bucket_plan(s, lds_max, &p)) {
      p.plan = kPlanSharedBucket;
      return p;
    }
    if ((few || !one_wg) && shared_split_plan(s, lds_max, &p)) { p.plan = kPlanSharedSplit; return p; }
    if (one_wg) p.plan = kPlanShared;
    return p;
  }
  // Few units with long caches: the digit-bucket plan, where it was measured faster than one workgroup per unit, or as
  // fast (H = 32, r = 32, k = S / 16, bucket / one-workgroup us per decode at 32, 64, 96, 128 units; S = 4096: 20/16, 21/17,
  // 23/18, 25/18; 8192: 22/24, 25/25, 29/26, 34/28; 12 288: 24/32, 29/34, 36/35, 41/37; 16 384: 26/40, 33/42, 43/44, 52/46;
  // 24 576: 30/56, 41/59, 57/62, 83/65; 32 768: 34/74, 51/77, 86/82, 102/88), and whatever one workgroup's LDS cannot hold.
  const int64_t units = (int64_t)s->B * s->H;
  const bool one_wg_fits = decode_lds_bytes(s->S_max, s->d_h) <= lds_max;
  const bool bucket_faster = ((s->S_max >= 16384 && units <= 96) || (s->S_max >= 12288 && units <= 64)) && (by_size || !helped_faster(s));
  if (units <= kSplitMaxUnits && s->S_max >= 8192 && (bucket_faster || !one_wg_fits) && bucket_plan(s, lds_max, &p)) {
    p.plan = kPlanBucket;
    return p;
  }
  if (one_wg_fits) { p.plan = kPlanFused; return p; }
  if (two_level_plan(s, kLongSpan, lds_max, &p)) p.plan = kPlanLong;
  return p;
}

struct GsLayout { size_t z, stat, esc, alpha, cnt, ckey, cpos, list, part, end; int list_stride; };

GsLayout gs_layout(const sparq_shape* s, const PlanInfo& p) {
  const size_t units = (size_t)s->B * s->H, ukv = (size_t)s->B * s->H_kv, g = (size_t)(s->H / s->H_kv);
  GsLayout l;
  const int kk = s->k < s->S_max ? s->k : s->S_max;
  l.list_stride = (kk + 7) & ~7;
  size_t off = kControlBytes;
  l.z = off; off = align256(off + units * s->S_max * sizeof(float));
  l.stat = off; off = align256(off + ukv * p.n1 * g * 2 * sizeof(float));
  l.esc = off; off = align256(off + units * sizeof(float));
  l.alpha = off; off = align256(off + units * sizeof(float));
  l.cnt = off; off = align256(off + ukv * p.n_span * sizeof(int32_t));
  l.ckey = off; off = align256(off + ukv * p.n_span * p.cand_cap * sizeof(uint32_t));
  l.cpos = off; off = align256(off + ukv * p.n_span * p.cand_cap * sizeof(int32_t));
  l.list = off; off = align256(off + ukv * l.list_stride * sizeof(int32_t));
  l.part = off; off = align256(off + units * p.n_split * (s->d_h + 2) * sizeof(float));
  l.end = off;
  return l;
}

struct BucketLayout { size_t tmax, zsum, anum, tau, zden, coarse, fine, skey, spos, part, z, stat, esc, end; };

BucketLayout bucket_layout(const sparq_shape* s, const PlanInfo& p) {
  const size_t units = (size_t)s->B * s->H, slots = units * p.n_span;
  BucketLayout l;
  size_t off = kControlBytes;
  l.tmax = off; off = align256(off + slots * sizeof(float));
  l.zsum = off; off = align256(off + slots * sizeof(float));
  l.anum = off; off = align256(off + slots * sizeof(float));
  l.tau = off; off = align256(off + units * sizeof(float));
  l.zden = off; off = align256(off + units * sizeof(float));
  l.coarse = off; off = align256(off + slots * 64 * sizeof(uint16_t));
  l.fine = off; off = align256(off + slots * bk_fine_len() * sizeof(uint16_t));
  l.skey = off; off = align256(off + slots * p.span_len * sizeof(uint32_t));
  l.spos = off; off = align256(off + slots * p.span_len * sizeof(uint32_t));
  l.part = off; off = align256(off + slots * (s->d_h + 2) * sizeof(float));
  l.z = l.stat = l.esc = off;
  if (p.plan == kPlanSharedBucket) {      // what gs_logits hands on: logit numerators, span statistics, temperatures
    const size_t ukv = (size_t)s->B * s->H_kv, g = (size_t)(s->H / s->H_kv);
    l.z = off; off = align256(off + units * s->S_max * sizeof(float));
    l.stat = off; off = align256(off + ukv * p.n1 * g * 2 * sizeof(float));
    l.esc = off; off = align256(off + units * sizeof(float));
  }
  l.end = off;
  return l;
}

struct LongLayout { size_t tmax, zsum, cnt, tau, ckey, cpos, end; };

LongLayout long_layout(const sparq_shape* s, const PlanInfo& p) {
  const size_t units = (size_t)s->B * s->H;
  LongLayout l;
  size_t off = kControlBytes;
  l.tmax = off; off = align256(off + units * p.n_span * sizeof(float));
  l.zsum = off; off = align256(off + units * p.n_span * sizeof(float));
  l.cnt = off; off = align256(off + units * p.n_span * sizeof(int32_t));
  l.tau = off; off = align256(off + units * sizeof(float));
  l.ckey = off; off = align256(off + units * p.n_span * p.cand_cap * sizeof(uint32_t));
  l.cpos = off; off = align256(off + units * p.n_span * p.cand_cap * sizeof(int32_t));
  // (a position list per unit, as this plan once kept: it decides which shapes sparq_decode_noalloc refuses)
  l.end = align256(off + units * s->S_max * sizeof(int32_t));
  return l;
}

size_t workspace_need(const sparq_shape* s) {
  size_t need = (size_t)kControlBytes + (size_t)s->B * s->H * dense_room(s) * (s->d_h + 2) * sizeof(float);
  const PlanInfo p = choose_plan(s, true);
  size_t e = 0;
  if (p.plan == kPlanLong) e = long_layout(s, p).end;
  if (p.plan == kPlanBucket || p.plan == kPlanSharedBucket) e = bucket_layout(s, p).end;
  if (p.plan == kPlanShared) e = (size_t)kControlBytes + (size_t)s->B * s->H * s->S_max * sizeof(float);
  if (p.plan == kPlanSharedSplit) e = gs_layout(s, p).end;
#ifdef SPARQ_STAGE_CLOCKS
  if (p.plan == kPlanFused) e = (size_t)kControlBytes + (size_t)s->B * s->H * kStageStamps * sizeof(unsigned long long);
#endif
  return e > need ? e : need;
}

int check_workspace(const sparq_shape* s, const void* ws, size_t bytes) {
  if (!ws || !aligned16(ws) || bytes < workspace_need(s)) return SPARQ_EWORKSPACE;
  return SPARQ_OK;
}

// the sizes of a call; the pointers are the caller's to set
DecodeArgs sized_args(const sparq_shape* shape, int S_stride) {
  DecodeArgs a{};
  a.B = shape->B; a.H = shape->H; a.H_kv = shape->H_kv; a.S_max = shape->S_max; a.S_stride = S_stride; a.d_h = shape->d_h;
  a.r = shape->r; a.k = shape->k; a.flags = shape->flags; a.local_window = shape->local_window;
  return a;
}

// enqueue one decode over `a` with the plan the shape calls for
hipError_t enqueue_decode(const sparq_shape* shape, const DecodeArgs& args, void* workspace, size_t workspace_bytes, hipStream_t s) {
  DecodeArgs a = args;
  a.group = a.H / a.H_kv;
  a.by_H = make_divider(a.H); a.by_H_kv = make_divider(a.H_kv); a.by_group = make_divider(a.group);
  PlanInfo p = choose_plan(shape);
  if (p.plan == kPlanNone) return hipErrorInvalidValue;
  // (a workspace that the call accepts may have been sized for another plan: then one workgroup per unit, which needs none)
  if (p.plan == kPlanSingleBucket && workspace_bytes < bucket_layout(shape, p).end) p.plan = kPlanSingleK;
#ifdef SPARQ_STAGE_CLOCKS
  if (p.plan == kPlanFused) {
    DecodeArgs c = a;
    c.clocks = reinterpret_cast<unsigned long long*>(static_cast<char*>(workspace) + kControlBytes);
    return launch_decode(c, shape->dtype, s);
  }
#endif
  if (p.plan == kPlanFused) return launch_decode(a, shape->dtype, s);
  const bool one_k = p.plan == kPlanSingleK || p.plan == kPlanSingleBucket;
  DecodeArgs d = a;
  if (a.k_new && (p.plan == kPlanSharedSplit || one_k)) {
    // the grouped-query rule over several workgroups and the single-copy kernels have no append built in: the append
    // kernel writes the *_next state, and they decode from that
    AppendArgs ap;
    ap.K = a.K; ap.Kt = one_k ? nullptr : a.Kt; ap.V = a.V; ap.v_mean = const_cast<float*>(a.v_mean); ap.seq_lens = const_cast<int32_t*>(a.seq_lens);
    ap.v_mean_out = a.v_mean_next; ap.seq_lens_out = a.seq_lens_next;
    ap.k_new = a.k_new; ap.v_new = a.v_new; ap.n_new_per_seq = nullptr; ap.err = a.err;
    ap.B = a.B; ap.H_kv = a.H_kv; ap.S_max = a.S_max; ap.S_stride = a.S_stride; ap.d_h = a.d_h; ap.n_new = 1; ap.tiled = tiled_k(shape) ? 1 : 0;
    hipError_t e = launch_append(ap, shape->dtype, s);
    if (e != hipSuccess) return e;
    d.v_mean = a.v_mean_next; d.seq_lens = a.seq_lens_next;
    d.k_new = nullptr; d.v_new = nullptr; d.v_mean_next = nullptr; d.seq_lens_next = nullptr;
  }
  if (p.plan == kPlanSingleK) return launch_decode_single_k(d, shape->dtype, s);
  if (p.plan == kPlanShared)
    return launch_decode_shared(d, reinterpret_cast<float*>(static_cast<char*>(workspace) + kControlBytes), shape->dtype, s);
  char* w = static_cast<char*>(workspace);
  if (p.plan == kPlanSharedSplit) {
    const GsLayout l = gs_layout(shape, p);
    GsArgs ga;
    ga.d = d;
    ga.n1 = p.n1; ga.span1 = p.span1; ga.n2 = p.n_span; ga.span2 = p.span_len; ga.cand_cap = p.cand_cap;
    ga.n_split = p.n_split; ga.list_stride = l.list_stride;
    ga.by_n1 = make_divider(ga.n1); ga.by_n2 = make_divider(ga.n2); ga.by_split = make_divider(ga.n_split);
    ga.z_ws = reinterpret_cast<float*>(w + l.z);
    ga.stat_ws = reinterpret_cast<float*>(w + l.stat);
    ga.esc_ws = reinterpret_cast<float*>(w + l.esc);
    ga.alpha_ws = reinterpret_cast<float*>(w + l.alpha);
    ga.cnt_ws = reinterpret_cast<int32_t*>(w + l.cnt);
    ga.cand_key_ws = reinterpret_cast<uint32_t*>(w + l.ckey);
    ga.cand_pos_ws = reinterpret_cast<int32_t*>(w + l.cpos);
    ga.list_ws = reinterpret_cast<int32_t*>(w + l.list);
    ga.part_ws = reinterpret_cast<float*>(w + l.part);
    return launch_decode_shared_split(ga, shape->dtype, s);
  }
  if (p.plan == kPlanBucket || p.plan == kPlanSharedBucket || p.plan == kPlanSingleBucket) {
    const BucketLayout l = bucket_layout(shape, p);
    BucketArgs ba;
    ba.d = d;
    ba.rows = p.plan == kPlanSingleBucket;
    ba.n_span = p.n_span; ba.span_len = p.span_len; ba.cand_cap = p.cand_cap;
    ba.by_span = make_divider(ba.n_span); ba.by_len = make_divider(ba.span_len);
    ba.tmax_ws = reinterpret_cast<float*>(w + l.tmax);
    ba.zsum_ws = reinterpret_cast<float*>(w + l.zsum);
    ba.anum_ws = reinterpret_cast<float*>(w + l.anum);
    ba.tau_ws = reinterpret_cast<float*>(w + l.tau);
    ba.zden_ws = reinterpret_cast<float*>(w + l.zden);
    // Up to 512 workgroups run at once (two per CU) and the unit's last one merges.  With more, each would hold its place for
    // the two round trips of its arrival while others wait (100 units of 60 000 positions, 800 workgroups: 147.8 us per
    // decode against 144.4 with a launch for the merges, 100 000 positions 209.2 / 203.3; 64 units of 60 000, 512: equal).
    ba.merge = (int64_t)d.B * d.H * p.n_span <= 512;
    ba.tickets = reinterpret_cast<int32_t*>(w + kTicketOffset);
    ba.coarse_ws = reinterpret_cast<uint16_t*>(w + l.coarse);
    ba.fine_ws = reinterpret_cast<uint16_t*>(w + l.fine);
    ba.skey_ws = reinterpret_cast<uint32_t*>(w + l.skey);
    ba.spos_ws = reinterpret_cast<uint32_t*>(w + l.spos);
    ba.part_ws = reinterpret_cast<float*>(w + l.part);
    if (p.plan == kPlanSharedBucket) {
      GsArgs ga{};
      ga.d = d;
      ga.n1 = p.n1; ga.span1 = p.span1;
      ga.by_n1 = make_divider(ga.n1);
      ga.z_ws = reinterpret_cast<float*>(w + l.z);
      ga.stat_ws = reinterpret_cast<float*>(w + l.stat);
      ga.esc_ws = reinterpret_cast<float*>(w + l.esc);
      hipError_t e = launch_group_logits(ga, shape->dtype, s);
      if (e != hipSuccess) return e;
      ba.group = shape->H / shape->H_kv; ba.n1 = p.n1;
      ba.z_ws = ga.z_ws; ba.stat_ws = ga.stat_ws; ba.esc_ws = ga.esc_ws;
      return launch_decode_bucket_group(ba, shape->dtype, s);
    }
    return launch_decode_bucket(ba, shape->dtype, s);
  }
  if (p.plan == kPlanLong) {
    const LongLayout l = long_layout(shape, p);
    LongArgs la;
    la.d = d;
    la.n_span = p.n_span; la.span_len = p.span_len; la.cand_cap = p.cand_cap;
    la.by_span = make_divider(la.n_span);
    la.tmax_ws = reinterpret_cast<float*>(w + l.tmax);
    la.zsum_ws = reinterpret_cast<float*>(w + l.zsum);
    la.cnt_ws = reinterpret_cast<int32_t*>(w + l.cnt);
    la.tau_ws = reinterpret_cast<float*>(w + l.tau);
    la.cand_key_ws = reinterpret_cast<uint32_t*>(w + l.ckey);
    la.cand_pos_ws = reinterpret_cast<int32_t*>(w + l.cpos);
    return launch_decode_long(la, shape->dtype, s);
  }
  return hipErrorInvalidValue;
}

// the build of the one-workgroup-per-head kernel that a call gets
const char* fused_name(const DecodeArgs& a) {
  if (decode_helped(a)) return "sparq_decode_fused (one workgroup per head, one launch), idle CUs fetch";
  if (decode_short(a)) return "sparq_decode_fused (one workgroup per head, one launch), workgroups of four waves";
  if (decode_runs(a))
    return decode_apart(a) ? "sparq_decode_fused (one workgroup per head, one launch), waves read apart, append of a step apart"
                           : "sparq_decode_fused (one workgroup per head, one launch), waves read apart";
  if (decode_apart(a)) return "sparq_decode_fused (one workgroup per head, one launch), append of a step apart";
  return "sparq_decode_fused (one workgroup per head, one launch)";
}

bool decode_supported(const sparq_shape* shape) { return choose_plan(shape).plan != kPlanNone; }

// ---- library-owned scratch for sparq_decode_noalloc ----
// One array per GPU (each device that loads this code object holds its own copy at its own address), kept
// until the process ends.  In host code the array's name is only a handle for hipGetSymbolAddress: kernels,
// fills and copies take the device address looked up below, never the name.
constexpr size_t kStaticScratchBytes = (size_t)32 << 20;
constexpr int kMaxDevices = 64;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

// Device address of `scratch` on the current device; looked up (and the control block cleared by a fill
// kernel on `s`) on the first call per device.  Returns nullptr if the runtime refuses.
void* static_scratch(hipStream_t s) {
  static void* ptr[kMaxDevices] = {};      // benign race: every thread computes the same value
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  if (!ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return nullptr;
    if (launch_clear(p, kControlBytes, s) != hipSuccess) return nullptr;
    ptr[dev] = p;
  }
  return ptr[dev];
}

}  // namespace

extern "C" {

int sparq_workspace_bytes(const sparq_shape* caller_shape, size_t* out_bytes) {
  int rc = check_shape(caller_shape);
  if (rc != SPARQ_OK) return rc;
  if (!out_bytes) return SPARQ_EINVAL;
  const sparq_shape sized = bounded(caller_shape);
  const sparq_shape* shape = &sized;
  // a bulk append is served by any workspace that the other calls accept, on fewer workgroups if that is short
  const size_t need = workspace_need(shape);
  const size_t append = tiled_k(shape) ? 0 : kAppendScratchOffset + append_scratch_bytes((int64_t)shape->B * shape->H_kv, shape->S_max, shape->d_h);
  *out_bytes = append > need ? append : need;
  // the digit-bucket plan for a key cache stored once is used where a caller brings the room for it
  const PlanInfo p = choose_plan(shape);
  if (p.plan == kPlanSingleBucket && bucket_layout(shape, p).end > *out_bytes) *out_bytes = bucket_layout(shape, p).end;
  return SPARQ_OK;
}

int sparq_workspace_init(void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!workspace || !aligned16(workspace) || workspace_bytes < (size_t)kControlBytes) return SPARQ_EWORKSPACE;
  return launch_clear(workspace, kControlBytes, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? SPARQ_OK : SPARQ_ELAUNCH;
}

int sparq_kv_append(const sparq_shape* caller_shape, const sparq_cache* cache, const void* k_new,
                    const void* v_new, int32_t n_new, const int32_t* n_new_per_seq,
                    void* workspace, size_t workspace_bytes, void* hip_stream) {
  int rc = check_shape(caller_shape);
  if (rc == SPARQ_OK) rc = check_cache(cache, caller_shape);
  if (rc != SPARQ_OK) return rc;
  const sparq_shape sized = bounded(caller_shape);
  const sparq_shape* shape = &sized;
  if (!k_new || !v_new || !aligned16(k_new) || !aligned16(v_new) || n_new < 1 || n_new > caller_shape->S_max) return SPARQ_EINVAL;
  rc = check_workspace(shape, workspace, workspace_bytes);
  if (rc != SPARQ_OK) return rc;
  AppendArgs a;
  a.K = cache->K; a.Kt = single_k(shape) ? nullptr : cache->Kt; a.V = cache->V; a.v_mean = cache->v_mean; a.seq_lens = cache->seq_lens;
  a.v_mean_out = cache->v_mean; a.seq_lens_out = cache->seq_lens;
  a.k_new = k_new; a.v_new = v_new; a.n_new_per_seq = n_new_per_seq; a.err = static_cast<int32_t*>(workspace);
  a.B = shape->B; a.H_kv = shape->H_kv; a.S_max = a.S_stride = caller_shape->S_max;   // S_bound does not limit an append
  a.d_h = shape->d_h; a.n_new = n_new; a.tiled = tiled_k(shape) ? 1 : 0;
  a.scratch = static_cast<char*>(workspace) + kAppendScratchOffset; a.scratch_bytes = workspace_bytes - kAppendScratchOffset;
  a.tickets = reinterpret_cast<int32_t*>(static_cast<char*>(workspace) + kTicketOffset);
  return launch_append(a, shape->dtype, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? SPARQ_OK : SPARQ_ELAUNCH;
}

int sparq_decode(const sparq_shape* caller_shape, const sparq_cache* cache, const void* q,
                 const int32_t* k_per_seq, void* out, float* alpha_out, int32_t* idx_out,
                 int32_t idx_stride, int32_t* chan_out, void* workspace, size_t workspace_bytes,
                 void* hip_stream) {
  int rc = check_shape(caller_shape);
  if (rc == SPARQ_OK) rc = check_cache(cache, caller_shape);
  if (rc != SPARQ_OK) return rc;
  const sparq_shape sized = bounded(caller_shape);
  const sparq_shape* shape = &sized;
  if (!q || !out || !aligned16(q) || !aligned16(out)) return SPARQ_EINVAL;
  if (idx_out && idx_stride < 1) return SPARQ_EINVAL;
  rc = check_workspace(shape, workspace, workspace_bytes);
  if (rc != SPARQ_OK) return rc;
  if (!decode_supported(shape)) return SPARQ_EUNSUPPORTED;
  DecodeArgs a = sized_args(shape, caller_shape->S_max);
  a.K = cache->K; a.Kt = cache->Kt; a.V = cache->V; a.v_mean = cache->v_mean; a.seq_lens = cache->seq_lens;
  a.q = q; a.k_per_seq = k_per_seq; a.out = out; a.alpha_out = alpha_out; a.idx_out = idx_out;
  a.k_new = nullptr; a.v_new = nullptr; a.v_mean_next = nullptr; a.seq_lens_next = nullptr;
  a.chan_out = chan_out; a.err = static_cast<int32_t*>(workspace);
  a.idx_stride = idx_out ? idx_stride : 0;
  return enqueue_decode(shape, a, workspace, workspace_bytes, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? SPARQ_OK : SPARQ_ELAUNCH;
}

int sparq_decode_noalloc(const sparq_shape* caller_shape, const sparq_cache* cache, const void* q,
                         const int32_t* k_per_seq, void* out, float* alpha_out, int32_t* idx_out,
                         int32_t idx_stride, int32_t* chan_out, int32_t* error_word, void* hip_stream) {
  int rc = check_shape(caller_shape);
  if (rc == SPARQ_OK) rc = check_cache(cache, caller_shape);
  if (rc != SPARQ_OK) return rc;
  const sparq_shape sized = bounded(caller_shape);
  const sparq_shape* shape = &sized;
  if (!q || !out || !aligned16(q) || !aligned16(out)) return SPARQ_EINVAL;
  if (idx_out && idx_stride < 1) return SPARQ_EINVAL;
  if (!decode_supported(shape)) return SPARQ_EUNSUPPORTED;
  if (workspace_need(shape) > kStaticScratchBytes) return SPARQ_ETOOLARGE;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  void* ws = static_scratch(s);
  if (!ws) return SPARQ_ELAUNCH;
  DecodeArgs a = sized_args(shape, caller_shape->S_max);
  a.K = cache->K; a.Kt = cache->Kt; a.V = cache->V; a.v_mean = cache->v_mean; a.seq_lens = cache->seq_lens;
  a.q = q; a.k_per_seq = k_per_seq; a.out = out; a.alpha_out = alpha_out; a.idx_out = idx_out;
  a.k_new = nullptr; a.v_new = nullptr; a.v_mean_next = nullptr; a.seq_lens_next = nullptr;
  a.chan_out = chan_out; a.err = error_word ? error_word : static_cast<int32_t*>(ws);
  a.idx_stride = idx_out ? idx_stride : 0;
  return enqueue_decode(shape, a, ws, kStaticScratchBytes, s) == hipSuccess ? SPARQ_OK : SPARQ_ELAUNCH;
}

int sparq_decode_step(const sparq_shape* caller_shape, const sparq_cache* cache, const void* k_new,
                      const void* v_new, float* v_mean_next, int32_t* seq_lens_next, const void* q,
                      const int32_t* k_per_seq, void* out, float* alpha_out, int32_t* idx_out,
                      int32_t idx_stride, int32_t* chan_out, void* workspace, size_t workspace_bytes,
                      void* hip_stream) {
  int rc = check_shape(caller_shape);
  if (rc == SPARQ_OK) rc = check_cache(cache, caller_shape);
  if (rc != SPARQ_OK) return rc;
  const sparq_shape sized = bounded(caller_shape);
  const sparq_shape* shape = &sized;
  if (!q || !out || !aligned16(q) || !aligned16(out)) return SPARQ_EINVAL;
  if (!k_new || !v_new || !aligned16(k_new) || !aligned16(v_new)) return SPARQ_EINVAL;
  if (!v_mean_next || !seq_lens_next || !aligned16(v_mean_next)) return SPARQ_EINVAL;
  if (v_mean_next == cache->v_mean || seq_lens_next == cache->seq_lens) return SPARQ_EINVAL;
  if (idx_out && idx_stride < 1) return SPARQ_EINVAL;
  rc = check_workspace(shape, workspace, workspace_bytes);
  if (rc != SPARQ_OK) return rc;
  if (!decode_supported(shape)) return SPARQ_EUNSUPPORTED;
  DecodeArgs a = sized_args(shape, caller_shape->S_max);
  a.K = cache->K; a.Kt = cache->Kt; a.V = cache->V; a.v_mean = cache->v_mean; a.seq_lens = cache->seq_lens;
  a.q = q; a.k_per_seq = k_per_seq; a.out = out; a.alpha_out = alpha_out; a.idx_out = idx_out;
  a.k_new = k_new; a.v_new = v_new; a.v_mean_next = v_mean_next; a.seq_lens_next = seq_lens_next;
  a.chan_out = chan_out; a.err = static_cast<int32_t*>(workspace);
  a.idx_stride = idx_out ? idx_stride : 0;
  return enqueue_decode(shape, a, workspace, workspace_bytes, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? SPARQ_OK : SPARQ_ELAUNCH;
}

int dense_decode(const sparq_shape* caller_shape, const sparq_cache* cache, const void* q, void* out,
                 void* workspace, size_t workspace_bytes, void* hip_stream) {
  int rc = check_shape(caller_shape);
  if (rc == SPARQ_OK) rc = check_cache(cache, caller_shape);
  if (rc != SPARQ_OK) return rc;
  const sparq_shape sized = bounded(caller_shape);
  const sparq_shape* shape = &sized;
  if (!q || !out || !aligned16(q) || !aligned16(out)) return SPARQ_EINVAL;
  rc = check_workspace(shape, workspace, workspace_bytes);
  if (rc != SPARQ_OK) return rc;
  if (tiled_k(shape)) return SPARQ_EUNSUPPORTED;   // the comparison kernel reads key rows
  DenseArgs a;
  a.K = cache->K; a.V = cache->V; a.seq_lens = cache->seq_lens; a.q = q; a.out = out;
  a.partials = reinterpret_cast<float*>(static_cast<char*>(workspace) + kControlBytes);
  a.tickets = reinterpret_cast<int32_t*>(static_cast<char*>(workspace) + kTicketOffset);
  a.err = static_cast<int32_t*>(workspace);
  a.B = shape->B; a.H = shape->H; a.H_kv = shape->H_kv; a.S_max = shape->S_max; a.S_stride = caller_shape->S_max; a.d_h = shape->d_h;
  dense_plan(shape, &a.n_split, &a.rows_per_split);
  return launch_dense(a, shape->dtype, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? SPARQ_OK : SPARQ_ELAUNCH;
}

int sparq_async_error(void* workspace, int32_t* host_flag, void* hip_stream) {
  if (!workspace || !host_flag) return SPARQ_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  if (hipMemcpyAsync(host_flag, workspace, sizeof(int32_t), hipMemcpyDeviceToHost, s) != hipSuccess) return SPARQ_ELAUNCH;
  if (launch_clear(workspace, kWorkspaceHeader, s) != hipSuccess) return SPARQ_ELAUNCH;
  return hipStreamSynchronize(s) == hipSuccess ? SPARQ_OK : SPARQ_ELAUNCH;
}

int sparq_copy_probe(void* dst, const void* src, size_t n_bytes, void* hip_stream) {
  if (!dst || !src || !aligned16(dst) || !aligned16(src) || n_bytes % 16 != 0) return SPARQ_EINVAL;
  return launch_copy_probe(dst, src, n_bytes, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? SPARQ_OK : SPARQ_ELAUNCH;
}

int sparq_read_probe(const void* src, size_t n_bytes, void* sink, size_t sink_bytes, void* hip_stream) {
  if (!src || !sink || !aligned16(src) || !aligned16(sink) || n_bytes % 16 != 0) return SPARQ_EINVAL;
  if (sink_bytes < (size_t)kProbeBlocks * 256 * sizeof(uint32_t)) return SPARQ_EWORKSPACE;
  return launch_read_probe(src, n_bytes, sink, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? SPARQ_OK : SPARQ_ELAUNCH;
}

const char* sparq_decode_plan(const sparq_shape* caller_shape) {
  if (check_shape(caller_shape) != SPARQ_OK) return "invalid shape";
  const sparq_shape sized = bounded(caller_shape);
  const sparq_shape* shape = &sized;
  switch (choose_plan(shape).plan) {
    case kPlanFused: return fused_name(sized_args(shape, caller_shape->S_max));
    case kPlanLong: return "long_scores + long_finish (two-level selection plan)";
    case kPlanBucket: return "bk_scores + bk_select_gather (digit-bucket plan)";
    case kPlanShared: return "sparq_decode_shared (grouped-query rule, one workgroup per KV head)";
    case kPlanSharedBucket: return "gs_logits + bk_group_scores + bk_select_gather (grouped-query rule on the digit-bucket plan)";
    case kPlanSharedSplit: return "gs_logits + gs_select + gs_merge + gs_gather + split_combine (grouped-query rule, several workgroups per KV head)";
    case kPlanSingleBucket: return "bk_scores + bk_select_gather (digit-bucket plan, key cache stored once)";
    case kPlanSingleK:
      return decode_single_k_short(sized_args(shape, caller_shape->S_max)) ? "sparq_decode_single_k (key cache stored once), workgroups of four waves"
                                                                           : "sparq_decode_single_k (key cache stored once)";
    default: return "unsupported";
  }
}

int sparq_stage_clocks(const sparq_shape* caller_shape, size_t* offset_bytes, int32_t* n_workgroups, int32_t* stamps_per_workgroup) {
  if (!offset_bytes || !n_workgroups || !stamps_per_workgroup) return SPARQ_EINVAL;
  const int rc = check_shape(caller_shape);
  if (rc != SPARQ_OK) return rc;
#ifdef SPARQ_STAGE_CLOCKS
  const sparq_shape sized = bounded(caller_shape);
  const sparq_shape* shape = &sized;
  if (choose_plan(shape).plan != kPlanFused) return SPARQ_EUNSUPPORTED;
  *offset_bytes = kControlBytes; *n_workgroups = shape->B * shape->H; *stamps_per_workgroup = kStageStamps;
  return SPARQ_OK;
#else
  return SPARQ_EUNSUPPORTED;
#endif
}

const char* sparq_status_string(int status) {
  switch (status) {
    case SPARQ_OK: return "ok";
    case SPARQ_EINVAL: return "invalid argument";
    case SPARQ_EUNSUPPORTED: return "unsupported shape or mode";
    case SPARQ_EWORKSPACE: return "workspace missing, misaligned or too small";
    case SPARQ_ELAUNCH: return "HIP launch failed";
    case SPARQ_ETOOLARGE: return "shape needs more scratch than the library's built-in buffer holds";
    default: return "unknown status";
  }
}

}  // extern "C"
