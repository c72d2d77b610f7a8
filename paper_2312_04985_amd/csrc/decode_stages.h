// The stages of the SparQ decode step (Section 4, Steps 1-3) as workgroup-level device functions.
// Every decode plan is a different distribution of these stages over workgroups: one workgroup per
// (sequence, head) (sparq_decode_fused.h), digit buckets over spans (sparq_decode_bucket.hip), two-level selection
// (sparq_decode_long.hip), the grouped-query rule (sparq_decode_shared.hip), the single-copy key cache
// (sparq_decode_single_k.hip); the append kernels use the column flush.
// Unless noted, functions are called by all NT threads of a workgroup (they contain barriers).
#pragma once
#include "common.h"
#include "params.h"
#include "two_ahead.h"

#include <type_traits>

// Waves per workgroup of what a source builds from the stages: 8, or what it defines before it includes this (4).  The two
// are namespaces of their own, so that no linker takes one's code for the other's.
#ifndef SPARQ_WAVES
#define SPARQ_WAVES 8
#endif
#if SPARQ_WAVES == 8
#define SPARQ_STAGES waves8
#elif SPARQ_WAVES == 4
#define SPARQ_STAGES waves4
#else
#error "4 or 8 waves"
#endif

namespace sparq {
inline namespace SPARQ_STAGES {

constexpr int NW = SPARQ_WAVES;   // waves per workgroup
constexpr int NT = NW * kWave;
static_assert(SPARQ_WAVES != 8 || NT == kDecodeThreads, "what the host sizes LDS for");
constexpr int kTieHeavy = 2048;  // a radix bin with more keys than this is counted tie-robustly in the next pass

// ------------------------------------------------------------------------------------------------
// small workgroup primitives

// Histogram bins are stored swizzled: the 32 consecutive digits that lane l sums in find_threshold_bin are row l of 32 words,
// its eight 16-byte pieces permuted by xor, so that 16 neighbouring lanes reading the same piece of their rows touch all 64
// banks once.
__device__ __forceinline__ uint32_t hist_slot(uint32_t digit) { return digit ^ ((digit >> 4) & 28u); }
// the 16 bytes of digits 32 lane + 4 piece .. + 3
__device__ __forceinline__ uint32_t hist_piece(int lane, int piece) { return ((uint32_t)lane << 5) | (((uint32_t)piece << 2) ^ (((uint32_t)lane << 1) & 28u)); }

// First-digit counts of 8 or 4 neighbouring keys per lane; n_valid = how many of them count (the leading ones).
// The atomics of lanes that meet in one address come one after the other.  8 keys: where most lanes of the wave hold one digit
// (duplicated keys), it is counted over the wave and added once; two of a lane's keys tell, so that no regular pattern of
// duplicates hides it.  us per decode of 2048 heads at 8192 positions, one atomic per run of equal neighbours / one for a lane
// whose keys are all equal / this: ordinary keys 132.8 / 128.7 / 128.3, all identical 189.8 / 178.6 / 179.1, one distinct in 8
// 181.7 / 200.0 / 172.1, one in 4 177.4 / 186.7 / 165.6, half of them identical 172.1 / 167.9 / 165.3.
// (Whole chunks without the test of n_valid per key: 0.1 of 9.5 us where a single head waits for it.)
__device__ __forceinline__ void hist_add_chunk(uint32_t* hist, const uint32_t (&kx)[8], int n_valid) {
  if (n_valid <= 0) return;
  constexpr int kHot = 40;                 // of 64 lanes
  const uint32_t d1 = kx[1] >> 21, d2 = kx[6] >> 21;
  const uint32_t h1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)d1), h2 = (uint32_t)__builtin_amdgcn_readfirstlane((int)d2);
  const int n1 = __popcll(__ballot(d1 == h1)), n2 = __popcll(__ballot(d2 == h2));
  if (__builtin_expect((n1 > n2 ? n1 : n2) > kHot, 0)) {
    const uint32_t hot = n1 > n2 ? h1 : h2;
    uint32_t n = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint32_t d = kx[e] >> 21;
      n += (uint32_t)__popcll(__ballot(e < n_valid && d == hot));
      if (e < n_valid && d != hot) atomicAdd(&hist[hist_slot(d)], 1u);
    }
    const uint64_t here = __ballot(true);
    if (__builtin_amdgcn_mbcnt_hi((uint32_t)(here >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)here, 0u)) == 0) atomicAdd(&hist[hist_slot(hot)], n);
    return;
  }
  if (n_valid >= 8) {
#pragma unroll
    for (int e = 0; e < 8; ++e) atomicAdd(&hist[hist_slot(kx[e] >> 21)], 1u);
    return;
  }
#pragma unroll
  for (int e = 0; e < 8; ++e)
    if (e < n_valid) atomicAdd(&hist[hist_slot(kx[e] >> 21)], 1u);
}
// 4 keys (spans whose keys are sorted afterwards, where duplicates take far longer): one atomic for a lane whose keys share the
// digit.  (Counted over the wave, ordinary keys took 0.2 of 58 us longer, 80 % identical ones 1 of 240 less.)
__device__ __forceinline__ void hist_add_chunk(uint32_t* hist, const uint32_t (&kx)[4], int n_valid) {
  if (n_valid <= 0) return;
  if (((kx[1] ^ kx[0]) | (kx[2] ^ kx[0]) | (kx[3] ^ kx[0])) >> 21 == 0) {
    atomicAdd(&hist[hist_slot(kx[0] >> 21)], (uint32_t)(n_valid < 4 ? n_valid : 4));
    return;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (e < n_valid) atomicAdd(&hist[hist_slot(kx[e] >> 21)], 1u);
}

// Count one key per lane into a histogram when many lanes may hold the same digit (exact ties: 64 LDS
// atomics on one address are serialised).  Up to four rounds: the first pending lane's digit is broadcast and
// all lanes holding it are counted with one atomic; what is left goes through plain atomics.  Called by all
// lanes of a wave together; lanes with valid = false contribute nothing.
__device__ __forceinline__ void hist_add_ties(uint32_t* hist, uint32_t digit, bool valid, int lane) {
  uint64_t todo = __ballot(valid);
#pragma unroll 1
  for (int it = 0; it < 4 && todo; ++it) {
    const int leader = __ffsll((unsigned long long)todo) - 1;
    const uint32_t dsel = (uint32_t)__builtin_amdgcn_readlane((int)digit, leader);
    const uint64_t same = __ballot(valid && digit == dsel) & todo;
    if (lane == leader) atomicAdd(&hist[hist_slot(dsel)], (uint32_t)__popcll(same));
    todo &= ~same;
  }
  if ((todo >> lane) & 1ull) atomicAdd(&hist[hist_slot(digit)], 1u);
}

// One wave locates the digit at which the count taken from the top digit downwards reaches `need`;
// writes {digit, how many keys of that digit are needed, keys with that digit} to ctl[0..2].
// Two levels: lane l sums digits 32l..32l+31 and a wave scan finds the lane, then the 32 digits of
// that lane are scanned across lanes.  Requires 1 <= need <= total count.
__device__ __forceinline__ void find_threshold_bin(const uint32_t* hist, int need, int lane, int* ctl) {
  uint32_t mine = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const uint4 v = *reinterpret_cast<const uint4*>(hist + hist_piece(lane, i));
    mine += (v.x + v.y) + (v.z + v.w);
  }
  const uint32_t incl = wave_scan_incl(mine);
  const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
  const uint32_t above = total - incl;      // keys with digits owned by higher lanes
  const uint64_t hit = __ballot(above < (uint32_t)need && (uint32_t)need <= above + mine);
  const int ls = hit ? __ffsll((unsigned long long)hit) - 1 : 0;
  const uint32_t need2 = (uint32_t)need - (uint32_t)__builtin_amdgcn_readlane((int)above, ls);
  // lane t < 32 takes digit 32*ls + 31 - t, so that the scan runs from the top digit down
  const uint32_t c = lane < 32 ? hist[hist_slot((uint32_t)(ls * 32 + 31 - lane))] : 0u;
  const uint32_t inc2 = wave_scan_incl(c);
  if (lane < 32 && (inc2 - c) < need2 && need2 <= inc2) {
    ctl[0] = ls * 32 + 31 - lane; ctl[1] = (int)(need2 - (inc2 - c)); ctl[2] = (int)c;
  }
}

// Workgroup -> (unit, span) of a launch over U units of n_span spans each.
__device__ __forceinline__ void map_span(int U, int n_span, Divider by_span, int& u, int& s) {
  const int bid = blockIdx.x;
  const bool shared = (U & 7) == 0;      // the spans of a unit, and the heads of a KV group, share an XCD
  const int slot = shared ? bid >> 3 : bid, q = divided(slot, by_span);
  u = shared ? (bid & 7) * (U >> 3) + q : q;
  s = slot - q * n_span;
}

// The length a launch of a multi-launch plan works on.  Inside sparq_decode_step (d.k_new set) the row being appended counts as position
// S_b although it reaches the cache only in the plan's last launch: every launch adds it the same way.
__device__ __forceinline__ int visible_length(const DecodeArgs& d, int b, bool& appended, bool& bad, bool& full) {
  int S = d.seq_lens[b];
  bad = S < 0 || S > d.S_max;
  if (bad) S = S < 0 ? 0 : d.S_max;
  appended = false; full = false;
  if (d.k_new) {
    if (S + 1 <= d.S_max) { appended = true; S += 1; } else full = true;
  }
  return S;
}

struct Nothing {
  __device__ __forceinline__ void operator()() const {}
};

// ------------------------------------------------------------------------------------------------
// Step 1a: the r largest components of |q| (ties to the lower channel) and the temperature (Eq. 9)

struct QueryLds {
  float* qf;       // [DH] query as fp32
  float* qs;       // [DH] selected query components, channel-ascending, padded to a multiple of 8
  int* chan;       // [DH] selected channels, ascending, same padding
};

// The 16-bit codes of channels lane * DH / 64 .. + DH / 64 - 1 of a row of DH (16-byte aligned).
template <int DH>
struct LaneCodes {
  static constexpr int E = DH / kWave;
  uint32_t c[E];
};
template <int DH>
__device__ __forceinline__ LaneCodes<DH> load_lane_codes(const uint16_t* row, int lane) {
  LaneCodes<DH> v;
  if (DH == 64) {
    v.c[0] = row[lane];
  } else {
#pragma unroll
    for (int i = 0; i < DH / 128; ++i) {
      const uint32_t w = reinterpret_cast<const uint32_t*>(row)[lane * (DH / 128) + i];
      v.c[2 * i] = w & 0xffffu; v.c[2 * i + 1] = w >> 16;
    }
  }
  return v;
}

// The r largest of the 64 E keys of a wave (E per lane, key e of lane l belonging to channel l E + e; BITS significant bits),
// ties to the lower channel: from the top down, two bits at a time, the largest t that at least r keys reach, ending as soon
// as exactly r do.
// Returns per key whether it is taken, and the number of taken keys of lower channels.  No LDS and no barrier.
template <int E, int BITS, class K>
__device__ __forceinline__ void wave_top_r(const K (&key)[E], int r, bool (&sel)[E], int (&before)[E]) {
  K t = 0;
  int n = E * kWave;                       // keys that reach t
  for (int bit = (BITS - 1) & ~1; bit >= 0 && n != r; bit -= 2) {
    K cand[3];
    int c[3] = {0, 0, 0};
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      cand[i] = t | ((K)(i + 1) << bit);
#pragma unroll
      for (int e = 0; e < E; ++e) c[i] += __popcll(__ballot(key[e] >= cand[i]));
    }
#pragma unroll
    for (int i = 0; i < 3; ++i)
      if (c[i] >= r) { t = cand[i]; n = c[i]; }
  }
  if (__builtin_expect(n == r, 1)) {
#pragma unroll
    for (int e = 0; e < E; ++e) sel[e] = key[e] >= t;
  } else {                                 // more than r - (keys above t) keys equal t: the first of them
    uint64_t eq[E];
    int need = r, lower = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      eq[e] = __ballot(key[e] == t);
      need -= __popcll(__ballot(key[e] > t));
      lower += (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(eq[e] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)eq[e], 0u));
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
      sel[e] = key[e] > t || (key[e] == t && lower < need);
      lower += key[e] == t ? 1 : 0;
    }
  }
  int b = 0;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const uint64_t m = __ballot(sel[e]);
    b += (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
  }
#pragma unroll
  for (int e = 0; e < E; ++e) { before[e] = b; b += sel[e] ? 1 : 0; }
}

// The first wave selects, on the 15-bit magnitude codes in its registers (about ten rounds of compare, ballot and count), and
// writes the list, the query and the L1 norms of all and of the selected components (sums[0..1]): one barrier, which also
// publishes whatever the caller wrote to LDS before the call.  The caller turns the norms into the temperature when the first
// loads of Step 1b are under way.  The list is padded to a multiple of 8 with the last channel at weight 0, so that Step 1b
// works on whole batches of 8 rows.
// (Ranking by counting larger keys in LDS, the comparisons dealt out over the workgroup, took three barriers and 1.0 us of a
// call, every wave selecting for itself 0.7: the two waves of a SIMD take turns, so that one wave is done sooner.  Per
// step, every wave / the first: one head at 1024 positions 9.65 / 9.45 us, 32 heads at 3981 19.1 / 18.8, 32 heads on 8 KV heads
// at 32 768 32.2 / 31.8, under the group rule 35.9 / 35.3; nothing where workgroups fill the chip.)
template <class T, int DH>
__device__ __forceinline__ void select_channels(const QueryLds& Q, const LaneCodes<DH>& q, int r, float* sums, int lane, int wave) {
  constexpr int E = DH / kWave;
  if (wave == 0) {
    uint32_t mag[E];
    float qv[E];
#pragma unroll
    for (int e = 0; e < E; ++e) { mag[e] = q.c[e] & 0x7fffu; qv[e] = T::widen((uint16_t)q.c[e]); }
    bool sel[E];
    int at[E];
    wave_top_r<E, 15>(mag, r, sel, at);
    float l1a = 0.0f, l1s = 0.0f;
    const int r8 = (r + 7) & ~7;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int j = lane * E + e;
      const float aq = fabsf(qv[e]);
      l1a += aq; l1s += sel[e] ? aq : 0.0f;
      Q.qf[j] = qv[e];
      if (sel[e]) {
        Q.chan[at[e]] = j; Q.qs[at[e]] = qv[e];
        if (at[e] == r - 1)
          for (int pp = r; pp < r8; ++pp) { Q.chan[pp] = j; Q.qs[pp] = 0.0f; }
      }
    }
    l1a = wave_sum(l1a); l1s = wave_sum(l1s);
    if (lane == 0) { sums[0] = l1a; sums[1] = l1s; }
  }
  __syncthreads();
}

// The temperature actually used: Eq. (9), or one of the two fixed values of the ablation in Section 5.3
// (flag bits 3 and 4).
__device__ __forceinline__ float apply_tau_mode(float tau_l1, uint32_t flags, int d_h, int r) {
  if (flags & 8u) return sqrtf((float)d_h);
  if (flags & 16u) return sqrtf((float)r);
  return tau_l1;
}
__device__ __forceinline__ float temperature(const float* sums, uint32_t flags, int d_h, int r) {
  const float all = sums[0], sel = sums[1];
  return apply_tau_mode(all > 0.0f ? sqrtf((float)d_h * sel / all) : sqrtf((float)d_h), flags, d_h, r);
}

// Local window: the last n_local = min(l, kq) positions are selected unconditionally; the select then
// runs over the S - n_local older positions for kq - n_local of them.
struct Window {
  int n_local, S_old, k_old;
};
__device__ __forceinline__ Window make_window(int local_window, int S, int kq) {
  Window w;
  w.n_local = local_window < kq ? local_window : kq;
  w.S_old = S - w.n_local;
  w.k_old = kq - w.n_local;
  return w;
}

// ------------------------------------------------------------------------------------------------
// Step 1b: approximate logit numerators over the r selected rows of the S-contiguous key copy

// 16 bytes of each of 8 listed rows.  The list is read as two 16-byte words and a row's address is one wide multiply-add per
// lane: with the row numbers moved to scalar registers and multiplied there, requesting 16 rows took 0.7 us of a
// wave's time (one scalar instruction after the other), this way 0.3.
// V: u32x4 keeps the 16 bytes of a request in one register tuple, uint4 are four words that the compiler may part.
template <bool KEEP = false, class V>
__device__ __forceinline__ void issue_rows(V (&v)[8], const char* base, uint32_t row_bytes, const int* chan) {
  const int4 lo = reinterpret_cast<const int4*>(chan)[0], hi = reinterpret_cast<const int4*>(chan)[1];
  uint32_t ch[8] = {(uint32_t)lo.x, (uint32_t)lo.y, (uint32_t)lo.z, (uint32_t)lo.w, (uint32_t)hi.x, (uint32_t)hi.y, (uint32_t)hi.z, (uint32_t)hi.w};
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    asm("" : "+v"(ch[t]));               // (the same in every lane: kept in a vector register all the same)
    v[t] = load16_as<V, KEEP>(base + (uint64_t)ch[t] * row_bytes);
  }
}

// Chunks (8 consecutive positions = 16 bytes of every channel row) chunk_begin + tid + i * STRIDE belong to
// thread tid of STRIDE (all NT threads of the workgroup unless the caller divides the rows of a chunk among
// groups of threads).  RUNS: where that is more than two per thread, they are cut into runs of 64, one chunk per lane, and every wave
// takes consecutive runs (the first waves one more where they do not come out even), so that the NW waves read at places 1 / NW of the row
// apart and not side by side (for row strides at which that is faster: decode_runs).
// The (chunk, batch-of-8-rows) pairs a thread owns form one flat sequence that runs through
// a two-deep software pipeline: a batch of 8 loads is always in flight behind the one being accumulated,
// also across chunk boundaries.  fp32 FMA in ascending channel order.  finish(c, acc) is called with the
// 8 sums of chunk c.  requested() is called by whole waves once their first batches of loads are under way: work that
// Step 1b does not wait for.  No barrier.
// The buffers are tuples of four registers each (u32x4).  As uint4 the compiler carried them through the loop word by word:
// copies of words still in flight, each with its wait, and bf16 codes widened several rows ahead, which went to scratch memory
// with the append and was held back there, and in every other bf16 call of the one-workgroup kernel, by a scheduling barrier
// behind each row.  Per decode / step in bf16, barrier / tuples: 32 heads at 3981 positions 17.9 / 16.8 and 18.6 / 17.5 us, 64
// heads of 64 channels at 6000 15.0 / 14.2 and 16.4 / 15.1, 512 at 4096 44.3 / 45.0 and 51.1 / 49.5, 2048 at 8192 132.5 / 130.2
// and 138.5 / 137.9; 2048 in f16 130.6 / 129.0 and 137.5 / 136.8.
// Addressing: chunk c of channel row j lies at Kt_head + j * row_bytes + c * chunk_bytes.  The S-contiguous
// key copy has row_bytes = 2 S_max and chunk_bytes = 16; the tiled single-copy layout (tiles of 8 positions,
// channel-major inside a tile) has row_bytes = 16 and chunk_bytes = 16 d_h.
template <class T, int STRIDE = NT, bool KEEP = false, bool RUNS = false, class Finish, class Requested>
__device__ __forceinline__ void stream_channel_rows(const char* Kt_head, uint32_t row_bytes, const int* chan,
                                                    const float* qs, int r, int chunk_begin, int chunk_end,
                                                    int tid, Finish&& finish, Requested&& requested, uint32_t chunk_bytes = 16u) {
  const int n_batches = (r + 7) >> 3;
  const int n_chunks = chunk_end - chunk_begin;
  constexpr int W = STRIDE / kWave;
  int own = tid, my_chunks = n_chunks > tid ? (n_chunks - tid + STRIDE - 1) / STRIDE : 0, step = STRIDE;
  if (RUNS && n_chunks > 2 * STRIDE) {
    const int w = tid / kWave, runs = (n_chunks + kWave - 1) / kWave, per = runs / W, more = runs % W;
    own += (w * (per - 1) + (w < more ? w : more)) * kWave;
    my_chunks = (n_chunks - own + kWave - 1) / kWave;
    if (my_chunks > per + (w < more)) my_chunks = per + (w < more);
    step = kWave;
  }
  const int items = my_chunks * n_batches;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  int ic = 0, ib = 0, cc = 0, cb = 0;   // issue and consume cursors: (own chunk number, batch)
  auto issue_next = [&](u32x4 (&v)[8]) {
    issue_rows<KEEP>(v, Kt_head + (size_t)((uint32_t)(chunk_begin + own + ic * step) * chunk_bytes), row_bytes, chan + ib * 8);
    if (++ib == n_batches) { ib = 0; ++ic; }
  };
  auto consume_next = [&](const u32x4 (&v)[8]) {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const float qv = qs[cb * 8 + t];
      float f[8];
      unpack8<T>(make_uint4(v[t].x, v[t].y, v[t].z, v[t].w), f);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = fmaf(f[e], qv, acc[e]);
    }
    if (++cb == n_batches) {
      finish(chunk_begin + own + cc * step, acc);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = 0.0f;
      cb = 0; ++cc;
    }
  };
  u32x4 v[2][8];
  two_ahead(items, __any(items > 1), [&](auto buffer) { issue_next(v[buffer.value]); }, [&](auto buffer) { consume_next(v[buffer.value]); },
            requested, [&]() { ic = 0; });
}

// ------------------------------------------------------------------------------------------------
// The newest S mod 8 keys of a sequence.  The S-contiguous copy Kt is brought up to date 8 positions at
// a time (one aligned 16-byte store per channel row every 8th append, instead of a 2-byte store per
// channel on every append: those cost a 32-byte memory transaction each).  Positions 8 floor(S/8) .. S-1
// therefore are not in Kt yet; there are at most 7 of them and their approximate logit numerators come
// from the rows of K: wave w takes position 8 floor(S/8) + w, lane l the channels l, l + 64, ... of the
// padded list; with fewer than 8 waves a wave takes several.  The loads are issued before Step 1b streams Kt and used after it.
struct TailRow {
  uint16_t raw[4];   // up to 256 list entries over 64 lanes
};

__device__ __forceinline__ TailRow tail_row_issue(const uint16_t* krow, const int* chan, int r8, int lane) {
  TailRow t;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int jj = lane + i * kWave;
    t.raw[i] = jj < r8 ? krow[chan[jj]] : (uint16_t)0;
  }
  return t;
}

template <class T>
__device__ __forceinline__ float tail_row_dot(const TailRow& t, const float* qs, int r8, int lane) {
  float part = 0.0f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int jj = lane + i * kWave;
    if (jj < r8) part = fmaf(T::widen(t.raw[i]), qs[jj], part);
  }
  return wave_sum(part);
}

// Positions S-8 .. S-1 of channel j of one KV head, S a multiple of 8, as 16 bytes: rows S-8 .. S-2 of
// K_head (cached by earlier calls) and `newest`, the code of the row being appended.
__device__ __forceinline__ uint4 gather_key_columns(const uint16_t* K_head, int d_h, int S, int j, uint16_t newest) {
  uint32_t w[4];
#pragma unroll
  for (int e = 0; e < 8; e += 2) {
    const uint32_t lo = K_head[(size_t)(S - 8 + e) * d_h + j];
    const uint32_t hi = e + 1 < 7 ? K_head[(size_t)(S - 8 + e + 1) * d_h + j] : (uint32_t)newest;
    w[e >> 1] = lo | (hi << 16);
  }
  return make_uint4(w[0], w[1], w[2], w[3]);
}
// ... written as columns S-8 .. S-1 of Kt: one 16-byte store
__device__ __forceinline__ void flush_key_columns(uint16_t* Kt_head, const uint16_t* K_head, int S_stride, int d_h,
                                                  int S, int j, uint16_t newest) {
  // (a non-temporal store: each of these 16 bytes is a line of its own that nothing reads for the next 8 steps; with
  // 2048 KV heads the step is 1-2 % faster, with 512 it is 0.5 % slower)
  const uint4 c = gather_key_columns(K_head, d_h, S, j, newest);
  u32x4 v;
  v.x = c.x; v.y = c.y; v.z = c.z; v.w = c.w;
  __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(Kt_head + (size_t)j * S_stride + (S - 8)));
}

// ------------------------------------------------------------------------------------------------
// transpose 8 rows x 8 channels of 16-bit codes: w[c] = the 8 rows' codes of channel c
__device__ __forceinline__ void transpose_piece(const uint4 (&rows)[8], uint4 (&w)[8]) {
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    uint32_t o[4];
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      const uint32_t a = c < 2 ? rows[e].x : (c < 4 ? rows[e].y : (c < 6 ? rows[e].z : rows[e].w));
      const uint32_t b = c < 2 ? rows[e + 1].x : (c < 4 ? rows[e + 1].y : (c < 6 ? rows[e + 1].z : rows[e + 1].w));
      o[e >> 1] = (c & 1) ? (a >> 16) | (b & 0xffff0000u) : (a & 0xffffu) | (b << 16);
    }
    w[c] = make_uint4(o[0], o[1], o[2], o[3]);
  }
}

// The append of sparq_decode_step inside the decode's launch, for channel c of a KV head: the new row (codes kc, vc) into K and
// V at position S - 1, the mean that includes it into the *_next buffer, and with a row that completes a group of 8 the
// channel's 8 columns of Kt (TILED: its 16 bytes of the tile).  No workgroup of the launch reads what this writes: every head
// takes the row from k_new / v_new, the columns lie above its S_fl, the state it reads is the old one.
template <int DH, bool TILED>
__device__ __forceinline__ void append_channel(const DecodeArgs& a, size_t kv_head, int c, int S, bool appended, uint16_t kc, uint16_t vc, float mean) {
  a.v_mean_next[kv_head * DH + c] = mean;
  if (!appended) return;
  uint16_t* K_head = reinterpret_cast<uint16_t*>(a.K) + kv_head * a.S_stride * (size_t)DH;
  // rows by position: the rows of K, or the rows of the newest positions (tiled layout)
  uint16_t* rows = TILED ? reinterpret_cast<uint16_t*>(a.Kt) + kv_head * (size_t)(8 * DH) - (size_t)((S - 1) & ~7) * DH : K_head;
  reinterpret_cast<uint16_t*>(a.V)[(kv_head * a.S_stride + (S - 1)) * DH + c] = vc;
  if (!TILED || (S & 7) != 0) rows[(size_t)(S - 1) * DH + c] = kc;
  if ((S & 7) != 0) return;
  if (!TILED)
    flush_key_columns(reinterpret_cast<uint16_t*>(a.Kt) + kv_head * DH * (size_t)a.S_stride, rows, a.S_stride, DH, S, c, kc);
  else
    *reinterpret_cast<uint4*>(K_head + (size_t)(S - 8) * DH + (size_t)c * 8) = gather_key_columns(rows, DH, S, c, kc);
}

// ... by workgroups of their own, the last of the grid, which take the places that decoding workgroups have left: workgroup i of
// append_workgroups() has NT / (DH / 8) KV heads, a thread 8 channels of one.  Bound by the scattered stores of a completed group;
// few workgroups spread them over the launch's end.  (A channel per thread, eight times as many workgroups: 2048 heads at 4096
// positions 182 us per such step, so 179.)
inline int append_workgroups(int64_t heads, int d_h) { return (int)((heads * (d_h / 8) + NT - 1) / NT); }

template <class T, int DH, bool TILED>
__device__ __forceinline__ void append_heads(const DecodeArgs& a, int i) {
  constexpr int LPR = DH / 8;
  const int head = i * (NT / LPR) + (int)threadIdx.x / LPR, j0 = ((int)threadIdx.x % LPR) * 8;
  if (head >= a.B * a.H_kv) return;
  const int b = divided(head, a.by_H_kv);
  const size_t at = (size_t)head * DH + j0;
  const uint4 kc = load16(reinterpret_cast<const uint16_t*>(a.k_new) + at), vc = load16(reinterpret_cast<const uint16_t*>(a.v_new) + at);
  float m[8];
#pragma unroll
  for (int e = 0; e < 8; e += 4) {
    const float4 v = *reinterpret_cast<const float4*>(a.v_mean + at + e);
    m[e] = v.x; m[e + 1] = v.y; m[e + 2] = v.z; m[e + 3] = v.w;
  }
  bool appended, bad, full;               // (reported by the decoding workgroups)
  const int S = visible_length(a, b, appended, bad, full);
  if (appended) {
    uint16_t* K_head = reinterpret_cast<uint16_t*>(a.K) + (size_t)head * a.S_stride * DH;
    // rows by position: the rows of K, or the rows of the newest positions (tiled layout)
    uint16_t* rows = TILED ? reinterpret_cast<uint16_t*>(a.Kt) + (size_t)head * (8 * DH) - (size_t)((S - 1) & ~7) * DH : K_head;
    *reinterpret_cast<uint4*>(reinterpret_cast<uint16_t*>(a.V) + ((size_t)head * a.S_stride + (S - 1)) * DH + j0) = vc;
    if (!TILED || (S & 7) != 0) *reinterpret_cast<uint4*>(rows + (size_t)(S - 1) * DH + j0) = kc;
    if ((S & 7) == 0) {
      uint4 r[8], w[8];
#pragma unroll
      for (int e = 0; e < 7; ++e) r[e] = *reinterpret_cast<const uint4*>(rows + (size_t)(S - 8 + e) * DH + j0);
      r[7] = kc;
      transpose_piece(r, w);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        uint16_t* dst = TILED ? K_head + (size_t)(S - 8) * DH + (size_t)(j0 + e) * 8
                              : reinterpret_cast<uint16_t*>(a.Kt) + ((size_t)head * DH + j0 + e) * a.S_stride + (S - 8);
        const u32x4 c = {w[e].x, w[e].y, w[e].z, w[e].w};
        __builtin_nontemporal_store(c, reinterpret_cast<u32x4*>(dst));
      }
    }
    float f[8];
    unpack8<T>(vc, f);
#pragma unroll
    for (int e = 0; e < 8; ++e) {         // the mean of no rows is ignored
      if (S == 1) m[e] = 0.0f;
      m[e] += (f[e] - m[e]) * (1.0f / (float)S);
    }
  }
#pragma unroll
  for (int e = 0; e < 8; e += 4) *reinterpret_cast<float4*>(a.v_mean_next + at + e) = make_float4(m[e], m[e + 1], m[e + 2], m[e + 3]);
}

// ------------------------------------------------------------------------------------------------
// Step 2a: the kq positions with the largest keys (ties to the lower position)

struct SelectLds {
  uint32_t* hist;   // [2][kRadixBins] double-buffered digit histograms (swizzled slots)
  uint32_t* wcnt;   // [NW] wave totals of the compaction scan
  int* ctl;         // [8]
  float* red;       // [4 * NW]: the callers' maxima of the waves, then select_compact's sums ([30..31]: select_channels' until then)
};

// Exclusive prefix sum of v over the workgroup in thread order; *total gets the sum.
// One barrier; `wsum`: NW words.
__device__ __forceinline__ uint32_t block_scan_excl(uint32_t v, uint32_t* wsum, int lane, int wave,
                                                    uint32_t* total) {
  const uint32_t incl = wave_scan_incl(v);
  if (lane == kWave - 1) wsum[wave] = incl;
  __syncthreads();
  uint32_t before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const uint32_t t = wsum[w];
    if (w < wave) before += t;
    all += t;
  }
  *total = all;
  return before + incl - v;
}

// the largest of one value per wave
__device__ __forceinline__ float wave_values_max(const float* v) {
  float m = v[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) m = fmaxf(m, v[w]);
  return m;
}

// A thread's share of the softmax denominator, summed while the logit numerators are produced: relative to the
// largest value the thread has seen, brought to the sequence's maximum at the end.  (It starts at the lowest finite value, so
// that no maximum lies below it: a thread without positions brings 0.)
struct RunningSum {
  float ref = -3.402823466e38f, z = 0.0f;
  template <int M>
  __device__ __forceinline__ void add(const float (&d)[M], float esc) {
    float m = ref;
#pragma unroll
    for (int e = 0; e < M; ++e) m = fmaxf(m, d[e]);
    z *= exp2_weight((ref - m) * esc);
#pragma unroll
    for (int e = 0; e < M; ++e) z += exp2_weight((d[e] - m) * esc);
    ref = m;
  }
  __device__ __forceinline__ float relative_to(float dmax, float esc) const { return z * exp2_weight((ref - dmax) * esc); }
};

// What select_compact adds up beside the list.
enum class Sums {
  kNone,        // nothing
  kNumerator,   // alpha's numerator, sum over the selected of exp((d - dmax) / tau); the threads bring the denominator
  kBoth         // the numerator and the denominator, sum over all keys
};

// What alpha is made of beside the waves' sums in red[NW ..] (selected_mass() and all_mass()).
struct Selection {
  uint32_t first;   // the threshold: its decided bits, the others 0
  int need;         // how many of the keys that share them are taken
  bool whole;       // all of them
};
__device__ __forceinline__ float all_mass(const float* red) {
  float t = 0.0f;
#pragma unroll
  for (int w = 0; w < NW; ++w) t += red[NW + w];
  return t;
}
__device__ __forceinline__ float selected_mass(const Selection& s, const float* red, float dmax, float esc) {
  float t = 0.0f, e = 0.0f;
#pragma unroll
  for (int w = 0; w < NW; ++w) { t += red[2 * NW + w]; e += red[3 * NW + w]; }
  // Which of the equal keys are taken does not matter for the sum: either all of them are, or all 32 bits are decided and
  // they share one weight.
  return t + (s.whole ? e : (float)s.need * exp2_weight((key_to_float(s.first) - dmax) * esc));
}
// alpha's numerator and denominator are summed in different orders (and launches): a share is at most 1, and 1 where everything
// is selected (but not a number where they are none)
__device__ __forceinline__ float as_share(float alpha, bool everything) {
  return alpha > 1.0f || (everything && alpha == alpha) ? 1.0f : alpha;
}

// Step 2a as a whole: the k_old positions of largest key among keys[0..S_old) (ties to the lower position) and all
// positions S_old .. S-1 (the local window), ascending, into list[0 .. k_old + S - S_old).
// On entry hist[0] holds the counts of the first digit of keys[0..S_old), hist[1] is zero, and a barrier lies behind
// them.  Digits of 11, 11 and 10 bits from the top.  The threshold's first digit comes from hist[0]; then every lane
// keeps two bit masks of its keys, "above the bin" and "in the bin".  What follows concerns the keys in the bin only: they are
// counted by their next digit, one wave finds the threshold among them, and the masks are formed again, until the remaining
// bin is taken whole (with distinct keys: after the second digit as a rule).  A lane owns consecutive positions, so lane order
// is position order and one workgroup scan of the packed (above, in) counts orders the list, whatever the length (ties: the
// first `need` keys of the bin by position).
// Bound by vector instructions where workgroups share a CU, by the latency of one wave's instructions and of LDS where they
// do not.  Up to 8 keys per lane (S <= 8 NT) stay in registers and every step is straight code; beyond that a lane keeps the
// masks and reads the few keys that they name again.  Measured for the whole selection of one head at 1024 positions and at
// 3982: 3.0 and 3.5 us with the second form for every length and alpha summed here, 2.3 and 3.1.
// `list` may be the key array itself: it overwrites it from the front, a write never lands beyond the position it
// records, and all reads of keys precede the scan's barrier.  With key_out (receives the key of the n-th entry) the keys
// are read again after it: list must then be another array.  Entries of list / idx_out are offset by pos_base.
// esc = log2(e) / tau; zs = the calling thread's share of the denominator (kNumerator); dmax() = the largest logit numerator,
// called by every thread once the threshold is known.
// Ends with a barrier that also publishes the list and the waves' sums.
// found() is called when the threshold is known (a time stamp of a profiling build).
//
// The passes over the keys of the threshold's bin, for both forms: count(hist, shift, mask, heavy) counts the keys in the bin
// by a digit, narrow() forms the masks anew for keys above `last` and from `first` to `last`.
struct Bin {
  uint32_t first = 0xffffffffu, last = 0xffffffffu;       // keys that share the decided bits lie in first .. last
  int need, size;
};
__device__ __forceinline__ Bin first_bin(int k_old, const SelectLds& sl, int lane, int wave) {
  Bin b;
  b.need = b.size = k_old;
  if (k_old > 0) {                                        // (0: everything comes from the window)
    if (wave == 0) find_threshold_bin(sl.hist, k_old, lane, sl.ctl);
    __syncthreads();
    b.first = (uint32_t)sl.ctl[0] << 21; b.last = b.first | 0x1fffffu;
    b.need = sl.ctl[1]; b.size = sl.ctl[2];
  }
  return b;
}
template <class Count, class Narrow>
__device__ __forceinline__ void next_bins(Bin& b, const SelectLds& sl, int tid, int lane, int wave, Count&& count, Narrow&& narrow) {
  for (int pass = 1; pass < 3 && b.need != b.size; ++pass) {
    const int shift = pass == 1 ? 10 : 0;
    const uint32_t dmask = pass == 1 ? 0x7ffu : 0x3ffu;
    uint32_t* hist = sl.hist + (pass & 1) * kRadixBins;
    if (__builtin_expect(pass == 2, 0)) {                                      // hist[0] has served the first digit
      for (int i = tid; i < kRadixBins; i += NT) hist[i] = 0u;
      __syncthreads();
    }
    // heavy: thousands of keys share the decided bits (duplicated keys, underflowed scores): they may share the next digit
    // too, and plain atomics on one address would take microseconds; count per wave first
    count(hist, shift, dmask, b.size > kTieHeavy);
    __syncthreads();
    if (wave == 0) find_threshold_bin(hist, b.need, lane, sl.ctl);
    __syncthreads();
    b.first |= (uint32_t)sl.ctl[0] << shift; b.last = b.first | ((1u << shift) - 1u);
    b.need = sl.ctl[1]; b.size = sl.ctl[2];
    narrow();
  }
}

// a lane's sums and (above, in) counts -> its place in the list; the scan's barrier publishes the waves' sums too
template <Sums SUMS>
__device__ __forceinline__ Selection place_of(const Bin& b, uint32_t n_gt, uint32_t n_eq, float z, float asum, float esum,
                                              const SelectLds& sl, int lane, int wave, uint32_t& o, int& room) {
  if (SUMS != Sums::kNone) {
    z = wave_sum(z); asum = wave_sum(asum); esum = wave_sum(esum);
    if (lane == 0) { sl.red[NW + wave] = z; sl.red[2 * NW + wave] = asum; sl.red[3 * NW + wave] = esum; }
  }
  uint32_t total;
  const uint32_t ex = block_scan_excl(n_gt | (n_eq << 16), sl.wcnt, lane, wave, &total);
  const uint32_t eq_before = ex >> 16;
  o = (ex & 0xffffu) + (eq_before < (uint32_t)b.need ? eq_before : (uint32_t)b.need);
  room = b.need - (int)eq_before;                         // keys of the bin still to be taken from this lane on
  return Selection{b.first, b.need, (uint32_t)b.need >= (total >> 16)};
}

// M = 4 or 8 keys per lane, in registers
template <Sums SUMS, int M, class Max, class Found>
__device__ __forceinline__ Selection select_compact_regs(const uint32_t* keys, uint32_t* list, int S, int S_old, int k_old, Max&& dmax_of,
                                                         float esc, const RunningSum& zs, int32_t* idx_out, int idx_stride, const SelectLds& sl,
                                                         int tid, int lane, int wave, uint32_t* key_out, int pos_base, Found&& found) {
  const int own = tid * M;
  uint32_t kx[M] = {};
  if (own < S) {
#pragma unroll
    for (int i = 0; i < M; i += 4) {
      const uint4 v = *reinterpret_cast<const uint4*>(keys + own + i);
      kx[i] = v.x; kx[i + 1] = v.y; kx[i + 2] = v.z; kx[i + 3] = v.w;
    }
  }
  auto below = [&](int end) -> uint32_t { const int n = end - own; return n >= M ? (1u << M) - 1u : (n <= 0 ? 0u : (1u << n) - 1u); };
  const uint32_t all_mask = below(S), old_mask = below(S_old);
  Bin b = first_bin(k_old, sl, lane, wave);
  uint32_t gt, eq;
  auto narrow = [&]() {
    uint32_t g = 0, ge = 0;
#pragma unroll
    for (int e = M - 1; e >= 0; --e) {
      g = g + g + (kx[e] > b.last ? 1u : 0u);
      ge = ge + ge + (kx[e] >= b.first ? 1u : 0u);
    }
    eq = ge & ~g & old_mask;
    gt = (g & old_mask) | (all_mask & ~old_mask);
  };
  narrow();
  next_bins(b, sl, tid, lane, wave, [&](uint32_t* hist, int shift, uint32_t dmask, bool heavy) {
    if (__builtin_expect(!heavy, 1)) {
#pragma unroll
      for (int e = 0; e < M; ++e)
        if ((eq >> e) & 1u) atomicAdd(&hist[hist_slot((kx[e] >> shift) & dmask)], 1u);
    } else {
#pragma unroll
      for (int e = 0; e < M; ++e) hist_add_ties(hist, (kx[e] >> shift) & dmask, (eq >> e) & 1u, lane);
    }
  }, narrow);
  found();
  float z = 0.0f, asum = 0.0f, esum = 0.0f;
  if (SUMS != Sums::kNone) {
    const float dmax = dmax_of();
    if (SUMS == Sums::kNumerator) z = zs.relative_to(dmax, esc);
#pragma unroll
    for (int e = 0; e < M; ++e) {
      const float w = exp2_weight((key_to_float(kx[e]) - dmax) * esc);
      asum += (gt >> e) & 1u ? w : 0.0f;
      esum += (eq >> e) & 1u ? w : 0.0f;
      if (SUMS == Sums::kBoth) z += (all_mask >> e) & 1u ? w : 0.0f;
    }
  }
  uint32_t o;
  int room;
  const Selection s = place_of<SUMS>(b, __popc(gt), __popc(eq), z, asum, esum, sl, lane, wave, o, room);
  uint32_t take = gt;
  for (uint32_t t = eq; t && room > 0; --room, t &= t - 1) take |= t & (0u - t);
  for (; take; take &= take - 1) {
    const int e = __ffs(take) - 1, at = own + e;
    list[o] = (uint32_t)(pos_base + at);
    if (key_out) key_out[o] = keys[at];
    if (idx_out && (int)o < idx_stride) idx_out[o] = pos_base + at;
    ++o;
  }
  __syncthreads();
  return s;
}

// kOwnWords: bit masks of each kind per lane, for up to 32 NT kOwnWords positions.
template <Sums SUMS, int kOwnWords, class Max, class Found>
__device__ __forceinline__ Selection select_compact_words(const uint32_t* keys, uint32_t* list, int S, int S_old, int k_old, Max&& dmax_of,
                                                          float esc, const RunningSum& zs, int32_t* idx_out, int idx_stride,
                                                          const SelectLds& sl, int tid, int lane, int wave, uint32_t* key_out, int pos_base,
                                                          Found&& found) {
  Bin b = first_bin(k_old, sl, lane, wave);
  // this lane's positions: granules of 8, dealt out evenly, in order
  constexpr int gran = 8;
  const int n_gran = (S + gran - 1) / gran, per = n_gran / NT, rem = n_gran - per * NT;
  const int own = (tid * per + (tid < rem ? tid : rem)) * gran, n_own = (per + (tid < rem ? 1 : 0)) * gran;
  uint32_t gt[kOwnWords], eq[kOwnWords];                  // bit i of word w: position own + 32 w + i
  float z = 0.0f, dmax = 0.0f;
  if (SUMS == Sums::kBoth) dmax = dmax_of();
#pragma unroll
  for (int w = 0; w < kOwnWords; ++w) {
    gt[w] = eq[w] = 0;
    const int at = own + 32 * w;
    if (32 * w < n_own) {
      const int old_here = S_old - at, all_here = S - at < n_own - 32 * w ? S - at : n_own - 32 * w;   // of this lane's own
      const uint32_t old_mask = old_here >= 32 ? ~0u : (old_here <= 0 ? 0u : (1u << old_here) - 1u);
      const uint32_t all_mask = all_here >= 32 ? ~0u : (all_here <= 0 ? 0u : (1u << all_here) - 1u);
      uint32_t g = 0, ge = 0;
#pragma unroll
      for (int i = 7; i >= 0; --i) {
        if (32 * w + 4 * i < n_own) {
          const uint4 v = *reinterpret_cast<const uint4*>(keys + at + 4 * i);
          const uint32_t kx[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
          for (int e = 3; e >= 0; --e) {
            g = g + g + (kx[e] > b.last ? 1u : 0u);
            ge = ge + ge + (kx[e] >= b.first ? 1u : 0u);
            if (SUMS == Sums::kBoth) z += 4 * i + e < all_here ? exp2_weight((key_to_float(kx[e]) - dmax) * esc) : 0.0f;
          }
        }
      }
      eq[w] = ge & ~g & old_mask;
      gt[w] = (g & old_mask) | (all_mask & ~old_mask);
    }
  }
  auto each = [&](uint32_t (&bits)[kOwnWords], auto&& f) {      // f(word, bit, position) for every set bit
#pragma unroll
    for (int w = 0; w < kOwnWords; ++w)
      for (uint32_t t = bits[w]; t; t &= t - 1) f(w, t & (0u - t), own + 32 * w + __ffs(t) - 1);
  };
  next_bins(b, sl, tid, lane, wave, [&](uint32_t* hist, int shift, uint32_t dmask, bool heavy) {
    if (__builtin_expect(!heavy, 1)) {
      each(eq, [&](int, uint32_t, int at) { atomicAdd(&hist[hist_slot((keys[at] >> shift) & dmask)], 1u); });
    } else {
#pragma unroll
      for (int w = 0; w < kOwnWords; ++w)
        for (int i = 0; i < 32; ++i) {
          const bool on = (eq[w] >> i) & 1u;
          if (__ballot(on) == 0) continue;
          hist_add_ties(hist, (keys[on ? own + 32 * w + i : 0] >> shift) & dmask, on, lane);
        }
    }
  }, [&]() {
    each(eq, [&](int w, uint32_t bit, int at) {
      const uint32_t key = keys[at];
      if (key < b.first || key > b.last) eq[w] &= ~bit;
      if (key > b.last) gt[w] |= bit;
    });
  });
  found();
  float asum = 0.0f, esum = 0.0f;
  if (SUMS != Sums::kNone) {
    if (SUMS == Sums::kNumerator) { dmax = dmax_of(); z = zs.relative_to(dmax, esc); }
    each(gt, [&](int, uint32_t, int at) { asum += exp2_weight((key_to_float(keys[at]) - dmax) * esc); });
    each(eq, [&](int, uint32_t, int at) { esum += exp2_weight((key_to_float(keys[at]) - dmax) * esc); });
  }
  uint32_t n_gt = 0, n_eq = 0;
#pragma unroll
  for (int w = 0; w < kOwnWords; ++w) { n_gt += __popc(gt[w]); n_eq += __popc(eq[w]); }
  uint32_t o;
  int room;
  const Selection s = place_of<SUMS>(b, n_gt, n_eq, z, asum, esum, sl, lane, wave, o, room);
#pragma unroll
  for (int w = 0; w < kOwnWords; ++w) {
    uint32_t take = gt[w];
    for (uint32_t t = eq[w]; t && room > 0; --room, t &= t - 1) take |= t & (0u - t);
    for (; take; take &= take - 1) {
      const int at = own + 32 * w + __ffs(take) - 1;
      list[o] = (uint32_t)(pos_base + at);
      if (key_out) key_out[o] = keys[at];
      if (idx_out && (int)o < idx_stride) idx_out[o] = pos_base + at;
      ++o;
    }
  }
  __syncthreads();
  return s;
}

template <Sums SUMS, class Max, class Found = Nothing>
__device__ __forceinline__ Selection select_compact(const uint32_t* keys, uint32_t* list, int S, int S_old, int k_old, Max&& dmax_of, float esc,
                                                    const RunningSum& zs, int32_t* idx_out, int idx_stride, const SelectLds& sl, int tid,
                                                    int lane, int wave, uint32_t* key_out = nullptr, int pos_base = 0, Found&& found = Found{}) {
  if (S <= 4 * NT)
    return select_compact_regs<SUMS, 4>(keys, list, S, S_old, k_old, dmax_of, esc, zs, idx_out, idx_stride, sl, tid, lane, wave, key_out, pos_base, found);
  if (S <= 8 * NT)
    return select_compact_regs<SUMS, 8>(keys, list, S, S_old, k_old, dmax_of, esc, zs, idx_out, idx_stride, sl, tid, lane, wave, key_out, pos_base, found);
  if (S <= 32 * NT)
    return select_compact_words<SUMS, 1>(keys, list, S, S_old, k_old, dmax_of, esc, zs, idx_out, idx_stride, sl, tid, lane, wave, key_out, pos_base, found);
  return select_compact_words<SUMS, 3>(keys, list, S, S_old, k_old, dmax_of, esc, zs, idx_out, idx_stride, sl, tid, lane, wave, key_out, pos_base,
                                       found);      // LDS ends at about 40 000 keys
}

// ------------------------------------------------------------------------------------------------
// Step 2b: exact softmax attention over gathered rows (Eq. 8), online softmax in the exp2 domain

template <int DH>
struct RowGeometry {
  static constexpr int LPR = DH / 8;          // lanes per row (16 bytes each)
  static constexpr int RPW = kWave / LPR;     // rows per wave per load
  static constexpr int RPI = NW * RPW;        // rows per workgroup per load
  static constexpr int UNR = 4;
  static constexpr int GROUP = RPI * UNR;     // rows the workgroup covers per group of loads
};

// Rows list[n_begin..n_end) of K and V (K_head / V_head already offset by the lane's 16-byte column
// slice `sub`).  LPR lanes share a row, K and V rows are issued together, groups of UNR loads run
// through a two-deep software pipeline.  q8 = the lane's 8 query components times log2(e)/sqrt(d_h).
// Accumulates into (m_run, l_run, acc).  No barrier.
// TILED: the keys come from the tiled single-copy layout instead: K_head is the head's first tile (tiles of
// 8 positions, channel-major inside a tile: element (position p, channel j) at ((p / 8) d_h + j) 8 + p % 8),
// so a lane's 8 channels of one position are eight 2-byte loads 16 bytes apart; positions from tiled_below on
// (the up to 7 newest, not yet in a tile) are rows of K_stage (row p - tiled_below, already offset by `sub`).
// requested() is called by whole waves once the first group of loads is under way.
template <class T, int DH, bool TILED = false, bool KEEP = false, class Requested = Nothing>
__device__ __forceinline__ void attend_rows(const char* K_head, const char* V_head, const int* list, int n_begin,
                                            int n_end, const float (&q8)[8], int lane, int wave, float& m_run,
                                            float& l_run, float (&acc)[8], Requested&& requested = Requested{},
                                            const char* K_stage = nullptr, int tiled_below = 0) {
  using G = RowGeometry<DH>;
  const int slot = wave * G::RPW + lane / G::LPR;
  const int n_groups = (n_end - n_begin + G::GROUP - 1) / G::GROUP;
  auto issue = [&](uint4 (&kr)[G::UNR], uint4 (&vr)[G::UNR], int g) {
#pragma unroll
    for (int t = 0; t < G::UNR; ++t) {
      const int n = n_begin + g * G::GROUP + t * G::RPI + slot;
      const int p = list[n < n_end ? n : n_end - 1];
      const uint32_t off = (uint32_t)p * (uint32_t)(DH * 2);   // < S_max * 512 bytes
      if (!TILED) {
        kr[t] = load16_as<uint4, KEEP>(K_head + off);
      } else if (p >= tiled_below) {
        kr[t] = load16(K_stage + (uint32_t)(p - tiled_below) * (uint32_t)(DH * 2));
      } else {
        const uint16_t* tp = reinterpret_cast<const uint16_t*>(K_head) +
                             ((size_t)(p >> 3) * DH + (lane % G::LPR) * 8) * 8 + (p & 7);
        const uint32_t c0 = tp[0], c1 = tp[8], c2 = tp[16], c3 = tp[24], c4 = tp[32], c5 = tp[40], c6 = tp[48], c7 = tp[56];
        kr[t] = make_uint4(c0 | (c1 << 16), c2 | (c3 << 16), c4 | (c5 << 16), c6 | (c7 << 16));
      }
      vr[t] = load16_as<uint4, KEEP>(V_head + off);
    }
  };
  // The rows of a group are weighted against one maximum: one rescaling of the sums for UNR rows.  (One per row: 512 heads of
  // 4096 positions, two workgroups per CU and bound by vector instructions, 51.5 us per step, so 50.7.)
  auto consume = [&](const uint4 (&kr)[G::UNR], const uint4 (&vr)[G::UNR], int g) {
    const int n0 = n_begin + g * G::GROUP + slot;          // row t of the lane is n0 + t RPI
    float dot[G::UNR], m_new = m_run;
#pragma unroll
    for (int t = 0; t < G::UNR; ++t) {
      float f[8];
      unpack8<T>(kr[t], f);
      dot[t] = 0.0f;
#pragma unroll
      for (int e = 0; e < 8; ++e) dot[t] = fmaf(f[e], q8[e], dot[t]);
    }
#pragma unroll
    for (int t = 0; t < G::UNR; ++t) {
      dot[t] = lanes_sum<G::LPR>(dot[t]);
      m_new = n0 + t * G::RPI < n_end ? fmaxf(m_new, dot[t]) : m_new;
    }
    if (n0 < n_end) {
      const float sc = exp2_weight(m_run - m_new);
      l_run *= sc;
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] *= sc;
#pragma unroll
      for (int t = 0; t < G::UNR; ++t) {
        if (n0 + t * G::RPI < n_end) {
          const float pr = exp2_weight(dot[t] - m_new);
          float f[8];
          unpack8<T>(vr[t], f);
          l_run += pr;
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[e] = fmaf(pr, f[e], acc[e]);
        }
      }
      m_run = m_new;
    }
  };
  if (n_groups > 0) {
    uint4 ka[G::UNR], va[G::UNR], kb[G::UNR], vb[G::UNR];
    issue(ka, va, 0);
    requested();
    int g = 0;
    for (; g + 2 < n_groups; g += 2) {
      issue(kb, vb, g + 1);
      consume(ka, va, g);
      issue(ka, va, g + 2);
      consume(kb, vb, g + 1);
    }
    if (g + 1 < n_groups) {
      issue(kb, vb, g + 1);
      consume(ka, va, g);
      consume(kb, vb, g + 1);
    } else {
      consume(ka, va, g);
    }
  } else {
    requested();
  }
}

// Step 1b from the row-major keys: rows 0..S-1 of one KV head (or of a span), LPR lanes per row as in the gather of
// Step 2, groups of UNR loads through a two-deep software pipeline.  finish(position, dot) is called by
// the first lane of each row's lane group.  qm8 = the lane's 8 masked query components.
template <class T, int DH, class Finish>
__device__ __forceinline__ void stream_key_rows(const char* K_head_sub, int S, const float (&qm8)[8], int lane, int wave,
                                                Finish&& finish) {
  using G = RowGeometry<DH>;
  constexpr int UNR = 8, GROUP = G::RPI * UNR;
  const int slot = wave * G::RPW + lane / G::LPR;
  const bool first = lane % G::LPR == 0;
  const int n_groups = (S + GROUP - 1) / GROUP;
  auto issue = [&](uint4 (&kr)[UNR], int g) {
#pragma unroll
    for (int t = 0; t < UNR; ++t) {
      const int n = g * GROUP + t * G::RPI + slot;
      kr[t] = load16(K_head_sub + (size_t)(n < S ? n : S - 1) * (DH * 2));
    }
  };
  auto consume = [&](const uint4 (&kr)[UNR], int g) {
#pragma unroll
    for (int t = 0; t < UNR; ++t) {
      const int n = g * GROUP + t * G::RPI + slot;
      float f[8];
      unpack8<T>(kr[t], f);
      float dot = 0.0f;
#pragma unroll
      for (int e = 0; e < 8; ++e) dot = fmaf(f[e], qm8[e], dot);
      dot = lanes_sum<G::LPR>(dot);
      if (first && n < S) finish(n, dot);
    }
  };
  if (n_groups > 0) {
    uint4 ka[UNR], kb[UNR];
    issue(ka, 0);
    int g = 0;
    for (; g + 2 < n_groups; g += 2) {
      issue(kb, g + 1);
      consume(ka, g);
      issue(ka, g + 2);
      consume(kb, g + 1);
    }
    if (g + 1 < n_groups) {
      issue(kb, g + 1);
      consume(ka, g);
      consume(kb, g + 1);
    } else {
      consume(ka, g);
    }
  }
}

// One more row, given as 16-bit codes in LDS (the row a decode step appends), folded into the state of
// the lane group with slot 0.  Executed by all lanes; no barrier.
template <class T, int DH>
__device__ __forceinline__ void attend_row_from_codes(const uint16_t* krow, const uint16_t* vrow, const float (&q8)[8],
                                                      int lane, int wave, float& m_run, float& l_run, float (&acc)[8]) {
  using G = RowGeometry<DH>;
  const int sub = lane % G::LPR;
  float f[8];
  unpack8<T>(*reinterpret_cast<const uint4*>(krow + sub * 8), f);
  float dot = 0.0f;
#pragma unroll
  for (int e = 0; e < 8; ++e) dot = fmaf(f[e], q8[e], dot);
  dot = lanes_sum<G::LPR>(dot);
  if (wave == 0 && lane < G::LPR) {
    const float m_new = fmaxf(m_run, dot);
    const float sc = exp2_weight(m_run - m_new), pr = exp2_weight(dot - m_new);
    unpack8<T>(*reinterpret_cast<const uint4*>(vrow + sub * 8), f);
    l_run = l_run * sc + pr;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = acc[e] * sc + pr * f[e];
    m_run = m_new;
  }
}

// Merge the lane groups of a wave (butterfly over the group index) and store the wave's partial
// (acc[DH], m, l) to part[wave][DH + 2].  The caller puts a barrier after it.
template <int DH>
__device__ __forceinline__ void store_wave_partial(float m_run, float l_run, float (&acc)[8], float* part, int lane, int wave) {
  using G = RowGeometry<DH>;
  auto merge = [&](auto step) {
    constexpr int O = decltype(step)::value;
    float ma, mb, la, lb;
    lane_pair<O>(m_run, ma, mb);
    lane_pair<O>(l_run, la, lb);
    m_run = fmaxf(ma, mb);
    const float sa = weight_exp2(ma, m_run), sb = weight_exp2(mb, m_run);
    l_run = la * sa + lb * sb;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float a, b;
      lane_pair<O>(acc[e], a, b);
      acc[e] = a * sa + b * sb;
    }
  };
  if (G::LPR <= 8) merge(std::integral_constant<int, 8>{});
  if (G::LPR <= 16) merge(std::integral_constant<int, 16>{});
  merge(std::integral_constant<int, 32>{});
  float* mine = part + wave * (DH + 2);
  if (lane < G::LPR) {
#pragma unroll
    for (int e = 0; e < 8; ++e) mine[lane * 8 + e] = acc[e];
    if (lane == 0) { mine[DH] = m_run; mine[DH + 1] = l_run; }
  }
}

// Channel c of the merge of n_parts partials laid out [n_parts][DH + 2]: running max, denominator and
// un-normalised numerator (each partial's numerator and denominator are relative to its own max).
template <int DH>
__device__ __forceinline__ void combine_partials(const float* parts, int n_parts, int c, float& m_all, float& l_all, float& y) {
  m_all = -INFINITY;
  for (int w = 0; w < n_parts; ++w) m_all = fmaxf(m_all, parts[w * (DH + 2) + DH]);
  l_all = 0.0f; y = 0.0f;
  for (int w = 0; w < n_parts; ++w) {
    const float s = weight_exp2(parts[w * (DH + 2) + DH], m_all);
    l_all += parts[w * (DH + 2) + DH + 1] * s;
    y += parts[w * (DH + 2) + c] * s;
  }
}

}  // inline namespace
}  // namespace sparq
