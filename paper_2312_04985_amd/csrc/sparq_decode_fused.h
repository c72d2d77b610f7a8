// SparQ decode, one workgroup per (sequence, query head): Section 4, Steps 1-3, in one launch with
// no intermediate HBM traffic.
//   stage 0  top-r of |q| and the temperature (Eq. 9)
//   stage 1  stream the r selected rows of the S-contiguous key copy; the fp32 approximate logit
//            numerators of all cached positions stay in LDS as order-preserving integer keys and are
//            counted into the first radix histogram as they are produced
//   stage 2  radix select of the k-th largest key, ordered compaction of the selected positions
//            (ties to the lower position), alpha = selected share of the approximate softmax mass
//   stage 3  gather the selected K and V rows, online-softmax exact attention, blend with the
//            mean value vector (Eq. 10), round and store
#pragma once
#include "decode_stages.h"

namespace sparq {
inline namespace SPARQ_STAGES {

// A SPARQ_STAGE_CLOCKS build (a second library for profiling, never the default one) keeps nine time stamps per
// workgroup in scalar registers and stores them when the workgroup ends; otherwise the macro is empty.
#ifdef SPARQ_STAGE_CLOCKS
#define SPARQ_STAMP(i) stamp[i] = wall_clock64()
#else
#define SPARQ_STAMP(i) do {} while (0)
#endif


struct Lds {
  uint32_t* keys;   // [S_max]   stage 1-2: keys; after compaction: selected positions
  SelectLds sel;
  QueryLds qry;
  float* part;      // [NW * (DH + 2)] stage-3 partials
  float* mean;      // [DH] the mean value vector, parked until the blend
  uint16_t* knew;   // [DH] codes of the key row being appended (one-launch step only)
  uint16_t* vnew;   // [DH]
};

template <int DH>
__device__ __forceinline__ Lds carve(uint32_t* base, int S_max) {
  Lds l;
  l.keys = base; base += S_max;
  l.sel.hist = base; base += 2 * kRadixBins;
  l.part = reinterpret_cast<float*>(base); base += NW * (DH + 2);
  l.qry.qf = reinterpret_cast<float*>(base); base += DH;
  l.qry.qs = reinterpret_cast<float*>(base); base += DH;
  l.qry.chan = reinterpret_cast<int*>(base); base += DH;
  l.mean = reinterpret_cast<float*>(base); base += DH;
  l.sel.red = reinterpret_cast<float*>(base); base += 32;
  l.sel.wcnt = base; base += 16;
  l.sel.ctl = reinterpret_cast<int*>(base); base += 8;
  l.knew = reinterpret_cast<uint16_t*>(base); base += DH / 2;
  l.vnew = reinterpret_cast<uint16_t*>(base);
  return l;
}

// The arguments in front of the first loads, requested at once.  A helped workgroup's place in the grid may be no unit's, and the
// compiler moves every request that it can behind that branch: four round trips for arguments, one after the other, where the other
// builds have one or two.  us per step with the caches in L2, as it was / so / without helpers: one head at 1500 positions 9.65 / 9.43 / 9.34, at
// 2000 11.0 / 10.7 / 10.7; 32 heads at 1500 10.3 / 10.0 / 9.9.  (The append's inputs among them: 256 channels 1.5 % faster, 64 and 128 1 %
// slower, which is how the code comes to lie.)
template <int DH>
__device__ __forceinline__ void request_arguments(const DecodeArgs& a) {
  asm volatile("" :: "s"(a.seq_lens), "s"(a.q), "s"(a.B), "s"(a.H), "s"(a.H_kv), "s"(a.S_max), "s"(a.flags), "s"(a.per_xcd), "s"(a.by_xcd.mul),
               "s"(a.by_xcd.shift), "s"(a.by_H.mul), "s"(a.by_H.shift), "s"(a.by_group.mul), "s"(a.by_group.shift));
  if (DH == 256) asm volatile("" :: "s"(a.v_mean), "s"(a.k_new), "s"(a.v_new));
}

// APPEND = true is the one-launch decode step: the new key/value row of every KV head (k_new, v_new)
// counts as position S_b of its sequence without being read back from the cache.  Every workgroup
// takes that row from the inputs; the workgroup of the first query head of a KV group, or (APART) workgroups of the append's own
// behind the decoding ones, also write it into K, V and Kt and store the updated mean; lengths and means go to
// the *_next buffers, so no workgroup can observe another one's update of the state it reads.
// TILED = true reads the single-copy tiled key layout (flag bit 6): a.K holds tiles of 8 positions, channel-major
// inside a tile, a.Kt the up to 7 newest rows of every KV head (8 rows of d_h each) that do not fill a tile yet.
// Step 1b then strides through the tiles (16 bytes per position chunk and channel), Step 2b collects a row's
// components from its tile, and the append writes a row of the small buffer, or a whole tile with the eighth row.
// RUNS = true reads the channel rows in runs (stream_channel_rows).
// HELP = true is for few units: every unit has a.helpers more workgroups on its XCD, on CUs that would be idle, which write
// nothing.  Bound is what a CU can have on its way from beyond its L2 (60 GB/s; from L2 160): a helper goes through Step 1 as
// well, in another order of the channel rows, so that each brings a part of them into the L2 that all share, and once
// the threshold's first digit is known it touches its part of the rows of K and V that are or may be selected, while the unit's
// own workgroup still orders its list.  Nobody waits for a helper, and what it does cannot be seen but in time.
// Blocks that ordinary calls skip are marked (__builtin_expect, here and in the stages), so that the compiler moves them behind the
// code that runs: where few workgroups wait for instructions, jumping over them costs: the step of one head at 1023 positions 9.83 us, so
// 9.42; of 32 heads at 1500 12.3 / 11.9; 512 heads and more equal.
template <class T, int DH, bool APPEND, bool TILED, bool HELP, bool APART, bool RUNS>
__global__ __launch_bounds__(NT, 4) void sparq_decode_fused(const DecodeArgs a) {
  extern __shared__ __align__(16) uint32_t smem[];
  const Lds L = carve<DH>(smem, a.S_max);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int U = a.B * a.H;
  int u = blockIdx.x;
  int share = 0;                           // 0: the unit's own workgroup, 1 .. helpers: one that fetches for it
  if (HELP) {
    request_arguments<DH>(a);
    const int slot = u >> 3;
    share = divided(slot, a.by_xcd);
    u = (u & 7) * a.per_xcd + (slot - share * a.per_xcd);
    if (u >= U) return;
  } else if (APART && __builtin_expect(u >= U, 0)) {
    append_heads<T, DH, TILED>(a, u - U);
    return;
  }

#ifdef SPARQ_STAGE_CLOCKS
  unsigned long long stamp[kStageStamps];
#endif
  SPARQ_STAMP(0);
  // Workgroup -> unit.  Workgroups are dealt round-robin to the 8 XCDs and started in index order.
  // Default: every XCD gets a contiguous run of units, so the query heads of a KV group share an L2.
  // With the ragged-batch hint (and no grouped heads): workgroup i serves the sequence with the
  // (i / H)-th largest length, so the longest sequences start first and the short ones fill in behind.
  if (!HELP && __builtin_expect((a.flags & 4u) && a.H == a.H_kv && a.B > 1 && a.B <= NT, 0)) {
    int* lens = reinterpret_cast<int*>(L.keys);   // free until stage 1
    if (tid < a.B) lens[tid] = a.seq_lens[tid];
    __syncthreads();
    if (tid < a.B) {
      const int mine = lens[tid];
      int rank = 0;
      for (int j = 0; j < a.B; ++j) rank += (lens[j] > mine) || (lens[j] == mine && j < tid);
      if (rank == divided(u, a.by_H)) L.sel.ctl[7] = tid;
    }
    __syncthreads();
    u = L.sel.ctl[7] * a.H + (u - divided(u, a.by_H) * a.H);
  } else if (!HELP && (U & 7) == 0) {
    u = (u & 7) * (U >> 3) + (u >> 3);
  }
  u = __builtin_amdgcn_readfirstlane(u);   // the same in every lane (also where it came through LDS): keep what follows scalar
  const int b = divided(u, a.by_H), h = u - b * a.H;
  const int hk = divided(h, a.by_group);
  const size_t kv_head = (size_t)b * a.H_kv + hk;

  // everything the unit reads from small tensors is requested here, in one round trip; the mean value
  // vector is only needed for the blend at the very end
  const LaneCodes<DH> qcode = load_lane_codes<DH>(reinterpret_cast<const uint16_t*>(a.q) + (size_t)u * DH, lane);
  uint16_t kcode = 0, vcode = 0;
  float vm = 0.0f;
  const int late = tid - (NT - DH);         // a channel for each thread of the last waves, the first to run out of chunks
  if (late >= 0) {
    vm = a.v_mean[kv_head * DH + late];
    if (APPEND) {
      kcode = reinterpret_cast<const uint16_t*>(a.k_new)[kv_head * DH + late];
      vcode = reinterpret_cast<const uint16_t*>(a.v_new)[kv_head * DH + late];
    }
  }
  for (int i = tid; i < 2 * kRadixBins; i += NT) L.sel.hist[i] = 0u;
  int S = a.seq_lens[b];
  // a length beyond the bound of this call that the buffers can hold is carried over as it is (clamped only here)
  const int S_kept = (S > a.S_max && S <= a.S_stride) ? S : -1;
  if (__builtin_expect(S < 0 || S > a.S_max, 0)) {
    if (tid == 0 && share == 0) atomicOr(a.err, 8);
    S = S < 0 ? 0 : a.S_max;
  }
  bool appended = false;                                    // this sequence takes the new row (uniform)
  const bool owner = APPEND && !APART && share == 0 && h == hk * a.group;   // writes the row and the new mean
  if (APPEND) {
    if (S + 1 <= a.S_max) { appended = true; S += 1; }
    else if (__builtin_expect(tid == 0 && share == 0, 0)) atomicOr(a.err, 1);
    if (h == 0 && tid == 0 && share == 0) a.seq_lens_next[b] = S_kept >= 0 ? S_kept : S;
  }
  int kb = a.k_per_seq ? a.k_per_seq[b] : a.k;
  kb = kb < 1 ? 1 : (kb > a.k ? a.k : kb);
  const int kq = kb < S ? kb : S;

  uint16_t* out = reinterpret_cast<uint16_t*>(a.out) + (size_t)u * DH;
  int32_t* idx_out = a.idx_out ? a.idx_out + (size_t)u * a.idx_stride : nullptr;
  if (__builtin_expect(S == 0, 0)) {   // nothing cached: defined output, raise the flag
    if (share) return;
    if (tid < DH) out[tid] = 0;
    if (tid == 0) { atomicOr(a.err, 2); if (a.alpha_out) a.alpha_out[u] = 0.0f; }
    if (a.chan_out && tid < a.r) a.chan_out[(size_t)u * a.r + tid] = -1;
    if (idx_out) for (int n = tid; n < a.idx_stride; n += NT) idx_out[n] = -1;
    if (owner && late >= 0) a.v_mean_next[kv_head * DH + late] = vm;
    return;
  }

  // ---------------- stage 0 ----------------
  select_channels<T, DH>(L.qry, qcode, a.r, L.sel.red + 30, lane, wave);
  if (HELP && __builtin_expect(share != 0, 0)) {                     // begin with another batch of rows
    const int rows = (a.r + 7) & ~7;
    int ch = 0;
    float qv = 0.0f;
    if (tid < rows) {
      int from = tid + 8 * share;
      while (from >= rows) from -= rows;
      ch = L.qry.chan[from]; qv = L.qry.qs[from];
    }
    __syncthreads();
    if (tid < rows) { L.qry.chan[tid] = ch; L.qry.qs[tid] = qv; }
    __syncthreads();
  }
  const Window win = make_window(a.local_window, S, kq);
  // the newest S mod 8 positions are not in Kt: wave w gets position S_fl + w (and S_fl + w + NW) from its K row (from the
  // inputs if it is the row being appended); loads issued behind the stream's first, used after stage 1
  // (in the one-launch step Kt is up to date for the length before this call: the group of 8 that the new
  // row may complete is written during this launch, so up to 8 positions come from rows)
  const int S_fl = ((APPEND && appended) ? S - 1 : S) & ~7, n_tail = S - S_fl, r8 = (a.r + 7) & ~7;
  // rows of K by position (two-copy layout), or the rows of the newest positions S_fl .. (tiled layout)
  const uint16_t* K_rows = TILED ? reinterpret_cast<const uint16_t*>(a.Kt) + kv_head * (size_t)(8 * DH) - (size_t)S_fl * DH
                                 : reinterpret_cast<const uint16_t*>(a.K) + kv_head * a.S_stride * (size_t)DH;
  constexpr int TAILS = (8 + NW - 1) / NW;                  // per wave: positions S_fl + wave, S_fl + wave + NW, ...
  static_assert(TAILS * NW >= 8, "every one of up to 8 positions has a wave");
  TailRow tail[TAILS];

  SPARQ_STAMP(1);
  // ---------------- stage 1 ----------------
  const uint32_t row_bytes = TILED ? 16 : (uint32_t)a.S_stride * 2;
  const char* Kt_head = TILED ? reinterpret_cast<const char*>(a.K) + kv_head * a.S_stride * (size_t)(DH * 2)
                              : reinterpret_cast<const char*>(a.Kt) + kv_head * DH * row_bytes;
  float esc;
  RunningSum zs;
  auto requested = [&]() {
    if (late >= 0) {              // (these values arrive after the query: waited for in front of the stream they cost 0.2 us)
      if (APPEND) { L.knew[late] = kcode; L.vnew[late] = vcode; }
      if (APPEND && appended) {   // same update as append_one_row; the mean of no rows is ignored
        if (S == 1) vm = 0.0f;
        vm += (T::widen(vcode) - vm) * (1.0f / (float)S);
      }
      L.mean[late] = vm;
    }
#pragma unroll
    for (int t = 0; t < TAILS; ++t) {
      const int n = wave + t * NW;
      if (n < n_tail)
        tail[t] = tail_row_issue(APPEND && appended && n == n_tail - 1 ? reinterpret_cast<const uint16_t*>(a.k_new) + kv_head * DH
                                                                       : K_rows + (size_t)(S_fl + n) * DH, L.qry.chan, r8, lane);
    }
    esc = kLog2e / temperature(L.sel.red + 30, a.flags, DH, a.r);
  };
  auto finish = [&](int c, const float (&acc)[8]) {
    uint32_t kx[8];
    if (share == 0) zs.add(acc, esc);
#pragma unroll
    for (int e = 0; e < 8; ++e) kx[e] = float_to_key(acc[e]);
    hist_add_chunk(L.sel.hist, kx, win.S_old - c * 8);
    uint4* dst = reinterpret_cast<uint4*>(L.keys + c * 8);
    dst[0] = make_uint4(kx[0], kx[1], kx[2], kx[3]);
    dst[1] = make_uint4(kx[4], kx[5], kx[6], kx[7]);
  };
  stream_channel_rows<T, NT, HELP, RUNS>(Kt_head, row_bytes, L.qry.chan, L.qry.qs, a.r, 0, S_fl >> 3, tid, finish, requested, TILED ? DH * 16u : 16u);
#pragma unroll
  for (int t = 0; t < TAILS; ++t) {
    const int n = wave + t * NW;
    if (n < n_tail) {
      const float dot = tail_row_dot<T>(tail[t], L.qry.qs, r8, lane);
      if (lane == 0) {
        zs.add({dot}, esc);
        const uint32_t key = float_to_key(dot);
        L.keys[S_fl + n] = key;
        if (S_fl + n < win.S_old) atomicAdd(&L.sel.hist[hist_slot(key >> 21)], 1u);
      }
    }
  }
  SPARQ_STAMP(2);
  const float tmax = wave_max(zs.ref);
  if (lane == 0) L.sel.red[wave] = tmax;
  __syncthreads();
  SPARQ_STAMP(3);
  auto dmax_of = [&]() { return wave_values_max(L.sel.red); };
  if (HELP && __builtin_expect(share != 0, 0)) {
    // positions share - 1, share - 1 + helpers, ...: the keys of the threshold's first digit may be taken, those above are
    const Bin bin = first_bin(win.k_old, L.sel, lane, wave);
    const bool whole = bin.size <= 2 * bin.need + NT;        // (many equal keys: only those that are certain)
    constexpr int LINES = DH * 2 / 128;                      // of a row
    const char* K_head = reinterpret_cast<const char*>(a.K) + kv_head * a.S_stride * (size_t)(DH * 2);
    const char* V_head = reinterpret_cast<const char*>(a.V) + kv_head * a.S_stride * (size_t)(DH * 2);
    uint32_t seen = 0;
    for (int p = tid * a.helpers + share - 1; p < S - 1; p += NT * a.helpers) {   // (S - 1 may be the row being appended)
      const uint32_t key = L.keys[p];
      if (p >= win.S_old || key > bin.last || (whole && key >= bin.first)) {
#pragma unroll
        for (int l = 0; l < LINES; ++l) {
          seen |= *reinterpret_cast<const uint32_t*>(K_head + (size_t)p * (DH * 2) + l * 128);
          seen |= *reinterpret_cast<const uint32_t*>(V_head + (size_t)p * (DH * 2) + l * 128);
        }
      }
    }
    asm volatile("" :: "v"(seen));
    return;
  }

  // ---------------- stage 2 ----------------
  const Selection chosen = select_compact<Sums::kNumerator>(L.keys, L.keys, S, win.S_old, win.k_old, dmax_of, esc, zs, idx_out,
                                                            a.idx_stride, L.sel, tid, lane, wave, nullptr, 0, [&]() { SPARQ_STAMP(4); });
  SPARQ_STAMP(5);
  if (idx_out && tid == 0 && kq > a.idx_stride) atomicOr(a.err, 4);
  if (idx_out) for (int n = kq + tid; n < a.idx_stride; n += NT) idx_out[n] = -1;
  if (a.chan_out && tid < a.r) a.chan_out[(size_t)u * a.r + tid] = L.qry.chan[tid];

  // ---------------- stage 3 ----------------
  using G = RowGeometry<DH>;
  const int sub = lane % G::LPR;
  const int* list = reinterpret_cast<const int*>(L.keys);
  const char* K_head = reinterpret_cast<const char*>(a.K) + kv_head * a.S_stride * (size_t)(DH * 2) + sub * 16;
  const char* V_head = reinterpret_cast<const char*>(a.V) + kv_head * a.S_stride * (size_t)(DH * 2) + sub * 16;
  const float qscale = kLog2e / sqrtf((float)DH);
  float q8[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) q8[e] = L.qry.qf[sub * 8 + e] * qscale;
  // positions are ascending, so the appended row (position S - 1) can only be the last entry; it is
  // not read back from the cache but taken from the inputs
  const bool new_selected = APPEND && appended && list[kq - 1] == S - 1;
  float alpha = 0.0f;
  auto gathering = [&]() {
    if (tid < DH) alpha = as_share(selected_mass(chosen, L.sel.red, dmax_of(), esc) / all_mass(L.sel.red), kq == S);
  };
  float m_run = -INFINITY, l_run = 0.0f;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (TILED)
    attend_rows<T, DH, true>(Kt_head, V_head, list, 0, new_selected ? kq - 1 : kq, q8, lane, wave, m_run, l_run, acc, gathering,
                             reinterpret_cast<const char*>(K_rows + (size_t)S_fl * DH) + sub * 16, S_fl);
  else
    attend_rows<T, DH, false, HELP>(K_head, V_head, list, 0, new_selected ? kq - 1 : kq, q8, lane, wave, m_run, l_run, acc, gathering);
  if (APPEND && new_selected) attend_row_from_codes<T, DH>(L.knew, L.vnew, q8, lane, wave, m_run, l_run, acc);
  SPARQ_STAMP(6);
  store_wave_partial<DH>(m_run, l_run, acc, L.part, lane, wave);
  __syncthreads();
  SPARQ_STAMP(7);
  if (tid < DH) {
    float m_all, l_all, y3;
    combine_partials<DH>(L.part, NW, tid, m_all, l_all, y3);
    y3 /= l_all;
    if (tid == 0 && a.alpha_out) a.alpha_out[u] = alpha;
    float y = y3;
    if (!(a.flags & 1u)) y = alpha * y3 + (1.0f - alpha) * L.mean[tid];
    out[tid] = T::narrow(y);
  }
  // The append's stores come last.  (Measured at five places of the kernel: in front of stage 0 they sit
  // on the critical path of every wait that follows, because a wait for a load also waits for the stores
  // issued before it; after Step 1b, after the select, after the compaction and here cost the same within
  // noise when workgroups come in several rounds, and here is best when they all run at once.)
  if (APPEND && owner && tid < DH) append_channel<DH, TILED>(a, kv_head, tid, S, appended, L.knew[tid], L.vnew[tid], L.mean[tid]);
#ifdef SPARQ_STAGE_CLOCKS
  SPARQ_STAMP(8);
  if (a.clocks && tid == 0)
    for (int i = 0; i < kStageStamps; ++i) a.clocks[(size_t)(HELP ? u : (int)blockIdx.x) * kStageStamps + i] = stamp[i];
#endif
}

// LDS bytes for a cache of S_max rows and head dimension d_h
inline size_t fused_lds_bytes(int S_max, int d_h) {
  return 4 * ((size_t)S_max + 2 * kRadixBins + (size_t)NW * (d_h + 2) + 5 * (size_t)d_h + 32 + 16 + 8);
}

// One launch of `grid` workgroups.
template <class T, int DH, bool APPEND, bool TILED, bool HELP, bool APART, bool RUNS>
hipError_t launch_fused(const DecodeArgs& a, int grid, hipStream_t s) {
  const size_t lds = fused_lds_bytes(a.S_max, DH);
  auto kern = sparq_decode_fused<T, DH, APPEND, TILED, HELP, APART, RUNS>;
  hipError_t e = allow_lds<sparq_decode_fused<T, DH, APPEND, TILED, HELP, APART, RUNS>>(lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(NT), lds, s, a);
  return hipGetLastError();
}

// ... for the cache's type and head dimension
template <bool APPEND, bool TILED, bool HELP, bool APART, bool RUNS>
hipError_t launch_fused(const DecodeArgs& a, int dtype, int grid, hipStream_t s) {
  const bool bf = dtype == 1;
  switch (a.d_h) {
    case 64:  return bf ? launch_fused<BF16, 64, APPEND, TILED, HELP, APART, RUNS>(a, grid, s) : launch_fused<F16, 64, APPEND, TILED, HELP, APART, RUNS>(a, grid, s);
    case 128: return bf ? launch_fused<BF16, 128, APPEND, TILED, HELP, APART, RUNS>(a, grid, s) : launch_fused<F16, 128, APPEND, TILED, HELP, APART, RUNS>(a, grid, s);
    case 256: return bf ? launch_fused<BF16, 256, APPEND, TILED, HELP, APART, RUNS>(a, grid, s) : launch_fused<F16, 256, APPEND, TILED, HELP, APART, RUNS>(a, grid, s);
    default:  return hipErrorInvalidValue;
  }
}

}  // inline namespace
}  // namespace sparq
