// SparQ decode for many (sequence, head) units with sequences too long for one workgroup's LDS (one 4-byte
// key per cached position does not fit beyond ~35 000 positions; few units with long caches go through the
// digit-bucket plan instead).  The top-k of a sequence is contained in the union of the top-k of
// its parts (a position beaten by fewer than k others overall is beaten by fewer than k in its own part,
// ties to the lower position in both), so the selection of Step 2 is made in two levels:
//   long_scores    (units x n_span workgroups) Step 1 on a span of span_len positions, keys in LDS; the
//                  span's own top-min(k, span) positions go to the workspace as (key, position) candidates,
//                  position-ascending, with the span's largest logit and its softmax denominator
//   long_finish    (one workgroup per unit) the candidates of all spans into LDS (at most n_span x k),
//                  the same radix select and ordered compaction over them, alpha, the position list, exact attention over
//                  the selected rows, the blend, and inside sparq_decode_step the append
// (Measured for 512 units of 40 960 positions, k = 1024, per step: with the append, the merge, the gather and the last
// merge as launches of their own 313 us, so 300; everything in one launch, the workgroup of a unit's last span going
// on with the unit, 350-358: with the memory saturated each of its round trips to other workgroups' results takes
// microseconds.)
// The local window is part of both levels: its positions are the last ones of the sequence, every span
// hands on those it holds, and they are the last candidates of the merge.
#include "decode_stages.h"

namespace sparq {

namespace {

// LDS words of long_scores besides the span's keys
template <int DH>
__host__ __device__ constexpr size_t scores_fixed_words() {
  return 2 * (size_t)kRadixBins + 3 * (size_t)DH + 32 + 16 + 8;
}

template <class T, int DH>
__global__ __launch_bounds__(NT, 4) void long_scores(const LongArgs a) {
  extern __shared__ __align__(16) uint32_t smem[];
  uint32_t* keys = smem;                                        // [span_len]
  uint32_t* hist = keys + a.span_len;                           // [2][kRadixBins]
  float* qf = reinterpret_cast<float*>(hist + 2 * kRadixBins);  // [DH]
  float* qs = qf + DH;
  int* chan = reinterpret_cast<int*>(qs + DH);
  float* red = reinterpret_cast<float*>(chan + DH);             // [32]
  uint32_t* wcnt = reinterpret_cast<uint32_t*>(red + 32);       // [16]
  int* ctl = reinterpret_cast<int*>(wcnt + 16);                 // [8]
  const DecodeArgs& d = a.d;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int U = d.B * d.H;
  int u, s;
  map_span(U, a.n_span, a.by_span, u, s);
  const int b = divided(u, d.by_H), h = u - b * d.H;
  const size_t kv_head = (size_t)b * d.H_kv + divided(h, d.by_group);

  const LaneCodes<DH> qcode = load_lane_codes<DH>(reinterpret_cast<const uint16_t*>(d.q) + (size_t)u * DH, lane);
  for (int i = tid; i < 2 * kRadixBins; i += NT) hist[i] = 0u;
  bool appended, bad, full;      // inside a step the row being appended counts as position S_b; long_finish writes it
  const int S = visible_length(d, b, appended, bad, full);
  if (tid == 0 && s == 0 && (bad || full)) atomicOr(d.err, (bad ? 8 : 0) | (full ? 1 : 0));
  int32_t* idx_out = d.idx_out ? d.idx_out + (size_t)u * d.idx_stride : nullptr;
  if (S == 0) {   // nothing cached: span 0 writes the defined outputs, the later launches skip the unit
    if (s == 0) {
      if (tid < DH) reinterpret_cast<uint16_t*>(d.out)[(size_t)u * DH + tid] = 0;
      if (tid == 0) { atomicOr(d.err, 2); if (d.alpha_out) d.alpha_out[u] = 0.0f; }
      if (d.chan_out && tid < d.r) d.chan_out[(size_t)u * d.r + tid] = -1;
      if (idx_out) for (int n = tid; n < d.idx_stride; n += NT) idx_out[n] = -1;
    }
    return;
  }
  int kb = d.k_per_seq ? d.k_per_seq[b] : d.k;
  kb = kb < 1 ? 1 : (kb > d.k ? d.k : kb);
  const int kq = kb < S ? kb : S;
  const Window win = make_window(d.local_window, S, kq);
  const size_t slot = (size_t)u * a.n_span + s;
  const int p0 = s * a.span_len;
  if (p0 >= S) {   // a span beyond the end of this sequence
    if (tid == 0) { a.cnt_ws[slot] = 0; a.tmax_ws[slot] = -INFINITY; a.zsum_ws[slot] = 0.0f; }
    return;
  }
  const int len = S - p0 < a.span_len ? S - p0 : a.span_len;

  const QueryLds Q{qf, qs, chan};
  select_channels<T, DH>(Q, qcode, d.r, red + 30, lane, wave);

  // the newest S mod 8 positions are not in Kt (inside a step: up to 8, Kt being up to date for the length before the
  // call): the span that holds them takes them from the rows of K, the row being appended from the inputs
  const int S_fl = (appended ? S - 1 : S) & ~7, r8 = (d.r + 7) & ~7;
  const int n_tail = (S_fl >= p0 && S_fl < p0 + len) ? S - S_fl : 0;
  TailRow tail;
  float tau, esc;
  auto requested = [&]() {     // behind the stream's first loads
    if (wave < n_tail) {
      const uint16_t* krow = appended && wave == n_tail - 1
                                 ? reinterpret_cast<const uint16_t*>(d.k_new) + kv_head * DH
                                 : reinterpret_cast<const uint16_t*>(d.K) + (kv_head * d.S_stride + S_fl + wave) * (size_t)DH;
      tail = tail_row_issue(krow, chan, r8, lane);
    }
    tau = temperature(red + 30, d.flags, DH, d.r);
    esc = kLog2e / tau;
    if (s == 0) {
      if (d.chan_out && tid < d.r) d.chan_out[(size_t)u * d.r + tid] = chan[tid];
      if (tid == 0) a.tau_ws[u] = tau;
    }
  };

  const int end = p0 + len < S_fl ? p0 + len : S_fl;     // whole chunks of this span that are in Kt
  const uint32_t row_bytes = (uint32_t)d.S_stride * 2;
  const char* Kt_head = reinterpret_cast<const char*>(d.Kt) + kv_head * DH * row_bytes;
  RunningSum zs;
  stream_channel_rows<T>(Kt_head, row_bytes, chan, qs, d.r, p0 >> 3, end > p0 ? end >> 3 : p0 >> 3, tid,
                         [&](int c, const float (&acc)[8]) {
    uint32_t kx[8];
    zs.add(acc, esc);
#pragma unroll
    for (int e = 0; e < 8; ++e) kx[e] = float_to_key(acc[e]);
    hist_add_chunk(hist, kx, win.S_old - c * 8);
    uint4* dst = reinterpret_cast<uint4*>(keys + (c * 8 - p0));
    dst[0] = make_uint4(kx[0], kx[1], kx[2], kx[3]);
    dst[1] = make_uint4(kx[4], kx[5], kx[6], kx[7]);
  }, requested);
  if (wave < n_tail) {
    const float dot = tail_row_dot<T>(tail, qs, r8, lane);
    if (lane == 0) {
      zs.add({dot}, esc);
      const uint32_t key = float_to_key(dot);
      keys[S_fl + wave - p0] = key;
      if (S_fl + wave < win.S_old) atomicAdd(&hist[hist_slot(key >> 21)], 1u);
    }
  }
  const float tmax = wave_max(zs.ref);
  if (lane == 0) red[wave] = tmax;
  __syncthreads();
  auto dmax_of = [&]() { return wave_values_max(red); };

  // the span's own selection: its part of the window unconditionally, and as many of its older positions
  // as the whole sequence may take
  int n_old = win.S_old - p0;
  n_old = n_old < 0 ? 0 : (n_old > len ? len : n_old);
  const int k_old = win.k_old < n_old ? win.k_old : n_old;
  const SelectLds sel{hist, wcnt, ctl, red};
  uint32_t* cand_key = a.cand_key_ws + slot * a.cand_cap;
  uint32_t* cand_pos = reinterpret_cast<uint32_t*>(a.cand_pos_ws) + slot * a.cand_cap;
  select_compact<Sums::kNumerator>(keys, cand_pos, len, n_old, k_old, dmax_of, esc, zs, nullptr, 0, sel, tid, lane, wave, cand_key, p0);
  if (tid == 0) {
    a.cnt_ws[slot] = k_old + (len - n_old);
    a.tmax_ws[slot] = dmax_of();
    a.zsum_ws[slot] = all_mass(red);
  }
}

// One workgroup per unit: merge the candidates of the spans and do the rest of the unit.
template <class T, int DH>
__global__ __launch_bounds__(NT, 4) void long_finish(const LongArgs a) {
  extern __shared__ __align__(16) uint32_t smem[];
  const DecodeArgs& d = a.d;
  const int cap_all = a.n_span * a.cand_cap;
  uint32_t* keys = smem;                                          // [round_up(cap_all, 8)]; later the list
  uint32_t* hist = keys + ((cap_all + 7) & ~7);                   // [2][kRadixBins]; later the waves' partial results
  float* red = reinterpret_cast<float*>(hist + 2 * kRadixBins);   // [32]
  uint32_t* wcnt = reinterpret_cast<uint32_t*>(red + 32);         // [16]
  int* ctl = reinterpret_cast<int*>(wcnt + 16);                   // [8]
  int* off = ctl + 8;                                             // [kMaxSpans + 1] candidates before each span
  float* stat = reinterpret_cast<float*>(off + kMaxSpans + 8);    // [2]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int U = d.B * d.H;
  int u = blockIdx.x;
  if ((U & 7) == 0) u = (u & 7) * (U >> 3) + (u >> 3);            // the heads of a KV group share an XCD
  const int b = divided(u, d.by_H), h = u - b * d.H, hk = divided(h, d.by_group);
  const size_t kv_head = (size_t)b * d.H_kv + hk;
  bool appended, bad, full;
  const int S = visible_length(d, b, appended, bad, full);
  const bool owner = d.k_new && h == hk * d.group;         // writes the row and the new mean
  if (d.k_new && h == 0 && tid == 0) {   // a length beyond the bound of this call that the buffers can hold is carried over as it is
    const int S_in = d.seq_lens[b];
    d.seq_lens_next[b] = (S_in > d.S_max && S_in <= d.S_stride) ? S_in : S;
  }
  // what the end of the unit needs is requested early
  float vm = 0.0f;
  uint16_t kc = 0, vc = 0;
  if (tid < DH) {
    vm = d.v_mean[kv_head * DH + tid];
    if (appended) {
      kc = reinterpret_cast<const uint16_t*>(d.k_new)[kv_head * DH + tid];
      vc = reinterpret_cast<const uint16_t*>(d.v_new)[kv_head * DH + tid];
    }
  }
  if (S == 0) {                            // outputs written by long_scores
    if (owner && tid < DH) d.v_mean_next[kv_head * DH + tid] = vm;
    return;
  }
  int kb = d.k_per_seq ? d.k_per_seq[b] : d.k;
  kb = kb < 1 ? 1 : (kb > d.k ? d.k : kb);
  const int kq = kb < S ? kb : S;
  int32_t* idx_out = d.idx_out ? d.idx_out + (size_t)u * d.idx_stride : nullptr;
  const Window win = make_window(d.local_window, S, kq);
  const float tau = a.tau_ws[u];
  const float esc = kLog2e / tau;
  using G = RowGeometry<DH>;
  const int sub = lane % G::LPR;
  const uint4 qraw = load16(reinterpret_cast<const uint16_t*>(d.q) + (size_t)u * DH + sub * 8);

  for (int i = tid; i < 2 * kRadixBins; i += NT) hist[i] = 0u;
  if (wave == 0) {   // kMaxSpans = 64: one lane per span
    const size_t slot = (size_t)u * a.n_span + lane;
    const bool on = lane < a.n_span;
    const int cnt = on ? a.cnt_ws[slot] : 0;
    const float tm = on ? a.tmax_ws[slot] : -INFINITY;
    const float zs = on ? a.zsum_ws[slot] : 0.0f;
    const uint32_t incl = wave_scan_incl((uint32_t)cnt);
    off[lane + 1] = (int)incl;
    if (lane == 0) off[0] = 0;
    const float dmax = wave_max(tm);
    const float z = wave_sum(tm == -INFINITY ? 0.0f : zs * exp2f((tm - dmax) * esc));
    if (lane == 0) { stat[0] = dmax; stat[1] = z; }
  }
  __syncthreads();
  const int n_cand = off[a.n_span];
  const int n_free = n_cand - win.n_local;        // candidates that compete; the window's come last
  const float dmax = stat[0], zsum = stat[1];
  const uint32_t* unit_key = a.cand_key_ws + (size_t)u * a.n_span * a.cand_cap;
  const int32_t* unit_pos = a.cand_pos_ws + (size_t)u * a.n_span * a.cand_cap;
  auto entry = [&](int ci) {                      // candidate number -> entry of the unit's candidate arrays
    int lo = 0, hi = a.n_span - 1;                // the last span that starts at or before it
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (off[mid] <= ci) lo = mid; else hi = mid - 1;
    }
    return lo * a.cand_cap + (ci - off[lo]);
  };
  constexpr int FLY = 8;                          // eight loads in flight per thread, across the spans
  for (int n0 = tid; n0 < n_cand; n0 += FLY * NT) {
    uint32_t key[FLY];
#pragma unroll
    for (int j = 0; j < FLY; ++j) key[j] = n0 + j * NT < n_cand ? unit_key[entry(n0 + j * NT)] : 0u;
#pragma unroll
    for (int j = 0; j < FLY; ++j) {
      const int n = n0 + j * NT;
      if (n < n_cand) {
        keys[n] = key[j];
        if (n < n_free) atomicAdd(&hist[hist_slot(key[j] >> 21)], 1u);
      }
    }
  }
  __syncthreads();
  const SelectLds sel{hist, wcnt, ctl, red};
  const Selection chosen = select_compact<Sums::kNumerator>(keys, keys, n_cand, n_free, win.k_old, [&]() { return dmax; }, esc, RunningSum{},
                                                            nullptr, 0, sel, tid, lane, wave);
  const float alpha = as_share(selected_mass(chosen, red, dmax, esc) / zsum, kq == S);
  for (int n0 = tid; n0 < kq; n0 += FLY * NT) {   // candidate numbers -> positions, in place
    int pos[FLY];
#pragma unroll
    for (int j = 0; j < FLY; ++j) pos[j] = n0 + j * NT < kq ? unit_pos[entry((int)keys[n0 + j * NT])] : 0;
#pragma unroll
    for (int j = 0; j < FLY; ++j) {
      const int n = n0 + j * NT;
      if (n < kq) {
        keys[n] = (uint32_t)pos[j];
        if (idx_out && n < d.idx_stride) idx_out[n] = pos[j];
      }
    }
  }
  if (tid == 0) {
    if (d.alpha_out) d.alpha_out[u] = alpha;
    if (idx_out && kq > d.idx_stride) atomicOr(d.err, 4);
  }
  if (idx_out) for (int n = kq + tid; n < d.idx_stride; n += NT) idx_out[n] = -1;
  __syncthreads();

  // ---- exact attention over the selected rows, blend, append: as in sparq_decode_fused ----
  const int* list = reinterpret_cast<const int*>(keys);
  uint16_t* K_rows = reinterpret_cast<uint16_t*>(d.K) + kv_head * d.S_stride * (size_t)DH;
  const char* K_head = reinterpret_cast<const char*>(K_rows) + sub * 16;
  const char* V_head = reinterpret_cast<const char*>(d.V) + kv_head * d.S_stride * (size_t)(DH * 2) + sub * 16;
  const float qscale = kLog2e / sqrtf((float)DH);
  float q8[8];
  unpack8<T>(qraw, q8);
#pragma unroll
  for (int e = 0; e < 8; ++e) q8[e] *= qscale;
  // positions are ascending: the appended row can only be the last entry, and is taken from the inputs
  const bool new_selected = appended && list[kq - 1] == S - 1;
  float m_run = -INFINITY, l_run = 0.0f;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  attend_rows<T, DH>(K_head, V_head, list, 0, kq - (new_selected ? 1 : 0), q8, lane, wave, m_run, l_run, acc);
  if (new_selected)
    attend_row_from_codes<T, DH>(reinterpret_cast<const uint16_t*>(d.k_new) + kv_head * DH,
                                 reinterpret_cast<const uint16_t*>(d.v_new) + kv_head * DH, q8, lane, wave, m_run, l_run, acc);
  float* part = reinterpret_cast<float*>(hist);
  store_wave_partial<DH>(m_run, l_run, acc, part, lane, wave);
  __syncthreads();
  if (tid < DH) {
    float m_all, l_all, y3;
    combine_partials<DH>(part, NW, tid, m_all, l_all, y3);
    y3 /= l_all;
    if (appended) {                                // the mean with the new row; the mean of no rows is ignored
      if (S == 1) vm = 0.0f;
      vm += (T::widen(vc) - vm) * (1.0f / (float)S);
    }
    float y = y3;
    if (!(d.flags & 1u)) y = alpha * y3 + (1.0f - alpha) * vm;
    reinterpret_cast<uint16_t*>(d.out)[(size_t)u * DH + tid] = T::narrow(y);
    // nobody reads row S - 1 of K or V, or columns of Kt, in this launch; the mean goes to the *_next buffer
    if (owner) {
      d.v_mean_next[kv_head * DH + tid] = vm;
      if (appended) {
        reinterpret_cast<uint16_t*>(d.V)[(kv_head * d.S_stride + (S - 1)) * DH + tid] = vc;
        K_rows[(size_t)(S - 1) * DH + tid] = kc;
        if ((S & 7) == 0)
          flush_key_columns(reinterpret_cast<uint16_t*>(d.Kt) + kv_head * DH * (size_t)d.S_stride, K_rows, d.S_stride, DH, S, tid, kc);
      }
    }
  }
}

template <class T, int DH>
hipError_t launch_long(const LongArgs& a, hipStream_t s) {
  const int units = a.d.B * a.d.H;
  const size_t lds1 = 4 * ((size_t)a.span_len + scores_fixed_words<DH>()), lds2 = long_merge_lds_bytes(a.n_span, a.cand_cap);
  hipError_t e;
  if ((e = allow_lds<long_scores<T, DH>>(lds1)) != hipSuccess) return e;
  if ((e = allow_lds<long_finish<T, DH>>(lds2)) != hipSuccess) return e;
  hipLaunchKernelGGL((long_scores<T, DH>), dim3(units * a.n_span), dim3(NT), lds1, s, a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL((long_finish<T, DH>), dim3(units), dim3(NT), lds2, s, a);
  return hipGetLastError();
}

}  // namespace

size_t long_scores_lds_bytes(int span_len, int d_h) {
  switch (d_h) {
    case 64: return 4 * ((size_t)span_len + scores_fixed_words<64>());
    case 128: return 4 * ((size_t)span_len + scores_fixed_words<128>());
    case 256: return 4 * ((size_t)span_len + scores_fixed_words<256>());
    default: return 0;
  }
}

size_t long_merge_lds_bytes(int n_span, int cand_cap) {
  return 4 * ((((size_t)n_span * cand_cap + 7) & ~(size_t)7) + 2 * kRadixBins + 32 + 16 + 8 + kMaxSpans + 8 + 8);
}

hipError_t launch_decode_long(const LongArgs& a, int dtype, hipStream_t s) {
  const bool bf = dtype == 1;
  switch (a.d.d_h) {
    case 64:  return bf ? launch_long<BF16, 64>(a, s) : launch_long<F16, 64>(a, s);
    case 128: return bf ? launch_long<BF16, 128>(a, s) : launch_long<F16, 128>(a, s);
    case 256: return bf ? launch_long<BF16, 256>(a, s) : launch_long<F16, 256>(a, s);
    default:  return hipErrorInvalidValue;
  }
}

}  // namespace sparq
