// SparQ decode with the paper's grouped-query rule (Section 4, "Grouped query attention";
// Appendix B): the G query heads that share a KV head select ONE channel set from the group sum of
// |q| and ONE position set from the group sum of their approximate scores s-hat; the temperature,
// alpha and the exact attention stay per query head.  One workgroup per (sequence, KV head).
//   stage 0  group sums of |q| in fp64 (head order, as the definition is written), top-r, per-head tau
//   pass A   stream the r channel rows once for all G heads: the G logit numerators of every position go to
//            the workspace (fp32), per-head max and sum-exp stay in registers
//   pass B   read them back: score_i = sum_h softmax_h(z)_i as integer keys in LDS
//   stage 2  radix select of the k largest scores, ordered position list
//   stage 3  gather each selected K and V row once for the G heads: exact attention per head; per-head
//            alpha from the stored logits of the selected positions
//   blend    y_h = alpha_h y3_h + (1 - alpha_h) v_mean (Eq. 10), round and store
// The group sum of softmaxes is not monotone in any one head's logits, so the logits themselves are needed
// twice (statistics, then scores) and a third time for alpha; G x S floats do not fit in LDS for long
// sequences, so they live in the workspace (16 bytes per position for G = 4, against 2 r bytes for streaming
// the key rows again), written and read by the same workgroup.
#include "group_stages.h"

namespace sparq {

namespace {

template <int DH, int G>
struct SharedLds {
  uint32_t* keys;      // [S_max]
  SelectLds sel;       // hist [2][kRadixBins], wcnt, ctl, red
  float* part;         // [NW][G][DH + 2], aliases hist after the select
  float* qf;           // [G][DH]
  float* qs;           // [G][DH] per-head components on the shared channel list (padded, weight 0)
  int* chan;           // [DH]
  float* stat;         // [NW][G][2]
};

template <int DH, int G>
__host__ __device__ constexpr size_t shared_part_words() { return (size_t)NW * G * (DH + 2); }

// words after the key array
template <int DH, int G>
__host__ __device__ constexpr size_t shared_fixed_words() {
  size_t hist_part = 2 * kRadixBins;
  if (hist_part < shared_part_words<DH, G>()) hist_part = shared_part_words<DH, G>();
  return hist_part + 2 * (size_t)G * DH /* qf, qs */ + DH /* chan */ + 32 + 16 + 8 + NW * G * 2;
}

// One workgroup serves lengths up to which the keys and this many words fit the LDS.  More than the arrays take: the line between
// the plans, and with it the workspace of a shape, stays where the plans were compared.
template <int DH, int G>
__host__ __device__ constexpr size_t shared_limit_words() {
  size_t hist_part = 2 * kRadixBins + NT;
  if (hist_part < shared_part_words<DH, G>()) hist_part = shared_part_words<DH, G>();
  constexpr size_t others = 2 * (size_t)G * DH + 3 * DH + 56 + NW * G * 2 + G * 4;
  return hist_part + others;
}

template <int DH, int G>
__device__ __forceinline__ SharedLds<DH, G> carve_shared(uint32_t* base, int S_max) {
  SharedLds<DH, G> l;
  l.keys = base; base += S_max;
  size_t hist_part = 2 * kRadixBins;
  if (hist_part < shared_part_words<DH, G>()) hist_part = shared_part_words<DH, G>();
  l.sel.hist = base;
  l.part = reinterpret_cast<float*>(base);
  base += hist_part;
  l.qf = reinterpret_cast<float*>(base); base += G * DH;
  l.qs = reinterpret_cast<float*>(base); base += G * DH;
  l.chan = reinterpret_cast<int*>(base); base += DH;
  l.sel.red = reinterpret_cast<float*>(base); base += 32;
  l.sel.wcnt = base; base += 16;
  l.sel.ctl = reinterpret_cast<int*>(base); base += 8;
  l.stat = reinterpret_cast<float*>(base);
  return l;
}

template <class T, int DH, int G>
__global__ __launch_bounds__(NT, 2) void sparq_decode_shared(const DecodeArgs a, float* __restrict__ z_ws) {
  extern __shared__ __align__(16) uint32_t smem[];
  const SharedLds<DH, G> L = carve_shared<DH, G>(smem, a.S_max);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const size_t kv_head = blockIdx.x;                 // (b, hk)
  const int b = divided((int)kv_head, a.by_H_kv), hk = (int)(kv_head - (size_t)b * a.H_kv);
  const size_t u0 = (size_t)b * a.H + (size_t)hk * G;   // first query head of the group

  LaneCodes<DH> qcode[G];
#pragma unroll
  for (int h = 0; h < G; ++h) qcode[h] = load_lane_codes<DH>(reinterpret_cast<const uint16_t*>(a.q) + (u0 + h) * DH, lane);
  // Inside sparq_decode_step the row being appended counts as position S_b: it is taken from the inputs, and this workgroup,
  // the only one of its KV head, writes it at the end (an append launch in front took 5-14 us: 128 KV heads
  // at 4000 positions 51 -> 44 us per step, two at 500 19.7 -> 15.0).
  bool appended, bad, full;
  const int S = visible_length(a, b, appended, bad, full);
  if (tid == 0) {
    if (hk == 0 && (bad || full)) atomicOr(a.err, (bad ? 8 : 0) | (full ? 1 : 0));
    if (a.k_new && hk == 0) {   // a length beyond the bound of this call that the buffers can hold is carried over as it is
      const int S_in = a.seq_lens[b];
      a.seq_lens_next[b] = (S_in > a.S_max && S_in <= a.S_stride) ? S_in : S;
    }
  }
  int kb = a.k_per_seq ? a.k_per_seq[b] : a.k;
  kb = kb < 1 ? 1 : (kb > a.k ? a.k : kb);
  const int kq = kb < S ? kb : S;
  uint16_t* out = reinterpret_cast<uint16_t*>(a.out) + u0 * DH;
  if (S == 0) {
    for (int i = tid; i < G * DH; i += NT) out[i] = 0;
    if (tid < G) { if (a.alpha_out) a.alpha_out[u0 + tid] = 0.0f; }
    if (tid == 0) atomicOr(a.err, 2);
    if (a.chan_out) for (int i = tid; i < G * a.r; i += NT) a.chan_out[u0 * a.r + i] = -1;
    if (a.idx_out) for (int i = tid; i < G * a.idx_stride; i += NT) a.idx_out[u0 * a.idx_stride + i] = -1;
    if (a.k_new && tid < DH) a.v_mean_next[kv_head * DH + tid] = a.v_mean[kv_head * DH + tid];
    return;
  }

  // ---------------- stage 0: shared channel set, per-head temperature ----------------
  for (int i = tid; i < 2 * kRadixBins; i += NT) L.sel.hist[i] = 0u;
  float esc[G];        // log2(e) / tau_h
  const GroupQueryLds GQ{L.qf, L.qs, L.chan};
  select_channels_group<T, DH, G>(GQ, qcode, a.r, a.flags, L.sel.red, lane, wave, esc);
  if (a.chan_out)
    for (int i = tid; i < G * a.r; i += NT) a.chan_out[u0 * a.r + i] = L.chan[i % a.r];

  const Window win = make_window(a.local_window, S, kq);

  // ---------------- pass A: per-head max and sum-exp of the approximate logits ----------------
  const uint32_t row_bytes = (uint32_t)a.S_stride * 2;
  const char* Kt_head = reinterpret_cast<const char*>(a.Kt) + kv_head * DH * row_bytes;
  // whole chunks that are in Kt: the newest S mod 8 positions are not in it yet (inside a step: up to 8, Kt being up to
  // date for the length before the call)
  const int S_fl = (appended ? S - 1 : S) & ~7, n_chunks = S_fl >> 3, n_tail = S - S_fl, r8 = (a.r + 7) & ~7;
  uint16_t* K_rows = reinterpret_cast<uint16_t*>(a.K) + kv_head * a.S_stride * (size_t)DH;
  const uint16_t* k_row = reinterpret_cast<const uint16_t*>(a.k_new) + kv_head * DH;     // used where `appended`
  const uint16_t* v_row = reinterpret_cast<const uint16_t*>(a.v_new) + kv_head * DH;
  float tdot[G];          // wave w: the logit numerators of position S_fl + w for the G heads, from its K row
#pragma unroll
  for (int h = 0; h < G; ++h) tdot[h] = 0.0f;
  if (wave < n_tail) {
    const TailRow tail = tail_row_issue(appended && wave == n_tail - 1 ? k_row : K_rows + (size_t)(S_fl + wave) * DH, L.chan, r8, lane);
#pragma unroll
    for (int h = 0; h < G; ++h) tdot[h] = tail_row_dot<T>(tail, L.qs + h * DH, r8, lane);
  }
  RunningSum rs[G];     // running max of the logit numerator, sum of exp2((d - max) * esc)
  float* z_unit = z_ws + u0 * (size_t)a.S_max;        // [G][S_max] logit numerators of this group
  stream_channel_rows_group<T, G>(Kt_head, row_bytes, L.chan, L.qs, DH, a.r, 0, n_chunks, tid,
                                  [&](int c, const float (&acc)[G][8]) {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      float4* dst = reinterpret_cast<float4*>(z_unit + (size_t)h * a.S_max + c * 8);
      dst[0] = make_float4(acc[h][0], acc[h][1], acc[h][2], acc[h][3]);
      dst[1] = make_float4(acc[h][4], acc[h][5], acc[h][6], acc[h][7]);
      rs[h].add(acc[h], esc[h]);
    }
  });
  if (wave < n_tail && lane == 0) {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      const float v = tdot[h];
      z_unit[(size_t)h * a.S_max + S_fl + wave] = v;
      rs[h].add({v}, esc[h]);
    }
  }
  float mh[G], inv_z[G], log_z[G];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    float m, z;
    wave_merge(rs[h], esc[h], m, z);
    if (lane == 0) { L.stat[(wave * G + h) * 2] = m; L.stat[(wave * G + h) * 2 + 1] = z; }
  }
  __syncthreads();
#pragma unroll
  for (int h = 0; h < G; ++h) {
    float m = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) m = fmaxf(m, L.stat[(w * G + h) * 2]);
    float z = 0.0f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float mw = L.stat[(w * G + h) * 2];
      z += L.stat[(w * G + h) * 2 + 1] * exp2f((mw - m) * esc[h]);    // 0 of a wave without positions
    }
    mh[h] = m; inv_z[h] = 1.0f / z; log_z[h] = log2f(inv_z[h]);
  }

  // ---------------- pass B: group score = sum over heads of s-hat, as keys ----------------
  // (the barrier above also orders this workgroup's stores of pass A before these loads)
  for (int c = tid; c < n_chunks; c += NT) {
    float4 lo[G], hi[G];
#pragma unroll
    for (int h = 0; h < G; ++h) {
      const float4* src = reinterpret_cast<const float4*>(z_unit + (size_t)h * a.S_max + c * 8);
      lo[h] = src[0]; hi[h] = src[1];
    }
    uint32_t kx[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float dv[G];
#pragma unroll
      for (int h = 0; h < G; ++h) dv[h] = e < 4 ? (&lo[h].x)[e] : (&hi[h].x)[e - 4];
      kx[e] = float_to_key(group_score<G>(dv, mh, esc, log_z));
      if (c * 8 + e < win.S_old) atomicAdd(&L.sel.hist[hist_slot(kx[e] >> 21)], 1u);
    }
    uint4* dst = reinterpret_cast<uint4*>(L.keys + c * 8);
    dst[0] = make_uint4(kx[0], kx[1], kx[2], kx[3]);
    dst[1] = make_uint4(kx[4], kx[5], kx[6], kx[7]);
  }
  if (wave < n_tail && lane == 0) {
    const uint32_t key = float_to_key(group_score<G>(tdot, mh, esc, log_z));
    L.keys[S_fl + wave] = key;
    if (S_fl + wave < win.S_old) atomicAdd(&L.sel.hist[hist_slot(key >> 21)], 1u);
  }
  __syncthreads();

  // ---------------- stage 2: the kq positions of largest group score ----------------
  int32_t* idx_out = a.idx_out ? a.idx_out + u0 * a.idx_stride : nullptr;
  select_compact<Sums::kNone>(L.keys, L.keys, S, win.S_old, win.k_old, []() { return 0.0f; }, 0.0f, RunningSum{}, idx_out, a.idx_stride, L.sel, tid, lane, wave);
  if (idx_out) {
    if (tid == 0 && kq > a.idx_stride) atomicOr(a.err, 4);
    for (int n = kq + tid; n < a.idx_stride; n += NT) idx_out[n] = -1;
    // the other heads of the group report the same list
    const int shown = kq < a.idx_stride ? kq : a.idx_stride;
    for (int h = 1; h < G; ++h)
      for (int n = tid; n < a.idx_stride; n += NT)
        idx_out[(size_t)h * a.idx_stride + n] = n < shown ? (int)L.keys[n] : -1;
  }

  // alpha_h = sum over the selected positions of s-hat_h, from the stored logits (the same values the
  // normaliser was summed from)
  float asum[G];
#pragma unroll
  for (int h = 0; h < G; ++h) asum[h] = 0.0f;
  for (int n = tid; n < kq; n += NT) {
    const int pos = (int)L.keys[n];
#pragma unroll
    for (int h = 0; h < G; ++h) asum[h] += exp2f((z_unit[(size_t)h * a.S_max + pos] - mh[h]) * esc[h]);
  }

  // ---------------- stage 3: one gather for the G heads ----------------
  const int sub = lane % RowGeometry<DH>::LPR;
  const int* list = reinterpret_cast<const int*>(L.keys);
  const char* K_head = reinterpret_cast<const char*>(a.K) + kv_head * a.S_stride * (size_t)(DH * 2) + sub * 16;
  const char* V_head = reinterpret_cast<const char*>(a.V) + kv_head * a.S_stride * (size_t)(DH * 2) + sub * 16;
  const float qscale = kLog2e / sqrtf((float)DH);
  float q8[G][8];   // query slices, exp2 domain
  float m_run[G], l_run[G], acc[G][8];
#pragma unroll
  for (int h = 0; h < G; ++h) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float qv = L.qf[h * DH + sub * 8 + e];
      q8[h][e] = qv * qscale;
      acc[h][e] = 0.0f;
    }
    m_run[h] = -INFINITY; l_run[h] = 0.0f;
  }
  // positions are ascending: the appended row can only be the last entry
  const bool new_selected = appended && list[kq - 1] == S - 1;
  attend_rows_group<T, DH, G>(K_head, V_head, list, 0, kq - (new_selected ? 1 : 0), q8, lane, wave, m_run, l_run, acc);
  if (new_selected) {
#pragma unroll
    for (int h = 0; h < G; ++h) attend_row_from_codes<T, DH>(k_row, v_row, q8[h], lane, wave, m_run[h], l_run[h], acc[h]);
  }
  __syncthreads();   // hist is dead: `part` may overwrite them
#pragma unroll
  for (int h = 0; h < G; ++h) {
    const float a_w = wave_sum(asum[h]);
    if (lane == 0) L.stat[(wave * G + h) * 2] = a_w;
    store_wave_partial<DH>(m_run[h], l_run[h], acc[h], L.part + h * (DH + 2), lane, wave * G);   // part[wave][h]
  }
  __syncthreads();
  for (int i = tid; i < G * DH; i += NT) {
    const int h = i / DH, c = i - h * DH;
    float m_all = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) m_all = fmaxf(m_all, L.part[(w * G + h) * (DH + 2) + DH]);
    float l_all = 0.0f, y3 = 0.0f, a_all = 0.0f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float s = weight_exp2(L.part[(w * G + h) * (DH + 2) + DH], m_all);
      l_all += L.part[(w * G + h) * (DH + 2) + DH + 1] * s;
      y3 += L.part[(w * G + h) * (DH + 2) + c] * s;
      a_all += L.stat[(w * G + h) * 2];
    }
    y3 /= l_all;
    // inv_z of head h: recompute from the broadcast statistics is not needed, every thread holds all G
    float alpha = 0.0f;
#pragma unroll
    for (int hh = 0; hh < G; ++hh) if (hh == h) alpha = a_all * inv_z[hh];
    alpha = as_share(alpha, kq == S);
    float vm = a.v_mean[kv_head * DH + c];
    if (appended) {                        // the mean with the new row; the mean of no rows is ignored
      if (S == 1) vm = 0.0f;
      vm += (T::widen(v_row[c]) - vm) * (1.0f / (float)S);
    }
    float y = y3;
    if (!(a.flags & 1u)) y = alpha * y3 + (1.0f - alpha) * vm;
    out[(size_t)h * DH + c] = T::narrow(y);
    if (c == 0 && a.alpha_out) a.alpha_out[u0 + h] = alpha;
    if (a.k_new && h == 0) {               // everything this workgroup reads of the cache has been read
      a.v_mean_next[kv_head * DH + c] = vm;
      if (appended) {
        reinterpret_cast<uint16_t*>(a.V)[(kv_head * a.S_stride + (S - 1)) * DH + c] = v_row[c];
        K_rows[(size_t)(S - 1) * DH + c] = k_row[c];
        if ((S & 7) == 0)
          flush_key_columns(reinterpret_cast<uint16_t*>(a.Kt) + kv_head * DH * (size_t)a.S_stride, K_rows, a.S_stride, DH, S, c, k_row[c]);
      }
    }
  }
}

template <class T, int DH, int G>
hipError_t launch_shared_g(const DecodeArgs& a, float* z_ws, hipStream_t s) {
  static_assert(shared_limit_words<DH, G>() >= shared_fixed_words<DH, G>(), "what the plan admits fits");
  const size_t lds = 4 * ((size_t)a.S_max + shared_fixed_words<DH, G>());
  auto kern = sparq_decode_shared<T, DH, G>;
  hipError_t e = allow_lds<sparq_decode_shared<T, DH, G>>(lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(a.B * a.H_kv), dim3(NT), lds, s, a, z_ws);
  return hipGetLastError();
}

template <class T, int DH>
hipError_t launch_shared_dh(const DecodeArgs& a, float* z_ws, hipStream_t s) {
  switch (a.H / a.H_kv) {
    case 2: return launch_shared_g<T, DH, 2>(a, z_ws, s);
    case 4: return launch_shared_g<T, DH, 4>(a, z_ws, s);
    default: return hipErrorInvalidValue;
  }
}

template <int DH>
size_t shared_limit(int S_max, int g) {
  return 4 * ((size_t)S_max + (g == 2 ? shared_limit_words<DH, 2>() : shared_limit_words<DH, 4>()));
}

}  // namespace

// LDS bytes that admit a length to the grouped-query kernel, 0 if the group size or head dimension has no kernel
size_t decode_shared_lds_bytes(int S_max, int d_h, int g) {
  if (g != 2 && g != 4) return 0;
  switch (d_h) {
    case 64: return shared_limit<64>(S_max, g);
    case 128: return shared_limit<128>(S_max, g);
    case 256: return shared_limit<256>(S_max, g);
    default: return 0;
  }
}

hipError_t launch_decode_shared(const DecodeArgs& a, float* z_ws, int dtype, hipStream_t s) {
  const bool bf = dtype == 1;
  switch (a.d_h) {
    case 64:  return bf ? launch_shared_dh<BF16, 64>(a, z_ws, s) : launch_shared_dh<F16, 64>(a, z_ws, s);
    case 128: return bf ? launch_shared_dh<BF16, 128>(a, z_ws, s) : launch_shared_dh<F16, 128>(a, z_ws, s);
    case 256: return bf ? launch_shared_dh<BF16, 256>(a, z_ws, s) : launch_shared_dh<F16, 256>(a, z_ws, s);
    default:  return hipErrorInvalidValue;
  }
}

}  // namespace sparq
