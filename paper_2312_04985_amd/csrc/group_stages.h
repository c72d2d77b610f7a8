// Stages of the grouped-query rule (Section 4, "Grouped query attention"; Appendix B) that several kernels
// share: the channel selection from the group sum of |q| with the per-head temperatures, and Step 1b for G
// query heads at once.
#pragma once
#include "decode_stages.h"

namespace sparq {

// The group score of a position is sum_h s-hat_h = sum_h exp2((d_h - max_h) esc_h) / Z_h.  Only its order
// matters (alpha is summed from the logits), so the key is formed from log2 of it, as
// max_h x_h + log2(sum_h exp2(x_h - max_h x_h)) with x_h = (d_h - max_h) esc_h - log2 Z_h.  The plain sum
// underflows to 0 for every position far below all heads' maxima: thousands of exactly equal keys, which the
// fp64 definition does not have, and which serialise the histogram atomics of the select (6 us per pass over
// 8192 keys instead of 1).  The logarithm keeps them apart at the same relative accuracy (the rounding of x_h
// dominates either way).  log_z = log2(1 / Z_h).
template <int G>
__device__ __forceinline__ float group_score(const float (&d)[G], const float (&mh)[G], const float (&esc)[G],
                                             const float (&log_z)[G]) {
  float x[G], mx = -INFINITY;
#pragma unroll
  for (int h = 0; h < G; ++h) { x[h] = (d[h] - mh[h]) * esc[h] + log_z[h]; mx = fmaxf(mx, x[h]); }
  float s = 0.0f;
#pragma unroll
  for (int h = 0; h < G; ++h) s += exp2_weight(x[h] - mx);
  return mx + log2_normal(s);             // 1 <= s <= G
}

// Per-head softmax statistics of a whole sequence from the n1 span partials {max, sum-exp relative to it}:
// executed by wave 0 (one lane per span, n1 <= 64); results to out[h] = {max, 1 / sum-exp}.
template <int G>
__device__ __forceinline__ void combine_span_stats(const float* stat_unit, int n1, const float* esc_unit, int lane, float* out) {
  const bool on = lane < n1;
  float m[G], z[G], esc[G];
#pragma unroll
  for (int h = 0; h < G; ++h) {      // all loads first: one round trip
    m[h] = on ? stat_unit[(lane * G + h) * 2] : -INFINITY;
    z[h] = on ? stat_unit[(lane * G + h) * 2 + 1] : 0.0f;
    esc[h] = esc_unit[h];
  }
#pragma unroll
  for (int h = 0; h < G; ++h) {
    const float m_all = wave_max(m[h]);
    const float z_all = wave_sum(m[h] == -INFINITY ? 0.0f : z[h] * exp2f((m[h] - m_all) * esc[h]));
    if (lane == 0) { out[h * 2] = m_all; out[h * 2 + 1] = 1.0f / z_all; }
  }
}

// One head's (running maximum, sum) over the 64 lanes of a wave: the sum relative to the common maximum.
__device__ __forceinline__ void wave_merge(const RunningSum& rs, float esc, float& m, float& z) {
  m = wave_max(rs.ref);
  z = wave_sum(rs.relative_to(m, esc));
}

struct GroupQueryLds {
  float* qf;       // [G][DH] the group's queries as fp32
  float* qs;       // [G][DH] per-head components on the shared channel list (padded to a multiple of 8, weight 0)
  int* chan;       // [DH] shared channel list, ascending, same padding
};

// Step 1a under the group rule: channel j is ranked by sum_h |q_h,j| (fp64, heads in order, ties to the lower
// channel); esc[h] = log2(e) / tau_h with tau_h from Eq. (9) on the shared channel set (or the fixed
// temperature the flags ask for).  q: the codes of the group's queries.  As select_channels: by the
// first wave, one barrier, which also publishes whatever the caller wrote to LDS before the call.  out: [G] floats of LDS.
template <class T, int DH, int G>
__device__ __forceinline__ void select_channels_group(const GroupQueryLds& Q, const LaneCodes<DH> (&q)[G], int r, uint32_t flags,
                                                      float* out, int lane, int wave, float (&esc)[G]) {
  constexpr int E = DH / kWave;
  if (wave == 0) {
    uint64_t mag[E];                                                        // sums >= 0: their bits order like they do
#pragma unroll
    for (int e = 0; e < E; ++e) {
      double m = 0.0;
#pragma unroll
      for (int h = 0; h < G; ++h) m += (double)fabsf(T::widen((uint16_t)q[h].c[e]));   // head order, as in the definition
      mag[e] = (uint64_t)__double_as_longlong(m);
    }
    bool sel[E];
    int at[E];
    wave_top_r<E, 63>(mag, r, sel, at);
    const int r8 = (r + 7) & ~7;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int j = lane * E + e;
#pragma unroll
      for (int h = 0; h < G; ++h) Q.qf[h * DH + j] = T::widen((uint16_t)q[h].c[e]);
      if (sel[e]) {
        Q.chan[at[e]] = j;
#pragma unroll
        for (int h = 0; h < G; ++h) Q.qs[h * DH + at[e]] = T::widen((uint16_t)q[h].c[e]);
        if (at[e] == r - 1)
          for (int pp = r; pp < r8; ++pp) {
            Q.chan[pp] = j;
#pragma unroll
            for (int h = 0; h < G; ++h) Q.qs[h * DH + pp] = 0.0f;
          }
      }
    }
#pragma unroll
    for (int h = 0; h < G; ++h) {
      float l1a = 0.0f, l1s = 0.0f;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const float aq = fabsf(T::widen((uint16_t)q[h].c[e]));
        l1a += aq; l1s += sel[e] ? aq : 0.0f;
      }
      const float all = wave_sum(l1a), part = wave_sum(l1s);
      const float tau = part > 0.0f ? sqrtf((float)DH * part / all) : sqrtf((float)DH);   // all logits 0 then
      if (lane == 0) out[h] = kLog2e / apply_tau_mode(tau, flags, DH, r);
    }
  }
  __syncthreads();
#pragma unroll
  for (int h = 0; h < G; ++h) esc[h] = out[h];
}

// Step 1b for G heads at once: like stream_channel_rows, every loaded 16-byte chunk feeds G accumulators.
// Thread tid of STRIDE owns chunks chunk_begin + tid + i * STRIDE (STRIDE < NT: the caller divides the channel
// rows of a chunk among NT / STRIDE groups of threads).
template <class T, int G, int STRIDE = NT, class Finish>
__device__ __forceinline__ void stream_channel_rows_group(const char* Kt_head, uint32_t row_bytes, const int* chan,
                                                          const float* qs, int qs_stride, int r, int chunk_begin,
                                                          int chunk_end, int tid, Finish&& finish) {
  const int n_batches = (r + 7) >> 3;
  const int n_chunks = chunk_end - chunk_begin;
  const int my_chunks = n_chunks > tid ? (n_chunks - tid + STRIDE - 1) / STRIDE : 0;
  const int items = my_chunks * n_batches;
  float acc[G][8];
#pragma unroll
  for (int h = 0; h < G; ++h)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[h][e] = 0.0f;
  int ic = 0, ib = 0, cc = 0, cb = 0;
  auto issue_next = [&](uint4 (&v)[8]) {
    issue_rows(v, Kt_head + (size_t)((uint32_t)(chunk_begin + tid + ic * STRIDE) * 16u), row_bytes, chan + ib * 8);
    if (++ib == n_batches) { ib = 0; ++ic; }
  };
  auto consume_next = [&](const uint4 (&v)[8]) {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      float f[8];
      unpack8<T>(v[t], f);
#pragma unroll
      for (int h = 0; h < G; ++h) {
        const float qv = qs[h * qs_stride + cb * 8 + t];
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[h][e] = fmaf(f[e], qv, acc[h][e]);
      }
    }
    if (++cb == n_batches) {
      finish(chunk_begin + tid + cc * STRIDE, acc);
#pragma unroll
      for (int h = 0; h < G; ++h)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[h][e] = 0.0f;
      cb = 0; ++cc;
    }
  };
  uint4 va[8], vb[8];
  if (items > 0) {
    issue_next(va);
    int i = 0;
    for (; i + 2 < items; i += 2) {
      issue_next(vb);
      consume_next(va);
      issue_next(va);
      consume_next(vb);
    }
    if (i + 1 < items) {
      issue_next(vb);
      consume_next(va);
      consume_next(vb);
    } else {
      consume_next(va);
    }
  }
}

// Step 2b for the G query heads of a group at once: attend_rows with every loaded row weighted for each head.  Two rows per
// lane and load (registers), one rescaling of a head's sums for both.  Bound by vector instructions: with a rescaling per row,
// exponentials that scale denormals first, and group_score's the same, one workgroup per KV head with 4 heads took 73.5 us
// per step for 512 KV heads of 4096 positions, so 70.2; 128 of 8192 77.5 / 69.7; 4 of 3000 34.9 / 30.9.
template <class T, int DH, int G>
__device__ __forceinline__ void attend_rows_group(const char* K_head, const char* V_head, const int* list, int n_begin, int n_end,
                                                  const float (&q8)[G][8], int lane, int wave, float (&m_run)[G], float (&l_run)[G],
                                                  float (&acc)[G][8]) {
  using Geo = RowGeometry<DH>;
  constexpr int UNR = 2, GROUP = Geo::RPI * UNR;
  const int slot = wave * Geo::RPW + lane / Geo::LPR;
  const int n_groups = (n_end - n_begin + GROUP - 1) / GROUP;
  auto issue = [&](uint4 (&kr)[UNR], uint4 (&vr)[UNR], int g) {
#pragma unroll
    for (int t = 0; t < UNR; ++t) {
      const int n = n_begin + g * GROUP + t * Geo::RPI + slot;
      const uint32_t off = (uint32_t)list[n < n_end ? n : n_end - 1] * (uint32_t)(DH * 2);
      kr[t] = load16(K_head + off);
      vr[t] = load16(V_head + off);
    }
  };
  auto consume = [&](const uint4 (&kr)[UNR], const uint4 (&vr)[UNR], int g) {
    const int n0 = n_begin + g * GROUP + slot;             // row t of the lane is n0 + t RPI
    float kf[UNR][8], vf[UNR][8];
#pragma unroll
    for (int t = 0; t < UNR; ++t) { unpack8<T>(kr[t], kf[t]); unpack8<T>(vr[t], vf[t]); }
#pragma unroll
    for (int h = 0; h < G; ++h) {
      float dot[UNR], m_new = m_run[h];
#pragma unroll
      for (int t = 0; t < UNR; ++t) {
        dot[t] = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) dot[t] = fmaf(kf[t][e], q8[h][e], dot[t]);
        dot[t] = lanes_sum<Geo::LPR>(dot[t]);
        m_new = n0 + t * Geo::RPI < n_end ? fmaxf(m_new, dot[t]) : m_new;
      }
      if (n0 < n_end) {
        const float sc = exp2_weight(m_run[h] - m_new);
        l_run[h] *= sc;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[h][e] *= sc;
#pragma unroll
        for (int t = 0; t < UNR; ++t) {
          if (n0 + t * Geo::RPI < n_end) {
            const float pr = exp2_weight(dot[t] - m_new);
            l_run[h] += pr;
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[h][e] = fmaf(pr, vf[t][e], acc[h][e]);
          }
        }
        m_run[h] = m_new;
      }
    }
  };
  if (n_groups > 0) {
    uint4 ka[UNR], va[UNR], kb[UNR], vb[UNR];
    issue(ka, va, 0);
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
  }
}

}  // namespace sparq
