// Dense single-query attention (Section 3, Eq. 2): the in-library comparison for SparQ.
// Split along the sequence: each workgroup streams a run of K and V rows of one KV head once
// for G query heads of its group (online softmax, fp32).  The last of a KV head's workgroups to finish merges their
// partial results.
#include "common.h"
#include "params.h"

namespace sparq {

namespace {

constexpr int DT = 256;            // threads per workgroup; two workgroups per CU (256 registers)
constexpr int DW = DT / kWave;

// A wave takes groups of TPG tiles of 16 rows, two groups in flight.  The scores of a tile are one chain of matrix
// instructions (16 rows x 16 query heads, of which G are distinct: the heads repeat), which leaves every lane the
// scores of one row; the softmax then costs one exponential per (row, head) instead of one in each of the d_h / 8
// lanes that share a row, and the running maximum is looked at once per group: the accumulators are rescaled only
// when it rises.  The weights go through LDS to the lanes that hold the row's slice of V, as fp32, and V is
// accumulated by plain fp32 FMAs.  Products of 16-bit inputs are exact in the matrix unit and summed in fp32.
// Bound by HBM.  Measured (before: scores by FMAs and lane sums, two exponentials and a rescaling per row, head and lane,
// and a second launch for the merge): 8 KV heads of 32 768 rows, 4 query heads each, bf16 44.2 -> 26.9 us (134 MB); 64 KV heads
// of 8192 rows, 8 heads each 120 -> 53; 512 KV heads of 4096 rows, one head each 170 -> 157 (6.8 TB/s); one row group of one
// head 9.5 -> 7.6.  Registers decide: with twice the rows per group and four copies of the group's code in every
// instance, f16 with 4 and 8 heads went to scratch memory (64 KV heads of 5000 rows, 4 heads 47 us, now 31; 8 heads 68, now 39).
template <class T, int DH, int G>
struct DenseGeometry {
  static constexpr int LPR = DH / 8, RPW = kWave / LPR;      // lanes per row of V, rows per load of a wave
  static constexpr int KK = DH / 32;                         // matrix instructions (16-byte pieces per lane) per tile
  static constexpr int TPG = DH == 64 ? 2 : 1;               // two groups of 4 to 8 KB of K in flight fit the registers
  static constexpr bool TIGHT = G == 8 || (G == 4 && DH == 256);   // ... with two copies of the group's code and no more
  static constexpr int R = 16 * TPG;                         // rows per group
  static constexpr int NV = R / RPW;                         // loads of V per group
  static constexpr int NH = G < 4 ? G : 4;                   // scores of a row that one lane holds
};

template <class T>
__device__ __forceinline__ void store_out4(uint16_t* dst, const float4& y, float scale) {
  const uint32_t lo = T::narrow(y.x * scale) | ((uint32_t)T::narrow(y.y * scale) << 16);
  const uint32_t hi = T::narrow(y.z * scale) | ((uint32_t)T::narrow(y.w * scale) << 16);
  *reinterpret_cast<uint2*>(dst) = make_uint2(lo, hi);
}

template <class T, int DH, int G>
__global__ __launch_bounds__(DT, 2) void dense_partial(const DenseArgs a) {
  using Geo = DenseGeometry<T, DH, G>;
  constexpr int LPR = Geo::LPR, RPW = Geo::RPW, KK = Geo::KK, TPG = Geo::TPG, R = Geo::R, NV = Geo::NV, NH = Geo::NH;
  __shared__ __align__(16) float ps[DW][R][G];   // weights of a wave's group of rows
  __shared__ float part[DW][G][DH + 2];
  __shared__ float stat[kDenseSplits * G * 2];      // the last workgroup's merge: (max, denominator) of every partial
  __shared__ float4 red[DT];
  __shared__ int ticket;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = a.H / a.H_kv, gpk = dense_bundles(g, DH), per = (g + gpk - 1) / gpk;   // bundles per KV head, heads of a bundle
  // Workgroups are dealt round-robin to the 8 XCDs: the KV head varies fastest and the split slowest, so that every XCD gets
  // its share of the splits at the ends of the sequences, which a ragged batch leaves empty; the bundles of a KV head, which
  // read the same rows, are 8 apart and share an XCD's L2.
  const int heads = a.B * a.H_kv, pairs = heads * a.n_split;      // pairs: (KV head, split)
  const int chunk = blockIdx.x / (8 * gpk), in_chunk = blockIdx.x - chunk * 8 * gpk;   // 8 pairs, or what is left of them
  const int width = pairs - chunk * 8 < 8 ? pairs - chunk * 8 : 8, bundle = in_chunk / width;
  const int pair = chunk * 8 + in_chunk - bundle * width, split = pair / heads, head = pair - split * heads;
  const int unit = head * gpk + bundle;          // (sequence, KV head, bundle)
  const int hk = head % a.H_kv, b = head / a.H_kv;
  const int h0 = hk * g + bundle * per;          // first query head served here
  const int n_heads = g - bundle * per < per ? g - bundle * per : per;   // <= G; the others repeat the last one
  int S = a.seq_lens[b];
  S = S < 0 ? 0 : (S > a.S_max ? a.S_max : S);
  const int s0 = split * a.rows_per_split;
  const int s1 = (s0 + a.rows_per_split) < S ? (s0 + a.rows_per_split) : S;
  uint16_t* out = reinterpret_cast<uint16_t*>(a.out) + ((size_t)b * a.H + h0) * DH;
  if (s0 >= S) {                                 // nothing of this sequence here; an empty sequence: zeros
    if (S == 0 && split == 0)
      for (int i = tid; i < n_heads * DH; i += DT) out[i] = 0;
    return;
  }
  const int n_live = (S + a.rows_per_split - 1) / a.rows_per_split;   // workgroups of this unit that have rows

  const size_t kv_head = (size_t)b * a.H_kv + hk;
  const int row16 = lane & 15, quarter = lane >> 4;
  const int sub = lane % LPR, vrow = lane / LPR;
  // This run of rows.  Offsets inside it fit 32 bits, those inside a whole head need not: a run is the (units x n_split)-th
  // part of K, and dense_plan's smallest such product is 128.
  const char* K_run = reinterpret_cast<const char*>(a.K) + (kv_head * a.S_stride + s0) * (size_t)(DH * 2);
  const char* V_run = reinterpret_cast<const char*>(a.V) + (kv_head * a.S_stride + s0) * (size_t)(DH * 2);
  const int q_row = row16 % G < n_heads ? row16 % G : n_heads - 1;
  const uint16_t* qp = reinterpret_cast<const uint16_t*>(a.q) + ((size_t)b * a.H + h0 + q_row) * DH + quarter * 8;
  uint4 qf[KK];                                  // row (lane % 16) % G of the query, channels 32 kk + 8 quarter ..
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) qf[kk] = *reinterpret_cast<const uint4*>(qp + kk * 32);
  const float qscale = kLog2e / sqrtf((float)DH);
  float acc[G][8], m_ref[NH], l_run[NH];
#pragma unroll
  for (int t = 0; t < G; ++t)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[t][e] = 0.0f;
#pragma unroll
  for (int i = 0; i < NH; ++i) { m_ref[i] = -INFINITY; l_run[i] = 0.0f; }

  auto issue = [&](uint4 (&kr)[TPG][KK], uint4 (&vr)[NV], int r0) {
#pragma unroll
    for (int t = 0; t < TPG; ++t) {
      const int n = r0 + t * 16 + row16;
      const uint32_t off = (uint32_t)(n < s1 ? n - s0 : 0) * (uint32_t)(DH * 2) + quarter * 16;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) kr[t][kk] = load16(K_run + off + kk * 64);
    }
#pragma unroll
    for (int u = 0; u < NV; ++u) {
      const int n = r0 + u * RPW + vrow;
      vr[u] = load16(V_run + ((uint32_t)(n < s1 ? n - s0 : 0) * (uint32_t)(DH * 2) + sub * 16));
    }
  };
  auto consume = [&](const uint4 (&kr)[TPG][KK], const uint4 (&vr)[NV], int r0) {
    float sc[TPG][NH];                           // scores of row r0 + 16 t + lane % 16, heads (4 quarter + i) % G
    bool above = false;
#pragma unroll
    for (int t = 0; t < TPG; ++t) {
      f32x4 c = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) c = T::mfma_16x16x32(qf[kk], kr[t][kk], c);
      const bool ok = r0 + t * 16 + row16 < s1;
#pragma unroll
      for (int i = 0; i < NH; ++i) {
        sc[t][i] = ok ? c[i] * qscale : -INFINITY;
        above = above || sc[t][i] > m_ref[i];
      }
    }
    if (__ballot(above)) {                       // the maximum of some head rises: uniform, rare after the first groups
      float w[NH];
#pragma unroll
      for (int i = 0; i < NH; ++i) {
        float mx = sc[0][i];
#pragma unroll
        for (int t = 1; t < TPG; ++t) mx = fmaxf(mx, sc[t][i]);
        mx = fmaxf(group_max<16>(mx), m_ref[i]);
        w[i] = weight_exp2(m_ref[i], mx);
        m_ref[i] = mx;
        l_run[i] *= w[i];
      }
#pragma unroll
      for (int t = 0; t < G; ++t) {
        const float wt = lane_f(w[t % NH], t / NH * 16);      // head t lives in quarter t / 4
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[t][e] *= wt;
      }
    }
#pragma unroll
    for (int t = 0; t < TPG; ++t) {
      float p[NH];
#pragma unroll
      for (int i = 0; i < NH; ++i) { p[i] = exp2_weight(sc[t][i] - m_ref[i]); l_run[i] += p[i]; }
      if (quarter < (G + 3) / 4) {               // the other quarters hold copies
#pragma unroll
        for (int i = 0; i < NH; ++i) ps[wave][t * 16 + row16][quarter * 4 + i] = p[i];
      }
    }
    wave_lds_fence();
#pragma unroll
    for (int u = 0; u < NV; ++u) {
      float f[8], w[G];
#pragma unroll
      for (int t = 0; t < G; ++t) w[t] = ps[wave][u * RPW + vrow][t];
      unpack8<T>(vr[u], f);
#pragma unroll
      for (int t = 0; t < G; ++t)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[t][e] = fmaf(w[t], f[e], acc[t][e]);
    }
    wave_lds_fence();                            // the next group overwrites the weights
  };

  int r0 = s0 + wave * R;
  if (r0 < s1) {
    uint4 ka[TPG][KK], va[NV], kb[TPG][KK], vb[NV];
    issue(ka, va, r0);
    if constexpr (Geo::TIGHT) {
      for (;;) {                                 // (past the end of the run the loads repeat its first row, and nothing uses them)
        const int r1 = r0 + DW * R;
        issue(kb, vb, r1);
        consume(ka, va, r0);
        if (r1 >= s1) break;
        r0 = r1 + DW * R;
        issue(ka, va, r0);
        consume(kb, vb, r1);
        if (r0 >= s1) break;
      }
    } else {
      for (;;) {
        const int r1 = r0 + DW * R, r2 = r1 + DW * R;
        if (r1 >= s1) { consume(ka, va, r0); break; }
        issue(kb, vb, r1);
        consume(ka, va, r0);
        if (r2 >= s1) { consume(kb, vb, r1); break; }
        issue(ka, va, r2);
        consume(kb, vb, r1);
        r0 = r2;
      }
    }
  }
  // merge the row groups of a wave (they share the reference maximum), then the waves, per query head
#pragma unroll
  for (int t = 0; t < G; ++t) {
#pragma unroll
    for (int o = LPR; o < kWave; o <<= 1)
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[t][e] += __shfl_xor(acc[t][e], o);
    if (lane < LPR) {
#pragma unroll
      for (int e = 0; e < 8; ++e) part[wave][t][sub * 8 + e] = acc[t][e];
    }
  }
#pragma unroll
  for (int i = 0; i < NH; ++i) {
    const float l = group_sum<16>(l_run[i]);
    if (row16 == 0 && quarter < (G + 3) / 4) { part[wave][quarter * 4 + i][DH] = m_ref[i]; part[wave][quarter * 4 + i][DH + 1] = l; }
  }
  __syncthreads();
  // partial (y, m, l) of this workgroup: 4 channels of a head per thread
  constexpr int SLOTS = G * DH / 4, GRPS = DT / SLOTS;
  static_assert(GRPS >= 1, "a slot of 4 channels per thread");
  const int slot = tid % SLOTS, grp = tid / SLOTS, t_s = slot / (DH / 4), c_s = slot % (DH / 4) * 4;
  const int slots = n_heads * (DH / 4);          // the slots of real heads come first
  float4 y4 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  float m_all = -INFINITY, l_all = 0.0f;
  const size_t first = ((size_t)b * a.H + h0) * a.n_split;
  const float* y_parts = a.partials + first * DH;                                           // [n_split][n_heads][DH]
  float* s_parts = a.partials + (size_t)a.B * a.H * a.n_split * DH + first * 2;             // [n_split][n_heads][2]
  if (grp == 0 && slot < slots) {
#pragma unroll
    for (int w = 0; w < DW; ++w) m_all = fmaxf(m_all, part[w][t_s][DH]);
#pragma unroll
    for (int w = 0; w < DW; ++w) {
      const float s = weight_exp2(part[w][t_s][DH], m_all);
      const float* y = &part[w][t_s][c_s];
      l_all += part[w][t_s][DH + 1] * s;
      y4.x += y[0] * s; y4.y += y[1] * s; y4.z += y[2] * s; y4.w += y[3] * s;
    }
    if (n_live == 1) {                           // (a denominator that is no positive number: zeros)
      if (!(l_all > 0.0f)) { y4 = make_float4(0.0f, 0.0f, 0.0f, 0.0f); l_all = 1.0f; }
      store_out4<T>(out + slot * 4, y4, 1.0f / l_all);
    } else {
      store_agent4(y_parts, (uint32_t)(split * slots + slot) * 16, y4);
      if (c_s == 0) { store_agent(s_parts + (split * n_heads + t_s) * 2, m_all); store_agent(s_parts + (split * n_heads + t_s) * 2 + 1, l_all); }
    }
  }
  if (n_live == 1) return;
  if (!last_to_arrive(a.tickets + unit, n_live, &ticket)) return;
  // the merge: the partials of a channel are shared by GRPS threads, eight in flight each; n_live <= kDenseSplits
  constexpr int FLY = 8;
  float4 v[FLY];
  auto fetch = [&](int s0) {
#pragma unroll
    for (int j = 0; j < FLY; ++j) {
      const int s = s0 + j * GRPS;
      v[j] = load_agent4(y_parts, (uint32_t)((s < n_live ? s : 0) * slots + (slot < slots ? slot : 0)) * 16);
    }
  };
  fetch(grp);
  for (int i = tid; i < n_live * n_heads; i += DT) { stat[i * 2] = load_agent(s_parts + i * 2); stat[i * 2 + 1] = load_agent(s_parts + i * 2 + 1); }
  __syncthreads();
  for (int t = wave; t < n_heads; t += DW) {           // two partials per lane: their weights, with the denominator in them
    float m[2], l[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int p = (lane + j * kWave) * n_heads + t;
      const bool on = lane + j * kWave < n_live;
      m[j] = on ? stat[p * 2] : -INFINITY; l[j] = on ? stat[p * 2 + 1] : 0.0f;
    }
    const float m_max = wave_max(fmaxf(m[0], m[1]));
    const float w0 = weight_exp2(m[0], m_max), w1 = weight_exp2(m[1], m_max);
    const float l_sum = wave_sum(l[0] * w0 + l[1] * w1);
    if (lane < n_live) stat[(lane * n_heads + t) * 2] = w0 / l_sum;
    if (lane == 0) stat[t * 2 + 1] = l_sum;
    if (lane + kWave < n_live) stat[((lane + kWave) * n_heads + t) * 2] = w1 / l_sum;
  }
  __syncthreads();
  y4 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  for (int s0 = grp;;) {
#pragma unroll
    for (int j = 0; j < FLY; ++j) {
      const int s = s0 + j * GRPS;
      const float w = s < n_live ? stat[(s * n_heads + t_s) * 2] : 0.0f;
      if (s < n_live) { y4.x += v[j].x * w; y4.y += v[j].y * w; y4.z += v[j].z * w; y4.w += v[j].w * w; }
    }
    s0 += FLY * GRPS;
    if (s0 - grp >= n_live) break;
    fetch(s0);
  }
  if (GRPS > 1) {
    red[tid] = y4;
    __syncthreads();
    if (grp == 0) {
#pragma unroll
      for (int k = 1; k < GRPS; ++k) {
        const float4 o = red[k * SLOTS + slot];
        y4.x += o.x; y4.y += o.y; y4.z += o.z; y4.w += o.w;
      }
    }
  }
  if (!(stat[t_s * 2 + 1] > 0.0f)) y4 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  if (grp == 0 && slot < slots) store_out4<T>(out + slot * 4, y4, 1.0f);
}

template <class T, int DH, int G>
hipError_t launch_g(const DenseArgs& a, hipStream_t s) {
  const int blocks = a.B * a.H_kv * dense_bundles(a.H / a.H_kv, DH) * a.n_split;
  hipLaunchKernelGGL((dense_partial<T, DH, G>), dim3(blocks), dim3(DT), 0, s, a);
  return hipGetLastError();
}

template <class T, int DH>
hipError_t launch_dh(const DenseArgs& a, hipStream_t s) {
  switch (dense_width(a.H / a.H_kv, DH)) {
    case 8:
      if constexpr (DH <= 128) return launch_g<T, DH, 8>(a, s);
      return hipErrorInvalidValue;
    case 4: return launch_g<T, DH, 4>(a, s);
    case 2: return launch_g<T, DH, 2>(a, s);
    default: return launch_g<T, DH, 1>(a, s);
  }
}

}  // namespace

hipError_t launch_dense(const DenseArgs& a, int dtype, hipStream_t s) {
  const bool bf = dtype == 1;
  switch (a.d_h) {
    case 64:  return bf ? launch_dh<BF16, 64>(a, s) : launch_dh<F16, 64>(a, s);
    case 128: return bf ? launch_dh<BF16, 128>(a, s) : launch_dh<F16, 128>(a, s);
    case 256: return bf ? launch_dh<BF16, 256>(a, s) : launch_dh<F16, 256>(a, s);
    default:  return hipErrorInvalidValue;
  }
}

}  // namespace sparq
