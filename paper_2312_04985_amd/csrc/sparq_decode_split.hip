// The last launch of the grouped-query plan over several workgroups per KV head: one workgroup per query head merges
// the partial results of the gather, blends with the mean value vector (Eq. 10) and stores.
#include "decode_stages.h"

namespace sparq {

namespace {

template <class T, int DH>
__global__ __launch_bounds__(DH) void split_combine(const SplitArgs a) {
  const DecodeArgs& d = a.d;
  const int u = blockIdx.x, c = threadIdx.x;
  const int b = divided(u, d.by_H), h = u - b * d.H;
  const size_t kv_head = (size_t)b * d.H_kv + divided(h, d.by_group);
  const int S = d.seq_lens[b];
  if (S <= 0) return;                      // outputs written by the plan's first launch
  // all partials of this channel in flight at once (n_split <= kMaxSplit)
  const float* parts = a.part_ws + (size_t)u * a.n_split * (DH + 2);
  float pm[kMaxSplit], pl[kMaxSplit], py[kMaxSplit];
#pragma unroll
  for (int w = 0; w < kMaxSplit; ++w) {
    const bool on = w < a.n_split;
    pm[w] = on ? parts[w * (DH + 2) + DH] : -INFINITY;
    pl[w] = on ? parts[w * (DH + 2) + DH + 1] : 0.0f;
    py[w] = on ? parts[w * (DH + 2) + c] : 0.0f;
  }
  const float alpha = a.alpha_ws[u];
  const float vm = d.v_mean[kv_head * DH + c];
  float m_all = -INFINITY;
#pragma unroll
  for (int w = 0; w < kMaxSplit; ++w) m_all = fmaxf(m_all, pm[w]);
  float l_all = 0.0f, y3 = 0.0f;
#pragma unroll
  for (int w = 0; w < kMaxSplit; ++w) {
    const float sw = weight_exp2(pm[w], m_all);
    l_all += pl[w] * sw;
    y3 += py[w] * sw;
  }
  y3 /= l_all;
  float y = y3;
  if (!(d.flags & 1u)) y = alpha * y3 + (1.0f - alpha) * vm;
  reinterpret_cast<uint16_t*>(d.out)[(size_t)u * DH + c] = T::narrow(y);
}

}  // namespace

template <class T, int DH>
hipError_t launch_combine_only(const SplitArgs& a, hipStream_t s) {
  hipLaunchKernelGGL((split_combine<T, DH>), dim3(a.d.B * a.d.H), dim3(DH), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_split_combine(const SplitArgs& a, int dtype, hipStream_t s) {
  const bool bf = dtype == 1;
  switch (a.d.d_h) {
    case 64:  return bf ? launch_combine_only<BF16, 64>(a, s) : launch_combine_only<F16, 64>(a, s);
    case 128: return bf ? launch_combine_only<BF16, 128>(a, s) : launch_combine_only<F16, 128>(a, s);
    case 256: return bf ? launch_combine_only<BF16, 256>(a, s) : launch_combine_only<F16, 256>(a, s);
    default:  return hipErrorInvalidValue;
  }
}

}  // namespace sparq
