// Launches of the one-workgroup-per-head kernel.
#include "sparq_decode_fused.h"

namespace sparq {

namespace {

template <class T, int DH, bool APPEND, bool TILED>
hipError_t launch_one(const DecodeArgs& a, hipStream_t s) {
  const size_t lds = decode_lds_bytes(a.S_max, DH);
  hipError_t e = allow_lds<sparq_decode_fused<T, DH, APPEND, TILED, false>>(lds);
  if (e != hipSuccess) return e;
  DecodeArgs d = a;
  d.append_apart = APPEND && append_apart((int64_t)a.B * a.H);
  hipLaunchKernelGGL((sparq_decode_fused<T, DH, APPEND, TILED, false>), dim3(a.B * a.H + (d.append_apart ? append_workgroups<DH>((int64_t)a.B * a.H_kv) : 0)), dim3(NT), lds, s, d);
  return hipGetLastError();
}

template <bool APPEND, bool TILED>
hipError_t launch_any(const DecodeArgs& a, int dtype, hipStream_t s) {
  const bool bf = dtype == 1;
  switch (a.d_h) {
    case 64:  return bf ? launch_one<BF16, 64, APPEND, TILED>(a, s) : launch_one<F16, 64, APPEND, TILED>(a, s);
    case 128: return bf ? launch_one<BF16, 128, APPEND, TILED>(a, s) : launch_one<F16, 128, APPEND, TILED>(a, s);
    case 256: return bf ? launch_one<BF16, 256, APPEND, TILED>(a, s) : launch_one<F16, 256, APPEND, TILED>(a, s);
    default:  return hipErrorInvalidValue;
  }
}

}  // namespace

size_t decode_lds_bytes(int S_max, int d_h) { return fused_lds_bytes(S_max, d_h); }

hipError_t launch_decode(const DecodeArgs& a, int dtype, hipStream_t s) {
  if (decode_helped(a)) return launch_decode_helped(a, dtype, s);
  if (decode_short(a)) return launch_decode_short(a, dtype, s);
  if (a.flags & 64u) return a.k_new ? launch_any<true, true>(a, dtype, s) : launch_any<false, true>(a, dtype, s);
  return a.k_new ? launch_any<true, false>(a, dtype, s) : launch_any<false, false>(a, dtype, s);
}

}  // namespace sparq
