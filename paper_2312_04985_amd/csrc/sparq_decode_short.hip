// The one-workgroup-per-head kernel for short caches of many units: workgroups of four waves, four of them on a CU.
#define SPARQ_WAVES 4
#include "sparq_decode_fused.h"

namespace sparq {

namespace {

template <class T, int DH, bool APPEND>
hipError_t launch_one(const DecodeArgs& a, hipStream_t s) {
  const size_t lds = fused_lds_bytes(a.S_max, DH);
  hipError_t e = allow_lds<sparq_decode_fused<T, DH, APPEND, false, false>>(lds);
  if (e != hipSuccess) return e;
  DecodeArgs d = a;
  d.append_apart = APPEND && append_apart((int64_t)a.B * a.H);
  hipLaunchKernelGGL((sparq_decode_fused<T, DH, APPEND, false, false>), dim3(a.B * a.H + (d.append_apart ? append_workgroups<DH>((int64_t)a.B * a.H_kv) : 0)), dim3(NT), lds, s, d);
  return hipGetLastError();
}

template <bool APPEND>
hipError_t launch_any(const DecodeArgs& a, int dtype, hipStream_t s) {
  const bool bf = dtype == 1;
  switch (a.d_h) {
    case 64:  return bf ? launch_one<BF16, 64, APPEND>(a, s) : launch_one<F16, 64, APPEND>(a, s);
    case 128: return bf ? launch_one<BF16, 128, APPEND>(a, s) : launch_one<F16, 128, APPEND>(a, s);
    case 256: return bf ? launch_one<BF16, 256, APPEND>(a, s) : launch_one<F16, 256, APPEND>(a, s);
    default:  return hipErrorInvalidValue;
  }
}

}  // namespace

// More units than run at once in workgroups of eight waves (two per CU), as long as four of these fit the LDS of a CU and a unit's
// reads do not bind the call: a unit is a chain of serial stages, so that twice as many units under way hide twice as much of it;
// with much to read both wait for the memory.  us per step, eight waves / four, 128 channels, r 32 unless said: 2048 heads at 200
// positions 48.1 / 28.1, 500 49.3 / 32.9, 1020 (k 128) 58.4 / 47.5, 1500 64.9 / 57.6, 1800 with k 256 84.5 / 82.3, 3000 105.6 / 104.7,
// 4090 with k 512 (524 KB per unit) 165.2 / 166.3; r 16 at 2500 61.2 / 45.9; of 64 channels, r 16, at 4700 82.1 / 72.6; of 256, r 64, 1024 heads at 1500
// 58.6 / 56.6; 544 heads at 1000 24.8 / 18.2, 512 16.8 / 16.7, 256 13.0 / 13.0.
bool decode_short(const DecodeArgs& a) {
  if ((a.flags & 64u) || (int64_t)a.B * a.H <= 512) return false;      // (not for the tiled layout)
  const int64_t reads = (int64_t)a.S_max * a.r * 2 + (int64_t)(a.k < a.S_max ? a.k : a.S_max) * a.d_h * 4;
  return 4 * fused_lds_bytes(a.S_max, a.d_h) <= 160 * 1024 && reads <= 350000;
}

hipError_t launch_decode_short(const DecodeArgs& a, int dtype, hipStream_t s) {
  return a.k_new ? launch_any<true>(a, dtype, s) : launch_any<false>(a, dtype, s);
}

}  // namespace sparq
