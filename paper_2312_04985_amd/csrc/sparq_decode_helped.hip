// The one-workgroup-per-head kernel for few units, whose idle CUs fetch for the units' workgroups.
#include "sparq_decode_fused.h"

namespace sparq {

namespace {

// Workgroups of a unit, its own and those that fetch for it: one for each of the XCD's 32 CUs, at most 8 (of 32 heads at 4096
// positions, the caches in HBM: 4 per unit 16.7 us per decode, 8 16.8; at 12 200 positions 23.2 and 22.6).
int units_per_xcd(const DecodeArgs& a) { return (a.B * a.H + 7) / 8; }
int workgroups_per_unit(int per_xcd) { return 32 / per_xcd < 8 ? 32 / per_xcd : 8; }

template <class T, int DH, bool APPEND>
hipError_t launch_one(const DecodeArgs& a, hipStream_t s) {
  const size_t lds = decode_lds_bytes(a.S_max, DH);
  hipError_t e = allow_lds<sparq_decode_fused<T, DH, APPEND, false, true>>(lds);
  if (e != hipSuccess) return e;
  DecodeArgs d = a;
  d.per_xcd = units_per_xcd(a);
  d.by_xcd = make_divider(d.per_xcd);
  const int n = workgroups_per_unit(d.per_xcd);
  d.helpers = n - 1;
  hipLaunchKernelGGL((sparq_decode_fused<T, DH, APPEND, false, true>), dim3(8 * d.per_xcd * n), dim3(NT), lds, s, d);
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

// Where CUs are idle.  With three or more workgroups per unit (80 units) it is always faster but for the smallest calls, whose
// loads are all on their way at once; with two (128 units) as long as what the units read stays in the L2 of their
// XCD.  us per decode without / with helpers, caches in HBM (40 caches in turn) and in the memory-side cache (3 in turn): 32 heads at
// 1500 positions 12.7 / 11.6 and 12.0 / 11.1, 4096 18.3 / 15.9 and 17.5 / 14.8, 8192 23.2 / 19.3 and 22.7 / 17.6; 8 heads at 11 000 26.9 /
// 22.2 and 23.3 / 20.4; 16 of 256 channels at 4096 27.7 / 22.3 and 26.4 / 20.9; 72 at 12 000 31.4 / 27.5 and 29.2 / 22.9; 96 at 6500
// 25.8 / 24.9 and 23.5 / 19.2, at 10 000 30.7 / 31.9 and 27.6 / 27.0; 128 at 4096 20.5 / 19.7 and 19.9 / 17.7, at 8192 26.6 / 29.6 and
// 26.2 / 25.9.  The smallest calls gain in the first column and lose in the second: a step of one head at 1023 10.6 / 10.1 and 9.4 / 9.6, 56
// heads of 256 channels at 217 12.0 / 11.7 and 10.9 / 11.2, 64 at 300 10.5 / 10.0 and 9.6 / 9.8; 32 at 700 10.7 / 10.2 and 10.1 / 9.9, 64 at 500 11.6 /
// 10.9 and 10.7 / 10.5, 128 at 134 11.8 / 11.3 and 11.3 / 10.9.
bool decode_helped(const DecodeArgs& a) {
  const int64_t units = (int64_t)a.B * a.H;
  if ((a.flags & 64u) || units > 128) return false;      // (not for the tiled layout)
  if (a.S_max <= 1024 && units * a.S_max < 22000) return false;
  return workgroups_per_unit(units_per_xcd(a)) >= 3 || units * a.S_max <= 640 * 1024;
}

hipError_t launch_decode_helped(const DecodeArgs& a, int dtype, hipStream_t s) {
  return a.k_new ? launch_any<true>(a, dtype, s) : launch_any<false>(a, dtype, s);
}

}  // namespace sparq
