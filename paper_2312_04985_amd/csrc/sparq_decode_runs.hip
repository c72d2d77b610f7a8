// The one-workgroup-per-head kernel for row strides of Kt near a multiple of 32 KiB: the waves of a workgroup read an eighth of the row apart.
#include "sparq_decode_fused.h"

namespace sparq {

// Side by side, the workgroup advancing 8 KB of every row at a time, all requests of a moment lie at one offset of rows whose
// stride is 32 KiB or nearly.  us per decode, side by side / apart, 128 channels, r 32, k 512 unless said:
// Strides of 16 320, 16 448, 32 640, 32 704, 32 832, 32 896 positions are up to 28 % faster, whatever the units, groups, r and d_h: 256 heads at 16 320 63.5 / 56.9,
// 16 448 62.6 / 58.0, 32 640 105.2 / 99.8, 32 896 107.8 / 102.2; 512 on 128 KV heads at 16 320 93.6 / 81.1, 16 448 96.0 / 83.6; 256 on 128, r 64, at 16 320 102.7 / 80.3;
// 160 of 64 channels, r 16, at 16 320 28.5 / 25.6; 512 of 256, r 64, 264.1 / 247.8; the least with r 8 at 32 704: equal.
// Exact multiples, 512 KV heads and more: 16 384 120.2 / 108.7, r 16 64.6 / 63.0, r 64 220.8 / 185.1; 64 channels, r 16, 60.9 / 58.2, r 48 159.4 / 139.9; 256, r 64, equal; with r 8
// equal.  With fewer KV heads it goes either way: 160 heads 46.6 / 52.5, 192 with r 48 69.9 / 72.5 and with r 64 90.9 / 73.2, 256 of 64 channels, r 16, 31.7 / 34.7, on
// 128 KV heads 30.2 / 37.0.
// Everywhere else as fast or slower (14 336 52.3 / 56.1, 18 432 on 128 KV heads 88.2 / 93.6, 33 024 109.2 / 113.3, 8256 67.2 / 68.0).
// In a build of its own, as the append's workgroups.
bool decode_runs(const DecodeArgs& a) {
  if ((a.flags & 64u) || a.S_max <= 2 * 8 * kDecodeThreads) return false;       // (not for the tiled layout; up to two chunks per thread)
  const int m = (a.S_stride + 8192) / 16384, off = a.S_stride - m * 16384;
  if (m > 2) return false;
  if (off == 0) return a.r >= 16 && (int64_t)a.B * a.H_kv >= 512;
  return off <= 64 * m && -off <= 64 * m;
}

hipError_t launch_decode_runs(const DecodeArgs& a, int dtype, hipStream_t s) {
  const int units = a.B * a.H;
  if (!a.k_new) return launch_fused<false, false, false, false, true>(a, dtype, units, s);
  if (!decode_apart(a)) return launch_fused<true, false, false, false, true>(a, dtype, units, s);
  return launch_fused<true, false, false, true, true>(a, dtype, units + append_workgroups((int64_t)a.B * a.H_kv, a.d_h), s);
}

}  // namespace sparq
