// Launches of the one-workgroup-per-head kernel.
#include "sparq_decode_fused.h"

namespace sparq {

namespace {

// Whether a step's append has workgroups of its own.  At the end of a decoding workgroup its stores hold the place on the CU
// until the memory has taken them; where more workgroups wait for it, that adds up over the rounds, most of all in the steps
// that complete a group of 8 (d_h 16-byte stores to as many lines per KV head).  Where all run at once, or in two rounds,
// nobody waits for the last stores of a workgroup, and the others would only begin then.  us per step, in the decoding
// workgroups / apart, at 4096 positions of 128 channels, k = 512, a step that completes a group and one that does not: 512 units
// 47.5 / 52.1 and 44.3 / 45.5; 1024 94.1 / 95.0 and 86.4 / 86.4; 1536 143.2 / 141.2; 2048 189.4 / 182.8 and 169.4 / 168.4;
// 2048 at 8192 positions, k = 256, 162.6 / 146.5 and 137.8 / 131.0.
// (The append's workgroups in front of the decoding ones, or a quarter, half or three quarters into the grid: 2-11 % more.)
constexpr bool append_apart(int64_t units) { return units > 1024; }

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

size_t decode_lds_bytes(int S_max, int d_h) {
  return 4 * ((size_t)S_max + 2 * kRadixBins + (size_t)NW * (d_h + 2) + 5 * (size_t)d_h + 32 + 16 + 8);
}

hipError_t launch_decode(const DecodeArgs& a, int dtype, hipStream_t s) {
  if (decode_helped(a)) return launch_decode_helped(a, dtype, s);
  if (a.flags & 64u) return a.k_new ? launch_any<true, true>(a, dtype, s) : launch_any<false, true>(a, dtype, s);
  return a.k_new ? launch_any<true, false>(a, dtype, s) : launch_any<false, false>(a, dtype, s);
}

}  // namespace sparq
