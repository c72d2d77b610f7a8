// The one-workgroup-per-head kernel for short caches of many units: workgroups of four waves, four of them on a CU.
#define SPARQ_WAVES 4
#include "sparq_decode_fused.h"

namespace sparq {

// More units than run at once in workgroups of eight waves (two per CU), as long as four of these fit the LDS of a CU and a unit's
// reads do not bind the call: a unit is a chain of serial stages, so that twice as many units under way hide twice as much of it;
// with much to read both wait for the memory.  us per step, eight waves / four, 128 channels, r 32 unless said: 2048 heads at 200
// positions 48.1 / 28.1, 500 49.3 / 32.9, 1020 (k 128) 58.4 / 47.5, 1500 64.9 / 57.6, 1800 with k 256 84.5 / 82.3, 3000 105.6 / 104.7,
// 4090 with k 512 (524 KB per unit) 165.2 / 166.3; r 16 at 2500 61.2 / 45.9; of 64 channels, r 16, at 4700 82.1 / 72.6; of 256, r 64, 1024 heads at 1500
// 58.6 / 56.6; 544 heads at 1000 24.8 / 18.2, 512 16.8 / 16.7, 256 13.0 / 13.0.
// A step appends in the decoding workgroups, whatever their number (decode_apart is for the build of eight waves).  us per step so / in
// workgroups of the append's own, a step that completes a group of 8 positions and one that does not: 1536 heads at 200 28.8 / 32.7 and 23.4 /
// 23.7, 2048 34.7 / 36.6 and 26.0 / 26.6, 3072 48.9 / 53.6 and 37.5 / 37.8; 1536 at 1000 35.7 / 39.4 and 26.4 / 27.1, 2048 41.2 / 42.2 and 29.6 /
// 30.1, 3072 62.0 / 61.1 and 43.5 / 42.8; 2048 on 512 KV heads at 1000 31.4 / 30.1 and 26.8 / 26.9.
bool decode_short(const DecodeArgs& a) {
  if ((a.flags & 64u) || (int64_t)a.B * a.H <= 512) return false;      // (not for the tiled layout)
  const int64_t reads = (int64_t)a.S_max * a.r * 2 + (int64_t)(a.k < a.S_max ? a.k : a.S_max) * a.d_h * 4;
  return 4 * fused_lds_bytes(a.S_max, a.d_h) <= 160 * 1024 && reads <= 350000;
}

hipError_t launch_decode_short(const DecodeArgs& a, int dtype, hipStream_t s) {
  const int units = a.B * a.H;
  return a.k_new ? launch_fused<true, false, false, false, false>(a, dtype, units, s) : launch_fused<false, false, false, false, false>(a, dtype, units, s);
}

}  // namespace sparq
