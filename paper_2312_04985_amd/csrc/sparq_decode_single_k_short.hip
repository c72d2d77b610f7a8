// The kernel for a key cache stored once in workgroups of four waves, four of them on a CU: short caches of many units.
#define SPARQ_WAVES 4
#include "sparq_decode_single_k.h"

namespace sparq {

// As decode_short, by what a unit reads: its key rows whole and the selected ones.  us per decode, eight waves / four, 2048 heads of 128
// channels, k 64: 64 positions 41.2 / 23.0, 200 48.5 / 33.8, 500 66.3 / 53.7; k 128: 1000 103.7 / 101.1, 1500 (449 KB per unit) 138.7 /
// 140.8, 2000 178 / 186; on 512 KV heads at 1000 74.9 / 69.2, 4000 195 / 233; of 64 channels at 1000 66.1 / 53.3, 2000 94.0 / 91.6; 3584
// on 896 KV heads at 314 positions, all of them selected, 113.2 / 79.9.
bool decode_single_k_short(const DecodeArgs& a) {
  const int64_t reads = ((int64_t)a.S_max * 2 + (int64_t)(a.k < a.S_max ? a.k : a.S_max) * 4) * a.d_h;
  return (int64_t)a.B * a.H > 512 && reads <= 330000;
}

hipError_t launch_decode_single_k_short(const DecodeArgs& a, int dtype, hipStream_t s) { return launch_1k_any(a, dtype, s); }

}  // namespace sparq
