// Launches of the one-workgroup-per-head kernel.
#include "sparq_decode_fused.h"

namespace sparq {

size_t decode_lds_bytes(int S_max, int d_h) { return fused_lds_bytes(S_max, d_h); }

hipError_t launch_decode(const DecodeArgs& a, int dtype, hipStream_t s) {
  if (decode_helped(a)) return launch_decode_helped(a, dtype, s);
  if (decode_short(a)) return launch_decode_short(a, dtype, s);
  if (decode_runs(a)) return launch_decode_runs(a, dtype, s);
  if (a.k_new && decode_apart(a)) return launch_step_apart(a, dtype, s);
  const int units = a.B * a.H;
  if (a.flags & 64u) return a.k_new ? launch_fused<true, true, false, false, false>(a, dtype, units, s) : launch_fused<false, true, false, false, false>(a, dtype, units, s);
  return a.k_new ? launch_fused<true, false, false, false, false>(a, dtype, units, s) : launch_fused<false, false, false, false, false>(a, dtype, units, s);
}

}  // namespace sparq
