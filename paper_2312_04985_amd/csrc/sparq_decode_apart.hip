// The one-launch step of many units: its append has workgroups of its own, behind the decoding ones.
#include "sparq_decode_fused.h"

namespace sparq {

// At the end of a decoding workgroup the append's stores hold the place on the CU until the memory has taken them; where more
// workgroups wait for it, that adds up over the rounds, most of all in the steps
// that complete a group of 8 (d_h 16-byte stores to as many lines per KV head).  Where all run at once, or in two rounds,
// nobody waits for the last stores of a workgroup, and the others would only begin then.  us per step, in the decoding
// workgroups / apart, at 4096 positions of 128 channels, k = 512, a step that completes a group and one that does not: 512 units
// 47.5 / 52.1 and 44.3 / 45.5; 1024 94.1 / 95.0 and 86.4 / 86.4; 1536 143.2 / 141.2; 2048 189.4 / 182.8 and 169.4 / 168.4;
// 2048 at 8192 positions, k = 256, 162.6 / 146.5 and 137.8 / 131.0.
// Not with 512 KV heads or fewer, however many query heads: that is how many rows there are to append, and what is gained
// in the steps that complete a group is lost in the seven others: 1344 heads on 336 of 128 channels at 2100, k 700, 101.2 / 99.6 and 95.7 /
// 96.6; 2048 on 512 140.4 / 139.5 and 131.8 / 132.6; 2048 on 512 at 4100 139.4 / 135.3 and 129.2 / 129.7; 4096 on 512 of 64 channels at 6000, k 1000, 213.4 /
// 208.1 and 199.2 / 204.9.  (2048 on 1024 at 4100 167.1 / 155.7 and 147.8 / 147.4.)
// (The append's workgroups in front of the decoding ones, or a quarter, half or three quarters into the grid: 2-11 % more.
// In a build of its own because the code of the append's workgroups, in the kernel of all steps, took 0.5-1 % of a step of up to 1024
// units that never runs it: 176 units of 128 channels at 3630 22.5 / 22.7, 320 of 64 at 300 11.7 / 11.8, 224 at 485 13.5 / 13.6.)
bool decode_apart(const DecodeArgs& a) { return (int64_t)a.B * a.H > 1024 && (int64_t)a.B * a.H_kv > 512; }

hipError_t launch_step_apart(const DecodeArgs& a, int dtype, hipStream_t s) {
  const int grid = a.B * a.H + append_workgroups((int64_t)a.B * a.H_kv, a.d_h);
  return (a.flags & 64u) ? launch_fused<true, true, false, true, false>(a, dtype, grid, s) : launch_fused<true, false, false, true, false>(a, dtype, grid, s);
}

}  // namespace sparq
