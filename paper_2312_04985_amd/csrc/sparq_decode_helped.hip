// The one-workgroup-per-head kernel for few units, whose idle CUs fetch for the units' workgroups.
#include "sparq_decode_fused.h"

namespace sparq {

namespace {

// Workgroups of a unit, its own and those that fetch for it: one for each of the XCD's 32 CUs, at most 8 (of 32 heads at 4096
// positions, the caches in HBM: 4 per unit 16.7 us per decode, 8 16.8; at 12 200 positions 23.2 and 22.6).
int units_per_xcd(const DecodeArgs& a) { return (a.B * a.H + 7) / 8; }
int workgroups_per_unit(int per_xcd) { return 32 / per_xcd < 8 ? 32 / per_xcd : 8; }

}  // namespace

// Where CUs are idle: with three or more workgroups per unit (80 units) always, with two (128 units) as long as what the units
// read stays in the L2 of their XCD.  us per step without / with helpers, 128 channels, r 16 unless said, every line from HBM (a gigabyte
// read between the calls) and with the caches in L2 or in the memory-side cache (3 in turn):
// 1 head at 100 positions, k 16, 12.2 / 11.8 and 9.1 / 9.1; 300, k 64, 12.5 / 11.9 and 9.2 / 9.2; 1023, k 128, 13.4 / 12.3 and 9.5 / 9.5; 4000, k 128, 14.7 /
// 13.1 and 10.4 / 10.4; 32 heads at 300, k 64, 13.1 / 12.6 and 9.7 / 9.7; 1500, k 128, 14.3 / 13.1 and 10.1 / 10.1; 6000, r 32, k 512, 24.0 / 19.5 and 20.0 /
// 16.0; 128 at 100, k 16, 12.9 / 12.5 and 9.7 / 9.6; 500, k 64, 13.7 / 13.0 and 10.2 / 10.1; 2000, r 32, k 256, 17.9 / 16.1 and 14.4 / 12.9; at 8192, not
// helped, k 512, 40 caches in turn 26.6 / 29.6 and 3 in turn 26.2 / 25.9.
// (There was a line below which small calls had none, drawn when the helped build itself cost them 0.2 us.)
bool decode_helped(const DecodeArgs& a) {
  const int64_t units = (int64_t)a.B * a.H;
  if ((a.flags & 64u) || units > 128) return false;      // (not for the tiled layout)
  return workgroups_per_unit(units_per_xcd(a)) >= 3 || units * a.S_max <= 640 * 1024;
}

hipError_t launch_decode_helped(const DecodeArgs& a, int dtype, hipStream_t s) {
  DecodeArgs d = a;
  d.per_xcd = units_per_xcd(a);
  d.by_xcd = make_divider(d.per_xcd);
  const int n = workgroups_per_unit(d.per_xcd), grid = 8 * d.per_xcd * n;
  d.helpers = n - 1;
  return a.k_new ? launch_fused<true, false, true, false, false>(d, dtype, grid, s) : launch_fused<false, false, true, false, false>(d, dtype, grid, s);
}

}  // namespace sparq
