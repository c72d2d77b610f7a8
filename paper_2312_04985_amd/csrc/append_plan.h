// How the rows of a bulk append are dealt to workgroups: arithmetic shared by the kernel and its launcher (kv_append.hip).
// Nothing here needs a device compiler, so a test on the host runs the same code.
#pragma once
#include <stdint.h>

namespace sparq {

constexpr int kAppendThreads = 256;
// positions per tile: 256, 128, 64 for d_h = 64, 128, 256 (32 KB of keys)
constexpr int append_tile(int d_h) { return 8 * kAppendThreads / (d_h / 8); }

// Workgroups per KV head of a bulk append of `tiles` tiles per head: about kAppendGroups in all (8 per CU; three of them
// run at once, by registers), at most 128 per head, so that append_finish reads few partial sums.
constexpr int64_t kAppendGroups = 2048;
constexpr int64_t append_groups(int64_t heads, int64_t tiles) {
  const int64_t per = (tiles * heads + kAppendGroups - 1) / kAppendGroups, n = (tiles + per - 1) / per;
  return n < 128 ? n : 128;
}

// Up to so many workgroups one launch does a bulk append.  Device us per call, two launches / one: 8 KV heads x 8 rows 8.6 /
// 7.5, 64 x 64 9.5 / 9.2, 128 x 8 8.4 / 8.3, 192 x 8 9.0 / 9.6, 512 x 8 9.7 / 14.0; a program that does not capture its calls
// pays 2.5 us of host time for the second launch, so the line lies a little higher than where the device times cross.
constexpr int64_t kAppendOneLaunch = 192;

// Short appends for many KV heads, by append_rows_short: up to a quarter of a tile, and up to kAppendShort rows where there
// are rows enough to fill the memory's pipes with a workgroup per head (append_rows asks for 16 pieces per thread at once,
// but 8 rows keep 16 to 64 of its 256 threads busy).  Device us per call, short / tiles: 512 heads of 128 x 8 rows 8.1 / 9.5,
// x 33 10.8 / 11.3, x 64 15.6 / 13.9; 768 x 64 20.3 / 17.9; 1024 x 64 24.3 / 27.3; 2048 x 8 17.6 / 22.1, x 64 45.3 / 43.9; heads of
// 64, 512 x 64 11.0 / 11.2, 1536 x 33 15.2 / 19.1; heads of 256, 256 x 48 16.2 / 13.0, 512 x 33 18.4 / 19.9, 768 x 64 31.2 / 35.8.
constexpr int kAppendShort = 64;
constexpr bool append_short(int64_t heads, int64_t n_new, int d_h) {
  return n_new <= kAppendShort && (n_new <= append_tile(d_h) / 4 || heads * d_h >= 131072);
}

// Workgroups per KV head: one per tile until there are kAppendGroups in all, then longer runs of tiles, and no
// more than the scratch holds partial sums of (512 KV heads, up to 512 rows each: 4 per head 51 us, 2 per head
// 67 us).  A call on a cache that is not aligned to 64 positions may touch one tile more.
struct AppendSplit {
  int n_split, tiles_per_split;
};
constexpr AppendSplit append_split(int64_t heads, int64_t n_new, int d_h, int64_t held) {
  const int64_t tiles = (n_new + 63 + append_tile(d_h) - 1) / append_tile(d_h);
  int64_t n = append_groups(heads, tiles);
  if (n > held) n = held > 1 ? held : 1;
  const int64_t per = (tiles + n - 1) / n;
  return {(int)((tiles + per - 1) / per), (int)per};
}

// What workgroup `split` of a KV head does for a sequence of S cached and n > 0 new rows: positions begin .. end - 1
// (end <= begin: none of the rows fall to it).  `used`: the workgroups 0 .. used - 1 of the head have rows.
struct AppendRun {
  int begin, end, used;
};
constexpr AppendRun append_run(int S, int n, int split, AppendSplit p, int d_h) {
  const int per = p.tiles_per_split * append_tile(d_h), first = S & ~63, e = S + n, begin = first + split * per;
  return {begin, begin + per < e ? begin + per : e, (e - first + per - 1) / per};
}
// Arrivals at a head's counter before its mean, and then its sequence's length, is written in the same launch: every
// workgroup of the head, since each decides by that length what falls to it.
constexpr int append_arrivals(AppendSplit p) { return p.n_split; }

}  // namespace sparq
