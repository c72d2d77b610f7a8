// The hand-overs of a bulk append in one launch, followed on the host with the launcher's and the kernel's own arithmetic:
// the workgroups of one KV head run one after the other, a chosen one last, and each reads the sequence's length when it
// starts.  0: every row was written by exactly one workgroup, the length advanced once and the counter is back at 0.
#include <stdint.h>

#include <vector>

#include "../paper_2312_04985_amd/csrc/append_plan.h"

using namespace sparq;

namespace {

int follow(int S, int n, int d_h, AppendSplit p, int late, bool rows_only) {
  const int E = S + n, positions = 2 * E + 64;
  std::vector<int> writes(positions, 0);
  int length = S, counter = 0, times = 0;
  for (int i = 0; i < p.n_split; ++i) {
    const int w = i == p.n_split - 1 ? late : (i < late ? i : i + 1);
    const int seen = length;
    const AppendRun run = append_run(seen, n, w, p, d_h);
    for (int q = run.begin > seen ? run.begin : seen; q < run.end; ++q) ++writes[q];
    if (rows_only && run.begin >= run.end) continue;      // the mistake that the test plants: counted only with rows
    if (++counter == (rows_only ? run.used : append_arrivals(p))) { counter = 0; length = seen + n; ++times; }
  }
  for (int q = 0; q < positions; ++q)
    if (writes[q] != (q >= S && q < E ? 1 : 0)) return 1;
  int used = 0;
  for (int w = 0; w < p.n_split; ++w) {
    const AppendRun run = append_run(S, n, w, p, d_h);
    if (run.end > run.begin) used = used == w ? w + 1 : -1;   // the first ones, without a gap
  }
  if (used != append_run(S, n, 0, p, d_h).used) return 2;
  return length == E && times == 1 && counter == 0 ? 0 : 3;
}

}  // namespace

// the first failure over all last workgroups and every number of rows in 1 .. n_new (steps of `step`)
extern "C" int append_model(int S, int n_new, int step, int d_h, int64_t heads, int64_t held, int rows_only) {
  const AppendSplit p = append_split(heads, n_new, d_h, held);
  for (int n = n_new; n >= 1; n -= step)
    for (int late = 0; late < p.n_split; ++late) {
      const int rc = follow(S, n, d_h, p, late, rows_only != 0);
      if (rc) return rc;
    }
  return 0;
}

extern "C" int append_workgroups(int n_new, int d_h, int64_t heads, int64_t held) {
  return append_split(heads, n_new, d_h, held).n_split;
}
