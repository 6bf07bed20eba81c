// Which task each launch slot of the attention kernel runs, the shares of the
// task list that the XCD groups take, the slices of a row, how many slots a
// launch has, and the merge's grid.  Plain code: the kernel evaluates
// task_of_slot on the device (a constexpr function is callable from device
// code), the planner and the host tests on the host.
#pragma once

#include <cstdint>
#include <vector>

namespace bsa {

// Map launch slot `slot` to a task index in [0, nt), or -1.  Slot i runs on
// XCD i % 8.  The XCDs form 8 / group groups of `group` XCDs; group g works
// through the g-th contiguous share of the task list, and inside it its XCDs
// take turns over runs of `run` consecutive tasks (XCD member m takes runs m,
// m + group, ...), so neighbouring tasks still share an XCD while the group's
// XCDs stay on the same stretch of the list.  group = 1 gives each XCD its
// own contiguous eighth; group = 8 keeps all XCDs on one stretch.  The shares
// are equal in task count, or given (share_lo non-null: group g takes
// [share_lo[g], share_lo[g + 1]), cut by the planner so that the shares hold
// equal work; group >= 2).  The tail of a share that does not fill whole
// rounds of runs is dealt out one task per XCD.  With default_slots(nt)
// slots for equal shares, or shares_slots(...) for given ones, every task of
// [0, nt) has exactly one slot.
constexpr int64_t task_of_slot(int64_t slot, int64_t nt, int64_t group, int64_t run, const int32_t* share_lo) {
  const int64_t xcd = slot & 7, local = slot >> 3;
  if (group <= 1) {
    const int64_t per = (nt + 7) / 8;
    const int64_t t = xcd * per + local;
    return (local < per && t < nt) ? t : -1;
  }
  const int64_t ngroups = 8 / group, gi = xcd / group, mi = xcd % group;
  int64_t lo = 0, n = 0;
  if (share_lo) {
    // a select over the (at most four) groups keeps the bounds in scalar
    // registers on the device; an indexed read of the kernel argument array
    // would place it in scratch memory
    int64_t a0 = 0, a1 = 0;
    for (int i = 0; i < 4; ++i)
      if (i == gi) {
        a0 = share_lo[i];
        a1 = share_lo[i + 1];
      }
    lo = a0;
    n = a1 - a0;
  } else {
    const int64_t per = (nt + ngroups - 1) / ngroups;
    lo = gi * per;
    n = (nt < lo + per ? nt : lo + per) - lo;
    if (n < 0) n = 0;
  }
  const int64_t whole = n / (group * run);  // complete rounds of runs
  const int64_t t = local < whole * run ? (local / run) * group * run + mi * run + local % run
                                        : whole * group * run + (local - whole * run) * group + mi;
  return t < n ? lo + t : -1;
}

// Launch slots for equal shares: the task count rounded up to a multiple of 8.
constexpr int64_t default_slots(int64_t nt) { return (nt + 7) / 8 * 8; }

// Slices per physical row for the kernel.  A request of few rows leaves CUs
// idle however long its rows are, and the plan's Split-K factor ends at 8, so
// its rows are cut further where that is expected to pay.  The partial states
// merge as for Split-K; the plan, its tasks and their exports stay what they
// are.
//
// Expected time of a row's slices: the keys of one slice of the longest row, at
// the rate of a workgroup that has its SIMDs to itself (slower where tiles mask
// their members), or where more workgroups run than that the keys of one slice of
// a mean row at the rate of the CU or the L2 behind it; and the partial states' way through memory.  The rates are
// fitted to 1550 measurements of 1 to 64 slices (seven kernels, 2 to 256 rows,
// 0.2K to 130K keys a row, K/V of 2 to 64 MB a head).  Over them the slices
// chosen take 1.05 times the time of the fastest number, one slice takes 2.9
// times, and none of the chosen takes 3% more than one slice.  (A cut until 512
// tasks run or a slice has 448 keys took 1.16 times, and up to 1.6 times one
// slice: T = (256, 64), 160 rows of 1024 keys 38 us in one slice, 60 in three.)
// (Those rows were of equal length.  The longest row waits alone: 64 rows of 614
// keys, the longest 1024, T = (64, 64) 20.5 us by the mean row, uncut, 19.0 by the
// longest; four heads of 2048 tokens under 25% top-k of (32, 16) blocks 30 and 26
// us.  Of 389 requests with few rows 21 are faster by 3% and 13 slower, nearly all
// of these within 5%; the geometric mean is unchanged.)
constexpr int64_t kSliceTasks = 512;  // tasks that cut rows may become
constexpr int64_t kSliceKeys = 192;   // keys a slice keeps at least
constexpr int32_t kSliceMost = 64;
struct SliceQuery {
  int32_t tq, tkv, split;
  int64_t rows;     // physical rows
  double keys;      // keys of a physical row
  bool masked;      // tiles have several member blocks
  int64_t kv_bytes; // K and V of one head
  double longest;   // keys of the longest row (0: the rows are equal)
};
inline int32_t row_slices(const SliceQuery& z) {
  if (z.rows < 1 || z.rows * z.split * 2 > kSliceTasks) return z.split;
  const int i = z.tq <= 64 ? 0 : z.tq <= 128 ? 1 : 2;
  // us per 1024 keys: alone (plus masking), and per workgroup on each of 256
  // CUs (T_Q = 64 streams the most K/V per key: less from an XCD's own L2); us
  // per task and merge
  const double alone = (i == 0 ? (z.tkv >= 64 ? 14.0 : 17.0) : i == 1 ? 16.0 : 17.0) +
                       (z.masked ? (i == 0 ? 2.5 : i == 1 ? 2.0 : 3.5) : 0.0);
  const double shared = i == 0 ? (z.kv_bytes <= (4 << 20) ? 8.0 : 11.5) : i == 1 ? 14.0 : 26.0;
  const double state = i == 0 ? 0.018 : i == 1 ? 0.03 : 0.06, merge = i == 2 ? 4.0 : 1.5;
  auto time = [&](int32_t s) -> double {
    const int64_t tasks = z.rows * s;
    // whole rounds of CUs weigh more than the mean: the last round waits
    const double load = 0.6 * (double)((tasks + 255) / 256) + 0.4 * (double)tasks / 256.0;
    const double last = (z.longest > z.keys ? z.longest : z.keys) * alone, all = z.keys * shared * load;
    return (last > all ? last : all) / s / 1024.0 + (s > 1 ? merge + state * (double)tasks : 0.0);
  };
  int32_t best = z.split;
  double best_time = time(z.split) - 1.0;  // (a microsecond has to be won)
  for (int32_t s = z.split + 1; s <= kSliceMost && z.rows * s <= kSliceTasks && z.keys >= (double)kSliceKeys * s; ++s) {
    const double t = time(s);
    if (t < best_time) {
      best = s;
      best_time = t;
    }
  }
  return best;
}

// Launch slots per kernel launch; 0: all tasks in one launch.  The tasks an
// XCD runs at once read the same head's K/V in the same order, and share L2
// lines while they are about equally far.  They start together but drift
// apart over the generations of a long launch; a launch per generation lines
// them up again, for the wait on its slowest task and about 7 us.  That pays
// for the T_Q = 64 kernels, which read the most K/V per flop, and there
// - where a head's K/V is several times an XCD's L2 (4 MB): over the rule's
//   other conditions a mean of 0.83 of the time at 115200 tokens (none of 258
//   slower by 3%), 0.89 at 65536 (none of 174), 0.98 at 32768 (33 of 162);
// - where the rows are about equally long (with the longest above 1.4 times
//   the mean the wait costs more: 0.89 within, 1.0 above), and of up to about
//   two generations with a block's rows to a task nearly equal, since the wait
//   is then for half of the tasks: 65536 tokens, 2 heads, 15% and 40%
//   Bernoulli of (64, 64) blocks 0.92 -> 0.96 and 2.25 -> 2.39 ms (longest
//   rows 1.26 and 1.13 times the mean), top-k 0.64 -> 0.65 and, in two slots,
//   0.79 -> 0.68; at 2304 tasks 0.93 to 1.01, at 3072 0.90 to 0.98;
// - where they are scattered: the long runs of windows share lines between
//   neighbours anyway (5% window of 131072 tokens 4.20 and 4.59 ms);
// - where a query block is at most one task's rows: the tasks of a larger
//   block share their list and run side by side (128-token blocks: 0.97, the
//   fastest plan unchanged);
// - where a task has about 2048 keys or more: 131072 tokens x 24 heads with
//   equally long random rows under the three T_Q = 64 kernels 1.6 times at none,
//   1.25 at 512, 1.08 to 1.15 at 1024, 0.99 to 1.06 at 1536, 0.94 to 1.0 at
//   2048 and 0.70 to 0.92 at 8192 keys a row; of 32-token blocks, two to a
//   task, 0.97 to 1.06 at 512 and 0.84 to 0.97 at 1024.
// 12% top-k of 64-token blocks, T = (64, 32) in two slots, 24 heads x 115200
// tokens 35.1 -> 21.9 ms (the fastest without: 24.5 ms), 12 x 65536 4.83 ->
// 3.39; 12% Bernoulli 12 x 65536 5.45 -> 4.19; T_Q = 128 within 2%.
constexpr int64_t kGenerationSlots = 1024;      // four 2-wave workgroups on each of 256 CUs
constexpr int64_t kGenerationKvBytes = 32 << 20;
constexpr int64_t kGenerationKeys = 2048;
constexpr int64_t kGenerationTasksUneven = 2304;  // tasks from which rows may be uneven
struct GenerationQuery {
  int32_t tq, bq, bkv, slices;
  int64_t tasks, logical_rows, nnz, max_row_nnz, run_blocks;
  int64_t kv_bytes;  // K and V of one head
};
constexpr int64_t generation_slots(const GenerationQuery& z) {
  if (z.tq != 64 || z.bq > 64 || z.slices != 1 || z.tasks < 2 * kGenerationSlots) return 0;
  if (z.kv_bytes < kGenerationKvBytes) return 0;
  if (z.max_row_nnz * z.logical_rows * 5 > z.nnz * 7 || z.run_blocks * 3 > z.nnz * 2) return 0;
  if (z.bq == z.tq && z.tasks < kGenerationTasksUneven && z.max_row_nnz * z.logical_rows * 10 > z.nnz * 11) return 0;
  // a task's keys are at most the keys of its query blocks' rows together,
  // and close to them where few blocks are active
  if (z.nnz * z.bkv / z.logical_rows * (z.tq / z.bq) < kGenerationKeys) return 0;
  return kGenerationSlots;
}

// Workgroups of the Split-K merge, kMergeRows query rows each: (physical rows,
// parts of a row).  A launch dimension holds fewer than 2^32 threads, so with
// kMergeThreads a workgroup the rows of the largest plans (below 2^24) have one
// to themselves.
constexpr int64_t kMergeRows = 8;
constexpr int64_t kMergeThreads = 32 * kMergeRows;
constexpr int64_t merge_grid_x(int64_t nrows) { return nrows; }
constexpr int64_t merge_grid_y(int64_t tq) { return tq / kMergeRows; }

// Launch slots for given shares share_lo[0 .. 8 / group] (group >= 2): eight
// times the most tasks one XCD of any group takes.
constexpr int64_t shares_slots(const int32_t* share_lo, int64_t group, int64_t run) {
  int64_t most = 0;
  for (int64_t g = 0; g < 8 / group; ++g) {
    const int64_t n = (int64_t)share_lo[g + 1] - share_lo[g], whole = n / (group * run);
    const int64_t r = n - whole * group * run;
    const int64_t per_xcd = whole * run + (r + group - 1) / group;
    if (per_xcd > most) most = per_xcd;
  }
  return 8 * most;
}

// Shares of the XCD groups (group >= 2) over a split-free task list:
// contiguous stretches holding equal work.  The task list holds npq tasks
// per (b, h) in (b, head) order, whatever the dispatch order does inside a
// head, and work[k] is the work of the k-th (b, h) (its active logical
// blocks), taken as spread evenly over its tasks, so a cut may fall inside a
// head.  Requests whose heads carry equal work get equal task counts when
// the heads divide evenly among the groups.  Fills lo[0..4] (lo[g] = nt
// past the last group).
inline void balanced_shares(const std::vector<int64_t>& work, int64_t npq, int32_t group, int32_t* lo) {
  const int ngroups = 8 / group;
  const int64_t nbh = (int64_t)work.size(), nt = nbh * npq;
  std::vector<int64_t> cw(nbh + 1, 0);
  for (int64_t k = 0; k < nbh; ++k) cw[k + 1] = cw[k] + work[k];
  const int64_t total = cw[nbh];
  for (int g = 0; g <= 4; ++g) lo[g] = (int32_t)nt;
  lo[0] = 0;
  for (int g = 1; g < ngroups; ++g) {
    int64_t pos;
    if (total == 0) {
      pos = (nt * g + ngroups - 1) / ngroups;
    } else {
      const int64_t target = total * g / ngroups;
      int64_t k = 0;
      while (k + 1 < nbh && cw[k + 1] <= target) ++k;
      pos = k * npq + (work[k] > 0 ? ((target - cw[k]) * npq + work[k] / 2) / work[k] : 0);
    }
    if (pos < lo[g - 1]) pos = lo[g - 1];
    if (pos > nt) pos = nt;
    lo[g] = (int32_t)pos;
  }
}

}  // namespace bsa
