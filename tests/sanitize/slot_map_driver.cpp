// Host check of the attention kernel's slot map (slot_map.h): for equal
// shares and for work-balanced shares, every task of [0, nt) has exactly one
// launch slot and every other slot maps to -1; and of the rules for slices and
// for a launch per generation, and the merge's grid.  Exit status 0 and "ok N" when all
// configurations pass; the first failure is printed and exits 1.
#include <cstdint>
#include <cstdio>
#include <random>
#include <vector>

#include "slot_map.h"

namespace {

bool covers_once(int64_t nt, int64_t nslots, int64_t group, int64_t run, const int32_t* share_lo, const char* what) {
  std::vector<int> seen((size_t)nt, 0);
  for (int64_t s = 0; s < nslots; ++s) {
    const int64_t t = bsa::task_of_slot(s, nt, group, run, share_lo);
    if (t < -1 || t >= nt) {
      std::printf("FAIL %s: slot %lld maps to %lld outside [0, %lld)\n", what, (long long)s, (long long)t,
                  (long long)nt);
      return false;
    }
    if (t >= 0 && ++seen[(size_t)t] > 1) {
      std::printf("FAIL %s: task %lld twice (nt %lld group %lld run %lld)\n", what, (long long)t, (long long)nt,
                  (long long)group, (long long)run);
      return false;
    }
  }
  for (int64_t t = 0; t < nt; ++t)
    if (!seen[(size_t)t]) {
      std::printf("FAIL %s: task %lld has no slot (nt %lld group %lld run %lld, %lld slots)\n", what, (long long)t,
                  (long long)nt, (long long)group, (long long)run, (long long)nslots);
      return false;
    }
  return true;
}

}  // namespace

int main() {
  std::mt19937_64 rng(12345);
  long checks = 0;
  const int64_t groups[] = {1, 2, 4, 8};
  const int64_t runs[] = {1, 3, 8};
  // equal shares, with the default launch size
  for (int64_t nt = 0; nt <= 700; ++nt)
    for (int64_t g : groups)
      for (int64_t r : runs) {
        if (!covers_once(nt, bsa::default_slots(nt), g, r, nullptr, "equal shares")) return 1;
        ++checks;
      }
  for (int i = 0; i < 200; ++i) {
    const int64_t nt = (int64_t)(rng() % 200000);
    for (int64_t g : groups) {
      if (!covers_once(nt, bsa::default_slots(nt), g, 8, nullptr, "equal shares, large")) return 1;
      ++checks;
    }
  }
  // work-balanced shares: heads of zero, equal, skewed and random work
  for (int i = 0; i < 4000; ++i) {
    const int64_t nbh = 1 + (int64_t)(rng() % 64), npq = 1 + (int64_t)(rng() % 300);
    std::vector<int64_t> work((size_t)nbh);
    const int kind = i % 4;
    for (int64_t k = 0; k < nbh; ++k) {
      if (kind == 0) work[(size_t)k] = 0;
      else if (kind == 1) work[(size_t)k] = 1000;
      else if (kind == 2) work[(size_t)k] = (k % 7 == 0) ? 100000 : (int64_t)(rng() % 3);
      else work[(size_t)k] = (int64_t)(rng() % 5000);
    }
    for (int32_t g : {2, 4}) {
      int32_t lo[5];
      bsa::balanced_shares(work, npq, g, lo);
      const int ngroups = 8 / g;
      const int64_t nt = nbh * npq;
      if (lo[0] != 0 || lo[ngroups] != nt) {
        std::printf("FAIL shares: ends %d %d for nt %lld\n", lo[0], lo[ngroups], (long long)nt);
        return 1;
      }
      for (int k = 0; k < ngroups; ++k)
        if (lo[k] > lo[k + 1]) {
          std::printf("FAIL shares: not monotone at %d\n", k);
          return 1;
        }
      // equal work over heads that divide evenly: the shares are equal in count
      if (kind == 1 && nbh % ngroups == 0)
        for (int k = 0; k <= ngroups; ++k)
          if (lo[k] != nt / ngroups * k) {
            std::printf("FAIL shares: equal heads, share %d at %d not %lld\n", k, lo[k], (long long)(nt / ngroups * k));
            return 1;
          }
      for (int64_t r : runs) {
        if (!covers_once(nt, bsa::shares_slots(lo, g, r), g, r, lo, "balanced shares")) return 1;
        ++checks;
      }
    }
  }
  // slices: never fewer than the plan's or more tasks and shorter slices than
  // allowed, none that was measured to lose, and enough where few rows are long
  {
    struct Known {
      int32_t tq, tkv;
      int64_t rows;
      double keys;
      int32_t lo, hi;
      double longest = 0;
    };
    const Known known[] = {{256, 64, 160, 1024, 1, 1}, {256, 32, 192, 4096, 1, 1}, {256, 64, 224, 16384, 1, 1},
                           {128, 64, 256, 1638, 1, 1}, {128, 32, 224, 1024, 1, 1}, {64, 64, 256, 1024, 1, 1},
                           {64, 32, 224, 1024, 1, 1},  {64, 64, 104, 10000, 4, 4}, {64, 32, 2, 13000, 24, 64},
                           {128, 64, 64, 8192, 4, 8},  {256, 64, 32, 8192, 4, 8},
                           // two heads of 2048 tokens: even rows, and 30% Bernoulli
                           {64, 64, 64, 512, 1, 1},    {64, 64, 64, 614, 2, 4, 1024}};
    for (const Known& k : known) {
      bsa::SliceQuery z{k.tq, k.tkv, 1, k.rows, k.keys, false, int64_t(32768) * 512, k.longest};
      const int32_t got = bsa::row_slices(z);
      if (got < k.lo || got > k.hi) {
        std::printf("FAIL slices: T (%d, %d), %lld rows of %.0f keys: %d\n", k.tq, k.tkv, (long long)k.rows, k.keys, got);
        return 1;
      }
      ++checks;
    }
    for (int i = 0; i < 20000; ++i) {
      bsa::SliceQuery z{};
      z.tq = 64 << (rng() % 3);
      z.tkv = 32 << (rng() % 2);
      z.split = 1 << (rng() % 4);
      z.rows = 1 + (int64_t)(rng() % 600);
      z.keys = (double)(rng() % 200000);
      z.masked = rng() % 2;
      z.kv_bytes = (int64_t)(rng() % 200000) * 512;
      const int32_t got = bsa::row_slices(z);
      if (got < z.split || got > 64 || (got > z.split && (z.rows * got > 512 || z.keys < 192.0 * got))) {
        std::printf("FAIL slices: %d of %lld rows\n", got, (long long)z.rows);
        return 1;
      }
      ++checks;
    }
  }
  // a launch per generation: rows of no, one, few and enough keys
  {
    bsa::GenerationQuery z{};
    z.tq = 64;
    z.bq = 64;
    z.bkv = 64;
    z.slices = 1;
    z.tasks = z.logical_rows = 24 * 2048;
    z.kv_bytes = int64_t(131072) * 512;
    for (int64_t blocks : {0, 1, 8, 31, 32, 256})
      for (int32_t bq : {64, 32, 16}) {
        z.bq = bq;
        z.logical_rows = z.tasks * (64 / bq);
        z.max_row_nnz = blocks;
        z.nnz = blocks * z.logical_rows;
        z.run_blocks = z.nnz / 16;
        const int64_t want = blocks * 64 * (64 / bq) >= 2048 ? 1024 : 0;
        if (bsa::generation_slots(z) != want) {
          std::printf("FAIL generations: %lld slots for %lld blocks a row of %d\n",
                      (long long)bsa::generation_slots(z), (long long)blocks, bq);
          return 1;
        }
        ++checks;
      }
  }
  // about two generations: only where a task's rows are nearly equal, or
  // several query blocks make up a task; from 2304 tasks on up to 1.4 times the mean
  {
    bsa::GenerationQuery z{};
    z.tq = 64;
    z.bkv = 64;
    z.slices = 1;
    z.kv_bytes = int64_t(65536) * 512;
    for (int32_t bq : {64, 32})
      for (int64_t tasks : {2047, 2048, 2303, 2304, 4096})
        for (int64_t longest : {100, 110, 111, 140, 141}) {
          z.bq = bq;
          z.tasks = tasks;
          z.logical_rows = tasks * (64 / bq);
          z.nnz = 100 * z.logical_rows;
          z.max_row_nnz = longest;
          const bool want = tasks >= 2048 && longest <= (bq == 64 && tasks < 2304 ? 110 : 140);
          if (bsa::generation_slots(z) != (want ? 1024 : 0)) {
            std::printf("FAIL generations: %lld tasks of %d, longest row %lld%%\n", (long long)tasks, bq,
                        (long long)longest);
            return 1;
          }
          ++checks;
        }
  }
  // the merge's grid: 8 query rows per workgroup, and launchable (fewer than
  // 2^32 threads a dimension) for every row count whose tasks are
  for (int64_t tq : {64, 128, 256})
    for (int64_t nrows : {int64_t(1), int64_t(1) << 21, (int64_t(1) << 24) - 1}) {
      const int64_t x = bsa::merge_grid_x(nrows), y = bsa::merge_grid_y(tq);
      if (x * y != nrows * tq / 8 || x * bsa::kMergeThreads >= (int64_t(1) << 32) || y > 65535) {
        std::printf("FAIL merge grid: %lld x %lld for %lld rows of %lld\n", (long long)x, (long long)y,
                    (long long)nrows, (long long)tq);
        return 1;
      }
      ++checks;
    }
  std::printf("ok %ld\n", checks);
  return 0;
}
