// Small joins: a query whose tables stay within a few thousand rows runs all
// its remaining steps in one workgroup and one launch (small.hip).
#pragma once

#include "common.hpp"

namespace gsmat {

constexpr int64_t kSmallRows = 4096;        // rows of a table inside the launch
constexpr int64_t kSmallFin = 64 << 10;     // bytes of a final table of its own
// Blocks the answer may be left in: it takes the smallest that holds it, so a
// kept answer holds at most four times its bytes (or 1 KiB).
constexpr int kSmallFins = 4;
constexpr int64_t kFinBytes[kSmallFins] = {1 << 10, 4 << 10, 16 << 10, kSmallFin};

// Offsets in a query's work area: two tables of up to `cols` columns (the
// first at 0, the second at tab), the row starts and lengths of every
// candidate expansion, and the output offsets of an expansion left to be
// written.
struct SmallLayout {
  int64_t tab, starts, lens, offs, bytes;
  SmallLayout(int np, int cols) {
    tab = 4 * kSmallRows * (cols < 1 ? 1 : cols > kMaxCols ? kMaxCols : cols);
    starts = 2 * tab;
    lens = starts + 4 * kSmallRows * np;
    offs = lens + 4 * kSmallRows * np;
    bytes = offs + 8 * (kSmallRows + 32);
  }
};

enum : int32_t { kSmallDone = 1, kSmallMore = 2, kSmallWrite = 3 };
// where a reported table's columns are: where they were at the start (or in
// the store), in the work area, in final block i
enum : int32_t { kAtStart = 0, kAtWork = 1, kAtFin = 2 /* + i */ };

struct SmallPat {
  int32_t s, p, o;
};
struct SmallStep {
  int8_t kind, tp, orient, var;
  uint32_t members;
};

// One query: its plan, the table it starts from (column c holds variable
// var[c]) and the memory of its tables.
struct SmallArgs {
  int32_t np, nsteps, adaptive, k;
  int32_t si;
  uint32_t rem;
  int64_t n;
  int64_t budget;
  char* work;       // laid out by these (SmallLayout)
  int64_t tab, starts, lens, offs;
  char* fin[kSmallFins];  // kFinBytes[i] bytes (null: none)
  SmallPat pats[kMaxPats];
  SmallStep steps[kMaxPats + 1];
  LookupRes lk[kMaxPats];       // of the patterns with a constant ...
  uint32_t lk_valid;            // ... where this bit is set (else looked up)
  const int32_t* col[kMaxCols];
  int8_t var[kMaxCols];
};

// What the host reads when the launch is done: the table reached and the
// steps' row counts.  kSmallDone: the table is the query's answer (n = 0:
// none).  kSmallMore: it is the table before step si, which the general path
// takes on from there.  kSmallWrite: likewise, but step si has been counted:
// an expansion of pattern tp (orient 0 from its subject) with m rows, its
// offsets (int64) at `offs` of the work area and its rows' starts at start.
struct SmallReport {
  int64_t n;
  int32_t k, si;
  uint32_t rem;
  int32_t status, place, tp, orient;
  int64_t m;
  const int32_t* start;
  const int32_t* col[kMaxCols];
  int32_t var[kMaxCols];
  int64_t step_in[kMaxPats + 1], step_out[kMaxPats + 1];
  uint32_t seq;  // written last
};

// The store, alike for every query of a launch.
struct SmallStore {
  const PredDesc* dout;
  const PredDesc* din;
  OriPtrs out, in;
  const int32_t* out_src;
};

// Runs n queries, each from its a.rem / a.si on in a workgroup of its own.
// args and reps are host memory the device can reach; reps[i] is complete once
// reps[i].seq == seq.
void launch_small(const SmallStore& st, const SmallArgs* args, SmallReport* reps, int n,
                  uint32_t seq, hipStream_t s);

// An expansion counted by a small join: output j < m belongs to the last of
// the n <= kSmallRows rows whose offset is at most j.  Column c of the output
// is at out + c * stride.  offs null: the m = n rows as they are, k columns.
struct SmallWriteTask {
  const int64_t* offs;
  const int32_t* start;
  const int32_t* nbr;
  int32_t* out;
  int64_t m, stride;
  int32_t n, k;
  const int32_t* col[kMaxCols];
};

// Writes n counted expansions, `most` rows the largest; tasks is host memory
// the device can reach (n = 1: passed by value).
void launch_small_write(const SmallWriteTask* tasks, int n, int64_t most, double bytes,
                        hipStream_t s);

}  // namespace gsmat
