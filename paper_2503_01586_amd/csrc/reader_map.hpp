// Several queries per sequence: which work-group of the attention launch reads what.  All work-groups stand on a line, those
// that read the same rows (a split of one sequence: every query and head group of it) next to each other; this says which
// place of the line a work-group of the grid takes.  Plain C++ apart from the function attributes: the host can run it.
#pragma once

#if defined(__HIPCC__)
#define EKV_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define EKV_HOST_DEVICE inline
#endif

namespace ekv {

// Work-groups that stay together when a line of `all` of them is dealt out, `readers` of which read the same rows: the first of
// a run fetches the rows, the others find them in the L2.  A line that the chip (256 compute units) holds at once is one run:
// nothing waits for a compute unit, so nothing has to be dealt evenly, and an XCD keeps to as few sequences and their queries
// as it can (4 x 5 queries of 4096 tokens without the append: 70.6 us, dealt in runs of five 71.5).  Longer runs than sixteen
// are unequal shares of a prompt's queries (runs of 32 give an XCD up to 1.9 times its share of 257 to 400 of them).  us, one
// line spread as it came / in contiguous eighths / dealt out: 2048 queries over their own prompt, 1024 columns and sixteen
// elite chunks, 1668 / 2217 / 1545; 512 243 / 260 / 235; 7B 12.5 %, 64 x 4 queries, lengths falling from 2048 203 / 186 / 168.
constexpr int kReaderRun = 16;

inline int reader_run(int readers, int all) { return all <= 256 ? all : readers < kReaderRun ? readers : kReaderRun; }

// How often every XCD gets a run (a division less at the start of every work-group: 4 x 5 queries of 4096 tokens 86.0 -> 85.7 us)
inline int reader_turns(int all, int run) { return all / (8 * run); }

// Place on the line of `all` work-groups that work-group `block` takes (-1: none).  Work-groups go to the eight XCDs
// round-robin by index.  The line is dealt out in runs, there and back (XCD 0 .. 7, 7 .. 0, ...): the rows that a query sees
// grow along the line where the queries are a prompt's, or fall where a batch is sorted by length, and every XCD gets its
// share of both ends.  What is left, less than a run per XCD, is divided in eighths, so that no XCD has more than one
// work-group more than another.
EKV_HOST_DEVICE int reader_place(int block, int all, int run, int turns) {
  const int xcd = block & 7, slot = block >> 3;
  const int turn = slot / run;
  if (turn < turns) return (turn * 8 + (turn & 1 ? 7 - xcd : xcd)) * run + slot % run;
  const int rest = all - turns * 8 * run, share = (rest + 7) / 8, k = slot - turns * run;
  const int at = turns * 8 * run + xcd * share + k;
  return k < share && at < all ? at : -1;
}

}  // namespace ekv
