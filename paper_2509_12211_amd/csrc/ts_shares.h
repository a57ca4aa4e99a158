// Shares in proportion to the work: the arithmetic of one sequence, without anything of the
// device in it, so that a test can run it on the CPU as well.
#pragma once

#include <math.h>

namespace ts {

#define TS_BOTH __host__ __device__ __forceinline__

constexpr int kBalanceMembers = 32;   // most members of a cluster (more only lengthen its merge)

// What a sequence asks of the workgroups that share one of its KV heads, in metadata rows (a
// token's K and V are as long as a page's box): rows every member reads in full, rows divided
// among them, and the most members it may have.
struct SeqWork {
  float whole, rows, most;
};

// P pages, Kb of them kept, of at most Kmax that any sequence keeps.  At least one row, so that
// an empty sequence has its workgroup too.
// exchange: the members divide the scoring as well and hand each other the scores.  The limit
// then goes by the longest list (a page per wave of every member at the least there, as with
// clusters of one size), not by the sequence's own: one that keeps 4 pages of 8000 has 8000 to
// score, and on one workgroup did so for the whole launch (one of 128 K tokens and five of
// 1600, 8 KV heads of 128 channels: 116 us; 28.9 now, 42 with even clusters).
// Otherwise every member scores all pages, and there is no use for one without pages to attend.
TS_BOTH SeqWork seq_work(int P, int Kb, int Kmax, int S, bool exchange) {
  SeqWork w;
  w.whole = exchange ? 0.f : (float)P;
  w.rows = fmaxf((float)(Kb * S) + (exchange ? (float)P : 0.f), 1.f);
  const int most = ((exchange ? Kmax : Kb) + 3) / 4;
  w.most = (float)(most < kBalanceMembers ? most : kBalanceMembers);
  return w;
}

// Rows the busiest workgroup of a sequence reads with a cluster of g workgroups, which divide the
// scoring evenly and the pages kept in pieces of `chunk`.
TS_BOTH float even_rows(int P, int Kb, int chunk, int S, float inv_g) {
  return (float)P * inv_g + (float)((Kb < chunk ? Kb : chunk) * S);
}

// Members of a cluster at `inv`, the reciprocal of how many divided rows a member may take (the
// rows per workgroup less those read in full; 0: no limit).
TS_BOTH float members_of(const SeqWork& w, float inv) {
  return fmaxf(fminf(ceilf(w.rows * inv), w.most), 1.f);
}

// Every cached token, two rounds of units and more (of kRound at once): whether each unit is best
// left to one workgroup (kWhole).  total, longest: pages of the B sequences.  A few sequences much
// longer than the rest would decide the finish time (kFewLong); even lengths are divided where
// they would leave the last round mostly empty (kHalves).
constexpr int kRound = 256;
enum Rounds { kWhole, kHalves, kFewLong };
TS_BOTH Rounds rounds_of(int total, int longest, int B, int units) {
  const float mean = (float)total / (float)B, most = (float)longest;
  const int last = units % kRound;
  if (mean < 0.4f * most) return kFewLong;
  return mean < 0.9f * most || last == 0 || last > kRound * 5 / 8 ? kWhole : kHalves;
}

}  // namespace ts
