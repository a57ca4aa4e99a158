// Shares in proportion to the work: the arithmetic of one sequence, without anything of the
// device in it, so that a test can run it on the CPU as well.
#pragma once

#include <math.h>

namespace ts {

#define TS_BOTH __host__ __device__ __forceinline__

// Most members of a cluster.  Measured when the last member merged all partials, which more of them only made
// longer; from nine members on the merge is dealt out now, and the limit has not been looked at again.
constexpr int kBalanceMembers = 32;

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

// Kept pages of each member where K are divided among g: whole groups of pages that are smaller
// than an MFMA tile.
TS_BOTH int chunk_of(int K, int g, int S) {
  const int c = (K + g - 1) / g;
  return S < 16 ? (c + 3) / 4 * 4 : c;
}

// Members of a cluster in a launch of `units` of them, at most `most`, each with a table of P pages, K
// kept, d channels: the number whose launch is worked out to be the shortest.  What it takes beyond
// what all have in common, in us: a round of scoring with more than one group of pages a wave; the
// member's rows and tiles at 100 B/ns; each fragment of a wave after the first; each sixteen partials
// merged after the first; and, with more than 96 workgroups, every further one (their polls, arrivals
// and dispatch).  sweep.py --clusters times 48 layouts of 1 to 85 units with 100 to 8000 pages at up to
// eleven sizes each: where these costs were fitted, 1.0 % above the best size on average, 9.4 % at the most (1 unit, 120 of
// 1000 pages: 30 members 12.0 us, 16 11.0), and as many members as fit the device with four pages each 4.8 % above
// it, 38 % at the most (4 units, 250 of 1000 pages: 63 members 17.1 us, 17 12.4; 16 units, 48 of 250: 12
// 11.1, 6 10.1; 8 units, 120 of 1000: 30 13.7, 16 11.6).  Since then more than eight members divide the merge and six to
// nine groups a wave are one round, which the costs do not know of: 2.4 % and 21 % now, as many members as fit 2.4 % and 15.5 %.
struct ClusterTime {
  float grows;   // what only grows with fewer members
  float all;
};
TS_BOTH ClusterTime cluster_us(int units, int members, int chunk, int P, int S, int d) {
  const int group = 512 / d, groups = (P + group - 1) / group;
  const int rows = ((groups + members - 1) / members + 7) / 8;
  const int frags = S < 16 ? (chunk * S + 15) / 16 : chunk * (S > 32 ? S / 32 : 1);
  const int rounds = (frags + 7) / 8, batches = members > 17 ? (members + 14) / 16 : 1, wgs = units * members;
  const float scoring = rows <= 1 ? 0.f : rows <= 3 ? 0.5f : rows <= 5 ? 1.f : 1.f + 0.35f * (float)(rows - 5);
  const float bytes = ((float)P / (float)members + (float)(chunk * S)) * 4.f * (float)d;
  ClusterTime t;
  t.grows = scoring + bytes * 1e-5f + 0.3f * (float)(rounds - 1);
  t.all = t.grows + 0.7f * (float)(batches - 1) + (wgs > 96 ? 0.012f * (float)(wgs - 96) : 0.f);
  return t;
}
// (Worked out in every call.  Only sizes that divide the list differently are looked at, and none
// below the one at which the growing part alone is no less than the best: 0.01 to 0.27 us a call, where
// all sizes take 0.06 to 0.64.)
TS_BOTH int cluster_members(int units, int most, int P, int K, int S, int d) {
  int best = most, g = most;
  float least = INFINITY;
  while (g >= 2) {
    const int chunk = chunk_of(K, g, S), members = (K + chunk - 1) / chunk;
    const ClusterTime t = cluster_us(units, members, chunk, P, S, d);
    if (t.all < least) {
      least = t.all;
      best = g;
    }
    if (t.grows >= least) break;
    g = members - 1;
  }
  return best;
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
