// Shares in proportion to the work: the arithmetic of one sequence, without anything of the
// device in it, so that a test can run it on the CPU as well.
#pragma once

#include <math.h>

namespace ts {

#define TS_BOTH __host__ __device__ __forceinline__

constexpr int kBalanceMembers = 32;   // most members of a cluster (more only lengthen its merge)

// What a sequence asks of the workgroups that share one of its KV heads, in metadata rows (a
// token's K and V are as long as a page's box), and the most members it may have.
struct SeqWork {
  float rows, most;
};

// P pages, Kb of them kept, of at most Kmax that any sequence keeps.  At least one row, so that
// an empty sequence has its workgroup too.  The limit goes by the longest list (a page per wave
// of every member at the least there, as with clusters of one size), not by the sequence's own:
// one that keeps 4 pages of 8000 has 8000 to score, and on one workgroup did so for the whole
// launch (one of 128 K tokens and five of 1600, 8 KV heads of 128 channels: 116 us; 28.9 now,
// 42 with even clusters).
TS_BOTH SeqWork seq_work(int P, int Kb, int Kmax, int S) {
  SeqWork w;
  w.rows = fmaxf((float)P + (float)(Kb * S), 1.f);
  const int most = (Kmax + 3) / 4;
  w.most = (float)(most < kBalanceMembers ? most : kBalanceMembers);
  return w;
}

// Members of a cluster at `inv_t`, the reciprocal of the rows per workgroup (0: one).
TS_BOTH float members_of(const SeqWork& w, float inv_t) {
  return fmaxf(fminf(ceilf(w.rows * inv_t), w.most), 1.f);
}

}  // namespace ts
