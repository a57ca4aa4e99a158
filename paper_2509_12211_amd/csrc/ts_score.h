// Page scoring (Eq. 2): the directional bounding-box bound, group-summed.
#pragma once
#include "ts_device.h"

namespace ts {

// For a group of G query heads sharing one KV head,
//   sum_g sum_c max(q_gc * m_c, q_gc * M_c) = sum_c (Qp_c * M_c + Qn_c * m_c)
// with Qp_c = sum_g max(q_gc, 0) and Qn_c = sum_g min(q_gc, 0): a term takes
// M when q >= 0 and m otherwise (the sign test of Eq. 2), so the per-head sum
// factorises.  Two FMAs per channel per page, whatever G is.
//
// The sum is accumulated in fp64 and rounded to fp32 once at the end: with
// temporally correlated keys the terms are large and of mixed sign, the bound
// itself can be 1e3-1e4 times smaller than their magnitudes, and an fp32
// running sum then misses the 1e-5 relative tolerance on the score.  Qp, Qn
// (sums of <= 16 bf16 values) and the bf16 x fp64 products are exact in fp64.
//
// Lane layout: a metadata row (D bf16) is read as D/8 chunks of 16 bytes, so
// one wave-wide 16-byte load covers 64 / (D/8) consecutive pages; each lane
// keeps Qp / Qn for its 8 channels.
template <int D, bool kHalf = false, int NW = kWaves>
struct ScoreLanes {
  static constexpr int NT = NW * kWave;     // threads of the workgroup
  static constexpr int LPR = D / 8;         // lanes per metadata row
  static constexpr int PPW = kWave / LPR;   // pages per wave-wide load
  double qp[8], qn[8];

  // Qp / Qn of the unit.  Split in three so the caller can issue other loads between the query load
  // and its first use (loads return in issue order: what is needed first is
  // issued first), and more while the waves wait for each other.  stage: LDS scratch of
  // query_stage_bytes(G) bytes, headed by the raw rows when share_query returns.
  //
  // Two forms.  kShort is for launches that score several groups a wave in one round, where this is a link of
  // the chain they are made of:
  //   G = 1: a lane's sums are its own chunk of the row, which it has fetched itself: no exchange.
  //   G <= 8: a wave fetches the G values of each of its D / NW channels, a lane per (row, channel),
  //   sums them across its lanes, and the sums go round through LDS behind one barrier (ready 0.3 us sooner).
  // Otherwise, and for larger groups, the rows themselves go through LDS, a thread sums a channel over
  // the heads (a loop of loads per lane would pay one memory round trip per head), and the sums go
  // round behind a second barrier: fewer loads, and 1-2 % faster where other workgroups' work
  // covers the wait (352 units of 52 pages 18.3 against 18.55 us).
  static constexpr size_t query_stage_bytes(int G) { return (size_t)G * D * 2 + 2 * D * 8; }
  static constexpr int kQueryLoads = 16 * D / 8 / NT > 0 ? 16 * D / 8 / NT : 1;
  static constexpr int kChannels = D / NW;            // channels a wave sums over the rows
  static constexpr int kRows = kWave / kChannels;     // rows of them its lanes cover
  static constexpr int kSumLoads = 8 / kRows > 0 ? 8 / kRows : 1;

  template <bool kShort, int kDummy = 0>
  struct QueryRegs {
    uint4 w[kQueryLoads];
  };
  template <int kDummy>
  struct QueryRegs<true, kDummy> {
    uint4 w[kQueryLoads];
    uint16_t e[kSumLoads];
  };

  // Every thread loads and every thread stages what it loaded (thread i takes
  // chunk i, threads past the last chunk take the last one again; duplicates carry
  // identical data): a
  // load under a branch makes the compiler wait for ALL outstanding loads
  // wherever it needs one of them, instead of counting, and a load whose only
  // use sits under a branch is moved down into that branch.
  template <bool kShort>
  __device__ __forceinline__ static void issue_query(QueryRegs<kShort>& r, const uint16_t* q_group, int G) {
    const int n16 = G * D / 8, lane = lane_id();
    if constexpr (kShort) {
#pragma unroll
      for (int k = 0; k < kSumLoads; ++k)
        r.e[k] = q_group[min(k * kRows + lane / kChannels, G - 1) * D + wave_id() * kChannels + lane % kChannels];
    }
#pragma unroll
    for (int k = 0; k < kQueryLoads; ++k)
      r.w[k] = reinterpret_cast<const uint4*>(q_group)[kShort && G == 1 ? lane % LPR : min((int)threadIdx.x + k * NT, n16 - 1)];
  }

  // To be called by the whole workgroup, like share_query behind it: here the query is waited for
  // and summed; what the caller sends out in between is on its way while the waves wait for each other.
  template <bool kShort>
  __device__ __forceinline__ void sum_query(const QueryRegs<kShort>& r, int G, unsigned char* stage) {
    uint4* raw = reinterpret_cast<uint4*>(stage);
    double* red = reinterpret_cast<double*>(stage + (size_t)G * D * 2);   // [2][D]
    const int n16 = G * D / 8, lane = lane_id();
    if (kShort && G == 1) {
      raw[lane % LPR] = r.w[0];
      float f[8];
      unpack8e<kHalf>(r.w[0], f);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        qp[i] = static_cast<double>(fmaxf(f[i], 0.f));
        qn[i] = static_cast<double>(fminf(f[i], 0.f));
      }
      return;
    }
#pragma unroll
    for (int k = 0; k < kQueryLoads; ++k) {
      raw[min((int)threadIdx.x + k * NT, n16 - 1)] = r.w[k];
    }
    TS_MARK(20);
    bool summed = false;
    if constexpr (kShort) {
      if (TS_USUALLY(G <= 8)) {
        static_assert(kRows * kSumLoads == 8 && kChannels <= 32, "a wave sums up to eight rows");
        double p = 0.0, n = 0.0;
#pragma unroll
        for (int k = 0; k < kSumLoads; ++k) {
          const float f = k * kRows + lane / kChannels < G ? elem_to_f32<kHalf>(r.e[k]) : 0.f;
          p += static_cast<double>(fmaxf(f, 0.f));
          n += static_cast<double>(fminf(f, 0.f));
        }
        // the lower half of the wave goes on with the positive sums, the upper half with the negative
        double s = sum_halves_f64(p, n);
        if (kChannels <= 16) s = sum_row_pairs_f64(s);
        if (kChannels <= 8) s += dpp_move_f64<kDppRowRor8>(s);
        if ((lane & 31) < kChannels) red[(lane >> 5) * D + wave_id() * kChannels + lane % kChannels] = s;
        summed = true;
      }
    }
    if (!summed) {
      __syncthreads();
      if (threadIdx.x < D) {
        const uint16_t* col = reinterpret_cast<const uint16_t*>(stage) + threadIdx.x;
        double p = 0.0, n = 0.0;
        for (int g = 0; g < G; ++g) {
          const float f = elem_to_f32<kHalf>(col[g * D]);
          p += static_cast<double>(fmaxf(f, 0.f));
          n += static_cast<double>(fminf(f, 0.f));
        }
        red[threadIdx.x] = p;
        red[D + threadIdx.x] = n;
      }
    }
    TS_MARK(21);
  }
  // (One head: the barrier is for the rows and for what the caller has asked for ahead of the sums,
  // see before_share of scan_finish.)
  template <bool kShort>
  __device__ __forceinline__ void share_query(int G, const unsigned char* stage) {
    __syncthreads();
    if (kShort && G == 1) return;
    const double* red = reinterpret_cast<const double*>(stage + (size_t)G * D * 2);
    const int cg = lane_id() % LPR;
#pragma unroll
    for (int i = 0; i < 8; ++i) { qp[i] = red[cg * 8 + i]; qn[i] = red[D + cg * 8 + i]; }
  }

  // Two chains of eight (the max terms, the min terms) instead of one of sixteen: with
  // four rows a wave has eight independent chains to interleave.
  __device__ __forceinline__ double row_partial(const uint4& mn, const uint4& mx) const {
    float lo[8], hi[8];
    unpack8e<kHalf>(mn, lo);
    unpack8e<kHalf>(mx, hi);
    double sp = 0.0, sn = 0.0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      sp = fma(qp[i], static_cast<double>(hi[i]), sp);
      sn = fma(qn[i], static_cast<double>(lo[i]), sn);
    }
    return sp + sn;
  }
};

// The metadata rows one wave has in flight: U wave-wide loads of min and of max,
// each covering PPW consecutive pages, the u-th starting at page base + u * rstep
// (rstep = PPW: the pages [base, base + PPI); larger when the groups of PPW pages
// are dealt out in turn to several workgroups).  Rows up to Pmax are always
// readable (whatever they hold), so the loads do not wait for the sequence length.
template <int D, bool kHalf = false, int NW = kWaves, int U = 4>
struct MetaTile {
  uint4 mn[U], mx[U];

  // Plimit >= 1.  Pages at or past Plimit read row Plimit - 1 instead (no branch
  // around the loads); reduce() never reports them.
  template <int U0 = 0, int U1 = U>
  __device__ __forceinline__ void load(const uint16_t* pmin_u, const uint16_t* pmax_u, int base,
                                       int Plimit, int rstep) {
    constexpr int LPR = ScoreLanes<D, kHalf>::LPR;
    const int lane = lane_id(), cg = lane % LPR, prow = lane / LPR;
#pragma unroll
    for (int u = U0; u < U1; ++u) {
      const int pg = min(base + u * rstep + prow, Plimit - 1);
      mn[u] = load_stream16(pmin_u + (size_t)pg * D + cg * 8);
      mx[u] = load_stream16(pmax_u + (size_t)pg * D + cg * 8);
    }
  }

  // The tile's scores: a lane ends up with at most one.  patch(min_row, max_row, page) may first
  // amend the row chunks this lane holds (a token appended in the same launch).
  struct Score {
    double s;
    int page;    // of this lane's score
    bool mine;   // it is this lane that reports it
  };
  template <typename Patch>
  __device__ __forceinline__ Score scores(const ScoreLanes<D, kHalf, NW>& ql, int base, int rstep, Patch patch) {
    constexpr int LPR = ScoreLanes<D, kHalf>::LPR;
    static_assert(U == 8 || U == 4 || U == 2 || U == 1, "rows folded in one butterfly");
    const int lane = lane_id(), cg = lane % LPR, prow = lane / LPR;
    double part[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      patch(mn[u], mx[u], base + u * rstep + prow);
      part[u] = ql.row_partial(mn[u], mx[u]);
    }
    // of a page's first eight lanes, 8 / U at a time hold the sum of a row, and the first of
    // those reports it
    constexpr int LPS = 8 / U;
    Score r;
    if constexpr (U == 8) r.s = group_sum8_f64<LPR>(part, cg);
    else if constexpr (U == 4) r.s = group_sum4_f64<LPR>(part, cg);
    else if constexpr (U == 2) r.s = group_sum2_f64<LPR>(part, cg);
    else r.s = group_sum1_f64<LPR>(part[0]);
    r.page = base + cg / LPS * rstep + prow;
    r.mine = cg % LPS == 0 && cg < 8;
    return r;
  }
  // sink(page, score) is called once per page < Pmax by one lane; pages >= Pb get -inf.
  template <typename Sink>
  __device__ __forceinline__ static void report(const Score& r, int Pb, int Pmax, Sink sink) {
    if (r.mine && r.page < Pmax) sink(r.page, r.page < Pb ? static_cast<float>(r.s) : -INFINITY);
  }
  template <typename Patch, typename Sink>
  __device__ __forceinline__ void reduce(const ScoreLanes<D, kHalf, NW>& ql, int base, int Pb, int Pmax,
                                         int rstep, Patch patch, Sink sink) {
    report(scores(ql, base, rstep, patch), Pb, Pmax, sink);
  }
  // Everything of the tile has arrived (the first use of its registers, pinned to this place).
  __device__ __forceinline__ void arrived() {
#pragma unroll
    for (int u = 0; u < U; ++u)
      asm volatile("" : "+v"(mn[u].x), "+v"(mn[u].y), "+v"(mn[u].z), "+v"(mn[u].w), "+v"(mx[u].x),
                   "+v"(mx[u].y), "+v"(mx[u].z), "+v"(mx[u].w));
  }
};

// Scoring one (sequence, KV head) is split in two so that a kernel can put the
// first loads of a unit as early as it likes (before unrelated set-up work):
// scan_issue sends out the query rows and the wave's first metadata tile,
// scan_finish does everything else.  A wave's iterations are it = first_iter,
// first_iter + iter_stride, ..., each covering U groups of PPW consecutive pages
// (PPI pages in all).  With gs == 1 these are the pages [it * PPI, (it + 1) * PPI);
// in general the sequence's groups of PPW pages are dealt out in turn to gs
// parties, and the caller, party goff, gets the groups (it * U + u) * gs + goff:
// its share is then spread as evenly as can be over the whole sequence.
//
// R = 0: any number of iterations of U = 4.  R > 0: the build for launches in which a wave has at
// most R groups of pages: one tile and, with more than one group, a last group of its own.
template <int D, bool kHalf = false, int NW = kWaves, int R = 0>
struct ScanRegs {
  static constexpr int U = R == 0 ? 4 : (R == 1 ? 1 : R - 1);
  static constexpr bool kTail = R > 1;
  static constexpr int kHead = R < 3 ? U : 2;                     // groups asked for ahead of the query's sums
  static constexpr int PPI = ScoreLanes<D, kHalf, NW>::PPW * U;   // pages one wave covers per iteration
  typename ScoreLanes<D, kHalf, NW>::template QueryRegs<(R > 1)> q;
  MetaTile<D, kHalf, NW, U> tile;
  MetaTile<D, kHalf, NW, 1> tail;
};

struct Nothing {
  __device__ __forceinline__ void operator()() const {}
};

template <int D, bool kHalf, int NW, int R>
__device__ __forceinline__ void scan_issue_query(ScanRegs<D, kHalf, NW, R>& r, const uint16_t* q_group, int G) {
  ScoreLanes<D, kHalf, NW>::template issue_query<(R > 1)>(r.q, q_group, G);
}
template <int D, bool kHalf, int NW, int R>
__device__ __forceinline__ void scan_issue_tile(ScanRegs<D, kHalf, NW, R>& r, const uint16_t* pmin_u,
                                                const uint16_t* pmax_u, int Pmax, int first_iter,
                                                int gs = 1, int goff = 0) {
  using Regs = ScanRegs<D, kHalf, NW, R>;
  constexpr int PPW = ScoreLanes<D, kHalf>::PPW;
  r.tile.template load<0, Regs::kHead>(pmin_u, pmax_u, first_iter * Regs::PPI * gs + goff * PPW, Pmax, PPW * gs);
}
// The rest of the first loads.  A compute unit's memory pipeline takes the loads of eight waves only as
// earlier ones drain, and a wave whose loads are not taken stands still: with all of them ahead of the
// query's sums, those were ready 3.7 us after the kernel's entry (16 x 4 units of 1024 pages) where the
// query had arrived after 0.9.  Two groups go out ahead of the sums, the others between them and the
// barrier: 18.8 -> 18.4 us, one query head each (8 x 16 units of 512 pages) 17.05 -> 16.95, 4 x 4 of 4097 pages
// 19.2 -> 18.5, the INT8 cache 17.95 -> 17.55 (with the sums' own shorter way).
template <int D, bool kHalf, int NW, int R>
__device__ __forceinline__ void scan_issue_rest(ScanRegs<D, kHalf, NW, R>& r, const uint16_t* pmin_u,
                                                const uint16_t* pmax_u, int Pmax, int first_iter, int iter_stride,
                                                int gs, int goff) {
  using Regs = ScanRegs<D, kHalf, NW, R>;
  constexpr int PPW = ScoreLanes<D, kHalf>::PPW, PPI = Regs::PPI;
  if constexpr (!Regs::kTail) return;
  asm volatile("" ::: "memory");
  r.tile.template load<Regs::kHead, Regs::U>(pmin_u, pmax_u, first_iter * PPI * gs + goff * PPW, Pmax, PPW * gs);
  if constexpr (Regs::kTail)
    r.tail.load(pmin_u, pmax_u, (iter_stride * PPI + first_iter * PPW) * gs + goff * PPW, Pmax, 0);
  __builtin_amdgcn_sched_barrier(0);
}

// `before_share` runs ahead of the barrier of share_query, `after_query` once the query is in
// registers; it returns Pb.  Must be
// called by the whole workgroup (the query may go through LDS, q_stage, with
// barriers).
//
// fill_to_pmax: the sink also wants the -inf of the pages from Pb to Pmax (a
// caller that writes scores out for others to read); otherwise the scan stops at
// the sequence's last page.
//
// kBranchless: the next tile is fetched without a branch around the loads even
// when there is none (the clamped loads then cost a cache line or two), so the
// compiler can count outstanding loads and overlap the fetch with the reduction
// of the current tile.  That is what a latency-bound launch wants; a launch with
// thousands of units is bound by bandwidth and overlaps across workgroups, and
// there the plain branch is a little cheaper.  (Putting the branch around the
// fetch AND the reduction it overlaps with, two copies of the reduction, so that
// no load is issued where there is no next tile, measured 0.7 us slower on the
// 16-sequence configuration.)
template <int D, bool kBranchless, bool kHalf, int NW, int R, typename AfterQuery, typename Patch, typename Sink,
          typename BeforeReport = Nothing, typename BeforeShare = Nothing>
__device__ __forceinline__ void scan_finish(ScanRegs<D, kHalf, NW, R>& r, const uint16_t* pmin_u,
                                            const uint16_t* pmax_u, int G, int Pmax, int first_iter,
                                            int iter_stride, unsigned char* q_stage,
                                            AfterQuery after_query, Patch patch, Sink sink,
                                            int gs = 1, int goff = 0, bool fill_to_pmax = true,
                                            BeforeReport before_report = BeforeReport{},
                                            BeforeShare before_share = BeforeShare{}) {
  using Regs = ScanRegs<D, kHalf, NW, R>;
  constexpr int PPW = ScoreLanes<D, kHalf>::PPW, PPI = Regs::PPI;
  const int rstep = PPW * gs;
  TS_MARK(19);
  ScoreLanes<D, kHalf, NW> ql;
  ql.template sum_query<(R > 1)>(r.q, G, q_stage);
  scan_issue_rest(r, pmin_u, pmax_u, Pmax, first_iter, iter_stride, gs, goff);
  before_share();
  ql.template share_query<(R > 1)>(G, q_stage);
  TS_MARK(16);
  const int Pb = after_query();
  const int limit = uniform(fill_to_pmax ? Pmax : Pb);
  // only the first tile is fetched blind; later ones stop at the sequence's
  // last page (pages >= Pb still get their -inf through the sink)
  int base = first_iter * PPI * gs + goff * PPW;   // first page of the tile's first group
  if constexpr (R > 0) {
    const int end = min(Pmax, limit);
    const auto s = r.tile.scores(ql, base, rstep, patch);
    // (waited for here, ahead of the stores of the sink: behind them a wait would be one for
    // their acknowledgement too)
    if constexpr (Regs::kTail) r.tail.arrived();
    before_report();
    r.tile.report(s, Pb, end, sink);
    if constexpr (Regs::kTail) {
      const int last = (iter_stride * PPI + first_iter * PPW) * gs + goff * PPW;
      if (uniform(last) < end) r.tail.reduce(ql, last, Pb, end, 0, patch, sink);
    }
  } else if (kBranchless) {
    // The first tile is reduced whether or not it holds a page below the limit (the sink
    // sees no page at or past the limit).  With a path around the loop the tile's loads
    // would still be in flight where the two paths meet, and the compiler, which cannot
    // count across such a join, would wait there for EVERY outstanding memory operation:
    // the write-through stores of the scores included, a trip to memory and back in front
    // of the barrier that follows (measured, with the arrival count below: 0.3-0.5 us).
    do {
      const int next = base + iter_stride * PPI * gs;
      auto cur = r.tile;
      r.tile.load(pmin_u, pmax_u, next, max(Pb, 1), rstep);
      cur.reduce(ql, base, Pb, min(Pmax, limit), rstep, patch, sink);
      base = next;
    } while (base < limit);
  } else {
    while (base < limit) {
      const int next = base + iter_stride * PPI * gs;
      auto cur = r.tile;
      if (next < Pb) r.tile.load(pmin_u, pmax_u, next, Pb, rstep);
      cur.reduce(ql, base, Pb, Pmax, rstep, patch, sink);
      base = next;
    }
  }
}

}  // namespace ts
