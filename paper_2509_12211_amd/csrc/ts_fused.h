// The kernels that depend on the cache format (attention over the selected
// pages, and Algorithm 1 in one launch) and their host-side launch logic.  Each
// format and head_dim is compiled in a file of its own (fmt_*.hip instantiate
// launch_fused_format / launch_attention_format / append_capacity_format for
// one pair each, so that they build in parallel); tinyserve.hip holds the entry
// points and everything that does not depend on the format.
#pragma once
#include "../../include/tinyserve.h"

#include <hip/hip_runtime.h>

#include <map>
#include <mutex>
#include <tuple>
#include <utility>

#include "ts_attend.h"
#include "ts_device.h"
#include "ts_meta.h"
#include "ts_score.h"
#include "ts_select.h"
#include "ts_shares.h"

namespace ts {


// ---------------------------------------------------------------------------
// Work decomposition shared by host and device
// ---------------------------------------------------------------------------
// A unit is one (sequence, KV head).  A unit is worked on by a cluster of g
// workgroups: each scores 1/g of the unit's pages and attends 1/g of its
// selected pages.  g is chosen so that units * g is about one workgroup (eight
// waves) per compute unit; with thousands of units g = 1 and nothing is exchanged
// between workgroups at all.
constexpr int kCtrlWords = 64;   // control words at the head of the workspace
constexpr int kCtrlError = 2;    // sticky: a bounded wait expired
constexpr int kCtrlEpoch = 16;   // launches of the fused kernel with clusters so far (own 64-byte line)
constexpr int kCtrlArrive = 32;  // workgroups of the current launch that have read the epoch (own line)
// Behind them, for launches of up to 256 workgroups whose units may be shared without waiting:
// members of a unit that have handed on their partial, zero between launches.  (At the front of
// the workspace like the control words: layouts that use the same memory in turn find it zero.)
constexpr int kCtrlDone = kCtrlWords;
constexpr int kCtrlArea = kCtrlWords + 256;
constexpr int kSpinLimit = 1 << 20;  // polls (a few hundred ns each) before a wait gives up
constexpr int kTargetWorkgroups = 256;
constexpr int kMaxCluster = 64;
// Per-unit counters are bumped by every member of a cluster at about the same
// time.  Each gets a 256-byte slot of its own while the batch is small: sixteen
// units' counters packed into one 64-byte line made every workgroup of the
// launch hammer the same line (measured: 6 us of waiting with 16 x 16
// workgroups).  Only clusters (g > 1, at most a few hundred units) use the
// counters, so large batches keep them packed.
constexpr int kCounterPadUnits = 512;
constexpr int kCounterPadStride = 64;   // int32 words

struct Plan {
  int units;          // B * Hkv
  int g;              // workgroups per unit (= attention splits = score slices)
  int chunk;          // selected pages per workgroup
  size_t off_unit;    // int32 [units * cstride]: arrival counters of the staged attention
  int cstride;        // words between the counters of consecutive units
  size_t off_scores;  // {fp32 score, uint32 launch tag} [units][Pmax]
  size_t off_part;    // [units][g][G][d+2]: {fp32, launch tag} words (fused) or fp32 (staged attention)
  size_t total;
  size_t lds_fused;   // dynamic LDS of the fused kernel
  size_t lds_list;    // ... in front of this workgroup's selected pages, which come last
  bool small_units;   // many small units: small_units_decode_kernel
  bool shares;        // workgroups by the work if the lengths ask for it, per_head of them per KV head:
  int per_head;       // shares_decode_kernel (query-aware), dense_shares_kernel (every token)
  bool rounds;        // every token, two rounds of units and more: dense_rounds_kernel
  bool shares_uniform;   // ... also where all sequences have the same budget
  float min_rows;     // ... that is, if it saves the busiest workgroup that many metadata rows
};

static size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

struct FusedParams {
  AttendParams at;
  const uint16_t* page_min;
  const uint16_t* page_max;
  uint64_t* scores;     // [units][Pmax] exchange buffer (workspace): score | launch tag << 32
  float* scores_out;    // nullable, caller's
  int32_t* sel_out;     // nullable [units][Kmax]
  int32_t* sel_count;   // nullable [B]
  const int32_t* topk_per_seq;
  int32_t* ctrl;        // control words
  // One token per sequence appended by the same launch (k_new == nullptr: none).
  // (the pool, the metadata and the lengths are then written through the
  // pointers above: the caller's buffers are writable, the const is this
  // library's view of them in the calls that only read)
  const uint16_t* k_new;   // [B][Hkv][D]
  const uint16_t* v_new;
  int topk, S, units, g, cstride, B;
  int keep_first, keep_last;   // pages kept whatever their score (0, 0: the paper's selection)
  int spin_limit;              // polls before a cross-workgroup wait gives up
  int xcds;                    // > 1: clusters laid out one per XCD over that many XCDs (see cluster_of)
  int n_arrive;                // workgroups of the launch that count themselves in
  FastDiv div_g, div_xcds, div_hkv;   // divisions by g, xcds and the number of KV heads
  // (last: what stands in front of these is fetched in few loads, see decode_units)
  int per_head;                // shares: workgroups per KV head
  float inv_g, min_rows;       // ... see Plan
};

// What the first loads of a workgroup are addressed with, as kernel arguments of their own in front
// of the struct: these fourteen words are in scalar registers when a wave starts (the flag
// -amdgpu-kernarg-preload-count of the build), where the struct is a trip to memory away.  The
// loads go out 0.6 us after the kernel's entry instead of 0.9, and with them ends a launch: 4 units
// of 12 workgroups 10.0 -> 9.7 us, 16 of 16 (131072 tokens each) 19.6 -> 19.2.
struct FirstArgs {
  const uint16_t* q;
  const uint16_t* page_min;
  const uint16_t* page_max;
  const uint16_t* first;       // one group of pages a wave: the new tokens' keys and values;
  const uint16_t* second;      // more: the control words and the lengths
  uint32_t shape;              // pages of a table row | g << 16 | (G - 1) << 24 | log2 of the XCDs << 28
  uint32_t units;
  uint32_t magic_g, magic_hkv; // FastDiv::magic
  __device__ __forceinline__ const int32_t* ctrl() const { return reinterpret_cast<const int32_t*>(first); }
  __device__ __forceinline__ const int32_t* seq_lens() const { return reinterpret_cast<const int32_t*>(second); }
  __device__ __forceinline__ int Pmax() const { return (int)(shape & 0xffffu); }
  __device__ __forceinline__ int g() const { return (int)((shape >> 16) & 0xffu); }
  __device__ __forceinline__ int G() const { return (int)((shape >> 24) & 15u) + 1; }
  __device__ __forceinline__ int xcd_bits() const { return (int)(shape >> 28); }
};
static_assert(TS_MAX_PAGES_PER_SEQ <= 0xffff && kMaxCluster <= 0xff, "fields of FirstArgs::shape");

// Which cluster a workgroup belongs to, and as which member.  The hardware deals
// consecutive workgroup ids out to the XCDs in turn (on a part with eight of them,
// ids congruent modulo 8 share a die; the first id of a launch goes wherever the
// previous launch left off; ts_debug_xcc_ids lets a test look), and each XCD has an
// L2 of its own.
// With xcds > 1 the g members of a cluster are the workgroups
// id = xcd + xcds * (k * g + member): all on one XCD.  Nothing depends on it for
// correctness (everything the members hand each other goes through agent-scope
// accesses whichever die they run on); measured, it is worth 0.5 us on a single
// short sequence and nothing either way on the 16- and 4-sequence batches, whose
// exchanges wait for the slowest member rather than for the hand-off itself.  The
// host asks for it only when the grid is a multiple of xcds * g workgroups;
// clusters beyond the last unit then have nothing to do.  Otherwise the members
// are consecutive ids.
struct ClusterSlot { int cluster, member; };
__device__ __forceinline__ ClusterSlot cluster_of(int wg, const FastDiv& g, const FastDiv& xcds,
                                                  bool by_xcd) {
  ClusterSlot c;
  if (by_xcd) {
    const int slot = fast_div(wg, xcds), xcd = wg - slot * (int)xcds.d;
    c.cluster = fast_div(slot, g);
    c.member = slot - c.cluster * (int)g.d;
    c.cluster = c.cluster * (int)xcds.d + xcd;
  } else {
    c.cluster = fast_div(wg, g);
    c.member = wg - c.cluster * (int)g.d;
  }
  return c;
}

// The same from the first arguments: g >= 2, the number of XCDs a power of two (1: consecutive ids).
__device__ __forceinline__ ClusterSlot cluster_of(int wg, const FirstArgs& f) {
  const int bits = f.xcd_bits(), slot = wg >> bits, xcd = wg & ((1 << bits) - 1);
  const int c = (int)__umulhi((uint32_t)slot, f.magic_g);
  return ClusterSlot{(c << bits) + xcd, slot - c * f.g()};
}

__device__ __forceinline__ int pages_of(int len, int S) { return (len + S - 1) / S; }

// grid (g, units).  The last workgroup of a unit to deposit its partial merges
// them (unit_done counts arrivals and is left at zero again).
// A few microseconds of work behind a chain of look-ups: the count, the list, the table, the tiles,
// each a trip to memory.  A wave asks for the list entries and table rows of its first fragments
// without waiting for the count (the list is readable to its end), and its first arguments come
// in registers (see FirstArgs): 64 units of 128 kept pages of 16, 12.8 -> 12.1 us, of 256 of 8 12.6 -> 12.2.
template <int D, int S, bool kInt8, bool kHalf>
__global__ __launch_bounds__(kThreads) void sparse_attention_kernel(
    const uint16_t* q, const int32_t* sel, const int32_t* sel_count, const int32_t* seq_lens,
    const int32_t* block_table, uint32_t magic_hkv, int chunk, int Kmax, int shape, AttendParams p,
    int32_t* unit_done, int cstride) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int s_last;
  constexpr int NS = PageGeom<S>::NS;
  const int Pmax = shape & 0xffff, G = shape >> 16;
  const int u = blockIdx.y, b = fast_div(u, FastDiv{1, magic_hkv}), split = blockIdx.x;
  const int32_t* bt_row = block_table + (size_t)b * Pmax;
  // sel == nullptr: the dense baseline, every page of the sequence in order
  const int32_t* list = sel ? sel + (size_t)u * Kmax : bt_row;
  const int readable = sel ? Kmax : Pmax;
  const int len = seq_lens[b], listed = (sel ? sel_count : seq_lens)[b];
  FirstEntries<S> ready;
  int first_e[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    // (lanes past the chunk ask for its last entry: a table row each would be a line each)
    first_e[s] = split * chunk + min(first_entry<kWaves, S>(s), chunk - 1);
    ready.j[s] = list[min(first_e[s], readable - 1)];
  }
  QOperand<D, kInt8> qop;
  qop.load(q + (size_t)u * G * D, G);
  __builtin_amdgcn_sched_barrier(0);   // (all of these are on their way before one is waited for)
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    ready.j[s] = sel ? ready.j[s] : first_e[s];
    ready.phys[s] = bt_row[min(max(ready.j[s], 0), Pmax - 1)];   // (only looked at where the entry is one)
  }
  const int Kb = uniform(sel ? max(0, min(listed, Kmax)) : min((len + S - 1) / S, Kmax));
  const int h = u - b * p.Hkv;
  const int c0 = min(split * chunk, Kb), count = min(c0 + chunk, Kb) - c0;
  const NewToken none{-1, 0, q, q};
  attend_split<kWaves, D, S, false, kInt8, kHalf, true>(
      p, b, h, [&] { return SplitPlace{p.n_split, split, (size_t)u * p.n_split}; }, count, len, none,
      [&](int i) { return sel ? list[c0 + i] : c0 + i; }, [&](int j) { return bt_row[j]; },
      reinterpret_cast<float*>(smem), 0u, nullptr, 0, &qop, ready);
  if (p.n_split == 1) return;
  stores_complete();
  __syncthreads();
  if (threadIdx.x == 0) s_last = atomic_add_agent(&unit_done[u * cstride], 1) == p.n_split - 1;
  __syncthreads();
  if (!uniform(s_last)) return;
  combine_splits<D>(p, b, h, (size_t)u * p.n_split, p.n_split, reinterpret_cast<float*>(smem));
  if (threadIdx.x == 0) atomic_store_agent(&unit_done[u * cstride], 0);
}

// ---------------------------------------------------------------------------
// Shares in proportion to the work (ragged batches).
//
// With clusters of one size a launch over sequences of different lengths ends with the
// longest one, while the workgroups of the short ones have long left.  Here the workgroups
// of a launch, N per KV head, are dealt out to the sequences by the bytes each has to
// read: every wave works the same shares out for itself from the lengths, a lane per
// sequence, and finds the one that belongs to its workgroup.
// ---------------------------------------------------------------------------
constexpr int kBalanceSeqs = kWave;   // a lane per sequence
constexpr int kShareWords = 8;        // of LDS, in which a workgroup's place in its unit waits until it is needed
constexpr int kBalanceTryAll = 12;    // sequences up to which trying all shares at once is the quicker way

struct UnitShare {
  int b, h, member, g;   // g == 0: nothing to do
  int chunk;             // selected pages per member
  int part_row;          // the cluster's first row of the partial area
  int L, K;              // the sequence's length and page budget as given
};

// The smallest share t (rows per workgroup) with which the members of all sequences fit into N
// workgroups.  Lane s < B comes with sequence s, the other lanes with nothing.  INFINITY: one
// workgroup each.  Not below total / N nor below what a member reads in full (`lo`); total /
// (N - B) on top of the latter does in any case, and so does one workgroup each.
__device__ __forceinline__ float share_floor(int N, const SeqWork& w) {
  return fmaxf(wave_sum_f32(w.rows) * __builtin_amdgcn_rcpf((float)N), wave_max_f32(w.whole));
}
__device__ __forceinline__ float smallest_share(int B, int N, const SeqWork& w, float lo) {
  const int lane = lane_id();
  const bool on = lane < B;
  const float spread = wave_max_f32(w.whole) + wave_sum_f32(w.rows) * __builtin_amdgcn_rcpf((float)max(N - B, 1));
  const float hi = 1.001f * fminf(wave_max_f32(w.whole + w.rows), spread);
  float best = INFINITY;
  if (B <= kBalanceTryAll) {   // 64 values of t at once, a lane each
    const float t = fmaf(fmaxf(hi - lo, 0.f), (float)lane * (1.f / 63.f), lo);
    float n = 0.f;
    for (int s = 0; s < B; ++s) {
      SeqWork ws;
      ws.whole = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w.whole), s));
      ws.rows = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w.rows), s));
      ws.most = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w.most), s));
      n += members_of(ws, __builtin_amdgcn_rcpf(t - ws.whole));
    }
    const uint64_t fits = __ballot(n <= (float)N);
    if (fits) best = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), __builtin_ctzll(fits)));
  } else {                       // halving, a lane per sequence
    float a = lo, z = hi;
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      const float mid = i == 0 ? z : 0.5f * (a + z);
      if (wave_sum_f32(on ? members_of(w, __builtin_amdgcn_rcpf(mid - w.whole)) : 0.f) <= (float)N) {
        z = mid;
        best = mid;
      } else {
        a = mid;
      }
    }
  }
  return best;
}

// The share of workgroup blockIdx.x at t rows per workgroup.  Lane s < B comes with sequence s:
// its work, the pages Kb to deal out to its members; L and K are handed through.
template <int S>
__device__ __forceinline__ UnitShare take_share(int B, int N, int Hkv, const FastDiv& div_hkv, const SeqWork& w,
                                                float t, int Kb, int L, int K) {
  const int gl = lane_id() < B ? (int)members_of(w, __builtin_amdgcn_rcpf(t - w.whole)) : 0;
  const int incl = wave_inclusive_sum(gl);
  // workgroup x: KV head x mod Hkv (so that with eight heads or a multiple a cluster stays on
  // one XCD), place x / Hkv among the head's N
  const int place = fast_div(blockIdx.x, div_hkv);
  UnitShare u{};
  u.h = (int)blockIdx.x - place * Hkv;
  const uint64_t after = __ballot(incl > place);
  if (after == 0ull) return u;   // more workgroups than members
  const int s = __builtin_ctzll(after);
  const int first = __builtin_amdgcn_readlane(incl - gl, s);
  u.b = s;
  u.g = __builtin_amdgcn_readlane(gl, s);
  u.member = place - first;
  u.part_row = u.h * N + first;
  u.L = __builtin_amdgcn_readlane(L, s);
  u.K = __builtin_amdgcn_readlane(K, s);
  const int kept = __builtin_amdgcn_readlane(Kb, s);
  u.chunk = max((int)ceilf((float)kept * __builtin_amdgcn_rcpf((float)u.g) - 1e-3f), 1);
  if (u.chunk * u.g < kept) ++u.chunk;   // (the reciprocal is a bit short)
  if (S < 16) u.chunk = (u.chunk + 3) / 4 * 4;   // whole groups of small pages
  return u;
}

// Whether the batch goes by shares, and this workgroup's if so.  Lane s < B comes with the
// length L and the budget K of sequence s (the lanes past them with the last one's).  Every wave
// of the launch works it out from the same numbers by the same operations.
// Batches of one length leave at the first test: there is nothing to gain, whatever the block
// tables and the pool have room for.  The next one asks what shares could save at the very
// best, and only then they are worked out.
template <int S, bool kApp, bool kExchange>
__device__ __forceinline__ bool by_shares(const FusedParams& p, int L, int K, UnitShare& share) {
  const AttendParams& at = p.at;
  if (__ballot(((L ^ uniform(L)) | (K ^ uniform(K))) != 0) == 0ull) return false;
  const bool on = lane_id() < p.B;
  const int len = L + (kApp && L / S < at.Pmax ? 1 : 0);
  const int P = min(pages_of(len, S), at.Pmax), Kb = max(0, min(min(K, P), at.Kmax));
  SeqWork w = seq_work(P, Kb, at.Kmax, S, kExchange);
  if (!on) w = SeqWork{0.f, 0.f, 0.f};
  const float even = wave_max_f32(even_rows(P, Kb, at.chunk, S, p.inv_g));
  const float lo = share_floor(p.per_head, w);
  if (even - lo < p.min_rows) return false;
  const float t = smallest_share(p.B, p.per_head, w, lo);
  if (even - t < p.min_rows) return false;
  share = take_share<S>(p.B, p.per_head, at.Hkv, p.div_hkv, w, t, Kb, L, K);
  return true;
}

// Attention over every cached token, the sequences' workgroups in proportion to their pages.
// Bound by HBM, and by how the work divides over the compute units: the attention's registers
// leave room for one workgroup of eight waves each, so a launch runs in rounds of 256, and
// every round past the first pays another start (1.5-5 us) and ends with a partial one.
// Clusters of one size over the longest possible sequence, four rounds of them, also left
// the work of a ragged batch where the round-robin over the XCDs put it.  One round, dealt
// out by the lengths on the device, against four (bf16): 16 sequences x 4 KV heads of 16 K
// tokens, 64 channels, 56.3 -> 48.0 us (5.6 TB/s); 4 x 4 of 128 K 118 -> 93 (5.8); 3 x 8 of
// 16 K, 128 channels, 67 -> 43; 7 x 8 of 4-50 K 156 -> 132; 24 x 8 of 512-8192 109 -> 94;
// 24 layouts of 12 to 256 units 1.03 to 1.9 times faster.
template <int D, int S, bool kHalf>
__global__ __launch_bounds__(kThreads) void dense_shares_kernel(AttendParams p, int32_t* unit_done,
                                                                int cstride, int B, int per_head,
                                                                FastDiv div_hkv) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int s_last;
  const int lane = lane_id(), len = p.seq_lens[min(lane, B - 1)];
  const int pages = lane < B ? max(0, min(pages_of(len, S), p.Pmax)) : 0;
  const SeqWork w = lane < B ? SeqWork{0.f, fmaxf((float)pages, 1.f), (float)min((pages + 3) / 4, kMaxCluster)}
                             : SeqWork{0.f, 0.f, 0.f};
  const float t = smallest_share(B, per_head, w, share_floor(per_head, w));
  const UnitShare share = take_share<S>(B, per_head, p.Hkv, div_hkv, w, t, pages, len, pages);
  const int g = uniform(share.g);
  if (g == 0) return;   // a workgroup too many
  const int b = share.b, h = share.h, u = b * p.Hkv + h;
  const int c0 = min(share.member * share.chunk, share.K), count = min(c0 + share.chunk, share.K) - c0;
  const int32_t* bt_row = p.block_table + (size_t)b * p.Pmax;
  const NewToken none{-1, 0, p.q, p.q};
  attend_split<kWaves, D, S, false, false, kHalf>(
      p, b, h, [&] { return SplitPlace{g, share.member, (size_t)share.part_row}; }, count, share.L, none,
      [&](int i) { return c0 + i; }, [&](int j) { return bt_row[j]; }, reinterpret_cast<float*>(smem));
  if (g == 1) return;
  stores_complete();
  __syncthreads();
  if (threadIdx.x == 0) s_last = atomic_add_agent(&unit_done[u * cstride], 1) == g - 1;
  __syncthreads();
  if (!uniform(s_last)) return;
  combine_splits<D>(p, b, h, (size_t)share.part_row, g, reinterpret_cast<float*>(smem));
  if (threadIdx.x == 0) atomic_store_agent(&unit_done[u * cstride], 0);
}

// Attention over every cached token, two rounds of units and more: one workgroup each, or the
// sequences longer than half the longest in two parts, as the lengths have it (see
// rounds_of).  A workgroup alone gets 35 GB/s of the 5800, so that a few sequences much
// longer than the rest would decide the finish time.
// Workgroup x < units has unit x or its first part, and workgroup units + x the second: those
// with nothing to do come last, when the compute units run out of work anyway.  With a few
// long sequences workgroups 2 u and 2 u + 1 have unit u, so that their second parts do not come last
// (64 x 8 units, three of 16 K tokens and the rest of 800: 142 -> 117 us; 600 units of 300 tokens the
// other way round, 21.6 against 20.4).
// bf16, against two parts at half the table's width for all, split with its partials whatever
// the length: 48 x 16 units of 500-4096 tokens, pages of 32, 105.4 -> 79.4 us; 31 x 32 of 100-2000,
// 128 channels, 131 -> 97; 64 x 8 of 4096, 128 channels, 181 -> 173; 56 x 16 of 2-8 K 229 -> 210.
template <int D, int S, bool kHalf>
__global__ __launch_bounds__(kThreads) void dense_rounds_kernel(AttendParams p, int32_t* unit_done,
                                                                int cstride, int B, int units,
                                                                FastDiv div_hkv) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int s_last;
  const int x = (int)blockIdx.x, u_far = x < units ? x : x - units, u_near = x >> 1;
  const int len_far = p.seq_lens[fast_div(u_far, div_hkv)], len_near = p.seq_lens[fast_div(u_near, div_hkv)];
  int total = 0, longest = 0;
  for (int i = lane_id(); i < B; i += kWave) {
    const int pages = max(0, min(pages_of(p.seq_lens[i], S), p.Pmax));
    total += pages;
    longest = max(longest, pages);
  }
  total = __builtin_amdgcn_readlane(wave_inclusive_sum(total), 63);
  longest = (int)wave_max_u32((uint32_t)longest);
  const Rounds way = (Rounds)uniform(rounds_of(total, longest, B, units));
  const bool near = way == kFewLong;
  const int split = near ? x & 1 : (int)(x >= units), u = near ? u_near : u_far;
  const int b = fast_div(u, div_hkv), h = u - b * p.Hkv, len = uniform(near ? len_near : len_far);
  const int pages = max(0, min(pages_of(len, S), p.Pmax));
  int chunk = longest;
  if (way != kWhole) {
    chunk = (longest + 1) / 2;
    if (S < 16) chunk = (chunk + 3) / 4 * 4;   // whole groups of small pages
  }
  const int n_split = pages > chunk ? 2 : 1;
  if (split >= n_split) return;
  const int c0 = split * chunk, count = min(chunk, pages - c0);
  const int32_t* bt_row = p.block_table + (size_t)b * p.Pmax;
  const NewToken none{-1, 0, p.q, p.q};
  attend_split<kWaves, D, S, false, false, kHalf>(
      p, b, h, [&] { return SplitPlace{n_split, split, (size_t)u * 2}; }, count, len, none,
      [&](int i) { return c0 + i; }, [&](int j) { return bt_row[j]; }, reinterpret_cast<float*>(smem));
  if (n_split == 1) return;
  stores_complete();
  __syncthreads();
  if (threadIdx.x == 0) s_last = atomic_add_agent(&unit_done[u * cstride], 1) == 1;
  __syncthreads();
  if (!uniform(s_last)) return;
  combine_splits<D>(p, b, h, (size_t)u * 2, 2, reinterpret_cast<float*>(smem));
  if (threadIdx.x == 0) atomic_store_agent(&unit_done[u * cstride], 0);
}

// ---------------------------------------------------------------------------
// Fused kernel (Algorithm 1 in one launch).
//
// Workgroup w belongs to cluster w / g as member w % g; a cluster takes units
// cluster, cluster + n_clusters, ...  For each unit a member
//   1. scores every g-th group of the unit's pages (metadata loads are issued
//      before anything else; the unit's block-table row is copied to LDS
//      meanwhile),
//   2. g > 1: publishes each score as a word tagged with the launch tag and
//      polls (bounded) the unit's score row until every word carries the tag,
//      counting the scores into the selection's bins as they come in;
//      g == 1: the scores never leave LDS,
//   3. runs the top-K selection itself (every member computes the same list),
//   4. attends its own 1/g of the selected pages,
//   5. g > 1: hands its partial softmax state on as words tagged with the launch
//      tag; the cluster's last member polls for all g partials (data and flag
//      arrive together) and merges them, or each member its slices of the
//      output in clusters of nine members and more (kDealt).
// Members only ever wait for members of their own cluster, all of which are
// resident: the host launches at most as many workgroups as fit on the device
// at once.  Every wait is bounded and raises the workspace's error word.
//
// Every thread-0-only block sits between two barriers and every value that
// steers a branch around a barrier is pinned uniform.
// ---------------------------------------------------------------------------
//
// kLoop = false is the build for launches in which every workgroup has exactly one
// unit (all but clusters of a forced size that do not fit the device).  Without
// the loop around the body the compiler has nothing to hoist: with it, every
// unit-independent value of the whole body (several hundred instructions, most
// of them spilled at once) is computed ahead of the first unit, that is ahead of
// the first load.
//
// kApp = true is the build that first appends one token per sequence
// (ts_append_and_decode); the plain build carries none of its registers.  With
// the INT8 cache the token's bf16 rows are quantised in the launch, by the few
// waves that need the codes (the one that scores the token's page, the one that
// writes the pool, the one that attends the page).
//
// The host launches at most one workgroup (eight waves) per compute unit, that is
// two waves per SIMD: saying so lets the compiler schedule for latency with the
// registers of that occupancy instead of saving registers for waves that never
// come (measured: 0.5 us of 26 on the 16-sequence configuration).
//
// NW: waves per workgroup.
//
// kCluster says whether a unit is shared by several workgroups (p.g > 1): the
// build for one workgroup per unit carries nothing of the exchange, the build
// for clusters nothing of the selection's stand-alone first stages.
//
// kRound > 0: a wave scores its share of the pages in one round of at most that many groups (see
// ScanRegs), and what the first loads need comes in the arguments in front (f).
//
// kInRegs: what the first loads are addressed with is in registers already (see with_args).
//
// kDecide: the lengths decide between clusters of one size and shares in proportion to the
// work (see by_shares), ahead of the first loads.
//
// kDealt: clusters of more than kMergedByOne members deal the merge of their partials out (see attend_split).
template <int NW, int D, int S, bool kLoop, bool kApp, bool kInt8, bool kHalf, bool kCluster,
          bool kDecide = false, int kRound = 0, bool kInRegs = false, bool kDealt = kDecide>
__device__ __forceinline__ void decode_units(const FusedParams& p, const FirstArgs& f = FirstArgs{}) {
  constexpr bool kFirst = kRound > 0;
  static_assert(!kFirst || (kCluster && !kLoop && !kDecide), "one round of scoring: clusters with one unit each");
  constexpr int NT = NW * kWave;
  static_assert(!(kLoop && kApp), "the append is folded only into the loop-free build");
  static_assert(!kLoop || kCluster, "a single workgroup per unit needs no loop");
  static_assert(!(kDecide && kLoop), "shares are worked out once, at the head");
  static_assert(!kInRegs || (!kApp && !kCluster && !kDecide), "leading arguments of with_args: one workgroup per unit, no append");
  extern __shared__ __align__(16) unsigned char smem[];
  TS_MARK_INIT();
  TS_MARK(22);
  const AttendParams& at = p.at;
  // Everything the unit's first loads are addressed with is asked for here, ahead of the
  // first branch: the compiler fetches a kernel argument in the block that first uses it,
  // and arguments first used behind the tests below came in a second and a third trip to
  // memory, each waited for, before the first load could go out.
  // In the builds of one workgroup per unit nothing else: fetched here and first used behind the rare
  // blocks, which lie out of the way, the cluster's arguments and those of the end were parked in
  // vector lanes (16 registers, and a second trip, with 128 channels, pages of 64 and an append).
  // 192 units of 4096 tokens with an append, 64 channels, pages of 32 15.0 -> 14.8 us, the INT8 cache
  // 16.2 -> 15.7.  Builds with clusters ask for all of it: clusters that take several units in turn, 128
  // units of four workgroups, are at 33.1 us so and 33.6 with the short list.
  if constexpr (kCluster && !kFirst) {
    asm volatile("" ::"s"(p.ctrl), "s"(p.page_min), "s"(p.page_max), "s"(p.topk_per_seq), "s"(p.k_new),
                 "s"(p.v_new), "s"(p.topk), "s"(p.units), "s"(p.g), "s"(p.xcds), "s"(p.div_hkv.d),
                 "s"(p.div_hkv.magic), "s"(p.div_g.d), "s"(p.div_g.magic), "s"(p.div_xcds.d),
                 "s"(p.div_xcds.magic), "s"(at.q), "s"(at.block_table), "s"(at.seq_lens), "s"(at.Hq),
                 "s"(at.Hkv), "s"(at.G), "s"(at.Pmax), "s"(at.lse), "s"(at.k_scale),
                 "s"(at.v_scale));
  } else if constexpr (!kFirst && !kInRegs) {
    asm volatile("" ::"s"(p.ctrl), "s"(p.page_min), "s"(p.page_max), "s"(p.topk_per_seq), "s"(p.topk),
                 "s"(p.div_hkv.d), "s"(p.div_hkv.magic), "s"(at.q), "s"(at.block_table), "s"(at.seq_lens),
                 "s"(at.Hq), "s"(at.Hkv), "s"(at.G), "s"(at.Pmax));
    if constexpr (kApp) asm volatile("" ::"s"(p.k_new), "s"(p.v_new));
  }
  const int G = kFirst ? f.G() : at.G, Pmax = kFirst ? f.Pmax() : at.Pmax;
  // which unit this workgroup works on, as which of how many members, and the size of a
  // member's chunk of the selected pages
  int epoch_raw, L_raw, K_raw;
  ClusterSlot where{(int)blockIdx.x, 0};
  if constexpr (kFirst) where = cluster_of(blockIdx.x, f);
  else if constexpr (kCluster) where = cluster_of(blockIdx.x, p.div_g, p.div_xcds, p.xcds > 1);
  int g = kCluster ? (kFirst ? f.g() : p.g) : 1, member = kCluster ? where.member : 0;
  int chunk = at.chunk;
  const int n_clusters = kCluster ? fast_div(gridDim.x, p.div_g) : (int)gridDim.x;
  // (a launch laid out by XCD is padded to whole rounds of the XCDs: clusters past
  // the last unit leave before any barrier, see below, and are not counted in)
  const bool padding = (kCluster || kDecide) && !kLoop && where.cluster >= (kFirst ? (int)f.units : p.units);
  const SelectLds sl = carve_select<NW>(smem, Pmax);
  const uint32_t sel_bytes = (uint32_t)select_lds_bytes(Pmax, NW), att_bytes = (uint32_t)(kParts<NW, kInt8> * G * (D + 2) * 4);
  const uint32_t q_off = sel_bytes > att_bytes ? sel_bytes : att_bytes;
  constexpr bool exchange = kCluster;
  unsigned char* q_stage = smem + q_off;
  int32_t* words = reinterpret_cast<int32_t*>(q_stage + ScoreLanes<D, kHalf, NW>::query_stage_bytes(G));
  int32_t* bt_lds = words + (kDecide ? kShareWords : 0);
  int32_t* my_sel = bt_lds + Pmax;  // [chunk]
  int u = padding ? 0 : where.cluster;
  int b = kFirst ? fast_div(u, FastDiv{1, f.magic_hkv}) : fast_div(u, p.div_hkv), h = u - b * at.Hkv;

  // The first loads of a unit (sequence length, K, query rows, block-table row,
  // first metadata tile) are sent out ahead of everything else: for the first
  // unit right here, before the set-up work that follows, for later units at the
  // end of the unit before.  What they fetch is only looked at inside the loop.
  // Which pages a member scores: the sequence's groups of PPW consecutive pages
  // (one wave-wide load each) are dealt out to the cluster's members in turn.
  // The selection bins the scores over a range it estimates from the member's
  // own share (see the exchange below), so that share has to be a fair sample
  // of the sequence; dealing out whole tiles of PPI pages reads 0.3 us faster on
  // the 16-sequence configuration, but where the scores vary smoothly along the
  // sequence the few pages that matter then lie in tiles most members never see.
  constexpr int kBtRegs = kRound == 1 ? 4 : 8;  // block-table entries per thread fetched through registers
  int bt_regs[kBtRegs];
  ScanRegs<D, kHalf, NW, kRound> scan;
  // Append mode: the new token's key / value rows of this unit, as the 16-byte
  // chunk (channels 8 * (lane % (D/8)) .. + 7) every lane needs for the box update
  // and the pool write (bf16 also for the INT8 cache, which quantises them).
  constexpr bool app = kApp;
  constexpr int LPR = ScoreLanes<D, kHalf>::LPR;
  uint4 kn16 = make_uint4(0, 0, 0, 0), vn16 = make_uint4(0, 0, 0, 0);
  bool leave = padding;
  if constexpr (kDecide) {
    const int lane = min(lane_id(), p.B - 1);
    epoch_raw = p.ctrl[kCtrlEpoch];
    const int L_lane = at.seq_lens[lane], K_lane = (p.topk_per_seq ? p.topk_per_seq : at.seq_lens)[lane];
    UnitShare share{b, h, member, g, chunk, u * at.n_split};
    if (uniform(by_shares<S, kApp, kCluster>(p, L_lane, p.topk_per_seq ? K_lane : p.topk, share))) {
      leave = share.g == 0;
      g = share.g;
      member = share.member;
      chunk = share.chunk;
      b = share.b;
      h = share.h;
      u = b * at.Hkv + h;
    }
    L_raw = __builtin_amdgcn_readlane(L_lane, b);
    K_raw = p.topk_per_seq ? __builtin_amdgcn_readlane(K_lane, b) : p.topk;
    // What only the end of the attention needs waits for it in LDS: in scalar registers it was
    // spilled in the ring of fragments (24 sequences x 8 KV heads of 8192 tokens: 50.6 -> 50.0 us).
    if (threadIdx.x == 0) {
      words[0] = g;
      words[1] = member;
      words[2] = share.part_row;
      *reinterpret_cast<int32_t**>(words + 4) = &p.ctrl[kCtrlDone + u];   // (no cluster: u < 256)
    }
  }
  auto issue_unit = [&](int uu) {
    if constexpr (!kDecide) {
      b = fast_div(uu, p.div_hkv);
      h = uu - b * at.Hkv;
      epoch_raw = p.ctrl[kCtrlEpoch];
      L_raw = at.seq_lens[b];
      K_raw = p.topk_per_seq ? p.topk_per_seq[b] : p.topk;
    }
    scan_issue_query(scan, at.q + ((size_t)b * at.Hq + (size_t)h * G) * D, G);
    if (app) {  // behind the query (needed first), ahead of the metadata (needed with it)
      const size_t row = ((size_t)b * at.Hkv + h) * D + (lane_id() % LPR) * 8;
      kn16 = *reinterpret_cast<const uint4*>(p.k_new + row);
      vn16 = *reinterpret_cast<const uint4*>(p.v_new + row);
    }
    const int32_t* bt_row = at.block_table + (size_t)b * Pmax;
#pragma unroll
    for (int k = 0; k < kBtRegs; ++k)   // no branch around the loads
      bt_regs[k] = bt_row[min((int)threadIdx.x + k * NT, Pmax - 1)];
    scan_issue_tile(scan, p.page_min + (size_t)uu * Pmax * D, p.page_max + (size_t)uu * Pmax * D,
                       Pmax, wave_id(), kCluster ? g : 1, kCluster ? member : 0);
  };
  if constexpr (kFirst || kInRegs) {
    // (the same loads; those whose addresses need the struct, or that the struct's would be waited
    // for with, come last, and with one round of scoring wait in registers until the scores are
    // worked out.  With several groups a wave the length and the epoch, which everything behind the
    // query's sums waits for, go out on leading arguments ahead of the metadata, through vector
    // addresses: scalar loads come back in any order, and with one of these under way the wait for the
    // struct would be one for it too)
    constexpr bool kWordsFirst = kRound > 1;
    const size_t new_chunk = (size_t)u * D + (lane_id() % LPR) * 8;
    scan_issue_query(scan, (kFirst ? f.q : at.q) + (size_t)u * G * D, G);
    if constexpr (kWordsFirst) {
      epoch_raw = f.ctrl()[kCtrlEpoch + vector_zero()];
      L_raw = f.seq_lens()[b + vector_zero()];
    } else if constexpr (app) {
      kn16 = *reinterpret_cast<const uint4*>(f.first + new_chunk);
      vn16 = *reinterpret_cast<const uint4*>(f.second + new_chunk);
    }
    scan_issue_tile(scan, (kFirst ? f.page_min : p.page_min) + (size_t)u * Pmax * D,
                    (kFirst ? f.page_max : p.page_max) + (size_t)u * Pmax * D, Pmax, wave_id(), kCluster ? g : 1,
                    kCluster ? member : 0);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (kWordsFirst) {
      // (three groups: what the rest is addressed with in one trip; see above.  With five the registers run
      // out: others were parked, and waited for, ahead of the first load)
      if constexpr (kRound < 5)
        asm volatile("" ::"s"(at.block_table), "s"(p.topk_per_seq), "s"(p.k_new), "s"(p.v_new), "s"(p.topk));
      if constexpr (app) {
        kn16 = *reinterpret_cast<const uint4*>(p.k_new + new_chunk);
        vn16 = *reinterpret_cast<const uint4*>(p.v_new + new_chunk);
      }
      K_raw = p.topk_per_seq ? p.topk_per_seq[b + vector_zero()] : p.topk;
    } else {
      epoch_raw = exchange ? p.ctrl[kCtrlEpoch] : 0;
      L_raw = at.seq_lens[b];
      K_raw = p.topk_per_seq ? p.topk_per_seq[b] : p.topk;
    }
    const int32_t* bt_row = at.block_table + (size_t)b * Pmax;
#pragma unroll
    for (int k = 0; k < kBtRegs; ++k)   // no branch around the loads
      bt_regs[k] = bt_row[min((int)threadIdx.x + k * NT, Pmax - 1)];
  } else {
    if (kLoop ? u < p.units : true) issue_unit(u);   // the host launches no idle cluster
  }
  // (The empty asm keeps the loads where they are: in front of anything that waits for one of
  // them, in the order of their use.  Left to the scheduler, the query's went out last and was waited
  // for with everything else.)
  if (!kLoop && (!kFirst || kRound == 3)) asm volatile("" : : "s"(q_off) : "memory");
  // (a padding workgroup leaves only here, behind the loads of unit 0, whose results it
  // drops: with an exit ahead of them the kernel's arguments would be fetched in two
  // dependent trips, the second one behind the test.  The expectation is for clusters that score in
  // one round or look at the lengths first, 12 x 8 units of 5600-8192 tokens with an append 26.0 -> 25.85 us:
  // in the other builds the compiler, with the exit out of the way, parks 2 to 10 scalar registers in
  // vector lanes ahead of the first load, none without it)
  if (kFirst || (kDecide && kCluster) ? TS_RARELY(leave) : leave) {
    // A workgroup too many counts itself in like the others, once all its waves have read the
    // lengths and the epoch: lengths advanced while it still looks at them could send it
    // another way.
    if (kDecide && (kCluster || kApp)) {
      asm volatile("" ::"v"(epoch_raw));
      __syncthreads();
      if (threadIdx.x == 0) (void)atomic_add_agent(&p.ctrl[kCtrlArrive], 1);
    }
    return;
  }
  TS_MARK(23);

  // Launch tag of the score exchange.  The epoch word is read by every wave of a
  // workgroup before the workgroup counts itself in; the launch's first workgroup advances it
  // for the next launch on its way out, once the count says that every workgroup
  // has read it.
  uint32_t tag = 0;
  bool counted = false;
  while (kLoop ? u < p.units : true) {
    TS_MARK(0);
    const int32_t* bt_row = at.block_table + (size_t)b * Pmax;
    uint64_t* srow = p.scores + (size_t)u * Pmax;
    float* srow_out = p.scores_out && (exchange || member == 0) ? p.scores_out + (size_t)u * Pmax : nullptr;

    // 1. score my share of the pages; the unit's block-table row is parked in LDS
    KeyLayout kl;
    int L_unit = 0, j_new = -1, slot_new = 0;  // length after the append; the new token's page / slot
    int pb_scan = 0;                         // the unit's page count, known once the scan runs
    int K_unit = 0;                          // the sequence's page budget (read with the length)
    uint32_t tmin = 0xffffffffu, tmax = 0u;  // this thread's share of the key range
    uint4 box_lo = make_uint4(0, 0, 0, 0), box_hi = make_uint4(0, 0, 0, 0);   // this lane's chunk of the
    bool has_box = false;                    // new token's box, if it has to write it back
    auto park_table = [&] {
#pragma unroll
      for (int k = 0; k < kBtRegs; ++k) {
        // (threads past the row's end write its last entry once more: a test would be a branch each)
        bt_lds[min((int)threadIdx.x + k * NT, Pmax - 1)] = bt_regs[k];
      }
      if (TS_RARELY(Pmax > kBtRegs * NT))
        for (int j = threadIdx.x + kBtRegs * NT; j < Pmax; j += NT) bt_lds[j] = bt_row[j];
    };
    scan_finish<D, !kLoop>(
        scan, p.page_min + (size_t)u * Pmax * D, p.page_max + (size_t)u * Pmax * D, G, Pmax,
        wave_id(), NW, q_stage,
        [&] {
          if (!kFirst) park_table();
          // (the empty asm pins the first use of the two values to this point:
          // using them earlier would put a memory round trip in front of the scan)
          if (!kFirst) asm volatile("" : "+v"(L_raw), "+v"(K_raw), "+v"(epoch_raw));
          // the tag is fixed by the first unit: the epoch word may already have
          // been advanced (by the launch's first workgroup, once it is through
          // with its own units) when a later unit's loads go out
          // (0 is never a tag: it marks words nobody has written since
          // ts_workspace_init, so the count skips it when it wraps)
          if (tag == 0u) tag = max((uint32_t)uniform(epoch_raw) + 1u, 1u);
          L_unit = uniform(L_raw);
          if (!kFirst) K_unit = uniform(K_raw);
          if (app && L_unit / S < Pmax) {  // a sequence with no room left is not extended
            j_new = L_unit / S;
            slot_new = L_unit % S;
            L_unit += 1;
          }
          pb_scan = uniform(min(pages_of(L_unit, S), Pmax));
          kl = KeyLayout::make<NW>(pb_scan);
          return pb_scan;
        },
        [&](uint4& mn, uint4& mx, int pg) {
          // the wave that scores the new token's page first widens (or opens)
          // its box in registers (the outer test is uniform over the wave: all the
          // others jump over the block instead of executing it with every lane masked
          // off).  It is written back with the token, below: the other members wait for this
          // wave's scores, which a store in front of them would hold up (16 units of 16
          // workgroups: 13.75 -> 14.1 us).
          if constexpr (kInt8) {
            // INT8 cache: the box takes the dequantised key rounded outwards; the
            // whole wave works out the row's scale (the LPR lanes of a row each
            // hold one chunk of it), the page's lanes do the rest
            if (kApp && TS_RARELY(__ballot(pg == j_new) != 0ull)) {
              float amax = chunk_amax_bf16(kn16);
#pragma unroll
              for (int m = 1; m < LPR; m <<= 1) amax = fmaxf(amax, shfl_xor_f(amax, m));
              if (pg == j_new) {
                uint4 lo, hi;
                i8_chunk_box(kn16, i8_row_scale(amax), lo, hi);
                mn = slot_new == 0 ? lo : widen_box<false>(mn, lo, true);
                mx = slot_new == 0 ? hi : widen_box<false>(mx, hi, false);
                box_lo = mn;
                box_hi = mx;
                has_box = true;
              }
            }
          } else if (kApp && TS_RARELY(__ballot(pg == j_new) != 0ull) && pg == j_new) {
            mn = slot_new == 0 ? kn16 : widen_box<kHalf>(mn, kn16, true);
            mx = slot_new == 0 ? kn16 : widen_box<kHalf>(mx, kn16, false);
            // (where every member scores the page, each widens it for itself and the first writes
            // it back; a member that reads the row behind that write widens it once more, to the
            // same box)
            if (exchange || member == 0) {
              box_lo = mn;
              box_hi = mx;
              has_box = true;
            }
          }
        },
        [&](int pg, float s) {
          if (exchange) store_agent_tagged(srow + pg, s, tag);
          if (pg < pb_scan) {   // (with an exchange: the range of my own share of the scores)
            const uint32_t k = score_key(s);
            if (!exchange) sl.keys[kl.at(pg)] = k;
            tmin = min(tmin, k);
            tmax = max(tmax, k);
          }
          if (TS_RARELY(srow_out != nullptr)) srow_out[pg] = s;
        },
        kCluster ? g : 1, kCluster ? member : 0, srow_out != nullptr,
        [&] {
          if constexpr (kFirst) {
            park_table();
            K_unit = uniform(K_raw);
          }
        },
        [&] {
          // Each wave has the epoch and the length by the barrier behind the query's sums: past it the
          // first thread may count the workgroup in.  (The builds that fetch the two words with scalar
          // loads wait for those at that barrier as it is.)
          if constexpr (kRound > 1) asm volatile("" : "+v"(L_raw), "+v"(epoch_raw));
        });
    TS_MARK_WAVE(32);
    const int L = uniform(L_unit);
    const int Pb = uniform(min(pages_of(L, S), Pmax));
    const int Kb = uniform(max(0, min(min(K_unit, Pb), at.Kmax)));

    // count this workgroup in (once): all its waves have read the epoch and, in append mode,
    // the sequence length, ahead of the barrier inside the scan.  The count's value is not asked
    // for: an atomic that returns one would hold this wave, and with it the barrier below, for a trip
    // to memory and back.
    if (exchange || app) {
      if (!counted && threadIdx.x == 0) (void)atomic_add_agent(&p.ctrl[kCtrlArrive], 1);
      counted = true;
    }

    // (the attention's query operand, out of the rows the scoring staged in LDS: fetched
    // here, where the waves are about to wait for the other members anyway)
    QOperand<D, kInt8> qop;
    qop.load(reinterpret_cast<const uint16_t*>(q_stage), G);   // the raw rows head the staging area
    // 2. exchange the scores inside the cluster
    TS_MARK(1);
    // The new token lands in its pool slot (one member's first lanes; the
    // block-table row is complete in LDS once the barrier above is passed).
    // Nothing in this launch reads it from there: the attention splices it in
    // from the caller's arrays.  It is done now rather than at the end (stores
    // issued last would hold up the completion of the kernel), by the first
    // lanes of the last wave (the first wave carries the workgroup's atomics).
    // All of it is written through (see store_through): what the pool and the boxes of a layer
    // receive in a step are parts of some 20 lines a unit (with 64 channels and pages of 16: 16 of the
    // value tile, whose D rows are S * 2 bytes each, one of the key tile, two boxes), whose
    // write-back otherwise starts when the kernel is done.
    auto store_new_token = [&] {
      const int t = (int)threadIdx.x - (NT - kWave);
      if (TS_RARELY(__ballot(has_box) != 0ull) && has_box) {
        const size_t row = ((size_t)u * Pmax + j_new) * D + (lane_id() % LPR) * 8;
        store_through16(const_cast<uint16_t*>(p.page_min) + row, box_lo);
        store_through16(const_cast<uint16_t*>(p.page_max) + row, box_hi);
      }
      if constexpr (kInt8) {
        if (TS_RARELY(j_new >= 0 && member == 0 && wave_id() == NW - 1)) {   // (uniform) the whole last wave
          float ka = chunk_amax_bf16(kn16), va = chunk_amax_bf16(vn16);
#pragma unroll
          for (int m = 1; m < LPR; m <<= 1) {
            ka = fmaxf(ka, shfl_xor_f(ka, m));
            va = fmaxf(va, shfl_xor_f(va, m));
          }
          const int phys = bt_lds[j_new];
          if (t < LPR && phys >= 0 && phys < at.n_phys) {
            const float ksc = i8_row_scale(ka), vsc = i8_row_scale(va);
            const size_t tile = ((size_t)phys * at.Hkv + h) * (size_t)at.tile_stride;
            uint8_t* k8 = reinterpret_cast<uint8_t*>(const_cast<uint16_t*>(at.k_pool));
            uint8_t* v8 = reinterpret_cast<uint8_t*>(const_cast<uint16_t*>(at.v_pool));
            store_through8(k8 + tile + (size_t)slot_new * D + t * 8, i8_chunk_codes(kn16, ksc));
            const uint2 vc = i8_chunk_codes(vn16, vsc);
#pragma unroll
            for (int i = 0; i < 8; ++i)
              store_through(&v8[tile + (size_t)(t * 8 + i) * S + slot_new],
                            (uint8_t)((i < 4 ? vc.x : vc.y) >> (8 * (i & 3))));
            if (t == 0) {
              const size_t so = ((size_t)phys * at.Hkv + h) * (size_t)S + slot_new;
              store_agent(const_cast<float*>(at.k_scale) + so, ksc);
              store_agent(const_cast<float*>(at.v_scale) + so, vsc);
            }
          }
        }
        return;
      }
      if (TS_RARELY(j_new >= 0 && member == 0 && wave_id() == NW - 1) && t < LPR) {
        const int phys = bt_lds[j_new];
        if (phys >= 0 && phys < at.n_phys) {
          const size_t tile = ((size_t)phys * at.Hkv + h) * (size_t)at.tile_stride;
          uint16_t* k_pool_w = const_cast<uint16_t*>(at.k_pool);
          uint16_t* v_pool_w = const_cast<uint16_t*>(at.v_pool);
          store_through16(k_pool_w + tile + (size_t)slot_new * D + t * 8, kn16);
          const uint32_t vw[4] = {vn16.x, vn16.y, vn16.z, vn16.w};
#pragma unroll
          for (int i = 0; i < 8; ++i)
            store_through(&v_pool_w[tile + (size_t)(t * 8 + i) * S + slot_new],
                          (uint16_t)(vw[i >> 1] >> (16 * (i & 1))));
        }
      }
    };

    const ForcedPages forced = ForcedPages::make(p.keep_first, p.keep_last, Pb);
    BinMap bins{0.f, 0.f};
    if (exchange) {
      // The selection's first stage (counting the pages into score bins) is done
      // here, key by key as the scores come in, instead of in a pass of its own
      // after them.  The bins need a score range before the first score of the
      // other members is looked at: the range of this workgroup's own share
      // (every g-th group of pages: a fair sample), widened; any monotone map
      // keeps the selection exact.  Each member bins in its own way and all
      // arrive at the same pages.
      select_begin<NW>(sl, tmin, tmax);
      __syncthreads();
      if (kApp) store_new_token();   // (the block-table row is complete behind this barrier)
      {
        uint32_t lo_key, hi_key;
        select_deposited_range<NW>(sl, lo_key, hi_key);
        bins = BinMap::widened(lo_key, hi_key);
      }
      // every thread polls its own entries of the row until all carry this
      // launch's tag (all loads of a round in flight together; bounded)
      bool expired = false;
      int spins = 0;
      auto poll = [&](auto np_tag) {
        constexpr int NP = decltype(np_tag)::value;
        for (int j0 = threadIdx.x; j0 < Pb; j0 += NT * NP) {
          uint64_t v[NP];
          for (;;) {
            bool all = true;
#pragma unroll
            for (int i = 0; i < NP; ++i) {
              v[i] = load_agent_u64(srow + min(j0 + i * NT, Pb - 1));  // no branch around the load
              all = all && (uint32_t)(v[i] >> 32) == tag;
            }
            if (all) break;
            if (++spins > p.spin_limit) { expired = true; break; }
            __builtin_amdgcn_s_sleep(1);
          }
#pragma unroll
          for (int i = 0; i < NP; ++i) {
            const int j = j0 + i * NT;
            if (j < Pb) {
              const bool always = j < forced.first || j >= forced.last_begin;
              const uint32_t k = always ? kForcedKey : score_key(__uint_as_float((uint32_t)v[i]));
              sl.keys[kl.at(j)] = k;
              atomicAdd(&sl.hist[bin_slot_index(bins.slot<true>(k))], 1u);
            }
          }
        }
      };
      const int per_thread = uniform((Pb + NT - 1) / NT);
      if (per_thread <= 1) poll(std::integral_constant<int, 1>{});
      else if (per_thread <= 2) poll(std::integral_constant<int, 2>{});
      else if (per_thread <= 4) poll(std::integral_constant<int, 4>{});
      else poll(std::integral_constant<int, 8>{});
      if (TS_RARELY(expired)) atomic_store_agent(&p.ctrl[kCtrlError], 1);
      TS_MARK(3);
      TS_MARK_WAVE(40);
    } else {
      select_begin<NW>(sl, tmin, tmax);
    }
    __syncthreads();
    TS_MARK(4);
    if (kApp && !exchange) store_new_token();

    // 3. select; keep my own chunk of the ascending list
    const int c0 = min(member * chunk, Kb), count = min(c0 + chunk, Kb) - c0;
    int32_t* sel_row = (p.sel_out && member == 0) ? p.sel_out + (size_t)u * at.Kmax : nullptr;
    if (TS_RARELY(sel_row != nullptr))
      for (int i = Kb + threadIdx.x; i < at.Kmax; i += NT) sel_row[i] = -1;
    if (TS_RARELY(p.sel_count && member == 0 && h == 0) && threadIdx.x == 0) p.sel_count[b] = Kb;
    auto keep_page = [&](int rank, int page) {
      if (rank >= c0 && rank < c0 + count) my_sel[rank - c0] = page;
      if (TS_RARELY(sel_row != nullptr)) sel_row[rank] = page;
    };
    if (exchange) select_topk_lds<NW, true>(sl, kl, Pb, Kb, forced, keep_page, bins);
    else select_topk_lds<NW, false>(sl, kl, Pb, Kb, forced, keep_page);
    __syncthreads();
    TS_MARK(5);
    // 4. attend my chunk (the wave-merge area reuses the select scratch)
    const size_t new_row = ((size_t)b * at.Hkv + h) * D;
    const NewToken nt{j_new, slot_new, app ? p.k_new + new_row : at.q, app ? p.v_new + new_row : at.q};
    // 5. (inside the same call) the cluster's partials are handed on as tagged
    // words; the cluster's last member (its chunk of the list is the one that
    // can be short) keeps its own in registers, polls for the others and writes
    // the output, or in large clusters every member its part of it (see attend_split).
    // Shares without an exchange wait for nothing at all: the member that finds itself the
    // last to have handed on its partial merges them.
    constexpr bool apart = kDecide && !kCluster;
    // Clusters that take several units in turn, INT8 cache, 128 channels: the expanded codes, the scales and what
    // the loop keeps for the next unit fill the registers, and the ring's rounds put 88 bytes a lane in
    // scratch memory (pages of 32 and 64).  128 units of four workgroups, pages of 16 43.8 -> 42.4 us, of 32
    // 54.5 -> 49.0, of 64 54.9 -> 48.5.  With smaller pages or 64 channels the rounds are the faster way
    // (pages of 8 57.0 against 57.7, 64 channels and pages of 16 31.6 against 33.2).
    constexpr bool plain = kLoop && kInt8 && D == 128 && S >= 16;
    constexpr int hand = !exchange ? kPlain : kDealt ? kTaggedDealt : kTagged;
    const bool merged = attend_split<NW, D, S, kApp, kInt8, kHalf, true, apart, plain, hand>(
        at, b, h,
        [&] {
          if constexpr (kDecide) {
            return SplitPlace{uniform(words[0]), uniform(words[1]), (size_t)uniform(words[2])};
          } else {
            return SplitPlace{at.n_split, member, (size_t)u * at.n_split};
          }
        },
        count, L, nt, [&](int i) { return my_sel[i]; }, [&](int j) { return bt_lds[j]; },
        reinterpret_cast<float*>(smem), tag, nullptr, p.spin_limit, &qop);
    if (apart && uniform(words[0]) > 1) {
      int* last = reinterpret_cast<int*>(smem);   // (free behind the barrier that ends the attention)
      stores_complete();
      __syncthreads();
      int32_t* done = *reinterpret_cast<int32_t**>(words + 4);
      if (threadIdx.x == 0) *last = atomic_add_agent(done, 1) == words[0] - 1;
      __syncthreads();
      if (uniform(*last)) {
        combine_splits<D, true>(at, b, h, (size_t)uniform(words[2]), uniform(words[0]), reinterpret_cast<float*>(smem) + 64);
        if (threadIdx.x == 0) atomic_store_agent(done, 0);
      }
    }
    TS_MARK(6);
    if (TS_RARELY(!merged)) atomic_store_agent(&p.ctrl[kCtrlError], 1);
    if (!kLoop) break;
    u += n_clusters;
    if (u >= p.units) break;
    issue_unit(u);
  }
  // The launch's first workgroup, at the end of its own work, closes the books: once
  // the count shows that every workgroup has read the epoch word and, with one unit per
  // workgroup, its sequence length (all of them did so microseconds ago), its first
  // wave re-arms the count, advances the epoch and (append mode) the lengths.
  // (No expectation in the builds of one workgroup per unit: out of the way, the block has registers
  // parked for it at the kernel's head.)
  const bool closes = blockIdx.x == 0 && wave_id() == 0;
  if ((exchange || app) && (kCluster ? TS_RARELY(closes) : closes)) {
    if (!wait_at_least(&p.ctrl[kCtrlArrive], p.n_arrive, p.spin_limit))
      atomic_store_agent(&p.ctrl[kCtrlError], 1);
    if (lane_id() == 0) {
      atomic_store_agent(&p.ctrl[kCtrlArrive], 0);
      if (exchange) atomic_store_agent(&p.ctrl[kCtrlEpoch], (int)tag);
    }
    if (app) {
      int32_t* seq_lens_w = const_cast<int32_t*>(at.seq_lens);
      for (int i = lane_id(); i < p.B; i += kWave) {
        const int len = seq_lens_w[i];
        if (len / S < Pmax) store_through(&seq_lens_w[i], len + 1);
      }
    }
  }
}

template <int D, int S, bool kLoop, bool kApp, bool kInt8, bool kHalf, bool kCluster>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void
query_aware_decode_kernel(FusedParams p) {
  decode_units<kWaves, D, S, kLoop, kApp, kInt8, kHalf, kCluster>(p);
}

// Clusters with one unit each, as in query_aware_decode_kernel's loop-free build, whose waves score
// their share of the pages in one round of at most R groups of 8 (64 channels) or 4 pages.  These
// launches are bound by the chain of their phases, and scoring is one of its links: 300
// instructions for the four groups of a tile and as many again for the next tile's loads, whose
// pages mostly do not exist.  R = 1 (8 waves, a group each): 4 units of 12 workgroups with 188
// pages 11.5 -> 10.3 us, 1 of 8 with 257 10.6 -> 9.8; R = 3: 128 of 2 with 257 16.8 -> 16.1, 4 of 32
// with 4098 17.9 -> 17.0; R = 5: 16 to 128 units of 513-4097 pages -0.1 us, without an append 18.5 -> 17.9;
// R = 9, 128 channels: 64 units of 1002 pages 27.5 -> 26.8, 32 of 1565 21.3 -> 20.5, the INT8 cache, 22 of 2910 28.0
// -> 25.9; 64 channels: 64 of 1565 21.3 -> 20.75, 128 of 1002 24.7 -> 24.4.
// The first loads' arguments come ahead of the others (FirstArgs).
template <int D, int S, bool kApp, bool kInt8, bool kHalf, int R>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void
one_round_decode_kernel(const uint16_t* q, const uint16_t* page_min, const uint16_t* page_max,
                        const uint16_t* first, const uint16_t* second, uint32_t shape, uint32_t units,
                        uint32_t magic_g, uint32_t magic_hkv, FusedParams p) {
  decode_units<kWaves, D, S, false, kApp, kInt8, kHalf, true, false, R, false, (R > 1)>(
      p, FirstArgs{q, page_min, page_max, first, second, shape, units, magic_g, magic_hkv});
}

// R = 1 for clusters of more than kMergedByOne.  The smaller ones, the shortest of all launches, do not carry the merge
// that is dealt out to the members: 16 layers in a graph, each 1 unit of eight members, 257 pages, 8.70 -> 8.64 us, 4 of
// eight, 188 pages 9.44 -> 9.34, the INT8 cache, 128 channels, 2 of six, 94 pages 12.63 -> 12.42; nine such shapes 0.3 % on
// average, from -0.5 to +1.6 % (where in memory the same instructions lie makes up to 3 % by itself).  With more
// groups a wave it is 0.4 % at the most, which no second build is for.
template <int D, int S, bool kApp, bool kInt8, bool kHalf>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void
one_group_dealt_decode_kernel(const uint16_t* q, const uint16_t* page_min, const uint16_t* page_max,
                              const uint16_t* first, const uint16_t* second, uint32_t shape, uint32_t units,
                              uint32_t magic_g, uint32_t magic_hkv, FusedParams p) {
  decode_units<kWaves, D, S, false, kApp, kInt8, kHalf, true, false, 1, false, true>(
      p, FirstArgs{q, page_min, page_max, first, second, shape, units, magic_g, magic_hkv});
}

// Up to 255 units of batches that may be ragged: see by_shares.  kCluster: the members of a
// cluster divide the scoring and wait for each other's scores and partials, by shares as with
// clusters of one size.  Batches that have one workgroup per unit otherwise (129 to 255 units) do
// not: their launches never waited, so that several streams could run them side by side, and
// must not start to.  Every member scores all pages, the pages kept are divided, and the last
// member to finish merges the partials.
template <int D, int S, bool kApp, bool kHalf, bool kCluster>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void
shares_decode_kernel(FusedParams p) {
  decode_units<kWaves, D, S, false, kApp, false, kHalf, kCluster, true>(p);
}

// Batches of more units than compute units whose units are not small: one workgroup of eight
// waves per unit, one resident per compute unit, the next one handed out by the hardware as
// one ends, so that the spread of sequence lengths does not decide the finish time and
// workgroups are in different phases at any time.  (Workgroups that stayed and took the
// units from a counter, the looping build, needed all unit-independent values of the body
// ahead of the loop and spilled with 128 channels and pages of 32 and 64: 80 layouts of
// 272-900 units 4 % slower on average and up to 20 %, the 64-sequence batch 890 against
// 880 us.)  Bound by HBM: 6.3 TB/s on the 64-sequence batch.
template <int D, int S, bool kInt8, bool kHalf>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void
many_units_decode_kernel(FusedParams p) {
  decode_units<kWaves, D, S, false, false, kInt8, kHalf, false>(p);
}

// One workgroup per unit: the struct with what the unit's first loads are addressed with taken from
// leading arguments, which are in registers when a wave starts (see FirstArgs).  The query and the
// first metadata tile go out on them alone, 25 instructions in, before anything of the struct or the
// lengths is asked for: with those fetches in front, scalar loads like the lengths', the first vector
// load stood behind a wait for them and 70 instructions.  512 units of 125 pages 14.2 -> 13.8 us, with 128
// channels 20.0 -> 19.6, 480 of 125 pages of 32 13.9 -> 13.6, 504 of 174 11.8 -> 11.8 (and 14.5, 20.3, 14.1
// and 12.2 with the struct alone).  Units that are not small do not feel it.
// shape: pages of a table row | G << 16.
__device__ __forceinline__ FusedParams with_args(FusedParams p, const uint16_t* q, const uint16_t* page_min,
                                                 const uint16_t* page_max, const int32_t* block_table,
                                                 const int32_t* seq_lens, const int32_t* topk_per_seq, uint32_t shape,
                                                 uint32_t magic_hkv) {
  p.at.q = q;
  p.page_min = page_min;
  p.page_max = page_max;
  p.at.block_table = block_table;
  p.at.seq_lens = seq_lens;
  p.topk_per_seq = topk_per_seq;
  p.at.Pmax = (int)(shape & 0xffffu);
  p.at.G = (int)(shape >> 16);
  p.div_hkv.magic = magic_hkv;
  return p;
}

// Batches of more units than compute units, as long as a unit is small (kSmallUnitBytes): one
// workgroup of four waves per unit, two of them resident per compute unit, handed out by the
// hardware.  Such a unit is bound by the chain of its phases, 10-13 us of which little is
// data: two half-size workgroups run two such chains side by side on a compute unit, where
// workgroups of eight waves run them one after the other.  Against the looping build that
// did so, 40 layouts of 264 to 1568 units: 1.0 to 2.4
// times faster, geometric mean 1.52 (504 units of 176 pages, 6 kept: 35.2 -> 15.7 us).
// An append runs as a kernel of its own in front: folding it in gained 3 % here and would
// make the first workgroup wait for ones not yet resident.
constexpr int kSmallWaves = 4;
template <int D, int S, bool kHalf>
__global__ __launch_bounds__(kSmallWaves * kWave) __attribute__((amdgpu_waves_per_eu(2, 2))) void
small_units_decode_kernel(const uint16_t* q, const uint16_t* page_min, const uint16_t* page_max,
                          const int32_t* block_table, const int32_t* seq_lens, const int32_t* topk_per_seq,
                          uint32_t shape, uint32_t magic_hkv, FusedParams p) {
  decode_units<kSmallWaves, D, S, false, false, false, kHalf, false, false, 0, true>(
      with_args(p, q, page_min, page_max, block_table, seq_lens, topk_per_seq, shape, magic_hkv));
}

// The same for the INT8 cache, whose list stays cut for eight waves: a wave takes two of its parts in turn.
template <int D, int S>
__global__ __launch_bounds__(kSmallWaves * kWave) __attribute__((amdgpu_waves_per_eu(2, 2))) void
small_units_i8_decode_kernel(const uint16_t* q, const uint16_t* page_min, const uint16_t* page_max,
                             const int32_t* block_table, const int32_t* seq_lens, const int32_t* topk_per_seq,
                             uint32_t shape, uint32_t magic_hkv, FusedParams p) {
  decode_units<kSmallWaves, D, S, false, false, true, false, false, false, 0, true>(
      with_args(p, q, page_min, page_max, block_table, seq_lens, topk_per_seq, shape, magic_hkv));
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
static int launch_status() { return hipGetLastError() == hipSuccess ? TS_OK : TS_ERR_LAUNCH; }

static int num_compute_units() {
  static int cus = 0;
  if (cus == 0) {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    cus = n;
  }
  return cus;
}

// XCDs (dies with an L2 of their own) the device deals workgroups out to: eight
// on the full part (32 compute units each), one in the single-die partition modes.
constexpr int kCusPerXcd = 32;
static int num_xcds() {
  const int cus = num_compute_units();
  return cus >= 2 * kCusPerXcd && cus % kCusPerXcd == 0 ? cus / kCusPerXcd : 1;
}

template <typename KernelT>
static int allow_lds(KernelT kernel, size_t bytes) {
  if (bytes <= 64 * 1024) return TS_OK;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                             hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)bytes) == hipSuccess
             ? TS_OK
             : TS_ERR_LAUNCH;
}

// Workgroups of `kernel`, of eight waves (only such workgroups ever wait for each other, and
// only of them anyone asks), that can be resident on the whole device at once.  The
// runtime's answer is remembered per (device, kernel, LDS size): the query costs more
// host time than the launch itself.
template <typename KernelT>
static int resident_capacity(KernelT kernel, size_t lds) {
  static std::mutex mu;
  static std::map<std::tuple<int, const void*, size_t>, int> known;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  const std::tuple<int, const void*, size_t> key(dev, reinterpret_cast<const void*>(kernel), lds);
  std::lock_guard<std::mutex> lock(mu);
  auto it = known.find(key);
  if (it != known.end()) return it->second;
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kThreads, lds) != hipSuccess)
    return 0;
  const int cap = per_cu * num_compute_units();
  if (cap > 0) known[key] = cap;
  return cap;
}

// CALL(DD, S) for the layout's page_size (check_layout has admitted it).
#define TS_DISPATCH_PAGE(DD, S, CALL) \
  switch (S) {                        \
    case 4: CALL(DD, 4); break;       \
    case 8: CALL(DD, 8); break;       \
    case 16: CALL(DD, 16); break;     \
    case 32: CALL(DD, 32); break;     \
    default: CALL(DD, 64); break;     \
  }

// The launches below: max_resident is the number of workgroups the launch may count on being
// resident together.  An append is folded into the launch where all units are worked on at
// once; otherwise it runs as a kernel of its own in front: those launches are bound by
// bandwidth or have the latency of one unit hidden behind others.

// One workgroup per unit (pl.g == 1); no workgroup waits for another unit's.
template <int D, int S, int kFmt>
static int launch_single(const ts_layout* layout, FusedParams& p, const Plan& pl, const void* k_new,
                         const void* v_new, int max_resident, void* stream) {
  constexpr bool kInt8 = kFmt == TS_KV_INT8, kHalf = kFmt == TS_KV_FP16;
  hipStream_t s = (hipStream_t)stream;
  auto one_kernel = query_aware_decode_kernel<D, S, false, false, kInt8, kHalf, false>;
  auto app_kernel = query_aware_decode_kernel<D, S, false, true, kInt8, kHalf, false>;
  auto many_kernel = many_units_decode_kernel<D, S, kInt8, kHalf>;
  const unsigned grid = (unsigned)pl.units;
  int st;
  p.xcds = 0;
  p.n_arrive = pl.units;
  if (!pl.small_units) {
    auto kernel = k_new ? app_kernel : one_kernel;
    if ((st = allow_lds(kernel, pl.lds_fused)) != TS_OK) return st;
    int cap = resident_capacity(kernel, pl.lds_fused);
    if (cap > max_resident) cap = max_resident;
    if (pl.units <= cap) {
      kernel<<<grid, kThreads, pl.lds_fused, s>>>(p);
      return TS_OK;
    }
  }
  if (k_new) {
    if ((st = ts_append_token_meta(layout, k_new, v_new, 1, stream)) != TS_OK) return st;
    p.k_new = p.v_new = nullptr;
  }
  if (pl.small_units) {
    auto small_kernel = [] {
      if constexpr (kInt8) return small_units_i8_decode_kernel<D, S>;
      else return small_units_decode_kernel<D, S, kHalf>;
    }();
    if ((st = allow_lds(small_kernel, pl.lds_fused)) != TS_OK) return st;
    small_kernel<<<grid, kSmallWaves * kWave, pl.lds_fused, s>>>(
        p.at.q, p.page_min, p.page_max, p.at.block_table, p.at.seq_lens, p.topk_per_seq,
        (uint32_t)p.at.Pmax | (uint32_t)p.at.G << 16, p.div_hkv.magic, p);
    return TS_OK;
  }
  if ((st = allow_lds(many_kernel, pl.lds_fused)) != TS_OK) return st;
  many_kernel<<<grid, kThreads, pl.lds_fused, s>>>(p);
  return TS_OK;
}

// A grid whose clusters of pl.g workgroups lie one per XCD is padded to whole rounds of the XCDs,
// where that many can be resident at once: the number of workgroups, p.xcds and p.div_xcds.
static unsigned cluster_grid(FusedParams& p, const Plan& pl, int cap) {
  const int xcds = num_xcds();
  const unsigned padded = (unsigned)((pl.units + xcds - 1) / xcds * xcds * pl.g);
  p.xcds = 0;
  if (xcds <= 1 || (int)padded > cap) return (unsigned)(pl.units * pl.g);
  p.xcds = xcds;
  p.div_xcds = make_fast_div(xcds);
  return padded;
}

// Up to 255 units of a batch that may be ragged (pl.shares): clusters of one size or in
// proportion to the work, as the lengths have it.  False: not all workgroups fit the
// device at once (a part of one).
template <int D, int S, int kFmt, bool kCluster>
static bool launch_shares(const ts_layout* layout, FusedParams& p, const Plan& pl, const void* k_new,
                          int max_resident, void* stream, int& st) {
  constexpr bool kHalf = kFmt == TS_KV_FP16;
  auto kernel = k_new ? shares_decode_kernel<D, S, true, kHalf, kCluster>
                      : shares_decode_kernel<D, S, false, kHalf, kCluster>;
  if ((st = allow_lds(kernel, pl.lds_fused)) != TS_OK) return true;
  int cap = resident_capacity(kernel, pl.lds_fused);
  if (cap > max_resident) cap = max_resident;
  unsigned grid = kCluster ? cluster_grid(p, pl, cap) : (unsigned)pl.units;
  if (!kCluster) p.xcds = 0;
  if (grid < (unsigned)(pl.per_head * layout->num_kv_heads)) grid = (unsigned)(pl.per_head * layout->num_kv_heads);
  if ((int)grid > cap) return false;
  p.n_arrive = (int)grid;
  p.per_head = pl.per_head;
  p.inv_g = 1.f / (float)pl.g;
  p.min_rows = pl.min_rows;
  kernel<<<grid, kThreads, pl.lds_fused, (hipStream_t)stream>>>(p);
  return true;
}

// The build for clusters whose waves score their pages in one round, nullptr where that takes more
// than nine groups each: a tile of eight and one more group are the longest that is built.
using OneRound = void (*)(const uint16_t*, const uint16_t*, const uint16_t*, const uint16_t*, const uint16_t*,
                          uint32_t, uint32_t, uint32_t, uint32_t, FusedParams);
static int round_groups(int D, int Pmax, int g) {   // groups of pages a wave has at the most
  const int group = kWave / (D / 8), groups = (Pmax + group - 1) / group;
  return ((groups + g - 1) / g + kWaves - 1) / kWaves;
}
template <int D, int S, bool kApp, int kFmt>
static OneRound one_round_kernel(int rows, int g) {
  constexpr bool kInt8 = kFmt == TS_KV_INT8, kHalf = kFmt == TS_KV_FP16;
  if (rows <= 1 && g > kMergedByOne) return one_group_dealt_decode_kernel<D, S, kApp, kInt8, kHalf>;
  if (rows <= 1) return one_round_decode_kernel<D, S, kApp, kInt8, kHalf, 1>;
  if (rows <= 3) return one_round_decode_kernel<D, S, kApp, kInt8, kHalf, 3>;
  if (rows <= 5) return one_round_decode_kernel<D, S, kApp, kInt8, kHalf, 5>;
  if (rows <= 9) return one_round_decode_kernel<D, S, kApp, kInt8, kHalf, 9>;
  return nullptr;
}

// A cluster of pl.g > 1 workgroups per unit: the loop-free builds where all clusters are
// resident at once, otherwise (a forced cluster size) the looping one, each cluster taking
// several units in turn.
template <int D, int S, int kFmt>
static int launch_clusters(const ts_layout* layout, FusedParams& p, const Plan& pl,
                           const void* k_new, const void* v_new, int max_resident, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  constexpr bool kInt8 = kFmt == TS_KV_INT8, kHalf = kFmt == TS_KV_FP16;
  auto loop_kernel = query_aware_decode_kernel<D, S, true, false, kInt8, kHalf, true>;
  auto one_kernel = query_aware_decode_kernel<D, S, false, false, kInt8, kHalf, true>;
  auto app_kernel = query_aware_decode_kernel<D, S, false, true, kInt8, kHalf, true>;
  int st;
  const int rows = round_groups(D, p.at.Pmax, p.g);
  const OneRound round_kernel = k_new ? one_round_kernel<D, S, true, kFmt>(rows, p.g)
                                      : one_round_kernel<D, S, false, kFmt>(rows, p.g);
  if (round_kernel) {
    if ((st = allow_lds(round_kernel, pl.lds_fused)) != TS_OK) return st;
    int cap = resident_capacity(round_kernel, pl.lds_fused);
    if (cap > max_resident) cap = max_resident;
    const unsigned grid = cluster_grid(p, pl, cap);
    int xcd_bits = 0;
    while (p.xcds > 1 << xcd_bits) ++xcd_bits;
    if (pl.units * pl.g <= cap && (p.xcds == 0 || p.xcds == 1 << xcd_bits)) {
      p.n_arrive = pl.units * pl.g;
      const uint32_t shape = (uint32_t)p.at.Pmax | (uint32_t)p.g << 16 | (uint32_t)(p.at.G - 1) << 24 |
                             (uint32_t)xcd_bits << 28;
      const uint16_t *words = reinterpret_cast<const uint16_t*>(p.ctrl),
                     *lens = reinterpret_cast<const uint16_t*>(p.at.seq_lens);   // (see FirstArgs)
      round_kernel<<<grid, kThreads, pl.lds_fused, s>>>(p.at.q, p.page_min, p.page_max, rows <= 1 ? p.k_new : words,
                                                        rows <= 1 ? p.v_new : lens, shape, (uint32_t)pl.units,
                                                        p.div_g.magic, p.div_hkv.magic, p);
      return TS_OK;
    }
  }
  if ((st = allow_lds(loop_kernel, pl.lds_fused)) != TS_OK ||
      (st = allow_lds(one_kernel, pl.lds_fused)) != TS_OK ||
      (st = allow_lds(app_kernel, pl.lds_fused)) != TS_OK)
    return st;
  int cap1 = resident_capacity(k_new ? app_kernel : one_kernel, pl.lds_fused);
  if (cap1 > max_resident) cap1 = max_resident;
  const bool one_unit_each = pl.units * pl.g <= cap1;
  if (k_new && !one_unit_each) {
    if ((st = ts_append_token_meta(layout, k_new, v_new, 1, stream)) != TS_OK) return st;
    p.k_new = p.v_new = nullptr;
  }
  const int xcds = num_xcds();
  p.xcds = 0;
  if (one_unit_each) {
    const unsigned grid = cluster_grid(p, pl, cap1);
    p.n_arrive = pl.units * pl.g;
    if (p.k_new)
      app_kernel<<<grid, kThreads, pl.lds_fused, s>>>(p);
    else
      one_kernel<<<grid, kThreads, pl.lds_fused, s>>>(p);
    return TS_OK;
  }
  int cap = resident_capacity(loop_kernel, pl.lds_fused);
  if (cap > max_resident) cap = max_resident;
  int clusters = cap / pl.g;
  if (clusters < 1) return TS_ERR_DEVICE;   // a cluster must be co-resident
  if (clusters > pl.units) clusters = pl.units;
  if (xcds > 1 && clusters >= xcds) {
    clusters = clusters / xcds * xcds;
    p.xcds = xcds;
    p.div_xcds = make_fast_div(xcds);
  }
  p.n_arrive = clusters * pl.g;
  loop_kernel<<<(unsigned)(clusters * pl.g), kThreads, pl.lds_fused, s>>>(p);
  return TS_OK;
}

// The fused launch for the layout's page_size in one cache format and head_dim.
template <int kFmt, int kD>
int launch_fused_format(const ts_layout* layout, FusedParams& p, const Plan& pl, const void* k_new,
                        const void* v_new, int max_resident, void* stream) {
  int st = TS_ERR_UNSUPPORTED;
#define TS_LAUNCH_FUSED(DD, SS)                                                                     \
  if constexpr (kFmt != TS_KV_INT8) {                                                              \
    if (pl.shares &&                                                                               \
        (pl.g > 1 ? launch_shares<DD, SS, kFmt, true>(layout, p, pl, k_new, max_resident, stream, st)  \
                  : launch_shares<DD, SS, kFmt, false>(layout, p, pl, k_new, max_resident, stream, st))) \
      return st;                                                                                   \
  }                                                                                                \
  st = pl.g > 1                                                                                    \
           ? launch_clusters<DD, SS, kFmt>(layout, p, pl, k_new, v_new, max_resident, stream)       \
           : launch_single<DD, SS, kFmt>(layout, p, pl, k_new, v_new, max_resident, stream)
  TS_DISPATCH_PAGE(kD, layout->page_size, TS_LAUNCH_FUSED)
#undef TS_LAUNCH_FUSED
  return st;
}

// The staged attention kernel (grid (g, units)); sel == nullptr: every page.
template <int kFmt, int kD>
int launch_attention_format(const ts_layout* layout, const AttendParams& a, const Plan& pl,
                            const int32_t* sel, const int32_t* sel_count, int32_t* unit_done,
                            void* stream) {
  constexpr bool kInt8 = kFmt == TS_KV_INT8, kHalf = kFmt == TS_KV_FP16;
  const size_t lds = (size_t)kWaves * a.G * (layout->head_dim + 2) * 4;
  dim3 grid(pl.g, pl.units);
  hipStream_t s = (hipStream_t)stream;
  if constexpr (!kInt8) {
    if (!sel && pl.shares) {
      const FastDiv div_hkv = make_fast_div(a.Hkv);
#define TS_LAUNCH_DENSE(DD, SS)                                                  \
  dense_shares_kernel<DD, SS, kHalf><<<pl.per_head * a.Hkv, kThreads, lds, s>>>( \
      a, unit_done, pl.cstride, layout->num_seqs, pl.per_head, div_hkv)
      TS_DISPATCH_PAGE(kD, layout->page_size, TS_LAUNCH_DENSE)
#undef TS_LAUNCH_DENSE
      return launch_status();
    }
  }
  if constexpr (!kInt8) {
    if (!sel && pl.rounds) {
      const FastDiv div_hkv = make_fast_div(a.Hkv);
#define TS_LAUNCH_ROUNDS(DD, SS)                                          \
  dense_rounds_kernel<DD, SS, kHalf><<<2 * pl.units, kThreads, lds, s>>>( \
      a, unit_done, pl.cstride, layout->num_seqs, pl.units, div_hkv)
      TS_DISPATCH_PAGE(kD, layout->page_size, TS_LAUNCH_ROUNDS)
#undef TS_LAUNCH_ROUNDS
      return launch_status();
    }
  }
#define TS_LAUNCH_ATTENTION(DD, SS)                                                                     \
  sparse_attention_kernel<DD, SS, kInt8, kHalf><<<grid, kThreads, lds, s>>>(                            \
      a.q, sel, sel_count, a.seq_lens, a.block_table, make_fast_div(a.Hkv).magic, a.chunk, a.Kmax,     \
      a.Pmax | a.G << 16, a, unit_done, pl.cstride)
  TS_DISPATCH_PAGE(kD, layout->page_size, TS_LAUNCH_ATTENTION)
#undef TS_LAUNCH_ATTENTION
  return launch_status();
}

// Workgroups of the loop-free build with the append folded in that can be
// resident at once.
template <int kFmt, int kD>
int append_capacity_format(const ts_layout* layout, const Plan& pl) {
  constexpr bool kInt8 = kFmt == TS_KV_INT8, kHalf = kFmt == TS_KV_FP16;
  int cap = 0;
#define TS_CAPACITY(DD, SS)                                                                        \
  cap = pl.g > 1 ? resident_capacity(query_aware_decode_kernel<DD, SS, false, true, kInt8, kHalf, true>, \
                                     pl.lds_fused)                                                 \
                 : resident_capacity(query_aware_decode_kernel<DD, SS, false, true, kInt8, kHalf, false>, \
                                     pl.lds_fused)
  TS_DISPATCH_PAGE(kD, layout->page_size, TS_CAPACITY)
#undef TS_CAPACITY
  return cap;
}

#ifdef TS_PROFILE
// The timestamp buffer of the translation unit that holds this format's kernels.
template <int kFmt, int kD>
int set_profile_buffer_format(void* buf) {
  return hipMemcpyToSymbol(HIP_SYMBOL(g_profile_buf), &buf, sizeof(buf)) == hipSuccess ? TS_OK
                                                                                        : TS_ERR_LAUNCH;
}
#define TS_FORMAT_PROFILE(LINKAGE, FMT, DD) LINKAGE template int set_profile_buffer_format<FMT, DD>(void*);
#else
#define TS_FORMAT_PROFILE(LINKAGE, FMT, DD)
#endif

// Instantiated once per format and head_dim, each in its own file.
#define TS_FORMAT_FUNCTIONS(LINKAGE, FMT, DD)                                                      \
  TS_FORMAT_PROFILE(LINKAGE, FMT, DD)                                                              \
  LINKAGE template int launch_fused_format<FMT, DD>(const ts_layout*, FusedParams&, const Plan&,   \
                                                    const void*, const void*, int, void*);         \
  LINKAGE template int launch_attention_format<FMT, DD>(const ts_layout*, const AttendParams&,     \
                                                        const Plan&, const int32_t*,               \
                                                        const int32_t*, int32_t*, void*);          \
  LINKAGE template int append_capacity_format<FMT, DD>(const ts_layout*, const Plan&);

// CALL(FMT, DD) for the layout's cache format and head_dim (check_layout has admitted them).
#define TS_DISPATCH_FORMAT(layout, CALL)                            \
  do {                                                              \
    const bool d64 = (layout)->head_dim == 64;                      \
    switch ((layout)->kv_format) {                                  \
      case TS_KV_INT8:                                              \
        if (d64) { CALL(TS_KV_INT8, 64); } else { CALL(TS_KV_INT8, 128); } \
        break;                                                      \
      case TS_KV_FP16:                                              \
        if (d64) { CALL(TS_KV_FP16, 64); } else { CALL(TS_KV_FP16, 128); } \
        break;                                                      \
      default:                                                      \
        if (d64) { CALL(TS_KV_BF16, 64); } else { CALL(TS_KV_BF16, 128); } \
    }                                                               \
  } while (0)

}  // namespace ts
