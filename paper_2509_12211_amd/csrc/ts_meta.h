// Page metadata kernels: bulk rebuild (Eq. 1) and per-token incremental update.
#pragma once
#include "ts_device.h"

namespace ts {

struct MetaParams {
  const uint16_t* k_pool;
  uint16_t* k_pool_w;
  uint16_t* v_pool_w;
  const int32_t* block_table;
  int32_t* seq_lens;
  uint16_t* page_min;
  uint16_t* page_max;
  int B, Hkv, S, Pmax, n_phys, tile_stride;
  float* k_scale;   // INT8 cache only: fp32 [n_phys][Hkv][S]
  float* v_scale;
};

// Bytes of boxes from which on a bulk rebuild writes them through (pages of up to 16 tokens).
constexpr size_t kBoxesThrough = 18 << 20;

// One lane's 16 bytes of a unit's boxes (`bytes` of them at base), written through.
__device__ __forceinline__ void store_row_through(uint16_t* base, int bytes, int at, const uint4& v) {
  constexpr int kRawBuffer = 0x00020000, kSc1 = 16;   // third word of a raw descriptor; cache policy: agent scope
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(base, (short)0, bytes, kRawBuffer);
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(stream_u4, v), r, at, 0, kSc1);
}

// A wavefront summarises kWave / (D/8) logical pages of one (sequence, KV head) at
// a time: a page's D/8 consecutive lanes each own eight channels (one 16-byte
// chunk of a token row) and walk down the page's tokens, so a lane takes the
// channel-wise min / max over the tokens in its own registers and nothing is
// folded across lanes.  A wave-wide load reads one token row of every page of
// the group (128 or 256 contiguous bytes each); up to NT = 16 of them are in
// flight per wave before the first is used (16 KiB), behind ONE dependent
// look-up of the sequence length and the block-table entries, so the kernel
// streams the pool at memory speed instead of paying that chain per page.
// NT: token rows fetched together, min(page_size, 16); longer pages take several
// rounds.  Slots past the sequence's last token are read (they lie inside the
// page's tile) and ignored.  The rows are fetched with streaming loads (each
// instruction takes whole lines that nobody reads again): -9 % on the 128 MiB pool.
// The boxes of pages of up to 16 tokens (11 to 33 % of what the kernel moves) are written through,
// whole lines at a time, where there are many: they fill the 32 MiB of the L2 caches with lines that
// the kernel's end writes back.  64 channels, pages of 16, 66 MB of boxes 128.3 -> 118.1 us, 33 MB 70.2 ->
// 67.1, 25 MB 54.6 -> 53.9; 128 channels, 33 MB 58.6 -> 57.3, 25 MB 44.0 -> 43.3; pages of 8, 33 MB 33.2 ->
// 32.2, 25 MB 25.3 -> 25.0.  At 19 MB the two are equal.  Fewer would lose: 18 MB 1 % (128 channels 33.0 -> 33.5), 16
// MB 1 to 2 %, 6 to 8 MB 6 % (15.7 -> 16.7, pages of 8 10.8 -> 11.5).  With pages of 32 it costs 0.5 %.
// (A build of its own: a test at the stores cost the others 1 %, 8 units of 1327 pages 11.54 -> 11.70 us.)
template <int D, bool kHalf, int NT, bool kThrough>
__global__ __launch_bounds__(kThreads) void build_page_meta_kernel(MetaParams p) {
  constexpr int LPR = D / 8;        // lanes per page (one per 16-byte chunk of a token row)
  constexpr int PPW = kWave / LPR;  // pages per wave
  const int lane = lane_id(), cg = lane % LPR;
  const int j = (blockIdx.y * kWaves + wave_id()) * PPW + lane / LPR;
  const int h = blockIdx.x, b = blockIdx.z;
  const int L = p.seq_lens[b];
  const int Pb = min((L + p.S - 1) / p.S, p.Pmax);
  if (uniform((blockIdx.y * kWaves + wave_id()) * PPW) >= Pb) return;   // the whole group is past the end
  const bool page_on = j < Pb;
  const int phys = p.block_table[(size_t)b * p.Pmax + min(j, Pb - 1)];
  const bool on = page_on && phys >= 0 && phys < p.n_phys;
  const int valid = min(p.S, L - j * p.S);   // tokens the page holds (only looked at when `on`)
  const uint16_t* tile =
      p.k_pool + ((size_t)(on ? phys : 0) * p.Hkv + h) * (size_t)p.tile_stride + cg * 8;
  float lo[8], hi[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) { lo[i] = INFINITY; hi[i] = -INFINITY; }
  for (int t0 = 0; t0 < p.S; t0 += NT) {
    uint4 w[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) w[t] = load_stream16(tile + (size_t)(t0 + t) * D);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      float f[8];
      unpack8e<kHalf>(w[t], f);
      const bool tok = t0 + t < valid;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        lo[i] = fminf(lo[i], tok ? f[i] : INFINITY);
        hi[i] = fmaxf(hi[i], tok ? f[i] : -INFINITY);
      }
    }
  }
  if (on) {
    const size_t row = (((size_t)b * p.Hkv + h) * p.Pmax + j) * D + cg * 8;
    // back to 16-bit elements: the values are elements of the cache, so this is exact
    // (bf16: the upper half of the fp32 pattern)
    auto pack = [](float x, float y) -> uint32_t {
      if (kHalf) return (uint32_t)f32_to_half(x) | ((uint32_t)f32_to_half(y) << 16);
      return (__float_as_uint(x) >> 16) | (__float_as_uint(y) & 0xffff0000u);
    };
    const uint4 a = make_uint4(pack(lo[0], lo[1]), pack(lo[2], lo[3]), pack(lo[4], lo[5]),
                               pack(lo[6], lo[7]));
    const uint4 c = make_uint4(pack(hi[0], hi[1]), pack(hi[2], hi[3]), pack(hi[4], hi[5]),
                               pack(hi[6], hi[7]));
    if constexpr (kThrough) {
      const size_t unit = ((size_t)b * p.Hkv + h) * p.Pmax * D;
      const int bytes = p.Pmax * D * 2, at = (j * D + cg * 8) * 2;
      store_row_through(p.page_min + unit, bytes, at, a);
      store_row_through(p.page_max + unit, bytes, at, c);
    } else {
      *reinterpret_cast<uint4*>(p.page_min + row) = a;
      *reinterpret_cast<uint4*>(p.page_max + row) = c;
    }
  }
}

// Element-wise box update of eight packed bf16: lo = k where k < lo, hi = k
// where k > hi (strict, as the stand-alone append kernel does it).
template <bool kHalf = false>
__device__ __forceinline__ uint32_t widen_pair(uint32_t box, uint32_t k, bool is_min) {
  const float bl = elem_lo<kHalf>(box), bh = elem_hi<kHalf>(box), kl = elem_lo<kHalf>(k),
              kh = elem_hi<kHalf>(k);
  const bool tl = is_min ? kl < bl : kl > bl, th = is_min ? kh < bh : kh > bh;
  return ((tl ? k : box) & 0x0000ffffu) | ((th ? k : box) & 0xffff0000u);
}
template <bool kHalf = false>
__device__ __forceinline__ uint4 widen_box(const uint4& box, const uint4& k, bool is_min) {
  return make_uint4(widen_pair<kHalf>(box.x, k.x, is_min), widen_pair<kHalf>(box.y, k.y, is_min),
                    widen_pair<kHalf>(box.z, k.z, is_min), widen_pair<kHalf>(box.w, k.w, is_min));
}

// One workgroup per sequence.  A thread takes eight channels of one KV head at a
// time: it widens (or opens) the 16-byte chunk of the box of page seq_len / S
// and, when v_new is given, puts the token into its pool slot (one 16-byte store
// for the key; the value tile is channel-major, so eight 2-byte stores).  The
// kernel is a chain of dependent memory round trips, arranged to need only two:
// the token's values (which do not depend on the length) go out together with
// the length, then the block-table entry and the old box together.  All threads
// read seq_lens[b] before the barrier; thread 0 advances it after.
// kHalf: the cache holds IEEE half (the comparison is the only thing that differs).
template <bool kHalf>
__global__ __launch_bounds__(kThreads) void append_token_meta_kernel(MetaParams p, int D,
                                                                      const uint16_t* k_new,
                                                                      const uint16_t* v_new,
                                                                      int advance) {
  const int b = blockIdx.x, n8 = p.Hkv * D / 8, cpr = D / 8;   // chunks, chunks per head row
  const uint4* k_src = reinterpret_cast<const uint4*>(k_new + (size_t)b * p.Hkv * D);
  const uint4* v_src = reinterpret_cast<const uint4*>((v_new ? v_new : k_new) + (size_t)b * p.Hkv * D);
  const int first = min((int)threadIdx.x, n8 - 1);
  const uint4 k0 = k_src[first], v0 = v_src[first];   // fetched ahead of the length
  const int L = p.seq_lens[b];
  const int sh = __builtin_ctz(p.S);  // page sizes are powers of two
  const int j = L >> sh, slot = L & (p.S - 1);
  const bool fits = j < p.Pmax;
  const int jc = fits ? j : 0;
  const int phys = p.block_table[(size_t)b * p.Pmax + jc];
  for (int i0 = threadIdx.x; i0 < n8; i0 += kThreads) {
    const int h = i0 / cpr, c8 = (i0 % cpr) * 8;
    const size_t m = (((size_t)b * p.Hkv + h) * p.Pmax + jc) * D + c8;
    const uint4 lo = *reinterpret_cast<const uint4*>(p.page_min + m);   // before phys is looked at
    const uint4 hi = *reinterpret_cast<const uint4*>(p.page_max + m);
    const uint4 kn = i0 == (int)threadIdx.x ? k0 : k_src[i0];
    const uint4 vn = i0 == (int)threadIdx.x ? v0 : v_src[i0];
    const bool ok = fits && (v_new == nullptr || (phys >= 0 && phys < p.n_phys));
    if (ok) {
      *reinterpret_cast<uint4*>(p.page_min + m) = slot == 0 ? kn : widen_box<kHalf>(lo, kn, true);
      *reinterpret_cast<uint4*>(p.page_max + m) = slot == 0 ? kn : widen_box<kHalf>(hi, kn, false);
      if (v_new != nullptr) {
        const size_t tile = ((size_t)phys * p.Hkv + h) * (size_t)p.tile_stride;
        *reinterpret_cast<uint4*>(p.k_pool_w + tile + (size_t)slot * D + c8) = kn;
        const uint32_t vw[4] = {vn.x, vn.y, vn.z, vn.w};
#pragma unroll
        for (int i = 0; i < 8; ++i)
          p.v_pool_w[tile + (size_t)(c8 + i) * p.S + slot] = (uint16_t)(vw[i >> 1] >> (16 * (i & 1)));
      }
    }
  }
  const bool ok = fits && (v_new == nullptr || (phys >= 0 && phys < p.n_phys));
  __syncthreads();
  if (ok && advance && threadIdx.x == 0) p.seq_lens[b] = L + 1;
}

// ---------------------------------------------------------------------------
// INT8 cache.  The key of a token is code * scale (one fp32 scale per token and
// KV head) as a real number; a page's box has to contain those numbers for
// Eq. 2 to remain an upper bound, so the minimum is rounded DOWN to bf16 and
// the maximum UP.  int8 x fp32 is exact in fp64.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint16_t bf16_directed(double x, bool up) {
  float f = static_cast<float>(x);   // nearest; then moved to the right side of x
  uint32_t b = __float_as_uint(f);
  if (up ? static_cast<double>(f) < x : static_cast<double>(f) > x) {
    const bool away = up ? !(b >> 31) : (b >> 31) != 0;   // a step away from zero
    if ((b & 0x7fffffffu) == 0u) b = up ? 0x00000001u : 0x80000001u;
    else b = away ? b + 1u : b - 1u;
  }
  uint16_t hi = static_cast<uint16_t>(b >> 16);
  if ((b & 0xffffu) != 0u) {
    // dropping the low bits moves towards zero: down for positive values, up for negative
    const bool negative = (b >> 31) != 0;
    if (negative ? !up : up) hi = static_cast<uint16_t>(hi + 1);
  }
  return hi;
}

// The dequantised values of a chunk rounded outwards to bf16: lo <= code * scale <= hi.
__device__ __forceinline__ void i8_chunk_box(const uint4& c, float scale, uint4& lo, uint4& hi) {
  const uint32_t w[4] = {c.x, c.y, c.z, c.w};
  uint32_t l[4], h[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const double a = static_cast<double>(i8_code(bf16_lo(w[i]), scale)) * static_cast<double>(scale);
    const double b = static_cast<double>(i8_code(bf16_hi(w[i]), scale)) * static_cast<double>(scale);
    l[i] = bf16_directed(a, false) | (static_cast<uint32_t>(bf16_directed(b, false)) << 16);
    h[i] = bf16_directed(a, true) | (static_cast<uint32_t>(bf16_directed(b, true)) << 16);
  }
  lo = make_uint4(l[0], l[1], l[2], l[3]);
  hi = make_uint4(h[0], h[1], h[2], h[3]);
}

// The same for a value known as its nearest fp32 f, where f is no bf16 number (its lower
// half is not zero): the exact value then lies between the same two bf16 numbers as f.
__device__ __forceinline__ uint32_t bf16_directed_off_grid(float f, bool up) {
  const uint32_t b = __float_as_uint(f);
  return (b >> 16) + (((b >> 31) != 0u) != up ? 1u : 0u);
}

// Bulk rebuild for the INT8 cache, laid out like build_page_meta_kernel: the eight
// consecutive lanes of a page each own sixteen channels and walk down the page's tokens, a
// wave-wide load takes 128 contiguous bytes of each of eight pages (one token row with
// D = 128, two with D = 64), NI of them in flight, and the tokens' scales come in fours.
// Bound by memory, as long as the arithmetic stays in fp32: code * scale is one fused
// multiply-add with ONE rounding (u * s - 128 * s for the biased code u), rounding keeps the
// order, and so the smallest rounded product is the rounded smallest product.  From that
// the bf16 below it follows without the exact value, unless the rounded one is itself a bf16
// number (about one in 65536, or scales with few bits); those channels are worked out
// again in fp64.  (One thread per channel with a byte load and three fp64 operations per
// token, each page waiting for its own look-ups, ran at 0.9 TB/s.)
// Slots past the sequence's last token repeat that token.
template <int D, int NI>
__global__ __launch_bounds__(kThreads) void build_page_meta_i8_kernel(MetaParams p) {
  constexpr int R = 128 / D;     // token rows per load
  constexpr int NS = NI * R;     // tokens per round
  static_assert(NS % 4 == 0, "scales are fetched in fours");
  const int lane = lane_id(), li = lane & 7;
  // (with two rows the second row's chunks run backwards, so that the lane with the same
  // channels is the mirror image within the eight)
  const int r = R == 2 ? li >> 2 : 0, cg = r ? 7 - li : li;
  const int first = (blockIdx.y * kWaves + wave_id()) * 8, j = first + lane / 8;
  const int h = blockIdx.x, b = blockIdx.z;
  const int L = p.seq_lens[b];
  const int Pb = min((L + p.S - 1) / p.S, p.Pmax);
  if (uniform(first) >= Pb) return;   // the whole group is past the end
  const int phys = p.block_table[(size_t)b * p.Pmax + min(j, Pb - 1)];
  const bool on = j < Pb && phys >= 0 && phys < p.n_phys;
  const int last = on ? min(p.S, L - j * p.S) - 1 : 0;   // the page's last token
  const size_t tile_id = (size_t)(on ? phys : 0) * p.Hkv + h;
  const uint8_t* tile = reinterpret_cast<const uint8_t*>(p.k_pool) + tile_id * (size_t)p.tile_stride + cg * 16;
  const float* sc = p.k_scale + tile_id * (size_t)p.S;
  const float s_last = sc[last];
  float lo[16], hi[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) { lo[i] = INFINITY; hi[i] = -INFINITY; }
  for (int t0 = 0; t0 < p.S; t0 += NS) {
    uint4 w[NI];
    float4 s4[NS / 4];
#pragma unroll
    for (int i = 0; i < NI; ++i) w[i] = load_stream16(tile + (size_t)min(t0 + i * R + r, last) * D);
#pragma unroll
    for (int q = 0; q < NS / 4; ++q) s4[q] = *reinterpret_cast<const float4*>(sc + t0 + 4 * q);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const float4 q = s4[i * R / 4];
      const int e = i * R % 4;
      float s = e == 0 ? q.x : e == 1 ? q.y : e == 2 ? q.z : q.w;
      if (R == 2) s = r ? (e == 0 ? q.y : q.w) : s;
      s = t0 + i * R + r <= last ? s : s_last;
      const float bias = -128.0f * s;
      const uint32_t x[4] = {w[i].x ^ 0x80808080u, w[i].y ^ 0x80808080u, w[i].z ^ 0x80808080u,
                             w[i].w ^ 0x80808080u};
#pragma unroll
      for (int c = 0; c < 16; ++c) {
        const float v = fmaf(static_cast<float>((x[c >> 2] >> (8 * (c & 3))) & 0xffu), s, bias);
        lo[c] = fminf(lo[c], v);
        hi[c] = fmaxf(hi[c], v);
      }
    }
  }
  // the lane's channels: all sixteen, or with two rows the half that it takes over from (and
  // the other half that it leaves to) the lane of the other row
  constexpr int NC = 16 / R;
  const int c0 = cg * 16 + r * 8;
  float klo[NC], khi[NC];
  if constexpr (R == 2) {
    auto mirror = [](float v) {
      return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), kDppHalfMirror, 0xf, 0xf, true));
    };
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      klo[c] = fminf(r ? lo[8 + c] : lo[c], mirror(r ? lo[c] : lo[8 + c]));
      khi[c] = fmaxf(r ? hi[8 + c] : hi[c], mirror(r ? hi[c] : hi[8 + c]));
    }
  } else {
#pragma unroll
    for (int c = 0; c < NC; ++c) { klo[c] = lo[c]; khi[c] = hi[c]; }
  }
  uint32_t mn[NC], mx[NC];
  uint32_t redo = 0;   // channels with an extreme that is a bf16 number (zeros of either sign too)
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    mn[c] = bf16_directed_off_grid(klo[c], false);
    mx[c] = bf16_directed_off_grid(khi[c], true);
    if ((__float_as_uint(klo[c]) & 0xffffu) == 0u || (__float_as_uint(khi[c]) & 0xffffu) == 0u) redo |= 1u << c;
  }
  if (!on) return;
  if (redo != 0u) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      if ((redo >> c) & 1u) {
        double dlo = INFINITY, dhi = -INFINITY;
        for (int t = 0; t <= last; ++t) {
          const int8_t code = static_cast<int8_t>(tile[(size_t)t * D + r * 8 + c]);
          const double k = static_cast<double>(code) * static_cast<double>(sc[t]);
          dlo = fmin(dlo, k);
          dhi = fmax(dhi, k);
        }
        mn[c] = bf16_directed(dlo, false);
        mx[c] = bf16_directed(dhi, true);
      }
    }
  }
  const size_t row = (((size_t)b * p.Hkv + h) * p.Pmax + j) * D + c0;
#pragma unroll
  for (int q = 0; q < NC / 8; ++q) {
    auto pack = [&](const uint32_t (&m)[NC]) {
      return make_uint4(m[8 * q] | (m[8 * q + 1] << 16), m[8 * q + 2] | (m[8 * q + 3] << 16),
                        m[8 * q + 4] | (m[8 * q + 5] << 16), m[8 * q + 6] | (m[8 * q + 7] << 16));
    };
    *reinterpret_cast<uint4*>(p.page_min + row + 8 * q) = pack(mn);
    *reinterpret_cast<uint4*>(p.page_max + row + 8 * q) = pack(mx);
  }
}

// Append to the INT8 cache: one workgroup per sequence, a wave per KV head at a
// time.  The bf16 key and value are quantised (scale = max |x| / 127, 1 for a
// zero vector; code = x / scale rounded half to even, in fp32 with correctly
// rounded division), stored with their scales when v_new is given, and the
// page's box is opened / widened with the dequantised key rounded outwards.  As above two round trips
// for the first head of a wave: the token's rows go out with the length, the old box with the block-table entry.
static __global__ __launch_bounds__(kThreads) void append_token_i8_kernel(MetaParams p, int D,
                                                                   const uint16_t* k_new,
                                                                   const uint16_t* v_new,
                                                                   int advance) {
  const int b = blockIdx.x, lane = lane_id();
  const int mine = wave_id(), c1 = D > kWave ? lane + kWave : lane;   // channels lane, c1
  auto fetch = [&](const uint16_t* rows, int h, float (&x)[2]) {
    const uint16_t* row = rows + ((size_t)b * p.Hkv + h) * D;
    x[0] = bf16_to_f32(row[lane]);
    x[1] = bf16_to_f32(row[c1]);   // (64 channels: the first again, not used)
  };
  float k0[2], v0[2];
  fetch(k_new, min(mine, p.Hkv - 1), k0);
  fetch(v_new ? v_new : k_new, min(mine, p.Hkv - 1), v0);
  const int L = p.seq_lens[b];
  const int sh = __builtin_ctz(p.S);
  const int j = L >> sh, slot = L & (p.S - 1);
  const bool fits = j < p.Pmax;
  const int jc = fits ? j : 0;
  const int phys = p.block_table[(size_t)b * p.Pmax + jc];
  const bool ok = fits && (v_new == nullptr || (phys >= 0 && phys < p.n_phys));
  for (int h = mine; h < p.Hkv; h += kWaves) {
    const size_t row = (((size_t)b * p.Hkv + h) * p.Pmax + jc) * D;
    float kv[2] = {k0[0], k0[1]}, vv[2] = {v0[0], v0[1]};
    const uint16_t lo_was[2] = {p.page_min[row + lane], p.page_min[row + c1]};
    const uint16_t hi_was[2] = {p.page_max[row + lane], p.page_max[row + c1]};
    if (h != mine) {
      fetch(k_new, h, kv);
      fetch(v_new ? v_new : k_new, h, vv);
    }
    const float ksc = i8_row_scale(wave_max_f32(fmaxf(fabsf(kv[0]), fabsf(kv[1]))));
    const float vsc = i8_row_scale(wave_max_f32(fmaxf(fabsf(vv[0]), fabsf(vv[1]))));
    if (!ok) continue;
    const size_t tile = ((size_t)phys * p.Hkv + h) * (size_t)p.tile_stride;
    int8_t* k8 = reinterpret_cast<int8_t*>(p.k_pool_w);
    int8_t* v8 = reinterpret_cast<int8_t*>(p.v_pool_w);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int c = lane + 64 * i;
      if (c < D) {
        const int kq = i8_code(kv[i], ksc), vq = i8_code(vv[i], vsc);
        if (v_new != nullptr) {
          k8[tile + (size_t)slot * D + c] = static_cast<int8_t>(kq);
          v8[tile + (size_t)c * p.S + slot] = static_cast<int8_t>(vq);
        }
        const double kd = static_cast<double>(kq) * static_cast<double>(ksc);
        const uint16_t lo = bf16_directed(kd, false), hi = bf16_directed(kd, true);
        if (slot == 0 || bf16_to_f32(lo) < bf16_to_f32(lo_was[i])) p.page_min[row + c] = lo;
        if (slot == 0 || bf16_to_f32(hi) > bf16_to_f32(hi_was[i])) p.page_max[row + c] = hi;
      }
    }
    if (v_new != nullptr && lane == 0) {
      const size_t so = ((size_t)phys * p.Hkv + h) * (size_t)p.S + slot;
      p.k_scale[so] = ksc;
      p.v_scale[so] = vsc;
    }
  }
  __syncthreads();   // every thread has read seq_lens[b]
  if (ok && advance && threadIdx.x == 0) p.seq_lens[b] = L + 1;
}

}  // namespace ts
