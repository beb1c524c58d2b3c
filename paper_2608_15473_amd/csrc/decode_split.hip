// Split-KV decode sweep over a paged grouped-query KV cache (gfx950).
//
// Computes, for every (request b, shard s, query head h), the pair (O, ln Z) of the shard's cached
// positions (Q-First, arXiv:2608.15473, §5: Z = sum exp(s_i), O = sum exp(s_i) v_i / Z, scores
// s_i = scale * q . k_i as in §2).  The kernel is bound by HBM bandwidth: every cached byte of K
// and V is read exactly once, and the G query heads that share a KV head are all served from that
// one read.
//
// Work decomposition.  One workgroup = one unit (b, s, c, g): KV head g of chunk c of shard s of
// request b (chunks > 1 only when a shape has too few units to fill the GPU).  Its W wavefronts
// take the unit's pages round-robin.  Inside a wavefront the 64 lanes form 4 rows of 16; a page
// (16 positions x 128 dims of bf16 = 4 KB per tensor) is read with 4 fully coalesced 16-byte
// loads per lane, load j covering positions 4j..4j+3, so lane (row r, column c) holds dims
// 8c..8c+7 of position 4j + r.  Each row is an independent online-softmax sweeper over the
// positions r, r+4, r+8, r+12 of every page; rows and wavefronts merge once, at the end.
//
// Per page and lane, scores: at G = 4 or 8 query heads per KV head, on the matrix cores (the K
// tile passes through LDS into the operand layout of four v_mfma_f32_16x16x32_bf16, which leave
// each lane the scores of exactly the positions whose V it holds, for one head; the other heads'
// come from neighbouring lanes by DPP); otherwise with v_dot2c_f32_bf16 on the packed bf16 pairs and a 16-lane
// DPP all-reduce per score.  Both take exact bf16 products and fp32 sums.  Then exp2 in the log2
// domain and fp32 FMAs for PV with the bf16 values unpacked by shift/mask.  The running max is
// raised lazily (only when a score exceeds it by more than kLazy), so the O rescale is rare after
// a shard's first pages.
#include <math.h>

#include <atomic>

#include "linear_mfma.h"
#include "merge_body.h"
#include "qf_internal.h"

namespace qf {
namespace {

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

constexpr int D = kHeadDim;
constexpr int P = kPage;
constexpr float kLn2 = 0.6931471805599453f;
constexpr int kNonTemporal = 2;  // buffer-load cache-policy bit "nt" on gfx950
constexpr float kLazy = 8.0f;  // log2 units: p = exp2(s - m) stays <= 256 between rescales

__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a),
                                         __builtin_bit_cast(bf16x2_t, b), c, false);
}

using mrg::row_sum16;  // sum over the 16 lanes of a DPP row, the same bits on each

// Lane 4*(c/4) + h's value in every lane c of its quad (DPP quad_perm [h,h,h,h]).
__device__ __forceinline__ float quad_bcast(float x, int h) {
  const int v = __float_as_int(x);
  switch (h) {
    case 0: return __int_as_float(__builtin_amdgcn_mov_dpp(v, 0x00, 0xF, 0xF, true));
    case 1: return __int_as_float(__builtin_amdgcn_mov_dpp(v, 0x55, 0xF, 0xF, true));
    case 2: return __int_as_float(__builtin_amdgcn_mov_dpp(v, 0xAA, 0xF, 0xF, true));
    default: return __int_as_float(__builtin_amdgcn_mov_dpp(v, 0xFF, 0xF, 0xF, true));
  }
}

// Lane 8*(c/8) + h's value in every lane c of its 8-lane group (G = 8), or the quad's (G <= 4),
// for the matrix path, where lane c holds the values of head c % G.  For G = 8 the quad broadcast
// gives one half of each 8-lane group the right head, and a 4-lane row shift written only into
// the other half's DPP banks (quads) completes it.
template <int G>
__device__ __forceinline__ float group_bcast(float x, int h) {
  if constexpr (G == 1) {
    return x;
  } else if constexpr (G <= 4) {
    return quad_bcast(x, h);
  } else {
    const float t = quad_bcast(x, h & 3);
    return h < 4 ? __builtin_amdgcn_update_dpp(t, t, 0x114, 0xF, 0xA, false)   // row_shr:4 -> quads 1, 3
                 : __builtin_amdgcn_update_dpp(t, t, 0x104, 0xF, 0x5, false);  // row_shl:4 -> quads 0, 2
  }
}

// Rows (16 lanes) or halves (32 lanes) of two registers exchanged: x = (a's even, b's even),
// y = (a's odd, b's odd), in lane order.
__device__ __forceinline__ void swap_rows(float a, float b, float& x, float& y) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  x = __uint_as_float(r[0]);
  y = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap_halves(float a, float b, float& x, float& y) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  x = __uint_as_float(r[0]);
  y = __uint_as_float(r[1]);
}

// 16-byte slot of chunk `ch` (dims 8ch..8ch+7) of position `pos` in a wavefront's 4 KB K tile in
// LDS.  The XOR swizzle makes both the row-wise writes and the column-wise operand reads free of
// bank conflicts: a position's 16 chunks stay in its 256 bytes, and the 16 positions read together
// for one chunk land in 16 different slots of their rows.
__device__ __forceinline__ int kslot(int pos, int ch) {
  return pos * 16 + (ch ^ (4 * (pos & 3) + (pos >> 2)));
}

// Block-table entries are wave-uniform: read them through the constant address space so they
// become scalar loads (own counter), never vector loads that would join the page loads' vmcnt.
typedef const __attribute__((address_space(4))) int32_t* const_i32_ptr;

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

__device__ __forceinline__ void unpack8(const uint4& w, float* f) {
  f[0] = bf16_lo(w.x); f[1] = bf16_hi(w.x);
  f[2] = bf16_lo(w.y); f[3] = bf16_hi(w.y);
  f[4] = bf16_lo(w.z); f[5] = bf16_hi(w.z);
  f[6] = bf16_lo(w.w); f[7] = bf16_hi(w.w);
}

// Sweep and merge in one launch: every unit of a (request, KV head) counts itself in once its
// partial states are stored; the unit that completes the count merges the group's G query heads
// over all max_shards x chunks slots with the merge kernels' own code (merge_body.h).  The XCDs'
// L2 caches are not coherent with each other, and a device-scope fence would write back and
// invalidate a whole L2 per workgroup, so no fence is used: the partial states are written and
// read with device-scope accesses (which go through to the coherent level), every wavefront waits
// until its own stores have completed before the workgroup barrier, and the count is a
// device-scope atomic.  The last unit then sets the counter back to 0 for the next call.
// Nothing ever waits for another workgroup.
// The G query heads of one (request, KV head) merged over their `entries` slots by the last unit
// of the group.  When one 16-slot group per wavefront covers the slots with W / G wavefronts per
// head (or W / 2, ...), heads are merged side by side by teams of wavefronts, and every wavefront
// loads its log-partitions and O rows at once (one memory round trip; the O rows of empty slots
// are read and discarded); each team sums exactly what merge_row's wavefronts sum, with the same
// code (mrg::WaveMerge), so the bits are merge_row's.  Otherwise head by head with merge_row.  The partial states
// were written by other workgroups of this launch: read with device-scope loads.
template <int G, int W>
__device__ __forceinline__ void merge_group(const float* __restrict__ part_o,
                                            const float* __restrict__ part_lse,
                                            uint16_t* __restrict__ merged_o,
                                            float* __restrict__ merged_lse, int b, int g, int hq,
                                            int entries) {
  constexpr int K = mrg::K;
  const int groups = (entries + K - 1) / K;
  const int hpw = min(G, W / max(groups, 1));   // heads merged side by side
  if (hpw < 2) {
#pragma unroll 1
    for (int h = 0; h < G; ++h)
      mrg::merge_row<true, false, W, true>(part_o, part_lse, merged_o, merged_lse, entries, hq, b,
                                           g * G + h, nullptr, nullptr, nullptr, 1, 0.0f);
    return;
  }
  const int wph = W / hpw;                       // wavefronts per head, >= groups
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int sub = wave / wph, wl = wave % wph;
  const bool in_team = sub < hpw;
  const int i0 = K * wl;
  __shared__ mrg::WaveMergeLds<W> lds;
#pragma unroll 1
  for (int h0 = 0; h0 < G; h0 += hpw) {
    const int h = g * G + h0 + min(sub, hpw - 1);
    const float* lse = part_lse + (size_t)b * entries * hq + h;
    const float* o = part_o + ((size_t)b * entries * hq + h) * mrg::D + 2 * lane;
    const int32_t o_step = hq * mrg::D;
    const float* o_i0 = o + (size_t)i0 * o_step;
    float x = -INFINITY;
    if (in_team && lane < K && i0 + lane < entries)
      x = __hip_atomic_load(&lse[(size_t)(i0 + lane) * hq], __ATOMIC_RELAXED,
                            __HIP_MEMORY_SCOPE_AGENT);
    float2 v[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const bool in = in_team && i0 + k < entries;
      v[k] = __builtin_bit_cast(
          float2, in ? __hip_atomic_load(reinterpret_cast<const uint64_t*>(o_i0 + k * o_step),
                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                     : 0ull);
    }
    // This wavefront's group, as one round of merge_row's loop.
    mrg::WaveMerge st;
    st.add(x, v);
    lds.put(wave, lane, st);
    __syncthreads();
    if (in_team && wl == 0) {   // the team's first wavefront: merge_row's final merge
      float lse_out;
      const float2 a = lds.finish(sub * wph, wph, lane, lse_out);
      const size_t out_idx = ((size_t)b * hq + h) * mrg::D / 2 + lane;
      reinterpret_cast<uint32_t*>(merged_o)[out_idx] = mrg::bf16_rne(a.x) | (mrg::bf16_rne(a.y) << 16);
      if (merged_lse && lane == 0) merged_lse[(size_t)b * hq + h] = lse_out;
    }
    __syncthreads();
  }
}

template <int G, int W>
__device__ __forceinline__ void merge_if_last(const float* __restrict__ part_o,
                                              const float* __restrict__ part_lse,
                                              int32_t* __restrict__ counters,
                                              uint16_t* __restrict__ merged_o,
                                              float* __restrict__ merged_lse, int b, int g,
                                              int hq, int hkv, int entries, int counter_step) {
  __shared__ int s_last;
  int32_t* const counter = &counters[((size_t)b * hkv + g) * counter_step];
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wavefront's partial stores are complete
  __syncthreads();
  if (threadIdx.x == 0) {
    const int prev = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_last = (prev == entries - 1);
  }
  __syncthreads();
  if (!s_last) return;
  merge_group<G, W>(part_o, part_lse, merged_o, merged_lse, b, g, hq, entries);
  if (threadIdx.x == 0)
    __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Pages [p0, p1) of shard s of request b (the split rule of the interface: K = ceil(pages / S_b)
// whole pages per shard, the last ones shorter or empty), with the request's shape checked: an out-of-range
// context length or shard count is clamped (so nothing is read out of bounds) and reported in
// `poison`.  n is the clamped context length.
struct ShardRange {
  int n, p0, p1;
  bool poison;
};
__device__ __forceinline__ ShardRange shard_range(const int32_t* __restrict__ ctx_lens,
                                                 const int32_t* __restrict__ n_shards, int b,
                                                 int s, int32_t max_pages, int32_t max_shards) {
  ShardRange r;
  int n = ctx_lens[b];
  int S = n_shards[b];
  r.poison = false;
  const int cap = max_pages * P;
  if (n < 0 || n > cap) { r.poison = true; n = n < 0 ? 0 : cap; }
  if (S < 1 || S > max_shards) { r.poison = true; S = S < 1 ? 1 : max_shards; }
  const int pages = (n + P - 1) / P;
  const int per = (pages + S - 1) / S;
  r.n = n;
  r.p0 = r.p1 = 0;
  if (s < S) {
    r.p0 = (int)min((int64_t)s * per, (int64_t)pages);
    r.p1 = (int)min((int64_t)(s + 1) * per, (int64_t)pages);
  }
  return r;
}

// The sweep of one unit by one workgroup; `bid` plays the role of the workgroup index (it is the
// index itself in decode_split_kernel, the sweep's share of the indices in a shared launch).
// With MERGE, the unit also takes part in the fused merge (merge_if_last).
template <int G, int W, int NBUF, bool MERGE = false>
__device__ __forceinline__ void sweep_unit(
    const uint16_t* __restrict__ qp, const uint16_t* __restrict__ kp,
    const uint16_t* __restrict__ vp, const int32_t* __restrict__ block_table,
    const int32_t* __restrict__ ctx_lens, const int32_t* __restrict__ n_shards,
    float* __restrict__ out_o, float* __restrict__ out_lse, int32_t hq, int32_t hkv,
    int32_t max_pages, int32_t num_pages, int32_t max_shards, int32_t chunks, int32_t n_units,
    int32_t batch, int32_t run, UnitDivisors by, float scale_log2, const unsigned bid,
    int32_t* __restrict__ counters = nullptr, uint16_t* __restrict__ merged_o = nullptr,
    float* __restrict__ merged_lse = nullptr, const int32_t* __restrict__ unit_order = nullptr,
    int32_t counter_step = 1) {
  // Which unit this workgroup sweeps.  Workgroups are dispatched in index order, round-robin over
  // the 8 XCDs.
  //  * Short shards (run > 0): items of `run` units (the KV heads of some consecutive (shard, chunk)
  //    slots of a request, in (request, shard, chunk, KV head) order) are dealt to the XCDs in rows
  //    of 8 consecutive items, each row rotated against the one before, so that the slots of one
  //    request, and the first slots of all requests, spread over every XCD whatever the shard
  //    counts: in a ragged batch a few long requests hold most of the pages, and with each XCD
  //    taking a contiguous range of units those requests' sweeps ran on one or two XCDs.  Measured:
  //    12 requests of 27 to 7,003 positions at 16 shards, sweep + fold 37 -> 28 us a layer; 14 of up to
  //    25,056 at 35 shards 109 -> 65 us; uniform batches +-0.5%.
  //  * Long shards (run == 0): units in (shard descending, request, KV head) order,
  //    round-robin over the XCDs, so the largest shards (high indices exist only in long requests)
  //    start first and every XCD gets an even share; the small shards fill the tail.  With
  //    sub-shard chunks the chunk index runs fastest, so the chunks of a shard alternate between
  //    even- and odd-numbered XCDs (the unit index modulo 8 is the XCD), and their sizes are
  //    weighted by that parity (kXcdWeightEven / kXcdWeightOdd): measured on MI355X, odd-numbered
  //    XCDs stream 8-17% slower than even ones under the long-shard sweep, whatever KV head they
  //    read, so equal chunks leave the even XCDs idle while the odd ones finish.
  //    Without chunks (and with at most kRankMaxPairs (request, shard) pairs), a unit order
  //    written by rank_units_kernel replaces both: each workgroup index names its unit, longest
  //    shard first, and the odd XCDs get fewer of the long units.
  int g, c, s, b;
  int pair = 0;  // long shards with chunks: index of the (request, shard, KV head) in unit order
  if (run > 0) {
    const unsigned j = bid / 8u;
    const unsigned r = by.run.of(j);
    const unsigned i = (bid - (r + (r >> 1) + (r >> 2) + (r >> 3))) & 7u;   // XCD bid % 8, rotated
    const unsigned item_unit = (8u * r + i - r) * (unsigned)run + j;        // item * run + j % run
    if (item_unit >= (unsigned)n_units) return;
    unsigned rest = by.hkv.of(item_unit);
    g = (int)(item_unit - rest * (unsigned)hkv);
    unsigned q = by.chunks.of(rest);
    c = (int)(rest - q * (unsigned)chunks);
    rest = q;
    q = by.shards.of(rest);
    s = (int)(rest - q * (unsigned)max_shards);
    b = (int)q;
  } else {
    const int unit = unit_order != nullptr ? unit_order[bid] : (int)bid;
    if (unit < 0 || unit >= n_units) return;
    int rest;
    if (chunks > 1) {
      c = unit % chunks;
      pair = unit / chunks;
      g = pair % hkv;
      rest = pair / hkv;
    } else {
      c = 0;
      g = unit % hkv;
      rest = unit / hkv;
    }
    b = rest % batch;
    s = max_shards - 1 - rest / batch;
  }

  // The request's shape, checked: an out-of-range value poisons this unit's log-sum-exp with NaN.
  const ShardRange range = shard_range(ctx_lens, n_shards, b, s, max_pages, max_shards);
  const int n = range.n;
  bool poison = range.poison;
  const int p0 = range.p0;
  const int len = range.p1 - p0;
  int c0, c1;
  if (run == 0 && chunks > 1) {
    // Chunk j of this shard runs on an XCD of parity (pair * chunks + j) % 2; the pages before
    // chunk c weigh kXcdWeightEven per even-XCD chunk and kXcdWeightOdd per odd one.
    const int first_odd = (int)(((int64_t)pair * chunks) & 1);
    auto weight_before = [&](int cc) -> int64_t {
      const int64_t even = first_odd ? cc / 2 : (cc + 1) / 2;
      return even * kXcdWeightEven + (cc - even) * kXcdWeightOdd;
    };
    const int64_t total = weight_before(chunks);
    c0 = p0 + (int)((int64_t)len * weight_before(c) / total);
    c1 = p0 + (int)((int64_t)len * weight_before(c + 1) / total);
  } else {
    const int cper = (len + chunks - 1) / chunks;
    c0 = p0 + (int)min((int64_t)c * cper, (int64_t)len);
    c1 = p0 + (int)min((int64_t)(c + 1) * cper, (int64_t)len);
  }

  // An empty unit (a slot past the request's shards, or an empty shard or chunk) reads nothing:
  // its ln Z is -inf (NaN if the request's shape was out of range), its O is never read, so it
  // stops here, before the query loads and the merge.  (Ragged batches are mostly such units.)
  if (c0 >= c1) {
    if (threadIdx.x < G) {
      const size_t slot = (((size_t)b * max_shards + s) * chunks + c) * hq + (size_t)g * G;
      if constexpr (MERGE)
        __hip_atomic_store(&out_lse[slot + threadIdx.x], poison ? NAN : -INFINITY,
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      else
        __builtin_nontemporal_store(poison ? NAN : -INFINITY, &out_lse[slot + threadIdx.x]);
    }
    if constexpr (MERGE)
      merge_if_last<G, W>(out_o, out_lse, counters, merged_o, merged_lse, b, g, hq, hkv,
                          max_shards * chunks, counter_step);
    return;
  }

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row = lane >> 4;
  const int col = lane & 15;

  // With 4 or 8 heads per KV head the scores come from the matrix cores (process_mf below);
  // otherwise the VALU computes them (process_valu).  Measured: the matrix path is 1-5% faster at
  // G = 4 and 27-32% faster at G = 8, where the VALU path spends most of its issue slots on the
  // dot products and reductions, and 1-2.5% slower at G = 2, where the VALU has slack and the LDS
  // round trip only adds latency.
  constexpr bool MF = G >= 4;

  // Queries of the group (not requested before the shape is known: 82% of a ragged batch's units are empty,
  // and their queries cost it 0.5%).  VALU path: dims 8col..8col+7 of every head as packed bf16 pairs.
  // Matrix path: the queries are the 16 columns of the B operand of S^T = K Q^T (column c holds
  // head c % G), split over the dims in 4 steps of 32: lane (row, col) holds dims
  // 32kk + 8row .. 32kk + 8row + 7 of head col % G for step kk.
  uint32_t qv[G][4];
  bf16x8_t qb[4];
  if constexpr (MF) {
    const uint4* qrow = reinterpret_cast<const uint4*>(qp + ((size_t)b * hq + (size_t)g * G + col % G) * D);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) qb[kk] = __builtin_bit_cast(bf16x8_t, qrow[4 * kk + row]);
  } else {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      const uint4 t = reinterpret_cast<const uint4*>(qp + ((size_t)b * hq + (size_t)g * G + h) * D)[col];
      qv[h][0] = t.x; qv[h][1] = t.y; qv[h][2] = t.z; qv[h][3] = t.w;
    }
  }

  // Online-softmax state.  VALU path: every lane keeps (m, l) of all G heads for its row.  Matrix
  // path: lane (row, col) keeps them for head col % G only (m1, l1); the other heads' values sit
  // in the same quad (8-lane group at G = 8) and are broadcast when needed.  acc: dims 8col..8col+7 of every head.
  float m[G], l[G], acc[G][8];
  float m1 = -INFINITY, l1 = 0.0f;
#pragma unroll
  for (int h = 0; h < G; ++h) {
    m[h] = -INFINITY;
    l[h] = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[h][e] = 0.0f;
  }

  const const_i32_ptr bt =
      block_table ? (const_i32_ptr)(block_table + (size_t)b * max_pages) : nullptr;
  const size_t page_stride = (size_t)hkv * P * D;  // elements between physical pages
  const uint16_t* kbase = kp + (size_t)g * P * D;
  const uint16_t* vbase = vp + (size_t)g * P * D;

  // This wavefront's pages: c0 + wave + i * W for i < mine.
  const int mine = (c1 - c0 > wave) ? (c1 - c0 - wave + W - 1) / W : 0;
  auto page_of = [&](int i) { return c0 + wave + i * W; };
  // Raw block-table entry of page i, checked only when used; past either end, that of the page there
  // (so that the entries of a group of buffers are read without a test, in one go).
  auto entry = [&](int i) -> int {
    const int pg = page_of(min(max(i, 0), mine - 1));
    return bt ? bt[pg] : b * max_pages + pg;
  };
  // One 4 KB page of one KV head through a buffer resource whose size covers the page's cached
  // positions only: loads past it return zeros, so the slots
  // past the last position of a partial page read as zeros instead of whatever the pool holds
  // there (a zero V meets a zero weight; the scores of those slots are set to -inf).  The loads
  // are non-temporal (cache policy nt): every cached byte is read exactly once per sweep, and on
  // gfx950 streaming reads marked nt reach a markedly higher share of HBM bandwidth than
  // default-policy reads.
  auto issue = [&](uint4* kk, uint4* vv, int ph, int i) {
    if ((unsigned)ph >= (unsigned)num_pages) {
      poison = true;
      ph = 0;
    }
    const int bytes = min(n - page_of(i) * P, P) * D * 2;
    const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(kbase + (size_t)ph * page_stride), (short)0, bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(vbase + (size_t)ph * page_stride), (short)0, bytes, 0x00020000);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      kk[j] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rk, lane * 16, j * 1024, kNonTemporal));
#pragma unroll
    for (int j = 0; j < 4; ++j)
      vv[j] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rv, lane * 16, j * 1024, kNonTemporal));
  };

  // P V for the 4 positions of this row, weights pr[j][h] of position 4j + row.  (The slots past
  // the last position of a partial page were loaded as zeros and have zero weights.)
  auto accumulate = [&](uint4* vc, auto&& weight) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float vf[8];
      unpack8(vc[j], vf);
#pragma unroll
      for (int h = 0; h < G; ++h) {
        const float p = weight(j, h);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[h][e] = fmaf(p, vf[e], acc[h][e]);
      }
    }
  };

  // Matrix path.  The page's K tile goes through this wavefront's 4 KB of LDS: the coalesced
  // loads give lane (row, col) dims 8col.. of position 4j + row, and the operand reads give lane
  // (row, col) dims 32kk + 8row.. of position pi(col) = 4(col % 4) + col / 4, so that the
  // 16 x 16 result S^T = K Q^T lands with lane (row, col) holding the scores of positions
  // 4i + row (i = 0..3), the very positions whose V this lane reads, for head col % G.  Four
  // v_mfma_f32_16x16x32_bf16 (exact bf16 products, fp32 sums) replace 4G dot products and 4G
  // 16-lane reductions per position quad.
  __shared__ uint4 s_k[MF ? W : 1][MF ? P * 16 : 1];
  auto process_mf = [&](uint4* kc, uint4* vc, int pg) {
    const int valid = n - pg * P;  // slots [0, valid) of this page are cached positions
    uint4* tile = s_k[wave];
#pragma unroll
    for (int j = 0; j < 4; ++j) tile[kslot(4 * j + row, col)] = kc[j];
    // LDS operations of one wavefront complete in order; the fence only keeps the compiler from
    // moving the operand reads above the writes of other lanes' slots.
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int pos = 4 * (col & 3) + (col >> 2);
    f32x4_t st = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
      st = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
          __builtin_bit_cast(bf16x8_t, tile[kslot(pos, 4 * kk + row)]), qb[kk], st, 0, 0, 0);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");

    float sc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) sc[i] = st[i] * scale_log2;
    if (valid < P) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (4 * i + row >= valid) sc[i] = -INFINITY;
    }
    const float mx = fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3]));
    const bool raise = mx > m1 + kLazy;
    float alpha = 1.0f;
    if (raise) {
      alpha = __builtin_amdgcn_exp2f(m1 - mx);  // m1 = -inf -> 0
      l1 *= alpha;
      m1 = mx;
    }
    if (__builtin_amdgcn_ballot_w64(raise)) {   // rare after a shard's first page
#pragma unroll
      for (int h = 0; h < G; ++h) {
        const float a = group_bcast<G>(alpha, h);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[h][e] *= a;
      }
    }
    const float base = (m1 == -INFINITY) ? 0.0f : m1;
    float pr[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) pr[i] = __builtin_amdgcn_exp2f(sc[i] - base);
    l1 += (pr[0] + pr[1]) + (pr[2] + pr[3]);
    accumulate(vc, [&](int j, int h) { return group_bcast<G>(pr[j], h); });
  };

  auto process_valu = [&](uint4* kc, uint4* vc, int pg) {
    const int valid = n - pg * P;  // slots [0, valid) of this page are cached positions

    // Scores of this row's 4 positions for the G heads, log2 domain.
    float sc[4][G];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
      for (int h = 0; h < G; ++h) {
        float d = dot2(kc[j].x, qv[h][0], 0.0f);
        d = dot2(kc[j].y, qv[h][1], d);
        d = dot2(kc[j].z, qv[h][2], d);
        d = dot2(kc[j].w, qv[h][3], d);
        sc[j][h] = row_sum16(d) * scale_log2;
      }
    }
    if (valid < P) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (4 * j + row >= valid) {
#pragma unroll
          for (int h = 0; h < G; ++h) sc[j][h] = -INFINITY;
        }
    }

    float pr[4][G];
#pragma unroll
    for (int h = 0; h < G; ++h) {
      const float mx = fmaxf(fmaxf(sc[0][h], sc[1][h]), fmaxf(sc[2][h], sc[3][h]));
      if (mx > m[h] + kLazy) {
        const float alpha = __builtin_amdgcn_exp2f(m[h] - mx);  // m = -inf -> 0
        l[h] *= alpha;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[h][e] *= alpha;
        m[h] = mx;
      }
      const float base = (m[h] == -INFINITY) ? 0.0f : m[h];
#pragma unroll
      for (int j = 0; j < 4; ++j) pr[j][h] = __builtin_amdgcn_exp2f(sc[j][h] - base);
      l[h] += (pr[0][h] + pr[1][h]) + (pr[2][h] + pr[3][h]);
    }
    accumulate(vc, [&](int j, int h) { return pr[j][h]; });
  };

  // Rotation over NBUF register buffers, all of them in flight while the oldest is waited for: page
  // i is computed, then page i + NBUF requested into its buffer.  No load is issued for a page that does
  // not exist: it would move no data but still take the compute unit's address path 16 cycles a load,
  // 8 loads a page, which a unit of a few pages per wavefront cannot hide.  So the wavefront's pages
  // are preceded by `pad` slots without a page, which only the first group and the computing skip (by
  // uniform branches): the loop's loads are unconditional and its wait counts exact.
  // Block-table entries come a group at a time: scalar loads may return out of order, so waiting for
  // one waits for all, and a group is requested once the one before has been used.
  uint4 kbuf[NBUF][4], vbuf[NBUF][4];
  if (mine > 0) {
    const int pad = (NBUF - mine % NBUF) % NBUF;
    int ent[NBUF];
#pragma unroll
    for (int t = 0; t < NBUF; ++t) ent[t] = entry(t - pad);
    auto process = [&](int t, int i) {
      if constexpr (MF)
        process_mf(kbuf[t], vbuf[t], page_of(i));
      else
        process_valu(kbuf[t], vbuf[t], page_of(i));
    };
#pragma unroll
    for (int t = 0; t < NBUF; ++t)
      if (t == NBUF - 1 || t >= pad) issue(kbuf[t], vbuf[t], ent[t], t - pad);
    int next = NBUF - pad;   // the first page not requested yet; the buffers hold next - NBUF + t
#pragma unroll
    for (int t = 0; t < NBUF; ++t) ent[t] = entry(next + t);
    auto group = [&](bool first) {
      int now[NBUF];
#pragma unroll
      for (int t = 0; t < NBUF; ++t) {
        if (!first || next - NBUF + t >= 0) process(t, next - NBUF + t);
        if (t == 0) {
#pragma unroll
          for (int u = 0; u < NBUF; ++u) now[u] = ent[u];
        }
        issue(kbuf[t], vbuf[t], now[t], next + t);
        if (t == 0) {
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int u = 0; u < NBUF; ++u) ent[u] = entry(next + NBUF + u);
        }
      }
      next += NBUF;
    };
    // The first group apart where there are more than two buffers: its waits must hold for any pad.
    if (NBUF > 2 && next < mine) group(true);
    while (next < mine) group(NBUF <= 2);
#pragma unroll
    for (int t = 0; t < NBUF; ++t)
      if (t == NBUF - 1 || next - NBUF + t >= 0) process(t, next - NBUF + t);
  }
  if constexpr (MF) {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      m[h] = group_bcast<G>(m1, h);
      l[h] = group_bcast<G>(l1, h);
    }
  }

  // Merge the 4 rows of the wavefront (lanes col, col+16, col+32, col+48 hold the same dims), by
  // swapping registers between rows: the sums of 8 dims take 4 row swaps and 2 half swaps, and leave
  // each row with 2 of them (rows 0..3: dims 0-1, 4-5, 2-3, 6-7), each (r0 + r1) + (r2 + r3).
  __shared__ float s_acc[W][G][D];
  __shared__ float s_m[W][G];
  __shared__ float s_l[W][G];
  __shared__ int s_bad[W];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    float M = m[h], x, y;
    swap_rows(M, M, x, y);
    M = fmaxf(x, y);
    swap_halves(M, M, x, y);
    M = fmaxf(x, y);
    const float f = (M == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f(m[h] - M);
    float lh = l[h] * f;
    swap_rows(lh, lh, x, y);
    lh = x + y;
    swap_halves(lh, lh, x, y);
    l[h] = x + y;
    m[h] = M;
    float c[4], d[2];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      swap_rows(acc[h][e] * f, acc[h][e + 4] * f, x, y);
      c[e] = x + y;
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      swap_halves(c[e], c[e + 2], x, y);
      d[e] = x + y;
    }
    // Merge the W wavefronts through LDS and write the unit's (O, ln Z).
    *reinterpret_cast<float2*>(&s_acc[wave][h][col * 8 + (row & 1) * 4 + (row & 2)]) =
        make_float2(d[0], d[1]);
  }
  // Any poisoned wavefront poisons the unit: a ballot per wavefront, met in LDS at the barrier
  // the merge needs anyway (cheaper in registers than __syncthreads_or, which rebuilds a flat
  // thread index from the y and z indices).
  const bool wave_bad = __builtin_amdgcn_ballot_w64(poison) != 0;
  if (lane == 0) {
#pragma unroll
    for (int h = 0; h < G; ++h) { s_m[wave][h] = m[h]; s_l[wave][h] = l[h]; }
    s_bad[wave] = wave_bad ? 1 : 0;
  }
  __syncthreads();
  int bad = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) bad |= s_bad[w];

  const size_t slot = (((size_t)b * max_shards + s) * chunks + c) * hq + (size_t)g * G;
  for (int idx = threadIdx.x; idx < G * D; idx += 64 * W) {
    const int h = idx / D;
    const int d = idx % D;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < W; ++w) M = fmaxf(M, s_m[w][h]);
    float L = 0.0f, A = 0.0f;
    if (M != -INFINITY) {
#pragma unroll
      for (int w = 0; w < W; ++w) {
        const float f = __builtin_amdgcn_exp2f(s_m[w][h] - M);
        L = fmaf(f, s_l[w][h], L);
        A = fmaf(f, s_acc[w][h][d], A);
      }
    } else {
      // No finite score: no position at all (every l is 0; an empty shard) or only NaN scores
      // (a NaN query element; l is NaN), which must come out NaN like any NaN input.
#pragma unroll
      for (int w = 0; w < W; ++w) L += s_l[w][h];
      A = L;
    }
    const bool nan_only = M == -INFINITY && __builtin_isnan(L);
    if (M != -INFINITY || nan_only) {
      // Non-temporal: a thin stream of default-policy writes interleaved with the sweep's
      // reads costs far more HBM time than its bytes (measured ~4% of the sweep).
      if constexpr (MERGE)   // read by another workgroup of this launch (merge_if_last)
        __hip_atomic_store(&out_o[(slot + h) * D + d], A / L, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
      else
        __builtin_nontemporal_store(A / L, &out_o[(slot + h) * D + d]);
    }
    if (d == 0) {
      float lse = nan_only ? NAN : (M == -INFINITY) ? -INFINITY : (M + log2f(L)) * kLn2;
      if (bad) lse = NAN;
      if constexpr (MERGE)
        __hip_atomic_store(&out_lse[slot + h], lse, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      else
        __builtin_nontemporal_store(lse, &out_lse[slot + h]);
    }
  }
  if constexpr (MERGE)
    merge_if_last<G, W>(out_o, out_lse, counters, merged_o, merged_lse, b, g, hq, hkv,
                        max_shards * chunks, counter_step);
}

// Three wavefronts per SIMD with two page buffers (the long-shard sweep) and with three at G <= 2: the matrix path at G = 4
// needs the hint to stay within 168 registers (it does, without spills); deeper buffers take two.
template <int G, int W, int NBUF>
__global__ void __launch_bounds__(64 * W)
__attribute__((amdgpu_waves_per_eu((NBUF == 2 && G <= 4) || (NBUF == 3 && G <= 2) ? 3 : 2)))
decode_split_kernel(const uint16_t* __restrict__ qp, const uint16_t* __restrict__ kp,
                    const uint16_t* __restrict__ vp, const int32_t* __restrict__ block_table,
                    const int32_t* __restrict__ ctx_lens, const int32_t* __restrict__ n_shards,
                    float* __restrict__ out_o, float* __restrict__ out_lse, int32_t hq,
                    int32_t hkv, int32_t max_pages, int32_t num_pages, int32_t max_shards,
                    int32_t chunks, int32_t n_units, int32_t batch, int32_t run, UnitDivisors by,
                    float scale_log2, const int32_t* __restrict__ unit_order) {
  sweep_unit<G, W, NBUF>(qp, kp, vp, block_table, ctx_lens, n_shards, out_o, out_lse, hq, hkv,
                         max_pages, num_pages, max_shards, chunks, n_units, batch, run, by,
                         scale_log2, blockIdx.x, nullptr, nullptr, nullptr, unit_order);
}

// The XCD dealing cycle of rank_units_kernel: kXcdWeightEven : kXcdWeightOdd in lowest terms
// (27 : 23), one cycle holding that many entries of every even and every odd XCD, spread by
// smooth weighted round-robin so that every prefix of the cycle is near the weights.
constexpr int kXcdCycleMax = 256;
struct XcdCycle {
  int len;
  int count[8];                  // entries of XCD x in one cycle
  uint8_t xcd[kXcdCycleMax];     // XCD of entry i
  uint16_t before[kXcdCycleMax]; // entries of the same XCD before entry i
};
constexpr int gcd_of(int a, int b) { return b ? gcd_of(b, a % b) : a; }
constexpr XcdCycle make_xcd_cycle() {
  XcdCycle c{};
  const int gd = gcd_of(kXcdWeightEven, kXcdWeightOdd);
  const int we = kXcdWeightEven / gd, wo = kXcdWeightOdd / gd;
  c.len = 4 * (we + wo);
  int cur[8] = {};
  for (int i = 0; i < c.len; ++i) {
    int best = 0;
    for (int x = 0; x < 8; ++x) cur[x] += (x & 1) ? wo : we;
    for (int x = 1; x < 8; ++x)
      if (cur[x] > cur[best]) best = x;
    cur[best] -= c.len;
    c.xcd[i] = (uint8_t)best;
    c.before[i] = (uint16_t)c.count[best]++;
  }
  return c;
}
static_assert(kXcdWeightEven >= kXcdWeightOdd, "even XCDs take the larger share");
constexpr int kXcdCycleLen = make_xcd_cycle().len;
static_assert(kXcdCycleLen <= kXcdCycleMax, "XCD weights too fine for the cycle table");
static_assert(kXcdCycleMax <= kRankBuckets && kRankBuckets % 8 == 0,
              "the ordering kernel loads the cycle one entry per thread, fills queue t % 8");
__constant__ XcdCycle kXcdCycle = make_xcd_cycle();

// The dispatch order of an unchunked long-shard sweep, [8 * units_per_xcd] (workgroup index ->
// unit, -1 for none).  Workgroups are dispatched in index order, index i on XCD i % 8, and the
// long shards' workgroups live long, so
//  * the (request, shard) pairs are ranked by page count, longest first: a request's shards are
//    of one length, but across a ragged batch they differ 2x, and in shard-index order the last
//    units to start were full-length shards that streamed alone at the end of the launch
//    (longest-processing-time-first list scheduling);
//  * the ranked units (all KV heads of a pair in turn) are dealt to the 8 XCDs' queues in the
//    kXcdWeightEven : kXcdWeightOdd cycle, since the odd-numbered XCDs stream slower, when the
//    even XCDs' queues hold that many (else round-robin); the empty units and the padding fill
//    the rest of every queue.
// Measured on a ragged batch of 64 requests: ranking -4% step time, the weighted dealing -2.4%
// more.  Counting sort in one workgroup over kRankBuckets length buckets of 2^shift pages (the
// last bucket holds the empty shards only); pairs of one bucket keep no particular order among
// themselves.  The order decides only when and where a unit runs, never what it computes.
__global__ void __launch_bounds__(kRankBuckets)
rank_units_kernel(const int32_t* __restrict__ ctx_lens, const int32_t* __restrict__ n_shards,
                  int32_t batch, int32_t max_pages, int32_t max_shards, int32_t hkv,
                  int32_t units_per_xcd, int32_t shift, int32_t* __restrict__ unit_order) {
  __shared__ int32_t count[kRankBuckets];
  __shared__ int32_t scan[2][kRankBuckets];
  __shared__ int32_t ranked[kRankMaxPairs];  // pair index of rank r (unit order: r % B, S-1-r/B)
  __shared__ uint16_t key[kRankMaxPairs];    // bucket of pair r
  __shared__ uint8_t cyc_xcd[kXcdCycleMax];
  __shared__ uint16_t cyc_before[kXcdCycleMax];
  __shared__ int32_t cyc_count[8];
  __shared__ int32_t s_live;
  __shared__ int32_t used[8], first_free[8];
  const int t = threadIdx.x, lane = t & 63;
  const int n_pairs = batch * max_shards;
  constexpr int cycle = kXcdCycleLen;
  // x / hkv and x % hkv: a shift and a mask for the usual power-of-two head counts.
  const int hkv_log2 = (hkv & (hkv - 1)) == 0 ? __builtin_ctz(hkv) : -1;
  auto unit_of = [&](int rank, int j) {  // KV head j % hkv of the pair of rank rank + j / hkv
    return hkv_log2 >= 0 ? ranked[rank + (j >> hkv_log2)] * hkv + (j & (hkv - 1))
                         : ranked[rank + j / hkv] * hkv + j % hkv;
  };
  if (t < cycle) {
    cyc_xcd[t] = kXcdCycle.xcd[t];
    cyc_before[t] = kXcdCycle.before[t];
  }
  if (t < 8) {
    cyc_count[t] = kXcdCycle.count[t];
    used[t] = 0;
  }
  count[t] = 0;
  __syncthreads();
  // Every pair's bucket, kept and counted.  Most pairs of a ragged batch are empty (slots past a
  // request's shards): the empty bucket takes one atomic per wavefront.  (The loops run
  // uniformly over the workgroup, so every ballot sees whole wavefronts.)
  for (int r0 = 0; r0 < n_pairs; r0 += kRankBuckets) {
    const int r = r0 + t;
    int k = 0;
    if (r < n_pairs) {
      const ShardRange range = shard_range(ctx_lens, n_shards, r % batch,
                                           max_shards - 1 - r / batch, max_pages, max_shards);
      const int len = range.p1 - range.p0;
      k = len == 0 ? kRankBuckets - 1 : kRankBuckets - 2 - min(len >> shift, kRankBuckets - 2);
      key[r] = (uint16_t)k;
    }
    const bool empty = r < n_pairs && k == kRankBuckets - 1;
    const uint64_t m = __ballot(empty);
    if (r < n_pairs && !empty) atomicAdd(&count[k], 1);
    if (lane == 0 && m != 0) atomicAdd(&count[kRankBuckets - 1], (int)__popcll(m));
  }
  __syncthreads();
  if (t == 0) s_live = n_pairs - count[kRankBuckets - 1];
  // Exclusive prefix sums of the counts (Hillis-Steele over the shifted counts).
  int cur = 0;
  scan[0][t] = t > 0 ? count[t - 1] : 0;
  __syncthreads();
  for (int d = 1; d < kRankBuckets; d <<= 1) {
    scan[cur ^ 1][t] = scan[cur][t] + (t >= d ? scan[cur][t - d] : 0);
    cur ^= 1;
    __syncthreads();
  }
  count[t] = scan[cur][t];  // first rank of bucket t
  __syncthreads();
  for (int r0 = 0; r0 < n_pairs; r0 += kRankBuckets) {
    const int r = r0 + t;
    const int k = r < n_pairs ? key[r] : 0;
    const bool empty = r < n_pairs && k == kRankBuckets - 1;
    const uint64_t m = __ballot(empty);
    int base = 0;
    if (lane == 0 && m != 0) base = atomicAdd(&count[kRankBuckets - 1], (int)__popcll(m));
    base = __shfl(base, 0);
    if (r < n_pairs) {
      const int at = empty ? base + (int)__popcll(m & ((1ull << lane) - 1))
                           : atomicAdd(&count[k], 1);
      ranked[at] = r;
    }
  }
  __syncthreads();

  // Live unit k (k < R) is KV head k % hkv of the pair of rank k / hkv.  Its XCD and place in that
  // XCD's queue: entry k % cycle of the weighted cycle, or round-robin.
  const int R = s_live * hkv;
  const int full = R / cycle;
  const bool weighted = (int64_t)(full + 1) * cyc_count[0] <= units_per_xcd;
  if (weighted && t < R % cycle) atomicAdd(&used[cyc_xcd[t]], 1);
  __syncthreads();
  if (t < 8) used[t] += weighted ? full * cyc_count[t] : (R + 7 - t) / 8;
  __syncthreads();
  if (t == 0) {
    int acc = 0;
    for (int x = 0; x < 8; ++x) {
      first_free[x] = acc;
      acc += units_per_xcd - used[x];
    }
  }
  __syncthreads();
  for (int k = t; k < R; k += kRankBuckets) {
    int x, pos;
    if (weighted) {
      const int i = k % cycle;
      x = cyc_xcd[i];
      pos = (k / cycle) * cyc_count[x] + cyc_before[i];
    } else {
      x = k & 7;
      pos = k >> 3;
    }
    unit_order[8 * pos + x] = unit_of(0, k);
  }
  // The rest of every queue: empty unit e is KV head e % hkv of the pair of rank s_live + e / hkv
  // (then -1).  Thread t fills queue t % 8 (kRankBuckets is a multiple of 8), places
  // t / 8, t / 8 + 128, ... from the queue's first free one on.
  const int n_empty = n_pairs * hkv - R;
  const int x = t & 7;
  constexpr int kStride = kRankBuckets / 8;
  const int lo = used[x];
  int pos = t >> 3;
  if (pos < lo) pos += (lo - pos + kStride - 1) / kStride * kStride;
  for (int e = first_free[x] + pos - lo; pos < units_per_xcd; pos += kStride, e += kStride)
    unit_order[8 * pos + x] = e < n_empty ? unit_of(s_live, e) : -1;
}

// Fill p.unit_order (when the sweep has one) on `stream`, ahead of the sweep.
hipError_t launch_rank(const SplitParams& p, hipStream_t stream) {
  if (p.unit_order == nullptr) return hipSuccess;
  hipLaunchKernelGGL(rank_units_kernel, dim3(1), dim3(kRankBuckets), 0, stream, p.ctx_lens,
                     p.n_shards, p.batch, p.max_pages, p.max_shards, p.hkv, p.units_per_xcd,
                     p.rank_shift, p.unit_order);
  return hipGetLastError();
}

template <int G, int W, int NBUF>
__global__ void __launch_bounds__(64 * W)
__attribute__((amdgpu_waves_per_eu(G >= 8 ? 2 : 3)))   // the unfused sweep's occupancy
decode_fused_kernel(const uint16_t* __restrict__ qp, const uint16_t* __restrict__ kp,
                    const uint16_t* __restrict__ vp, const int32_t* __restrict__ block_table,
                    const int32_t* __restrict__ ctx_lens, const int32_t* __restrict__ n_shards,
                    float* __restrict__ out_o, float* __restrict__ out_lse, int32_t hq,
                    int32_t hkv, int32_t max_pages, int32_t num_pages, int32_t max_shards,
                    int32_t chunks, int32_t n_units, int32_t batch, int32_t run, UnitDivisors by,
                    float scale_log2, int32_t* __restrict__ counters,
                    uint16_t* __restrict__ merged_o, float* __restrict__ merged_lse,
                    int32_t counter_step) {
  sweep_unit<G, W, NBUF, true>(qp, kp, vp, block_table, ctx_lens, n_shards, out_o, out_lse, hq,
                               hkv, max_pages, num_pages, max_shards, chunks, n_units,
                               batch, run, by, scale_log2, blockIdx.x, counters,
                               merged_o, merged_lse, nullptr, counter_step);
}

template <int G>
hipError_t launch_fused_g(const SplitParams& p, int32_t* counters, int32_t counter_step, void* out,
                          float* lse, hipStream_t stream) {
  const unsigned grid = 8u * (unsigned)p.units_per_xcd;
  hipLaunchKernelGGL((decode_fused_kernel<G, kSplitWaves, kSplitBuffers>), dim3(grid),
                     dim3(64 * kSplitWaves), 0, stream, p.q, p.k, p.v, p.block_table, p.ctx_lens,
                     p.n_shards, p.out_o, p.out_lse, p.hq, p.hkv, p.max_pages, p.num_pages,
                     p.max_shards, p.chunks, p.n_units, p.batch, p.run, p.by, p.scale_log2, counters,
                     static_cast<uint16_t*>(out), lse, counter_step);
  return hipGetLastError();
}

template <int G, int NBUF>
hipError_t launch_gn(const SplitParams& p, hipStream_t stream) {
  const hipError_t e = launch_rank(p, stream);
  if (e != hipSuccess) return e;
  const unsigned grid = 8u * (unsigned)p.units_per_xcd;
  hipLaunchKernelGGL((decode_split_kernel<G, kSplitWaves, NBUF>), dim3(grid), dim3(64 * kSplitWaves),
                     0, stream, p.q, p.k, p.v, p.block_table, p.ctx_lens, p.n_shards, p.out_o,
                     p.out_lse, p.hq, p.hkv, p.max_pages, p.num_pages, p.max_shards, p.chunks,
                     p.n_units, p.batch, p.run, p.by, p.scale_log2, p.unit_order);
  return hipGetLastError();
}

// The host picks deep buffers from the shard length (short shards of at least kDeepMinPages);
// NBUF only changes how far ahead pages are requested, never the arithmetic.
template <int G>
hipError_t launch_g(const SplitParams& p, hipStream_t stream) {
  if (p.deep && G <= 2 && p.n_units < kDeepManyUnits)
    return launch_gn<G, G <= 2 ? kFewUnitsBuffers : kSplitBuffers>(p, stream);
  if (p.deep) return launch_gn<G, split_buffers_deep(G)>(p, stream);
  return launch_gn<G, kSplitBuffers>(p, stream);
}

// One launch, two roles: the sweep's workgroups and those of a fused product (linear_body.h) share
// one grid, so the hardware dispatcher runs both at once on every CU (the sweep beside the
// feed-forward, §3).  Groups of 8 consecutive workgroup indices (one per XCD) are dealt to the two
// roles in proportion to their sizes, so both start together and each keeps its index modulo 8;
// every workgroup does exactly what it would do in its own launch.
// MB: rows of a product on the vector path, one or several behind the SwiGLU prologue; products on the
// tiles, of any number of rows, are in the kernels of kTilesBucket.
// The occupancy the sweep alone reaches (registers), asked of the shared kernel too, so that
// the product's role does not lower it.
constexpr int kTilesBucket = 2;

template <int G, int MB>
__global__ void __launch_bounds__(64 * kSplitWaves)
__attribute__((amdgpu_waves_per_eu(G >= 8 ? 2 : 3)))
sweep_beside_linear_kernel(
    const uint16_t* __restrict__ qp, const uint16_t* __restrict__ kp,
    const uint16_t* __restrict__ vp, const int32_t* __restrict__ block_table,
    const int32_t* __restrict__ ctx_lens, const int32_t* __restrict__ n_shards,
    float* __restrict__ out_o, float* __restrict__ out_lse, int32_t hq, int32_t hkv,
    int32_t max_pages, int32_t num_pages, int32_t max_shards, int32_t chunks, int32_t n_units,
    int32_t units_per_xcd, int32_t batch, int32_t run, UnitDivisors by, float scale_log2,
    const int32_t* __restrict__ unit_order, const uint16_t* __restrict__ x,
    const uint16_t* __restrict__ w,
    const uint16_t* __restrict__ gain, const uint16_t* __restrict__ residual,
    uint16_t* __restrict__ out_a, uint16_t* __restrict__ out_b, int32_t M, int32_t N, int32_t K,
    int32_t n_split, float eps, int32_t prologue, int32_t glu, int32_t tiles /* one row: rows a wavefront */,
    int32_t linear_groups) {
  static_assert(64 * kSplitWaves == lin::kThreads, "both roles use the same workgroup size");
  const unsigned j = blockIdx.x / 8u, lane8 = blockIdx.x % 8u;
  const unsigned long long S = (unsigned)units_per_xcd, T = S + (unsigned)linear_groups;
  const unsigned before = (unsigned)(j * S / T);          // sweep groups dealt before group j
  if ((unsigned)((j + 1ull) * S / T) > before) {
    sweep_unit<G, kSplitWaves, kSplitBuffers>(qp, kp, vp, block_table, ctx_lens, n_shards, out_o,
                                              out_lse, hq, hkv, max_pages, num_pages, max_shards,
                                              chunks, n_units, batch, run, by,
                                              scale_log2, 8u * before + lane8, nullptr, nullptr,
                                              nullptr, unit_order);
    return;
  }
  constexpr int R = lin::beside_rows(MB);
  const unsigned lb = 8u * (j - before) + lane8;
  if (MB > 1 && (MB > kTilesBucket || tiles == 0)) {   // several rows behind the SwiGLU prologue
    lin::linear_rows<kProSwiglu, MB, 2, R>(x, w, gain, residual, out_a, out_b, M, N, K, n_split, eps, lb);
    return;
  }
  if constexpr (MB == kTilesBucket) {
    __shared__ lin::TileLds<2, kSplitWaves> lds;
    auto tile = [&](auto t) {
      constexpr int T = decltype(t)::value, RW = T * lin::kTileRows;
      auto& l = reinterpret_cast<lin::TileLds<T, kSplitWaves>&>(lds);
      const int n0 = (int)lb * RW;
      if (prologue == kProRmsNorm) {
        if (glu)
          lin::linear_tiles<kProRmsNorm, T, kSplitWaves, 1, true>(
              x, w, gain, residual, out_a, out_b, M, N, K, n_split, eps, n0, RW, l);
        else
          lin::linear_tiles<kProRmsNorm, T, kSplitWaves, 1, false>(
              x, w, gain, residual, out_a, out_b, M, N, K, n_split, eps, n0, RW, l);
      } else {
        if (glu)
          lin::linear_tiles<kProNone, T, kSplitWaves, 1, true>(
              x, w, gain, residual, out_a, out_b, M, N, K, n_split, eps, n0, RW, l);
        else
          lin::linear_tiles<kProNone, T, kSplitWaves, 1, false>(
              x, w, gain, residual, out_a, out_b, M, N, K, n_split, eps, n0, RW, l);
      }
    };
    if (tiles == 1)
      tile(std::integral_constant<int, 1>{});
    else
      tile(std::integral_constant<int, 2>{});
  } else if constexpr (MB == 1) {
    // K in groups of three chunks of 512 from 1,024 to 10,240 inputs, else of two (with two rows a wavefront
    // always three).  Fewer waits are worth the loads past the end that three may add: one row beside the
    // sweep of one request of 4,608 positions, us with groups of two and three: 1,024 x 2,048 7.43 / 7.35,
    // 2,048 x 2,560 9.62 / 9.22, 1,024 x 3,072 8.05 / 7.41, 2,560 x 4,096 11.6 / 11.2, but 4,096 x 14,336
    // 29.7 / 30.2, where many groups hide a wait.
    auto rows = [&](auto unroll, auto per) {
      constexpr int U = decltype(unroll)::value, RW = decltype(per)::value;
      if (prologue == kProRmsNorm)
        lin::linear_rows<kProRmsNorm, 1, U, RW>(x, w, gain, residual, out_a, out_b, M, N, K, n_split, eps, lb);
      else if (prologue == kProSwiglu)
        lin::linear_rows<kProSwiglu, 1, U, RW>(x, w, gain, residual, out_a, out_b, M, N, K, n_split, eps, lb);
      else
        lin::linear_rows<kProNone, 1, U, RW>(x, w, gain, residual, out_a, out_b, M, N, K, n_split, eps, lb);
    };
    auto gated = [&](auto unroll) {
      constexpr int U = decltype(unroll)::value;
      if (prologue == kProRmsNorm)
        lin::linear_rows<kProRmsNorm, 1, U, R, true>(x, w, gain, residual, out_a, out_b, M, N, K, n_split,
                                                     eps, lb);
      else
        lin::linear_rows<kProNone, 1, U, R, true>(x, w, gain, residual, out_a, out_b, M, N, K, n_split, eps,
                                                  lb);
    };
    using std::integral_constant;
    const bool three = K > 1024 && K <= 10240;
    if (glu && three) gated(integral_constant<int, 3>{});
    else if (glu) gated(integral_constant<int, 2>{});
    else if (tiles == 2) rows(integral_constant<int, 3>{}, integral_constant<int, 2>{});
    else if (three) rows(integral_constant<int, 3>{}, integral_constant<int, R>{});
    else rows(integral_constant<int, 2>{}, integral_constant<int, R>{});
  }
}

// Tiles of a product's workgroup beside the sweep: one, so that a long K is dealt to many workgroups, but
// two
//  * where the tiles one by one would be two rounds of a compute unit or more and K is short, so that
//    starting and meeting is most of a workgroup's life (two rows beside the sweep of one request of 9,000
//    positions, us: 6,144 x 1,024 with GLU 18.5 -> 13.2, 19,456 x 2,560 32.1 -> 27.1; 14.5 and 29.2 on the
//    vector path.  4,096 x 2,048 12.7 -> 13.7, 4,096 x 14,336 28.7 -> 38.7);
//  * where that leaves every workgroup of the launch a compute unit of its own (1,024 x 1,024 beside 192
//    workgroups of the sweep 8.6 -> 7.0, vector path 7.9; 1,024 x 3,072 8.9 -> 7.7).
// Most units of a ragged batch are empty, so the count is of what may run, not of what does.
int beside_tiles(const SplitParams& p, const LinearParams& l) {
  constexpr int kUnits = 256, R = lin::kTileRows;
  const int64_t sweep = 8 * (int64_t)p.units_per_xcd;
  const bool rounds = l.N > 2 * kUnits * R && l.K <= 4096;
  const bool own = sweep + (l.N + R - 1) / R > kUnits && sweep + (l.N + 2 * R - 1) / (2 * R) <= kUnits;
  return rounds || own ? 2 : 1;
}

// Whether one row's product beside the sweep has two output rows a wavefront, not beside_rows: a long K is
// then dealt to twice the wavefronts (us, four and two: 2,048 x 5,632 13.5 / 11.6, 2,560 x 9,728 18.4 /
// 16.2, 4,096 x 11,008 26.3 / 22.9, beside 32 KV heads 44.4 / 34.0).  A short one is better in few
// workgroups (1,024 x 3,072 7.8 / 9.3, 6,144 x 1,024 with GLU 9.2 / 10.6), a very long one keeps enough
// loads in flight with four (5,120 x 25,600 52.3 / 59.3).
bool beside_two_rows(const LinearParams& l) {
  return l.M == 1 && !l.glu && l.N >= 2048 && l.K > 4096 && l.K <= 16384;
}

template <int G, int MB>
hipError_t launch_beside(const SplitParams& p, const LinearParams& l, hipStream_t stream) {
  const bool two = MB == 1 && beside_two_rows(l);
  const int tiles = lin::takes_tiles(l) ? beside_tiles(p, l) : two ? 2 : 0;
  const int per_group = lin::takes_tiles(l) ? tiles * lin::kTileRows
                                            : lin::kRowsPerBlock * (two ? 2 : lin::beside_rows(MB));
  const int linear_groups = ((l.N + per_group - 1) / per_group + 7) / 8;
  const unsigned grid = 8u * ((unsigned)p.units_per_xcd + (unsigned)linear_groups);
  const hipError_t e = launch_rank(p, stream);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((sweep_beside_linear_kernel<G, MB>), dim3(grid), dim3(64 * kSplitWaves), 0,
                     stream, p.q, p.k, p.v, p.block_table, p.ctx_lens, p.n_shards, p.out_o,
                     p.out_lse, p.hq, p.hkv, p.max_pages, p.num_pages, p.max_shards, p.chunks,
                     p.n_units, p.units_per_xcd, p.batch, p.run, p.by, p.scale_log2, p.unit_order,
                     l.x, l.w, l.gain,
                     l.residual, l.out_a, l.out_b, l.M, l.N, l.K, l.n_split, l.eps, l.prologue,
                     l.glu ? 1 : 0, tiles, linear_groups);
  return hipGetLastError();
}

template <int G>
hipError_t launch_beside_g(const SplitParams& p, const LinearParams& l, hipStream_t stream) {
  switch (lin::takes_tiles(l) ? kTilesBucket : lin::rows_bucket(l.M)) {
    case 1: return launch_beside<G, 1>(p, l, stream);
    case 2: return launch_beside<G, 2>(p, l, stream);
    case 4: return launch_beside<G, 4>(p, l, stream);
    default: return launch_beside<G, 8>(p, l, stream);
  }
}

// Workgroups of the two-buffer kernel that the chunk rule counts as resident per compute unit: those of
// the kernel's earlier register counts, which the rule was measured with (per-GPU share of a 2^20
// request, 1,024 instead of 768 at G = 2: 90.4 -> 91.3 us, more workgroups in flight only add
// contention), never more than the device holds.
constexpr int counted_per_unit(int group) { return group == 1 ? 4 : group == 8 ? 2 : 3; }

template <int G>
int resident_g() {
  int dev = 0, cus = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(
          &per_cu, decode_split_kernel<G, kSplitWaves, kSplitBuffers>, 64 * kSplitWaves, 0) !=
          hipSuccess) {
    (void)hipGetLastError();  // leave no error behind for the next launch check
    return 0;
  }
  return cus * (per_cu < counted_per_unit(G) ? per_cu : counted_per_unit(G));
}

}  // namespace

int split_resident_workgroups(int group) {
  static std::atomic<int> cached[4] = {{-1}, {-1}, {-1}, {-1}};
  const int k = group == 1 ? 0 : group == 2 ? 1 : group == 4 ? 2 : group == 8 ? 3 : -1;
  if (k < 0) return 0;
  int v = cached[k].load(std::memory_order_relaxed);
  if (v < 0) {
    v = k == 0 ? resident_g<1>() : k == 1 ? resident_g<2>() : k == 2 ? resident_g<4>() : resident_g<8>();
    if (v > 0) cached[k].store(v, std::memory_order_relaxed);
  }
  return v;
}

hipError_t launch_decode_split(const SplitParams& p, int group, hipStream_t stream) {
  switch (group) {
    case 1: return launch_g<1>(p, stream);
    case 2: return launch_g<2>(p, stream);
    case 4: return launch_g<4>(p, stream);
    case 8: return launch_g<8>(p, stream);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_decode_split_beside(const SplitParams& p, int group, const LinearParams& l,
                                     hipStream_t stream) {
  if (lin::takes_single_rows(l)) {
    const hipError_t e = launch_decode_split(p, group, stream);
    return e != hipSuccess ? e : launch_linear(l, stream);
  }
  switch (group) {
    case 1: return launch_beside_g<1>(p, l, stream);
    case 2: return launch_beside_g<2>(p, l, stream);
    case 4: return launch_beside_g<4>(p, l, stream);
    case 8: return launch_beside_g<8>(p, l, stream);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_decode_fused(const SplitParams& p, int group, int32_t* counters,
                               int32_t counter_step, void* out, float* lse, hipStream_t stream) {
  switch (group) {
    case 1: return launch_fused_g<1>(p, counters, counter_step, out, lse, stream);
    case 2: return launch_fused_g<2>(p, counters, counter_step, out, lse, stream);
    case 4: return launch_fused_g<4>(p, counters, counter_step, out, lse, stream);
    case 8: return launch_fused_g<8>(p, counters, counter_step, out, lse, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace qf
