// Internal interface between the host library (qfattn_api.hip) and the kernel files.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace qf {

constexpr int kHeadDim = 128;     // D
constexpr int kPage = 16;         // P
constexpr int kSplitWaves = 4;    // waves per workgroup of the sweep kernel
// Pages in registers per wave of the sweep, all in flight while the oldest is waited for.  Long shards
// keep three wavefronts per SIMD with 2 (long ragged shards lose 4% at two wavefronts).  Short shards of
// some length (a handful of pages per wavefront, so a workgroup's life is mostly its first pages'
// latency) go deeper, at two wavefronts per SIMD: measured on MI355X, 32-page shards at G=2 2% faster.
// Shorter ones keep 2: 3 pages per wavefront all at once (4,608 positions in units of 12 pages) took
// 11.1 us a layer against 10.5.
constexpr int kSplitBuffers = 2;
constexpr int split_buffers_deep(int group) { return group <= 2 ? 4 : group == 4 ? 3 : 2; }
constexpr int kDeepMinPages = 4 * kSplitWaves;   // shard pages (at full capacity) for deep buffers
// At G <= 2, launches of fewer units than kDeepManyUnits (5 rounds of resident workgroups) take 3 buffers,
// which keep three wavefronts per SIMD: with few rounds what is resident counts (12 ragged requests of up
// to 7,003 positions at 16 shards 26.8 -> 25.5 us a layer, 8 requests of 4,608 at 8 shards 35.1 -> 33.9),
// with many the depth (32 requests of 32,768 at 64 shards 676 us with 3; 4 and 5 alike within 0.5%).
constexpr int kFewUnitsBuffers = 3;
constexpr int kDeepManyUnits = 4096;

// Shards at least this long (pages, at full capacity) are swept in the long-shard order (largest
// shard first), shorter ones in the short-shard order (dealt to the XCDs by items; decode_split.hip).
constexpr int kLongShardPages = 128;
// Items of the short-shard order (units_per_item in qfattn_api.hip).
constexpr int kDealManyUnits = 4096;
constexpr int kDealFewUnits = 256;
constexpr int kDealItemUnits = 8;
constexpr int kDealMostSlots = 1024;
constexpr int kDealMostUnits = 1 << 23;
// Relative page shares of the sub-shard chunks of a long shard that run on even- and odd-numbered
// XCDs (decode_split.hip): the odd XCDs stream slower.
constexpr int kXcdWeightEven = 1080;
constexpr int kXcdWeightOdd = 920;
// The one-workgroup kernel that orders the units of an unchunked long-shard sweep
// (decode_split.hip): length buckets (= its threads), and the most (request, shard) pairs it
// ranks (held in LDS).
constexpr int kRankBuckets = 1024;
constexpr int kRankMaxPairs = 8192;

// Division of n < 2^31 by a launch constant d: (n * mul) >> shift with mul = ceil(2^shift / d),
// shift = 31 + ceil(log2 d); exact, since n (mul d - 2^shift) < 2^31 d <= 2^shift.
struct Divisor {
  uint32_t mul = 1u << 31, shift = 31;
  Divisor() = default;
  explicit Divisor(uint32_t d) {
    uint32_t l = 0;
    while ((uint64_t(1) << l) < d) ++l;
    shift = 31 + l;
    mul = (uint32_t)(((uint64_t(1) << shift) + d - 1) / d);
  }
  __host__ __device__ uint32_t of(uint32_t n) const { return (uint32_t)(((uint64_t)n * mul) >> shift); }
};
// The divisors that turn a workgroup index into a unit of the short-shard order.
struct UnitDivisors {
  Divisor run, hkv, chunks, shards;
};

// One launch of the sweep kernel.  A workgroup handles one unit (request b, shard s, chunk c,
// KV head g); its output slot is [((b * max_shards + s) * chunks + c) * hq + g * G + h].
struct SplitParams {
  const uint16_t* q;            // bf16 [B, Hq, D]
  const uint16_t* k;            // bf16 [num_pages, Hkv, P, D]
  const uint16_t* v;
  const int32_t* block_table;   // [B, max_pages] or null (identity)
  const int32_t* ctx_lens;      // [B]
  const int32_t* n_shards;      // [B]
  float* out_o;                 // fp32 [B, max_shards, chunks, Hq, D]
  float* out_lse;               // fp32 [B, max_shards, chunks, Hq]
  int32_t batch, hq, hkv, max_pages, num_pages, max_shards, chunks;
  int32_t n_units;              // B * max_shards * chunks * Hkv
  // Short-shard order: units of an item, which run on one XCD; long-shard order: 0.
  int32_t run;
  UnitDivisors by;
  int32_t units_per_xcd;        // workgroup indices per XCD: whole items (run > 0), ceil(n_units / 8)
  // The long-shard order with chunks == 1 only, or null: [8 * units_per_xcd] int32 that an ordering
  // kernel, launched just before the sweep, fills with the unit each workgroup index sweeps (-1:
  // none): longest shard first, dealt to the XCDs by kXcdWeightEven / kXcdWeightOdd
  // (rank_shift: log2 of the length buckets' width in pages).
  int32_t* unit_order;
  int32_t rank_shift;
  bool deep;                    // short shards of >= kDeepMinPages pages: split_buffers_deep(G)
  float scale_log2;             // softmax scale * log2(e)
};

// Merge of `entries` partial states per (row, head):
//   in  O [rows, entries, hq, D] fp32, lse [rows, entries, hq] fp32 (natural log)
//   out O [rows, hq, D] (fp32 or bf16), lse [rows, hq] fp32 (may be null)
// With q non-null (final output only) the current token is folded in after the merge:
//   q bf16 [rows, hq, D], k_cur / v_cur bf16 [rows, hkv, D].
struct AppendParams;

struct MergeParams {
  const float* in_o;
  const float* in_lse;
  void* out_o;
  float* out_lse;
  int32_t rows, entries, hq;
  const uint16_t* q = nullptr;
  const uint16_t* k_cur = nullptr;
  const uint16_t* v_cur = nullptr;
  int32_t hkv = 1;
  float scale = 0.0f;
  // With the current token (q, k_cur, v_cur): also append k_cur and v_cur to the cache and
  // advance ctx_lens (AppendParams below; k_new / v_new / advance there are not used).
  const AppendParams* append = nullptr;
};

// Cache append: write the current token's key and value at position ctx_lens[b] of request b.
struct AppendParams {
  uint16_t* k;                  // bf16 [num_pages, Hkv, P, D]
  uint16_t* v;
  const int32_t* block_table;   // [B, max_pages] or null (identity)
  int32_t* ctx_lens;            // [B]; advanced by one after the write when advance != 0
  const uint16_t* k_new;        // bf16 [B, Hkv, D]
  const uint16_t* v_new;
  int32_t* status;              // optional: set to 1 when an append is skipped
  int32_t batch, hkv, max_pages, num_pages, advance;
};

hipError_t launch_kv_append(const AppendParams& p, hipStream_t stream);
// out = W . P(x) (+ residual) for a few input rows (block_ops.hip).
constexpr int kProNone = 0, kProRmsNorm = 1, kProSwiglu = 2;
constexpr int kLinearMaxRows = 8;
struct LinearParams {
  const uint16_t* x;         // bf16 [M, K] ([M, 2K] for kProSwiglu: gate, then up)
  const uint16_t* w;         // bf16 [N, K]
  const uint16_t* gain;      // bf16 [K] (kProRmsNorm)
  const uint16_t* residual;  // bf16 [M, N] or nullptr
  uint16_t* out_a;           // bf16 [M, n_split]
  uint16_t* out_b;           // bf16 [M, N - n_split]
  int M, N, K, n_split, prologue;
  float eps;
  bool glu;                  // rows of W alternate gate / up; out = silu(gate) * up, N / 2 columns
};
hipError_t launch_linear(const LinearParams& p, hipStream_t stream);
hipError_t launch_linear_pair(const LinearParams& a, const LinearParams& b, hipStream_t stream);
hipError_t launch_linear_merge(const LinearParams& l, const MergeParams& m, hipStream_t stream);
// out = W . attn (+ residual) for one request, attn being the current token folded into the merged pair
// (m.in_o, merged_lse) of its cache, written to m.out_o / m.out_lse, and the token appended (a).
hipError_t launch_linear_attn(const LinearParams& l, const MergeParams& m, const float* merged_lse,
                              const AppendParams& a, hipStream_t stream);
// The sweep with the merge fused into its last workgroup per (request, KV head)
// (decode_split.hip): p.out_o / p.out_lse hold the partial states; the counter of request b and KV head g
// is counters[(b * hkv + g) * counter_step], zero before and after.
hipError_t launch_decode_fused(const SplitParams& p, int group, int32_t* counters,
                               int32_t counter_step, void* out, float* lse, hipStream_t stream);
// Counters this far apart lie in cache lines of their own (128 bytes).
constexpr int kCounterStep = 32;
// The sweep and a fused product in one launch (decode_split.hip).
hipError_t launch_decode_split_beside(const SplitParams& p, int group, const LinearParams& l,
                                      hipStream_t stream);

// Host simulation of the layer-wise decode schedule (schedule.cpp).
int simulate_schedule(int R, const double* arrival, const double* attn_time, int L, int wiring,
                      double ffn_time, int min_batch, double max_wait, double* finish,
                      double* sweep_start, double* sweep_end, double* ffn_depart,
                      double* ffn_return);

hipError_t launch_decode_split(const SplitParams& p, int group, hipStream_t stream);

// The allocation-free decode's fixed scratch (decode_noalloc.hip): one device array per GPU for the partial
// states.  The sizes that a call may have are the interface's (the bound on (request, KV head) groups and
// the 256 KiB below the 64 MiB date from a form with arrival counters in the array).
constexpr size_t kNoallocStateBytes = (size_t(64) << 20) - (size_t(256) << 10);
constexpr int64_t kNoallocMaxGroups = 65536;
// This device's scratch (looked up on the first call on the device).
hipError_t noalloc_states(void** states);

// Workgroups of the long-shard sweep (kSplitBuffers) at group size `group` that are resident on
// the current device at once (compute units x workgroups per unit); 0 when there is no device to
// ask.  Queried once per group size and kept.
int split_resident_workgroups(int group);
// to_bf16 = false: partial-state output (fp32 O not written for an empty row);
// to_bf16 = true:  final output (bf16, +0 for an empty row).
// max_waves: at most this many wavefronts per row (a row of more slots than one round of them covers
// takes more rounds; the sums of a row depend on it only then).
hipError_t launch_merge(const MergeParams& p, bool to_bf16, hipStream_t stream, int max_waves = 16);

}  // namespace qf
