// The two ends of a decoder block's attention at one request, each in a launch with the product next to
// it (Q-First, arXiv:2608.15473, §2): at one request every launch of a block costs 3 to 5 us of latency
// against 1 us of bytes, so the number of launches is what bounds a step.
//
//  * linear_merge_kernel (block_ops.hip): the merge of the shard slots into one (O, ln Z) per query head
//    beside a product (W_k|W_v N1(z)): neither reads what the other writes.
//  * attn_rows: out = W . attn (+ residual) where attn is the current token folded into that pair
//    (merge_body.h), computed by every workgroup for itself into LDS: 16 lanes hold one head, 8 dims
//    each, so the score of the current token is a 16-lane reduction.  The weights are requested first.
//    One more workgroup writes the folded attention and its log-sum-exp, and appends the token's key
//    and value.
//
// Measured on steps of one request in a HIP graph (the merge, fold and append in a launch between the
// two products before): Qwen3-0.6B sizes, 4,608 positions, 28 blocks 688 -> 598 us; 400 positions, 10
// blocks 220 -> 205 against the fold in every wavefront's registers (which took Qwen3-4B's 32 heads from
// 477 to 500 us for 6 blocks; with the fold in LDS 479).
#pragma once

#include "append_body.h"
#include "linear_body.h"
#include "merge_body.h"

namespace qf {
namespace lin {

// Merged attention of one request's cached positions and its current token (device pointers).
struct AttnFold {
  const float* o;          // fp32 [Hq, D]; where lse is -inf it may hold anything: selected out
  const float* lse;        // fp32 [Hq]
  const uint16_t* q;       // bf16 [Hq, D]
  const uint16_t* k_cur;   // bf16 [Hkv, D]
  const uint16_t* v_cur;
  int32_t hq, group;
  float scale;
};

struct FoldInputs {
  uint4 o[2], q, k, v;
  float lse;
};

// Elements 8 vec .. 8 vec + 7 of [Hq, D], for vec = 16 head + lane % 16; `in`: the head exists.
__device__ __forceinline__ FoldInputs load_fold(const AttnFold& f, int vec, bool in) {
  FoldInputs x{};
  x.lse = -INFINITY;
  if (in) {
    const int h = vec >> 4, cur = (h / f.group) * 16 + (vec & 15);
    x.o[0] = reinterpret_cast<const uint4*>(f.o)[2 * vec];
    x.o[1] = reinterpret_cast<const uint4*>(f.o)[2 * vec + 1];
    x.q = reinterpret_cast<const uint4*>(f.q)[vec];
    x.k = reinterpret_cast<const uint4*>(f.k_cur)[cur];
    x.v = reinterpret_cast<const uint4*>(f.v_cur)[cur];
    x.lse = f.lse[h];
  }
  return x;
}

// The folded attention of this lane's 8 dims, rounded to bf16 (packed), and its log-sum-exp.
__device__ __forceinline__ uint4 fold8(const FoldInputs& x, float scale, float& lse_out) {
  float q[8], k[8], v[8], a[8];
  unpack8(x.q, q);
  unpack8(x.k, k);
  unpack8(x.v, v);
  float dot = 0.0f;
#pragma unroll
  for (int j = 0; j < 8; ++j) dot = fmaf(q[j], k[j], dot);
  const float s_jj = mrg::row_sum16(dot) * scale;
  const float t = 1.0f / (1.0f + expf(-(x.lse - s_jj)));   // weight of the cached history
  const bool empty = x.lse == -INFINITY;
  const uint32_t o[8] = {x.o[0].x, x.o[0].y, x.o[0].z, x.o[0].w, x.o[1].x, x.o[1].y, x.o[1].z, x.o[1].w};
#pragma unroll
  for (int j = 0; j < 8; ++j)
    a[j] = (1.0f - t) * v[j] + t * (empty ? 0.0f : __uint_as_float(o[j]));
  const float mx = fmaxf(x.lse, s_jj);
  float joined = mx + log1pf(expf(-fabsf(x.lse - s_jj)));  // stabilised logaddexp
  if (mx == -INFINITY) joined = -INFINITY;
  lse_out = (x.lse != x.lse || s_jj != s_jj) ? NAN : joined;
  auto pair = [&](int j) { return bf16_rne(a[j]) | (bf16_rne(a[j + 1]) << 16); };
  return make_uint4(pair(0), pair(2), pair(4), pair(6));
}

// Output rows R (4 bid + wavefront) .. + R - 1 of out = W . attn (+ residual) for one request, U chunks of
// 4 heads in a group; s_x: 64 U entries.  The sum of a row is that of linear_rows.
template <int U, int R>
__device__ __forceinline__ void attn_rows(const AttnFold& f, const LinearParams& p, unsigned bid,
                                          uint4* s_x) {
  const int lane = threadIdx.x & 63;
  const int n0 = ((int)bid * kRowsPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * R;
  const int vecs = p.K / 8;
  __amdgpu_buffer_rsrc_t rw[R];
  uint16_t res[R];
  float acc[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const bool in = n0 + r < p.N;   // rows past the end read as zeros
    rw[r] = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(p.w + (size_t)(in ? n0 + r : 0) * p.K), (short)0, in ? p.K * 2 : 0,
        0x00020000);
    res[r] = p.residual && in ? p.residual[n0 + r] : 0;
    acc[r] = 0.0f;
  }
  for (int c0 = 0; c0 < vecs; c0 += 64 * U) {
    uint4 wv[U][R];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int r = 0; r < R; ++r)
        wv[u][r] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(
                                                 rw[r], (c0 + u * 64 + lane) * 16, 0, 2));
    if (c0 > 0) __syncthreads();   // the last group's values have been read
    for (int i = threadIdx.x; i < 64 * U; i += kThreads) {   // whole rows of 16 lanes
      float lse;
      s_x[i] = fold8(load_fold(f, c0 + i, c0 + i < vecs), f.scale, lse);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float xf[8];
      unpack8(s_x[u * 64 + lane], xf);
      if (c0 + u * 64 + lane < vecs)
#pragma unroll
        for (int r = 0; r < R; ++r) {
          float wf[8];
          unpack8(wv[u][r], wf);
#pragma unroll
          for (int j = 0; j < 8; ++j) acc[r] = fmaf(wf[j], xf[j], acc[r]);
        }
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc[r] += __shfl_xor(acc[r], o);
    const int n = n0 + r;
    if (lane == 0 && n < p.N) {
      if (p.residual) acc[r] += lo(res[r]);
      const uint16_t b = (uint16_t)bf16_rne(acc[r]);
      if (n < p.n_split)
        p.out_a[n] = b;
      else
        p.out_b[n - p.n_split] = b;
    }
  }
}

// The folded attention and its log-sum-exp, written by one workgroup (the values attn_rows reads).
__device__ __forceinline__ void write_fold(const AttnFold& f, uint16_t* __restrict__ attn,
                                           float* __restrict__ lse) {
  for (int vec = threadIdx.x; vec < f.hq * 16; vec += blockDim.x) {   // whole rows of 16 lanes
    float l;
    const uint4 a = fold8(load_fold(f, vec, true), f.scale, l);
    reinterpret_cast<uint4*>(attn)[vec] = a;
    if (lse && (vec & 15) == 0) lse[vec >> 4] = l;
  }
}

}  // namespace lin
}  // namespace qf
