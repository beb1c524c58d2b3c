// The fused products of linear_body.h for several input rows, on the matrix cores.
//
// With more than a couple of input rows the vector path's cost is instructions, not bytes: every
// wavefront unpacks and normalises every input row again for each output row, and spends a
// fused multiply-add per weight and input row.  Here one v_mfma_f32_16x16x32_bf16 takes 512 weights
// for all input rows at once, so the product is a weight stream again.  Measured with 8 input rows
// (vector path -> here, us a launch in a HIP graph, weights from HBM): 6,144 x 1,024 with the RMS
// prologue 12.0 -> 5.2, 2,048 x 1,024 8.2 -> 4.0, 1,024 x 3,072 7.4 -> 4.7, 19,456 x 2,560 39.0 -> 21.1
// (4.7 TB/s), 2,560 x 9,728 29.1 -> 12.9.  With 2 rows the tiles are 1 to 46% faster but for products of
// a few hundred outputs and inputs (64 x 512: 2.1 -> 2.4); with one row the vector path is faster where
// launches are short (300 x 1,000: 2.6 against 3.2, 6,144 x 1,024 4.8 against 5.1, 2,048 x 1,024 3.5
// against 3.6) and within 8% either way elsewhere.
//
// Tiles.  The 16 rows of the A operand are 8 output rows times 2 slices of K, and the 16 columns of
// the B operand 8 input rows times the same slices; the product's diagonal blocks (equal slices) are
// the sums wanted, the others are not read.  So a tile has 8 output rows, not 16, and one load
// instruction reads 128 contiguous bytes (a cache line) of each.  A workgroup takes any number of
// output rows up to 8 T: up to 10,240 outputs the launch deals them evenly over the compute units, one
// workgroup each, because all of them stream at once and the one with the most rows ends last (2,560 x
// 9,728: 320 workgroups of 8 rows, two on a quarter of the units, took 20.3 us; 256 of 10 rows 13.2).
//
// Sums.  K is dealt in blocks of 64 inputs to 16 slots, a round of 1,024 inputs after the other; each
// slot's sum is one chain of matrix instructions, and the slots' sums meet in one fixed tree.  A
// workgroup of W = 4 or 8 wavefronts keeps 16 / W slots in each: T, W, the rows of a workgroup and the rounds
// in flight change nothing in any sum, so every launch of a product gives the same bits.
//
// With the RMS prologue the factor x * gain has up to 16 significant bits, so it is fed exactly as two
// bf16 halves (its upper 8 bits and the rest); r = 1 / sqrt(mean x^2 + eps) is applied at the end, as
// on the vector path.  An infinite factor's lower half is inf - inf, and an infinite weight meets lower
// halves that are 0: such an output may come out NaN where the exact sum is infinite, so with this
// prologue a NaN is summed again without halves.  Not where the row's sum of squares is not finite (an
// input row that holds a NaN or an infinity, as every row after a request whose cache was refused):
// r is then 0 or NaN and the output NaN whatever the sum was, and one such row of eight made 19,456 x
// 2,560 outputs take 294 us instead of 21 (21 now).  What is left are infinite weights and gains.
#pragma once

#include <type_traits>

#include "linear_body.h"

namespace qf {
namespace lin {

typedef __attribute__((ext_vector_type(8))) __bf16 mf_bf16x8;
typedef __attribute__((ext_vector_type(4))) float mf_f32x4;

// The upper 16 bits of a float as a float, and those of 8 floats as packed bf16.
__device__ __forceinline__ float hi_half(float p) {
  return __uint_as_float(__float_as_uint(p) & 0xffff0000u);
}
__device__ __forceinline__ uint4 pack_upper(const float* p) {
  auto pair = [&](int j) {
    return __builtin_amdgcn_perm(__float_as_uint(p[j + 1]), __float_as_uint(p[j]), 0x07060302u);
  };
  return make_uint4(pair(0), pair(2), pair(4), pair(6));
}

constexpr int kTileRows = 8;    // output rows of a tile, and most input rows
constexpr int kSlots = 16;
constexpr int kBlockK = 64;     // inputs of one step of a wavefront
constexpr int kRoundK = kSlots * kBlockK;

template <int T, int W>
struct TileLds {
  float sum[W][2][T * kTileRows][kTileRows + 1];   // [wavefront][slice][output row][input row]
  float ss[W][2][kTileRows];                       // sums of squares (RMS prologue)
};

// One output behind the RMS prologue summed by one thread without halves (and without the final factor).
__device__ __attribute__((noinline)) inline float plain_sum(const uint16_t* x, const uint16_t* w,
                                                            const uint16_t* gain, int32_t K) {
  float y = 0.0f;
  for (int k = 0; k < K; ++k) y = fmaf(lo(w[k]), lo(x[k]) * lo(gain[k]), y);
  return y;
}

// Output rows n0 .. n0 + rows - 1 (rows <= 8 T, even with GLU) of out = W . P(x) (+ residual),
// M <= 8 input rows, by a workgroup of W (4 or 8) wavefronts with the loads of RB rounds in
// flight.  lds: one per workgroup.
template <int PRO, int T, int W, int RB, bool GLU>
__device__ __forceinline__ void linear_tiles(
    const uint16_t* __restrict__ x, const uint16_t* __restrict__ w,
    const uint16_t* __restrict__ gain, const uint16_t* __restrict__ residual,
    uint16_t* __restrict__ out_a, uint16_t* __restrict__ out_b, int32_t M, int32_t N, int32_t K,
    int32_t n_split, float eps, const int32_t n0, const int32_t rows, TileLds<T, W>& lds) {
  static_assert(PRO == kProNone || PRO == kProRmsNorm, "the SwiGLU input has 24 significant bits");
  static_assert(W == 4 || W == 8, "the tree of the slots");
  constexpr int R = kTileRows;
  constexpr bool RMS = PRO == kProRmsNorm;
  constexpr int A = kSlots / W;                  // slots (steps per round) of a wavefront
  constexpr int kOut = 0x7fffffff;               // an offset past every resource: the load gives 0
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row = lane & (R - 1);                // output row of the A operand, input row of the B one
  const int kk = ((lane & 8) / 2 + (lane >> 4)) * 8;   // this lane's 8 inputs of a block
  if (n0 >= N) return;

  // One resource over the workgroup's weight rows, the input rows and the gains: rows past the
  // workgroup's or M, and inputs past K, read as zeros and cost no traffic.
  const int n_rows = min(N - n0, rows);
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(w + (size_t)n0 * K), (short)0, n_rows * K * 2, 0x00020000);
  const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(x), (short)0, M * K * 2, 0x00020000);
  const __amdgpu_buffer_rsrc_t rg = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(RMS ? gain : w), (short)0, RMS ? K * 2 : 0, 0x00020000);

  // Thread o < M n_rows finishes output (input row o / n_rows, output row o % n_rows), with GLU a
  // pair of output rows; its residual comes ahead of the weights.
  const int per = GLU ? n_rows / 2 : n_rows;
  const int om = (int)threadIdx.x / per, on = (GLU ? 2 : 1) * ((int)threadIdx.x % per);
  uint16_t res = 0;
  if constexpr (!GLU)
    if (residual != nullptr && om < M) res = residual[(size_t)om * N + n0 + on];

  struct Step {
    uint4 w[T], x, g;
  };
  // Block a of round j of this wavefront: inputs k .. k + 7 of this lane.
  auto issue = [&](Step& st, int j, int a) {
    const int k = ((j * A + a) * W + wave) * kBlockK + kk;
    const bool in = k < K;
    const int off = (row * K + k) * 2;
#pragma unroll
    for (int t = 0; t < T; ++t)
      st.w[t] = __builtin_bit_cast(
          uint4, __builtin_amdgcn_raw_buffer_load_b128(rw, in ? off + t * R * K * 2 : kOut, 0, 2));
    st.x = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rx, in ? off : kOut, 0, 0));
    if constexpr (RMS)
      st.g = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rg, in ? k * 2 : kOut, 0, 0));
    // Loads return in order and are waited for by count: the steps keep their order, so that a
    // step's wait leaves the steps after it in flight.
    __builtin_amdgcn_sched_barrier(0);
  };

  mf_f32x4 acc[A][T];
  float ss[A];
#pragma unroll
  for (int a = 0; a < A; ++a) {
    ss[a] = 0.0f;
#pragma unroll
    for (int t = 0; t < T; ++t) acc[a][t] = mf_f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  }
  auto compute = [&](const Step& st, int a) {
    auto mac = [&](const uint4& b) {
#pragma unroll
      for (int t = 0; t < T; ++t)
        acc[a][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            __builtin_bit_cast(mf_bf16x8, st.w[t]), __builtin_bit_cast(mf_bf16x8, b), acc[a][t], 0, 0, 0);
    };
    if constexpr (RMS) {
      float xf[8], gf[8], p[8], low[8];
      unpack8(st.x, xf);
      unpack8(st.g, gf);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        ss[a] = fmaf(xf[j], xf[j], ss[a]);
        p[j] = xf[j] * gf[j];
        low[j] = p[j] - hi_half(p[j]);                    // exact, at most 8 significant bits
      }
      mac(pack_upper(low));
      mac(pack_upper(p));
    } else {
      mac(st.x);
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  // A last, partial round comes first, then the whole ones in order, RB in flight.  A load past K
  // moves no data but takes the compute unit's address path 16 cycles like any other, so none is
  // issued to keep the loop simple: the last RB rounds are computed after it, by the copy of the
  // code that starts at the right buffer.  (With such loads a product of 6,144 x 1,024 took 9.0 us for
  // 8 rows instead of 6.1, then with 16 wavefronts a workgroup.)
  const int whole = K / kRoundK;
  const int rounds = whole + (whole * kRoundK < K ? 1 : 0);
  auto round_at = [&](int i) { return rounds > whole ? (i == 0 ? whole : i - 1) : i; };
  Step buf[RB][A];
  if (rounds < RB) {   // a short K: everything is in flight at once
#pragma unroll
    for (int b = 0; b < RB - 1; ++b)
      if (b < rounds)
#pragma unroll
        for (int a = 0; a < A; ++a) issue(buf[b][a], round_at(b), a);
#pragma unroll
    for (int b = 0; b < RB - 1; ++b)
      if (b < rounds)
#pragma unroll
        for (int a = 0; a < A; ++a) compute(buf[b][a], a);
  } else {
#pragma unroll
    for (int b = 0; b < RB; ++b)
#pragma unroll
      for (int a = 0; a < A; ++a) issue(buf[b][a], round_at(b), a);
    int i = RB;
    for (; i + RB <= rounds; i += RB)
#pragma unroll
      for (int b = 0; b < RB; ++b)
#pragma unroll
        for (int a = 0; a < A; ++a) {
          compute(buf[b][a], a);
          issue(buf[b][a], round_at(i + b), a);
        }
    auto drain = [&](auto left) {
      constexpr int kLeft = decltype(left)::value;
#pragma unroll
      for (int b = 0; b < kLeft; ++b)
#pragma unroll
        for (int a = 0; a < A; ++a) {
          compute(buf[b][a], a);
          issue(buf[b][a], round_at(i + b), a);
        }
#pragma unroll
      for (int b = 0; b < RB; ++b)
#pragma unroll
        for (int a = 0; a < A; ++a) compute(buf[(kLeft + b) % RB][a], a);
    };
    const int left = rounds - i;
    if (RB < 2 || left == 0) drain(std::integral_constant<int, 0>{});
    else if (RB < 3 || left == 1) drain(std::integral_constant<int, RB < 2 ? 0 : 1>{});
    else if (RB < 4 || left == 2) drain(std::integral_constant<int, RB < 3 ? 0 : 2>{});
    else drain(std::integral_constant<int, RB < 4 ? 0 : 3>{});
    static_assert(RB <= 4, "one copy per remainder");
  }

  // The tree: slots s and s + 8, then s and s + 4, then the slots and slices in order.  Wavefront s of
  // W holds the slots s, s + W, ...
  if constexpr (RMS) {
#pragma unroll
    for (int a = 0; a < A; ++a) {
      ss[a] += __shfl_xor(ss[a], 16);
      ss[a] += __shfl_xor(ss[a], 32);
    }
  }
#pragma unroll
  for (int d = A / 2; d > 0; d /= 2)
#pragma unroll
    for (int a = 0; a < d; ++a) {
      ss[a] += ss[a + d];
#pragma unroll
      for (int t = 0; t < T; ++t) acc[a][t] += acc[a + d][t];
    }

  // Lane (quarter q, column c) holds rows 4q .. 4q + 3 of the 16 x 16 result: slice q / 2 of output
  // rows 4 (q % 2) .. + 3, against slice c / 8 of input row c % 8; equal slices are stored.
  const int q = lane >> 4, c = lane & 15;
  if (RMS && q == 0) lds.ss[wave][c / R][c % R] = ss[0];
  if (q / 2 == c / R) {
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        lds.sum[wave][c / R][t * R + 4 * (q % 2) + i][c % R] = acc[0][t][i];
  }
  __syncthreads();
  if (om >= M) return;

  // Slot v's share of a sum over the workgroup's wavefronts.
  auto over_waves = [&](int v, auto&& at) {
    if constexpr (W == 4) return at(v);
    else return at(v) + at(v + 4);
  };
  float scale = 1.0f;
  if constexpr (RMS) {
    float t = 0.0f;
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int s = 0; s < 2; ++s) t += over_waves(v, [&](int i) { return lds.ss[i][s][om]; });
    scale = 1.0f / sqrtf(t / (float)K + eps);
  }
  auto value = [&](int n) {
    float y = 0.0f;
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int s = 0; s < 2; ++s) y += over_waves(v, [&](int i) { return lds.sum[i][s][n][om]; });
    if constexpr (RMS)
      if (__builtin_isnan(y) && scale > 0.0f)   // a finite sum of squares
        y = plain_sum(x + (size_t)om * K, w + (size_t)(n0 + n) * K, gain, K);
    return y;
  };
  const int n = n0 + on;
  if constexpr (GLU) {
    const float g = value(on) * scale, v = value(on + 1) * scale;
    out_a[(size_t)om * (N / 2) + n / 2] = (uint16_t)bf16_rne(silu(g) * v);
  } else {
    float y = value(on) * scale;
    if (residual != nullptr) y += lo(res);
    const uint16_t b = (uint16_t)bf16_rne(y);
    if (n < n_split)
      out_a[(size_t)om * n_split + n] = b;
    else
      out_b[(size_t)om * (N - n_split) + (n - n_split)] = b;
  }
}

// Whether a product takes the tiles: more than kVectorRows rows (below, the vector path), a prologue that
// two bf16 halves carry exactly, and 32-bit offsets (40 rows of K weights).
constexpr int kVectorRows = 1;
inline bool takes_tiles(const LinearParams& p) {
  return p.M > kVectorRows && p.prologue != kProSwiglu && p.K <= (1 << 24);
}
// Whether its rows are taken one by one, on the vector path: what is left of several rows without SwiGLU.
inline bool takes_single_rows(const LinearParams& p) {
  return p.M > kVectorRows && p.prologue != kProSwiglu && !takes_tiles(p);
}

}  // namespace lin
}  // namespace qf
