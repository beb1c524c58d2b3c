// Standalone launch of the fused decode-block products (bodies in linear_body.h and linear_mfma.h).
#include "attn_linear.h"
#include "linear_mfma.h"

namespace qf {
namespace {

template <int PRO, int MB, int U, int R, bool GLU>
__global__ void __launch_bounds__(lin::kThreads)
linear_kernel(const uint16_t* __restrict__ x, const uint16_t* __restrict__ w,
              const uint16_t* __restrict__ gain, const uint16_t* __restrict__ residual,
              uint16_t* __restrict__ out_a, uint16_t* __restrict__ out_b, int32_t M, int32_t N,
              int32_t K, int32_t n_split, float eps) {
  lin::linear_rows<PRO, MB, U, R, GLU>(x, w, gain, residual, out_a, out_b, M, N, K, n_split,
                                       eps, blockIdx.x);
}

template <int PRO, int T, int W, int RB, bool GLU>
__global__ void __launch_bounds__(64 * W)
linear_tiles_kernel(const uint16_t* __restrict__ x, const uint16_t* __restrict__ w,
                    const uint16_t* __restrict__ gain, const uint16_t* __restrict__ residual,
                    uint16_t* __restrict__ out_a, uint16_t* __restrict__ out_b, int32_t M,
                    int32_t N, int32_t K, int32_t n_split, float eps, int32_t rows) {
  __shared__ lin::TileLds<T, W> lds;
  lin::linear_tiles<PRO, T, W, RB, GLU>(x, w, gain, residual, out_a, out_b, M, N, K, n_split, eps,
                                        (int)blockIdx.x * rows, rows, lds);
}

// The output rows of a workgroup (even) for products of n and m outputs in one launch.  Up to 40 rows (5
// tiles) for each of the 256 compute units, one workgroup a unit takes an even share; above, as few
// workgroups a unit as keep one within `most` rows, all of one size.  `most` is 40 where five tiles leave
// room for two workgroups on a unit (128 registers at 8 wavefronts) and 32 behind the RMS prologue
// without GLU, where they take 143 (two rows of input, 60,000 x 1,024: 27.3 us with 40 rows, 24.0 with 32;
// eight rows, 151,936 x 1,024: 73.3 and 54.8).  From three workgroups a unit on, they run in rounds.
constexpr int kTileUnits = 256, kTileMost = 40;
int tile_rows(int64_t n, int64_t m, int most) {
  if (n + m <= kTileUnits * kTileMost) most = kTileMost;
  const int64_t per_unit = (n + m + kTileUnits * most - 1) / (kTileUnits * most);
  int64_t rows = ((n + m + kTileUnits * per_unit - 1) / (kTileUnits * per_unit) + 1) / 2 * 2;
  while (rows < most && (n + rows - 1) / rows + (m + rows - 1) / rows > kTileUnits * per_unit) rows += 2;
  return (int)rows;
}
constexpr int tile_most(int prologue, bool glu) { return prologue == kProRmsNorm && !glu ? 32 : kTileMost; }

// Calls launch(T, W, RB) for workgroups of `rows` output rows, RB rounds of K in flight: 8 wavefronts,
// without a prologue 4 for one tile (each holds more of the slots: fewer wavefronts to start, and less to
// add at the end).  With few tiles a workgroup is alone on its unit and has more rounds in flight; from
// three tiles on, the registers of one round let two workgroups share a unit.
// Sixteen wavefronts kept one workgroup a unit at 128 registers (with three rounds in flight behind the RMS
// prologue 3 of them in memory), us: 64 x 512 with two rows of input 2.54 -> 2.43, 1,024 x 3,072 4.29 -> 3.95,
// 4,096 x 2,560 (RMS) 7.04 -> 6.51, 6,144 x 1,024 (RMS, GLU) 5.60 -> 5.16, 9,728 x 2,560 (RMS, GLU) 12.9 ->
// 11.5; with eight rows 2.74 -> 2.56, 5.02 -> 4.77, 7.64 -> 7.24, 5.77 -> 5.23, 13.3 -> 11.9.
template <int PRO, class Launch>
void with_tiles(int rows, Launch&& launch) {
  constexpr bool RMS = PRO == kProRmsNorm;
  auto go = [&](auto t, auto w, auto rb) { launch(t, w, rb); };
  constexpr std::integral_constant<int, 1> i1{};
  constexpr std::integral_constant<int, 2> i2{};
  constexpr std::integral_constant<int, 8> w8{};
  switch ((rows + lin::kTileRows - 1) / lin::kTileRows) {
    case 1: go(i1, std::integral_constant<int, RMS ? 8 : 4>{}, i2); break;
    case 2: go(i2, w8, std::integral_constant<int, RMS ? 1 : 3>{}); break;
    case 3: go(std::integral_constant<int, 3>{}, w8, i1); break;
    case 4: go(std::integral_constant<int, 4>{}, w8, i1); break;
    default: go(std::integral_constant<int, 5>{}, w8, i1); break;
  }
}

template <int PRO, bool GLU>
void launch_tiles_pro(const LinearParams& p, hipStream_t stream) {
  const int rows = tile_rows(p.N, 0, tile_most(PRO, GLU));
  with_tiles<PRO>(rows, [&](auto t, auto w, auto rb) {
    constexpr int T = decltype(t)::value, W = decltype(w)::value, RB = decltype(rb)::value;
    hipLaunchKernelGGL((linear_tiles_kernel<PRO, T, W, RB, GLU>), dim3((p.N + rows - 1) / rows),
                       dim3(64 * W), 0, stream, p.x, p.w, p.gain, p.residual, p.out_a, p.out_b, p.M,
                       p.N, p.K, p.n_split, p.eps, rows);
  });
}

// One row per wavefront; two (a gate row and its up row) with the GLU output.
template <int PRO, int MB, int U>
void launch_u(const LinearParams& p, hipStream_t stream) {
  if constexpr (PRO != kProSwiglu) {   // the host rejects a GLU output after a SwiGLU input
    if (p.glu) {
      hipLaunchKernelGGL((linear_kernel<PRO, MB, U, 2, true>), dim3(lin::linear_blocks(p.N, 2)),
                         dim3(lin::kThreads), 0, stream, p.x, p.w, p.gain, p.residual, p.out_a,
                         p.out_b, p.M, p.N, p.K, p.n_split, p.eps);
      return;
    }
  }
  hipLaunchKernelGGL((linear_kernel<PRO, MB, U, 1, false>), dim3(lin::linear_blocks(p.N, 1)),
                     dim3(lin::kThreads), 0, stream, p.x, p.w, p.gain, p.residual, p.out_a,
                     p.out_b, p.M, p.N, p.K, p.n_split, p.eps);
}

template <int PRO, int MB>
void launch_pro(const LinearParams& p, hipStream_t stream) {
  constexpr int cap = (MB <= 1) ? 8 : (MB <= 2) ? 4 : (MB <= 4) ? 2 : 1;
  switch (lin::pick_unroll(p.M, p.K)) {
    case 1: launch_u<PRO, MB, 1>(p, stream); break;
    case 2: launch_u<PRO, MB, (cap >= 2 ? 2 : 1)>(p, stream); break;
    case 3: launch_u<PRO, MB, (cap >= 3 ? 3 : 1)>(p, stream); break;
    case 4: launch_u<PRO, MB, (cap >= 4 ? 4 : 1)>(p, stream); break;
    case 5: launch_u<PRO, MB, (cap >= 5 ? 5 : 1)>(p, stream); break;
    case 6: launch_u<PRO, MB, (cap >= 6 ? 6 : 1)>(p, stream); break;
    case 7: launch_u<PRO, MB, (cap >= 7 ? 7 : 1)>(p, stream); break;
    default: launch_u<PRO, MB, (cap >= 8 ? 8 : 1)>(p, stream); break;
  }
}

// Two products of the same input rows in one launch: the workgroups of the first, then those of the
// second, each doing what it would in its own launch.
template <int U>
__global__ void __launch_bounds__(lin::kThreads)
linear_pair_kernel(const LinearParams a, const LinearParams b, int32_t blocks_a) {
  if ((int)blockIdx.x < blocks_a)
    lin::linear_rows<kProRmsNorm, 1, U, 1, false>(a.x, a.w, a.gain, a.residual, a.out_a, a.out_b, a.M,
                                                  a.N, a.K, a.n_split, a.eps, blockIdx.x);
  else
    lin::linear_rows<kProRmsNorm, 1, U, 2, true>(b.x, b.w, b.gain, b.residual, b.out_a, b.out_b, b.M,
                                                 b.N, b.K, b.n_split, b.eps, blockIdx.x - blocks_a);
}

template <int T, int W, int RB>
__global__ void __launch_bounds__(64 * W)
linear_pair_tiles_kernel(const LinearParams a, const LinearParams b, int32_t blocks_a, int32_t rows) {
  __shared__ lin::TileLds<T, W> lds;
  if ((int)blockIdx.x < blocks_a)
    lin::linear_tiles<kProRmsNorm, T, W, RB, false>(a.x, a.w, a.gain, a.residual, a.out_a, a.out_b,
                                                    a.M, a.N, a.K, a.n_split, a.eps,
                                                    (int)blockIdx.x * rows, rows, lds);
  else
    lin::linear_tiles<kProRmsNorm, T, W, RB, true>(b.x, b.w, b.gain, b.residual, b.out_a, b.out_b, b.M,
                                                   b.N, b.K, b.n_split, b.eps,
                                                   ((int)blockIdx.x - blocks_a) * rows, rows, lds);
}

// The merge of one request's shard slots beside a product of one row behind the RMS prologue: the
// product's workgroups, then one per query head.
template <int U>
__global__ void __launch_bounds__(lin::kThreads)
linear_merge_kernel(const LinearParams a, int32_t blocks_a, const float* __restrict__ in_o,
                    const float* __restrict__ in_lse, float* __restrict__ out_o,
                    float* __restrict__ out_lse, int32_t entries, int32_t hq) {
  if ((int)blockIdx.x < blocks_a)
    lin::linear_rows<kProRmsNorm, 1, U, 1, false>(a.x, a.w, a.gain, a.residual, a.out_a, a.out_b, a.M,
                                                  a.N, a.K, a.n_split, a.eps, blockIdx.x);
  else
    mrg::merge_row<false, false, lin::kRowsPerBlock>(in_o, in_lse, out_o, out_lse, entries, hq, 0,
                                                     (int)blockIdx.x - blocks_a, nullptr, nullptr,
                                                     nullptr, 1, 0.0f);
}

// W . attn of one request: the first workgroup writes the folded attention and appends the current
// token, the others take 4 R output rows each.
template <int U, int R>
__global__ void __launch_bounds__(lin::kThreads)
linear_attn_kernel(const lin::AttnFold f, const LinearParams p, uint16_t* __restrict__ attn,
                   float* __restrict__ lse, const AppendParams a) {
  if (blockIdx.x == 0) {
    lin::write_fold(f, attn, lse);
    app::append_request(a.k, a.v, a.block_table, a.ctx_lens, f.k_cur, f.v_cur, a.status, a.hkv,
                        a.max_pages, a.num_pages, 1, 0);
    return;
  }
  __shared__ uint4 s_x[64 * U];
  lin::attn_rows<U, R>(f, p, blockIdx.x - 1, s_x);
}

template <int U>
void launch_linear_merge_u(const LinearParams& l, const MergeParams& m, hipStream_t stream) {
  const int blocks = lin::linear_blocks(l.N, 1);
  hipLaunchKernelGGL((linear_merge_kernel<U>), dim3(blocks + m.hq), dim3(lin::kThreads), 0, stream, l,
                     blocks, m.in_o, m.in_lse, static_cast<float*>(m.out_o), m.out_lse, m.entries,
                     m.hq);
}

template <int U>
void launch_pair_u(const LinearParams& a, const LinearParams& b, hipStream_t stream) {
  const int blocks_a = lin::linear_blocks(a.N, 1);
  hipLaunchKernelGGL((linear_pair_kernel<U>), dim3(blocks_a + lin::linear_blocks(b.N, 2)),
                     dim3(lin::kThreads), 0, stream, a, b, blocks_a);
}

}  // namespace

hipError_t launch_linear(const LinearParams& p, hipStream_t stream) {
  if (p.M == 0 || p.N == 0) return hipSuccess;
  if (lin::takes_single_rows(p)) {
    for (int m = 0; m < p.M; ++m) {
      LinearParams row = p;
      row.M = 1;
      row.x += (size_t)m * p.K;
      if (p.residual) row.residual += (size_t)m * p.N;
      row.out_a += (size_t)m * (p.glu ? p.N / 2 : p.n_split);
      if (p.out_b) row.out_b += (size_t)m * (p.N - p.n_split);
      const hipError_t e = launch_linear(row, stream);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  if (lin::takes_tiles(p)) {
    if (p.prologue == kProRmsNorm)
      p.glu ? launch_tiles_pro<kProRmsNorm, true>(p, stream) : launch_tiles_pro<kProRmsNorm, false>(p, stream);
    else
      p.glu ? launch_tiles_pro<kProNone, true>(p, stream) : launch_tiles_pro<kProNone, false>(p, stream);
    return hipGetLastError();
  }
  if (p.prologue == kProRmsNorm) launch_pro<kProRmsNorm, 1>(p, stream);
  else if (p.prologue == kProNone) launch_pro<kProNone, 1>(p, stream);
  else switch (lin::rows_bucket(p.M)) {
    case 1: launch_pro<kProSwiglu, 1>(p, stream); break;
    case 2: launch_pro<kProSwiglu, 2>(p, stream); break;
    case 4: launch_pro<kProSwiglu, 4>(p, stream); break;
    default: launch_pro<kProSwiglu, 8>(p, stream); break;
  }
  return hipGetLastError();
}

// A projection and the gated product of the same rows behind RMS prologues (W_q and W_gate|W_up of a
// block) share a launch; any other two products are launched one after the other.
hipError_t launch_linear_pair(const LinearParams& a, const LinearParams& b, hipStream_t stream) {
  const bool pair = a.M > 0 && a.M == b.M && a.K == b.K && a.prologue == kProRmsNorm &&
                    b.prologue == kProRmsNorm && !a.glu && b.glu &&
                    (a.M == 1 || lin::takes_tiles(a)) &&
                    (int64_t)a.N + b.N <= INT32_MAX / 2;
  if (!pair) {
    const hipError_t e = launch_linear(a, stream);
    return e != hipSuccess ? e : launch_linear(b, stream);
  }
  if (!lin::takes_tiles(a)) {
    switch (lin::pick_unroll(1, a.K)) {
      case 1: launch_pair_u<1>(a, b, stream); break;
      case 2: launch_pair_u<2>(a, b, stream); break;
      case 3: launch_pair_u<3>(a, b, stream); break;
      case 4: launch_pair_u<4>(a, b, stream); break;
      case 5: launch_pair_u<5>(a, b, stream); break;
      case 6: launch_pair_u<6>(a, b, stream); break;
      case 7: launch_pair_u<7>(a, b, stream); break;
      default: launch_pair_u<8>(a, b, stream); break;
    }
    return hipGetLastError();
  }
  const int rows = tile_rows(a.N, b.N, tile_most(kProRmsNorm, false));
  const int blocks_a = (a.N + rows - 1) / rows;
  with_tiles<kProRmsNorm>(rows, [&](auto t, auto w, auto rb) {
    constexpr int T = decltype(t)::value, W = decltype(w)::value, RB = decltype(rb)::value;
    hipLaunchKernelGGL((linear_pair_tiles_kernel<T, W, RB>), dim3(blocks_a + (b.N + rows - 1) / rows),
                       dim3(64 * W), 0, stream, a, b, blocks_a, rows);
  });
  return hipGetLastError();
}

// A product and the merge of shard slots into fp32 pairs: one launch for one request and one row behind
// the RMS prologue, else two.
hipError_t launch_linear_merge(const LinearParams& l, const MergeParams& m, hipStream_t stream) {
  if (l.M != 1 || m.rows != 1 || l.prologue != kProRmsNorm || l.glu || l.N > INT32_MAX / 2) {
    const hipError_t e = l.M > 0 ? launch_linear(l, stream) : hipSuccess;
    return e != hipSuccess ? e : launch_merge(m, false, stream);
  }
  switch (lin::pick_unroll(1, l.K)) {
    case 1: launch_linear_merge_u<1>(l, m, stream); break;
    case 2: launch_linear_merge_u<2>(l, m, stream); break;
    case 3: launch_linear_merge_u<3>(l, m, stream); break;
    case 4: launch_linear_merge_u<4>(l, m, stream); break;
    case 5: launch_linear_merge_u<5>(l, m, stream); break;
    case 6: launch_linear_merge_u<6>(l, m, stream); break;
    case 7: launch_linear_merge_u<7>(l, m, stream); break;
    default: launch_linear_merge_u<8>(l, m, stream); break;
  }
  return hipGetLastError();
}

hipError_t launch_linear_attn(const LinearParams& l, const MergeParams& m, const float* merged_lse,
                              const AppendParams& a, hipStream_t stream) {
  const lin::AttnFold f{m.in_o, merged_lse, m.q, m.k_cur, m.v_cur, m.hq, m.hq / m.hkv, m.scale};
  // Every workgroup folds all heads: two rows a wavefront where there are more rows than 8 a compute
  // unit.
  const int rows = l.N > 2048 ? 2 : 1;
  const dim3 grid(1 + lin::linear_blocks(l.N, rows)), block(lin::kThreads);
  uint16_t* attn = static_cast<uint16_t*>(m.out_o);
  auto launch = [&](auto u) {
    constexpr int U = decltype(u)::value;
    if (rows == 1)
      hipLaunchKernelGGL((linear_attn_kernel<U, 1>), grid, block, 0, stream, f, l, attn, m.out_lse, a);
    else
      hipLaunchKernelGGL((linear_attn_kernel<U, 2>), grid, block, 0, stream, f, l, attn, m.out_lse, a);
  };
  const int chunks = (l.K + 511) / 512;   // of 4 heads
  if (chunks <= 1) launch(std::integral_constant<int, 1>{});
  else if (chunks == 2) launch(std::integral_constant<int, 2>{});
  else if (chunks <= 4) launch(std::integral_constant<int, 4>{});
  else launch(std::integral_constant<int, 8>{});
  return hipGetLastError();
}

}  // namespace qf
