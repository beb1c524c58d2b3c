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

template <int PRO, int T, int W, int RB, bool GLU>
void launch_tiles(const LinearParams& p, int rows, hipStream_t stream) {
  hipLaunchKernelGGL((linear_tiles_kernel<PRO, T, W, RB, GLU>), dim3((p.N + rows - 1) / rows),
                     dim3(64 * W), 0, stream, p.x, p.w, p.gain, p.residual, p.out_a, p.out_b, p.M,
                     p.N, p.K, p.n_split, p.eps, rows);
}

// The output rows of a workgroup (even) for products of n and m outputs in one launch, and the
// workgroups per compute unit that makes: as few as keep a workgroup within 40 rows (5 tiles), all of
// them of one size.
struct TileShare {
  int per_unit, rows;
};
TileShare tile_share(int64_t n, int64_t m) {
  constexpr int64_t kUnits = 256, kMost = 40;
  const int64_t per_unit = (n + m + kUnits * kMost - 1) / (kUnits * kMost);
  int64_t rows = ((n + m + kUnits * per_unit - 1) / (kUnits * per_unit) + 1) / 2 * 2;
  while (rows < kMost && (n + rows - 1) / rows + (m + rows - 1) / rows > kUnits * per_unit) rows += 2;
  return {(int)per_unit, (int)rows};
}

template <int PRO, bool GLU>
void launch_tiles_pro(const LinearParams& p, hipStream_t stream) {
  const auto [per_unit, rows] = tile_share(p.N, 0);
  const int t = (rows + lin::kTileRows - 1) / lin::kTileRows;
  // Rounds in flight: as many as 128 registers hold (the RMS prologue also keeps the gains and the
  // halves).
  constexpr bool RMS = PRO == kProRmsNorm;
  if (per_unit == 1) {
    switch (t) {
      case 1: launch_tiles<PRO, 1, 16, RMS ? 3 : 4, GLU>(p, rows, stream); break;
      case 2: launch_tiles<PRO, 2, 16, RMS ? 2 : 3, GLU>(p, rows, stream); break;
      case 3: launch_tiles<PRO, 3, 16, 2, GLU>(p, rows, stream); break;
      case 4: launch_tiles<PRO, 4, 16, RMS ? 1 : 2, GLU>(p, rows, stream); break;
      default: launch_tiles<PRO, 5, 16, 1, GLU>(p, rows, stream); break;
    }
  } else {
    switch (t) {
      case 3: launch_tiles<PRO, 3, 8, 1, GLU>(p, rows, stream); break;
      case 4: launch_tiles<PRO, 4, 8, 1, GLU>(p, rows, stream); break;
      default: launch_tiles<PRO, 5, 8, 1, GLU>(p, rows, stream); break;
    }
  }
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

template <int T, int W, int RB>
void launch_pair_tiles(const LinearParams& a, const LinearParams& b, int rows, hipStream_t stream) {
  const int blocks_a = (a.N + rows - 1) / rows;
  hipLaunchKernelGGL((linear_pair_tiles_kernel<T, W, RB>), dim3(blocks_a + (b.N + rows - 1) / rows),
                     dim3(64 * W), 0, stream, a, b, blocks_a, rows);
}

template <int PRO>
void launch_rows(const LinearParams& p, hipStream_t stream) {
  switch (lin::rows_bucket(p.M)) {
    case 1: launch_pro<PRO, 1>(p, stream); break;
    case 2: launch_pro<PRO, 2>(p, stream); break;
    case 4: launch_pro<PRO, 4>(p, stream); break;
    default: launch_pro<PRO, 8>(p, stream); break;
  }
}

}  // namespace

hipError_t launch_linear(const LinearParams& p, hipStream_t stream) {
  if (p.M == 0 || p.N == 0) return hipSuccess;
  if (lin::takes_tiles(p)) {
    if (p.prologue == kProRmsNorm)
      p.glu ? launch_tiles_pro<kProRmsNorm, true>(p, stream) : launch_tiles_pro<kProRmsNorm, false>(p, stream);
    else
      p.glu ? launch_tiles_pro<kProNone, true>(p, stream) : launch_tiles_pro<kProNone, false>(p, stream);
    return hipGetLastError();
  }
  if (p.prologue == kProRmsNorm)
    launch_rows<kProRmsNorm>(p, stream);
  else if (p.prologue == kProSwiglu)
    launch_rows<kProSwiglu>(p, stream);
  else
    launch_rows<kProNone>(p, stream);
  return hipGetLastError();
}

// A projection and the gated product of the same rows behind RMS prologues (W_q and W_gate|W_up of a
// block) share a launch; any other two products are launched one after the other.
hipError_t launch_linear_pair(const LinearParams& a, const LinearParams& b, hipStream_t stream) {
  const bool pair = a.M > 0 && a.M == b.M && a.K == b.K && a.prologue == kProRmsNorm &&
                    b.prologue == kProRmsNorm && !a.glu && b.glu &&
                    lin::takes_tiles(a) == lin::takes_tiles(b) && (a.M == 1 || lin::takes_tiles(a)) &&
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
  const auto [per_unit, rows] = tile_share(a.N, b.N);
  const int t = (rows + lin::kTileRows - 1) / lin::kTileRows;
  if (per_unit == 1) {
    switch (t) {
      case 1: launch_pair_tiles<1, 16, 3>(a, b, rows, stream); break;
      case 2: launch_pair_tiles<2, 16, 2>(a, b, rows, stream); break;
      case 3: launch_pair_tiles<3, 16, 2>(a, b, rows, stream); break;
      case 4: launch_pair_tiles<4, 16, 1>(a, b, rows, stream); break;
      default: launch_pair_tiles<5, 16, 1>(a, b, rows, stream); break;
    }
  } else {
    switch (t) {
      case 3: launch_pair_tiles<3, 8, 1>(a, b, rows, stream); break;
      case 4: launch_pair_tiles<4, 8, 1>(a, b, rows, stream); break;
      default: launch_pair_tiles<5, 8, 1>(a, b, rows, stream); break;
    }
  }
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
