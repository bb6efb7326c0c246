// One translation unit's share of the chain kernels (fft_chain.h): the including
// file defines CGH_CHAIN_PART, and the kernels of the chain lengths whose index
// is that part modulo kChainParts are compiled here (they are split only so
// that they compile in parallel).
#include <algorithm>
#include <array>
#include <utility>

#include "fft_chain.h"

namespace cgh {
namespace {

struct MP {
  int M, P;
};

template <bool (*BUILT)(int, int)>
constexpr int count_lengths() {
  int n = 0;
  for (int P : {4, 2})
    for (int M = kMinChain; M <= kMaxFft / P; ++M) n += BUILT(M, P);
  return n;
}

// the lengths of this part
template <bool (*BUILT)(int, int)>
constexpr auto part_lengths() {
  constexpr int all = count_lengths<BUILT>();
  std::array<MP, (all + kChainParts - 1) / kChainParts> r{};
  int n = 0;
  for (int P : {4, 2})
    for (int M = kMinChain; M <= kMaxFft / P; ++M)
      if (BUILT(M, P)) {
        if (n % kChainParts == CGH_CHAIN_PART) r[n / kChainParts] = MP{M, P};
        ++n;
      }
  return r;
}

constexpr auto kRowLengths = part_lengths<row_chain>();
constexpr auto kColLengths = part_lengths<col_chain>();

template <int M, int P>
void launch_row(const RowArgs &a, hipStream_t s) {
  static_assert(row_plan(M, P, row_threads(M, P)).n > 0, "no row plan");
  // pipelined rows: as many workgroups as run at once, each taking every grid-th row
  // (a multiple of 16 workgroups, so that a pair of rows stays on one XCD)
  const int most = row_pipe(M, P) ? std::max(16, a.num_cu * row_groups(M, P) / 16 * 16) : a.rows;
  const dim3 grid(a.rows), block(row_threads(M, P));
  if (a.pass == 0)
    hipLaunchKernelGGL((k_row_fwd_q<M, P>), dim3(std::min(a.rows, most)), block, 0, s, a.field, a.H, a.W, a.rows, a.twf_x,
                       a.S);
  else if (a.pass == 1)
    hipLaunchKernelGGL((k_row_inv_q<M, P>), dim3(a.rows + a.sums.blocks), block, 0, s, a.S, a.H,
                       a.W, a.rows, a.twf_x, a.out, a.sums);
  else
    hipLaunchKernelGGL((k_row_loss_q<M, P>), grid, block, 0, s, a.S, a.H, a.W, a.rows, a.twf_x,
                       a.target, a.grad_I, a.mask, a.mcg, a.intensity, a.u_out, a.loss_part,
                       a.gscale, a.make_grad);
}

template <int M, int P>
void launch_col(const ColArgs &a, hipStream_t s) {
  static_assert(col_plan(M).r2 > 0, "no column plan");
  const int pairs = a.C * ((a.Wt + 1) / 2);
  const dim3 grid((pairs + 7) / 8 * 16 * P), block(col_threads(col_plan(M)));
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, block, 0, s, a.io, a.Hq, a.H, a.Wp, a.Wt, a.C, a.twf_y);
  };
  if constexpr (planes_chain(M, P)) {
    if (a.io.planes > 1) {
      a.conj_h ? go(k_col_wave<M, P, true, true>) : go(k_col_wave<M, P, false, true>);
      return;
    }
  }
  a.conj_h ? go(k_col_wave<M, P, true, false>) : go(k_col_wave<M, P, false, false>);
}

template <size_t I>
bool try_row(int M, int P, const RowArgs &a, hipStream_t s) {
  constexpr MP mp = kRowLengths[I];
  if constexpr (mp.M > 0) {
    if (mp.M != M || mp.P != P) return false;
    launch_row<mp.M, mp.P>(a, s);
    return true;
  }
  return false;
}
template <size_t I>
bool try_col(int M, int P, const ColArgs &a, hipStream_t s) {
  constexpr MP mp = kColLengths[I];
  if constexpr (mp.M > 0) {
    if (mp.M != M || mp.P != P) return false;
    launch_col<mp.M, mp.P>(a, s);
    return true;
  }
  return false;
}

template <size_t... I>
bool any_row(std::index_sequence<I...>, int M, int P, const RowArgs &a, hipStream_t s) {
  return (try_row<I>(M, P, a, s) || ...);
}
template <size_t... I>
bool any_col(std::index_sequence<I...>, int M, int P, const ColArgs &a, hipStream_t s) {
  return (try_col<I>(M, P, a, s) || ...);
}

}  // namespace

#define CGH_CAT2(a, b) a##b
#define CGH_CAT(a, b) CGH_CAT2(a, b)
bool CGH_CAT(row_chain_part_, CGH_CHAIN_PART)(int M, int P, const RowArgs &a, hipStream_t s) {
  return any_row(std::make_index_sequence<kRowLengths.size()>{}, M, P, a, s);
}
bool CGH_CAT(col_chain_part_, CGH_CHAIN_PART)(int M, int P, const ColArgs &a, hipStream_t s) {
  return any_col(std::make_index_sequence<kColLengths.size()>{}, M, P, a, s);
}

}  // namespace cgh
