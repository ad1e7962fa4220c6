// Router scores and the REFLEX counts in one launch (Sections 3.2, 4.2, 4.3).  The
// two are independent, so the first B workgroups compute the counts of one sequence
// each while the rest compute split-K partial score tiles (router_split_tile); the
// counts' long dependent chain then overlaps the score tiles instead of following
// them.  The route kernel adds the partials of each score.
#include "budget_impl.h"
#include "router_impl.h"

namespace rfx {
namespace {

__global__ __launch_bounds__(RS_THREADS) void front_kernel(
    const uint16_t* __restrict__ h, const float* __restrict__ w, float* __restrict__ parts, int T,
    int d, int E, int gy, int n_slices, BudgetArgs a, BudgetConsts p,
    int32_t* __restrict__ zero_word) {
  __shared__ BudgetLds lds;
  const int b = blockIdx.x;
  if (zero_word != nullptr && b == 0 && threadIdx.x == 0) *zero_word = 0;
  if (b < a.B) {
    budget_sequence<RS_THREADS>(lds, b, a.block_idx, a.masked, a.hist_len, a.c1, a.c2, a.seq_offsets,
                                a.active_block, T, p, a.k_out, nullptr, nullptr);
    return;
  }
  // score tiles: K slice fastest, then expert block, then token block
  const int r = b - a.B;
  const int ks = r % n_slices, rest = r / n_slices;
  router_split_tile(rest / gy, rest % gy, ks, h, w, parts, T, d, E);
}

}  // namespace

// The 32-token x 64-expert x 256-column tiles suit few scores: every tile is a workgroup, and
// its 80 KB pass through one CU.  From 2^17 scores (T = 2048 at E = 64, 512 at E = 256) the
// 128 x 64 tiles of launch_router, which re-read a quarter of the bytes, are faster
// (stage times, E = 256: T = 512 / 1024 / 2048 / 3000 19.6 / 25.9 / 43.0 / 54.7 us here and
// 15.3 / 20.7 / 22.7 / 26.1 there; E = 64: T = 1024 / 2048 / 3000 17.8 / 21.2 / 25.1 and 16.9 /
// 16.8 / 18.3; d = 2048), given that their K range splits into enough slices (router_slices).
bool front_fits(int T, int d, int E) {
  return T < 4096 && d % RS_KS == 0 && router_slices(T, d, E) == 1;
}

int front_slices(int d) { return d / RS_KS; }

int launch_front(const uint16_t* h, const float* w, float* parts, int T, int d, int E,
                 const BudgetArgs& budget, hipStream_t s, int32_t* zero_word) {
  const int gx = (T + RS_TM - 1) / RS_TM, gy = (E + RS_TE - 1) / RS_TE, ns = front_slices(d);
  hipLaunchKernelGGL(front_kernel, dim3(budget.B + gx * gy * ns), dim3(RS_THREADS), 0, s, h, w, parts,
                     T, d, E, gy, ns, budget, budget_consts(budget.params), zero_word);
  return launch_status();
}

}  // namespace rfx
