// The dispatch's kernels and the tile choice, run on the CPU.
#include "dispatch.hip"

namespace tg {
int gemm_grid() { return 256; }
}  // namespace tg

extern "C" {

// dispatch_one_block_kernel over npairs pairs with a schedule area: block 0
// (routing) sees the mask alive0, block 1 (plan) alive1, as when the mask is
// written between the two.
void one_block(const int32_t* ids, int npairs, int k, const int32_t* ert, int E, int R,
               const uint8_t* alive0, const uint8_t* alive1, int S, int d, int I, int grid,
               int32_t* counts, int32_t* offsets, int32_t* pair_slot, int32_t* perm,
               int32_t* pair_row, int32_t* n_unserved, int32_t* sched) {
  const int sbits = S > 1 ? 32 - __builtin_clz((unsigned)(S - 1)) : 0;
  for (int b = 0; b < 2; ++b)
    hip_host::run_block(b, 2, tg::kOneBlock, [&] {
      tg::dispatch_one_block_kernel<false>(ids, npairs, k, ert, E, R, b ? alive1 : alive0, S, sbits,
                                           nullptr, nullptr, pair_slot, counts, offsets, perm,
                                           pair_row, n_unserved, nullptr, sched,
                                           tg::GemmDims{d, I, grid});
    });
}

// The tile shape of a gate/up (swiglu) or down launch over the given rows.
int choose(int swiglu, const int32_t* rows, int S, int grid, int K, int cols) {
  int shape = -1;
  hip_host::run_block(0, 1, tg::kWave, [&] {
    const tg::Census cs = tg::census(S, [&](int s) { return rows[s]; });
    const int c = swiglu ? tg::choose_shape<true, false>(cs, grid, K, cols)
                         : tg::choose_shape<false, true>(cs, grid, K, cols);
    if (tg::lane_id() == 0) shape = c;
  });
  return shape;
}

}  // extern "C"
