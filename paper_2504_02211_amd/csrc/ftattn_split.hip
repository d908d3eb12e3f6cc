// Instantiations of the fused attention kernel for calls whose row tiles are split by their keys, and of the kernel that
// puts the shares together, kept apart from the main translation unit so that they compile side by side.
#include "ftattn_main.h"

namespace ftattn {

template <int D, bool FT>
static kernel_fn pick_split(bool causal) {
  return causal ? ftattn_main<D, FT, true, false, 0, true> : ftattn_main<D, FT, false, false, 0, true>;
}

template <int D, bool FT>
static kernel_fn pick_finish(bool causal) { return causal ? ftattn_finish<D, FT, true> : ftattn_finish<D, FT, false>; }

kernel_fn select_split(int D, bool ft, bool causal) {
  if (D == 128) return ft ? pick_split<128, true>(causal) : pick_split<128, false>(causal);
  if (D == 64) return ft ? pick_split<64, true>(causal) : pick_split<64, false>(causal);
  return nullptr;
}

kernel_fn select_finish(int D, bool ft, bool causal) {
  if (D == 128) return ft ? pick_finish<128, true>(causal) : pick_finish<128, false>(causal);
  if (D == 64) return ft ? pick_finish<64, true>(causal) : pick_finish<64, false>(causal);
  return nullptr;
}

}  // namespace ftattn
