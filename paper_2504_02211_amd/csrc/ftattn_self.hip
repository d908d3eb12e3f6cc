// Instantiations of the fused attention kernel for calls in one launch, whose workgroups encode the key and value tiles
// themselves; a translation unit of its own, so that all of them compile side by side.
#include "ftattn_main.h"

namespace ftattn {

template <int D, bool FT>
static kernel_fn pick_self(bool causal) {
  return causal ? ftattn_main<D, FT, true, false, 0, false, true> : ftattn_main<D, FT, false, false, 0, false, true>;
}

kernel_fn select_self(int D, bool ft, bool causal) {
  if (D == 128) return ft ? pick_self<128, true>(causal) : pick_self<128, false>(causal);
  if (D == 64) return ft ? pick_self<64, true>(causal) : pick_self<64, false>(causal);
  return nullptr;
}

}  // namespace ftattn
