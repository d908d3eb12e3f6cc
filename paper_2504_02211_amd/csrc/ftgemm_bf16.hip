// Instantiations of the fault-tolerant GEMM kernel for bf16 operands, one translation unit per type so that
// they compile side by side.
#include "ftgemm_main.h"

namespace ftgemm {
gemm_fn tile_kernel_bf16(int tile, bool ft, bool inject) { return tile_kernel_of<true>(tile, ft, inject); }
gemm_fn finish_kernel_bf16(bool ft) { return ft ? ftgemm_finish<true, true> : ftgemm_finish<false, true>; }
}  // namespace ftgemm
