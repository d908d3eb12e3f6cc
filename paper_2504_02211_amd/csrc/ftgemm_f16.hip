// Instantiations of the fault-tolerant GEMM kernel for fp16 operands, one translation unit per type so that
// they compile side by side.
#include "ftgemm_main.h"

namespace ftgemm {
gemm_fn tile_kernel_f16(int tile, bool ft, bool inject) { return tile_kernel_of<false>(tile, ft, inject); }
gemm_fn finish_kernel_f16(bool ft) { return ft ? ftgemm_finish<true, false> : ftgemm_finish<false, false>; }
}  // namespace ftgemm
