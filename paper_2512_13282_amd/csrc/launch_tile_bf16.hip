// launch_tile_bf16.hip -- the register-staged instances for bf16 inputs.
#include "launch_tile.h"

namespace gemm {
template hipError_t launch_tile_family<DT_BF16>(int32_t, const KernelArgs &, int64_t, hipStream_t);
}  // namespace gemm
