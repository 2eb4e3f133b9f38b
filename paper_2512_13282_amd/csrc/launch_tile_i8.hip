// launch_tile_i8.hip -- the register-staged instances for int8 inputs.
#include "launch_tile.h"

namespace gemm {
template hipError_t launch_tile_family<DT_I8>(int32_t, const KernelArgs &, int64_t, hipStream_t);
}  // namespace gemm
