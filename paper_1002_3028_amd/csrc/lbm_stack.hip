// lbm_stack.hip -- instances of the stacked-row kernel.
#include "lbm_stack.hpp"
#include "lbm_runtime.hpp"

namespace lbmx {

#define LBM_STACK_FN(LT)                                                         \
  {(const void *)&stack_kernel<CodecF32, LT>, (const void *)&stack_kernel<CodecF16, LT>,  \
   (const void *)&stack_kernel<CodecBF16, LT>, (const void *)&stack_kernel<CodecF16SR, LT>}
#define LBM_STACK(K)                                                             \
  {64, STACK_ROWS, 1, 1, 4, 0, K, (int)sizeof(StackRows) + MARCH_TABLE * 16,     \
   LBM_STACK_FN(true), LBM_STACK_FN(false), STACK_ROWS - 2 * (K - 1)}

const TileShape kStack[4] = {LBM_STACK(4), LBM_STACK(5), LBM_STACK(6), LBM_STACK(8)};

}  // namespace lbmx
