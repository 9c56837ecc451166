// lbm_march.hip -- instances of the marching kernel.
#include "lbm_march.hpp"
#include "lbm_runtime.hpp"

namespace lbmx {

#define LBM_MARCH_FN(K, NW, W, CP, LT)                                           \
  {(const void *)&march_kernel<CodecF32, K, NW, W, CP, LT>,                      \
   (const void *)&march_kernel<CodecF16, K, NW, W, CP, LT>,                      \
   (const void *)&march_kernel<CodecBF16, K, NW, W, CP, LT>,                     \
   (const void *)&march_kernel<CodecF16SR, K, NW, W, CP, LT>}
#define LBM_MARCH(K, NW, W, CP)                                                  \
  {64, NW, 1, 1, W, CP, K, MARCH_TABLE * 16, LBM_MARCH_FN(K, NW, W, CP, true),   \
   LBM_MARCH_FN(K, NW, W, CP, false), 0}

const TileShape kMarch4 = LBM_MARCH(4, 4, 2, 0);
const TileShape kMarch5 = LBM_MARCH(5, 4, 2, 0);

bool big_table(const lbm_config *c) { return c->table_n > MARCH_TABLE; }

}  // namespace lbmx
