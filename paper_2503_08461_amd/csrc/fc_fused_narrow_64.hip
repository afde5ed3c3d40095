// Fused kernels for head size 64, workgroups of four wavefronts.
#include "fc_unit.h"

namespace fc {

hipError_t launch_fused_narrow_64(const BatchParams& p, int query_tiles, size_t lds, hipStream_t s) {
  return launch_fused_d<64, false>(p, query_tiles, lds, s);
}

}  // namespace fc
