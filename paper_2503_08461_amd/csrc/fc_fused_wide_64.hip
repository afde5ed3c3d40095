// Fused kernels for head size 64, wide workgroups (one per CU).
#include "fc_unit.h"

namespace fc {

hipError_t fused_wide_setup_64() { return wide_setup_d<64>(); }

hipError_t launch_fused_wide_64(const BatchParams& p, int query_tiles, size_t lds, hipStream_t s) {
  return launch_fused_d<64, true>(p, query_tiles, lds, s);
}

}  // namespace fc
