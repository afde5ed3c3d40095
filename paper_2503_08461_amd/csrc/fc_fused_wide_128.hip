// Fused kernels for head size 128, wide workgroups (one per CU).
#include "fc_unit.h"

namespace fc {

hipError_t fused_wide_setup_128() { return wide_setup_d<128>(); }

hipError_t launch_fused_wide_128(const BatchParams& p, int query_tiles, size_t lds, hipStream_t s) {
  return launch_fused_d<128, true>(p, query_tiles, lds, s);
}

}  // namespace fc
