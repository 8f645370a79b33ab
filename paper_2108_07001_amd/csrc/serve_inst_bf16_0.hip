// serve_inst_bf16_0.hip -- instances of the batched serving kernels
// (bfloat16 splits, D = 1..4); split across files so that hipcc runs in parallel.
#include "serve_kernels.h"

namespace air {
#define AIR_SERVE_INST(D)                                                                       \
  hipError_t launch_serve_bf16_d##D(const JobDesc* j, int n, int64_t items, int64_t units, bool half, int g, \
                                   hipStream_t s) {                                            \
    return launch_serve_td<D, true>(j, n, items, units, half, g, s);                                  \
  }
AIR_SERVE_INST(1)
AIR_SERVE_INST(2)
AIR_SERVE_INST(3)
AIR_SERVE_INST(4)
#undef AIR_SERVE_INST
}  // namespace air
