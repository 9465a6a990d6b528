// The hop kernels in FP16 storage.
#include "hop_kernels.h"

namespace dp {

hipError_t launch_hop_f16(const HopArgs& a, hipStream_t st, int* nparts) {
  return a.dag ? launch_epi<F16, true>(a, st, nparts) : launch_epi<F16, false>(a, st, nparts);
}

}  // namespace dp
