// The hop kernels in FP64 storage.
#include "hop_kernels.h"

namespace dp {

hipError_t launch_hop_f64(const HopArgs& a, hipStream_t st, int* nparts) {
  return a.dag ? launch_epi<F64, true>(a, st, nparts) : launch_epi<F64, false>(a, st, nparts);
}

}  // namespace dp
