// The hop kernels in FP32 storage.
#include "hop_kernels.h"

namespace dp {

hipError_t launch_hop_f32(const HopArgs& a, hipStream_t st, int* nparts) {
  return a.dag ? launch_epi<F32, true>(a, st, nparts) : launch_epi<F32, false>(a, st, nparts);
}

}  // namespace dp
