// Dispatch of the hop kernels (hop_kernels.h) by storage precision.
#include <algorithm>

#include "dp_common.h"

namespace dp {

hipError_t launch_hop_f64(const HopArgs& a, hipStream_t st, int* nparts);
hipError_t launch_hop_f32(const HopArgs& a, hipStream_t st, int* nparts);
hipError_t launch_hop_f16(const HopArgs& a, hipStream_t st, int* nparts);

int reduction_blocks(const Geom& g) { return (g.Vh + kBlock - 1) / kBlock; }

int hop_parts(const Geom& g) { return g.T * ((g.Vsh + 63) / 64); }

int hop_blocks(const Geom& g) { return std::max(reduction_blocks(g), hop_parts(g)); }

hipError_t launch_hop(const HopArgs& a, hipStream_t st, int* nparts) {
  *nparts = 0;
  if (a.nslots <= 0 || a.g.Vh <= 0) return hipErrorInvalidValue;
  if (a.in.prec != a.out.prec || a.link_prec != a.in.prec) return hipErrorInvalidValue;
  switch (a.in.prec) {
    case F64: return launch_hop_f64(a, st, nparts);
    case F32: return launch_hop_f32(a, st, nparts);
    case F16: return launch_hop_f16(a, st, nparts);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace dp
