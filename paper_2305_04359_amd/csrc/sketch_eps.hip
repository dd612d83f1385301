// The beam search on rows with sketches, variants with the (1 + eps) rule of Sec. 4.5 compiled in.
#include "ann_dispatch.hpp"
#include "search_kernel.hpp"

namespace annmi {

template <int KIND, int NCH, int SK>
static hipError_t launch_eps(const SearchArgs& a, const VecTable& T, hipStream_t s) {
  return launch_search_sketched<KIND, NCH, SK, true, false>(a, T, s);
}

hipError_t launch_search_sketch_eps(const DistCfg& cfg, const SearchArgs& a, const VecTable& T, hipStream_t s) {
  ANN_DISPATCH_SKETCH(launch_eps, a, T, s);
}

}  // namespace annmi
