// bssn_batch_o4.hip -- order-4 instantiations of the batched stage kernels
// (many patches per launch).
#include "bssn_kernels.h"
#include "bssn_split.h"
#include "bssn_stage.h"

namespace bssn {

hipError_t launch_batch_o4(const BatchLaunch& B, const Gauge& G, int stage,
                           int precision, hipStream_t st) {
  return launch_batch_t<4>(B, G, stage, precision, st);
}

template <>
hipError_t launch_f64tiles<4>(const Patch& P, const Gauge& G, int stage,
                              const TileMap& M, int nwg, hipStream_t st,
                              double* kout) {
  return launch_f64tiles_t<4>(P, G, stage, M, nwg, st, kout);
}

}  // namespace bssn
