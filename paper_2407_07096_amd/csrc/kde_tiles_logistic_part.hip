// Exact kernel density tiles, epilogue mode kModeLogisticPart (the logistic kernel
// in launches with several workgroups per chunk).
#include "kde_tiles.h"

namespace stag {

stag_status launch_tiles_logistic_part(const Operands& xo, const Operands& qo, double* partial, const TileExtra& ex,
                               hipStream_t st) {
  return tiles::launch_tiles<tiles::kModeLogisticPart>(xo, qo, partial, ex, st);
}

}  // namespace stag
