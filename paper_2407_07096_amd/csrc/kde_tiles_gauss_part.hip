// Exact kernel density tiles, epilogue mode kModeGaussPart (the Gaussian sums
// in launches with several workgroups per chunk).
#include "kde_tiles.h"

namespace stag {

stag_status launch_tiles_gauss_part(const Operands& xo, const Operands& qo, double* partial, const TileExtra& ex,
                               hipStream_t st) {
  return tiles::launch_tiles<tiles::kModeGaussPart>(xo, qo, partial, ex, st);
}

}  // namespace stag
